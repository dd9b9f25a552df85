// Block-sparse x block-sparse product C = (Gamma A)(Omega B)^t, 8x8 blocks (paper Section
// III-A).  A block product is done only where both operands keep the block column.
//
// A workgroup owns a 128 x 128 tile of C: sixteen block rows of A against sixteen of B.  It
// walks the block columns in segments of 16 to 64 (as many sixteens as fit the payload area
// of LDS) and, per segment, copies the kept blocks of its 32 block rows from their compressed
// block rows into LDS (each row's blocks of the segment are one contiguous run, found through
// the per-sixteen row pointers seg_ptr) and scatters a one-byte position table per row from
// col_idx.  A wave owns one pair of A block rows and meets every pair of B block rows in
// turn (a 16 x 16 MFMA tile each).  For such a tile the columns worth multiplying are those
// kept by one of the two A rows and by one of the two B rows: the two rows' column sets are
// united, the two sides intersected (the merge of the sorted index lists of Section III-A,
// done on 64-bit column sets), and the surviving columns are compacted so that every MFMA
// 16x16x32 takes four of them; columns kept on one side only are never multiplied.
#include "bsp_device.h"
#include "bsp_launch.h"
#include "bsp_spgemm_pick.h"
#include <algorithm>
#ifdef BSP_ROWS_TUNE
#include <cstdlib>
#endif

namespace {

constexpr int kRows = 16;     // block rows of each operand per workgroup
constexpr int kSub = 16;      // block columns per seg_ptr entry
constexpr int kMaxSub = 4;    // a segment is one to four of those
constexpr int kCap = 592;     // blocks the payload area holds (>= 2 * kRows * kSub); slot kCap stays zero
constexpr int kTabOff = (kCap + 1) * 128;           // position tables, two sets of [32 rows][64 columns] bytes
constexpr int kTabBytes = 2 * kRows * 64;
constexpr int kLdsBytes = kTabOff + 2 * kTabBytes;
static_assert(kCap >= 2 * kRows * kSub, "one sixteen of columns must always fit");
static_assert(2 * kLdsBytes <= 160 * 1024, "two workgroups share a CU");

struct SpParams {
  const int32_t* sa;   // seg_ptr of A: [ra][nsub + 1]
  const int32_t* sb;
  const int32_t* ca;   // col_idx
  const int32_t* cb;
  const unsigned char* pa;  // [nnzb][8][8] bf16
  const unsigned char* pb;
  float* C;            // [ra*8][rb*8]
  int32_t ra, rb, nsub;
  int32_t nnzb_a, nnzb_b;   // both positive
  int32_t tiles_i, tiles_j;  // workgroup tiles along A's and B's block rows
  int32_t sbj, nsb;          // 8 x 8 groups of tiles: along j, in all
#ifdef BSP_ROWS_TUNE
  long long* trace;
#endif
};

#ifdef BSP_ROWS_TUNE
#define SP_CLOCK() wall_clock64()
#define SP_ADD(k, t0)                          \
  do {                                         \
    const long long t1_ = wall_clock64();      \
    tacc[k] += t1_ - (t0);                     \
    (t0) = t1_;                                \
  } while (0)
#else
#define SP_CLOCK() 0ll
#define SP_ADD(k, t0)
#endif

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// What a wave keeps of the next segment between asking for its row pointers and using them.
struct SegRows {
  int first, d[kMaxSub];
};
// A segment as every wave sees it: lane r < 32 holds row r's first block, slot in LDS and number
// of blocks; ks (the same in all lanes) is the segment's width in sixteens.
struct SegPlan {
  int first, off, cnt, ks;
};

// C = 0: an operand without a kept block.
__global__ __launch_bounds__(256) void spgemm_zero(float* C, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) C[i] = 0.f;
}

template <int U>
__global__ __launch_bounds__(512) void spgemm_nt_bf16(SpParams q) {
  kernarg_touch<SpParams>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, jn = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroups go to different XCDs; each XCD takes whole 8 x 8 groups of tiles so
  // that the operand rows its workgroups share stay in its L2
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int grp = (slot >> 6) * 8 + xcd, within = slot & 63;
  if (grp >= q.nsb) return;
  const int gi = grp / q.sbj, gj = grp - gi * q.sbj;
  const int ti = gi * 8 + (within >> 3), tj = gj * 8 + (within & 7);
  if (ti >= q.tiles_i || tj >= q.tiles_j) return;
#ifdef BSP_ROWS_TUNE
  long long tacc[6] = {0, 0, 0, 0, 0, 0};
  const long long tentry = wall_clock64();
#endif
  long long tm = SP_CLOCK();

  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  const int half = jn >> 3, lr = jn & 7;  // which row of the pair, which row of the block
  constexpr uint32_t kZero = (uint32_t)kCap;           // the slot that holds zeros
  constexpr uint32_t kZZ = kZero | (kZero << 16);

  f32x4_t acc[8];
#pragma unroll
  for (int jp = 0; jp < 8; ++jp) acc[jp] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Every wave plans the segments for itself (the same few loads and shuffles in each, no
  // table in LDS and no barrier for it): lane r < 32 stands for row r of the 32 (A's sixteen,
  // then B's).
  const int mrow = lane & 31;
  const bool m_isA = mrow < kRows;
  const int m_row = m_isA ? ti * kRows + mrow : tj * kRows + mrow - kRows;
  const bool m_ok = lane < 32 && m_row < (m_isA ? q.ra : q.rb);
  const int32_t* m_sp = (m_isA ? q.sa : q.sb) + (int64_t)(m_ok ? m_row : 0) * (q.nsub + 1);
  auto seg_load = [&](int x, SegRows& sr) {
    sr.first = 0;
#pragma unroll
    for (int k = 0; k < kMaxSub; ++k) sr.d[k] = 0;
    if (m_ok && x < q.nsub) {
      const int kmax = min(kMaxSub, q.nsub - x);
      sr.first = m_sp[x];
#pragma unroll
      for (int k = 0; k < kMaxSub; ++k)
        if (k < kmax) sr.d[k] = m_sp[x + k + 1];
    }
  };
  // how many sixteens fit (the same answer in every wave), where each row's blocks start and go
  auto seg_plan = [&](int x, const SegRows& sr, SegPlan& pl) {
    const int kmax = min(kMaxSub, q.nsub - x);
    int ks = 1, cnt = m_ok ? sr.d[0] - sr.first : 0;
#pragma unroll
    for (int k = 1; k < kMaxSub; ++k) {
      const int dk = (m_ok && k < kmax) ? sr.d[k] - sr.first : 0;
      int t = dk;
#pragma unroll
      for (int m = 1; m < 32; m <<= 1) t += __shfl_xor(t, m);
      t = __builtin_amdgcn_readfirstlane(t);  // lanes 0-31 hold the total of the 32 rows
      if (k < kmax && t <= kCap) {            // totals grow with k: the last k that fits wins
        ks = k + 1;
        cnt = dk;
      }
    }
    int incl = cnt;
#pragma unroll
    for (int m = 1; m < 32; m <<= 1) {
      const int v = __shfl_up(incl, m);
      if (lane >= m) incl += v;
    }
    pl.first = sr.first;
    pl.off = incl - cnt;
    pl.cnt = cnt;
    pl.ks = ks;
  };
  // wave w brings rows 4w .. 4w + 3 (waves 0-3: A's, waves 4-7: B's); the columns of their
  // blocks, asked for one segment ahead
  const int32_t* my_col = wave < 4 ? q.ca : q.cb;
  const unsigned char* my_pay = wave < 4 ? q.pa : q.pb;
  // (every lane loads, the lanes past the row's blocks an entry they do not use: a load under a
  // condition would be waited for on the spot)
  const int my_last = (wave < 4 ? q.nnzb_a : q.nnzb_b) - 1;
  auto col_load = [&](const SegPlan& pl, int (&col)[4]) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int first = __builtin_amdgcn_readlane(pl.first, wave * 4 + rr);
      col[rr] = my_col[min(first + lane, my_last)];
    }
  };

  // ---- before the first segment: its plan and columns, an empty table, the zero block
  if (tid < 8) ((u32x4_t*)lds)[kCap * 8 + tid] = u32x4_t{0u, 0u, 0u, 0u};
  ((uint32_t*)(lds + kTabOff))[tid] = 0xFFFFFFFFu;  // 512 threads x 4 bytes: no block anywhere
  SegRows sr;
  SegPlan pl, pn;
  int col[4], coln[4];
  seg_load(0, sr);
  seg_plan(0, sr, pl);
  pn = pl;
  col_load(pl, col);
  __syncthreads();
  SP_ADD(0, tm);

  int buf = 0;
  for (int x = 0; x < q.nsub; buf ^= 1) {
    uint8_t* tab = lds + kTabOff + buf * kTabBytes;
    const int xn = x + __builtin_amdgcn_readfirstlane(pl.ks);

    // ---- copies: the position tables first (their columns came long ago), then the blocks
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int r = wave * 4 + rr;
      const int n = __builtin_amdgcn_readlane(pl.cnt, r);
      if (lane < n) tab[r * 64 + ((col[rr] - x * kSub) & 63)] = (uint8_t)lane;
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int r = wave * 4 + rr;
      const int first = __builtin_amdgcn_readlane(pl.first, r), off = __builtin_amdgcn_readlane(pl.off, r);
      const int n = __builtin_amdgcn_readlane(pl.cnt, r);
      const unsigned char* pay = my_pay + (int64_t)first * 128;
      const int pieces = n * 8;  // 16 bytes each
      for (int it = 0; it < pieces; it += 64) {
        if (it + lane < pieces)
          __builtin_amdgcn_global_load_lds((gptr_t)(pay + (it + lane) * 16),
                                           (lptr_t)(uintptr_t)(lds0 + (uint32_t)(off * 8 + it) * 16u), 16, 0, 0);
      }
    }
    // the next segment: its row pointers asked for now, its table emptied
    seg_load(xn, sr);
    ((uint32_t*)(lds + kTabOff + (buf ^ 1) * kTabBytes))[tid] = 0xFFFFFFFFu;
    SP_ADD(1, tm);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    SP_ADD(2, tm);
    seg_plan(xn, sr, pn);  // past the last segment: rows without blocks, loads of entries nobody uses
    col_load(pn, coln);

    // ---- products: this wave's pair of A rows against the eight pairs of B rows
    {
      const int ra0 = 2 * wave;
      const uint32_t a0 = tab[ra0 * 64 + lane], a1 = tab[(ra0 + 1) * 64 + lane];  // this lane's column
      const uint32_t oa0 = (uint32_t)__builtin_amdgcn_readlane(pl.off, ra0);
      const uint32_t oa1 = (uint32_t)__builtin_amdgcn_readlane(pl.off, ra0 + 1);
      const unsigned long long ma = __ballot(a0 != 255u) | __ballot(a1 != 255u);
      const uint32_t mineA = (a0 == 255u ? kZero : oa0 + a0) | ((a1 == 255u ? kZero : oa1 + a1) << 16);
      const int sh = half * 16;
      const uint32_t rowb = (uint32_t)lr * 16u;
      // per pair of B rows: the columns both sides keep, compacted: lane n gets the slots of the
      // n-th such column, the lanes past their number get the zero block
      int pA[8], pB[8], cnt[8];
#pragma unroll
      for (int jp = 0; jp < 8; ++jp) {
        const int rb0 = kRows + 2 * jp;
        const uint32_t b0 = tab[rb0 * 64 + lane], b1 = tab[(rb0 + 1) * 64 + lane];
        const uint32_t ob0 = (uint32_t)__builtin_amdgcn_readlane(pl.off, rb0);
        const uint32_t ob1 = (uint32_t)__builtin_amdgcn_readlane(pl.off, rb0 + 1);
        const unsigned long long m = ma & (__ballot(b0 != 255u) | __ballot(b1 != 255u));
        cnt[jp] = __popcll(m);
        const uint32_t mineB = (b0 == 255u ? kZero : ob0 + b0) | ((b1 == 255u ? kZero : ob1 + b1) << 16);
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        const bool isset = (m >> lane) & 1ull;
        const int dest = (isset ? rank : cnt[jp] + lane - rank) << 2;
        pA[jp] = __builtin_amdgcn_ds_permute(dest, (int)(isset ? mineA : kZZ));
        pB[jp] = __builtin_amdgcn_ds_permute(dest, (int)(isset ? mineB : kZZ));
      }
#pragma unroll
      for (int jp = 0; jp < 8; ++jp) {
        for (int s0 = 0; s0 < cnt[jp]; s0 += 4 * U) {
          uint32_t va[U], vb[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int n = (s0 + 4 * u + g) & 63;
            va[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(n << 2, pA[jp]);
            vb[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(n << 2, pB[jp]);
          }
          u32x4_t a[U], b[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (u > 0 && s0 + 4 * u >= cnt[jp]) continue;
            a[u] = *(const u32x4_t*)(lds + (((va[u] >> sh) & 0xFFFFu) * 128u + rowb));
            b[u] = *(const u32x4_t*)(lds + (((vb[u] >> sh) & 0xFFFFu) * 128u + rowb));
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u == 0 || s0 + 4 * u < cnt[jp]) acc[jp] = mfma_bf16_16x16x32(a[u], b[u], acc[jp]);
        }
      }
    }
    SP_ADD(3, tm);
    __syncthreads();  // every wave is done with the tables and the blocks
    SP_ADD(4, tm);
    x = xn;
    pl = pn;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) col[rr] = coln[rr];
  }

  // lane holds C[128 ti + 16 wave + 4 g + r][128 tj + 16 jp + jn], r = 0..3
  const int ncol = q.rb * 8;
#pragma unroll
  for (int jp = 0; jp < 8; ++jp) {
    const int col = 128 * tj + 16 * jp + jn;
    if (col >= ncol) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 128 * ti + 16 * wave + 4 * g + r;
      if (row < q.ra * 8) q.C[(int64_t)row * ncol + col] = acc[jp][r];
    }
  }
#ifdef BSP_ROWS_TUNE
  if (q.trace && lane == 0) {
    __builtin_amdgcn_s_waitcnt(0);
    SP_ADD(5, tm);
    long long* t = q.trace + ((size_t)blockIdx.x * 8 + wave) * 8;
    t[0] = tentry;
    for (int k = 0; k < 6; ++k) t[1 + k] = tacc[k];
    t[7] = tm;
  }
#endif
}

// ---------------------------------------------------------------------------------------------
// The same product as a tiled dense one, absent blocks staged as zeros.  A 16 x 16 tile of the
// kernel above can skip a column only if both rows of a side drop it, (1 - d)^2 of them, and its
// operands serve no other tile, so LDS gives it a quarter of the matrix rate; here a fragment
// serves a whole wave tile.  4096^3, half of the blocks kept on both sides: 344 -> 112 us (1.2 PFLOP/s
// of multiply-adds issued), all kept 533 -> 128, a quarter 159 -> 113, a tenth 98 / 111 (the kernel
// above stays); 1024^3 52 -> 9.9, 512^3 19.9 -> 7.0.
//
// A workgroup owns GM x GN wave tiles of 16 MI x 16 NI elements and walks the block columns eight
// at a time.  MV waves only move data: lane group l / 8 of a request brings the eight 16-byte rows
// of one block, from its place in the compressed row or from a line of zeros, so a request fills
// 1 KiB of LDS: the blocks of eight block rows in one block column.  They run NBUF - 1 steps ahead.
// Blocks lie column by column in LDS ([column][row]), which puts the two blocks that sixteen lanes
// read side by side.  Which blocks a row keeps in a step, and where they start, is a word per (step,
// row) of a table that all waves build first from seg_ptr and col_idx.
//
// What bounds it: the requests' issue, nine instructions each (128 x 128 tiles with two, four and
// eight movers at 2048^3: 43, 32, 25 us), then LDS: operands read and staged take 2048 clocks of a
// 256 x 256 tile's step, its products as many.  Reading half a step ahead of the products changed
// nothing.
//
// Zero times infinity: a product of an absent block with an infinity or NaN is no part of the
// result.  It leaves a non-finite sum, so a 16 x 16 tile with one is computed once more from
// the columns that both of its sides keep (redo_tile), the kernel above's rule, and what was
// not finite is replaced.
__device__ const u32x4_t g_zeros[1] = {};

struct DnParams {
  const int32_t* sa;
  const int32_t* sb;
  const int32_t* ca;
  const int32_t* cb;
  const unsigned char* pa;
  const unsigned char* pb;
  float* C;
  int32_t ra, rb, nsub, nsteps;   // nsteps: eights of block columns
  int32_t nnzb_a, nnzb_b;         // both positive
  int32_t tiles_i, tiles_j, per_xcd, total;
  int32_t band;                   // tile rows that consecutive workgroups share operand columns over
};

// One 16 x 16 tile once more (block rows la, la + 1 of the workgroup's A against lb, lb + 1 of its B, from
// the step table in LDS) from the columns that one of the two rows of each side keeps.  Four steps of
// loads are out at a time; bound by their latency.  4096^3, half kept, with one NaN in A 187 us, with all
// of A infinite 726, where finite operands take 124 (one column at a time from col_idx: 1248 and 8517).
template <int R>
__device__ __forceinline__ f32x4_t redo_tile(const DnParams& q, const uint32_t* tab, int la, int lb, const unsigned char* pa,
                                             const unsigned char* pb, int lane) {
  constexpr int U = 4;
  const int jn = lane & 15, g = lane >> 4, h = jn >> 3;
  pa += (jn & 7) * 16;
  pb += (jn & 7) * 16;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < q.nsteps; s0 += U) {
    u32x4_t a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t* t = tab + min(s0 + u, q.nsteps - 1) * R;
      const uint32_t a0 = t[la], a1 = t[la + 1], b0 = t[lb], b1 = t[lb + 1];
      const uint32_t both = s0 + u < q.nsteps ? (a0 | a1) & (b0 | b1) & 0xFFu : 0u, wa = h ? a1 : a0, wb = h ? b1 : b0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t c = 4u * k + g, before = (1u << c) - 1u, on = both >> c & 1u;
        a[u][k] = b[u][k] = u32x4_t{0u, 0u, 0u, 0u};
        if (on & wa >> c) a[u][k] = *(const u32x4_t*)(pa + (int64_t)((wa >> 8) + __popc(wa & before)) * 128);
        if (on & wb >> c) b[u][k] = *(const u32x4_t*)(pb + (int64_t)((wb >> 8) + __popc(wb & before)) * 128);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) acc = mfma_bf16_16x16x32(b[u][k], a[u][k], acc);
  }
  return acc;
}

template <int MI, int NI, int GM, int GN, int MV, int NBUF>
__global__ __launch_bounds__((GM * GN + MV) * 64) void spgemm_dense_bf16(DnParams q) {
  kernarg_touch<DnParams>();
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int RA = GM * MI * 2, RB = GN * NI * 2, R = RA + RB;  // block rows
  constexpr int NC = GM * GN, kBuf = R * 1024;                    // compute waves; bytes of a step
  // a mover brings GPM groups of eight rows, eight columns of them or a share of the eight
  constexpr int CS = MV > R / 8 ? MV / (R / 8) : 1, NCOL = 8 / CS, GPM = R / 8 * CS / MV;
  static_assert(GPM * MV == R / 8 * CS && NCOL * CS == 8 && (RA / 8) % GPM == 0, "movers share the rows evenly");
  constexpr int kAhead = (NBUF - 2) * GPM * NCOL;                   // requests that may be in flight while a step is used
  static_assert(kAhead <= 63, "vmcnt counts to 63");
  uint32_t* tab = (uint32_t*)(lds + NBUF * kBuf);                 // [step][R]: kept columns, first block << 8
  const int tid = threadIdx.x, lane = tid & 63, jn = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // an XCD takes a run of tiles: bands of `band` tile rows, column by column, whose operands its L2 keeps
  const int qi = (int)(blockIdx.x & 7u) * q.per_xcd + (int)(blockIdx.x >> 3);
  if (qi >= q.total) return;
  const int bt = q.band * q.tiles_j, b0 = qi / bt, rem = qi - b0 * bt;
  const int bh = min(q.band, q.tiles_i - b0 * q.band);
  const int ti = b0 * q.band + rem % bh, tj = rem / bh;

  // seg_ptr row of the tile's block row r (A's, then B's); past the matrix, the last row's, and ok = false
  auto seg_row = [&](int r, bool* ok) {
    const bool isA = r < RA;
    const int row = isA ? ti * RA + r : tj * RB + r - RA, rows = isA ? q.ra : q.rb;
    *ok = row < rows;
    return (isA ? q.sa : q.sb) + (int64_t)min(row, rows - 1) * (q.nsub + 1);
  };

  // ---- the table: sixteen lanes per (row, sixteen columns), four of those in flight per lane
  constexpr int kPer = 4 * (NC + MV);  // entries per round of the workgroup
  for (int e0 = tid >> 4; e0 < R * q.nsub; e0 += 4 * kPer) {
    int first[4], n[4], rel[4], c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = min(e0 + u * kPer, R * q.nsub - 1), r = e % R, x = e / R;
      bool ok;
      const int32_t* sp = seg_row(r, &ok);
      first[u] = sp[x];
      n[u] = sp[x + 1];
      rel[u] = sp[0];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = min(e0 + u * kPer, R * q.nsub - 1), r = e % R;
      // (every lane loads, those past the row's blocks an entry they do not use)
      c[u] = (r < RA ? q.ca : q.cb)[min(first[u] + jn, (r < RA ? q.nnzb_a : q.nnzb_b) - 1)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * kPer, r = e % R, x = e / R;
      bool ok;
      seg_row(r, &ok);
      uint32_t m = ok && jn < n[u] - first[u] ? 1u << ((c[u] - x * kSub) & 15) : 0u;
#pragma unroll
      for (int s = 1; s < 16; s <<= 1) m |= __shfl_xor(m, s);
      if (jn < 2 && e < R * q.nsub && 2 * x + jn < q.nsteps)
        tab[(2 * x + jn) * R + r] = (uint32_t)(first[u] - rel[u] + (jn ? __popc(m & 0xFFu) : 0)) << 8 | ((m >> (8 * jn)) & 0xFFu);
    }
  }
  __syncthreads();

  if (wave >= NC) {
    // =================================================================== data movers
    const int grp0 = (wave - NC) / CS * GPM, c0 = (wave - NC) % CS * NCOL;
    const bool isA = grp0 * 8 < RA;  // (all of a mover's groups are one operand's)
    const unsigned char* src[GPM];
    uint32_t tb[GPM];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
#pragma unroll
    for (int k = 0; k < GPM; ++k) {
      const int r = (grp0 + k) * 8 + (lane >> 3);
      bool ok;
      src[k] = (isA ? q.pa : q.pb) + (int64_t)seg_row(r, &ok)[0] * 128 + (lane & 7) * 16;
      tb[k] = lds0 + (uint32_t)(NBUF * kBuf + r * 4);
    }
    const unsigned char* zero = (const unsigned char*)g_zeros;
    auto issue = [&](int s, int buf) {
#pragma unroll
      for (int k = 0; k < GPM; ++k) {
        // (read and waited for in one: the compiler would wait for the requests in flight as well)
        uint32_t w;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(w) : "v"(tb[k] + (uint32_t)(s * R * 4)) : "memory");
        if (CS > 1) w += (uint32_t)__popc(w & ((1u << c0) - 1u)) << 8;
        const unsigned char* p = src[k] + (w >> 8) * 128u;
        const uint32_t dst = lds0 + (uint32_t)(buf * kBuf + (isA ? (grp0 + k) * 1024 : RA * 1024 + ((grp0 + k) * 8 - RA) * 128));
#pragma unroll
        for (int c = 0; c < NCOL; ++c) {
          const bool kept = (w >> (c0 + c)) & 1u;
          __builtin_amdgcn_global_load_lds((gptr_t)(kept ? p : zero),
                                           (lptr_t)(uintptr_t)(dst + (uint32_t)((c0 + c) * (isA ? RA : RB) * 128)), 16, 0, 0);
          p += kept ? 128 : 0;
        }
      }
    };
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s)
      if (s < q.nsteps) issue(s, s);
    int buf = NBUF - 1;
    if (NBUF - 2 < q.nsteps)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kAhead) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile(".p2align 6");  // (the loop's instructions start on a line: 2 % of 256 x 256 x 32768)
    for (int s = 0; s < q.nsteps; ++s) {
      __builtin_amdgcn_s_barrier();  // step s is there; everyone is done with step s - 1
      if (s + NBUF - 1 < q.nsteps) {
        issue(s + NBUF - 1, buf);
        buf = buf + 1 == NBUF ? 0 : buf + 1;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kAhead) : "memory");  // step s + 1 has landed
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
    }
    return;
  }

  // ===================================================================== compute waves
  const int wm = wave / GN, wn = wave - wm * GN;
  f32x4_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const unsigned char* la = lds + ((g * RA + wm * MI * 2 + (jn >> 3)) * 128 + (jn & 7) * 16);
  const unsigned char* lb = lds + (RA * 1024 + (g * RB + wn * NI * 2 + (jn >> 3)) * 128 + (jn & 7) * 16);
  int off = 0;
  for (int s = 0; s < q.nsteps; ++s) {
    __builtin_amdgcn_s_barrier();  // step s has landed
    asm volatile("" ::: "memory");
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      u32x4_t a[MI], b[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = *(const u32x4_t*)(la + off + kk * 4 * RA * 128 + i * 256);
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = *(const u32x4_t*)(lb + off + kk * 4 * RB * 128 + j * 256);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mfma_bf16_16x16x32(b[j], a[i], acc[i][j]);
    }
    off = off + kBuf == NBUF * kBuf ? 0 : off + kBuf;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (no read of the step may still be out at the next barrier)
  }

  // ---- results: the lane has C[row jn][columns 4 g .. 4 g + 3] of each 16 x 16 tile
  const int64_t ncol = (int64_t)q.rb * 8;
  auto put = [&](int r0, int c0, f32x4_t v) {
    if (r0 + (jn >> 3) < q.ra && c0 + (g >> 1) < q.rb)
      __builtin_memcpy(q.C + (int64_t)(r0 * 8 + jn) * ncol + c0 * 8 + 4 * g, &v, 16);
  };
  const int ar0 = ti * RA + wm * MI * 2, bc0 = tj * RB + wn * NI * 2;  // the wave's first block rows
  uint32_t redo = 0, bad[4] = {0, 0, 0, 0};  // tiles with a sum that is not finite; the lane's own of these
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const f32x4_t v = acc[i][j];
      put(ar0 + 2 * i, bc0 + 2 * j, v);
      // (the difference is not zero for an infinity or NaN)
      if (__ballot((v.x - v.x) + (v.y - v.y) + (v.z - v.z) + (v.w - v.w) != 0.f)) {
        redo |= 1u << (i * NI + j);
#pragma unroll
        for (int r = 0; r < 4; ++r) bad[r] |= v[r] - v[r] == 0.f ? 0u : 1u << (i * NI + j);
      }
    }
  for (; redo; redo &= redo - 1) {
    const int t = __ffs((int)redo) - 1, i = t / NI, j = t % NI;
    const int r0 = ar0 + 2 * i, c0 = bc0 + 2 * j, h = jn >> 3;
    // the lane's block rows; their first blocks (past the matrix: no blocks, any place)
    const unsigned char* pa = q.pa + (int64_t)q.sa[(int64_t)min(r0 + h, q.ra - 1) * (q.nsub + 1)] * 128;
    const unsigned char* pb = q.pb + (int64_t)q.sb[(int64_t)min(c0 + h, q.rb - 1) * (q.nsub + 1)] * 128;
    const f32x4_t v = redo_tile<R>(q, tab, wm * MI * 2 + 2 * i, RA + wn * NI * 2 + 2 * j, pa, pb, lane);
    if (r0 + h < q.ra && c0 + (g >> 1) < q.rb) {
      float* at = q.C + (int64_t)(r0 * 8 + jn) * ncol + c0 * 8 + 4 * g;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (bad[r] >> t & 1u) at[r] = v[r];
    }
  }
}

constexpr int kU = 2;  // MFMA steps whose fragments are asked for together

template <int U>
int launch_u(const SpParams& q, unsigned grid, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)spgemm_nt_bf16<U>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) !=
        hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((spgemm_nt_bf16<U>), dim3(grid), dim3(512), kLdsBytes, st, q);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

template <int TILE, int MI, int NI, int GM, int GN, int MV>
int launch_dense(DnParams q, hipStream_t st) {
  constexpr int RA = GM * MI * 2, RB = GN * NI * 2, NBUF = kSpTile[TILE].nbuf;
  static_assert(RA == kSpTile[TILE].ra && RB == kSpTile[TILE].rb, "the instance is the tile that was chosen");
  const int64_t ldsb = sp_tile_lds(kSpTile[TILE], q.nsteps);
  if (ldsb > kSpLds) return BSP_ERR_UNSUPPORTED;
  q.tiles_i = (q.ra + RA - 1) / RA;
  q.tiles_j = (q.rb + RB - 1) / RB;
  const int64_t total = (int64_t)q.tiles_i * q.tiles_j;
  if (total > 1 << 28) return BSP_ERR_UNSUPPORTED;
  q.total = (int32_t)total;
  q.per_xcd = (q.total + 7) / 8;
  q.band = std::min(q.tiles_i, 8);
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)spgemm_dense_bf16<MI, NI, GM, GN, MV, NBUF>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSpLds) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((spgemm_dense_bf16<MI, NI, GM, GN, MV, NBUF>), dim3((unsigned)(q.per_xcd * 8)),
                     dim3((GM * GN + MV) * 64), (size_t)ldsb, st, q);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

}  // namespace

extern "C" int bsp_spgemm_nt(const bsp_bcsr* A, const bsp_bcsr* B, float* C, void* stream) {
  if (!A || !B || !C) return BSP_ERR_NULL;
  if (!A->seg_ptr || !B->seg_ptr || (A->nnzb > 0 && (!A->payload || !A->col_idx)) ||
      (B->nnzb > 0 && (!B->payload || !B->col_idx)))
    return BSP_ERR_NULL;
  if (A->rows <= 0 || B->rows <= 0 || A->cols <= 0 || A->cols != B->cols || A->nnzb < 0 || B->nnzb < 0)
    return BSP_ERR_SHAPE;
  if (A->k != 8 || B->k != 8) return BSP_ERR_UNSUPPORTED;
  if (A->dtype != BSP_BF16 || B->dtype != BSP_BF16) return BSP_ERR_DTYPE;
  if ((int64_t)A->rows * 8 * B->rows * 8 > 0x7FFFFFFFll * 4 || A->nnzb > 0x7FFFFFFFll || B->nnzb > 0x7FFFFFFFll)
    return BSP_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(A->payload) & 15u) || (reinterpret_cast<uintptr_t>(B->payload) & 15u) ||
      (reinterpret_cast<uintptr_t>(C) & 3u))
    return BSP_ERR_ALIGN;
  if (A->nnzb == 0 || B->nnzb == 0) {
    const int64_t n = (int64_t)A->rows * 8 * B->rows * 8;
    hipLaunchKernelGGL(spgemm_zero, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0,
                       (hipStream_t)stream, C, n);
    return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
  }
  SpParams q;
  q.nnzb_a = (int32_t)A->nnzb;
  q.nnzb_b = (int32_t)B->nnzb;
  q.sa = A->seg_ptr;
  q.sb = B->seg_ptr;
  q.ca = A->col_idx;
  q.cb = B->col_idx;
  q.pa = (const unsigned char*)A->payload;
  q.pb = (const unsigned char*)B->payload;
  q.C = C;
  q.ra = A->rows;
  q.rb = B->rows;
  q.nsub = (A->cols + kSub - 1) / kSub;
  q.tiles_i = (A->rows + kRows - 1) / kRows;
  q.tiles_j = (B->rows + kRows - 1) / kRows;
  q.sbj = (q.tiles_j + 7) / 8;
  const int64_t nsb = (int64_t)((q.tiles_i + 7) / 8) * q.sbj;
  if (nsb * 64 > 0x7FFFFFFF) return BSP_ERR_SHAPE;
  q.nsb = (int32_t)nsb;
  DnParams d{q.sa, q.sb, q.ca, q.cb, q.pa, q.pb, C, q.ra, q.rb, q.nsub, (A->cols + 7) / 8, q.nnzb_a, q.nnzb_b, 0, 0, 0, 0, 0};
  {
    hipStream_t st = (hipStream_t)stream;
    int rc = BSP_ERR_UNSUPPORTED;
    switch (sp_pick(d.ra, d.rb, d.nsteps, (double)A->nnzb / ((double)A->rows * A->cols), (double)B->nnzb / ((double)B->rows * B->cols))) {
      case SP_TILE_64: rc = launch_dense<SP_TILE_64, 2, 2, 2, 2, 4>(d, st); break;
      case SP_TILE_128: rc = launch_dense<SP_TILE_128, 2, 4, 4, 2, 8>(d, st); break;
      case SP_TILE_128W: rc = launch_dense<SP_TILE_128W, 4, 4, 2, 4, 6>(d, st); break;
      case SP_TILE_256: rc = launch_dense<SP_TILE_256, 8, 4, 2, 4, 4>(d, st); break;
    }
    if (rc != BSP_ERR_UNSUPPORTED) return rc;
  }
#ifdef BSP_ROWS_TUNE
  q.trace = nullptr;
  if (const char* e = std::getenv("BSP_PW_TRACE_PTR")) q.trace = (long long*)std::strtoull(e, nullptr, 16);
#endif
  const unsigned grid = (unsigned)(((nsb + 7) / 8) * 8 * 64);
#ifdef BSP_ROWS_TUNE
  if (const char* e = std::getenv("BSP_SP_U")) {
    const int u = std::atoi(e);
    if (u == 2) return launch_u<2>(q, grid, (hipStream_t)stream);
    if (u == 3) return launch_u<3>(q, grid, (hipStream_t)stream);
    if (u == 6) return launch_u<6>(q, grid, (hipStream_t)stream);
  }
#endif
  return launch_u<kU>(q, grid, (hipStream_t)stream);
}
