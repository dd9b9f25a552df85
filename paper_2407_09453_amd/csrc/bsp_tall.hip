// Three-row windows (3x3, 3x1, ...; stride 1, bf16) with work enough to keep every CU busy for
// many steps: persistent workgroups, fourteen output rows to a weight fragment.
//
// What bounds such a layer is the weights' way from L2: every tile of pixels reads every strip's
// fragments again, and a CU gets about 65 bytes per ns.  The row-band kernel multiplies a fragment
// with seven rows of sixteen columns; here a wave holds fourteen accumulators (fourteen rows of one
// lane tile, or seven rows of two), which halves that traffic, and a tile's opening and end are
// hidden: data-mover waves stage the next slab or the next tile's first slab while the compute
// waves multiply.
//
// Work split.  An item is a pixel tile (NI images x NB bands of BR output rows x TW columns) x SG
// strips; a workgroup walks items nslot apart (one workgroup per CU).  The units of the walk are an
// item's channel slabs, one after the other through all items: unit u lies in patch buffer u & 1.
// Eight compute waves = SG strips x PTW column groups x KS shares of the contraction; the last NM
// waves only move data (their requests leave no LDS read of theirs waiting).  A share of the contraction
// ends in LDS: each of the KS waves of a strip then owns every KS-th pair of rows, which also deals out
// the stores.
//
// Strips differ by a quarter in the steps that they have in one slab, so no barrier ends a slab: movers
// and compute waves count what has landed and what is done in LDS, and a wave goes on to the next unit as
// soon as that has landed, up to one unit ahead of the others.  Two waves share a SIMD: the strips are
// dealt out so that a heavy one (they are stored heaviest first) shares with a light one.
//
// A step's fragments are read R patch rows ahead of the matrix instructions that use them; the weights
// of the next step are asked for when a step begins, on through slabs and items.
// Measured (row-band kernel -> here, in a replayed graph): 3x3 28x28x512 batch 16 52 -> 40.5 us, 56x56x256
// 47 -> 42, 28x28x256->512 27 -> 24, 58x76x544->336 batch 3 71 -> 29.  Of 56x56x256's 42 us the products are 45.5
// thousand cycles of a SIMD, 24 us at the 1.87 GHz that the chip keeps under this load.  Without the reads and
// the weights' loads it is 39 us, so the rest is not those; what it is has not been timed.
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>

namespace {

struct TallArgs {
  const unsigned char* X;
  unsigned char* Y;
  const float* bias;
  const unsigned char* residual;
  const int32_t* rstrip;
  const int32_t* rslab;
  const unsigned char* rdesc;
  const unsigned char* rfrag;
  int32_t relu, nstrips, nslabs, sc;  // sc: 16-byte pieces of a pixel per slab
  int32_t B, L, J, I, O, M, N, ph, pw;
  int32_t TW, NB, NI, PR, PCp;        // patch rows per image, staged columns per row
  int32_t tiles_x, nrows, groups;     // staged rows (NI * PR), KiB requests per row
  int32_t lscp, swz_shift, swz_mask;  // log2 of the 16-byte slots of a staged pixel; slot = piece ^ ((column >> shift) & mask)
  int32_t SG, lsg, lptw, KS, NM, nsg;
  int32_t nitems, per_xcd, nslot;
  int32_t bufbytes, ncols, ybytes;
  int32_t bo4;                        // results leave as 8-byte pieces (4x16 blocks)
  int32_t count_off;                  // LDS offset of the counters
  int32_t alone;                      // every workgroup has one item: the sums of the shares may use both buffers
  FastDiv d_nsg, d_tpi, d_tx, d_pr, d_perimg, d_tw;
};

typedef const __attribute__((address_space(4))) int32_t* cptr_t;
typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

struct Pos {
  int img0, y0, x0, sg;
};

template <int BR>
__device__ __forceinline__ Pos tall_pos(const TallArgs& a, int item) {
  Pos t;
  const int tile = (int)fdiv((uint32_t)item, a.d_nsg);
  t.sg = item - tile * a.nsg;
  const int ig = (int)fdiv((uint32_t)tile, a.d_tpi), trem = tile - ig * (int)a.d_tpi.d;
  const int ty = (int)fdiv((uint32_t)trem, a.d_tx), tx = trem - ty * a.tiles_x;
  t.img0 = ig * a.NI;
  t.y0 = ty * a.NB * BR;
  t.x0 = tx * a.TW;
  return t;
}

// sixteen zero bytes: what is copied for staged pixels outside the image
__device__ __align__(16) const unsigned char tall_zero16[16] = {0};

// everything this wave has asked LDS for is there, then the workgroup's barrier (a fence would also
// wait for the weights in flight)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Counters in LDS: one lane of a wave adds one once the wave's own LDS accesses (movers: and copies) are
// over; a wave waits until a counter has reached what every other wave is bound to add.
__device__ __forceinline__ void count_up(int32_t* p) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wait_for(const int32_t* p, int n) {
  while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < n) __builtin_amdgcn_s_sleep(1);
  asm volatile("" ::: "memory");
}

template <int BR, int NT, bool CW4>
__global__ __launch_bounds__(768) void conv_tall(TallArgs a) {
  constexpr int H = 3, NF = BR + H - 1, SEQ = NT * NF;
  constexpr int R = NT == 1 ? NF / 2 : NF;  // fragments in registers
  constexpr int NP = NT * BR / 2;           // pairs of results of a lane
  static_assert(SEQ % R == 0 && (NT * BR) % 2 == 0, "");
  kernarg_touch<TallArgs>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ncomp = (int)(blockDim.x >> 6) - a.NM;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int first = xcd * a.per_xcd + slot, end = min((xcd + 1) * a.per_xcd, a.nitems);
  if (first >= end) return;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  const int rowbytes = a.PCp << (a.lscp + 4);
  // even and odd units landed x movers, done x compute waves.  (By parity: a mover is at most one unit ahead of
  // another, as a compute wave is; one count for all units could be reached with a unit that somebody still lacks)
  int32_t* count = (int32_t*)(lds + a.count_off);
  if (tid < 4) count[tid] = 0;
  lds_barrier();

  if (wave >= ncomp) {
    // ---- data movers: mover m takes every NM-th group of a row's columns, all rows of it
    const int m = wave - ncomp;
    const int lppi = 6 - a.lscp;
    const int sub_pix = lane >> a.lscp, sidx = lane & ((1 << a.lscp) - 1);
    int u = 0;
    for (int item = first; item < end; item += a.nslot) {
      const Pos t = tall_pos<BR>(a, item);
      constexpr uint32_t kPad = 0xFFFFFFFFu;
      uint32_t rowsrc = kPad;  // lane r: where staged row r starts in X
      if (lane < a.nrows) {
        const int img = (int)fdiv((uint32_t)lane, a.d_pr), pr = lane - img * a.PR;
        const int gi = t.img0 + img, gy = t.y0 - a.ph + pr;
        if (gi < a.B && (unsigned)gy < (unsigned)a.L) rowsrc = (uint32_t)((gi * a.L + gy) * a.J) * (uint32_t)a.I * 2u;
      }
      for (int sl = 0; sl < a.nslabs; ++sl, ++u) {
        const uint32_t buf = lds0 + (uint32_t)((u & 1) * a.bufbytes);
        wait_for(count + 2 + (u & 1), (u >> 1) * ncomp);  // unit u - 2 is done everywhere
        for (int gq = m; gq < a.groups; gq += a.NM) {
          const int pc = (gq << lppi) + sub_pix;
          const int piece = sidx ^ ((pc >> a.swz_shift) & a.swz_mask);
          const int gx = t.x0 - a.pw + pc, ch = (sl * a.sc + piece) * 8;
          const bool real = piece < a.sc && ch < a.I && (unsigned)gx < (unsigned)a.J;
          const unsigned char* base = real ? a.X + ((uint32_t)gx * (uint32_t)a.I + (uint32_t)ch) * 2u : tall_zero16;
          const uint32_t rmask = real ? ~0u : 0u;
          uint32_t dst = buf + ((uint32_t)(gq << lppi) << (a.lscp + 4));
          for (int r = 0; r < a.nrows; ++r, dst += rowbytes) {
            const uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)rowsrc, r);
            const unsigned char* p = src == kPad ? tall_zero16 : base + (src & rmask);
            __builtin_amdgcn_global_load_lds((gptr_t)p, (lptr_t)(uintptr_t)dst, 16, 0, 0);
          }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        count_up(count + (u & 1));
        if (sl == 0 && item != first && a.KS > 1) {  // the sums of the item before
          asm volatile("s_barrier" ::: "memory");
          asm volatile("s_barrier" ::: "memory");
        }
      }
    }
    if (a.KS > 1) {
      asm volatile("s_barrier" ::: "memory");
      asm volatile("s_barrier" ::: "memory");
    }
    return;
  }

  // ---- compute waves
  // (waves w and w + 4 share a SIMD)
  const int order = wave < 4 ? wave : 11 - wave;
  const int sl_local = order & (a.SG - 1), sub = order >> a.lsg;
  const int pt = sub & ((1 << a.lptw) - 1), ks = sub >> a.lptw, ksm = a.KS - 1;

  // this lane's columns of a tile: the staged pixel under the window's corner, where it lies
  int timg[NT], tband[NT], tx[NT];
  uint32_t pixrow[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = min((pt * NT + j) * 16 + c, a.ncols - 1);  // lanes past the tile repeat its last column (never stored)
    timg[j] = (int)fdiv((uint32_t)col, a.d_perimg);
    const int rem = col - timg[j] * (int)a.d_perimg.d;
    tband[j] = (int)fdiv((uint32_t)rem, a.d_tw);
    tx[j] = rem - tband[j] * a.TW;
    pixrow[j] = (uint32_t)((timg[j] * a.PR + tband[j] * BR) * rowbytes);
  }

  // strip groups take every nsg-th strip (they are stored heaviest first: the groups weigh the same)
  auto strip_of = [&](int item) { return item - (int)fdiv((uint32_t)item, a.d_nsg) * a.nsg + sl_local * a.nsg; };
  auto slab_table = [&](int strip) {
    const uint64_t v = (uint64_t)(uintptr_t)(a.rslab + (size_t)strip * (a.nslabs + 1));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (cptr_t)(uintptr_t)((uint64_t)lo | ((uint64_t)hi << 32));
  };

  // ---- the weights: a walk of their own over the steps of all items, one step ahead of the products
  u32x4_t w[H], wn[H];  // this step's fragments, the next one's
  int dn, dnn;          // descriptors of the next step and the one after it
  const uint32_t frag_lane = (uint32_t)lane * 16u, desc_lane = (uint32_t)g * 4u;
  int f_item = first - a.nslot, f_cs = 0, f_end = 0, f_step = a.KS;
  auto f_item_next = [&]() {  // the first step of the next item in which this wave has one; past the last: step 0 for ever, never used
    for (;;) {
      f_item += a.nslot;
      if (f_item >= end) {
        f_cs = f_step = 0;
        f_end = 1;
        return;
      }
      const int strip = strip_of(f_item);
      if (strip >= a.nstrips) continue;
      const cptr_t t = slab_table(strip);
      const int lo = t[0];
      f_end = t[a.nslabs];
      f_cs = lo + ((ks - lo) & ksm);
      if (f_cs < f_end) return;
    }
  };
  auto f_next = [&]() {
    const int cs = f_cs;
    f_cs += f_step;
    if (f_cs >= f_end) f_item_next();
    return cs;
  };
  auto get_desc = [&](int cs) { return *(const int*)(a.rdesc + ((uint32_t)cs * 16u + desc_lane)); };
  int w_cs;  // the step whose weights are asked for next
  auto get_weights = [&]() {
    const uint32_t off = (uint32_t)w_cs * (uint32_t)(H * 1024) + frag_lane;
#pragma unroll
    for (int dy = 0; dy < H; ++dy) wn[dy] = *(const u32x4_t*)(a.rfrag + off + dy * 1024);
  };
  f_item_next();
  const int cs0 = f_next();
  w_cs = cs0;
  dn = get_desc(cs0);
  get_weights();
  w_cs = f_next();
  dnn = get_desc(w_cs);

  f32x4_t acc[NT * BR];
  u32x4_t f[R];
  const unsigned char* buf = lds;

  // where the fragments of a step lie, patch row 0 (4-channel units: two pieces of 8 bytes)
  uint32_t ad0[NT], ad1[NT];
  auto addresses = [&](uint32_t desc) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (CW4) {
        const uint32_t u0 = desc & 0xFFu, u1 = (desc >> 16) & 0xFFu;
        const uint32_t c0 = (uint32_t)tx[j] + ((desc >> 8) & 0xFFu), c1 = (uint32_t)tx[j] + (desc >> 24);
        ad0[j] = pixrow[j] + (c0 << (a.lscp + 4)) + (((u0 >> 1) ^ ((c0 >> a.swz_shift) & (uint32_t)a.swz_mask)) << 4) + ((u0 & 1u) << 3);
        ad1[j] = pixrow[j] + (c1 << (a.lscp + 4)) + (((u1 >> 1) ^ ((c1 >> a.swz_shift) & (uint32_t)a.swz_mask)) << 4) + ((u1 & 1u) << 3);
      } else {
        const uint32_t c0 = (uint32_t)tx[j] + ((desc >> 8) & 0xFFu);
        ad0[j] = pixrow[j] + (c0 << (a.lscp + 4)) + (((desc & 0xFFu) ^ ((c0 >> a.swz_shift) & (uint32_t)a.swz_mask)) << 4);
        ad1[j] = 0;
      }
    }
  };
  uint32_t r0 = 0, r1 = 0;  // where the next fragment is read
  auto frag = [&]() {
    u32x4_t v;
    if (CW4) {
      const u32x2_t x = *(const u32x2_t*)(buf + r0), y = *(const u32x2_t*)(buf + r1);
      v = u32x4_t{x.x, x.y, y.x, y.y};
      r1 += (uint32_t)rowbytes;
    } else {
      v = *(const u32x4_t*)(buf + r0);
    }
    r0 += (uint32_t)rowbytes;
    return v;
  };
  // the first R fragments of the step whose addresses are in ad0, ad1
  auto preload = [&]() {
    r0 = ad0[0];
    r1 = ad1[0];
#pragma unroll
    for (int i = 0; i < R; ++i) f[i] = frag();
  };
  // One step.  Fragment i serves window rows dy = 0..2 of output rows i - dy; once it is used the
  // fragment R places on is asked for into its registers, from the next step past this one's end (read for
  // nothing, in bounds, where the next step lies in another unit).
  auto step = [&]() {
#pragma unroll
    for (int dy = 0; dy < H; ++dy) w[dy] = wn[dy];
    dn = dnn;
    get_weights();
    w_cs = f_next();
    dnn = get_desc(w_cs);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < SEQ; ++i) {
      const int j = i / NF, k = i % NF;
#pragma unroll
      for (int dy = 0; dy < H; ++dy) {
        const int r = k - dy;
        if (r < 0 || r >= BR) continue;
        acc[j * BR + r] = mfma_bf16_16x16x32(w[dy], f[i % R], acc[j * BR + r]);
      }
      const int q = i + R;
      if (NT == 2 && q == NF) {
        r0 = ad0[NT - 1];
        r1 = ad1[NT - 1];
      }
      if (q == SEQ) {
        addresses((uint32_t)dn);
        r0 = ad0[0];
        r1 = ad1[0];
      }
      f[i % R] = frag();
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // two lane rows hold the halves of an 8-channel block row: after the exchange an even lane row has all
  // eight channels of result x, an odd one those of result y
  auto paired = [&](const f32x4_t& x, const f32x4_t& y) {
    const auto s0 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x.x, x.y), pack_bf16x2(y.x, y.y), false, false);
    const auto s1 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x.z, x.w), pack_bf16x2(y.z, y.w), false, false);
    return u32x4_t{s0[0], s1[0], s0[1], s1[1]};
  };

  addresses((uint32_t)dn);
  const auto yres = __builtin_amdgcn_make_buffer_rsrc(a.Y, 0, a.ybytes, 0x00020000);
  // this lane's four output channels of an item (-1: none) and their biases
  auto channels = [&](int item) {
    const int strip = strip_of(item);
    return strip < a.nstrips ? a.rstrip[strip * 4 + g] : -1;
  };
  auto biases = [&](int ch) {
    f32x4_t b = {0.f, 0.f, 0.f, 0.f};
    if (a.bias) {
      const float* p = a.bias + max(ch, 0);
      b = f32x4_t{p[0], p[1], p[2], p[3]};
    }
    return b;
  };
  int chan = channels(first);
  f32x4_t bv = biases(chan);
  int u = 0;
  for (int item = first; item < end; item += a.nslot) {
    const Pos t = tall_pos<BR>(a, item);
    const int strip = t.sg + sl_local * a.nsg;
    const bool active = strip < a.nstrips;
    const cptr_t st = slab_table(active ? strip : 0);
    int lo = st[0];
    const bool more = item + a.nslot < end;
    int cnext = -1;  // the next item's channels
#pragma unroll
    for (int r = 0; r < NT * BR; ++r) acc[r] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int sl = 0; sl < a.nslabs; ++sl, ++u) {
      wait_for(count + (u & 1), ((u >> 1) + 1) * a.NM);  // unit u has landed
      // the wave that is behind goes first (left to itself the older wave of a SIMD runs ahead to the next
      // unit's buffer and waits there; the last unit is then the others' alone)
      switch (u & 3) {
        case 0: __builtin_amdgcn_s_setprio(3); break;
        case 1: __builtin_amdgcn_s_setprio(2); break;
        case 2: __builtin_amdgcn_s_setprio(1); break;
        default: __builtin_amdgcn_s_setprio(0);
      }
      if (more && sl + 1 == a.nslabs) cnext = channels(item + a.nslot);
      buf = lds + (u & 1) * a.bufbytes;
      const int hi = active ? st[sl + 1] : lo;
      int cs = lo + ((ks - lo) & ksm);
      if (cs < hi) {
        preload();
        for (; cs < hi; cs += a.KS) step();
      }
      lo = hi;
      if (a.KS == 1 || sl + 1 < a.nslabs) count_up(count + 2 + (u & 1));
    }

    // ---- results.  Pair q of a lane: results ia, ib; with a split contraction the pairs are dealt out
    // over the strip's KS waves, who get the others' shares through LDS
    if (a.KS > 1) {
      unsigned char* red = a.alone ? lds : lds + ((u - 1) & 1) * a.bufbytes;
      const int nw = a.SG << a.lptw, me = pt * a.SG + sl_local;
      lds_barrier();  // the patch is not read any more
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int ia = NT == 1 ? 2 * q : q, ib = NT == 1 ? 2 * q + 1 : BR + q, owner = q & ksm;
        if (owner == ks) continue;
        f32x4_t* dst = (f32x4_t*)(red + ((q * ksm + (ks < owner ? ks : ks - 1)) * nw + me) * 2048) + lane;
        dst[0] = acc[ia];
        dst[64] = acc[ib];
      }
      lds_barrier();
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int ia = NT == 1 ? 2 * q : q, ib = NT == 1 ? 2 * q + 1 : BR + q;
        if ((q & ksm) != ks) continue;
        for (int k = 0; k < ksm; ++k) {
          const f32x4_t* src = (const f32x4_t*)(red + ((q * ksm + k) * nw + me) * 2048) + lane;
          acc[ia] += src[0];
          acc[ib] += src[64];
        }
      }
      count_up(count + 2 + ((u - 1) & 1));
    }
    // the next item's biases: asked for ahead of this one's stores
    f32x4_t bnext = {0.f, 0.f, 0.f, 0.f};
    if (more) bnext = biases(cnext);
    int cb[NT], rows[NT];  // first output pixel of this lane's columns, rows that exist
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int gi = t.img0 + timg[j], gy = t.y0 + tband[j] * BR, gx = t.x0 + tx[j];
      const bool exists = (pt * NT + j) * 16 + c < a.ncols && gi < a.B && gx < a.N;
      cb[j] = (gi * a.M + gy) * a.N + gx;
      rows[j] = exists ? a.M - gy : 0;
    }
    if (!a.bo4) {
      const int ch8 = __builtin_amdgcn_ds_bpermute(((lane & 32) + c) << 2, chan);  // the even lane row's channel
      const int odd = g & 1;
      uint32_t off[NP];
      bool ok[NP];
      u32x4_t res[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int j = NT == 1 ? 0 : odd, r = NT == 1 ? 2 * q + odd : q;
        const int base = NT == 1 ? cb[0] : (j ? cb[NT - 1] : cb[0]), lim = NT == 1 ? rows[0] : (j ? rows[NT - 1] : rows[0]);
        ok[q] = (q & ksm) == ks && r < lim && ch8 >= 0;
        off[q] = ((uint32_t)(base + r * a.N) * (uint32_t)a.O + (uint32_t)ch8) * 2u;
        res[q] = u32x4_t{0, 0, 0, 0};
        if (a.residual && ok[q]) res[q] = *(const u32x4_t*)(a.residual + off[q]);
      }
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int ia = NT == 1 ? 2 * q : q, ib = NT == 1 ? 2 * q + 1 : BR + q;
        u32x4_t v = paired(acc[ia] + bv, acc[ib] + bv);
        if (a.residual || a.relu) {
          const u32x2_t l2 = post_bf16x4_reg(u32x2_t{v.x, v.y}, u32x2_t{res[q].x, res[q].y}, a.residual != nullptr, a.relu);
          const u32x2_t h2 = post_bf16x4_reg(u32x2_t{v.z, v.w}, u32x2_t{res[q].z, res[q].w}, a.residual != nullptr, a.relu);
          v = u32x4_t{l2.x, l2.y, h2.x, h2.y};
        }
        // (out of the buffer's range: not stored.  A branch would make the next step wait for the stores)
        __builtin_amdgcn_raw_buffer_store_b128(v, yres, ok[q] ? off[q] : 0xFFFFFFF0u, 0, 0);
      }
    } else {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        if ((q & ksm) != ks) continue;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int i = NT == 1 ? 2 * q + e : e * BR + q, j = i / BR, r = i % BR;
          if (r >= rows[j] || chan < 0) continue;
          const f32x4_t v = acc[i] + bv;
          u32x2_t o = {pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
          const uint32_t off = ((uint32_t)(cb[j] + r * a.N) * (uint32_t)a.O + (uint32_t)chan) * 2u;
          if (a.residual || a.relu) o = post_bf16x4(o, a.residual ? (const uint16_t*)(a.residual + off) : nullptr, 4, true, a.relu);
          *(u32x2_t*)(a.Y + off) = o;
        }
      }
    }
    chan = cnext;
    bv = bnext;
  }
}

constexpr int kLdsLimit = 160 * 1024;

int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, v = 0;
    cus = hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0 ? v : 256;
  }
  return cus;
}

inline int ceil_log2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Choice {
  int BR, NT, TW, NB, NI, SG, PTW, KS;
  double cost;
};

struct Geometry {
  int PR, PCp, lscp, tiles_x, tiles_y, nsg, nslot, alone;
  int64_t ntiles, nitems, per_xcd, bufbytes, ldsb;
};

bool tall_geometry(const ConvParams& p, const int32_t* rs, int cus, const Choice& c, Geometry* g) {
  const int slab = rs[BSP_ROWS_SLAB_W], nslabs = rs[BSP_ROWS_NSLABS_W], nstrips = rs[BSP_ROWS_NSTRIPS_W];
  if (c.NI * c.NB * c.TW > c.PTW * c.NT * 16 || c.SG * c.PTW * c.KS > 8) return false;
  g->PR = c.NB * c.BR + p.H - 1;
  if (c.NI * g->PR > 64) return false;  // the movers keep one staged row per lane
  g->lscp = std::max(2, ceil_log2((slab + 7) / 8));
  const int ppr = 64 >> g->lscp;  // pixels per request
  g->PCp = (int)cdiv(c.TW - 1 + p.K, ppr) * ppr;
  g->bufbytes = ((int64_t)c.NI * g->PR * g->PCp) << (g->lscp + 4);
  g->tiles_x = (int)cdiv(p.N, c.TW);
  g->tiles_y = (int)cdiv(cdiv(p.M, c.BR), c.NB);
  g->ntiles = cdiv(p.B, c.NI) * g->tiles_y * g->tiles_x;
  g->nsg = (int)cdiv(nstrips, c.SG);
  g->nitems = g->ntiles * g->nsg;
  g->per_xcd = cdiv(g->nitems, 8);
  g->nslot = (int)std::min<int64_t>(g->per_xcd, std::max(1, cus / 8));
  g->alone = g->per_xcd <= g->nslot;
  const bool two = !g->alone || nslabs > 1;
  const int64_t red = c.KS > 1 ? (int64_t)(c.NT * c.BR / 2) * (c.KS - 1) * c.SG * c.PTW * 2048 : 0;
  if (!g->alone && red > g->bufbytes) return false;
  g->ldsb = std::max((two ? 2 : 1) * g->bufbytes, red) + 16;
  return g->ldsb <= kLdsLimit;
}

// The tile: rounds of (slabs x the slower of the products and the copies of a slab, and the end of an item), in
// ns, plus the opening.  A SIMD has two compute waves; a request costs a mover about 25 ns and a CU gets
// 65 bytes per ns from L2.
bool tall_choose(const ConvParams& p, const int32_t* rs, int cus, Choice* best) {
  const int nstrips = rs[BSP_ROWS_NSTRIPS_W], nslabs = rs[BSP_ROWS_NSLABS_W];
  const double steps = (double)rs[BSP_ROWS_NCS_W] / nstrips / nslabs;  // of a strip in a slab
  best->cost = 1e300;
  for (int BR : {14, 7}) {
    const int NT = 14 / BR;
    for (int SG : {8, 4, 2, 1})
      for (int KS : {1, 2, 4}) {
        const int PTW = 8 / SG / KS, slots = PTW * NT * 16;
        if (PTW < 1 || (SG > 1 && SG / 2 >= nstrips)) continue;
        const int bands = (int)cdiv(p.M, BR);
        for (int mode = 0; mode < 3; ++mode) {
          Choice c{BR, NT, p.N, 1, 1, SG, PTW, KS, 0.0};
          if (mode == 0) {  // whole rows, as many bands as fit
            if (p.N > slots) continue;
            c.NB = std::min(slots / p.N, bands);
          } else if (mode == 1) {  // several images
            if (p.N * bands > slots) continue;
            c.NB = bands;
            c.NI = std::min(slots / (p.N * bands), p.B);
            if (c.NI < 2) continue;
          } else {  // part of a row
            if (p.N <= slots) continue;
            c.TW = (int)cdiv(p.N, cdiv(p.N, slots));
          }
          Geometry g;
          if (!tall_geometry(p, rs, cus, c, &g)) continue;
          const double products = std::ceil(steps / KS) * (p.H * 14) * 10.8 * 2 + 300.0;
          const double copies = std::max(g.bufbytes / 1024.0 / 4 * 25.0, g.bufbytes / 45.0) + 800.0;
          const double end = 900.0 + (KS > 1 ? 900.0 : 0.0);
          const double rounds = (double)cdiv(g.per_xcd, g.nslot);
          c.cost = 3500.0 + copies + rounds * (nslabs * std::max(products, copies) + end);
          if (c.cost < best->cost) *best = c;
        }
      }
  }
  return best->cost < 1e299;
}

template <int BR, int NT, bool CW4>
int launch_inst(const TallArgs& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_tall<BR, NT, CW4>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_tall<BR, NT, CW4>), grid, dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

}  // namespace

int bsp_launch_tall(const ConvParams& p, const void* plan_host, BspRival rival, hipStream_t st) {
  if (!plan_host) return BSP_ERR_UNSUPPORTED;
  const int32_t* hdr = (const int32_t*)plan_host;
  if (hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION || hdr[BSP_PLAN_O_W] != p.O ||
      hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H || hdr[BSP_PLAN_K_W] != p.K || hdr[BSP_PLAN_DTYPE_W] != BSP_BF16 ||
      hdr[BSP_PLAN_OFF_ROWS_W] == 0)
    return BSP_ERR_UNSUPPORTED;
  const int32_t* rs = hdr + hdr[BSP_PLAN_OFF_ROWS_W];
  if (p.H != 3 || p.sh != 1 || p.sw != 1 || rs[BSP_ROWS_NCS_W] == 0) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.B * p.L * p.J * p.I * 2 >= (1ll << 31) || (int64_t)p.P * p.O * 2 >= (1ll << 31)) return BSP_ERR_UNSUPPORTED;
  const int64_t mr = (int64_t)((p.P + 15) / 16) * rs[BSP_ROWS_NCS_W] * p.H;
#ifndef BSP_ROWS_TUNE
  // (no search where no cost would decide)
  if (!bsp_tall_beats(rival, mr, p.I, p.O, 0.0, 1.0)) return BSP_ERR_UNSUPPORTED;
#endif
  const int cus = device_cus();
  Choice ch;
  {
    // the search and the line are pure functions of these: remember the answers
    static std::mutex mu;
    static std::map<std::array<int32_t, 12>, Choice> memo;
    const std::array<int32_t, 12> key = {p.B, p.M, p.N, p.I, p.O, p.K, p.ph * 65536 + p.pw, rs[BSP_ROWS_NCS_W], rs[BSP_ROWS_NSTRIPS_W],
                                         rs[BSP_ROWS_CW_W], (int32_t)rival, cus};
    std::unique_lock<std::mutex> lock(mu);
    const auto it = memo.find(key);
    if (it != memo.end()) {
      ch = it->second;
    } else {
      lock.unlock();
      if (!tall_choose(p, rs, cus, &ch) || !bsp_tall_beats(rival, mr, p.I, p.O, ch.cost, rival == BSP_RIVAL_ROWS ? bsp_rows_cost(p, rs) : 0.0))
        ch.BR = 0;
      lock.lock();
      if (memo.size() > 4096) memo.clear();
      memo.emplace(key, ch);
    }
  }
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (const char* e = std::getenv("BSP_TALL")) {
    if (!std::atoi(e)) return BSP_ERR_UNSUPPORTED;
    if (!tall_choose(p, rs, cus, &ch)) return BSP_ERR_UNSUPPORTED;
  }
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "tall: M=%d N=%d B=%d I=%d O=%d | BR=%d NT=%d TW=%d NB=%d NI=%d SG=%d PTW=%d KS=%d cost=%.0f\n", p.M, p.N, p.B, p.I, p.O,
            ch.BR, ch.NT, ch.TW, ch.NB, ch.NI, ch.SG, ch.PTW, ch.KS, ch.cost);
#endif
  if (ch.BR == 0) return BSP_ERR_UNSUPPORTED;
  const int NM = 4;
  Geometry geo;
  if (!tall_geometry(p, rs, cus, ch, &geo)) return BSP_ERR_UNSUPPORTED;
  const int32_t* sec = p.plan + hdr[BSP_PLAN_OFF_ROWS_W];
  TallArgs a{};
  a.X = (const unsigned char*)p.X;
  a.Y = (unsigned char*)p.Y;
  a.bias = p.bias;
  a.residual = (const unsigned char*)p.residual;
  a.relu = p.relu;
  a.rstrip = sec + rs[BSP_ROWS_OFF_STRIP_W];
  a.rslab = sec + rs[BSP_ROWS_OFF_SLAB_W];
  a.rdesc = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_DESC_W]);
  a.rfrag = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_FRAG_W]);
  a.nstrips = rs[BSP_ROWS_NSTRIPS_W];
  a.nslabs = rs[BSP_ROWS_NSLABS_W];
  a.sc = rs[BSP_ROWS_SLAB_W] / 8;
  a.B = p.B;
  a.L = p.L;
  a.J = p.J;
  a.I = p.I;
  a.O = p.O;
  a.M = p.M;
  a.N = p.N;
  a.ph = p.ph;
  a.pw = p.pw;
  a.TW = ch.TW;
  a.NB = ch.NB;
  a.NI = ch.NI;
  a.PR = geo.PR;
  a.PCp = geo.PCp;
  a.tiles_x = geo.tiles_x;
  a.nrows = ch.NI * geo.PR;
  a.groups = geo.PCp >> (6 - geo.lscp);
  a.lscp = geo.lscp;
  const int bits = std::min(geo.lscp, 4);  // sixteen consecutive columns, sixteen bank groups
  a.swz_shift = 4 - bits;
  a.swz_mask = (1 << bits) - 1;
  a.SG = ch.SG;
  a.lsg = ceil_log2(ch.SG);
  a.lptw = ceil_log2(ch.PTW);
  a.KS = ch.KS;
  a.NM = NM;
  a.nsg = geo.nsg;
  a.nitems = (int32_t)geo.nitems;
  a.per_xcd = (int32_t)geo.per_xcd;
  a.nslot = geo.nslot;
  a.bufbytes = (int32_t)geo.bufbytes;
  a.ncols = ch.NI * ch.NB * ch.TW;
  a.ybytes = p.P * p.O * 2;
  a.bo4 = hdr[BSP_PLAN_BO_W] == 4;
  a.count_off = (int32_t)geo.ldsb - 16;
  a.alone = geo.alone;
  // multiply-high divisions are exact while dividend * divisor < 2^32
  if (geo.nitems >= (1ll << 24) || (geo.nitems + 8) * std::max<int64_t>(geo.nsg, (int64_t)geo.tiles_x * geo.tiles_y) >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  a.d_nsg = make_fastdiv((uint32_t)geo.nsg);
  a.d_tpi = make_fastdiv((uint32_t)(geo.tiles_x * geo.tiles_y));
  a.d_tx = make_fastdiv((uint32_t)geo.tiles_x);
  a.d_pr = make_fastdiv((uint32_t)geo.PR);
  a.d_perimg = make_fastdiv((uint32_t)(ch.NB * ch.TW));
  a.d_tw = make_fastdiv((uint32_t)ch.TW);
  const int threads = 64 * (ch.SG * ch.PTW * ch.KS + NM);
  const dim3 grid((unsigned)(geo.nslot * 8));
  const size_t ldsb = (size_t)geo.ldsb;
  if (rs[BSP_ROWS_CW_W] == 4)
    return ch.BR == 14 ? launch_inst<14, 1, true>(a, grid, threads, ldsb, st) : launch_inst<7, 2, true>(a, grid, threads, ldsb, st);
  return ch.BR == 14 ? launch_inst<14, 1, false>(a, grid, threads, ldsb, st) : launch_inst<7, 2, false>(a, grid, threads, ldsb, st);
}
