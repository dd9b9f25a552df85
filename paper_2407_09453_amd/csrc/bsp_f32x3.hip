// Single-precision layers in whole chunks of eight input channels on the bf16 matrix cores: every value is
// the sum of three bf16 parts (8 + 8 + 8 bits, exact: see kScale), and of the nine products of
// two values' parts the six largest are summed in fp32, the leading one by itself.  (Splitting a number into
// pieces whose products are exact is Dekker's, Numer. Math. 18, 1971.)  What is left out is below 2^-24 of
// a product, as much as one rounding; a sum of n terms is rounded n / 32 times per part instead of n times, so
// sums of two terms and more lie nearer to 64 bits than those of fp32 multiply-adds (2-norm of the error of 1x1
// sums of 1, 2, 8 and 64 terms, multiply-adds / here: 2.54e-8 / 2.61e-8, 3.10e-8 / 2.62e-8, 5.37e-8 / 2.89e-8, 1.44e-7 /
// 4.87e-8).  A sum of one term is the nearest float with a multiply-add and was not in 4 % of cases here; layers
// whose strips have at most kShort steps, those that scale or permute channels among them, sum eight of the
// nine: 2.54e-8, not the nearest in 0.2 %, by 0.506 of a last place at the most.  (Everywhere those two would cost
// 3x3 56x56x64 batch 32 37 -> 42 us.)
//
// Why: the fp32 matrix instructions reach 117 to 150 TFLOP/s, six bf16 ones per product 380, and a strip of
// sixteen rows gives back at most two thirds of that (the union of its block rows' columns).  Bound by
// LDS and the matrix cores alike: a step (four (chunk, tap) pairs) reads 3 KB of activations for six
// instructions of 16 cycles.  The weights' parts lie in the plan in operand order; activations are split
// once, where they are staged.  Measured (conv_f32 -> here, in a replayed graph): 3x3 56x56x64 batch 32 52 -> 35 us, of
// which the products are 15 by LDS or by the matrix cores; 28x28x128 batch 8 21.9 -> 12.0, 1x1 28x28x128->512 batch 8
// 15.2 -> 11.3; relative error of the first against 64 bits 3.1e-7 -> 1.0e-7.
//
// What three parts cannot hold takes another way: a lane tile that ends in an infinity or NaN (a value or sum past
// 2^111, an infinity times a zero that fills up a block row) is summed again in fp32, block row by block row,
// straight from memory (exact_tile); layers with weights that are not finite, below 2^-100 or from 2^127
// upwards stay with conv_f32.
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

struct X3Args {
  const float* X;
  float* Y;
  const float* bias;
  const float* residual;
  const int32_t* slab_ptr;
  const unsigned char* xdesc;
  const unsigned char* wfrag;      // DIRECT: where the weights lie in the payload
  int32_t relu;
  int32_t L, J, I, O, H, K, M, N;
  int32_t sh, sw, ph, pw, gsh, gsw, lsh, lsw;  // input pixels per staged pixel, staged pixels per output pixel
  int32_t CW, nchunk, tpc;         // output columns per chunk of columns, such chunks per row, tiles per chunk
  int32_t TPW, pitch, ppp;         // staged pixels per row, bytes per staged pixel, chunks staged of each
  int32_t nslabs, spst, nstages, slab_chunks;  // the plan's slabs, how many are staged at a time, chunks of one
  int32_t nstrips, NS, PG, ks, lpg, lks, nset; // strips per workgroup, pixel groups, waves that share a strip's steps; log2
  int32_t total, per_xcd;
  int32_t opitch, stream;
  int32_t lbo;
  const int32_t* plan;
  const float* payload;
  FastDiv d_nset, d_tpc, d_nchunk, d_cw, d_tpw, d_ppp, d_opp;
};

// Activations are multiplied by this where they are staged, and the sums divided by it: the smallest floats'
// last bits then lie at 2^-133, where bf16's end, so that no value below 2^111 loses any, and a product of 2^-126 keeps
// its last 39.  (Without it each tile that staged a value below 2^-100 was summed twice, the second time straight from
// memory: 3x3 56x56x64 batch 32 with one such value 213 us, with one in a hundred 656, now 37 as without any.)
constexpr float kScale = 65536.f;

// eight floats -> three times eight bf16
struct Parts {
  u32x4_t p[3];
};
__device__ __forceinline__ Parts split8(const f32x4_t lo, const f32x4_t hi) {
  Parts s;
  float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
      if (q < 2) {  // (exact: a part agrees with its value in the leading eight bits)
        v[2 * i] -= __uint_as_float(w[i] << 16);
        v[2 * i + 1] -= __uint_as_float(w[i] & 0xFFFF0000u);
      }
    }
    s.p[q] = u32x4_t{w[0], w[1], w[2], w[3]};
  }
  return s;
}

// The sums of one 16 x 16 tile (a strip, and one output pixel per lane column, whose window starts at
// iy0, ix0) in fp32 from kept blocks alone: every block row by itself, with zeros for the channels that it drops,
// where a value is an infinity or NaN, all of them in one where none is (a dropped channel then meets a zero weight).
// Straight from memory; four (chunk, tap) pairs to an instruction and twice those in flight, bound by two loads after
// each other: with one NaN 3x3 56x56x64 batch 32 takes 46 us (121 with one pair in flight), 28x28x128 batch 8 37 (113),
// 14x14x256 batch 2 with 16x4 blocks 59 (187).
__device__ __forceinline__ f32x4_t exact_tile(const X3Args& a, const float* xim, int strip, int iy0, int ix0, int lane) {
  constexpr int U = 2;
  const int g = lane >> 4, jn = lane & 15, HK = a.H * a.K;
  const PlanView pv = plan_view(a.plan);
  const int c0 = pv.strip_ptr[strip], npairs = (pv.strip_ptr[strip + 1] - c0) * HK;
  const int bi = 64 >> a.lbo, mine = jn >> a.lbo, at0 = (jn & ((1 << a.lbo) - 1)) * HK;
  const int nrows = BSP_STRIP >> a.lbo;  // block rows of a strip
  f32x4_t all = {0.f, 0.f, 0.f, 0.f}, acc[BSP_MAXSUB] = {};
#pragma unroll 1
  for (int q = 0; q < npairs; q += 4 * U) {
    int xc[U], at[U];
    i32x4_t src[U];
    bool in[U];
    const float* px[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int pair = min(q + 4 * u + g, npairs - 1), chunk = pair / HK, tap = pair - chunk * HK, th = tap / a.K;
      const int iy = iy0 + th, ix = ix0 + tap - th * a.K;
      xc[u] = pv.chunk_xc[c0 + chunk];
      src[u] = *(const i32x4_t*)(pv.chunk_src + (c0 + chunk) * BSP_MAXSUB);
      if (q + 4 * u + g >= npairs) src[u] = i32x4_t{-1, -1, -1, -1};  // (past the end: no weights, so no product)
      in[u] = src[u].x >= 0 || src[u].y >= 0 || src[u].z >= 0 || src[u].w >= 0;
      in[u] = in[u] && (unsigned)iy < (unsigned)a.L && (unsigned)ix < (unsigned)a.J;
      px[u] = xim + (int64_t)(iy * a.J + ix) * a.I;
      at[u] = (at0 + tap) * bi;
    }
    f32x4_t w[U][2], x[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // four channels at a time; 4-wide blocks: each from its own
        const int s = bi == 4 ? (h == 0 ? src[u].x : src[u].y) : mine == 0 ? src[u].x : mine == 1 ? src[u].y : mine == 2 ? src[u].z : src[u].w;
        w[u][h] = x[u][h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (s >= 0) w[u][h] = *(const f32x4_t*)(a.payload + (int64_t)s + at[u] + (bi == 4 ? 0 : 4 * h));
        if (in[u]) x[u][h] = *(const f32x4_t*)(px[u] + xc[u] * 8 + 4 * h);
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      bool odd = false;
#pragma unroll
      for (int i = 0; i < 8; ++i) odd |= (__float_as_uint(x[u][i >> 2][i & 3]) & 0x7F800000u) == 0x7F800000u;
      if (__ballot(odd) == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) all = mfma_f32_16x16x4(w[u][i >> 2][i & 3], x[u][i >> 2][i & 3], all);
      } else {
#pragma unroll
        for (int s = 0; s < BSP_MAXSUB; ++s) {
          if (s >= nrows) break;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bool kept = (bi == 4 && i >= 4 ? src[u].y : src[u][s]) >= 0;
            acc[s] = mfma_f32_16x16x4(w[u][i >> 2][i & 3], kept ? x[u][i >> 2][i & 3] : 0.f, acc[s]);
          }
        }
      }
    }
  }
  const int row = 4 * g >> a.lbo;  // the lane's four channels lie in one block row
  return all + (row == 0 ? acc[0] : row == 1 ? acc[1] : row == 2 ? acc[2] : acc[3]);
}

// One (tile of PT * 16 * PG output pixels) x (NS strips) per workgroup, as in conv_any: consecutive pixels of a
// chunk of image columns, the input patch staged with its halo, as many slabs at a time as LDS takes.  A staged
// pixel holds per chunk its three parts side by side, in an odd number of 16-byte pieces (no bank
// conflicts within a patch row).  Wave = (strip, pixel group, share of the strip's steps).  SHORT: eight products.
// DIRECT: the plan holds the weights' places in the payload and they are split here, step by step.
template <int PT, bool SHORT, bool DIRECT>
__global__ __launch_bounds__(512, 4) void conv_f32x3(X3Args a) {
  kernarg_touch<X3Args>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, jn = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthreads = (int)blockDim.x;
  // workgroups of one tile (other strips) are neighbours on one XCD: its L2 has the patch
  const uint32_t q = (blockIdx.x & 7u) * (uint32_t)a.per_xcd + (blockIdx.x >> 3);
  if (q >= (uint32_t)a.total) return;
  const uint32_t tile = fdiv(q, a.d_nset);
  const int set = (int)(q - tile * (uint32_t)a.nset);
  const uint32_t ic = fdiv(tile, a.d_tpc);
  const int px = PT * 16 * a.PG;
  const int p0 = (int)(tile - ic * (uint32_t)a.tpc) * px;
  const int img = (int)fdiv(ic, a.d_nchunk);
  const int col0 = (int)(ic - (uint32_t)img * (uint32_t)a.nchunk) * a.CW;
  const int m0 = (int)fdiv((uint32_t)p0, a.d_cw);
  const int plast = min(p0 + px, a.M * a.CW) - 1;
  const int rows = ((int)fdiv((uint32_t)plast, a.d_cw) - m0) * a.lsh + a.H;  // staged rows

  const int k = wave & (a.ks - 1), sp = wave >> a.lks, pg = sp & (a.PG - 1), si = sp >> a.lpg;
  const int strip = set * a.NS + si;
  const bool active = si < a.NS && strip < a.nstrips;
  // the strip's step ranges, one slab boundary per lane
  const int tab = a.slab_ptr[(active ? strip : 0) * (a.nslabs + 1) + min(lane, a.nslabs)];

  int base[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int p = min(p0 + (pg * PT + t) * 16 + jn, plast);
    const int y = (int)fdiv((uint32_t)p, a.d_cw), x = p - y * a.CW;
    base[t] = ((y - m0) * a.lsh * a.TPW + x * a.lsw) * a.pitch;
  }
  f32x4_t hi[PT], lo[PT];  // the leading products' sums, the others'
#pragma unroll
  for (int t = 0; t < PT; ++t) hi[t] = lo[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int iy0 = m0 * a.sh - a.ph, ix0 = col0 * a.sw - a.pw;
  const int pieces = rows * a.TPW * a.ppp;
  const float* xim = a.X + (int64_t)img * a.L * a.J * a.I;
  const uint32_t wrow = (uint32_t)(jn & ((1 << a.lbo) - 1)) * (256u >> a.lbo);  // bytes of a block's rows before this lane's
  const int rowpitch = a.TPW * a.pitch;

  for (int stg = 0; stg < a.nstages; ++stg) {
    const int sl0 = stg * a.spst, sl1 = min(sl0 + a.spst, a.nslabs);
    const int slo = __builtin_amdgcn_readlane(tab, sl0), shi = __builtin_amdgcn_readlane(tab, sl1);
    const int n = active && shi - slo > k ? (shi - slo - k + a.ks - 1) >> a.lks : 0;  // this wave's steps

    // ---- weights: one step ahead; descriptors: two
    u32x4_t w[3], wn[3];
    f32x4_t wl, wh;        // DIRECT: the next step's weights, and where they and those after them lie
    int lo0 = -1, hi0 = -1, lo1 = -1, hi1 = -1;
    int dn, an, dnn, ann;  // descriptor and place of the slab in a staged pixel, of the next step and the one after
    int fcs = slo + k, fsl = sl0, fadd = 0, fend = __builtin_amdgcn_readlane(tab, sl0 + 1), wcs = 0;
    auto ask_desc = [&]() {
      const int cs = min(fcs, shi - 1);  // (past the end: the last step again, never used)
      fcs += a.ks;
      while (cs >= fend) {
        fadd += a.slab_chunks * 48;
        ++fsl;
        fend = __builtin_amdgcn_readlane(tab, fsl + 1);
      }
      dnn = *(const int*)(a.xdesc + ((uint32_t)cs * 16u + (uint32_t)g * 4u));
      ann = fadd;
      wcs = cs;
      if constexpr (DIRECT) {
        const u32x2_t at = *(const u32x2_t*)(a.wfrag + ((uint32_t)cs * 128u + (uint32_t)(g * 4 + (jn >> a.lbo)) * 8u));
        lo1 = (int)at.x;
        hi1 = (int)at.y;
      }
    };
    auto ask_weights = [&]() {
      if constexpr (DIRECT) {
        lo0 = lo1;
        hi0 = hi1;
        wl = *(const f32x4_t*)((const unsigned char*)a.payload + ((uint32_t)max(lo0, 0) * 4u + wrow));
        wh = *(const f32x4_t*)((const unsigned char*)a.payload + ((uint32_t)max(hi0, 0) * 4u + wrow));
      } else {
        const unsigned char* p = a.wfrag + ((uint32_t)wcs * 3072u + (uint32_t)lane * 16u);
#pragma unroll
        for (int r = 0; r < 3; ++r) wn[r] = *(const u32x4_t*)(p + r * 1024);
      }
    };
    auto take_weights = [&]() {
      if constexpr (DIRECT) {
        const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
        const Parts s = split8(lo0 < 0 ? zero : wl, hi0 < 0 ? zero : wh);
#pragma unroll
        for (int r = 0; r < 3; ++r) w[r] = s.p[r];
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r) w[r] = wn[r];
      }
    };
    dn = dnn = an = ann = 0;
    if (n > 0) {  // their latency passes while the patch is staged
      ask_desc();
      ask_weights();
      dn = dnn;
      an = ann;
      ask_desc();
    }

    // ---- stage: a thread has two chunks of eight channels in flight (four: 30 registers more, a workgroup less
    // per CU, 1x1 28x28x128->512 batch 8 12.2 -> 15.3 us)
    const int c0 = sl0 * a.slab_chunks * 8;  // first channel that is staged
    if (stg > 0) __syncthreads();
    for (int f0 = tid; f0 < pieces; f0 += 2 * nthreads) {
      f32x4_t v[2][2];
      int dst[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int f = f0 + u * nthreads;
        const int pix = (int)fdiv((uint32_t)f, a.d_ppp), part = f - pix * a.ppp;
        const int r = (int)fdiv((uint32_t)pix, a.d_tpw), x = pix - r * a.TPW;
        const int iy = iy0 + r * a.gsh, ix = ix0 + x * a.gsw, ch = c0 + part * 8;
        dst[u] = f < pieces && ch < a.I ? pix * a.pitch + part * 48 : -1;
        v[u][0] = v[u][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (dst[u] >= 0 && (unsigned)iy < (unsigned)a.L && (unsigned)ix < (unsigned)a.J) {
          const f32x4_t* src = (const f32x4_t*)(xim + (uint32_t)(iy * a.J + ix) * (uint32_t)a.I + ch);
          v[u][0] = src[0];
          v[u][1] = src[1];
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (dst[u] < 0) continue;
        asm volatile("" : "+v"(v[u][0]), "+v"(v[u][1]));  // (scaled here: where they are loaded, each would be waited for by itself)
        const Parts s = split8(v[u][0] * kScale, v[u][1] * kScale);
#pragma unroll
        for (int r = 0; r < 3; ++r) *(u32x4_t*)(lds + dst[u] + r * 16) = s.p[r];
      }
    }
    __syncthreads();

    // ---- products, two lane tiles at a time: their fragments are read while the two before them are in the
    // matrix cores
    auto place = [&](int desc, int add) {
      asm volatile("" : "+v"(desc));  // decoded here, not where it is loaded: no early wait
      return ((uint32_t)desc & 0xFFFFu) * 48u + (uint32_t)add + (((uint32_t)desc >> 16) & 0xFFu) * (uint32_t)rowpitch +
             ((uint32_t)desc >> 24) * (uint32_t)a.pitch;
    };
    auto read = [&](uint32_t at, int t0, u32x4_t (&f)[2][3]) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 3; ++r) f[t][r] = *(const u32x4_t*)(lds + base[t0 + t] + at + r * 16);
    };
    auto mma = [&](int t0, const u32x4_t (&f)[2][3]) {
      constexpr int wi[8] = {0, 1, 2, 0, 1, 1, 2, 0}, xi[8] = {0, 2, 1, 2, 1, 0, 0, 1};
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        if (!SHORT && (m == 1 || m == 2)) continue;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f32x4_t& acc = m == 0 ? hi[t0 + t] : lo[t0 + t];
          acc = mfma_bf16_16x16x32(w[wi[m]], f[t][xi[m]], acc);
        }
      }
    };
    u32x4_t fa[2][3], fb[2][3];
    uint32_t at = 0;
    if (n > 0) {
      at = place(dn, an);
      read(at, 0, fa);
    }
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      take_weights();
      dn = dnn;
      an = ann;
      ask_weights();
      ask_desc();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PT == 4) {
        read(at, 2, fb);
        mma(0, fa);
        __builtin_amdgcn_sched_barrier(0);
        at = place(dn, an);
        read(at, 0, fa);
        mma(2, fb);
      } else {
        at = place(dn, an);
        read(at, 0, fb);
        mma(0, fa);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 3; ++r) fa[t][r] = fb[t][r];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  f32x4_t acc[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) acc[t] = hi[t] + lo[t];
  // ---- waves that share a strip: partial sums through LDS, the strip's matrix tiles dealt out to its waves
  if (a.ks > 1) {
    __syncthreads();
    f32x4_t* red = (f32x4_t*)lds;  // [wave][PT][64]
#pragma unroll
    for (int t = 0; t < PT; ++t) red[(wave * PT + t) * 64 + lane] = acc[t];
    __syncthreads();
    const f32x4_t* first = red + (wave - k) * (PT * 64) + lane;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      if ((t & (a.ks - 1)) != k) continue;
      f32x4_t v = first[t * 64];
      for (int s = 1; s < a.ks; ++s) v += first[(s * PT + t) * 64];
      acc[t] = v;
    }
  }
#pragma unroll
  for (int t = 0; t < PT; ++t) acc[t] *= 1.f / kScale;
  __syncthreads();  // everybody is done with the patch (the partial sums)

  // ---- results: bias, into an LDS image of the tile's output; then all waves copy that out, 16 contiguous
  // bytes per lane, with the residual and ReLU
  // (the lane anew: the rare path's pixels are those of `base`, and kept from there they were seven spilled
  // registers, whose 11 MB of scratch at 3x3 56x56x64 batch 32 were written by every launch and read by none)
  int el = lane;
  asm volatile("" : "+v"(el));
  const int eg = el >> 4, ejn = el & 15;
  const int opitch = a.opitch;
  if (active) {
    const int ch = strip * BSP_STRIP + 4 * eg;
    f32x4_t bv = {0.f, 0.f, 0.f, 0.f};
    if (a.bias) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (ch + r < a.O) bv[r] = a.bias[ch + r];
    }
    unsigned char* ot = lds + (pg * PT * 16 + ejn) * opitch + (si * BSP_STRIP + 4 * eg) * 4;
    uint32_t redo = 0;  // lane tiles with an infinity or NaN
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      if ((t & (a.ks - 1)) != k) continue;
      bool again = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) again |= (__float_as_uint(acc[t][r]) & 0x7F800000u) == 0x7F800000u;
      if (__ballot(again)) redo |= 1u << t;
      *(f32x4_t*)(ot + t * 16 * opitch) = acc[t] + bv;
    }
#pragma unroll 1
    for (; redo; redo &= redo - 1) {
      const int t = __builtin_ctz(redo), p = min(p0 + (pg * PT + t) * 16 + ejn, plast);
      const int y = (int)fdiv((uint32_t)p, a.d_cw), x = col0 + p - y * a.CW;
      *(f32x4_t*)(ot + t * 16 * opitch) = exact_tile(a, xim, strip, y * a.sh - a.ph, x * a.sw - a.pw, el) + bv;
    }
  }
  __syncthreads();
  const int run = min(a.NS * BSP_STRIP, a.O - set * a.NS * BSP_STRIP);  // a pixel's channels here
  const int opp = a.NS * 4;                                             // 16-byte pieces per pixel
  const int npix = plast + 1 - p0;
  const int64_t ybase = ((int64_t)img * a.M * a.N) * a.O + set * a.NS * BSP_STRIP;
  for (int i = tid; i < npix * opp; i += nthreads) {
    const int pix = (int)fdiv((uint32_t)i, a.d_opp), off = (i - pix * opp) * 4;
    const int y = (int)fdiv((uint32_t)(p0 + pix), a.d_cw), x = col0 + p0 + pix - y * a.CW;
    if (off >= run || x >= a.N) continue;
    const int64_t o = ybase + ((int64_t)y * a.N + x) * a.O + off;
    f32x4_t v = *(const f32x4_t*)(lds + pix * opitch + off * 4);
    if ((a.O & 3) == 0) {
      if (a.residual) v += *(const f32x4_t*)(a.residual + o);
      if (a.relu) v = f32x4_t{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
      if (a.stream)
        __builtin_nontemporal_store(v, (f32x4_t*)(a.Y + o));
      else
        *(f32x4_t*)(a.Y + o) = v;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (off + r >= run) break;
        float s = v[r];
        if (a.residual) s += a.residual[o + r];
        a.Y[o + r] = a.relu ? fmaxf(s, 0.f) : s;
      }
    }
  }
}

constexpr int kLdsLimit = 160 * 1024;
// Steps of a strip up to which eight products of nine are summed: sixteen rows with one weight each meet at most
// sixteen chunks of channels (4x16 blocks: thirty-two).  1x1 28x28x128->512 batch 8 10.8 -> 11.4 us, 56x56x64->64
// batch 32 15.1 -> 15.4, ->256 40.1 -> 42.0, 3x3 40x40x24->200 batch 16 the same.
constexpr int kShort = 4;

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct Pick {
  int32_t PT, PG, NS, ks, CW, nchunk, tpc, TPW, spst, lds;
  double cost;
};

// Tile, staging and split by a model of the busiest CU in clocks: the workgroups it runs, each with its
// steps (latency, or their share of LDS and matrix cores), what it stages and converts, what it stores, and a
// fixed chain, which resident workgroups hide of each other.
Pick choose(int B, int M, int N, int nstrips, int steps, int nslabs, int slab_chunks, int chunks, int H, int K, int lsh, int lsw, bool flat) {
  Pick best{};
  best.cost = 1e30;
  for (int PT : {2, 4})
    for (int PG : {1, 2, 4, 8}) {
      const int px = PT * 16 * PG;
      const auto width = [&](int cw) {
        const int64_t nchunk = cdiv(N, cw), tpc = cdiv((int64_t)M * cw, px), tiles = (int64_t)B * nchunk * tpc;
        const int orows = std::min(M, px % cw == 0 ? px / cw : (px - 2) / cw + 2);
        const int trows = (orows - 1) * lsh + H, tpw = (cw - 1) * lsw + K;
        const int64_t pix = (int64_t)trows * tpw;
        for (int spst = nslabs;; spst = (spst + 1) / 2) {
          const int ppp = std::min(spst * slab_chunks, chunks), nstages = cdiv(nslabs, spst);
          const int64_t patch = pix * ((ppp * 3 | 1) * 16);
          if (patch <= kLdsLimit)
            for (int ks : {1, 2, 4}) {
              if (PG * ks > 8 || ks > PT) continue;
              const int nsmax = std::min(nstrips, 8 / (PG * ks));
              const int NS = cdiv(nstrips, cdiv(nstrips, nsmax)), waves = NS * PG * ks;
              const int64_t ldsb = std::max({patch, ks > 1 ? (int64_t)waves * PT * 1024 : 0, (int64_t)px * (NS * 64 + 16)});
              if (ldsb > kLdsLimit) continue;
              const int64_t wgs = tiles * cdiv(nstrips, NS);
              const int resident = std::max(1, std::min((int)(kLdsLimit / ldsb), 16 / waves));
              const double percu = std::max(1.0, (double)cdiv(wgs, 256)), live = std::min<double>(percu, resident);
              const double mine = (double)steps / ks;
              const double comp = mine * std::max((12.0 + 27.0 * PT) * waves * live, 150.0 + 110.0 * PT) / live;
              const double stage = (double)pix * chunks * 32 / 12.0;
              const double store = (double)px * NS * 64 / 16.0;
              const double fix = (nstages * 1800.0 + 4000.0 + (ks > 1 ? 500.0 : 0.0)) / live;
              const double cost = percu * (comp + stage + store + fix);
              if (cost < best.cost)
                best = Pick{PT, PG, NS, ks, cw, (int32_t)nchunk, (int32_t)tpc, tpw, spst, (int32_t)ldsb, cost};
            }
          if (spst == 1) break;
        }
      };
      if (flat)
        width(px);
      else
        bsp_widths(N, 8, width);
    }
  return best;
}

template <int PT, bool SHORT, bool DIRECT>
int launch_inst(const X3Args& a, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_f32x3<PT, SHORT, DIRECT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_f32x3<PT, SHORT, DIRECT>), dim3((unsigned)(a.per_xcd * 8)), dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

}  // namespace

int bsp_launch_f32x3(const ConvParams& p, const void* plan_host, hipStream_t st) {
  const int32_t* hdr = (const int32_t*)plan_host;
  if (!hdr || hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION ||
      hdr[BSP_PLAN_O_W] != p.O || hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H || hdr[BSP_PLAN_K_W] != p.K ||
      hdr[BSP_PLAN_DTYPE_W] != BSP_F32 || hdr[BSP_PLAN_OFF_X3_W] == 0)
    return BSP_ERR_UNSUPPORTED;
  const int32_t* x3 = hdr + hdr[BSP_PLAN_OFF_X3_W];
  if (!x3[BSP_X3_USABLE_W] || x3[BSP_X3_NSTEPS_W] < 1) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.L * p.J * p.I * 4 >= (1ll << 32)) return BSP_ERR_UNSUPPORTED;
  const bool flat = p.H == 1 && p.K == 1 && p.ph == 0 && p.pw == 0 && p.sh == 1 && p.sw == 1;
  if (flat && p.P <= 256) return BSP_ERR_UNSUPPORTED;  // (straight from memory: fc_f32)
  const int nstrips = hdr[BSP_PLAN_NSTRIPS_W], steps = cdiv(x3[BSP_X3_NSTEPS_W], nstrips);
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (const char* e = std::getenv("BSP_X3")) {
    if (!std::atoi(e)) return BSP_ERR_UNSUPPORTED;
  } else
#endif
    if (!bsp_f32x3_beats(hdr[BSP_PLAN_BO_W], nstrips, steps, p.P, p.I, (int64_t)p.H * p.K)) return BSP_ERR_UNSUPPORTED;
  const int32_t* sec = p.plan + hdr[BSP_PLAN_OFF_X3_W];
  X3Args a{};
  a.X = (const float*)p.X;
  a.Y = (float*)p.Y;
  a.bias = p.bias;
  a.residual = (const float*)p.residual;
  a.slab_ptr = sec + x3[BSP_X3_OFF_SLAB_W];
  a.xdesc = (const unsigned char*)(sec + x3[BSP_X3_OFF_DESC_W]);
  a.wfrag = (const unsigned char*)(sec + x3[x3[BSP_X3_OFF_SRC_W] ? BSP_X3_OFF_SRC_W : BSP_X3_OFF_FRAG_W]);
  a.relu = p.relu;
  a.plan = p.plan;
  a.payload = (const float*)p.payload;
  a.lbo = __builtin_ctz(hdr[BSP_PLAN_BO_W]);
  a.I = p.I;
  a.O = p.O;
  a.H = p.H;
  a.K = p.K;
  a.nstrips = nstrips;
  a.nslabs = x3[BSP_X3_NSLABS_W];
  if (a.nslabs > 63) return BSP_ERR_UNSUPPORTED;
  a.slab_chunks = x3[BSP_X3_SLAB_W] / 8;
  int B = p.B;
  a.L = p.L;
  a.J = p.J;
  a.M = p.M;
  a.N = p.N;
  if (flat) {  // a plain matrix product over all pixels
    B = 1;
    a.L = a.M = 1;
    a.J = a.N = p.P;
    if ((int64_t)p.P * p.I >= (1ll << 32)) return BSP_ERR_UNSUPPORTED;
  }
  a.sh = p.sh;
  a.sw = p.sw;
  a.ph = p.ph;
  a.pw = p.pw;
  // a window of one row (column) needs only the rows (columns) it visits
  a.lsh = p.H == 1 ? 1 : p.sh;
  a.gsh = p.H == 1 ? p.sh : 1;
  a.lsw = p.K == 1 ? 1 : p.sw;
  a.gsw = p.K == 1 ? p.sw : 1;
  const int chunks = p.I / 8;
  Pick best;
  {
    // the search is a pure function of its arguments: remember its answers
    static std::mutex mu;
    static std::map<std::array<int32_t, 10>, Pick> memo;
    const std::array<int32_t, 10> key = {B, a.M, a.N, p.I, a.nstrips, p.H, p.K, p.sh * 2 + flat, p.sw, steps};
    std::unique_lock<std::mutex> lock(mu);
    const auto it = memo.find(key);
    if (it != memo.end()) {
      best = it->second;
    } else {
      lock.unlock();  // other layers' launches do not wait for this one's search
      best = choose(B, a.M, a.N, a.nstrips, steps, a.nslabs, a.slab_chunks, chunks, p.H, p.K, a.lsh, a.lsw, flat);
      lock.lock();
      if (memo.size() > 4096) memo.clear();
      memo.emplace(key, best);
    }
  }
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "x3: PT=%d PG=%d NS=%d ks=%d CW=%d nchunk=%d tpc=%d spst=%d/%d lds=%d cost=%.0f steps=%d\n", best.PT, best.PG, best.NS,
            best.ks, best.CW, best.nchunk, best.tpc, best.spst, a.nslabs, best.lds, best.cost, steps);
#endif
  if (best.PT == 0) return BSP_ERR_UNSUPPORTED;
  a.CW = best.CW;
  a.nchunk = best.nchunk;
  a.tpc = best.tpc;
  a.TPW = best.TPW;
  a.spst = best.spst;
  a.nstages = cdiv(a.nslabs, best.spst);
  a.ppp = std::min(best.spst * a.slab_chunks, chunks);
  a.pitch = (a.ppp * 3 | 1) * 16;
  a.NS = best.NS;
  a.PG = best.PG;
  a.ks = best.ks;
  a.lpg = __builtin_ctz(best.PG);
  a.lks = __builtin_ctz(best.ks);
  a.nset = cdiv(a.nstrips, best.NS);
  const int px = best.PT * 16 * best.PG;
  const int64_t tiles = (int64_t)B * a.nchunk * a.tpc, total = tiles * a.nset;
  if (total >= (1ll << 30)) return BSP_ERR_UNSUPPORTED;
  a.total = (int32_t)total;
  a.per_xcd = cdiv(total, 8);
  // multiply-high divisions are exact while dividend * divisor < 2^32 (the staging loop runs up to two
  // rounds of threads past the pieces, of which LDS holds at most 3413)
  const int64_t over = 3413 + 2 * 512;
  if ((total + 8) * a.nset >= (1ll << 32) || tiles * a.tpc >= (1ll << 32) ||
      (int64_t)B * a.nchunk * a.nchunk >= (1ll << 32) || (int64_t)a.tpc * px * a.CW >= (1ll << 32) ||
      over * std::max(a.ppp, a.TPW) >= (1ll << 32) || ((int64_t)px * best.NS * 4 + 512) * best.NS * 4 >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  a.d_nset = make_fastdiv((uint32_t)a.nset);
  a.d_tpc = make_fastdiv((uint32_t)a.tpc);
  a.d_nchunk = make_fastdiv((uint32_t)a.nchunk);
  a.d_cw = make_fastdiv((uint32_t)a.CW);
  a.d_tpw = make_fastdiv((uint32_t)a.TPW);
  a.d_ppp = make_fastdiv((uint32_t)a.ppp);
  a.d_opp = make_fastdiv((uint32_t)(best.NS * 4));
  a.opitch = best.NS * BSP_STRIP * 4 + 16;
  // whole 128-byte lines leave as streaming stores (nothing dirty is left for the kernel's end)
  a.stream = best.NS >= a.nstrips ? flat || p.O >= 32 : p.O % 32 == 0 && best.NS % 2 == 0;
  const int threads = 64 * best.NS * best.PG * best.ks;
  const size_t ldsb = (size_t)best.lds;
  auto launch = [&](auto direct) {
    constexpr bool D = decltype(direct)::value;
    if (steps <= kShort) return best.PT == 4 ? launch_inst<4, true, D>(a, threads, ldsb, st) : launch_inst<2, true, D>(a, threads, ldsb, st);
    return best.PT == 4 ? launch_inst<4, false, D>(a, threads, ldsb, st) : launch_inst<2, false, D>(a, threads, ldsb, st);
  };
  return x3[BSP_X3_OFF_SRC_W] ? launch(std::true_type{}) : launch(std::false_type{});
}
