// Layers of any shape on 16x16 matrix tiles, activations staged in LDS: bf16 layers whose channel
// counts are no multiple of eight, int8 layers (exact 32-bit sums, int8 or int32 results), and bf16
// layers of any channel count that are too small to fill the chip (bsp_rules.h).
//
// The weights come from the plan's step section (four (chunk, tap) pairs per step, a step's
// 16 x 64-byte operand contiguous), so only chunks that some block of a strip keeps have steps.  A
// chunk is 16 bytes of a pixel: eight bf16 channels or sixteen codes.
//
// What bounds it: on small layers the chain opening - patch - products - results, about 3.5 us with
// the launch, which the split of a strip's steps over waves shortens; instructions count there (a wave issues one
// per four clocks at best, its SIMD's second wave waits for the first, a taken branch is 28 clocks).  On large ones LDS (a
// step reads 1 KB per matrix instruction, half the matrix rate at best) and, with few steps per tile, the same
// chain times the tiles a CU works through, so what counts there is how many workgroups it holds:
// every instance keeps to 128 registers (144 in the four-tile one: 1x1 28x28x128->512 int8 28 us
// instead of 19).  Measured (general kernel / here): bf16 3x3 47x33x100->76 batch 3 36.9 / 5.9 us;
// 3x3 14x14x300->300 batch 16 150 / 22; 5x5 100x90x37->50 batch 2 52 / 9.4; 1x1 14x14x1001->333 batch 8
// 51 / 10.4; FC 32 x 1001 -> 999 28.6 / 5.4; int8 3x3 28x28x136->200 batch 8 28 / 8.2.  Which layers go
// to the other kernels instead: bsp_rules.h.
//
// A wait for everything before the patch's barrier, small outputs straight from the accumulators (bsp_any_direct), the
// bias asked for in the opening, zeros for a slab's unused pairs in its last step only and a strip's own partial sums kept in
// registers, together, data in the caches (cold): 1x7 17x17x160 batch 16 8.6 -> 7.3 us (9.3 -> 7.8), 5x5 35x35x48->64 batch 16
// 12.8 -> 10.2 (12.3 -> 9.6), 3x3 14x14x256 batch 1 5.6 -> 5.2 (5.8 -> 5.1), 7x7x512 batch 1 7.3 -> 6.9 (8.3 -> 7.0).
// The ring has four steps in every instance: eight for one lane tile cost a wave a SIMD and scratch for nothing.
#include "bsp_kept.h"
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
enum { kBf16 = 0, kI8 = 1 };

struct AnyArgs {
  const unsigned char* X;
  unsigned char* Y;
  const void* bias;                // fp32 or int32
  const unsigned char* residual;   // bf16
  const int32_t* slab_ptr;
  const unsigned char* xdesc;
  const unsigned char* wfrag;
  int32_t relu, shift, y32;        // y32: int32 results
  int32_t L, J, I, O, H, M, N;
  int32_t sh, sw, ph, pw, gsh, gsw, lsh, lsw;  // input pixels per staged pixel, staged pixels per output pixel
  int32_t CW, nchunk, tpc;         // output columns per chunk of columns, such chunks per row, tiles per chunk
  int32_t TPW, pitch, ppp;         // staged pixels per row, bytes per staged pixel, 16-byte pieces staged of each
  int32_t nslabs, spst, nstages, slab_bytes;   // the plan's slabs, how many are staged at a time
  int32_t nstrips, NS, PG, ks, lpg, lks, nset; // strips per workgroup, pixel groups, waves that share a strip's steps; log2
  int32_t total, per_xcd;
  int32_t opitch, stream;          // bytes per pixel of the output image; its pieces are whole output lines
  int32_t K, lbo;                  // log2 of the block rows' height (these and the two pointers: kept_only)
  const int32_t* plan;
  const unsigned char* payload;
  FastDiv d_nset, d_tpc, d_nchunk, d_cw;
  SmallDiv s_cw, s_tpw, s_ppp, s_opp;
};

template <int KIND>
__device__ __forceinline__ f32x4_t mma(u32x4_t a, u32x4_t b, f32x4_t c) {
  if constexpr (KIND == kI8)
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4_t, a),
                                                                           __builtin_bit_cast(i32x4_t, b),
                                                                           __builtin_bit_cast(i32x4_t, c), 0, 0, 0));
  else
    return mfma_bf16_16x16x32(a, b, c);
}
// the sum of two partial results, bit patterns of int32 or floats
template <int KIND>
__device__ __forceinline__ f32x4_t add4(f32x4_t a, f32x4_t b) {
  if constexpr (KIND == kI8)
    return __builtin_bit_cast(f32x4_t, __builtin_bit_cast(i32x4_t, a) + __builtin_bit_cast(i32x4_t, b));
  else
    return a + b;
}

// The first n of 16 bytes at any address (n >= 16: all of them).
__device__ __forceinline__ void store_first(unsigned char* p, u32x4_t v, int n, bool stream) {
  if (n >= 16) {
    if (stream)
      __builtin_nontemporal_store(v, (u32x4_t*)p);
    else
      __builtin_memcpy(p, &v, 16);
    return;
  }
  if (n & 8) {
    __builtin_memcpy(p, &v, 8);
    v = drop_low(v, 8);
    p += 8;
  }
  if (n & 4) {
    __builtin_memcpy(p, &v, 4);
    v = drop_low(v, 4);
    p += 4;
  }
  if (n & 2) {
    *(uint16_t*)p = (uint16_t)v.x;
    v = drop_low(v, 2);
    p += 2;
  }
  if (n & 1) *p = (uint8_t)v.x;
}
// The first n bytes (an even number) at any address, zeros for the others.
__device__ __forceinline__ u32x4_t load_first(const unsigned char* p, int n) {
  if (n >= 16) return load16(p);
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (n & 8) {
    __builtin_memcpy(&v, p, 8);
    p += 8;
  }
  uint32_t lo = 0;
  if (n & 4) {
    __builtin_memcpy(&lo, p, 4);
    p += 4;
  }
  const uint32_t hi = n & 2 ? *(const uint16_t*)p : 0u;
  const uint32_t a = n & 4 ? lo : hi, b = n & 4 ? hi : 0u;
  if (n & 8)
    v.z = a, v.w = b;
  else
    v.x = a, v.y = b;
  return v;
}

// The bias of channels ch to ch + 3; for those past the last channel some other channel's, which no result takes.  The same
// loads in every lane: with a path of its own for the end of the last strip (and for waves without a strip) that path's
// loads waited for everything in flight (int8 3x3 65x65x264->24 batch 4 with 16x4 blocks 10.3 -> 11.4 us, 1x1 8x8x232->35 3.4 -> 3.8).
template <int KIND>
__device__ __forceinline__ f32x4_t bias4(const AnyArgs& a, int ch) {
  u32x4_t b = {0u, 0u, 0u, 0u};
  if (a.bias) {
    const uint32_t* p = (const uint32_t*)a.bias;
    if (a.O % 4 == 0) {
      __builtin_memcpy(&b, p + min(ch, a.O - 4), 16);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) b[r] = p[min(ch + r, a.O - 1)];
    }
  }
  return __builtin_bit_cast(f32x4_t, b);
}

// One (tile of PT * 16 * PG output pixels) x (NS strips) per workgroup.  A tile is consecutive
// pixels of a chunk of image columns; its input patch, halo included, is staged as whole pixels
// (zeros outside the image and past the last channel), as many of the plan's slabs at a time as
// LDS takes.  A staged pixel is an odd number of 16-byte pieces, so pixels of a matrix tile that lie in
// one patch row read different banks; those of two rows can collide (bf16 3x3 47x33x100->76: 0.19 M of
// 0.51 M LDS cycles).  Wave = (strip, pixel group, share of the strip's steps): a step's
// weights come from the plan through a register ring of D, its activations from LDS one step ahead.  (A ring of eight
// with two or four steps read together, for one tile: 3x3 7x7x512 batch 1 as fast, 6.7 us, but a register budget that
// holds four waves a SIMD instead of five, and scalars in scratch; FC int8 20600 -> 120 batch 5 19.5 us instead of 17.7.)
// The bf16 instances keep up to eight scalars that only the results need in lanes of a vector register.  Reading
// them from the argument block again there spills none and costs more: 232 small layers 1.3 to 1.7 % slower, 350 others 0.6 %.
template <int KIND, int PT, bool VEC, bool DIRECT>
__global__ __launch_bounds__(512, 4) void conv_any(AnyArgs a) {
  kernarg_touch<AnyArgs>();
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int D = 4, ES = KIND == kI8 ? 1 : 2, U = 4;
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
  const int m0 = (int)fdiv((uint32_t)p0, a.d_cw), rel0 = p0 - m0 * a.CW;  // the tile's first row, its first pixel there
  const int plast = min(p0 + px, a.M * a.CW) - 1;
  const int rows = ((int)fdiv((uint32_t)plast, a.d_cw) - m0) * a.lsh + a.H;  // staged rows

  const int k = wave & (a.ks - 1), sp = wave >> a.lks, pg = sp & (a.PG - 1), si = sp >> a.lpg;
  const int strip = set * a.NS + si;
  const bool active = si < a.NS && strip < a.nstrips;
  // the strip's step ranges, one slab boundary per lane
  const int tab = a.slab_ptr[(active ? strip : 0) * (a.nslabs + 1) + min(lane, a.nslabs)];
  f32x4_t bv;

  const int iy0 = m0 * a.sh - a.ph, ix0 = col0 * a.sw - a.pw;
  const int pieces = rows * a.TPW * a.ppp;
  const int rowb = a.I * ES;  // bytes of a pixel
  const unsigned char* xim = a.X + (int64_t)img * a.L * a.J * rowb;
  const int rowpitch = a.TPW * a.pitch;

  // ---- staging: U 16-byte pieces per thread in flight.  Rounds of U pieces go out without a branch between them, the last
  // pieces one by one (not where the registers for both would not do)
  constexpr bool ROUNDS = VEC || PT < 4;
  u32x4_t v[U];
  int dst[U], off[U];
  auto ask = [&](int f0, int c0, auto whole) {  // f0: the wave's first piece, c0: first byte of a pixel that is staged
#pragma unroll
    for (int u = 0; u < U; ++u) {
      dst[u] = -1;
      if (!decltype(whole)::value && f0 + u * nthreads >= pieces) continue;
      const int f = f0 + u * nthreads + lane;
      const int pix = (int)sdiv((uint32_t)f, a.s_ppp), part = f - (int)__umul24(pix, a.ppp);
      const int r = (int)sdiv((uint32_t)pix, a.s_tpw), x = pix - (int)__umul24(r, a.TPW);
      const int iy = iy0 + (int)__umul24(r, a.gsh), ix = ix0 + (int)__umul24(x, a.gsw);
      off[u] = c0 + part * 16;
      if (f < pieces && off[u] < rowb) dst[u] = (int)__umul24(pix, a.pitch) + part * 16;
      v[u] = u32x4_t{0u, 0u, 0u, 0u};
      if (dst[u] >= 0 && (unsigned)iy < (unsigned)a.L && (unsigned)ix < (unsigned)a.J) {
        const unsigned char* src = xim + (uint32_t)(iy * a.J + ix) * (uint32_t)rowb;
        v[u] = VEC ? *(const u32x4_t*)(src + off[u]) : piece_ask(src, off[u], rowb);
      }
    }
  };
  auto place = [&] {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!VEC) {
        __builtin_amdgcn_sched_barrier(0);  // (one shift after the other: all at once take 40 registers)
        v[u] = piece_place(v[u], off[u], rowb);
      }
      if (dst[u] >= 0) *(u32x4_t*)(lds + dst[u]) = v[u];
    }
  };
  int base[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int p = min(rel0 + (pg * PT + t) * 16 + jn, plast - m0 * a.CW);
    const int y = (int)sdiv((uint32_t)p, a.s_cw), x = p - (int)__umul24(y, a.CW);
    base[t] = (int)__umul24(__umul24(__umul24(y, a.lsh), a.TPW) + __umul24(x, a.lsw), a.pitch);
  }
  f32x4_t acc[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  for (int stg = 0; stg < a.nstages; ++stg) {
    const int sl0 = stg * a.spst, sl1 = min(sl0 + a.spst, a.nslabs);
    const int slo = __builtin_amdgcn_readlane(tab, sl0), shi = __builtin_amdgcn_readlane(tab, sl1);
    const int n = active && shi - slo > k ? (shi - slo - k + a.ks - 1) >> a.lks : 0;  // this wave's steps

    // ---- weights: a ring of D steps
    u32x4_t wr[D];
    int dr[D];  // descriptors
    // Where a step's slab lies in a staged pixel, its first step, the next slab's first.  int8 finds that when it asks for a step,
    // bf16, which needs to know a slab's last step too, when it reads the step's activations (found at the request: 5x5
    // 35x35x48->64 batch 16 10.5 -> 11.2 us, 1500 random layers 1.5 % more; int8 the other way round, 3x3 65x65x264->24 batch 4
    // with 16x4 blocks 10.5 -> 11.1).
    [[maybe_unused]] int pos[D];
    int fcs = slo + k, fsl = sl0, fadd = 0, fbeg = slo, fend = __builtin_amdgcn_readlane(tab, sl0 + 1);
    auto find = [&](int cs) {
      while (cs >= fend) {
        fadd += a.slab_bytes;
        ++fsl;
        fbeg = fend;
        fend = __builtin_amdgcn_readlane(tab, fsl + 1);
      }
    };
    auto fetch = [&](int d) {
      const int cs = min(fcs, shi - 1);  // (past the end: the last step again, never used)
      fcs += a.ks;
      if constexpr (KIND == kI8) {
        find(cs);
        pos[d] = fadd;
      }
      dr[d] = *(const int*)(a.xdesc + ((uint32_t)cs * 16u + (uint32_t)g * 4u));
      wr[d] = *(const u32x4_t*)(a.wfrag + ((uint32_t)cs * 1024u + (uint32_t)lane * 16u));
    };
    const int c0 = sl0 * a.slab_bytes;
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < n) fetch(d);  // their latency passes while the patch is staged
    if (VEC && stg == 0) bv = bias4<KIND>(a, (active ? strip : 0) * BSP_STRIP + 4 * g);
    if (stg > 0) __syncthreads();
    int f0 = wave * 64;
    for (; ROUNDS ? f0 + (U - 1) * nthreads < pieces : f0 < pieces; f0 += U * nthreads) {
      ask(f0, c0, std::bool_constant<ROUNDS>{});
      place();
      __builtin_amdgcn_s_waitcnt(0);  // (once here, or the compiler waits before a round's first request, for the weights too)
    }
    if (ROUNDS && f0 < pieces) {
      ask(f0, c0, std::false_type{});
      place();
    }
    // (the weights asked for before the patch are there by now; the wait tells the compiler so, which otherwise
    // waits for the whole ring at every step)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // ---- products
    [[maybe_unused]] int rcs = slo + k;
    auto read = [&](int d, u32x4_t (&f)[PT]) {
      [[maybe_unused]] const int cs = min(rcs, shi - 1);
      if constexpr (KIND == kBf16) {
        rcs += a.ks;
        find(cs);
      }
      uint32_t desc = (uint32_t)dr[d];
      asm volatile("" : "+v"(desc));  // decoded here, not where it is loaded: no early wait
      const uint32_t o = ((desc & 0xFFFFu) << 4) + (uint32_t)(KIND == kI8 ? pos[d] : fadd) + __umul24((desc >> 16) & 0xFFu, rowpitch) +
                         __umul24(desc >> 24, a.pitch);
#pragma unroll
      for (int t = 0; t < PT; ++t) f[t] = *(const u32x4_t*)(lds + base[t] + o);
      if constexpr (KIND == kBf16) {
        // a pair that fills up a slab's last step multiplies zeros with zeros, not with whatever
        // (an infinity) lies at its descriptor's address
        if (cs == fend - 1) {
          const bool real = desc != 0u || (g == 0 && cs == fbeg);
#pragma unroll
          for (int t = 0; t < PT; ++t) f[t] = real ? f[t] : u32x4_t{0u, 0u, 0u, 0u};
        }
      }
    };
    auto mfmas = [&](int d, const u32x4_t (&f)[PT]) {
#pragma unroll
      for (int t = 0; t < PT; ++t) acc[t] = mma<KIND>(wr[d], f[t], acc[t]);
    };
    auto refill = [&](int d) {
      __builtin_amdgcn_sched_barrier(0);
      fetch(d);
      __builtin_amdgcn_sched_barrier(0);
    };
    u32x4_t fa[PT], fb[PT];
    int i = 0;
    if (n > 0) read(0, fa);
    for (; i + D < n; i += D) {
#pragma unroll
      for (int d = 0; d < D; d += 2) {
        read(d + 1, fb);
        mfmas(d, fa);
        refill(d);
        read((d + 2) % D, fa);
        mfmas(d + 1, fb);
        refill(d + 1);
      }
    }
#pragma unroll
    for (int d = 0; d < D; d += 2) {
      if (i + d + 1 < n) read(d + 1, fb);
      if (i + d < n) mfmas(d, fa);
      if (d + 2 < D && i + d + 2 < n) read(d + 2, fa);
      if (i + d + 1 < n) mfmas(d + 1, fb);
    }
  }

  // ---- waves that share a strip: partial sums through LDS.  The strip's matrix tiles are dealt out to
  // its waves, each adds up its tiles' sums in the order of the waves.
  if (a.ks > 1) {
    __syncthreads();
    f32x4_t* red = (f32x4_t*)lds;  // [wave][PT][64]
#pragma unroll
    for (int t = 0; t < PT; ++t)
      if ((t & (a.ks - 1)) != k) red[(wave * PT + t) * 64 + lane] = acc[t];
    __syncthreads();
    const f32x4_t* first = red + (wave - k) * (PT * 64) + lane;
    // (all of a tile's sums are asked for at once: one after the other they took most of a
    // microsecond of a small layer's five)
    auto add_up = [&](auto n) {
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        if ((t & (decltype(n)::value - 1)) != k) continue;
        f32x4_t v[decltype(n)::value];
#pragma unroll
        for (int s = 0; s < decltype(n)::value; ++s) v[s] = s == k ? acc[t] : first[(s * PT + t) * 64];
#pragma unroll
        for (int s = 1; s < decltype(n)::value; ++s) v[0] = add4<KIND>(v[0], v[s]);
        acc[t] = v[0];
      }
    };
    if (a.ks == 8)
      add_up(std::integral_constant<int, 8>{});
    else if (a.ks == 4)
      add_up(std::integral_constant<int, 4>{});
    else
      add_up(std::integral_constant<int, 2>{});
  }
  // ---- results: bias and the one rounding (or the rescale).  Small bf16 outputs leave from here, eight bytes per
  // lane; the others go into an LDS image of the tile's output, and then all waves copy that out, 16 contiguous
  // bytes per lane, with the residual and ReLU
  const int opitch = a.opitch;
  int id = tid;
  asm volatile("" : "+v"(id));  // (lane, column and group once more: no registers for them until here)
  const int ln = id & 63, lg = ln >> 4, lj = ln & 15;
  const int ch = strip * BSP_STRIP + 4 * lg;
  // (with pixels at any alignment its four registers are worth more until here: 1x1 64x64x417->72 batch 6 11.2 -> 8.6 us)
  if constexpr (!VEC) bv = bias4<KIND>(a, ch);
  u32x2_t out[PT];
  uint32_t bad = 0;  // bit 15 or 31: a result that is not finite (an exponent of ones carries over)
  auto not_finite = [](uint32_t pair) { return (pair & 0x7F807F80u) + 0x00800080u; };
  if constexpr (KIND == kBf16) {
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      if ((t & (a.ks - 1)) != k) continue;
      const f32x4_t v = acc[t] + bv;
      out[t] = u32x2_t{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
      bad |= not_finite(out[t].x) | not_finite(out[t].y);
    }
    bad = active && __ballot(bad & 0x80008000u);
  }
  [[maybe_unused]] auto send = [&] {
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      if ((t & (a.ks - 1)) != k) continue;
      const int i = (pg * PT + t) * 16 + lj, r = rel0 + i;
      const int dy = (int)sdiv((uint32_t)r, a.s_cw), x = col0 + r - (int)__umul24(dy, a.CW);
      if (p0 + i > plast || x >= a.N || ch >= a.O) continue;
      const uint32_t o = (((uint32_t)img * (uint32_t)a.M + (uint32_t)(m0 + dy)) * (uint32_t)a.N + (uint32_t)x) * (uint32_t)a.O + (uint32_t)ch;
      u32x2_t res = {0u, 0u};
      if (a.residual) res = *(const u32x2_t*)(a.residual + o * 2u);
      if (a.residual || a.relu) out[t] = post_bf16x4_reg(out[t], res, a.residual != nullptr, a.relu);
      *(u32x2_t*)(a.Y + o * 2u) = out[t];
    }
  };
  if constexpr (DIRECT)
    if (active && !bad) send();
  __syncthreads();  // everybody is done with the patch (the partial sums)
  if constexpr (DIRECT)
    if (!bad) return;
  if (active) {
    unsigned char* ot = lds + (pg * PT * 16 + lj) * opitch;
    const RescaleI8 rescale(__builtin_bit_cast(i32x4_t, bv), KIND == kI8 ? a.shift : 0);
#pragma unroll
    for (int t = 0; t < PT; ++t, ot += 16 * opitch) {
      if ((t & (a.ks - 1)) != k) continue;
      const int c = si * BSP_STRIP + 4 * lg;
      if constexpr (KIND == kBf16)
        *(u32x2_t*)(ot + c * 2) = out[t];
      else if (a.y32)
        *(f32x4_t*)(ot + c * 4) = add4<KIND>(acc[t], bv);
      else
        *(uint32_t*)(ot + c) = rescale(__builtin_bit_cast(i32x4_t, acc[t]));
    }
    if constexpr (KIND == kBf16) {
      if (bad) {
        // (the arguments once more: what only this needs takes no scalar registers before)
        auto* again = (const __attribute__((address_space(4))) AnyArgs*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(again));
        const AnyArgs& b = *(const AnyArgs*)again;
        auto place = [&](int tile) { return (u32x2_t*)(lds + (tile * 16 + lj) * opitch + (si * BSP_STRIP + 4 * lg) * 2); };
#pragma unroll 1
        for (int t = k; t < PT; t += b.ks) {
          const int tile = pg * PT + t;
          if (!__ballot((not_finite(place(tile)->x) | not_finite(place(tile)->y)) & 0x80008000u)) continue;
          const int p = min(p0 + tile * 16 + lj, plast);
          const int y = (int)fdiv((uint32_t)p, b.d_cw), x = col0 + p - y * b.CW;
          const f32x4_t v = kept_only<VEC>(b, b.X + (int64_t)img * b.L * b.J * b.I * 2, strip, y * b.sh - b.ph, x * b.sw - b.pw, ln) +
                            bias4<KIND>(b, ch);
          asm volatile("" ::: "memory");  // (read again, not kept)
          auto take = [&](uint32_t was, uint32_t now) {  // those of the results that are not finite
            const uint32_t m = (not_finite(was) >> 15 & 0x00010001u) * 0xFFFFu;
            return (was & ~m) | (now & m);
          };
          *place(tile) = u32x2_t{take(place(tile)->x, pack_bf16x2(v.x, v.y)), take(place(tile)->y, pack_bf16x2(v.z, v.w))};
        }
        if constexpr (DIRECT) {
#pragma unroll
          for (int t = 0; t < PT; ++t) out[t] = *place(pg * PT + t);
          send();
        }
      }
    }
  }
  if constexpr (DIRECT) return;
  __syncthreads();
  const int os = KIND == kBf16 ? 2 : a.y32 ? 4 : 1;  // bytes per result
  const int run = min(a.NS * BSP_STRIP, a.O - set * a.NS * BSP_STRIP) * os;  // a pixel's bytes here
  const int opp = a.NS * os;                         // 16-byte pieces per pixel
  const int npix = plast + 1 - p0;
  const int64_t ybase = ((int64_t)img * a.M * a.N) * a.O + set * a.NS * BSP_STRIP;
  for (int i = tid; i < npix * opp; i += nthreads) {
    const int pix = (int)sdiv((uint32_t)i, a.s_opp), off = (i - pix * opp) * 16;
    const int dy = (int)sdiv((uint32_t)(rel0 + pix), a.s_cw), y = m0 + dy, x = col0 + rel0 + pix - (int)__umul24(dy, a.CW);
    const int n = run - off;
    if (n <= 0 || x >= a.N) continue;
    const int64_t o = (ybase + ((int64_t)y * a.N + x) * a.O) * os + off;
    u32x4_t v = *(const u32x4_t*)(lds + pix * opitch + off);
    if constexpr (KIND == kBf16) {
      if (a.residual || a.relu) {
        u32x4_t r = {0u, 0u, 0u, 0u};
        if (a.residual) r = load_first(a.residual + o, n);
        const u32x2_t lo = post_bf16x4_reg(u32x2_t{v.x, v.y}, u32x2_t{r.x, r.y}, a.residual != nullptr, a.relu);
        const u32x2_t hi = post_bf16x4_reg(u32x2_t{v.z, v.w}, u32x2_t{r.z, r.w}, a.residual != nullptr, a.relu);
        v = u32x4_t{lo.x, lo.y, hi.x, hi.y};
      }
    }
    store_first(a.Y + o, v, n, a.stream);
  }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct Pick {
  int32_t PT, PG, NS, ks, CW, nchunk, tpc, TPW, spst, lds;
  double cost;
};

// Tile, staging and split by a model of the busiest CU in clocks: the workgroups it runs, each with
// its steps (their latency, or their share of the issue slots and LDS), the bytes it stages and the
// fixed chain, which resident workgroups hide of each other.  On 46 shapes (small, ragged and int8 layers) its choice measured 3 % above
// the best of up to 70 candidates in the mean, 0.3 % in the median, 9 to 17 % on six of them.
Pick choose(int B, int M, int N, int os, int nstrips, int steps, int nslabs, int slab_pieces, int pieces, int H, int K, int lsh,
            int lsw, bool flat) {
  Pick best{};
  double best_cost = 1e30;
  for (int PT : {1, 2, 4})
    for (int PG : {1, 2, 4, 8}) {
      const int px = PT * 16 * PG;
      const auto width = [&](int cw) {
        const int64_t nchunk = cdiv(N, cw), tpc = cdiv((int64_t)M * cw, px), tiles = (int64_t)B * nchunk * tpc;
        const int orows = std::min(M, px % cw == 0 ? px / cw : (px - 2) / cw + 2);
        const int trows = (orows - 1) * lsh + H, tpw = (cw - 1) * lsw + K;
        const int64_t pix = (int64_t)trows * tpw;
        for (int spst = nslabs;; spst = (spst + 1) / 2) {
          const int ppp = std::min(spst * slab_pieces, pieces), nstages = cdiv(nslabs, spst);
          const int64_t patch = pix * ((ppp | 1) * 16);
          if (patch <= 160 * 1024)
            for (int ks : {1, 2, 4, 8}) {
              if (PG * ks > 8) continue;
              const int nsmax = std::min(nstrips, 8 / (PG * ks));
              const int NS = cdiv(nstrips, cdiv(nstrips, nsmax)), waves = NS * PG * ks;
              const int64_t ldsb = std::max({patch, ks > 1 ? (int64_t)waves * PT * 1024 : 0, (int64_t)px * (NS * 16 * os + 16)});
              if (ldsb > 160 * 1024) continue;
              const int64_t wgs = tiles * cdiv(nstrips, NS);
              const int resident = std::max(1, std::min((int)(160 * 1024 / ldsb), 16 / waves));
              const double percu = std::max(1.0, (double)cdiv(wgs, 256)), live = std::min<double>(percu, resident);
              const double mine = (double)steps / ks;
              // a wave's step: its latency, or its share of a CU's issue, LDS and weight traffic
              const double wstep = 24.0 + 10.0 * PT;
              const double comp = mine * std::max(wstep * waves * live, 120.0 + 24.0 * PT) / live;
              const double stage = (double)pix * pieces * 16 / 20.0;
              const double fix = (nstages * 1600.0 + 4000.0 + (ks > 1 ? 500.0 : 0.0)) / live;
              const double cost = percu * (comp + stage + fix);
              if (cost < best_cost) {
                best_cost = cost;
                best = Pick{PT, PG, NS, ks, cw, (int32_t)nchunk, (int32_t)tpc, tpw, spst, (int32_t)ldsb, cost};
              }
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

template <int KIND, int PT, bool VEC, bool DIRECT>
int launch_inst(const AnyArgs& a, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_any<KIND, PT, VEC, DIRECT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) !=
        hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_any<KIND, PT, VEC, DIRECT>), dim3((unsigned)(a.per_xcd * 8)), dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}
// vec: pixels of X are whole 16-byte pieces; direct: results leave from the accumulators
template <int KIND, int PT>
int launch_conv(const AnyArgs& a, bool vec, bool direct, int threads, size_t ldsb, hipStream_t st) {
  if constexpr (KIND == kBf16)
    if (direct) return vec ? launch_inst<KIND, PT, true, true>(a, threads, ldsb, st) : launch_inst<KIND, PT, false, true>(a, threads, ldsb, st);
  return vec ? launch_inst<KIND, PT, true, false>(a, threads, ldsb, st) : launch_inst<KIND, PT, false, false>(a, threads, ldsb, st);
}

template <int KIND>
int launch_kind(const ConvParams& p, const int32_t* hdr, int y32, int shift, hipStream_t st) {
  constexpr int ES = KIND == kI8 ? 1 : 2;
  if (hdr[BSP_PLAN_NSTEPS_W] < 1 || p.I * ES < 16) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.L * p.J * p.I * ES >= (1ll << 31) || (int64_t)hdr[BSP_PLAN_NSTEPS_W] * 1024 >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  AnyArgs a{};
  a.X = (const unsigned char*)p.X;
  a.Y = (unsigned char*)p.Y;
  a.bias = p.bias;
  a.residual = (const unsigned char*)p.residual;
  a.slab_ptr = p.plan + hdr[BSP_PLAN_OFF_SLAB_W];
  a.xdesc = (const unsigned char*)(p.plan + hdr[BSP_PLAN_OFF_XDESC_W]);
  a.wfrag = (const unsigned char*)(p.plan + hdr[BSP_PLAN_OFF_WFRAG_W]);
  a.plan = p.plan;
  a.payload = (const unsigned char*)p.payload;
  a.lbo = __builtin_ctz(hdr[BSP_PLAN_BO_W]);
  a.K = p.K;
  a.relu = p.relu;
  a.shift = shift;
  a.y32 = y32;
  a.I = p.I;
  a.O = p.O;
  a.H = p.H;
  a.nstrips = hdr[BSP_PLAN_NSTRIPS_W];
  a.nslabs = hdr[BSP_PLAN_NSLABS_W];
  if (a.nslabs > 63) return BSP_ERR_UNSUPPORTED;
  a.slab_bytes = hdr[BSP_PLAN_SLAB_W] * ES;
  const bool vec = (p.I * ES) % 16 == 0 && (reinterpret_cast<uintptr_t>(p.X) & 15u) == 0;
  const bool flat = p.H == 1 && p.K == 1 && p.ph == 0 && p.pw == 0 && p.sh == 1 && p.sw == 1;
  int B = p.B;
  a.L = p.L;
  a.J = p.J;
  a.M = p.M;
  a.N = p.N;
  if (flat) {  // a plain matrix product over all pixels
    B = 1;
    a.L = a.M = 1;
    a.J = a.N = p.P;
    if ((int64_t)p.P * p.I * ES >= (1ll << 31)) return BSP_ERR_UNSUPPORTED;
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
  const int os = KIND == kBf16 ? 2 : y32 ? 4 : 1;
  const int pieces = cdiv(p.I * ES, 16), slab_pieces = a.slab_bytes / 16;
  Pick best;
  {
    // the search is a pure function of its arguments: remember its answers
    static std::mutex mu;
    static std::map<std::array<int32_t, 12>, Pick> memo;
    const int steps = cdiv(hdr[BSP_PLAN_NSTEPS_W], a.nstrips);
    const std::array<int32_t, 12> key = {B, a.M, a.N, p.I, p.O, p.H, p.K, p.sh * 2 + flat, p.sw, steps, a.nslabs, os};
    std::unique_lock<std::mutex> lock(mu);
    const auto it = memo.find(key);
    if (it != memo.end()) {
      best = it->second;
    } else {
      lock.unlock();  // other layers' launches do not wait for this one's search
      best = choose(B, a.M, a.N, os, a.nstrips, steps, a.nslabs, slab_pieces, pieces, p.H, p.K, a.lsh, a.lsw, flat);
      lock.lock();
      if (memo.size() > 4096) memo.clear();
      memo.emplace(key, best);
    }
  }
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (const char* e = std::getenv("BSP_ANY_TUNE")) {
    int t[6];  // PT, PG, NS, ks, chunks of columns, slabs per stage
    if (sscanf(e, "%d,%d,%d,%d,%d,%d", t, t + 1, t + 2, t + 3, t + 4, t + 5) == 6) {
      Pick b{};
      b.PT = t[0]; b.PG = t[1]; b.NS = t[2]; b.ks = t[3]; b.spst = std::min(t[5], a.nslabs);
      const int px = b.PT * 16 * b.PG;
      b.CW = flat ? px : cdiv(a.N, t[4]);
      b.nchunk = cdiv(a.N, b.CW);
      b.tpc = cdiv((int64_t)a.M * b.CW, px);
      const int orows = std::min(a.M, px % b.CW == 0 ? px / b.CW : (px - 2) / b.CW + 2);
      b.TPW = (b.CW - 1) * a.lsw + p.K;
      const int ppp = std::min(b.spst * slab_pieces, pieces);
      const int64_t patch = (int64_t)((orows - 1) * a.lsh + p.H) * b.TPW * ((ppp | 1) * 16);
      const int64_t l = std::max({patch, b.ks > 1 ? (int64_t)b.NS * b.PG * b.ks * b.PT * 1024 : 0, (int64_t)px * (b.NS * 16 * os + 16)});
      if (l > 160 * 1024 || b.NS * b.PG * b.ks > 8 || b.NS > a.nstrips) return BSP_ERR_UNSUPPORTED;
      b.lds = (int)l;
      best = b;
    }
  }
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "any: PT=%d PG=%d NS=%d ks=%d CW=%d nchunk=%d tpc=%d spst=%d/%d lds=%d\n", best.PT, best.PG, best.NS,
            best.ks, best.CW, best.nchunk, best.tpc, best.spst, a.nslabs, best.lds);
#endif
  if (best.PT == 0) return BSP_ERR_UNSUPPORTED;
  a.CW = best.CW;
  a.nchunk = best.nchunk;
  a.tpc = best.tpc;
  a.TPW = best.TPW;
  a.spst = best.spst;
  a.nstages = cdiv(a.nslabs, best.spst);
  a.ppp = std::min(best.spst * slab_pieces, pieces);
  a.pitch = (a.ppp | 1) * 16;
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
  // multiply-high divisions are exact while dividend * divisor < 2^32; what lies in a tile or a patch (at most 10240
  // pieces, 512 pixels) is divided and multiplied in 24 bits, input pixels per staged row or column too
  if ((total + 8) * a.nset >= (1ll << 32) || tiles * a.tpc >= (1ll << 32) ||
      (int64_t)B * a.nchunk * a.nchunk >= (1ll << 32) || (int64_t)a.tpc * px * a.CW >= (1ll << 32) ||
      (a.gsh >= (1 << 24) && a.M > 1) || (a.gsw >= (1 << 24) && a.N > 1))
    return BSP_ERR_UNSUPPORTED;
  a.d_nset = make_fastdiv((uint32_t)a.nset);
  a.d_tpc = make_fastdiv((uint32_t)a.tpc);
  a.d_nchunk = make_fastdiv((uint32_t)a.nchunk);
  a.d_cw = make_fastdiv((uint32_t)a.CW);
  a.s_cw = make_smalldiv((uint32_t)a.CW);
  a.s_tpw = make_smalldiv((uint32_t)a.TPW);
  a.s_ppp = make_smalldiv((uint32_t)a.ppp);
  a.s_opp = make_smalldiv((uint32_t)(best.NS * os));
  a.opitch = best.NS * BSP_STRIP * os + 16;
  // whole 128-byte lines leave as streaming stores (nothing dirty is left for the kernel's end)
  a.stream = p.O * os % 16 == 0 && (reinterpret_cast<uintptr_t>(p.Y) & 15u) == 0 &&
             (best.NS >= a.nstrips ? flat || p.O * os >= 128 : p.O * os % 128 == 0 && best.NS * BSP_STRIP * os % 128 == 0);
  const bool direct = KIND == kBf16 && bsp_any_direct(p.O, (int64_t)p.P * p.O);
  const int threads = 64 * best.NS * best.PG * best.ks;
  switch (best.PT) {
    case 1: return launch_conv<KIND, 1>(a, vec, direct, threads, (size_t)best.lds, st);
    case 2: return launch_conv<KIND, 2>(a, vec, direct, threads, (size_t)best.lds, st);
    case 4: return launch_conv<KIND, 4>(a, vec, direct, threads, (size_t)best.lds, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

const int32_t* plan_of(const ConvParams& p, int dtype, const void* plan_host) {
  const int32_t* hdr = (const int32_t*)plan_host;
  if (!hdr || hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION ||
      hdr[BSP_PLAN_O_W] != p.O || hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H || hdr[BSP_PLAN_K_W] != p.K ||
      hdr[BSP_PLAN_DTYPE_W] != dtype)
    return nullptr;
  return hdr;
}

}  // namespace

// The models of both kernels, weighed: a pure function of the layer, its plan and the device, so its answers are kept.
static bool model_beats_rows(const ConvParams& p, const int32_t* hdr, int64_t mm) {
  if (p.sh != p.sw || p.sh > 2 || hdr[BSP_PLAN_OFF_ROWS_W] == 0) return false;
  const int32_t* rs = hdr + hdr[BSP_PLAN_OFF_ROWS_W];
  const int nstrips = hdr[BSP_PLAN_NSTRIPS_W], nsteps = hdr[BSP_PLAN_NSTEPS_W];
  static std::mutex mu;
  static std::map<std::array<int32_t, 13>, bool> memo;
  const std::array<int32_t, 13> key = {p.B, p.M, p.N, p.I, p.O, p.H * 4 + p.K, p.sh, p.ph * 65536 + p.pw, nsteps, hdr[BSP_PLAN_NSLABS_W], rs[BSP_ROWS_NCS_W], rs[BSP_ROWS_NSTRIPS_W],
                                       rs[BSP_ROWS_CW_W] * 4096 + rs[BSP_ROWS_SLAB_W]};
  std::unique_lock<std::mutex> lock(mu);
  const auto it = memo.find(key);
  if (it != memo.end()) return it->second;
  lock.unlock();  // other layers' launches do not wait for this one's searches
  const Pick pick = choose(p.B, p.M, p.N, 2, nstrips, cdiv(nsteps, nstrips), hdr[BSP_PLAN_NSLABS_W], hdr[BSP_PLAN_SLAB_W] / 8, cdiv(p.I, 8), p.H, p.K, p.sh, p.sw, false);
  const bool beats = pick.PT && bsp_any_model_beats(p.sh > 1, mm, p.O, pick.cost, bsp_rows_cost(p, rs));
  lock.lock();
  if (memo.size() > 4096) memo.clear();
  memo.emplace(key, beats);
  return beats;
}

bool bsp_any_beats(const ConvParams& p, const void* plan_host, BspRival rival) {
  const int32_t* hdr = plan_of(p, BSP_BF16, plan_host);
  if (!hdr) return false;
  const int64_t mm = (int64_t)((p.P + 15) / 16) * hdr[BSP_PLAN_NSTEPS_W];
  const bool strided = p.sh > 1 || p.sw > 1;
  if (bsp_any_beats_bf16(rival, hdr[BSP_PLAN_BO_W], p.H, p.K, strided, mm, (int64_t)p.P * p.O, p.I, p.O)) return true;
  return rival == BSP_RIVAL_ROWS && bsp_any_models_decide(p.H, p.K, strided, mm, p.P, p.O) && model_beats_rows(p, hdr, mm);
}

bool bsp_any_beats_i8(const ConvParams& p, const void* plan_host) {
  const int32_t* hdr = plan_of(p, BSP_I8, plan_host);
  return hdr && bsp_any_beats_lds_i8(hdr[BSP_PLAN_NSLABS_W], (int64_t)p.H * p.K, p.P, p.O,
                                     (int64_t)((p.P + 15) / 16) * hdr[BSP_PLAN_NSTEPS_W]);
}

int bsp_launch_any(const ConvParams& p, const void* plan_host, hipStream_t st) {
  const int32_t* hdr = plan_of(p, BSP_BF16, plan_host);
  return hdr ? launch_kind<kBf16>(p, hdr, 0, 0, st) : BSP_ERR_UNSUPPORTED;
}

int bsp_launch_any_i8(const ConvParams& p, const void* plan_host, int y_i8, int shift, hipStream_t st) {
  const int32_t* hdr = plan_of(p, BSP_I8, plan_host);
  return hdr ? launch_kind<kI8>(p, hdr, !y_i8, shift, st) : BSP_ERR_UNSUPPORTED;
}
