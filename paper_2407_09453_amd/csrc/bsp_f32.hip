// Single-precision layers on the 4x4x1 matrix instruction (sixteen 4x4 tiles in one go).
//
// Why that instruction.  A 16x16x4 tile has sixteen rows, so with 8x8 blocks it runs the union of
// two block rows' kept columns (about 1.5 times the kept work at half density).  The 4x4x1 form
// multiplies sixteen independent 4x4 tiles; with its broadcast controls (cbsz = 4, abid = i) all
// sixteen take rows from group i of the A operand.  So lane = pixel (sixteen tiles of four pixels),
// and one A register holds a whole kept block at one window tap, whatever the granularity:
// lane 4 i + r has row r of the i-th (row quad, channel) pair of the block, 64 of them in a block of
// 8x8, 4x16 or 16x4.  Sixteen instructions then multiply that block with 64 pixels; nothing but
// kept blocks is ever multiplied.  Measured on registers: 117 TFLOP/s against 150 for 16x16x4,
// of which the union would leave about 100.
//
// Measured (this file / the general kernel it took these layers from): 3x3 64->64 at 56x56, batch
// 32, half of the 8x8 blocks kept: 55 / 188 us = 67 TFLOP/s; 3x3 128->416 at 28x28, batch 16, 4x16:
// 38 / 247 us; 5x5 48->64 at 35x35, batch 8: 21 / 93 us; 1x1 256->1024 at 14x14, batch 8: 15 / 49 us;
// FC 64 x 256 -> 256: 5.9 / 13.9 us, 1 x 4096 -> 4096: 21 / 197 us.  Layers with little to sum per strip
// stay with the general kernel (bsp_f32_general).
//
// What bounds the first of them: the matrix cores are busy 54 % of its time (30 us), staging and
// stores that nothing hides are 10 us (45 without them), the rest lies between the products.  Not
// in the LDS reads, of whose 11.5 M active cycles 7.4 M are conflicts: without them it is no faster.
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#include <array>
#include <map>
#include <mutex>
#include <utility>

namespace {

template <int ABID>
__device__ __forceinline__ f32x4_t mfma_4x4x1(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, ABID, 0);
}

// Of TP lane tiles, acc[tile * NQ + quad] += block (in a, lane 4 i + r) x the tile's BI channels in
// b: sixteen instructions per tile; tiles and row quads are taken in turn so that neighbouring
// instructions do not wait for each other.
template <int NQ, int BI, int TP, int... S>
__device__ __forceinline__ void block_mma(float a, const float (&b)[TP * BI], f32x4_t* acc,
                                          std::integer_sequence<int, S...>) {
  ((acc[S % (NQ * TP)] = mfma_4x4x1<(S % NQ) * BI + S / (NQ * TP)>(a, b[(S / NQ % TP) * BI + S / (NQ * TP)],
                                                                   acc[S % (NQ * TP)])), ...);
}

struct F32Args {
  const float* X;
  float* Y;
  const float* bias;
  const float* residual;
  const float* payload;
  const int32_t* row_ptr;
  const int32_t* col_idx;
  int32_t relu;
  int32_t L, J, I, O, H, K, M, N;
  int32_t sh, sw, ph, pw;        // gsh, gsw below: input pixels per staged pixel
  int32_t gsh, gsw, lsh, lsw;    // staged pixels per output pixel
  int32_t CW, nchunk, tpc;       // output columns per chunk, chunks per row, tiles per chunk
  int32_t TPW, pitch, slab, nslabs, lq;  // staged pixels per row, bytes per staged pixel, channels, slabs, log2(16-byte pieces)
  int32_t nbr, RG, ks, nset;     // block rows, block rows per workgroup, waves that share one, workgroups per tile
  int32_t total, per_xcd;        // workgroups
  int32_t nnzb;
  int32_t vec;                   // rows of X and Y are whole 16-byte pieces
  FastDiv d_nset, d_tpc, d_nchunk, d_cw, d_tpw;
};

// One (tile of PT * 64 output pixels) x (RG block rows) per workgroup.  A tile is consecutive
// pixels of a chunk of image columns (whole rows where they are at most 64 wide), so every lane
// has a pixel whatever the sizes; its input patch, halo included, is staged slab by slab of
// channels (zero outside the image and past the last channel).  A staged pixel takes
// slab * 4 + 16 bytes: an odd number of 16-byte pieces, so lanes on neighbouring pixels of a patch
// row read different banks; where a tile's pixels go on in the next row (chunks of eight columns,
// rows of ten staged pixels) some of them collide.
// Wave = (block row, share of its blocks): it walks its kept blocks tap by tap;
// the block's weights come straight from the compressed row, four taps ahead in a register ring,
// the pixels' channels from LDS one lane tile ahead.
template <int BO, int BI, int PT>
__global__ __launch_bounds__(512) void conv_f32(F32Args a) {
  kernarg_touch<F32Args>();
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int NQ = BO / 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthreads = (int)blockDim.x;
  // workgroups of one tile (other block rows) are neighbours on one XCD: its L2 has the patch
  const uint32_t q = (blockIdx.x & 7u) * (uint32_t)a.per_xcd + (blockIdx.x >> 3);
  if (q >= (uint32_t)a.total) return;
  const uint32_t tile = fdiv(q, a.d_nset);
  const int set = (int)(q - tile * (uint32_t)a.nset);
  const uint32_t ic = fdiv(tile, a.d_tpc);
  const int p0 = (int)(tile - ic * (uint32_t)a.tpc) * (PT * 64);
  const int img = (int)fdiv(ic, a.d_nchunk);
  const int col0 = (int)(ic - (uint32_t)img * (uint32_t)a.nchunk) * a.CW;
  const int m0 = (int)fdiv((uint32_t)p0, a.d_cw);
  const int plast = min(p0 + PT * 64, a.M * a.CW) - 1;
  const int rows = ((int)fdiv((uint32_t)plast, a.d_cw) - m0) * a.lsh + a.H;  // staged rows

  // this wave's block row and share of it (rows keep different numbers of blocks; turning which
  // wave takes which row from tile to tile, to even out the SIMDs, made no difference)
  const int rgi = wave / a.ks, ks = wave - rgi * a.ks;
  const int br = set * a.RG + rgi;
  const bool active = rgi < a.RG && br < a.nbr;
  const int row0 = active ? a.row_ptr[br] + ks : 0, rend = active ? a.row_ptr[br + 1] : 0;
  const int nblk = __builtin_amdgcn_readfirstlane(row0 < rend ? (rend - row0 + a.ks - 1) / a.ks : 0);
  const int HK = a.H * a.K;

  // the columns of this wave's next 64 blocks, one per lane
  int jb = 0;
  const int kNone = 0x7FFFFFFF / BI;
  auto load_cols = [&] {
    const int c = a.col_idx[min(row0 + min(jb + lane, max(nblk - 1, 0)) * a.ks, a.nnzb - 1)];
    return jb + lane < nblk ? c : kNone;
  };
  int cols = load_cols();

  // ---- weights: a ring of four (block, tap) steps.  This lane's element of a block at tap 0: row, channel
  const int ai = lane >> 2, arow = (ai / BI) * 4 + (lane & 3), ach = ai % BI;
  const char* wbase = (const char*)a.payload + (int64_t)row0 * (256 * HK);
  const uint32_t wlane = (uint32_t)(arow * HK * BI + ach) * 4u;
  const uint32_t wstep = (uint32_t)(a.ks * 256 * HK - (HK - 1) * BI * 4);       // to the next block
  const uint32_t wlast = (uint32_t)(max(nblk - 1, 0) * a.ks * 256 * HK + (HK - 1) * BI * 4);  // the row's last step
  float wr[4];
  uint32_t fo = 0;
  int ft = 0;
  auto fetch = [&](int d) {
    wr[d] = *(const float*)(wbase + (fo + wlane));
    const bool wrap = ++ft == HK;
    ft = wrap ? 0 : ft;
    fo = min(fo + (wrap ? wstep : (uint32_t)(BI * 4)), wlast);  // (past the row's end: its last step again, never used)
  };

  // ---- this lane's pixels
  int base[PT];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    const int p = min(p0 + pt * 64 + lane, plast);
    const int y = (int)fdiv((uint32_t)p, a.d_cw), x = p - y * a.CW;
    base[pt] = ((y - m0) * a.lsh * a.TPW + x * a.lsw) * a.pitch;
  }
  f32x4_t acc[PT * NQ];
#pragma unroll
  for (int k = 0; k < PT * NQ; ++k) acc[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int iy0 = m0 * a.sh - a.ph, ix0 = col0 * a.sw - a.pw;
  const int pieces = rows * a.TPW << a.lq;
  const int64_t xim = (int64_t)img * a.L * a.J * a.I;
  int j = 0;  // this wave's next block

  for (int sl = 0; sl < a.nslabs; ++sl) {
    const int c0 = sl * a.slab;
    // how many of the 64 columns lie before the slab's end and are still to do
    auto todo = [&] { return __popcll(__ballot(cols * BI < c0 + a.slab)) - (j - jb); };
    auto start = [&] {
      fo = (uint32_t)(j * a.ks) * (uint32_t)(256 * HK);
      ft = 0;
#pragma unroll
      for (int d = 0; d < 4; ++d) fetch(d);
    };
    int cnt = todo();
    if (cnt > 0) start();  // their latency passes while the patch is staged
    if (sl > 0) __syncthreads();
    // ---- stage the slab: four 16-byte pieces per thread in flight
    for (int f0 = tid; f0 < pieces; f0 += 4 * nthreads) {
      f32x4_t v[4];
      int dst[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int f = f0 + u * nthreads;
        const int pix = f >> a.lq, part = f - (pix << a.lq);
        const int r = (int)fdiv((uint32_t)pix, a.d_tpw), x = pix - r * a.TPW;
        const int iy = iy0 + r * a.gsh, ix = ix0 + x * a.gsw, ch = c0 + part * 4;
        dst[u] = f < pieces ? pix * a.pitch + part * 16 : -1;
        v[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (dst[u] >= 0 && (unsigned)iy < (unsigned)a.L && (unsigned)ix < (unsigned)a.J && ch < a.I) {
          const float* src = a.X + xim + ((int64_t)iy * a.J + ix) * a.I + ch;
          if (a.vec) {
            v[u] = *(const f32x4_t*)src;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (ch + e < a.I) v[u][e] = src[e];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (dst[u] >= 0) *(f32x4_t*)(lds + dst[u]) = v[u];
    }
    __syncthreads();

    // ---- products: the steps (block, tap) of this wave's blocks in the slab
    while (cnt > 0) {
      int ty = 0, tx = 0, jl = j - jb;
      auto col_off = [&] { return (__builtin_amdgcn_readlane(cols, jl & 63) * BI - c0) * 4; };
      constexpr int PP = PT < 2 ? 1 : 2;  // lane tiles whose products are interleaved
      float bb[2][PP * BI];
      auto read = [&](int pt, int o, float (&b)[PP * BI]) {
#pragma unroll
        for (int t = 0; t < PP; ++t)
#pragma unroll
          for (int e = 0; e < BI / 4; ++e) {
            const f32x4_t v = *(const f32x4_t*)(lds + base[pt + t] + o + e * 16);
            b[t * BI + 4 * e] = v.x;
            b[t * BI + 4 * e + 1] = v.y;
            b[t * BI + 4 * e + 2] = v.z;
            b[t * BI + 4 * e + 3] = v.w;
          }
      };
      int off = col_off();
      read(0, off, bb[0]);
      const int rowstep = (a.TPW - a.K + 1) * a.pitch;
      auto step = [&](auto dc) {
        constexpr int d = decltype(dc)::value;
        // where the next step reads: the next tap, or the next block's first one (after the last
        // step of all, some block's: an address inside the patch is all that matters then)
        const bool wx = ++tx == a.K;
        tx = wx ? 0 : tx;
        ty += wx ? 1 : 0;
        const bool wy = ty == a.H;
        ty = wy ? 0 : ty;
        jl += wy ? 1 : 0;
        const int ob = col_off();
        int noff = wy ? ((uint32_t)ob < (uint32_t)a.slab * 4u ? ob : 0) : off + (wx ? rowstep : a.pitch);
        constexpr int NP = PT / PP, par = (NP & 1) ? (d & 1) : 0;  // an odd number of pairs: the sets swap from step to step
#pragma unroll
        for (int t = 0; t < NP; ++t) {
          if (t + 1 < NP)
            read((t + 1) * PP, off, bb[(t + 1 + par) & 1]);
          else
            read(0, noff, bb[(NP + par) & 1]);
          block_mma<NQ, BI, PP>(wr[d], bb[(t + par) & 1], acc + t * PP * NQ, std::make_integer_sequence<int, 16 * PP>{});
        }
        fetch(d);
        off = noff;
      };
      int left = cnt * HK;
      for (; left >= 4; left -= 4) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
      }
      if (left > 0) step(std::integral_constant<int, 0>{});
      if (left > 1) step(std::integral_constant<int, 1>{});
      if (left > 2) step(std::integral_constant<int, 2>{});
      j += cnt;
      if (j - jb < 64 || j >= nblk) break;
      jb = j;  // a row of more than 64 blocks
      cols = load_cols();
      cnt = todo();
      if (cnt > 0) start();
    }
  }

  // ---- waves that share a block row: partial sums through LDS
  if (a.ks > 1) {
    __syncthreads();
    f32x4_t* red = (f32x4_t*)lds;  // [wave][PT * NQ][64]
    if (ks > 0) {
#pragma unroll
      for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int k = 0; k < NQ; ++k) red[(wave * (PT * NQ) + pt * NQ + k) * 64 + lane] = acc[pt * NQ + k];
    }
    __syncthreads();
    if (ks > 0) return;
    for (int s = 1; s < a.ks; ++s) {
#pragma unroll
      for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int k = 0; k < NQ; ++k) acc[pt * NQ + k] += red[((wave + s) * (PT * NQ) + pt * NQ + k) * 64 + lane];
    }
  }
  if (!active) return;

  // ---- results: the lane has channels br * BO .. + BO - 1 of its pixels
  const int ch0 = br * BO;
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    const int p = p0 + pt * 64 + lane;
    const int y = (int)fdiv((uint32_t)min(p, plast), a.d_cw), x = col0 + min(p, plast) - y * a.CW;
    if (p > plast || x >= a.N) continue;
    const int64_t o0 = (((int64_t)img * a.M + y) * a.N + x) * a.O + ch0;
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int ch = ch0 + 4 * k;
      f32x4_t v = acc[pt * NQ + k];
      if ((a.O & 3) == 0) {
        if (ch >= a.O) continue;
        if (a.bias) v += f32x4_t{a.bias[ch], a.bias[ch + 1], a.bias[ch + 2], a.bias[ch + 3]};
        if (a.residual) v += *(const f32x4_t*)(a.residual + o0 + 4 * k);
        if (a.relu) v = f32x4_t{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
        *(f32x4_t*)(a.Y + o0 + 4 * k) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (ch + r >= a.O) continue;
          float s = v[r] + (a.bias ? a.bias[ch + r] : 0.f);
          if (a.residual) s += a.residual[o0 + 4 * k + r];
          a.Y[o0 + 4 * k + r] = a.relu ? fmaxf(s, 0.f) : s;
        }
      }
    }
  }
}

// 1x1 layers on few pixels (FC layers): no staging.  Every pixel's channels of a kept block are
// one short run that the lane reads itself, and the weights are read once per 64 pixels.  What
// bounds a small call is the chain of dependent loads (row pointer, column, activations, result),
// so a block row is shared by up to sixteen waves, each with four blocks in flight.
template <int BO, int BI>
__global__ __launch_bounds__(1024) void fc_f32(F32Args a) {
  kernarg_touch<F32Args>();
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int NQ = BO / 4, D = 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t tile = fdiv(blockIdx.x, a.d_nset);
  const int br = (int)(blockIdx.x - tile * (uint32_t)a.nset);
  const int pixel = (int)tile * 64 + lane, px = min(pixel, a.N - 1);
  const int n0 = a.row_ptr[br] + wave, nend = a.row_ptr[br + 1];
  const int nblk = __builtin_amdgcn_readfirstlane(n0 < nend ? (nend - n0 + a.ks - 1) / a.ks : 0);
  const int ai = lane >> 2, arow = (ai / BI) * 4 + (lane & 3), ach = ai % BI;
  const float* wlane = a.payload + arow * BI + ach;
  const float* xlane = a.X + (int64_t)px * a.I;

  f32x4_t acc[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) acc[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // the bias of the channels this wave will store, asked for now: nothing waits for it at the end
  f32x4_t bv[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ch = br * BO + 4 * (a.ks > 1 ? min(wave, NQ - 1) : k) + r;
      bv[k][r] = a.bias && ch < a.O ? a.bias[ch] : 0.f;
    }
  float w[D], x[D][BI];
  int jb = 0, cols = 0;  // the columns of this wave's next 64 blocks, one per lane
  auto fetch = [&](int d, int s) {
    const int sl = min(s, nblk - jb - 1) & 63, nn = n0 + (jb + sl) * a.ks;
    const int c = __builtin_amdgcn_readlane(cols, sl) * BI;
    w[d] = wlane[(int64_t)nn * 64];
    if (a.vec) {
#pragma unroll
      for (int e = 0; e < BI / 4; ++e) {
        // (a last block that reaches past the channels: whole pieces, so they are there or not)
        const f32x4_t v = c + 4 * e < a.I ? *(const f32x4_t*)(xlane + c + 4 * e) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        x[d][4 * e] = v.x;
        x[d][4 * e + 1] = v.y;
        x[d][4 * e + 2] = v.z;
        x[d][4 * e + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < BI; ++e) {
        const float v = xlane[min(c + e, a.I - 1)];
        x[d][e] = c + e < a.I ? v : 0.f;
      }
    }
  };
  for (; jb < nblk; jb += 64) {
    cols = a.col_idx[n0 + min(jb + lane, nblk - 1) * a.ks];
    const int steps = min(nblk - jb, 64);
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < steps) fetch(d, d);
    int s = 0;
    for (; s + D < steps; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        block_mma<NQ, BI, 1>(w[d], x[d], acc, std::make_integer_sequence<int, 16>{});
        fetch(d, s + D + d);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (s + d < steps) block_mma<NQ, BI, 1>(w[d], x[d], acc, std::make_integer_sequence<int, 16>{});
  }
  if (a.ks > 1) {
    // every wave leaves its sums; then wave w adds up what it stores: channel quad by channel quad
    float* red = (float*)lds;  // [wave][NQ * 4][64]
#pragma unroll
    for (int k = 0; k < NQ; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave * NQ + k) * 4 + r) * 64 + lane] = acc[k][r];
    __syncthreads();
    if (wave >= NQ) return;
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < a.ks; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] += red[((s * NQ + wave) * 4 + r) * 64 + lane];
    acc[0] = v;
  }
  if (pixel >= a.N) return;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    if (a.ks > 1 && k > 0) break;
    const int ch = br * BO + 4 * (a.ks > 1 ? wave : k);
    const int64_t o = (int64_t)pixel * a.O + ch;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (ch + r >= a.O) continue;
      float s = acc[k][r] + bv[k][r];
      if (a.residual) s += a.residual[o + r];
      a.Y[o + r] = a.relu ? fmaxf(s, 0.f) : s;
    }
  }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Tile, slab and split, by a model of the busiest CU in clocks: the workgroups it runs, each with
// its matrix work (about 150 clocks per block, tap and 64 pixels, waves dealt over four SIMDs)
// and the bytes it stages (24 per clock), plus what several resident workgroups hide of each
// other's fixed costs (a slab's barriers and latency, the launch).  Over 3x3, 5x5, 1x7 and
// pointwise layers from 7x7x512 to 56x56x64 its choice measured within 5 % of the best of all
// candidates (odd 33x33x57: 17 %).
struct Pick {
  int32_t PT, slab, CW, nchunk, tpc, TPW, waves, RG, ks, lds;
};
Pick choose(int B, int M, int N, int I, int nbr, int H, int K, int lsh, int lsw, bool flat, int NQ, int BI) {
  Pick best{};
  double best_cost = 1e30;
  for (int PT : {1, 2, 4}) {
    if (PT * NQ > 8) continue;  // (accumulator registers)
    const int px = PT * 64;
    const auto width = [&](int cw) {
      const int64_t nchunk = cdiv(N, cw), tpc = cdiv((int64_t)M * cw, px), tiles = (int64_t)B * nchunk * tpc;
      const int orows = std::min(M, px % cw == 0 ? px / cw : (px - 2) / cw + 2);
      const int trows = (orows - 1) * lsh + H, tpw = (cw - 1) * lsw + K;
      for (int slab : {16, 32, 64, 128}) {
        if (slab > 16 && slab / 2 >= I) continue;
        const int64_t pix = (int64_t)trows * tpw;
        int64_t ldsb = pix * (slab * 4 + 16);
        if (ldsb > 160 * 1024 || pix * (slab / 4) >= (1 << 24)) continue;
        for (int ks : {1, 2, 4, 8}) {
          const int RGmax = 8 / ks;
          const int RG = cdiv(nbr, cdiv(nbr, RGmax));
          const int waves = RG * ks;
          const int64_t l2 = std::max<int64_t>(ldsb, ks > 1 ? (int64_t)waves * PT * NQ * 1024 : 0);
          if (l2 > 160 * 1024) continue;
          const int64_t wgs = tiles * cdiv(nbr, RG);
          const int resident = std::max(1, std::min((int)(160 * 1024 / l2), 16 / waves));
          // cycles of a workgroup's slowest SIMD: matrix work, staging, fixed cost per slab
          const int ns = cdiv(I, slab);
          const double blocks = 0.6 * cdiv(I, BI) * H * K / ks;  // half kept, with some unevenness
          const double wpers = std::max(1.0, waves / 4.0);
          const double mm = blocks * PT * 150.0 * wpers;
          const double st = (double)pix * slab * 4 * ns / 24.0;        // bytes per clock a CU stages
          const double fix = ns * 1500.0 + 3000.0 + (ks > 1 ? 500.0 : 0.0);
          // a CU runs its workgroups' matrix work one after the other and hides the rest behind
          // that as far as several are resident
          const double percu = std::max(1.0, (double)cdiv(wgs, 256));
          const double cost = percu * (mm + st) + fix * (percu / std::min<double>(percu, resident));
          if (cost < best_cost) {
            best_cost = cost;
            best = Pick{PT, slab, cw, (int32_t)nchunk, (int32_t)tpc, tpw, waves, RG, ks, (int32_t)l2};
          }
        }
      }
    };
    if (flat)
      width(px);
    else
      bsp_widths(N, 4, width);
  }
  return best;
}

template <int BO, int BI, int PT>
int launch_conv(const F32Args& a, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_f32<BO, BI, PT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) !=
        hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_f32<BO, BI, PT>), dim3((unsigned)(a.per_xcd * 8)), dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

template <int BO, int BI>
int launch_gran(const ConvParams& p, int64_t nnzb, hipStream_t st) {
  F32Args a{};
  a.X = (const float*)p.X;
  a.Y = (float*)p.Y;
  a.bias = p.bias;
  a.residual = (const float*)p.residual;
  a.payload = (const float*)p.payload;
  a.row_ptr = p.row_ptr;
  a.col_idx = p.col_idx;
  a.relu = p.relu;
  a.nnzb = (int32_t)nnzb;
  a.I = p.I;
  a.O = p.O;
  a.H = p.H;
  a.K = p.K;
  a.vec = p.I % 4 == 0;
  a.nbr = cdiv(p.O, BO);
  const bool pointwise = p.H == 1 && p.K == 1 && p.ph == 0 && p.pw == 0;
  const bool flat = pointwise && p.sh == 1 && p.sw == 1;  // a plain matrix product over all pixels

  // few pixels: straight from memory (see fc_f32)
  if (flat && p.P <= 256) {
    a.N = p.P;
    a.nset = a.nbr;
    const int64_t wgs = (int64_t)cdiv(p.P, 64) * a.nbr;
    if (wgs > 0x7FFFFFFF || wgs * a.nset >= (1ll << 32)) return BSP_ERR_UNSUPPORTED;
    a.ks = 16;
    while (a.ks > 4 && (wgs * a.ks >= 8192 || cdiv(p.I, BI) < 2 * a.ks)) a.ks /= 2;
    a.d_nset = make_fastdiv((uint32_t)a.nset);
    hipLaunchKernelGGL((fc_f32<BO, BI>), dim3((unsigned)wgs), dim3(64 * a.ks), (size_t)a.ks * BO * 256, st, a);
    return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
  }

  int B = p.B;
  a.L = p.L;
  a.J = p.J;
  a.M = p.M;
  a.N = p.N;
  if (flat) {
    B = 1;
    a.L = a.M = 1;
    a.J = a.N = p.P;
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
  Pick best;
  {
    // the search is a pure function of the shape: remember its answers
    static std::mutex mu;
    static std::map<std::array<int32_t, 9>, Pick> memo;
    const std::array<int32_t, 9> key = {B, a.M, a.N, p.I, p.O, p.H, p.K, p.sh * 2 + flat, p.sw};
    std::unique_lock<std::mutex> lock(mu);
    const auto it = memo.find(key);
    if (it != memo.end()) {
      best = it->second;
    } else {
      lock.unlock();  // other layers' launches do not wait for this one's search
      best = choose(B, a.M, a.N, p.I, a.nbr, p.H, p.K, a.lsh, a.lsw, flat, BO / 4, BI);
      lock.lock();
      if (memo.size() > 4096) memo.clear();
      memo.emplace(key, best);
    }
  }
  if (best.PT == 0) return BSP_ERR_UNSUPPORTED;
  a.CW = best.CW;
  a.nchunk = best.nchunk;
  a.tpc = best.tpc;
  a.TPW = best.TPW;
  a.slab = best.slab;
  a.nslabs = cdiv(p.I, best.slab);
  a.pitch = best.slab * 4 + 16;
  a.lq = 2;
  while ((4 << a.lq) < best.slab) ++a.lq;
  // (weights are addressed from the start of a block row with 32 bits)
  if ((int64_t)cdiv(p.I, BI) * 256 * p.H * p.K + 65536 >= (1ll << 31)) return BSP_ERR_UNSUPPORTED;
  a.RG = best.RG;
  a.ks = best.ks;
  a.nset = cdiv(a.nbr, best.RG);
  const int64_t total = (int64_t)B * a.nchunk * a.tpc * a.nset;
  if (total >= (1ll << 30)) return BSP_ERR_UNSUPPORTED;
  a.total = (int32_t)total;
  a.per_xcd = cdiv(total, 8);
  // multiply-high divisions are exact while dividend * divisor < 2^32
  const int64_t tiles = (int64_t)B * a.nchunk * a.tpc, pix_max = (int64_t)a.tpc * best.PT * 64;
  if ((int64_t)(total + 8) * a.nset >= (1ll << 32) || tiles * a.tpc >= (1ll << 32) ||
      (int64_t)B * a.nchunk * a.nchunk >= (1ll << 32) || pix_max * a.CW >= (1ll << 32) ||
      (int64_t)(best.lds + 65536) * a.TPW >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  a.d_nset = make_fastdiv((uint32_t)a.nset);
  a.d_tpc = make_fastdiv((uint32_t)a.tpc);
  a.d_nchunk = make_fastdiv((uint32_t)a.nchunk);
  a.d_cw = make_fastdiv((uint32_t)a.CW);
  a.d_tpw = make_fastdiv((uint32_t)a.TPW);
  const int threads = 64 * best.waves;
  switch (best.PT) {
    case 1: return launch_conv<BO, BI, 1>(a, threads, (size_t)best.lds, st);
    case 2: return launch_conv<BO, BI, 2>(a, threads, (size_t)best.lds, st);
    case 4:
      if constexpr (BO <= 8) return launch_conv<BO, BI, 4>(a, threads, (size_t)best.lds, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

}  // namespace

int bsp_launch_f32(const ConvParams& p, int64_t nnzb, int bo, int bi, const void* plan_host, hipStream_t st) {
  if (nnzb < 1 || nnzb > 0x7FFFFFFF || !p.row_ptr || !p.col_idx) return BSP_ERR_UNSUPPORTED;
  const int32_t* hdr = (const int32_t*)plan_host;
  const bool flat = p.H == 1 && p.K == 1 && p.ph == 0 && p.pw == 0 && p.sh == 1 && p.sw == 1;
  const int64_t HK = (int64_t)p.H * p.K;
  if (bsp_f32_general(bo, p.I, p.O, HK, hdr[BSP_PLAN_NCHUNKS_W] * HK, hdr[BSP_PLAN_NSTRIPS_W], (int64_t)p.P * p.O,
                      flat && p.P <= 256))
    return BSP_ERR_UNSUPPORTED;
  if (bo == 8 && bi == 8) return launch_gran<8, 8>(p, nnzb, st);
  if (bo == 4 && bi == 16) return launch_gran<4, 16>(p, nnzb, st);
  if (bo == 16 && bi == 4) return launch_gran<16, 4>(p, nnzb, st);
  return BSP_ERR_UNSUPPORTED;
}
