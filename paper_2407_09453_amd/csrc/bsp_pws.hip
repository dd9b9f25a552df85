// Pointwise (1x1) layers on many pixels: the pointwise kernel's steps (bsp_pw.hip) with the weights held in
// registers and the pixels streamed past them, bf16 or int8.
//
// Work split.  A workgroup of NW waves owns NS strips of 16 output channels and every so many-th tile of 16 * PT
// output pixels in its XCD's eighth of them.  A wave reads the weight fragments of its SW strips (wave, wave + NW)
// once, at most D steps each, and keeps them.  Per tile: the last tile's results leave, the input (QL loads of 16 bytes a
// lane, into registers) and residual of tiles to come are asked for; this tile's products from LDS, results into an
// LDS image of the output; the next tile's input to the other LDS buffer; one barrier.  Both buffers and both images
// are used in turn.  Steps, fragments and their order are the pointwise kernel's, so the results are the same bits.
//
// What bounds it: memory, at the rate of a copy of the same mix (64->256 at 56x56 batch 32 66 MB in 11.7 us; data cold, pointwise / here: 64->256 with a residual at
// 56x56 batch 32, 116 MB, 26.0 / 24.2 us; without 20.1 / 18.0; 256->128 there, 77 MB, 25.7 / 18.0), then LDS where strips
// are long (512->256 at 28x28 21.0 / 16.1: a fragment read from LDS feeds one product), and the results' arithmetic in
// int8 (64->256 13.4 / 9.2).  The pointwise kernel gives every tile a workgroup of its own, which walks launch, step
// ranges, weights, copy, products and results one after the other, two to seven times per CU; here the opening is
// paid once and every wait has another tile's work beside it.  Strips of up to four steps leave registers to ask for
// two tiles ahead, which is what a residual needs (64->256 27.1 with one, 24.2 with two); longer ones ask for one (256->64
// 15.0, two 15.5).  Streaming stores also where a line is shared by two workgroups (ordinary ones 1.2 times).
//
// Straight code: a wave runs U steps of every strip without a branch, steps that a strip does not have multiply no
// weights with a piece of zeros that lies behind every staged pixel (with the tile's own data there an infinity
// would reach channels that drop it).  With a branch per step and strip 64->256 took 14.4 us instead of 11.7, the
// int8 layer 11.9 instead of 9.2 (data warm).
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#ifdef BSP_ROWS_TUNE
#include <cstdio>
#include <cstdlib>
#endif
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

struct PwsArgs {
  const unsigned char* X;
  unsigned char* Y;
  const void* bias;
  const unsigned char* residual;
  const int32_t* rstrip;
  const int32_t* rslab;
  const unsigned char* rdesc;
  const unsigned char* rfrag;
  int32_t relu, nstrips, ncs;        // relu: int8 layers keep their rounding right shift here
  int32_t P, O;
  int32_t S, L, J, N, MN;            // S > 1: output pixel (img, y, x) reads input pixel (img, y*S, x*S)
  int32_t cpx, pitch;                // 16-byte pieces of a pixel; LDS bytes of a staged one
  int32_t NS, tiles, nsplit, per_xcd, groups;  // strips per workgroup; tiles of pixels, of an XCD; workgroups of an XCD that share them
  int32_t slot, out_off, oslot, opitch, bias_off, pair;
  FastDiv d_mn, d_n, d_cpx, d_nsplit, d_cpp;
};

// Four int8 results from four sums that hold their bias, half a unit and 128 units: shifted, saturated to 16 bits in
// pairs, then to bytes without a sign, from which 128 are taken again.  Ten instructions.
__device__ __forceinline__ uint32_t bytes_of(i32x4_t v, int shift) {
  const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_i16(v[0] >> shift, v[1] >> shift));
  const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_i16(v[2] >> shift, v[3] >> shift));
  uint32_t l8, h8;
  asm("v_sat_pk_u8_i16 %0, %1" : "=v"(l8) : "v"(lo));
  asm("v_sat_pk_u8_i16 %0, %1" : "=v"(h8) : "v"(hi));
  return (l8 | h8 << 16) ^ 0x80808080u;
}

// KIND: 8 or 4, the channels per unit of a bf16 layer; 16, an int8 layer.  RES: there is a residual.
template <int KIND, int PT, int SW, int D, int QL, bool RES>
__global__ __launch_bounds__(1024) void conv_pws(PwsArgs a) {
  constexpr int MT = 16 * PT;  // pixels of a tile
  constexpr bool CW4 = KIND == 4, I8 = KIND == 16;
  // Strips of many 4-channel units: the places of two steps a word, in units (one byte each), or 16x4 layers of 13 to 16 steps
  // with a residual spill (512->64 on 65536 pixels 27.8 us instead of 22.8, the pointwise kernel 26.6).
  constexpr bool BYTES = CW4 && D == 16 && QL == 2;
  constexpr int eb = I8 ? 1 : 2;
  kernarg_touch<PwsArgs>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = (int)blockDim.x, nwaves = nthr >> 6;
  // an XCD takes an eighth of the tiles, one after the other ; its consecutive workgroups share their pixels (the second reader hits that L2)
  const int xcd = blockIdx.x & 7, slot_wg = blockIdx.x >> 3;
  const int grp = (int)fdiv((uint32_t)slot_wg, a.d_nsplit), ns = slot_wg - grp * a.nsplit;
  const int first = xcd * a.per_xcd + grp, end = min(a.tiles, (xcd + 1) * a.per_xcd);
  if (first >= end) return;
  const int range0 = ns * a.NS * 16;  // the workgroup's strips cover the channels from here on

  // ---- the pieces of input this lane brings for every tile: pixel, bytes in it, place in a buffer.  Where registers held
  // for four of them would spill, a word each of pixel and place in pieces, decoded anew for every tile (1008->128 on 57344
  // pixels 16.2 us, spilled 16.9; where nothing spills the decoding costs up to 9 %).
  constexpr bool WORDS = I8 && QL == 4 && (D == 8 || SW == 2);
  uint32_t lpj[QL], pcj[WORDS ? 1 : QL], ldj[WORDS ? 1 : QL];
#pragma unroll
  for (int j = 0; j < QL; ++j) {
    const uint32_t idx = (uint32_t)(tid + j * nthr);
    const uint32_t lp = fdiv(idx, a.d_cpx), piece = idx - lp * (uint32_t)a.cpx;
    if constexpr (WORDS) {
      lpj[j] = lp << 16 | (lp * ((uint32_t)a.pitch >> 4) + piece);
    } else {
      lpj[j] = lp;
      pcj[j] = piece * 16u;
      ldj[j] = lp * (uint32_t)a.pitch + pcj[j];
    }
  }
  constexpr int AHEAD = D <= 4 ? 2 : 1;  // tiles asked for before their turn
  u32x4_t xr[AHEAD][QL];
  auto load_x = [&](u32x4_t (&x)[QL], int tile) {
#pragma unroll
    for (int j = 0; j < QL; ++j) {
      uint32_t lp = lpj[j];
      if constexpr (WORDS) {
        asm volatile("" : "+v"(lp));
        lp >>= 16;
      }
      // past the last pixel: that one again (a valid address, never used)
      const uint32_t p = min((uint32_t)tile * (uint32_t)MT + lp, (uint32_t)(a.P - 1));
      uint32_t ip = p;
      if (a.S > 1) {
        const uint32_t img = fdiv(p, a.d_mn), r2 = p - img * (uint32_t)a.MN;
        const uint32_t oy = fdiv(r2, a.d_n), ox = r2 - oy * (uint32_t)a.N;
        ip = (img * (uint32_t)a.L + oy * (uint32_t)a.S) * (uint32_t)a.J + ox * (uint32_t)a.S;
      }
      asm volatile("" : "+v"(ip));  // one load after the branch, not one in either: the waits count them
      uint32_t at;
      if constexpr (WORDS)
        at = (lpj[j] & 0xFFFFu) * 16u - (uint32_t)__mul24((int)lp, a.pitch);
      else
        at = pcj[j];
      x[j] = *(const u32x4_t*)(a.X + (ip * (uint32_t)a.cpx * 16u + at));
    }
  };
  auto write_x = [&](const u32x4_t (&x)[QL], uint32_t off) {
#pragma unroll
    for (int j = 0; j < QL; ++j) {
      if constexpr (WORDS) {
        uint32_t v = lpj[j];
        asm volatile("" : "+v"(v));
        if (v < (uint32_t)MT << 16) *(u32x4_t*)(lds + off + (v & 0xFFFFu) * 16u) = x[j];
      } else {
        if (lpj[j] < (uint32_t)MT) *(u32x4_t*)(lds + off + ldj[j]) = x[j];
      }
    }
  };
  load_x(xr[0], first);
  if constexpr (AHEAD == 2) load_x(xr[AHEAD - 1], first + a.groups);

  // ---- this wave's strips: weights, where a step's fragments lie in a lane's pixel of the tile (two 16-bit numbers
  // a word; CW4: both halves of a step), where this lane's results go in an image of the output, biases.  A strip's
  // missing steps multiply no weights with the zeros behind each staged pixel; missing channels go to the pad
  // behind each pixel of an image.
  using acc_t = typename std::conditional<I8, i32x4_t, f32x4_t>::type;
  u32x4_t w[SW][D];
  uint32_t un[SW][CW4 && !BYTES ? D : (D + 1) / 2];
  uint32_t img[SW], bch[SW];
  int nst[SW];
  i32x4_t cin[I8 ? SW : 1];
  const uint32_t none = (uint32_t)a.cpx * 16u;
  const bool odd = PT == 2 && !I8 && a.pair && (g & 1);
  bool wide = a.relu > 22;
#pragma unroll
  for (int s = 0; s < SW; ++s) {
    const int sidx = s * nwaves + wave, strip = ns * a.NS + sidx;
    const bool active = sidx < a.NS && strip < a.nstrips;
    const int sq = active ? strip : 0;
    const int lo = a.rslab[sq * 2], n = active ? a.rslab[sq * 2 + 1] - lo : 0;
    const int ch = a.rstrip[sq * 4 + g];
    const bool some = active && ch >= 0;
    nst[s] = n;
    img[s] = (uint32_t)(a.out_off + (c + (odd ? 16 : 0)) * a.opitch + (some ? (ch - range0 - (odd ? 4 : 0)) * eb : a.NS * 16 * eb));
    bch[s] = (uint32_t)(a.bias_off + (some ? ch - range0 : 0) * 4);
    if constexpr (I8) {
      i32x4_t b = {0, 0, 0, 0};
      const int32_t* bp = (const int32_t*)a.bias;
      if (bp && some) b = i32x4_t{bp[ch], bp[ch + 1], bp[ch + 2], bp[ch + 3]};
#pragma unroll
      for (int r = 0; r < 4; ++r) wide |= b[r] > (1 << 30) || b[r] < -(1 << 30);
      cin[s] = b;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const uint32_t cs = (uint32_t)min(lo + d, a.ncs - 1);
      w[s][d] = *(const u32x4_t*)(a.rfrag + (cs * 1024u + (uint32_t)lane * 16u));
      const uint32_t dv = *(const uint32_t*)(a.rdesc + (cs * 16u + (uint32_t)g * 4u));
      if (d >= n) w[s][d] = u32x4_t{0, 0, 0, 0};
      const uint32_t u0 = d < n ? (dv & 0xFFu) * (CW4 ? 8u : 16u) : none, u1 = d < n ? ((dv >> 16) & 0xFFu) * 8u : none;
      if constexpr (BYTES)
        un[s][d / 2] = (d & 1 ? un[s][d / 2] : 0u) | ((dv & 0xFFu) | (dv >> 16 & 0xFFu) << 8) << (d & 1 ? 16 : 0);
      else if constexpr (CW4)
        un[s][d] = u0 | u1 << 16;
      else if (d & 1)
        un[s][d / 2] |= u0 << 16;
      else
        un[s][d / 2] = u0;
    }
  }
  if constexpr (I8) {
    // the sums start from the bias, half a unit and 128 units; where one could then leave 32 bits, from nothing
    wide = __ballot(wide) != 0;
    const int plus = wide ? 0 : (a.relu ? 1 << (a.relu - 1) : 0) + (128 << a.relu);
#pragma unroll
    for (int s = 0; s < SW; ++s) cin[s] = wide ? i32x4_t{0, 0, 0, 0} : cin[s] + plus;
  } else {
    for (int i = tid; i < a.NS * 16; i += nthr)
      *(float*)(lds + a.bias_off + i * 4) = a.bias && range0 + i < a.O ? ((const float*)a.bias)[range0 + i] : 0.f;
  }
  // the zeros behind the pixels of both buffers
  for (int i = tid; i < 2 * MT; i += nthr) *(u32x4_t*)(lds + (uint32_t)i * (uint32_t)a.pitch + none) = u32x4_t{0, 0, 0, 0};

  // ---- the 16-byte pieces of output this lane stores for every tile
  constexpr int NIT = (PT * SW + (I8 ? 3 : 1)) / (I8 ? 4 : 2);  // MT * NS * 32 (16) bytes over 64 * NW lanes, NS <= NW * SW
  const int cpp = a.NS * (I8 ? 1 : 2);         // pieces per pixel
  int opix[NIT];  // the pixel of the tile, or none
  uint32_t lsrc[NIT], gofs[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = tid + it * nthr;
    const int pixel = (int)fdiv((uint32_t)i, a.d_cpp), k = i - pixel * cpp;
    opix[it] = pixel < MT && range0 + k * (16 / eb) < a.O ? pixel : (1 << 30);
    lsrc[it] = (uint32_t)(a.out_off + pixel * a.opitch + k * 16);
    gofs[it] = (uint32_t)(pixel * a.O) * (uint32_t)eb + (uint32_t)k * 16u;
  }
  const uint32_t obytes = (uint32_t)a.O * (uint32_t)(eb * MT);  // of a tile
  u32x4_t res[AHEAD][NIT];
  auto load_res = [&](u32x4_t (&r)[NIT], int next) {
    const int tile = min(next, a.tiles - 1);  // past the last tile: that one again (valid addresses, never used)
    const unsigned char* from = a.residual + ((uint32_t)tile * obytes + (uint32_t)range0 * 2u);
    const int left = a.P - tile * MT;
#pragma unroll
    for (int it = 0; it < NIT; ++it)  // (what is not stored reads the tile's first piece)
      r[it] = *(const u32x4_t*)(from + (opix[it] < left ? gofs[it] : 0u));
  };
  auto store = [&](const u32x4_t (&r)[NIT], int tile, uint32_t ooff) {
    unsigned char* to = a.Y + ((uint32_t)tile * obytes + (uint32_t)(range0 * eb));
    const int left = a.P - tile * MT;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (opix[it] >= left) continue;
      u32x4_t v = *(const u32x4_t*)(lds + ooff + lsrc[it]);
      if constexpr (RES) {
        const u32x2_t l2 = post_bf16x4_reg(u32x2_t{v.x, v.y}, u32x2_t{r[it].x, r[it].y}, true, a.relu);
        const u32x2_t h2 = post_bf16x4_reg(u32x2_t{v.z, v.w}, u32x2_t{r[it].z, r[it].w}, true, a.relu);
        v = u32x4_t{l2.x, l2.y, h2.x, h2.y};
      }
      __builtin_nontemporal_store(v, (u32x4_t*)(to + gofs[it]));
    }
  };

  const uint32_t base = (uint32_t)c * (uint32_t)a.pitch, tstep = 16u * (uint32_t)a.pitch;
  auto compute = [&](uint32_t xoff, uint32_t ooff, auto slow) {
    const uint32_t b0 = xoff + base, b1 = b0 + tstep;
    constexpr int U = D < 4 ? D : D / 2 + 1;  // steps that every strip takes, there or not; beyond them, the strip's own
    u32x4_t f[2][PT];
    auto read = [&](int s, int d) {
      u32x4_t (&fr)[PT] = f[(s * D + d) & 1];
      // decoded anew for every tile: kept across them, the steps' addresses would take the registers of the weights
      uint32_t& u = un[s][CW4 && !BYTES ? d : d / 2];
      asm volatile("" : "+v"(u));
      if constexpr (CW4) {
        uint32_t o0 = u & 0xFFFFu, o1 = u >> 16;
        if constexpr (BYTES) {
          const uint32_t v = d & 1 ? u >> 16 : u;
          o0 = (v & 0xFFu) * 8u;
          o1 = (v >> 8 & 0xFFu) * 8u;
          if (d < U && d >= nst[s]) o0 = o1 = none;
        }
#pragma unroll
        for (int t = 0; t < PT; ++t) {
          const u32x2_t x0 = *(const u32x2_t*)(lds + (t ? b1 : b0) + o0);
          const u32x2_t x1 = *(const u32x2_t*)(lds + (t ? b1 : b0) + o1);
          fr[t] = u32x4_t{x0.x, x0.y, x1.x, x1.y};
        }
      } else {
        const uint32_t o = d & 1 ? u >> 16 : u & 0xFFFFu;
#pragma unroll
        for (int t = 0; t < PT; ++t) fr[t] = *(const u32x4_t*)(lds + (t ? b1 : b0) + o);
      }
    };
    // a step's fragments are read while the step before it is in the matrix cores
    read(0, 0);
#pragma unroll
    for (int s = 0; s < SW; ++s) {
      acc_t acc[PT], bv = {0, 0, 0, 0};
      if constexpr (!I8) bv = *(const f32x4_t*)(lds + bch[s]);
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        if constexpr (I8)
          acc[t] = cin[s];
        else
          acc[t] = acc_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (d + 1 < D) {
          if (d + 1 < U || d + 1 < nst[s]) read(s, d + 1);
        } else if (s + 1 < SW) {
          read(s + 1, 0);
        }
        if (d >= U && d >= nst[s]) continue;
#pragma unroll
        for (int t = 0; t < PT; ++t) {
          const u32x4_t x = f[(s * D + d) & 1][t];
          if constexpr (I8)
            acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4_t, w[s][d]), __builtin_bit_cast(i32x4_t, x), acc[t], 0, 0, 0);
          else
            acc[t] = mfma_bf16_16x16x32(w[s][d], x, acc[t]);
        }
      }
      // bias, one rounding, into the image of the output lines
      unsigned char* ot = lds + ooff + img[s];
      if constexpr (I8) {
        uint32_t v[PT];
        if constexpr (decltype(slow)::value) {
          i32x4_t b = {0, 0, 0, 0};
          const int sidx = s * nwaves + wave, strip = ns * a.NS + sidx;
          if (a.bias && sidx < a.NS && strip < a.nstrips) {
            const int ch = a.rstrip[strip * 4 + g];
            const int32_t* bp = (const int32_t*)a.bias;
            if (ch >= 0) b = i32x4_t{bp[ch], bp[ch + 1], bp[ch + 2], bp[ch + 3]};
          }
          const RescaleI8 rescale(b, a.relu);
#pragma unroll
          for (int t = 0; t < PT; ++t) v[t] = rescale(acc[t]);
        } else {
#pragma unroll
          for (int t = 0; t < PT; ++t) v[t] = bytes_of(acc[t], a.relu);
        }
#pragma unroll
        for (int t = 0; t < PT; ++t) *(uint32_t*)(ot + t * 16 * a.opitch) = v[t];
      } else {
#pragma unroll
        for (int t = 0; t < PT; ++t) {
          acc[t] += bv;
          // (a rounding does not move a sum past zero: without a residual the activation may come first)
          if (!RES && a.relu) acc[t] = f32x4_t{fmaxf(acc[t].x, 0.f), fmaxf(acc[t].y, 0.f), fmaxf(acc[t].z, 0.f), fmaxf(acc[t].w, 0.f)};
        }
        if (PT == 2 && a.pair) {
          const uint32_t x0 = pack_bf16x2(acc[0].x, acc[0].y), y0 = pack_bf16x2(acc[0].z, acc[0].w);
          const uint32_t x1 = pack_bf16x2(acc[PT - 1].x, acc[PT - 1].y), y1 = pack_bf16x2(acc[PT - 1].z, acc[PT - 1].w);
          // lane rows 0/1 (and 2/3) hold the two halves of one 8-channel block row: after an exchange an
          // even row has all eight channels of the first lane tile, an odd row those of the second
          const auto sx = __builtin_amdgcn_permlane16_swap(x0, x1, false, false);
          const auto sy = __builtin_amdgcn_permlane16_swap(y0, y1, false, false);
          *(u32x4_t*)ot = u32x4_t{sx[0], sy[0], sx[1], sy[1]};
        } else {
#pragma unroll
          for (int t = 0; t < PT; ++t)
            *(u32x2_t*)(ot + t * 16 * a.opitch) = u32x2_t{pack_bf16x2(acc[t].x, acc[t].y), pack_bf16x2(acc[t].z, acc[t].w)};
        }
      }
    }
  };

  if constexpr (RES && AHEAD == 2) load_res(res[0], first);
  write_x(xr[0], 0);
  __syncthreads();
  int tile = first;
  auto step = [&](auto odd_tile) -> bool {
    constexpr uint32_t cur = decltype(odd_tile)::value, oth = cur ^ 1u;
    constexpr uint32_t mine = AHEAD == 2 ? cur : 0, other = AHEAD == 2 ? oth : 0;
    if (tile != first) store(res[other], tile - a.groups, oth * (uint32_t)a.oslot);
    load_x(xr[mine], tile + AHEAD * a.groups);
    if constexpr (RES) load_res(res[other], tile + (AHEAD - 1) * a.groups);
    if (I8 && wide)
      compute(cur * (uint32_t)a.slot, cur * (uint32_t)a.oslot, std::true_type{});
    else
      compute(cur * (uint32_t)a.slot, cur * (uint32_t)a.oslot, std::false_type{});
    write_x(xr[other], oth * (uint32_t)a.slot);
    __syncthreads();
    tile += a.groups;
    return tile < end;
  };
  for (;;) {
    if (!step(std::integral_constant<uint32_t, 0>{})) {
      store(res[0], tile - a.groups, 0);
      return;
    }
    if (!step(std::integral_constant<uint32_t, 1>{})) {
      store(res[AHEAD - 1], tile - a.groups, (uint32_t)a.oslot);
      return;
    }
  }
}

constexpr int kLdsLimit = 160 * 1024;

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

template <int KIND, int PT, int SW, int D, int QL, bool RES>
int launch_inst(const PwsArgs& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_pws<KIND, PT, SW, D, QL, RES>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_pws<KIND, PT, SW, D, QL, RES>), grid, dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

template <int KIND, int PT, int SW, int D, int QL>
int launch_res(const PwsArgs& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  if constexpr (KIND != 16)
    if (a.residual) return launch_inst<KIND, PT, SW, D, QL, true>(a, grid, threads, ldsb, st);
  return launch_inst<KIND, PT, SW, D, QL, false>(a, grid, threads, ldsb, st);
}

template <int KIND, int PT, int SW, int D>
int launch_q(const PwsArgs& a, int QL, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  switch (QL) {
    case 1: return launch_res<KIND, PT, SW, D, 1>(a, grid, threads, ldsb, st);
    case 2: return launch_res<KIND, PT, SW, D, 2>(a, grid, threads, ldsb, st);
    case 4:  // (long strips leave no registers for it)
      if constexpr (D <= 8) return launch_res<KIND, PT, SW, D, 4>(a, grid, threads, ldsb, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

template <int KIND>
int launch_k(const PwsArgs& a, int PT, int SW, int D, int QL, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  switch (PT * 1000 + SW * 100 + D) {
    case 2102: return launch_q<KIND, 2, 1, 2>(a, QL, grid, threads, ldsb, st);
    case 2104: return launch_q<KIND, 2, 1, 4>(a, QL, grid, threads, ldsb, st);
    case 2106: return launch_q<KIND, 2, 1, 6>(a, QL, grid, threads, ldsb, st);
    case 2108: return launch_q<KIND, 2, 1, 8>(a, QL, grid, threads, ldsb, st);
  }
  if constexpr (KIND == 16) {
    if (PT == 2 && SW == 2 && D == 1) return launch_q<KIND, 2, 2, 1>(a, QL, grid, threads, ldsb, st);
  } else {
    if (PT == 1 && SW == 1 && D == 12) return launch_q<KIND, 1, 1, 12>(a, QL, grid, threads, ldsb, st);
    if (PT == 1 && SW == 1 && D == 16) return launch_q<KIND, 1, 1, 16>(a, QL, grid, threads, ldsb, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

int launch_pws(const ConvParams& p, int dtype, const void* plan_host, int shift, hipStream_t st) {
  const bool i8 = dtype == BSP_I8;
  if (!plan_host) return BSP_ERR_UNSUPPORTED;
  const int32_t* hdr = (const int32_t*)plan_host;
  if (hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION || hdr[BSP_PLAN_O_W] != p.O ||
      hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H || hdr[BSP_PLAN_K_W] != p.K || hdr[BSP_PLAN_DTYPE_W] != dtype ||
      hdr[BSP_PLAN_OFF_ROWS_W] == 0)
    return BSP_ERR_UNSUPPORTED;
  const int32_t* rs = hdr + hdr[BSP_PLAN_OFF_ROWS_W];
  if (p.H != 1 || p.K != 1 || p.ph != 0 || p.pw != 0 || p.sh != p.sw || p.sh < 1) return BSP_ERR_UNSUPPORTED;
  if (rs[BSP_ROWS_NSLABS_W] != 1 || rs[BSP_ROWS_WINDOW_W] != 4 || rs[BSP_ROWS_NCS_W] < 1 || p.P <= 64) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.B * p.L * p.J * p.I * 2 >= (1ll << 31) || (int64_t)p.P * p.O * 2 >= (1ll << 31)) return BSP_ERR_UNSUPPORTED;
  const int eb = i8 ? 1 : 2, raw = p.I * eb, nstrips = rs[BSP_ROWS_NSTRIPS_W], steps = rs[BSP_ROWS_MAXSTRIPSTEPS_W];
  const int cw = rs[BSP_ROWS_CW_W];
  if (raw % 16 || steps > 16) return BSP_ERR_UNSUPPORTED;
  PwsArgs a{};
  a.cpx = raw / 16;
  a.pitch = (a.cpx + (a.cpx & 1 ? 2 : 1)) * 16;  // room for a piece of zeros, and an odd number of pieces: no two pixels of a lane tile share banks
  // Waves and strips of a workgroup (8900 random layers, their data cold, each on eight combinations).  One strip a
  // wave; two pay only where a strip is over after one step of int8 codes and its results are the work (5 to 7 %).
  // Workgroups of eight waves, of sixteen where strips are long (a tile staged once for twice the strips: 5 %), of four
  // where eight would leave strips over (18 strips, eight at a time, cost as 24 do), which costs 15 to 30 %, more in
  // int8, where results then are half lines.  16 waves a CU: the tiles asked for ahead do what more waves did (24: 2 to
  // 25 % slower).  Where the waves so chosen cannot bring a tile in four loads a lane (17 to 20 strips of up to four steps and
  // more than 256 channels, more than 512 channels past eight strips of up to eight steps) the layer stays with the pointwise
  // kernel: on eight or sixteen waves the former take 0.89 to 1.6 times as long there as here, the latter 1.0 to 1.7.
  int PT = steps <= 8 ? 2 : 1, SW = i8 && steps <= 1 && nstrips > 4 ? 2 : 1, NW = 8;
  if (nstrips <= 8) {
    if (SW == 2) NW = 4;  // (four strips of two steps: not taken, see bsp_pws_beats)
  } else {
    double best = 1e9;
    for (int nw = SW == 2 ? 4 : 8; nw; nw = SW == 2 ? (nw == 4 ? 8 : 0) : nw == 8 ? 16 : nw == 16 ? 4 : 0) {
      const int ns = std::min(nstrips, nw * SW);
      double c = (double)(cdiv(nstrips, ns) * ns) / nstrips;
      if (SW == 1) c *= nw == 4 ? (i8 ? 1.35 : steps <= 4 ? 1.15 : 1.30) : (nw == 8) == (steps <= 8) ? 1.0 : 1.04;
      if (c < best) best = c, NW = nw;
    }
  }
  int NS = std::min(nstrips, NW * SW);
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  int tuned = 0;
  if (const char* e = std::getenv("BSP_PWS_TUNE")) {
    int q[5];
    if (std::atoi(e) == 0) return BSP_ERR_UNSUPPORTED;
    if (sscanf(e, "%d,%d,%d,%d,%d", q, q + 1, q + 2, q + 3, q + 4) == 5) NW = q[0], SW = q[1], NS = std::min(q[2], nstrips), tuned = q[3], PT = q[4];
  }
#endif
  if (NS < nstrips) NS &= ~3;  // whole windows of output channels
  if (NS < 1 || NW < 1 || NW > 16 || NS > NW * SW) return BSP_ERR_UNSUPPORTED;
  const int D = SW == 2 ? 1 : steps <= 2 ? 2 : steps <= 4 ? 4 : steps <= 6 ? 6 : steps <= 8 ? 8 : steps <= 12 ? 12 : 16;
  if (D < steps) return BSP_ERR_UNSUPPORTED;
  const int threads = 64 * NW, MT = 16 * PT;
  int QL = cdiv((int64_t)MT * a.cpx, threads);
  QL = QL == 3 ? 4 : QL;
  if (QL > 4) return BSP_ERR_UNSUPPORTED;
  a.slot = MT * a.pitch;
  a.opitch = NS * 16 * eb + 16;
  a.out_off = 2 * a.slot;
  a.oslot = MT * a.opitch;
  a.bias_off = a.out_off + 2 * a.oslot;
  const int64_t ldsb = a.bias_off + (int64_t)NS * 64;
  if (ldsb > kLdsLimit) return BSP_ERR_UNSUPPORTED;
  int wgs = bsp_pws_held(NW, ldsb);
#ifdef BSP_ROWS_TUNE
  if (tuned) wgs = tuned;
#endif
  a.NS = NS;
  a.nsplit = cdiv(nstrips, NS);
  a.tiles = cdiv(p.P, MT);
  a.per_xcd = cdiv(a.tiles, 8);
  a.groups = std::min(a.per_xcd, std::max(1, wgs / 8 / a.nsplit));
#ifdef BSP_ROWS_TUNE
  if (!std::getenv("BSP_PWS_TUNE"))
#endif
    if (!bsp_pws_beats(i8, nstrips, steps, p.residual != nullptr, (double)a.tiles * a.nsplit / (256 * 16 / NW))) return BSP_ERR_UNSUPPORTED;
  const int32_t* sec = p.plan + hdr[BSP_PLAN_OFF_ROWS_W];
  a.X = (const unsigned char*)p.X;
  a.Y = (unsigned char*)p.Y;
  a.bias = p.bias;
  a.residual = (const unsigned char*)p.residual;
  a.relu = i8 ? shift : p.relu;
  a.rstrip = sec + rs[BSP_ROWS_OFF_STRIP_W];
  a.rslab = sec + rs[BSP_ROWS_OFF_SLAB_W];
  a.rdesc = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_DESC_W]);
  a.rfrag = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_FRAG_W]);
  a.nstrips = nstrips;
  a.ncs = rs[BSP_ROWS_NCS_W];
  a.P = p.P;
  a.O = p.O;
  a.S = p.sh;
  a.L = p.L;
  a.J = p.J;
  a.N = p.N;
  a.MN = p.M * p.N;
  a.pair = hdr[BSP_PLAN_BO_W] != 4;
  // multiply-high divisions are exact while dividend * divisor < 2^32 (at stride 1 no pixel number is divided)
  const int64_t pieces = (int64_t)QL * threads, outs = (int64_t)SW * threads;
  if ((a.S > 1 && (int64_t)p.P * std::max(a.MN, a.N) >= (1ll << 32)) || (int64_t)a.groups * a.nsplit * a.nsplit >= (1ll << 32) || ((int64_t)a.tiles + 2 * a.groups) * MT >= (1ll << 30) ||
      pieces * a.cpx >= (1ll << 32) || outs * NS * 2 >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  a.d_mn = make_fastdiv((uint32_t)a.MN);
  a.d_n = make_fastdiv((uint32_t)a.N);
  a.d_cpx = make_fastdiv((uint32_t)a.cpx);
  a.d_nsplit = make_fastdiv((uint32_t)a.nsplit);
  a.d_cpp = make_fastdiv((uint32_t)(NS * (i8 ? 1 : 2)));
#ifdef BSP_ROWS_TUNE
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "pws: PT=%d P=%d I=%d O=%d S=%d strips=%d steps=%d | NW=%d SW=%d D=%d QL=%d NS=%d tiles=%d wgs=%d lds=%d\n", PT, p.P, p.I, p.O, p.sh, nstrips,
            steps, NW, SW, D, QL, NS, a.tiles, 8 * a.groups * a.nsplit, (int)ldsb);
#endif
  dim3 grid((unsigned)(a.groups * a.nsplit * 8));
  switch (cw) {
    case 4: return launch_k<4>(a, PT, SW, D, QL, grid, threads, (size_t)ldsb, st);
    case 8: return launch_k<8>(a, PT, SW, D, QL, grid, threads, (size_t)ldsb, st);
    case 16: return launch_k<16>(a, PT, SW, D, QL, grid, threads, (size_t)ldsb, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

}  // namespace

int bsp_launch_pws(const ConvParams& p, int dtype, const void* plan_host, int shift, hipStream_t st) {
  if (dtype == BSP_I8 && (p.residual || p.relu)) return BSP_ERR_UNSUPPORTED;
  return launch_pws(p, dtype, plan_host, shift, st);
}
