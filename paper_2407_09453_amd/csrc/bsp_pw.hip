// Pointwise (1x1) layers as a block-sparse matrix product, bf16 with fp32 accumulation or int8 codes
// with exact 32-bit sums:
// Y[pixel][o] = bias[o] + sum over the kept blocks of row o of W[o][i] * X[pixel][i]
// (paper Eq. (5) with H = K = 1; only kept blocks are multiplied, Section I advantages 3-4).
//
// Work split.  A workgroup owns MT = 16 * PT * PG consecutive output pixels and NS strips of
// 16 output channels.  All input channels of its pixels are copied once from global memory
// straight into LDS (global_load_lds, one contiguous KiB per request); nothing is staged
// twice and there is no loop over channel slabs.  A staged pixel is `pitch` bytes; its
// 16-byte pieces are permuted by the pixel's position (slot = piece ^ f(pixel)) so that the
// sixteen pixels of a lane tile fall into sixteen different bank groups.  Wave (strip s,
// pixel group q) walks the strip's column steps: per step one weight fragment (streamed from
// the plan through a ring of D registers, requested D steps ahead), PT activation fragments
// from LDS at the channels the step's descriptor names, PT MFMAs.  Results leave straight
// from the accumulators; two lane tiles exchange halves across lane rows first so that every
// lane stores the 16 contiguous bytes of one 8-channel block row.
//
// int8: a 16-byte piece is sixteen codes and a step's product is the i32 16x16x64 one, so staging,
// weights and steps are byte for byte the same; the launcher counts input channels in pairs of codes.
// A lane's four results are four bytes, so they always leave through the LDS image of the output.
//
// A tile's pixels past the layer's last one are staged as copies of that one, and a pixel's pieces past its channels as copies of
// its last piece, so that no lane of a request is masked.  Nothing of either reaches a result: each MFMA column depends on its
// own pixel only and columns past the last pixel are not stored, and no descriptor names a piece past the channels.
#include "bsp_kept.h"
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

struct PwArgs {
  const unsigned char* X;
  unsigned char* Y;
  const float* bias;
  const unsigned char* residual;
  const int32_t* rstrip;
  const int32_t* rslab;
  const unsigned char* rdesc;
  const unsigned char* rfrag;
  int32_t relu, nstrips;           // relu: int8 layers keep their rounding right shift here (a word more in this
                                   // block moves the others over line borders: 0.08 us per launch)
  int32_t P, I, O;
  int32_t S, L, J, N, MN;          // S > 1: output pixel (img, y, x) reads input pixel (img, y*S, x*S)
  int32_t pitch, swz_shift, swz_mask;
  int32_t MT, lpg, NS, nreq;       // pixels per tile, log2 of the pixel groups, strips, KiB requests per tile
  int32_t mtiles, nsplit, per_xcd;
  int32_t pair;                    // results leave as 16-byte pieces (lane tiles paired)
  int32_t win_out, out_off, opitch;  // results gathered in LDS as whole output lines: where, bytes per pixel there
  int32_t adv_pix, adv_rem;        // (waves * 1024) / pitch and % pitch: a wave's step from request to request
  FastDiv d_mn, d_n, d_pitch, d_nsplit, d_cpp;
#ifdef BSP_ROWS_TUNE
  long long* trace;
#endif
};

// Up to 64 pixels, where the layers run that the streaming FC kernels and the any-shape kernel take otherwise: a
// sum that is no finite number is formed again from kept blocks alone, as those kernels do (looking for one: a ballot,
// a flag per wave and a barrier, 0.1 to 0.2 us of 1 x 512 -> 2048's 4.1).  Instances of their own keep the others
// as they are.
struct PwFewArgs : PwArgs {
  const int32_t* plan;
  const unsigned char* payload;
  int32_t H, K, lbo;               // 1, 1, log2 of the block rows' height
  int32_t flag_off;                // LDS offset of a flag per wave
};

#ifdef BSP_ROWS_TUNE
#define PW_MARK(k)                                                                                   \
  do {                                                                                               \
    if (a.trace && lane == 0) a.trace[((size_t)blockIdx.x * 16 + wave) * 8 + (k)] = wall_clock64(); \
  } while (0)
#else
#define PW_MARK(k)
#endif

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// KIND: 8 or 4, the channels per unit of a bf16 layer; 16, an int8 layer.
template <int PT, int KIND, int D, int MAXT, typename Args>
__global__ __launch_bounds__(MAXT) void conv_pw(Args a) {
  constexpr bool CW4 = KIND == 4, I8 = KIND == 16, FEW = std::is_same<Args, PwFewArgs>::value;
  kernarg_touch<Args>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwaves = (int)(blockDim.x >> 6);
  // consecutive workgroups of one XCD share a pixel tile (its second reader hits that L2)
  const int xcd = blockIdx.x & 7, slot_wg = blockIdx.x >> 3;
  if (slot_wg >= a.per_xcd) return;
  const int q = xcd * a.per_xcd + slot_wg;
  const int mt = (int)fdiv((uint32_t)q, a.d_nsplit);
  if (mt >= a.mtiles) return;
  const int ns = q - mt * a.nsplit;
  const int pix0 = mt * a.MT;
  PW_MARK(0);

  // ---- this wave's strip and pixel group.  Its step range and output channels are wave-uniform:
  // scalar loads, asked for here and waited for once the tile's copies are on their way (a
  // vector load would have to queue behind those copies, and a wait here would delay them)
  const int sidx = wave >> a.lpg, pg = wave & ((1 << a.lpg) - 1);
  const int strip = ns * a.NS + sidx;
  const bool active = sidx < a.NS && strip < a.nstrips;
  const int sq = active ? strip : 0;
  u32x2_t lohi;
  u32x4_t ch4;
  {
    const int32_t* ps = a.rslab + sq * 2;
    const int32_t* pc = a.rstrip + sq * 4;
    asm volatile("s_load_dwordx2 %0, %2, 0x0\n\ts_load_dwordx4 %1, %3, 0x0"
                 : "=&s"(lohi), "=&s"(ch4)
                 : "s"(ps), "s"(pc)
                 : "memory");
  }

  // ---- stage the tile: request rq fills LDS bytes [rq * 1024, rq * 1024 + 1024).  No lane is masked: a pixel past
  // the layer's last asks for the last one's bytes, a piece past a pixel's channels for the pixel's last piece (no
  // descriptor names it), so a request is a dozen instructions and no branch, and four go out between two jumps
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  {
    // lane state: the pixel its 16 bytes belong to and their offset in it; from one request of this wave to the
    // next both advance by constants
    const uint32_t o0 = (uint32_t)wave * 1024u + (uint32_t)lane * 16u;
    const uint32_t lp0 = fdiv(o0, a.d_pitch);
    uint32_t rem = o0 - lp0 * (uint32_t)a.pitch, p = (uint32_t)pix0 + lp0;  // (tiles are whole sixteens of pixels: p permutes as lp)
    const uint32_t rowb = (uint32_t)a.I * 2u, last = (uint32_t)a.P - 1u, swzm = (uint32_t)a.swz_mask << 4;
    const int swzs = 4 - a.swz_shift;
    auto request = [&](int rq, auto strided) {
      const uint32_t off = min(rem ^ ((p << swzs) & swzm), rowb - 16u);
      uint32_t ip = min(p, last);
      if constexpr (decltype(strided)::value) {
        const uint32_t img = fdiv(ip, a.d_mn), r2 = ip - img * (uint32_t)a.MN;
        const uint32_t oy = fdiv(r2, a.d_n), ox = r2 - oy * (uint32_t)a.N;
        ip = (img * (uint32_t)a.L + oy * (uint32_t)a.S) * (uint32_t)a.J + ox * (uint32_t)a.S;
      }
      __builtin_amdgcn_global_load_lds((gptr_t)(a.X + (ip * rowb + off)), (lptr_t)(uintptr_t)(lds0 + (uint32_t)rq * 1024u), 16, 0, 0);
      rem += (uint32_t)a.adv_rem;
      const bool over = rem >= (uint32_t)a.pitch;
      p += (uint32_t)a.adv_pix + (over ? 1u : 0u);
      rem = over ? rem - (uint32_t)a.pitch : rem;
    };
    int rq = wave;
    if (a.S == 1) {
      for (; rq + 3 * nwaves < a.nreq; rq += 4 * nwaves) {
#pragma unroll
        for (int u = 0; u < 4; ++u) request(rq + u * nwaves, std::false_type{});
      }
      for (; rq < a.nreq; rq += nwaves) request(rq, std::false_type{});
    } else {
      for (; rq < a.nreq; rq += nwaves) request(rq, std::true_type{});
    }
  }
  PW_MARK(1);
  // ---- the step range and channels asked for above have to be there now (the registers pass
  // through the wait, so that no use of them is moved above it)
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(lohi), "+s"(ch4) : : "memory");
  PW_MARK(2);
  const int lo = (int)lohi.x, hi = active ? (int)lohi.y : lo;
  const int nsteps = hi - lo;
  // first output channel of this lane's four rows
  const int chan = !active ? -1 : g == 0 ? (int)ch4.x : g == 1 ? (int)ch4.y : g == 2 ? (int)ch4.z : (int)ch4.w;

  const uint32_t frag_lane = (uint32_t)lane * 16u, desc_lane = (uint32_t)g * 4u;
  u32x4_t wr[D];  // weight fragments of the next D steps, oldest in slot 0
  int dr[D];      // their item descriptors
  int fnext = lo;
  // Slot d takes the next step; past the strip's end it asks for the last step again (a valid
  // address, never used).  Every pass of the ring loop thus issues the same loads whatever
  // the step count, so the wait before a slot's use can be for exactly that slot.
  auto fetch = [&](int d) {
    const int cs = min(fnext, hi - 1);
    ++fnext;
    dr[d] = *(const int*)(a.rdesc + ((uint32_t)cs * 16u + desc_lane));
    wr[d] = *(const u32x4_t*)(a.rfrag + ((uint32_t)cs * 1024u + frag_lane));
  };
  // the first D steps, and no more than the strip has
#pragma unroll
  for (int d = 0; d < D; ++d) {
    dr[d] = 0;
    wr[d] = u32x4_t{0, 0, 0, 0};
    if (d < nsteps) fetch(d);
  }
  using acc_t = typename std::conditional<I8, i32x4_t, f32x4_t>::type;
  using bias_t = typename std::conditional<I8, int32_t, float>::type;
  acc_t bv = {0, 0, 0, 0};
  const bias_t* bp = (const bias_t*)a.bias;
  if (bp && chan >= 0) bv = acc_t{bp[chan], bp[chan + 1], bp[chan + 2], bp[chan + 3]};

  acc_t acc[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) acc[t] = acc_t{0, 0, 0, 0};

  PW_MARK(3);
  __builtin_amdgcn_s_waitcnt(0);  // this wave's requests have landed
  PW_MARK(4);
  __syncthreads();                // everybody's have
  PW_MARK(5);
  if (!FEW && !active && !a.win_out) return;  // (with win_out every wave helps to store the tile)

  const int lp0 = pg * (PT * 16) + c;  // this lane's pixel of the wave's first lane tile
  const uint32_t swz = ((uint32_t)lp0 >> a.swz_shift) & (uint32_t)a.swz_mask;  // the same in every lane tile
  const uint32_t base = (uint32_t)lp0 * (uint32_t)a.pitch;
  const uint32_t tstep = 16u * (uint32_t)a.pitch;

  // the activation fragments of the step in slot d
  auto read = [&](int d, u32x4_t (&f)[PT]) {
    uint32_t desc = (uint32_t)dr[d];
    // the descriptor is decoded here, at its use: decoded where it is loaded, every
    // pass of the loop would wait for all the ring's loads at once
    asm volatile("" : "+v"(desc));
    if (CW4) {
      const uint32_t u0 = desc & 0xFFu, u1 = (desc >> 16) & 0xFFu;
      const uint32_t a0 = base + (((u0 >> 1) ^ swz) << 4) + ((u0 & 1u) << 3);
      const uint32_t a1 = base + (((u1 >> 1) ^ swz) << 4) + ((u1 & 1u) << 3);
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        const u32x2_t p0 = *(const u32x2_t*)(lds + a0 + t * tstep);
        const u32x2_t p1 = *(const u32x2_t*)(lds + a1 + t * tstep);
        f[t] = u32x4_t{p0.x, p0.y, p1.x, p1.y};
      }
    } else {
      const uint32_t ad = base + (((desc & 0xFFu) ^ swz) << 4);
#pragma unroll
      for (int t = 0; t < PT; ++t) f[t] = *(const u32x4_t*)(lds + ad + t * tstep);
    }
  };
  auto mfmas = [&](int d, const u32x4_t (&f)[PT]) {
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      if constexpr (I8)
        acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4_t, wr[d]), __builtin_bit_cast(i32x4_t, f[t]),
                                                       acc[t], 0, 0, 0);
      else
        acc[t] = mfma_bf16_16x16x32(wr[d], f[t], acc[t]);
    }
  };

  // A step's fragments are read from LDS while the step before it is in the matrix cores.
  u32x4_t fa[PT], fb[PT];
  int cs0 = lo;
  if (nsteps > 0) read(0, fa);
  // whole passes over the ring while more than D steps remain: every slot is used and then
  // refilled in place, after the MFMAs that read it
  for (; cs0 + D < hi; cs0 += D) {
#pragma unroll
    for (int d = 0; d < D; d += 2) {
      read(d + 1, fb);
      mfmas(d, fa);
      __builtin_amdgcn_sched_barrier(0);
      fetch(d);
      __builtin_amdgcn_sched_barrier(0);
      read((d + 2) % D, fa);
      mfmas(d + 1, fb);
      __builtin_amdgcn_sched_barrier(0);
      fetch(d + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the last steps (at most D): nothing is asked for any more
#pragma unroll
  for (int d = 0; d < D; d += 2) {
    if (cs0 + d + 1 < hi) read(d + 1, fb);
    if (cs0 + d < hi) mfmas(d, fa);
    if (d + 2 < D && cs0 + d + 2 < hi) read(d + 2, fa);
    if (cs0 + d + 1 < hi) mfmas(d + 1, fb);
  }

  // ---- results: bias, one rounding, then the optional residual add and ReLU
  if constexpr (!I8) {
#pragma unroll
    for (int t = 0; t < PT; ++t) acc[t] += bv;
  }
#ifdef BSP_ROWS_TUNE
  asm volatile("" ::"v"(acc[0]));
#endif
  PW_MARK(6);
  if constexpr (I8) {
    // + bias, rounding right shift (ties upward), saturation, into the image of the output lines
    unsigned char* ot = lds + a.out_off;
    const int range0 = ns * a.NS * 16, lpix = pg * (PT * 16) + c;
    const RescaleI8 rescale(bv, a.relu);
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const uint32_t v = rescale(acc[t]);
      if (chan >= 0) *(uint32_t*)(ot + (lpix + t * 16) * a.opitch + (chan - range0)) = v;
    }
    __syncthreads();
    const int cpp = a.NS, total = a.MT * cpp;  // 16-byte pieces per pixel, of the tile
    for (int i = tid; i < total; i += (int)blockDim.x) {
      const int pixel = (int)fdiv((uint32_t)i, a.d_cpp), k = i - pixel * cpp;
      const int ch = range0 + k * 16, gp = pix0 + pixel;
      if (gp < a.P && ch < a.O)
        __builtin_nontemporal_store(*(const u32x4_t*)(ot + pixel * a.opitch + k * 16),
                                    (u32x4_t*)(a.Y + ((uint32_t)gp * (uint32_t)a.O + (uint32_t)ch)));
    }
    return;
  }
  const int ptile0 = pix0 + pg * (PT * 16);
  if constexpr (FEW) {
    uint32_t* flags = (uint32_t*)(lds + a.flag_off);
    bool bad = false;
#pragma unroll
    for (int t = 0; t < PT; ++t)
      if (chan >= 0 && ptile0 + t * 16 + c < a.P) {  // (the other lanes hold copies of the last pixel)
#pragma unroll
        for (int r = 0; r < 4; ++r) bad |= (__float_as_uint(acc[t][r]) & 0x7F800000u) == 0x7F800000u;
      }
    const uint64_t mine = __ballot(bad);
    if (lane == 0) flags[wave] = mine != 0;
    __syncthreads();
    if (__ballot(lane < nwaves && flags[lane < nwaves ? lane : 0])) {
      // the workgroup's strips (whole windows of four) cover the channels of as many strips in natural order
      const int nat = ns * a.NS + sidx, ch = nat * BSP_STRIP + 4 * g;
      if (sidx >= a.NS || nat * BSP_STRIP >= a.O) return;
      f32x4_t b4 = {0.f, 0.f, 0.f, 0.f};
      if (a.bias && ch < a.O) b4 = f32x4_t{a.bias[ch], a.bias[ch + 1], a.bias[ch + 2], a.bias[ch + 3]};
#pragma unroll 1
      for (int t = 0; t < PT; ++t) {
        const int pixel = ptile0 + t * 16 + c, p = min(pixel, a.P - 1);
        const int img = (int)fdiv((uint32_t)p, a.d_mn), r2 = p - img * a.MN;
        const int oy = (int)fdiv((uint32_t)r2, a.d_n), ox = r2 - oy * a.N;
        const f32x4_t v = kept_only<true>(a, a.X + (int64_t)img * a.L * a.J * a.I * 2, nat, oy * a.S, ox * a.S, lane) + b4;
        if (pixel >= a.P || ch >= a.O) continue;
        u32x2_t o = {pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
        const uint32_t off = ((uint32_t)pixel * (uint32_t)a.O + (uint32_t)ch) * 2u;
        if (a.residual || a.relu) o = post_bf16x4(o, a.residual ? (const uint16_t*)(a.residual + off) : nullptr, 4, true, a.relu);
        *(u32x2_t*)(a.Y + off) = o;
      }
      return;
    }
    if (!active && !a.win_out) return;
  }
  // lane rows 0/1 (and 2/3) hold the two halves of one 8-channel block row: after an exchange
  // an even row has all eight channels of lane tile t, an odd row those of lane tile t + 1
  const int ch8 = __builtin_amdgcn_ds_bpermute(((lane & 32) + c) << 2, chan);  // the even row's channel
  const int odd = g & 1;
  auto paired = [&](int t) {
    const uint32_t x0 = pack_bf16x2(acc[t].x, acc[t].y), y0 = pack_bf16x2(acc[t].z, acc[t].w);
    const uint32_t x1 = pack_bf16x2(acc[t + 1].x, acc[t + 1].y), y1 = pack_bf16x2(acc[t + 1].z, acc[t + 1].w);
    const auto sx = __builtin_amdgcn_permlane16_swap(x0, x1, false, false);
    const auto sy = __builtin_amdgcn_permlane16_swap(y0, y1, false, false);
    return u32x4_t{sx[0], sy[0], sx[1], sy[1]};
  };
  if (a.win_out) {
    // The workgroup's strips cover a contiguous range of output channels: every wave puts its
    // pieces where they belong in an LDS image of the tile's output lines, then all threads
    // copy that image out, 16 contiguous bytes per lane.
    unsigned char* ot = lds + a.out_off;
    const int range0 = ns * a.NS * 16;
    const int lpix = pg * (PT * 16) + c;
    if (PT >= 2 && a.pair) {
#pragma unroll
      for (int t = 0; t + 1 < PT; t += 2) {
        const u32x4_t v = paired(t);
        if (ch8 >= 0) *(u32x4_t*)(ot + (lpix + (t + odd) * 16) * a.opitch + (ch8 - range0) * 2) = v;
      }
    } else {
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        const u32x2_t v = {pack_bf16x2(acc[t].x, acc[t].y), pack_bf16x2(acc[t].z, acc[t].w)};
        if (chan >= 0) *(u32x2_t*)(ot + (lpix + t * 16) * a.opitch + (chan - range0) * 2) = v;
      }
    }
    // what this thread copies out afterwards, and the residual that goes with it: asked for
    // now, used after the barrier
    const int cpp = a.NS * 2;  // 16-byte pieces per pixel
    const int total = a.MT * cpp;
    constexpr int NIT = PT >= 2 ? PT / 2 : 1;  // pieces per thread: 16 * PT * NS * 2 over 64 * NS * PG threads
    uint32_t ooff[NIT], lsrc[NIT];
    bool ovalid[NIT];
    u32x4_t res[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int i = tid + it * (int)blockDim.x;
      const int pixel = (int)fdiv((uint32_t)min(i, total - 1), a.d_cpp), k = min(i, total - 1) - pixel * cpp;
      const int ch = range0 + k * 8, gp = pix0 + pixel;
      ovalid[it] = i < total && gp < a.P && ch < a.O;
      ooff[it] = ((uint32_t)gp * (uint32_t)a.O + (uint32_t)ch) * 2u;
      lsrc[it] = (uint32_t)(pixel * a.opitch + k * 16);
      res[it] = u32x4_t{0, 0, 0, 0};
      if (ovalid[it] && a.residual) res[it] = *(const u32x4_t*)(a.residual + ooff[it]);
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (!ovalid[it]) continue;
      const u32x4_t v = *(const u32x4_t*)(ot + lsrc[it]);
      u32x2_t l2 = {v.x, v.y}, h2 = {v.z, v.w};
      if (a.residual || a.relu) {
        l2 = post_bf16x4_reg(l2, u32x2_t{res[it].x, res[it].y}, a.residual != nullptr, a.relu);
        h2 = post_bf16x4_reg(h2, u32x2_t{res[it].z, res[it].w}, a.residual != nullptr, a.relu);
      }
      // (whole output lines leave as streaming stores: no burst of dirty L2 lines is left for the
      // end of the kernel; pieces scattered over a line, below, are better merged in L2)
      __builtin_nontemporal_store(u32x4_t{l2.x, l2.y, h2.x, h2.y}, (u32x4_t*)(a.Y + ooff[it]));
    }
    // (a workgroup with several pixel groups has more pieces per thread than NIT covers)
    for (int i = tid + NIT * (int)blockDim.x; i < total; i += (int)blockDim.x) {
      const int pixel = (int)fdiv((uint32_t)i, a.d_cpp), k = i - pixel * cpp;
      const int ch = range0 + k * 8, gp = pix0 + pixel;
      if (gp >= a.P || ch >= a.O) continue;
      const u32x4_t v = *(const u32x4_t*)(ot + pixel * a.opitch + k * 16);
      const uint32_t off = ((uint32_t)gp * (uint32_t)a.O + (uint32_t)ch) * 2u;
      u32x2_t l2 = {v.x, v.y}, h2 = {v.z, v.w};
      if (a.residual || a.relu) {
        u32x4_t r = {0, 0, 0, 0};
        if (a.residual) r = *(const u32x4_t*)(a.residual + off);
        l2 = post_bf16x4_reg(l2, u32x2_t{r.x, r.y}, a.residual != nullptr, a.relu);
        h2 = post_bf16x4_reg(h2, u32x2_t{r.z, r.w}, a.residual != nullptr, a.relu);
      }
      __builtin_nontemporal_store(u32x4_t{l2.x, l2.y, h2.x, h2.y}, (u32x4_t*)(a.Y + off));
    }
  } else if (PT >= 2 && a.pair) {
#pragma unroll
    for (int t = 0; t + 1 < PT; t += 2) {
      u32x4_t v = paired(t);
      const int pixel = ptile0 + (t + odd) * 16 + c;
      if (pixel >= a.P || ch8 < 0) continue;
      const uint32_t off = ((uint32_t)pixel * (uint32_t)a.O + (uint32_t)ch8) * 2u;
      if (a.residual || a.relu) {
        const uint16_t* rp = a.residual ? (const uint16_t*)(a.residual + off) : nullptr;
        const u32x2_t l2 = post_bf16x4(u32x2_t{v.x, v.y}, rp, 4, true, a.relu);
        const u32x2_t h2 = post_bf16x4(u32x2_t{v.z, v.w}, rp ? rp + 4 : nullptr, 4, true, a.relu);
        v = u32x4_t{l2.x, l2.y, h2.x, h2.y};
      }
      *(u32x4_t*)(a.Y + off) = v;
    }
  } else {
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const int pixel = ptile0 + t * 16 + c;
      if (pixel >= a.P || chan < 0) continue;
      u32x2_t v = {pack_bf16x2(acc[t].x, acc[t].y), pack_bf16x2(acc[t].z, acc[t].w)};
      const uint32_t off = ((uint32_t)pixel * (uint32_t)a.O + (uint32_t)chan) * 2u;
      if (a.residual || a.relu)
        v = post_bf16x4(v, a.residual ? (const uint16_t*)(a.residual + off) : nullptr, 4, true, a.relu);
      *(u32x2_t*)(a.Y + off) = v;
    }
  }
#ifdef BSP_ROWS_TUNE
  __builtin_amdgcn_s_waitcnt(0);
#endif
  PW_MARK(7);
}

constexpr int kLdsLimit = 160 * 1024;

template <int PT, int KIND, int D, int MAXT, typename Args>
int launch_inst(const Args& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_pw<PT, KIND, D, MAXT, Args>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kLdsLimit) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_pw<PT, KIND, D, MAXT, Args>), grid, dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

// Ring depth D: strips of at most 2 (4) steps take instances with as many registers for
// weights, which leaves room for more waves per SIMD; otherwise 8.
template <int KIND, int D, typename Args>
int launch_d(const Args& a, int PT, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  constexpr int MAXT = 1024;
  if (threads > MAXT) return BSP_ERR_UNSUPPORTED;
  switch (PT) {
    case 1: return launch_inst<1, KIND, D, MAXT, Args>(a, grid, threads, ldsb, st);
    case 2: return launch_inst<2, KIND, D, MAXT, Args>(a, grid, threads, ldsb, st);
    case 4: return launch_inst<4, KIND, D, MAXT, Args>(a, grid, threads, ldsb, st);
    case 8:
      if constexpr (std::is_same<Args, PwArgs>::value)
        return launch_inst<8, KIND, D, (D >= 8 ? 512 : MAXT), Args>(a, grid, threads, ldsb, st);  // 8 lane tiles and a ring of 8 need more than 128 registers
  }
  return BSP_ERR_UNSUPPORTED;
}

template <int KIND, typename Args>
int launch_pt(const Args& a, int PT, int depth, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  if (PT == 8 && depth >= 8 && threads > 512) return BSP_ERR_UNSUPPORTED;
  switch (depth) {
    case 2: return launch_d<KIND, 2, Args>(a, PT, grid, threads, ldsb, st);
    case 4: return launch_d<KIND, 4, Args>(a, PT, grid, threads, ldsb, st);
    case 8: return launch_d<KIND, 8, Args>(a, PT, grid, threads, ldsb, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

int launch_pw(const ConvParams& p, int dtype, const void* plan_host, int shift, bool few, hipStream_t st) {
  const bool i8 = dtype == BSP_I8;
  if (!plan_host) return BSP_ERR_UNSUPPORTED;
  const int32_t* hdr = (const int32_t*)plan_host;
  if (hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION ||
      hdr[BSP_PLAN_O_W] != p.O || hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H ||
      hdr[BSP_PLAN_K_W] != p.K || hdr[BSP_PLAN_DTYPE_W] != dtype || hdr[BSP_PLAN_OFF_ROWS_W] == 0)
    return BSP_ERR_UNSUPPORTED;
  const int32_t* rs = hdr + hdr[BSP_PLAN_OFF_ROWS_W];
  if (p.H != 1 || p.K != 1 || p.ph != 0 || p.pw != 0 || p.sh != p.sw || p.sh < 1) return BSP_ERR_UNSUPPORTED;
  if (rs[BSP_ROWS_NSLABS_W] != 1 || few != (p.P <= 64)) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.B * p.L * p.J * p.I * 2 >= (1ll << 31) || (int64_t)p.P * p.O * 2 >= (1ll << 31))
    return BSP_ERR_UNSUPPORTED;
  const int nstrips = rs[BSP_ROWS_NSTRIPS_W];
  const int raw = p.I * (i8 ? 1 : 2);
  const int pitch = raw <= 128 ? 128 : (raw + 255) & ~255;
#ifdef BSP_ROWS_TUNE
  long long* a_trace = nullptr;
#endif
  const int maxsteps = rs[BSP_ROWS_MAXSTRIPSTEPS_W];
  const int depth = maxsteps <= 2 ? 2 : maxsteps <= 4 ? 4 : 8;
  BspPwChoice ch = bsp_pw_choose(p.P, raw / 2, i8 ? (1 << 30) : p.O, nstrips, pitch, rs[BSP_ROWS_WINDOW_W] == 4, i8);
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (const char* e = std::getenv("BSP_PWK_TUNE")) {
    int q[4];
    if (sscanf(e, "%d,%d,%d,%d", q, q + 1, q + 2, q + 3) == 4) ch = BspPwChoice{q[0], q[1], q[2], q[3]};
  }
  if (const char* e = std::getenv("BSP_PW_TRACE_PTR")) a_trace = (long long*)std::strtoull(e, nullptr, 16);
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "pw: P=%d I=%d O=%d S=%d strips=%d steps=%d | PT=%d PG=%d NS=%d wout=%d\n", p.P, p.I, p.O,
            p.sh, nstrips, rs[BSP_ROWS_NCS_W], ch.PT, ch.PG, ch.NS, ch.wout);
#endif
  if (ch.PT < 1 || ch.PG < 1 || ch.NS < 1) return BSP_ERR_UNSUPPORTED;
  PwArgs a{};
  const int32_t* sec = p.plan + hdr[BSP_PLAN_OFF_ROWS_W];
#ifdef BSP_ROWS_TUNE
  a.trace = a_trace;
#endif
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
  a.P = p.P;
  a.I = raw / 2;  // int8: pairs of codes
  a.O = p.O;
  a.S = p.sh;
  a.L = p.L;
  a.J = p.J;
  a.N = p.N;
  a.MN = p.M * p.N;
  a.pitch = pitch;
  if (pitch % 256 == 0) {
    a.swz_shift = 0;
    a.swz_mask = 15;
  } else {
    a.swz_shift = 1;
    a.swz_mask = 7;
  }
  a.MT = 16 * ch.PT * ch.PG;
  a.lpg = 0;
  while ((1 << a.lpg) < ch.PG) ++a.lpg;
  if ((1 << a.lpg) != ch.PG) return BSP_ERR_UNSUPPORTED;
  a.NS = ch.NS;
  const int64_t xbytes = (int64_t)a.MT * pitch;
  // whole-line output through LDS: the plan keeps windows of four strips together and the
  // workgroup takes whole windows (or every strip there is)
  a.win_out = ch.wout && rs[BSP_ROWS_WINDOW_W] == 4 && (ch.NS % 4 == 0 || ch.NS >= nstrips);
  a.out_off = (int32_t)xbytes;
  a.opitch = ch.NS * (i8 ? 16 : 32) + 16;
  if (i8 && !a.win_out) return BSP_ERR_UNSUPPORTED;
  const int64_t ldsb = xbytes + (a.win_out ? (int64_t)a.MT * a.opitch : 0);
  if (ldsb > kLdsLimit || ch.PG * ch.NS > 16 || ch.PG * ch.NS < 1) return BSP_ERR_UNSUPPORTED;
  a.nreq = (int32_t)(xbytes / 1024);
  a.d_cpp = make_fastdiv((uint32_t)(ch.NS * (i8 ? 1 : 2)));
  a.mtiles = cdiv(p.P, a.MT);
  a.nsplit = cdiv(nstrips, ch.NS);
  const int64_t wgs = (int64_t)a.mtiles * a.nsplit;
  a.per_xcd = cdiv(wgs, 8);
  a.pair = hdr[BSP_PLAN_BO_W] != 4 && ch.PT >= 2;
  // multiply-high divisions are exact while dividend * divisor < 2^32
  // (pixel numbers, which are divided where the stride is not 1; at stride 1 a line: larger layers go on to the kernels after)
  const int64_t pmax = (int64_t)a.mtiles * a.MT;
  if (pmax * std::max(a.MN, a.N) >= (1ll << 32) || (int64_t)a.per_xcd * 8 * a.nsplit >= (1ll << 32) ||
      xbytes * pitch >= (1ll << 32) || (int64_t)a.per_xcd * 8 >= (1ll << 31))
    return BSP_ERR_UNSUPPORTED;
  a.d_mn = make_fastdiv((uint32_t)a.MN);
  a.d_n = make_fastdiv((uint32_t)a.N);
  a.d_pitch = make_fastdiv((uint32_t)pitch);
  a.d_nsplit = make_fastdiv((uint32_t)a.nsplit);
  const int threads = 64 * ch.PG * ch.NS;
  a.adv_pix = (threads * 16) / pitch;
  a.adv_rem = (threads * 16) % pitch;
  dim3 grid((unsigned)(a.per_xcd * 8));
  const int cw = rs[BSP_ROWS_CW_W];
  if (few && !i8) {
    // (what is formed again is a workgroup's range of channels: the range that its strips cover)
    if (rs[BSP_ROWS_WINDOW_W] != 4 || (ch.NS % 4 && ch.NS < nstrips)) return BSP_ERR_UNSUPPORTED;
    PwFewArgs f{};
    static_cast<PwArgs&>(f) = a;
    f.plan = p.plan;
    f.payload = (const unsigned char*)p.payload;
    f.H = f.K = 1;
    f.lbo = __builtin_ctz(hdr[BSP_PLAN_BO_W]);
    f.flag_off = (int32_t)ldsb;
    if (ldsb + 64 > kLdsLimit) return BSP_ERR_UNSUPPORTED;
    return cw == 4 ? launch_pt<4>(f, ch.PT, depth, grid, threads, (size_t)ldsb + 64, st)
                   : launch_pt<8>(f, ch.PT, depth, grid, threads, (size_t)ldsb + 64, st);
  }
  switch (cw) {
    case 4: return launch_pt<4>(a, ch.PT, depth, grid, threads, (size_t)ldsb, st);
    case 8: return launch_pt<8>(a, ch.PT, depth, grid, threads, (size_t)ldsb, st);
    case 16: return launch_pt<16>(a, ch.PT, depth, grid, threads, (size_t)ldsb, st);
  }
  return BSP_ERR_UNSUPPORTED;
}

}  // namespace

int bsp_launch_pw(const ConvParams& p, int dtype, const void* plan_host, hipStream_t st) {
  return dtype == BSP_BF16 ? launch_pw(p, dtype, plan_host, 0, false, st) : BSP_ERR_UNSUPPORTED;
}

int bsp_launch_pw_few(const ConvParams& p, const void* plan_host, hipStream_t st) {
  return launch_pw(p, BSP_BF16, plan_host, 0, true, st);
}

int bsp_launch_pw_i8(const ConvParams& p, const void* plan_host, int shift, hipStream_t st) {
  const bool few = p.P <= 64;
  if (p.residual || p.relu || (few && !bsp_pw_few_beats_i8(p.I, p.O))) return BSP_ERR_UNSUPPORTED;
  return launch_pw(p, BSP_I8, plan_host, shift, few, st);
}
