// 3x3 layers (stride 1, padding 1 or 0, bf16, at most 128 input channels) on many pixels: the band kernel's steps
// (bsp_band.hip) with the weights held in registers and the bands streamed past them.
//
// Work split.  A workgroup is one wave per (strip, column tile of 16) and takes every so many-th tile of four output rows
// x CT column tiles in its XCD's eighth of them.  A wave reads its strip's weights once and keeps them (three fragments a
// step, six steps at the most).  Per tile: the next tile's input is asked for, into registers, by buffer loads whose
// bounds turn what lies outside the image into zeros; the last tile's results leave as whole output lines; this
// tile's products from LDS, a step's fragments read three patch rows ahead; results into an LDS image of the output; the
// next tile's input to the other LDS buffer; one barrier.  Steps and their order are the band kernel's, so the
// results are the same bits (the LDS-resident kernel's steps come in another order).  As in the band kernel, a strip's
// rows share what one of them keeps: an infinity or NaN in a channel that a row drops reaches it through the strip's
// other rows, and the first unit's through steps that are not full.
//
// What bounds it: memory, then the reads of the products (224x224x64 batch 16: 207 MB, 34 us at a copy's rate, in 48 to 51;
// matrix cores busy 32 % of the cycles, LDS 34 %).  The band kernel gives every tile a workgroup of its own, which walks
// launch, copy, weights, products and results one after the other (64 to 67 us there); on 149x149x32 batch 16 the
// LDS-resident kernel took 27.2 and this one takes 14.4.  Four rows rather than seven: a CU then holds twelve waves instead of eight (51 / 56 us), which is
// worth more than the halo rows; two tiles asked for ahead made no difference, a fragment read one row or five ahead
// neither.  With a branch per step the compiler waits for every read, so there is straight code for every number of steps.
#include "bsp_bands_map.h"
#include "bsp_launch.h"
#include "bsp_tile.h"

#include <algorithm>
#include <type_traits>
#ifdef BSP_ROWS_TUNE
#include <cstdio>
#include <cstdlib>
#endif

namespace {

struct BandsArgs {
  const unsigned char* X;
  unsigned char* Y;
  const float* bias;
  const unsigned char* residual;
  const int32_t* rstrip;
  const int32_t* rslab;
  const unsigned char* rdesc;
  const unsigned char* rfrag;
  int32_t relu, nstrips, ncs;
  int32_t xbytes, ybytes;       // of the whole input and output
  int32_t L, J, M, N, O, pad;
  int32_t cpx, pitch, rowpitch; // 16-byte pieces of a pixel; LDS bytes of a staged one and of a staged row
  int32_t pieces;               // of a patch
  int32_t ctiles, cw;           // column tiles and columns of a tile
  int32_t tiles, per_xcd, groups, tpi, nchunks;  // tiles, of an XCD; workgroups of an XCD that share them; of an image; of a band
  int32_t slot, out_off, oslot, opitch, single, bias_off;
  FastDiv d_cpx, d_jp, d_tpi, d_nchunks, d_cpp, d_ns;
};

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

constexpr int BR = kBandsRows, QL = kBandsPieces;

// D: the most steps of a strip; T: 256 times the waves that a SIMD is to hold.
template <int D, int T, bool RES>
__global__ __launch_bounds__(T) void conv_bands(BandsArgs a) {
  constexpr uint32_t kNone = 0x80000000u;  // an offset past the end of every tensor: reads as zero, is not written
  kernarg_touch<BandsArgs>();
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = (int)blockDim.x;
  // an XCD takes an eighth of the tiles, one after the other: the halo that neighbours share comes from its L2
  const int xcd = blockIdx.x & 7, grp = blockIdx.x >> 3;
  const int first = xcd * a.per_xcd + grp, end = min(a.tiles, (xcd + 1) * a.per_xcd);
  if (first >= end) return;
  const auto xsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, a.xbytes, 0x00020000);
  const auto ydst = __builtin_amdgcn_make_buffer_rsrc((void*)a.Y, 0, a.ybytes, 0x00020000);
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(RES ? a.residual : a.X), 0, RES ? a.ybytes : 0, 0x00020000);

  // ---- the pieces of input this lane brings for every tile
  uint32_t xofs[QL], xrc[QL], xlds[QL];  // offset from the patch's first pixel; row | column << 16; place in LDS
#pragma unroll
  for (int j = 0; j < QL; ++j) {
    const uint32_t idx = (uint32_t)(tid + j * nthr);
    const bool some = bsp_bands_some((int)idx, a.pieces);
    const uint32_t px = fdiv(idx, a.d_cpx), piece = idx - px * (uint32_t)a.cpx;
    const uint32_t row = fdiv(px, a.d_jp), col = px - row * a.d_jp.d;
    xofs[j] = some ? (row * (uint32_t)a.J + col) * (uint32_t)(a.cpx * 16) + piece * 16u : 0u;
    xrc[j] = some ? row | col << 16 : 0x7FFFu;
    xlds[j] = some ? row * (uint32_t)a.rowpitch + col * (uint32_t)a.pitch + piece * 16u : 0u;
  }
  struct Tile {
    int n, y0, x0;
  };
  auto locate = [&](int tile) {
    const int n = (int)fdiv((uint32_t)tile, a.d_tpi), r = tile - n * a.tpi;
    const int band = (int)fdiv((uint32_t)r, a.d_nchunks), chunk = r - band * a.nchunks;
    return Tile{n, band * BR, chunk * a.cw};
  };
  i32x4_t xr[QL];
  auto load_x = [&](Tile t, bool some) {
    const int yi = t.y0 - a.pad, xi = t.x0 - a.pad;
    const uint32_t base = (uint32_t)((t.n * a.L + yi) * a.J + xi) * (uint32_t)(a.cpx * 16);
    const bool inside = yi >= 0 && xi >= 0 && yi + BR + 2 <= a.L && xi + a.cw + 2 <= a.J;
    uint32_t at[QL];
    if (some && inside) {
#pragma unroll
      for (int j = 0; j < QL; ++j) at[j] = base + xofs[j];
    } else {
#pragma unroll
      for (int j = 0; j < QL; ++j) {
        const uint32_t row = (uint32_t)(yi + (int)(xrc[j] & 0xFFFFu)), col = (uint32_t)(xi + (int)(xrc[j] >> 16));
        const bool ok = (row < (uint32_t)a.L) & (col < (uint32_t)a.J) & some;
        at[j] = ok ? base + xofs[j] : kNone;
      }
    }
#pragma unroll
    for (int j = 0; j < QL; ++j) {
      asm volatile("" : "+v"(at[j]));  // one load after the branch, not one in either: the waits count them
      xr[j] = __builtin_bit_cast(i32x4_t, __builtin_amdgcn_raw_buffer_load_b128(xsrc, at[j], 0, 0));
    }
  };
  auto write_x = [&](uint32_t off) {
#pragma unroll
    for (int j = 0; j < QL; ++j)
      if (bsp_bands_some(tid + j * nthr, a.pieces)) *(i32x4_t*)(lds + off + xlds[j]) = xr[j];
  };
  Tile at = locate(first);
  load_x(at, true);

  // ---- this wave's strip and column tile.  Workgroups that share a CU (an XCD deals them out over its 32 one by one)
  // begin with different strips, so that a SIMD does not have the heaviest of each.
  const int ct = (int)fdiv((uint32_t)wave, a.d_ns);
  int strip = wave - ct * a.nstrips + (grp >> 5) % a.nstrips;
  if (strip >= a.nstrips) strip -= a.nstrips;
  const int lo = a.rslab[strip * 2], n = __builtin_amdgcn_readfirstlane(a.rslab[strip * 2 + 1] - lo);
  const int chan = a.rstrip[strip * 4 + g];
  u32x4_t w[D][3];
  uint32_t ad[(D + 1) / 2];  // where a step's first fragment lies in the patch, two 16-bit numbers a word (in pieces)
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const uint32_t cs = (uint32_t)min(lo + d, a.ncs - 1);
    const uint32_t dv = *(const uint32_t*)(a.rdesc + (cs * 16u + (uint32_t)g * 4u));
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) w[d][dy] = *(const u32x4_t*)(a.rfrag + ((cs * 3u + (uint32_t)dy) * 1024u + (uint32_t)lane * 16u));
    const uint32_t v = ((uint32_t)(ct * 16 + c) + ((dv >> 8) & 0xFFu)) * (uint32_t)(a.pitch >> 4) + (dv & 0xFFu);
    if (d & 1)
      ad[d / 2] |= v << 16;
    else
      ad[d / 2] = v;
  }
  const uint32_t bias_at = bsp_bands_bias((uint32_t)a.bias_off, (uint32_t)wave, (uint32_t)g);
  if (c < 4) *(float*)(lds + bias_at + c * 4) = a.bias && chan >= 0 ? a.bias[chan + c] : 0.f;
  const uint32_t img = (uint32_t)(a.out_off + (ct * 16 + c) * a.opitch + (chan >= 0 ? chan * 2 : a.O * 2));

  // ---- the 16-byte pieces of output this lane stores for every tile: its column and piece are the same in all, the
  // rows lie two apart (two rows have as many pieces as the workgroup lanes, counting whole strips)
  constexpr int NIT = (BR + 1) / 2;
  uint32_t ocol, lsrc, gofs, orow;
  {
    const uint32_t px = fdiv((uint32_t)tid, a.d_cpp), k = (uint32_t)tid - px * (uint32_t)(a.nstrips * 2);
    orow = px >= (uint32_t)a.cw;
    ocol = px - orow * (uint32_t)a.cw;
    lsrc = (uint32_t)a.out_off + px * (uint32_t)a.opitch + k * 16u;
    gofs = (orow * (uint32_t)a.N + ocol) * (uint32_t)(a.O * 2) + k * 16u;
    if (k * 8u >= (uint32_t)a.O) ocol = 0x7FFFu;
  }
  auto out_at = [&](Tile t, int it) {
    const uint32_t base = (uint32_t)((t.n * a.M + t.y0 + 2 * it) * a.N + t.x0) * (uint32_t)(a.O * 2);
    const int left = min(a.M - t.y0, BR) - 2 * it;
    return (((int)orow < left) & (t.x0 + (int)ocol < a.N)) ? base + gofs : kNone;
  };
  u32x4_t res[RES ? NIT : 1];
  auto load_res = [&](Tile t) {
    if constexpr (RES) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) res[it] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, out_at(t, it), 0, 0));
    }
  };
  auto store = [&](Tile t, uint32_t ooff) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      u32x4_t v = *(const u32x4_t*)(lds + (ooff + lsrc + (uint32_t)(2 * it * a.cw * a.opitch)));
      if constexpr (RES) {
        const u32x2_t l2 = post_bf16x4_reg(u32x2_t{v.x, v.y}, u32x2_t{res[it].x, res[it].y}, true, a.relu);
        const u32x2_t h2 = post_bf16x4_reg(u32x2_t{v.z, v.w}, u32x2_t{res[it].z, res[it].w}, true, a.relu);
        v = u32x4_t{l2.x, l2.y, h2.x, h2.y};
      }
      __builtin_amdgcn_raw_buffer_store_b128(v, ydst, out_at(t, it), 0, 2);  // (streaming)
    }
  };

  f32x4_t acc[BR];
  // N steps of the strip: a step's fragments are read R patch rows ahead of their products
  auto products = [&](auto steps, uint32_t xoff) __attribute__((always_inline)) {
    constexpr int N = decltype(steps)::value, FR = BR + 2, R = 3;
    u32x4_t f[R + 1];
    auto read = [&](int s) __attribute__((always_inline)) {
      f[s % (R + 1)] = *(const u32x4_t*)(lds + (xoff + ((s / FR & 1 ? ad[s / FR / 2] >> 16 : ad[s / FR / 2] & 0xFFFFu) << 4) + (uint32_t)(s % FR * a.rowpitch)));
    };
#pragma unroll
    for (int s = 0; s < R; ++s) read(s);
#pragma unroll
    for (int s = 0; s < N * FR; ++s) {
      const int d = s / FR, fr = s % FR;
      if (s + R < N * FR) read(s + R);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
        if (fr - dy >= 0 && fr - dy < BR) acc[fr - dy] = mfma_bf16_16x16x32(w[d][dy], f[s % (R + 1)], acc[fr - dy]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto compute = [&](uint32_t xoff) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < BR; ++r) acc[r] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // straight code for every number of steps: a branch per step makes the compiler wait for each read
#define BANDS_STEPS(k) \
  case k:              \
    if constexpr (k <= D) products(std::integral_constant<int, k>{}, xoff); \
    break;
    switch (n) {
      BANDS_STEPS(1) BANDS_STEPS(2) BANDS_STEPS(3) BANDS_STEPS(4) BANDS_STEPS(5) BANDS_STEPS(6)
    }
#undef BANDS_STEPS
  };
  auto write_out = [&](uint32_t ooff) {
    const f32x4_t bv = *(const f32x4_t*)(lds + bias_at);
    auto out = [&](auto act) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < BR; ++r) {
        f32x4_t v = acc[r] + bv;
        // (a rounding does not move a sum past zero: without a residual the activation may come first)
        if constexpr (decltype(act)::value) v = f32x4_t{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
        *(u32x2_t*)(lds + (ooff + img + (uint32_t)(r * a.cw * a.opitch))) = u32x2_t{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
      }
    };
    if (!RES && a.relu)
      out(std::true_type{});
    else
      out(std::false_type{});
  };

  write_x(0);
  __builtin_amdgcn_s_waitcnt(0);  // the weights too: left to the loop, their waits would catch every tile's loads
  __syncthreads();
  uint32_t cur = 0;
  Tile prev{};
  for (int tile = first;; tile += a.groups) {
    const bool last = tile + a.groups >= end;
    const uint32_t oth = cur ^ 1u;
    const Tile next = locate(last ? tile : tile + a.groups);
    load_x(next, !last);  // (older than the stores: the wait for it leaves those under way)
    if (tile != first) store(prev, oth * (uint32_t)a.oslot);
    load_res(at);
    compute(cur * (uint32_t)a.slot);
    if (a.single) __syncthreads();
    write_out(cur * (uint32_t)a.oslot);
    if (!last) write_x(oth * (uint32_t)a.slot);
    __syncthreads();
    if (last) {
      store(at, cur * (uint32_t)a.oslot);
      return;
    }
    cur = oth;
    prev = at;
    at = next;
  }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

template <int D, int T, bool RES>
int launch_inst(const BandsArgs& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  static bool raised = false;  // dynamic LDS above 64 KB has to be allowed once per kernel
  if (!raised) {
    if (hipFuncSetAttribute((const void*)conv_bands<D, T, RES>, hipFuncAttributeMaxDynamicSharedMemorySize, kBandsLds) != hipSuccess)
      return BSP_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL((conv_bands<D, T, RES>), grid, dim3(threads), ldsb, st, a);
  return hipGetLastError() == hipSuccess ? BSP_OK : BSP_ERR_HIP;
}

template <int D, int T>
int launch_res(const BandsArgs& a, dim3 grid, int threads, size_t ldsb, hipStream_t st) {
  return a.residual ? launch_inst<D, T, true>(a, grid, threads, ldsb, st) : launch_inst<D, T, false>(a, grid, threads, ldsb, st);
}

}  // namespace

int bsp_launch_bands(const ConvParams& p, const void* plan_host, hipStream_t st) {
  if (!plan_host) return BSP_ERR_UNSUPPORTED;
  const int32_t* hdr = (const int32_t*)plan_host;
  if (hdr[BSP_PLAN_MAGIC_W] != BSP_PLAN_MAGIC || hdr[BSP_PLAN_VERSION_W] != BSP_PLAN_VERSION || hdr[BSP_PLAN_O_W] != p.O ||
      hdr[BSP_PLAN_I_W] != p.I || hdr[BSP_PLAN_H_W] != p.H || hdr[BSP_PLAN_K_W] != p.K || hdr[BSP_PLAN_DTYPE_W] != BSP_BF16 ||
      hdr[BSP_PLAN_OFF_ROWS_W] == 0)
    return BSP_ERR_UNSUPPORTED;
  const int32_t* rs = hdr + hdr[BSP_PLAN_OFF_ROWS_W];
  if (p.H != 3 || p.K != 3 || p.sh != 1 || p.sw != 1 || p.ph != p.pw || p.ph < 0 || p.ph > 1) return BSP_ERR_UNSUPPORTED;
  if (rs[BSP_ROWS_NSLABS_W] != 1 || rs[BSP_ROWS_CW_W] != 8 || rs[BSP_ROWS_NCS_W] < 1 || p.I > 128) return BSP_ERR_UNSUPPORTED;
  if ((int64_t)p.B * p.L * p.J * p.I * 2 >= (1ll << 31) || (int64_t)p.P * p.O * 2 >= (1ll << 31)) return BSP_ERR_UNSUPPORTED;
  if (p.L >= 0x7000 || p.J >= 0x7000) return BSP_ERR_UNSUPPORTED;
  const int nstrips = rs[BSP_ROWS_NSTRIPS_W], steps = rs[BSP_ROWS_MAXSTRIPSTEPS_W];
  BandsMap m{};
  if (!bsp_bands_map(p.I, p.N, p.O, nstrips, steps, &m)) return BSP_ERR_UNSUPPORTED;
  const int threads = 64 * m.waves, Jp = m.cw + 2;
  BandsArgs a{};
  a.cpx = m.cpx;
  a.pitch = m.pitch;
  a.rowpitch = m.rowpitch;
  a.pieces = m.pieces;
  a.ctiles = m.ctiles;
  a.cw = m.cw;
  a.nchunks = cdiv(p.N, a.cw);
  a.slot = m.slot;
  a.out_off = m.out_off;
  a.oslot = m.oslot;
  a.opitch = m.opitch;
  a.single = m.single;
  a.bias_off = m.bias;
  a.tpi = cdiv(p.M, BR) * a.nchunks;
  const int64_t tiles = (int64_t)p.B * a.tpi;
  if (tiles >= (1ll << 30) || tiles * std::max(a.tpi, a.nchunks) >= (1ll << 32) || (int64_t)QL * threads * std::max(a.cpx, Jp) >= (1ll << 32) ||
      (int64_t)threads * 2 * nstrips >= (1ll << 32))
    return BSP_ERR_UNSUPPORTED;
  a.tiles = (int)tiles;
  a.per_xcd = cdiv(tiles, 8);
  a.groups = std::min(a.per_xcd, 32 * m.resident);
  const double rounds = (double)tiles / (256 * m.resident);
#ifdef BSP_ROWS_TUNE  // experiments only: never defined in the product build
  if (const char* e = std::getenv("BSP_BANDS_TUNE")) {
    if (std::atoi(e) == 0) return BSP_ERR_UNSUPPORTED;
  } else
#endif
    if (!bsp_bands_beats(nstrips, steps, p.P, p.I, rounds)) return BSP_ERR_UNSUPPORTED;
  // (the any-shape kernel's layers stay there: it forms sums that are no finite number again from kept blocks)
  if (bsp_any_beats(p, plan_host, BSP_RIVAL_LDS)) return BSP_ERR_UNSUPPORTED;
  const int32_t* sec = p.plan + hdr[BSP_PLAN_OFF_ROWS_W];
  a.X = (const unsigned char*)p.X;
  a.Y = (unsigned char*)p.Y;
  a.bias = p.bias;
  a.residual = (const unsigned char*)p.residual;
  a.rstrip = sec + rs[BSP_ROWS_OFF_STRIP_W];
  a.rslab = sec + rs[BSP_ROWS_OFF_SLAB_W];
  a.rdesc = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_DESC_W]);
  a.rfrag = (const unsigned char*)(sec + rs[BSP_ROWS_OFF_FRAG_W]);
  a.relu = p.relu;
  a.nstrips = nstrips;
  a.ncs = rs[BSP_ROWS_NCS_W];
  a.xbytes = (int32_t)((int64_t)p.B * p.L * p.J * p.I * 2);
  a.ybytes = (int32_t)((int64_t)p.P * p.O * 2);
  a.L = p.L;
  a.J = p.J;
  a.M = p.M;
  a.N = p.N;
  a.O = p.O;
  a.pad = p.ph;
  a.d_cpx = make_fastdiv((uint32_t)a.cpx);
  a.d_jp = make_fastdiv((uint32_t)Jp);
  a.d_tpi = make_fastdiv((uint32_t)a.tpi);
  a.d_nchunks = make_fastdiv((uint32_t)a.nchunks);
  a.d_cpp = make_fastdiv((uint32_t)(nstrips * 2));
  a.d_ns = make_fastdiv((uint32_t)nstrips);
#ifdef BSP_ROWS_TUNE
  if (std::getenv("BSP_ROWS_VERBOSE"))
    fprintf(stderr, "bands: B=%d %dx%d %d->%d strips=%d steps=%d | CT=%d D=%d single=%d resident=%d tiles=%d rounds=%.3f lds=%d\n", p.B, p.L, p.J, p.I, p.O, nstrips,
            steps, m.ctiles, m.depth, a.single, m.resident, a.tiles, rounds, m.lds);
#endif
  dim3 grid((unsigned)(a.groups * 8));
  switch (m.depth) {
    case 3: return launch_res<3, 1024>(a, grid, threads, (size_t)m.lds, st);
    case 5: return launch_res<5, 768>(a, grid, threads, (size_t)m.lds, st);
    default: return launch_res<6, 768>(a, grid, threads, (size_t)m.lds, st);
  }
}
