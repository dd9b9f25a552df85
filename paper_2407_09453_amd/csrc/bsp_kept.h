// bf16 sums from kept blocks alone, for the kernels whose strips multiply a channel that one of their block rows
// keeps with zeros for those that drop it: what they do again where a sum came out as no finite number
// (library private).
#ifndef BSP_KEPT_H
#define BSP_KEPT_H

#include "bsp_device.h"

namespace {

typedef __attribute__((ext_vector_type(4))) int kept_i32x4_t;

// 16 bytes from any address (the hardware has no alignment rule for them)
__device__ __forceinline__ u32x4_t load16(const unsigned char* p) {
  u32x4_t v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
// drops the low n bytes (0 .. 15), zeros come in from above
__device__ __forceinline__ u32x4_t drop_low(u32x4_t v, int n) {
  if (n & 8) v = u32x4_t{v.z, v.w, 0u, 0u};
  if (n & 4) v = u32x4_t{v.y, v.z, v.w, 0u};
  const uint32_t b = (uint32_t)(n & 3) * 8u;
  return u32x4_t{__builtin_amdgcn_alignbit(v.y, v.x, b), __builtin_amdgcn_alignbit(v.z, v.y, b),
                 __builtin_amdgcn_alignbit(v.w, v.z, b), v.w >> b};
}
// The bytes [off, off + 16) of a pixel of `row` >= 16 bytes, zeros past its end; nothing outside the
// pixel is read.  The first half asks for them (a chunk that reaches past the end is read from 16
// bytes before it), the second puts them in place.
__device__ __forceinline__ u32x4_t piece_ask(const unsigned char* px, int off, int row) {
  return load16(px + min(off, row - 16));
}
__device__ __forceinline__ u32x4_t piece_place(u32x4_t v, int off, int row) {
  return drop_low(v, max(off - (row - 16), 0));
}

// The sums of one 16 x 16 tile (a strip, and one output pixel per lane column, whose window starts at
// iy0, ix0) from kept blocks alone.  A step of the plan multiplies a channel that one block row of the
// strip keeps with zeros for those that drop it, which an infinity or NaN turns into NaN; here every
// block row is summed by itself, with zeros for the channels that it drops.  Straight from
// memory, and bound by its chain of two loads per two steps: with a NaN in one image FC
// 64 x 2048 -> 1000 takes 33 us instead of 6.3, 3x3 14x14x256 batch 1 34 instead of 5.4, 3x3
// 47x33x100->76 batch 3 22 instead of 6.4.  Tiles of finite sums never come here; looking for the
// others costs at most 0.05 us a layer.
template <bool VEC, typename Args>
__device__ __forceinline__ f32x4_t kept_only(const Args& a, const unsigned char* xim, int strip, int iy0, int ix0, int lane) {
  constexpr int U = 2;
  const int g = lane >> 4, jn = lane & 15;
  const int32_t* plan = a.plan;
  const unsigned char* payload = a.payload;
  int HK = a.H * a.K, K = a.K, rowb = a.I * 2;
  // (in vector registers: the scalar ones are full of what the kernel still needs)
  asm volatile("" : "+v"(plan), "+v"(payload), "+v"(xim), "+v"(HK), "+v"(K), "+v"(rowb), "+v"(strip));
  const PlanView pv = plan_view(plan);
  const int c0 = pv.strip_ptr[strip], npairs = (pv.strip_ptr[strip + 1] - c0) * HK;
  const int bi = 64 >> a.lbo, mine = jn >> a.lbo, at0 = (jn & ((1 << a.lbo) - 1)) * HK;
  f32x4_t acc[BSP_MAXSUB] = {};
  for (int q = g; q < npairs + g; q += 4 * U) {
    u32x4_t w[U], x[U];
    kept_i32x4_t src[U];  // where the chunk's block lies in the payload, by block row; 4-wide blocks: its two halves'
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int pair = q + 4 * u, chunk = pair / HK, tap = pair - chunk * HK, th = tap / K, tw = tap - th * K;
      const int iy = iy0 + th, ix = ix0 + tw;
      w[u] = x[u] = u32x4_t{0u, 0u, 0u, 0u};
      src[u] = kept_i32x4_t{-1, -1, -1, -1};
      if (pair >= npairs) continue;
      const int xc = pv.chunk_xc[c0 + chunk];
      src[u] = *(const kept_i32x4_t*)(pv.chunk_src + (c0 + chunk) * BSP_MAXSUB);
      const int at = (at0 + tap) * bi;
      if (bi == 4) {
        u32x2_t lo = {0u, 0u}, hi = {0u, 0u};
        if (src[u].x >= 0) lo = *(const u32x2_t*)(payload + (int64_t)(src[u].x + at) * 2);
        if (src[u].y >= 0) hi = *(const u32x2_t*)(payload + (int64_t)(src[u].y + at) * 2);
        w[u] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
      } else {
        const int s = mine == 0 ? src[u].x : mine == 1 ? src[u].y : mine == 2 ? src[u].z : src[u].w;
        if (s >= 0) w[u] = *(const u32x4_t*)(payload + (int64_t)(s + at) * 2);
      }
      if ((unsigned)iy >= (unsigned)a.L || (unsigned)ix >= (unsigned)a.J) continue;
      const unsigned char* px = xim + (uint32_t)(iy * a.J + ix) * (uint32_t)rowb;
      x[u] = VEC ? *(const u32x4_t*)(px + xc * 16) : piece_place(piece_ask(px, xc * 16, rowb), xc * 16, rowb);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (bi == 4) {
        if (src[u].x < 0) x[u].x = x[u].y = 0u;
        if (src[u].y < 0) x[u].z = x[u].w = 0u;
        src[u].x = 0;
      }
      // (a block row's sums are taken from its own instruction, whatever the others made of them)
#pragma unroll
      for (int s = 0; s < BSP_MAXSUB; ++s)
        acc[s] = mfma_bf16_16x16x32(w[u], src[u][s] >= 0 ? x[u] : u32x4_t{0u, 0u, 0u, 0u}, acc[s]);
    }
  }
  const int row = 4 * g >> a.lbo;  // the lane's four channels lie in one block row
  return row == 0 ? acc[0] : row == 1 ? acc[1] : row == 2 ? acc[2] : acc[3];
}

}  // namespace

#endif
