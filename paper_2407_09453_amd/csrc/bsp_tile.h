// Pieces shared by the LDS-tiled bf16 kernels: tile geometry, cheap integer
// division, MFMA step helpers (library private).
#ifndef BSP_TILE_H
#define BSP_TILE_H

#include "bsp_device.h"
#include "bsp_fastdiv.h"

// (both words are read and the product is formed whatever the divisor: a select instead of a
// branch around a second load, which in a kernel's opening was one more wait for the scalar
// cache per division)
__device__ __forceinline__ uint32_t fdiv(uint32_t x, FastDiv f) {
  const uint32_t q = __umulhi(x, f.mul);
  return f.d == 1 ? x : q;
}

__device__ __forceinline__ uint32_t sdiv(uint32_t x, SmallDiv f) { return __umul24(x, f.mul) >> f.shift; }

// XCD: consecutive workgroups of a launch go to the eight XCDs in turn, and each of those has an L2 of its own (4 MB) that
// keeps its lines from one launch to the next.  So a layer's kernel gives XCD x the x-th eighth of the batch's pixels, in
// order, whatever it cuts them into: what the layer before wrote there lies in that L2 (the band kernel only where the batch
// is no multiple of eight).  (16.8 MB as 64 KB a CU, written by the launch before on the same XCD and on another: landed in
// LDS after 0.62 and 2.0 us; 33.6 MB 1.2 and 4.0.)

struct TileCfg {
  int32_t TH, TW;            // output tile, pixels
  int32_t TPH, TPW;          // staged input patch, pixels
  int32_t lsh, lsw;          // LDS pixels per output pixel step
  int32_t gsh, gsw;          // input pixels per LDS pixel step
  int32_t tiles_y, tiles_x;  // tiles per image
  int32_t row_bytes;         // LDS bytes per staged pixel (slab*2 + pad)
  int32_t pitch;             // LDS bytes per staged patch row (TPW*row_bytes + pad)
  int32_t tile2x8;           // 1: a 16-pixel tile is 2 rows x 8 columns, 0: 16 consecutive pixels
  int32_t slab, nslabs;      // channels per slab, slabs
  int32_t spc;               // strips per workgroup (4 when nslabs > 1)
  int32_t nstrips;
  int32_t ntiles;            // B * tiles_y * tiles_x
  FastDiv d_pp, d_tpw, d_tw, d_tpr, d_ntiles, d_tpi, d_tiles_x;
};

constexpr int kStageBatch = 8;  // 16-byte pieces a thread keeps in flight while staging
#ifndef BSP_WDEPTH
#define BSP_WDEPTH 8
#endif
constexpr int kWDepth = BSP_WDEPTH;  // weight fragments fetched ahead

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
// two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Four bf16 results (v) plus four residual values already in registers (r), the activation,
// one more rounding: post_bf16x4's arithmetic without a trip through memory.
__device__ __forceinline__ u32x2_t post_bf16x4_reg(u32x2_t v, u32x2_t r, bool has_r, int relu) {
  float f[4] = {bf16_bits_to_f32((uint16_t)(v.x & 0xFFFF)), bf16_bits_to_f32((uint16_t)(v.x >> 16)),
                bf16_bits_to_f32((uint16_t)(v.y & 0xFFFF)), bf16_bits_to_f32((uint16_t)(v.y >> 16))};
  if (has_r) {
    f[0] += bf16_bits_to_f32((uint16_t)(r.x & 0xFFFF));
    f[1] += bf16_bits_to_f32((uint16_t)(r.x >> 16));
    f[2] += bf16_bits_to_f32((uint16_t)(r.y & 0xFFFF));
    f[3] += bf16_bits_to_f32((uint16_t)(r.y >> 16));
  }
  if (relu) {
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = fmaxf(f[k], 0.f);
  }
  return u32x2_t{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])};
}

// Four int8 results from four exact sums: + 32-bit bias, rounding right shift (ties upward),
// saturation to [-128, 127], lowest channel in the lowest byte; nothing wraps.  Up to a shift of 24 a
// sum that leaves 32 bits saturates either way, so one saturating addition of the bias and half a unit (put
// together once for all of a strip's pixels), a shift and a median do, and the bytes are put together by
// permutes: fifteen instructions for four results.  (A bias within half a unit of the largest integer takes
// the 64-bit way.)  1x1 56x56x64->256 at batch 32, whose strips have one step, in the pointwise kernel: 16.5
// us with 64 bits, 15.6 with the rounding bit added by itself (twenty-eight instructions); that form and this one
// in turn on another box 14.0 and 12.8; all ResNet50-shaped layers 542 -> 524.
typedef __attribute__((ext_vector_type(4))) int acc_i32x4_t;
struct RescaleI8 {
  acc_i32x4_t bias, plus;  // plus: the bias and half a unit
  int shift;
  bool wide;
  __device__ __forceinline__ RescaleI8(acc_i32x4_t b, int s) : bias(b), shift(s) {
    const int half = s && s <= 24 ? 1 << (s - 1) : 0;
    bool near = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      near |= b[r] > 0x7FFFFFFF - half;
      plus[r] = (int)((uint32_t)b[r] + (uint32_t)half);
    }
    wide = s > 24 || __ballot(near) != 0;
  }
  __device__ __forceinline__ uint32_t operator()(acc_i32x4_t sum) const {
    int q[4];
    if (!wide) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v = __builtin_elementwise_add_sat(sum[r], plus[r]) >> shift;
        q[r] = min(max(v, -128), 127);
      }
    } else {
      const long long half = shift ? 1ll << (shift - 1) : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long long w = ((long long)sum[r] + bias[r] + half) >> shift;
        q[r] = w < -128 ? -128 : (w > 127 ? 127 : (int)w);
      }
    }
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], 0x04000c0cu);
    return lo | hi;
  }
};

// The activations one step needs: every pixel tile of the wave reads its 16
// bytes at the offset the step's descriptor d (chunk, tap) selects.
template <int NT>
__device__ __forceinline__ void load_b(u32x4_t (&b)[NT], const int d, const unsigned char* lds,
                                       const int (&base)[NT], const int pitch,
                                       const int row_bytes) {
  const int xoff = ((d >> 16) & 0xFF) * pitch + ((d >> 24) & 0xFF) * row_bytes + (d & 0xFFFF) * 16;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) b[nt] = *(const u32x4_t*)(lds + base[nt] + xoff);
}
template <int NT>
__device__ __forceinline__ void do_mma(f32x4_t (&acc)[NT], const u32x4_t a,
                                       const u32x4_t (&b)[NT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma_bf16_16x16x32(a, b[nt], acc[nt]);
}


// Pick the output tile for a layer (most useful pixels per MFMA pixel slot,
// least halo, no LDS bank conflicts) and the LDS paddings; false if nothing fits
// in max_lds bytes.  Fills everything in *out except spc, ntiles and the dividers.
// The tile holds nt_scale * NT pixel tiles (nt_scale waves share a strip) and the LDS
// budget also has to cover out_row_bytes per output pixel (results staging), if any.
bool bsp_choose_tile(const ConvParams& p, int slab, int64_t max_lds, int max_pieces, int nt_scale,
                     int out_row_bytes, int min_nt, int slots, int* NT, TileCfg* out);

#endif
