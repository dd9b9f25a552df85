// Where the kernel that streams bands past weights in registers (bsp_bands.hip) keeps what in LDS (library private; plain
// C++, also compiled on the host by the tests): patches of the input, images of the output, biases.
#ifndef BSP_BANDS_MAP_H
#define BSP_BANDS_MAP_H

#include <stdint.h>

constexpr int kBandsRows = 4;        // output rows of a tile
constexpr int kBandsPieces = 4;      // pieces of input a lane brings for a tile
constexpr int kBandsLds = 160 * 1024;

struct BandsMap {
  int32_t ctiles, cw, waves;         // column tiles and columns of a tile; waves of a workgroup
  int32_t depth;                     // most steps that the instance holds
  int32_t cpx, pitch, rowpitch, pieces;  // 16-byte pieces of a pixel; LDS bytes of a staged one and of a staged row; pieces of a patch
  int32_t patch, opitch, image;      // LDS bytes of a patch, of a pixel of an image, of an image
  int32_t single, resident;          // one patch and one image instead of two; workgroups that a CU holds
  int32_t slot, out_off, oslot, bias, lds;
};

// I, N, O: channels in, output columns, channels out.  False: a layer that the kernel does not hold.
constexpr bool bsp_bands_map(int I, int N, int O, int nstrips, int steps, BandsMap* m) {
  auto least = [](int x, int y) { return x < y ? x : y; };
  if (nstrips < 1 || nstrips > 16 || steps > 6) return false;
  m->cpx = I / 8;
  m->pitch = (m->cpx | 1) * 16;  // an odd number of pieces: no two pixels of a lane tile share banks
  m->opitch = O * 2 + 16;
  // one column tile, more where fewer than four strips make a workgroup of four waves of them
  const int most = least(4 / nstrips, (N + 15) / 16);
  m->ctiles = most < 1 ? 1 : most;
  m->cw = 16 * m->ctiles;
  m->waves = nstrips * m->ctiles;
  // waves per SIMD that the registers of the instance for so many steps allow; a workgroup's waves are dealt over the
  // four SIMDs from the first one on
  m->depth = steps <= 3 ? 3 : steps <= 5 ? 5 : 6;
  const int held = (m->depth <= 3 ? 4 : 3) / ((m->waves + 3) / 4);
  if (held < 1) return false;
  m->rowpitch = (m->cw + 2) * m->pitch;
  m->pieces = (kBandsRows + 2) * (m->cw + 2) * m->cpx;
  if (m->pieces > kBandsPieces * 64 * m->waves) return false;
  // two patches and two images of the output in turn, so that one barrier ends a tile; one of each, and a second
  // barrier, where a CU then holds more workgroups
  m->patch = (kBandsRows + 2) * m->rowpitch;
  m->image = kBandsRows * m->cw * m->opitch;
  const int fixed = m->waves * 64;
  auto resident = [&](int sets) { return least(held, kBandsLds / (sets * (m->patch + m->image) + fixed)); };
  m->single = resident(1) > resident(2);
  const int sets = m->single ? 1 : 2;
  m->resident = resident(sets);
  if (m->resident < 1) return false;
  m->slot = m->single ? 0 : m->patch;
  m->out_off = sets * m->patch;
  m->oslot = m->single ? 0 : m->image;
  m->bias = sets * (m->patch + m->image);
  m->lds = m->bias + fixed;
  return true;
}

// The pieces that a lane brings: only the first `pieces` of the workgroup's are some, the others are not written.
constexpr bool bsp_bands_some(int index, int pieces) { return index < pieces; }

// Where a wave's four lane groups keep four biases each.
constexpr uint32_t bsp_bands_bias(uint32_t bias, uint32_t wave, uint32_t group) { return bias + (wave * 4 + group) * 16; }

#endif
