// Where the any-shape kernels and a specialised one both take a layer: which of the two runs it
// (library private; plain C++, also compiled on the host by the tests).
//
// A specialised kernel shares a patch or a weight fragment among more products, which pays once the
// chip is full of work; the any-shape one splits small layers finer (pixels, strips, contraction) and
// has the shorter opening.  The lines were drawn by timing both sides on 3800 layers (the networks' and
// random ones), along the matrix instructions of a layer (mm) and its results (po).  The last numbers
// of each entry are `the other / here` in microseconds, on either side of a line.
#ifndef BSP_RULES_H
#define BSP_RULES_H

#include <stdint.h>

enum BspRival { BSP_RIVAL_BAND, BSP_RIVAL_ROWS, BSP_RIVAL_LDS, BSP_RIVAL_TILE };

// bf16 windows: whether the any-shape kernel is to take the layer that `rival` could take (bo: output
// channels per block).
//   one row, row-band kernel: 1x7 17x17x160->192 batch 16 (100 861) 10.2 / 9.0, 17x17x192 batch 32 (220 218)
//     17.5 / 13.9, 57x57x272->192 batch 4 (252 030) 19 % slower here; more than 208 channels in: 29x29x456->168 batch 4 (188 845)
//     16.6 / 14.2, cold 17.9 / 17.6, 33x33x296->384 batch 2 (166 729) 14.5 / 9.6, 32x19x264->168 batch 9 (164 160) 11.3 / 12.0 the other
//     way, as 13x18x384->176 batch 16 (216 216, past the line), 1.05 to 1.14; with 16x4 blocks no line, 36x36x160->184 batch 31 (1.05 M) 66 / 40
//   one row, LDS kernel: 1x7 31x13x248->80 (32 382) 19.8 / 7.0; 37x37x32->184 batch 28 (201 264)
//     13.2 / 16.4; 1x3 98x32x8->144 batch 21 (37 044, po 9.5 M) 13.5 / 18.5; strided ones have no line
//   one column: 7x1 22x22x192->104 batch 8 (62 920) 9.4 / 7.8, 17x17x160->192 batch 16 (97 K) 10.0 / 9.5,
//     68x6x152->200 batch 11 (91 887) 9.4 / 11.0; 3x1 24x27x184 batch 20 (94 K) 11.5 / 11.6
//   3x3, band kernel: 56x56x64 batch 1 (14 112, po 201 K) 5.8 / 5.1; 35x35x64->96 batch 4 (28 244, po
//     470 K) 5.4 / 5.9
//   3x3, the others: 10x10x112->336 batch 5 (15 904) 8.6 / 5.4; 111x11x40->16 batch 30 (20 610) 5.6 / 6.9;
//     stride 2 35x35x72->224 batch 7 (58 424) 14.3 / 10.2, 39x39x8->160 batch 21 (59 910, po 5.1 M) 8.4 / 14.0
//   one column, row-band kernel, 8x8 blocks, more than 32 channels: 284 layers; 3x1 8x8x384 batch 16 (44 K) 8.5 / 6.5, 35x35x488->88 batch 3
//     (63 480, 3675 pixels) 0.54, 12x12x384->280 batch 15 (69 120, 2160) 1.12 the other way; past 5000 pixels as many lose as gain
//     (28x28x216->64 batch 18, 74 088, 1.24); strided ones 1.1 to 2.3 times faster here, all 92 up to 340 K
//   larger windows, row-band kernel (three or seven rows): 3x5 13x13x184->24 batch 8 (6 860) 8.8 / 5.3,
//     34x11x168->24 batch 27 (99 856) 7.9 / 14.4; 7x7 11x9x144->8 batch 6 (3 268) 8.0 / 5.8,
//     18x10x288->112 batch 15 (489 086) 16.5 / 31.5
//   larger windows, LDS kernel: 5x5 50x26x40->8 batch 7 (18 208) 11.3 / 6.4, with 4x16 blocks
//     73x73x24->32 batch 5 (63 308) 7.0 / 8.6, 7x7 64x48x8->152 batch 32 (638 976) 23 / 51
//   larger windows, ring-tile kernel: 5x5 25x25x248->16 batch 3 (po 30 K) 43 / 8.3, 85x85x16->448 batch 3
//     (po 9.7 M) 15.3 / 21.8; 7x7 32x32x232->32 batch 4 (po 131 K) 66 / 13, 37x8x64->144 batch 27 (po
//     1.2 M) 18.7 / 24.2
inline bool bsp_any_beats_bf16(BspRival rival, int bo, int H, int K, bool strided, int64_t mm, int64_t po, int64_t I, int64_t O) {
  if (H == 1 && K == 1) return rival == BSP_RIVAL_TILE;
  if (H == 1) {
    if (rival == BSP_RIVAL_ROWS) return bo == 16 || mm <= (I <= 208 ? 240000 : 200000);
    return rival == BSP_RIVAL_TILE || strided || (mm <= (bo == 16 ? 1000000 : 120000) && po <= 4000000);
  }
  if (K == 1) {
    if (rival == BSP_RIVAL_TILE) return true;
    if (H <= 3 && rival == BSP_RIVAL_ROWS && strided) return mm <= 340000 && po <= 10000000;
    if (H <= 3) return mm <= (rival == BSP_RIVAL_ROWS && bo == 8 && O > 32 && po <= 5000 * O ? 80000 : 45000) && po <= 4000000;
    if (rival == BSP_RIVAL_ROWS) return strided || mm <= 100000;
    return (mm <= 100000 && po <= 4000000) || (strided && po <= 10000000);
  }
  if (H <= 3 && K <= 3) {
    if (rival == BSP_RIVAL_TILE) return true;
    if (rival == BSP_RIVAL_BAND) return mm <= 25000 && po <= 250000;
    return mm <= (strided ? 60000 : 30000) && po <= 3000000;
  }
  if (rival == BSP_RIVAL_ROWS) return H <= 3 ? mm <= 80000 && po <= 300000 : mm <= 30000;
  if (rival == BSP_RIVAL_LDS) return mm <= (bo == 4 ? 25000 : 80000) && po <= 3000000;
  return H * K <= 25 ? O < 272 || po <= 1000000 : O < 136 || po <= 800000;
}

// 3x3 windows past those lines: whether the two kernels' own models of the layer decide between the any-shape and the row-band
// kernel, and how (`any`: clocks of the busiest CU, `rows`: rough ns).  Neither model knows the other's scale, and the row-band
// one gives 1.12 to 2.0 times what it takes (550 layers), so the line is a ratio, drawn where few lose.  Of 4966 random layers of at least
// 128 channels in, with data in the caches, with cold weights and with all data cold, those past the lines above:
//   stride 1, up to 8000 pixels (6500 of up to 64 channels out) and 115 K, of few pixels 200 K: 1177 of 2762 are taken, 0.78 of their time in
//     the mean; 37 lose more than 5 % somewhere (the worst 55x55x376->72 batch 2 1.29 to 1.36, 11x11x136->176 batch 25, dense, 1.25 to
//     1.35, 18x24x224->144 batch 8 1.25 to 1.28).  By matrix instructions, channels and rows alone 1234 were taken, 0.80, 108 of
//     them at a loss (cold 15x11x480->136 batch 11 11.0 / 14.7, 24x24x392->88 batch 6 10.3 / 13.0, 35x35x176->488 batch 2 9.8 / 12.0)
//   stride 2, more than 40 channels out, up to 300 K: 294 of 607, 0.755 of their time, 19 lose more than 5 % (47x47x416->56 batch 20 1.55
//     to 1.65, 45x50x448->72 batch 5 1.37 to 1.46; by lines alone 368, 0.84, 79 at a loss, cold 52x52x368->32 batch 17 16 / 30).  To 140 K
//     and past 72 channels out the ratio is another: there the row-band kernel is seldom the faster one (17x17x192->320 batch 16 11.0 / 8.1)
//   Left behind: 33x30x264->104 batch 4 of dense 16x4 blocks 0.40, stride 2 43x48x304->40 batch 12 0.42 to 0.48
inline bool bsp_any_models_decide(int H, int K, bool strided, int64_t mm, int64_t P, int64_t O) {
  if (H > 3 || K > 3 || H == 1 || K == 1 || P * O > 3000000) return false;
  return strided ? mm <= 300000 && O > 40 : mm <= (P <= 1500 ? 200000 : 115000) && P <= (O <= 64 ? 6500 : 8000);
}
inline bool bsp_any_model_beats(bool strided, int64_t mm, int64_t O, double any, double rows) {
  return any < (!strided ? 3.3 : mm <= 140000 && O > 72 ? 2.6 : 2.1) * rows;
}

// bf16 layers on the any-shape kernel: whether results leave straight from the accumulators, eight bytes a lane (po: results).
// That saves a barrier and the way through LDS; past some size an image's whole lines are worth more, and a narrow layer's
// pixels are part lines anyway.  1470 random layers, the geometric mean of direct / image (the slowest of a class):
//   fewer than 64 channels: 20 to 160 K results 0.94 to 0.96 (1.00), 160 to 200 K 0.96 (1.09; 40 channels), 320 to 460 K 1.01
//     (1.19), 460 K and more 1.03 (1.21; 3x1 50x50x64->48 batch 4 5.11 / 5.47 us)
//   others: 20 to 200 K 0.94 to 0.97 (1.00), 320 to 400 K 0.96 (1.03), 460 K and more 0.99 (1.09); 2.5 MB, 5x5 35x35x48->64
//     batch 16, 9.80 us through the image, 10.05 direct
// Instances of their own: with the choice made in the kernel the others paid for its registers and code, 3x1 82x108x43->347
// batch 3 16.6 -> 17.4 us.  (The entry points take results and residuals at multiples of 16 bytes only.)
inline bool bsp_any_direct(int64_t O, int64_t po) { return O % 4 == 0 && po <= (O < 64 ? 160000 : 400000); }

// bf16 windows of three rows at stride 1: whether the persistent kernel takes a layer from `rival`.  mr: matrix
// instructions of the row-band section's steps; cost: the two kernels' own models of a layer, which put
// the persistent one at 0.95 (0.85 to 1.10) of what it takes and the row-band kernel at 1.47 times (1.12 to 2.0)
// (rival / here in us, from 550 random layers):
//   row-band kernel, more than 128 channels in: 58x76x544->336 batch 3 71 / 29, 56x56x256 batch 16 47 / 42,
//     28x28x512 batch 16 52 / 40, 28x28x256->512 batch 16 27 / 24; 17x17x256->296 batch 4 10.4 / 12.7, 34x34x520->64
//     batch 6 14.3 / 18.2.  At this line 1 of 120 taken layers is more than a tenth slower (0.85), and the
//     geometric mean of the taken ones is 1.29 times faster.
//   band kernel: never; its workgroups stage whole lines, 73x73x80->192 batch 16 26 / 36 (bsp_bands_beats gives it to the
//     kernel that streams bands), 56x56x128->256 batch 16 26.9 / 27.9 (76x76x112->208 batch 3 30 / 17 is an exception)
//   LDS kernel (more strips than the band kernel has waves, 4-channel blocks, other widths): 104x104x72->344
//     16x4 blocks batch 9 98 / 61, 52x52x72->432 batch 10 39 / 29; 33x33x64->448 16x4 batch 10 14.6 / 15.7 (not
//     thinner pixels or fewer strips, most of which the kernel that streams bands takes before either)
//   Below 20 K matrix instructions a full chip's opening is longer than the layer.
inline bool bsp_tall_beats(BspRival rival, int64_t mr, int64_t I, int64_t O, double cost, double rows_cost) {
  if (mr < 20000) return false;
  if (rival == BSP_RIVAL_ROWS) return I > 128 && cost < 1.35 * rows_cost;
  return rival == BSP_RIVAL_LDS && I >= 64 && I <= 128 && O > 64 && mr > 120000;
}

// bf16, up to 64 pixels and short rows: staged once and split over strips and contraction (7x7x2048->512
// 9.0 -> 6.5 us, FC 64 x 2048 -> 1000 10.1 -> 6.8; from 17 pixels with 4x16 blocks, 7.7 -> 6.7; from
// 24 to 32 with 8x8 blocks, whose streaming kernel takes 6.0 against 6.5 at 17 and 7.2 against 6.5
// at 32; where the weights are the bulk the streaming kernels stay ahead: long rows, and with 4x16 and
// 16x4 blocks as many strips as there are CUs or somewhat fewer, 33 x 2048 -> 4096 8.7 there against
// 12.8, 52 x 1864 -> 3346 9.4 against 11.5).
inline bool bsp_any_few(int bo, int64_t P, int64_t I, int64_t O, bool pointwise) {
  if (P <= (bo == 8 ? 28 : 16) || P > 64 || I > 2048) return false;
  return !(pointwise && bo != 8 && P > 32 && O <= 4096 && I * O > 4400000);
}

// 1x1 layers of up to 64 pixels, stride 1 or more: the pointwise kernel, which copies a pixel tile's whole rows into LDS
// and walks each strip's weights behind one wait, against the kernels below it (streaming FC and any-shape in
// bf16).  The call costs a launch, two memory latencies and the tile's copy; the copy grows with I, and from
// some length on the streaming kernels' split of it is worth more.  Other us / pointwise us:
//   8x8   1 x 512 -> 4096 4.4 / 4.1, 16 x 64 -> 1000 4.1 / 3.4, 49 x 512 -> 2048 5.0 / 4.4; past 512 channels
//         only from 17 pixels: 28 x 1024 -> 1000 1.23x, 64 x 1280 -> 4096 1.43x, 1 x 1024 0.93x, 32 x 2048 -> 256 0.94x
//   4x16  1 x 512 -> 1000 1.28x, 8 x 1280 -> 1000 1.06x, 1 x 2048 -> 256 0.89x; from 8192 channels out 1.4x to 2.5x
//         whatever the length; past 16 pixels 512 channels 1.02x to 1.26x, 32 x 1024 -> 256 0.97x, -> 4096 1.09x
//   16x4  to 16 pixels 1.3x to 3x; past them 512 -> 1000 1.01x, 1024 -> 1000 0.97x, 1024 -> 4096 1.06x
inline bool bsp_pw_few_beats(int bo, int64_t P, int64_t I, int64_t O) {
  if (I <= 512) return true;
  if (I > 2048) return false;
  if (bo == 8) return P > 16 && I <= 1280;
  if (bo == 4) return P <= 16 ? I <= 1280 || O >= 8192 : I <= 1280 && O >= 4096;
  return P <= 16 || O >= 4096;
}

// The same in int8, against the any-shape kernel: 1.05x to 1.35x for up to 1024 channels (1 x 256 -> 256
// 1.31x, 49 x 512 -> 2048 1.29x, 64 x 1024 -> 1008 1.07x); 2048 -> 1008 0.92x, 2048 -> 4096 0.99x to 1.31x.
inline bool bsp_pw_few_beats_i8(int64_t I, int64_t O) { return I <= 1024 || (I <= 2048 && O >= 4096); }

// 1x1 layers: whether the kernel that streams the pixels past weights in registers takes the layer from the pointwise one.
// rounds: tiles of 32 pixels (16 where a strip has more than eight steps), times groups of strips, for each workgroup
// the chip holds.  Its opening brings every weight into registers before the first product, which two rounds pay for;
// below that a workgroup for each tile is over sooner.  8900 random layers with cold data, the geometric mean of
// pointwise / here in each class:
//   bf16, more than 8 strips: up to 2 steps 0.95 to 1 round, 0.98 to 1.02 to 2, 1.03 to 3, 1.10 past that, 3 or 4 steps 0.92, 0.96
//     to 0.99, 1.18, 1.15 to 1.30, 5 to 8 steps 0.93, 0.97 to 1.02, 1.21, 1.17 to 1.36; 9 to 16 steps 0.91, 0.92, 1.08, 1.02 to
//     4 (a third of them slower), 1.26 past that; 5 to 8 strips alike, but 9 to 16 steps 1.21 from 2 rounds on
//   up to 4 strips: up to 2 steps 0.97 to 1.02 however many rounds (64->64 on 100352 pixels 7.1 / 7.8), longer ones 1.03 to
//     1.20 from 2 rounds on, 9 to 16 steps 0.93 to 4 rounds, 1.08 to 1.15 past that; with their data in the caches, as a
//     layer has it from the one before, 0.92 to 0.96 from 2 to 3 rounds (256->64 on 19881 pixels 5.2 / 5.8), 0.84 to 1.17 to 4,
//     1.07 to 1.34 past that
//   more than 8 strips of up to 2 steps with their data in the caches: without a residual alike; with one, in the stack of a
//     ResNet50, 0.87 to 0.95 to 3.5 rounds (64->256 on 28224 pixels 6.4 / 7.6), 0.82 to 1.06 to 7 (on 39168 9.0 / 10.9), 1.00
//     to 1.07 past that, and with cold data 0.99 to 1.08 to 7 rounds
//   int8, more than 4 strips: 1 step 0.93 to 0.98 to 1.5 rounds, 1.15 to 1.38 past that in the stack of a ResNet50 (64->256 on
//     25600 pixels 6.1 / 5.1), 1.06 to 1.39 cold; 2 steps 0.94 to 1.04 to 3 rounds in the stack (128->512 on 11200
//     pixels 5.0 / 5.3), 0.92 to 1.20 cold, 1.04 to 1.24 and 1.00 to 1.21 past that; 3 or 4 steps and more
//     than 8 strips 0.94 to 1.05 and 0.94 to 1.06 to 3 rounds, 1.11 to 1.33 past that; up to 8 strips 0.86 to 1.00 and 0.94 to
//     0.95 to 2 rounds, 1.01 to 1.05 and 0.96 to 1.06 to 3; 5 to 8 steps 0.86 to 1.05 to 2 rounds, 1.13 to 1.32 past that; up to 4
//     strips 0.84 to 1.00 (0.84 to 0.95 cold); 9 to 16 steps 0.98 to 1.03 (0.84 to 1.1), left where they are
// 256->128 on 100352 pixels 25.7 / 18.0 us, 64->256 with a residual 26.0 / 24.2, in int8 13.4 / 9.2.
inline bool bsp_pws_beats(bool i8, int64_t strips, int64_t steps, bool residual, double rounds) {
  if (i8) return strips > 4 && steps <= 8 && rounds > (steps <= 1 ? 1.5 : steps == 2 || (steps <= 4 && strips > 8) ? 3 : 2);
  if (strips <= 4 && steps <= 2) return false;
  return rounds > (strips <= 4 || (strips > 8 && steps > 8) ? 4 : strips > 8 && steps <= 2 ? (residual ? 7 : 3.2) : 2);
}

// The workgroups of that kernel that the chip holds (waves and bytes of LDS of each): 16 waves a CU, fewer where LDS is
// short.  More than are held open twice: 512->128 at a tenth of the blocks (84480 bytes) on 42496 pixels 15.8 us instead of 14.8, on
// 57344 19.3 instead of 17.5.  (The rounds above count 16 waves whatever the LDS.)
inline int bsp_pws_held(int waves, int64_t lds) {
  const int64_t fit = 160 * 1024 / lds;
  return 256 * (int)(fit < 16 / waves ? fit : 16 / waves);
}

// 3x3 layers at stride 1 of at most 128 channels in: whether the kernel that streams bands past weights in registers takes
// the layer from the band and LDS-resident kernels.  rounds: tiles for each workgroup the chip holds.  900 random layers
// with cold data and with data in the caches, the other / here in us; below 4000 pixels 0.98 (long strips 0.64 to 0.9:
// every workgroup waits for all its weights before its first product).  Of 420 more, from 4000 pixels on, 145 are taken: 1.70
// times faster cold, 1.68 in the caches, three of them 5 to 8 % slower.
//   LDS kernel: 149x149x32 batch 16 27.2 / 14.4, 147x147x32->64 29.6 / 19.1, 97x83x72->104 batch 5 15.4 / 10.7
//   band kernel, more than 8 strips: 73x73x80->192 batch 16 28.2 / 23.2, 83x83x64->144 batch 28 81 / 53, but 0.91 to 1.0
//     below one round (37x37x48->184 batch 3 7.0 / 7.7)
//   up to 8 strips of more than three steps: past four rounds 224x224x64 batch 16 66.7 / 51.0, 112x112x64->128 31.2 / 29.5,
//     137x143x88->120 35.4 / 34.7; below them the same time (35x35x64->96 batch 16 7.4 / 7.6, 53x53x72->88 15.6 / 16.5), but
//     up to 4 strips to one and a half 56x56x64 batch 4 5.9 / 5.2, batch 9 7.8 / 6.2, batch 16 8.5 / 7.7 (batch 24 9.0 / 9.4)
//   more than six steps leave registers for two waves a SIMD: 56x56x128 batch 6 11.1 / 11.9, 28x28x128 batch 32 10.4 / 11.9
inline bool bsp_bands_beats(int64_t strips, int64_t steps, int64_t P, int64_t I, double rounds) {
  if (P < 4000 || steps > 6 || (strips > 8 && steps > 3 && rounds < 1)) return false;
  if (I >= 64 && strips <= 8 && steps > 3) return rounds >= 4 || (strips <= 4 && rounds <= 1.5);
  return true;
}

// int8 against the LDS-resident kernel, which keeps one slab's weights in LDS.  One slab (other us /
// any-shape us): below 20 K matrix instructions, 1x1 56x56x64->256 batch 2 6.4 / 5.0, batch 32 21 / 31.
// Several slabs: always for a window, 7x7x512 batch 32 15.2 / 11.5, 2x2 47x47x208->32 batch 61 21 / 14, 25x25x624->192
// batch 29 41 / 35 (a few of many channels out go the other way, 28x28x512 batch 16 49 / 52, 3x1 73x73x192->160
// batch 59 99 / 121, but their neighbours do not, 23x23x624->416 batch 37 102 / 73, 62x62x208->176 batch 45 57 /
// 53).  Not narrow 1x1 layers of large images (pixels times an image's pixels past 2^32, the pointwise kernels have the others):
// 600x600x640->16 57 / 95, ->32 58 / 69, ->48 62 / 62, 300x300x640->16 23 / 17.
inline bool bsp_any_beats_lds_i8(int nslabs, int64_t HK, int64_t P, int64_t O, int64_t mm) {
  if (nslabs == 1) return mm <= 20000;
  return HK > 1 || O >= 48 || P <= 100000;
}

// int8, layers of no other kernel (32-bit results, or channels that are not whole pieces): one or two
// products per pixel tile are over before a patch is staged (general / any-shape us: 16->16 on 6840 pixels
// 3.2 / 4.0, 24->40 on 6647 3.3 / 4.0; three products, 40->504 on 246, are 3.4 / 4.0 at the worst and even
// on the whole).  Many results leave better through the any-shape kernel's LDS image (16->32 on 114308
// 9.4 / 7.8) but for very many of whole rows (16->592 on 113535 62 / 82, 32->432 on 83810 32 / 41, 32->384 on
// 31000 16.8 / 16.2).  Channels in that are not whole eights are loaded one by one in the general kernel:
// two products 0.88 times its time, three 0.75.
inline bool bsp_i8_general(int64_t I, int64_t O, int64_t HK, int64_t po) {
  if (HK != 1 || I > 32 || I % 8) return false;
  return po <= 1000000 || (O % 16 == 0 && po > (I <= 16 ? 5000000 : 20000000));
}

// Pointwise kernel, int8 layers of one to three strips: lane tiles per wave.  A workgroup is as few waves
// as strips and keeps its pixels in LDS, so that a wide tile leaves a CU with hardly a wave to ask for the
// next one: tiles of 64 pixels stay while a CU holds 13 waves with them, of 32 while it holds 12 (64, 32
// and 16 pixels, in brackets the LDS-resident kernel: 112x112x288->16 batch 16 21.0 / 15.1 / 14.4 (15.6),
// 1008->16 58 / 44 / 36 (38), 1008->32 48 / 40 / 34 (39), 512->32 24.1 / 20.8 / 19.4 (20.1), 512->48 22.5 /
// 20.2 / 21.8 (20.6), 144->32 9.1 / 8.4 / 12.0 (12.8), 144->48 9.7 / 10.8 / 16.4 (13.7)).
inline int bsp_pw_thin(int PT, int64_t pitch, int NS) {
  auto waves = [&](int pt) { return 160 * 1024 / (16 * pt * (pitch + NS * 16 + 16)) * NS; };
  if (PT == 4 && waves(4) < 13) PT = 2;
  if (PT == 2 && waves(2) < 12) PT = 1;
  return PT;
}

// Pointwise kernel: tile of a layer of P pixels, I pairs of bytes per pixel in (2-byte channels, or pairs of codes) and O channels out (int8:
// any large number), pitch bytes per staged pixel; windowed: the plan keeps the strips in fours of neighbours.
//
// One pixel group; four lane tiles a wave unless the tile's channels then exceed 128 KiB of LDS; few strips per workgroup
// while pixels are plentiful or the tile is thin (many small workgroups hide each other's latencies), many when they are not (every
// strip group re-reads the tile from L2, which is what bounds deep layers).
//
// Then enough waves for the chip.  With fewer than five a CU, two lane tiles (and half as many pixels to stage) beat four by 0.3
// to 0.5 us (35x35x192->64 batch 16 4.65 -> 4.31, 14x14x512 batch 8 4.95 -> 4.51, 28x28x256->128 batch 8 4.26 -> 3.86; with six a CU
// 14x14x1024->256 batch 32 7.19 / 7.99), of many strips by more (18x18x1536->1504 int8 batch 2 10.4 -> 6.3), with fewer than two a CU one beats two (8x8x2048->192 batch 16
// 6.29 -> 5.36, with three 2048->384 6.52 / 7.09).  Eight strips share a tile then where they come in eights; where they do
// not, a tile that several workgroups stage stays wide on many pixels (9 strips, 20x20x936->136 batch 19 6.9 / 8.8; 17 strips,
// 28x28x800->272 batch 5 6.3 / 7.8) but not on few (15 strips, 12x12x888->232 batch 31 11.1 / 8.5).  Thinner tiles go by their number
// alone (56x56x64->256 batch 1 3.27 -> 3.03).  The line at five waves a CU over 2500 layers between one and eight, cold data, with all of this / four lane
// tiles or fewer strips: geometric mean 0.983; 38 layers gain a quarter or more, 9 lose 5 to 11 %, all within a tenth of the line
// (dense 32x32x376->120 batch 9 6.7 / 7.5, 25x25x288->272 stride 2 batch 28 5.4 / 5.9, int8 21x21x880->128 batch 22 7.4 / 7.9).
//
// Whole-line output for layers that widen (their output is the bulk of the traffic), and for narrowing ones whose channels come
// in eight strips, two whole lines of a pixel, where a CU holds as many workgroups with the image (cold 25x25x648->512 batch 6 9.0
// -> 8.4; 42 strips, 11x11x712->664 batch 17 7.0 / 7.9; 9 strips, 37x37x688->144 batch 8 8.8 / 9.4; 504 channels, 38x38x1360
// stride 2 batch 5 8.0 / 8.5).
struct BspPwChoice {
  int PT, PG, NS;
  int wout;      // results leave through an LDS image of whole output lines
};
inline BspPwChoice bsp_pw_choose(int64_t P, int I, int O, int nstrips, int pitch, bool windowed, bool i8) {
  constexpr int64_t lds = 160 * 1024;
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  auto least = [](int a, int b) { return a < b ? a : b; };
  BspPwChoice c{4, 1, 1, 0};
  while (c.PT > 1 && 16 * c.PT * pitch > 128 * 1024) c.PT /= 2;
  int ns = least((P >= 50000 || (I <= 128 && P >= 20000)) ? 4 : (I >= 512 ? 16 : 8), nstrips);
  if (ns >= 4) ns &= ~3;
  c.NS = ns > 1 ? ns : 1;
  const int64_t tiles = cdiv(P, 64);
  const bool few = tiles < 96 && nstrips <= 16;
  if (pitch > 128 && P > 64) {
    const int two = nstrips <= 8 ? nstrips : nstrips % 8 == 0 ? 8 : 4, sets = (int)cdiv(nstrips, two), pt0 = c.PT;
    if (c.PT == 4 && (few || (tiles * nstrips < 1280 && (sets == 1 || P * sets * pitch <= (25 << 20))))) c.PT = 2;
    if (c.PT == 2 && cdiv(P, 32) * nstrips < 448) c.PT = 1;
    if (c.PT < pt0) c.NS = c.PT == 1 ? least(nstrips, 4) : two;
  }
  // enough workgroups: fewer strips each first, then smaller pixel tiles (six strips in one workgroup, 42x42x848->88 batch 2, or
  // four and two with twice the pixels: 6.7 / 6.0)
  while (cdiv(P, 16 * c.PT) * cdiv(nstrips, c.NS) < 160) {
    if (c.NS >= 8)
      c.NS = (c.NS / 2) & ~3;
    else if (c.NS > 4)
      c.NS = 4;
    else if (c.PT > 1)
      c.PT /= 2;
    else
      break;
  }
  if ((pitch <= 128 || P <= 64) && c.PT == 4 && few) {
    c.PT = 2;
    c.NS = nstrips <= 8 ? nstrips : 4;
  }
  if (i8 && nstrips < 4) c.PT = bsp_pw_thin(c.PT, pitch, c.NS);
  const int64_t xb = (int64_t)16 * c.PT * pitch, ob = (int64_t)16 * c.PT * (c.NS * 32 + 16);
  const bool lines = O >= I || (c.NS == 8 && O % 128 == 0 && lds / (xb + ob) == lds / xb);
  c.wout = windowed && (c.NS % 4 == 0 || c.NS >= nstrips) && lines && xb + ob <= lds;
  return c;
}

// fp32: whether the general kernel is to take the layer.  It sums a strip of sixteen channels chunk by
// chunk and tap by tap (`pairs` of them over all strips), straight from memory: few of those are over
// before the other kernel has staged its first patch, and its results leave in longer runs.  Timed on
// 5500 layers, general / matrix tiles in us, pairs per strip in brackets: one chunk of input channels 1x1
// 15x5x5->125 batch 34 with 16x4 blocks 3.9 / 9.5, 3x3 50x12x3->323 batch 50 31 / 60, 5x5 43x43x1->496
// batch 8 [14] 51 / 23; 8x8 1x1 14x14x11->118 batch 6 [1.5] 4.3 / 6.7, 1x3 21x21x27 [7] and up the tiles, 1x3
// 111x111x20 batch 47 [6, 7 M results] 73 / 39; 16x4 1x1 49x49x79->180 batch 25 [10, 11 M] 165 / 51.
// The tiles' results leave as vectors where the channels out are a multiple of four, one by one where
// they are not, which moves the line down there, the further the more results, and up here: 4x16 1x1
// 58x58x25->108 batch 37 [3.7] 59 / 37, 44x44x21->85 batch 33 [3] 25 / 37; 8x8 52x52x33->236 batch 29 [2]
// 63 / 42, 16x4 41x41x80->234 batch 4 [10] 25 / 17 at 1.6 M results, 5x5x14->66 batch 2 3.5 / 3.8.  A block of
// sixteen channels is multiplied whole, also where the layer has eight: 4x16 3x1 110x110x1->248 batch 48
// 52 / 80.  One row of 4x16 blocks is one wave, which stages its patch alone: 1x1 35x35x81->4 batch 4 [4]
// 4.3 / 9.8, 287->4 on 84700 pixels [8] 14 / 32.  FC layers of up to 256 rows (`few`) are not staged: only a
// single chunk is left to the general kernel, 12x4x4x5->110 3.2 / 6.2.
inline bool bsp_f32_general(int bo, int64_t I, int64_t O, int64_t HK, int64_t pairs, int64_t strips, int64_t po, bool few) {
  if (few) return I <= 8;
  const bool vectors = O % 4 == 0, many = po > 1000000;
  if (I <= 8 && (HK == 1 || (HK <= 9 && (!vectors || !many || bo == 4)))) return true;
  int most;
  if (!vectors)
    most = bo == 4 ? 5 : many ? 6 : bo == 8 ? 7 : 12;
  else if (many)
    most = bo == 4 ? 2 : 1;
  else if (po > 300000)
    most = bo == 8 ? 4 : 2;
  else
    most = bo == 8 ? 5 : bo == 4 ? 3 : 7;
  if (HK == 1 && bo == 4 && O <= 4) most = 8;
  return pairs <= most * strips;
}

// fp32 in whole chunks of eight channels in: whether the three-part kernel takes the layer from the two
// above (steps: a strip's, on average).  6000 random layers, the others / here: 1.36 times faster over the 5237
// that this line takes, 104 of them (most with a tenth of their blocks kept, or one strip) more than a tenth slower, down
// to 3.9 / 9.5 us for 1x1 27x27x296->8 batch 5; 0.95 over the 137 that the one step of one strip and the few tiles send back.
//   One chunk and tap is over at once in the general kernel: 1x1 70x70x8->768 batch 5 23 / 28; so is one step of one
//   strip, 3x1 95x100x88->4 batch 24 6.8 / 24.3.
//   Strips of 4x16 blocks unite four block rows, which leaves little to skip, and one or two strips do not pay for the
//   splitting of a long pixel: 3x3 35x35x448->16 batch 2 at stride 2 28 / 45, 12x12x408->8 1x3 11.2 / 14.2; 8x8 1x1
//   18x105x1120->16 17.1 / 24.9.
//   Few tiles (of sixteen pixels and a strip) of many steps leave most of the chip idle for one long chain: 4x16 5x5
//   5x5x344->48 batch 6 23 / 42, 3x3 32x10x400->72 batch 2 18.2 / 22.6, 8x8 5x5 15x15x504->109 batch 6 at stride 2 48 / 82.
// 3x3 56x56x64 batch 32 55 / 36, 1x1 28x28x128->512 batch 8 15.2 / 11.3, 16x4 3x1 68x68x40->326 batch 11 31 / 21.
inline bool bsp_f32x3_beats(int bo, int64_t strips, int64_t steps, int64_t P, int64_t I, int64_t HK) {
  if (I * HK <= 8 || strips * steps == 1) return false;
  const int64_t tiles = strips * ((P + 15) / 16);
  if (bo == 4) return strips > 1 && (strips > 2 || steps <= 30) && steps * tiles >= 6000 && (steps <= 25 || tiles >= 256);
  return bo != 8 || ((strips > 1 || steps <= 30) && (steps <= 100 || tiles >= 400));
}

// The widths of at most 64 columns that up to ceil(N / least) even chunks of N columns have, each once, the
// widest first: 64 of them at the most, however wide the image is.
template <typename F>
inline void bsp_widths(int64_t N, int least, F&& each) {
  for (int64_t nc = (N + 63) / 64; nc <= (N + least - 1) / least;) {
    const int cw = (int)((N + nc - 1) / nc);
    each(cw);
    if (cw == 1) return;
    nc = (N + cw - 2) / (cw - 1);  // the fewest chunks that are narrower
  }
}

#endif
