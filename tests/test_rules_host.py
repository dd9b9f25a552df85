"""Which kernel takes a layer where several can (csrc/bsp_rules.h), compiled for the host: layers that
were timed on both sides of every line go to the side that was faster."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "bsp_rules.h"
static int wrong = 0;
static void is(bool got, bool want, const char* what) {
  if (got != want) {
    std::printf("%s\n", what);
    ++wrong;
  }
}
#define BEATS(want, ...) is(bsp_any_beats_bf16(__VA_ARGS__), want, #__VA_ARGS__)
#define FEW(want, ...) is(bsp_any_few(__VA_ARGS__), want, #__VA_ARGS__)
#define DIRECT(want, ...) is(bsp_any_direct(__VA_ARGS__), want, #__VA_ARGS__)
static void pw(int PT, int NS, int wout, int P, int I, int O, bool i8) {
  const int raw = i8 ? I : 2 * I, pitch = raw <= 128 ? 128 : (raw + 255) & ~255;
  const BspPwChoice c = bsp_pw_choose(P, raw / 2, i8 ? 1 << 30 : O, (O + 15) / 16, pitch, true, i8);
  if (c.PT != PT || c.NS != NS || c.wout != wout) {
    std::printf("P %d I %d O %d: %d %d %d, not %d %d %d\n", P, I, O, c.PT, c.NS, c.wout, PT, NS, wout);
    ++wrong;
  }
}
#define MODELS(want, ...) is(bsp_any_models_decide(__VA_ARGS__), want, #__VA_ARGS__)
#define LDS8(want, ...) is(bsp_any_beats_lds_i8(__VA_ARGS__), want, #__VA_ARGS__)
#define GEN8(want, ...) is(bsp_i8_general(__VA_ARGS__), want, #__VA_ARGS__)
#define THIN(want, ...) is(bsp_pw_thin(__VA_ARGS__) == want, true, #__VA_ARGS__)
#define TALL(want, ...) is(bsp_tall_beats(__VA_ARGS__), want, #__VA_ARGS__)
#define PWFEW(want, ...) is(bsp_pw_few_beats(__VA_ARGS__), want, #__VA_ARGS__)
#define PWFEW8(want, ...) is(bsp_pw_few_beats_i8(__VA_ARGS__), want, #__VA_ARGS__)
#define PWS(want, ...) is(bsp_pws_beats(__VA_ARGS__), want, #__VA_ARGS__)
#define BANDS(want, ...) is(bsp_bands_beats(__VA_ARGS__), want, #__VA_ARGS__)
#define X3(want, ...) is(bsp_f32x3_beats(__VA_ARGS__), want, #__VA_ARGS__)
#define F32(want, ...) is(bsp_f32_general(__VA_ARGS__), want, #__VA_ARGS__)
int main() {
  // rival, bo, H, K, strided, matrix instructions, results, channels in and out        the other / any-shape, us
  BEATS(true, BSP_RIVAL_ROWS, 8, 1, 7, false, 100861, 887808, 160, 192);      // 10.2 / 9.0
  BEATS(true, BSP_RIVAL_ROWS, 8, 1, 7, false, 220218, 1775616, 192, 192);      // 17.5 / 13.9
  BEATS(false, BSP_RIVAL_ROWS, 8, 1, 7, false, 252030, 2495232, 272, 192);     // 19 % slower
  BEATS(true, BSP_RIVAL_ROWS, 16, 1, 7, false, 1054620, 7392384, 160, 184);   // 66 / 40
  BEATS(true, BSP_RIVAL_LDS, 8, 1, 7, false, 32382, 161200, 248, 80);         // 19.8 / 7.0
  BEATS(false, BSP_RIVAL_LDS, 4, 1, 7, false, 201264, 7053088, 32, 184);      // 13.2 / 16.4
  BEATS(false, BSP_RIVAL_LDS, 16, 1, 3, false, 37044, 9483264, 8, 144);       // 13.5 / 18.5
  BEATS(true, BSP_RIVAL_LDS, 8, 1, 7, true, 53694, 4519800, 24, 200);         // 10.8 / 11.0: no line
  BEATS(true, BSP_RIVAL_LDS, 4, 7, 1, false, 62920, 402688, 192, 104);        // 9.4 / 7.8
  BEATS(true, BSP_RIVAL_ROWS, 8, 7, 1, false, 97104, 887808, 160, 192);       // 10.0 / 9.5
  BEATS(false, BSP_RIVAL_LDS, 8, 3, 1, false, 94000, 2384640, 184, 184);      // 11.5 / 11.6
  BEATS(true, BSP_RIVAL_ROWS, 4, 7, 1, true, 174202, 659456, 328, 128);       // 19.0 / 15.2
  BEATS(true, BSP_RIVAL_BAND, 8, 3, 3, false, 14112, 200704, 64, 64);         // 5.8 / 5.1
  BEATS(false, BSP_RIVAL_BAND, 8, 3, 3, false, 28244, 470400, 64, 96);        // 5.4 / 5.9
  BEATS(true, BSP_RIVAL_LDS, 8, 3, 3, false, 15904, 168000, 112, 336);        // 8.6 / 5.4
  BEATS(true, BSP_RIVAL_LDS, 16, 3, 3, true, 58424, 1920800, 72, 224);        // 14.3 / 10.2
  BEATS(false, BSP_RIVAL_LDS, 4, 3, 3, true, 59910, 5110560, 8, 160);         // 8.4 / 14.0
  BEATS(true, BSP_RIVAL_ROWS, 8, 3, 5, false, 6860, 37632, 184, 24);          // 8.8 / 5.3
  BEATS(false, BSP_RIVAL_ROWS, 4, 3, 5, false, 99856, 242352, 168, 24);       // 7.9 / 14.4
  BEATS(true, BSP_RIVAL_ROWS, 8, 7, 7, false, 3268, 4752, 144, 8);            // 8.0 / 5.8
  BEATS(false, BSP_RIVAL_ROWS, 4, 7, 7, false, 489086, 302400, 288, 112);     // 16.5 / 31.5
  BEATS(true, BSP_RIVAL_LDS, 8, 5, 5, false, 18208, 72800, 40, 8);            // 11.3 / 6.4
  BEATS(false, BSP_RIVAL_LDS, 4, 5, 5, false, 63308, 852640, 24, 32);         // 7.0 / 8.6
  BEATS(false, BSP_RIVAL_LDS, 4, 7, 7, false, 638976, 14942208, 8, 152);      // 23 / 51
  BEATS(true, BSP_RIVAL_TILE, 4, 5, 5, false, 21476, 30000, 248, 16);         // 43 / 8.3
  BEATS(false, BSP_RIVAL_TILE, 16, 5, 5, false, 230350, 9710400, 16, 448);    // 15.3 / 21.8
  BEATS(true, BSP_RIVAL_TILE, 8, 7, 7, false, 182272, 131072, 232, 32);       // 66 / 13
  BEATS(false, BSP_RIVAL_TILE, 8, 7, 7, false, 326500, 1150848, 64, 144);     // 18.7 / 24.2
  // row-band kernel, one row of more than 208 channels in: up to 200 K
  BEATS(true, BSP_RIVAL_ROWS, 8, 1, 7, false, 166181, 836352, 296, 384);      // 0.72 to 0.76 of the time here
  BEATS(true, BSP_RIVAL_ROWS, 8, 1, 7, false, 197010, 842400, 344, 160);      // 0.46
  BEATS(false, BSP_RIVAL_ROWS, 8, 1, 7, false, 216216, 658944, 384, 176);     // 1.05 to 1.14
  // one column: 8x8 blocks, more than 32 channels and up to 5000 pixels to 80 K, else to 45 K; strided to 340 K
  BEATS(true, BSP_RIVAL_ROWS, 8, 3, 1, false, 63480, 323400, 488, 88);        // 0.54
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 1, false, 74088, 903168, 216, 64);       // 1.24: 14 112 pixels
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 1, false, 48320, 618240, 208, 32);       // 1.23 to 1.39
  BEATS(false, BSP_RIVAL_ROWS, 4, 3, 1, false, 74556, 496128, 408, 136);      // 1.06 to 1.13
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 1, false, 83897, 1183200, 376, 232);     // 1.07 to 1.10
  BEATS(true, BSP_RIVAL_ROWS, 8, 3, 1, true, 214336, 1612800, 360, 256);      // 0.82 to 0.85
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 1, true, 351890, 5378688, 208, 368);     // not timed past the line but here (0.53 to 0.63)
  // 3x3: 30 K and, strided, 60 K; past them the two kernels' models decide
  BEATS(true, BSP_RIVAL_ROWS, 8, 3, 3, false, 29000, 300000, 256, 128);
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 3, false, 30001, 300000, 256, 128);
  BEATS(true, BSP_RIVAL_ROWS, 8, 3, 3, true, 60000, 300000, 256, 128);
  BEATS(false, BSP_RIVAL_ROWS, 8, 3, 3, true, 60001, 300000, 256, 128);
  // window, strided, matrix instructions, pixels, channels out
  MODELS(true, 3, 3, false, 115000, 8000, 128);
  MODELS(false, 3, 3, false, 115001, 8000, 128);
  MODELS(false, 3, 3, false, 115000, 8001, 128);
  MODELS(true, 3, 3, false, 115000, 6500, 64);
  MODELS(false, 3, 3, false, 115000, 6501, 64);                           // 57x35x224->24 batch 5 1.11 to 1.25
  MODELS(true, 3, 3, false, 200000, 1500, 128);
  MODELS(false, 3, 3, false, 200001, 1500, 128);
  MODELS(false, 3, 3, true, 117916, 11492, 32);                           // 52x52x368->32 stride 2 batch 17 16 / 30
  MODELS(true, 3, 3, true, 300000, 11492, 48);
  MODELS(false, 3, 3, true, 300001, 11492, 48);
  MODELS(false, 3, 3, false, 100000, 7000, 432);                          // more than 3 M results
  MODELS(false, 3, 1, false, 60000, 4000, 128);
  MODELS(false, 5, 3, false, 60000, 4000, 128);
  is(bsp_any_model_beats(false, 90000, 64, 3299., 1000.) && !bsp_any_model_beats(false, 90000, 64, 3300., 1000.), true, "models at stride 1");
  is(bsp_any_model_beats(true, 140000, 80, 2599., 1000.) && !bsp_any_model_beats(true, 140000, 80, 2600., 1000.), true, "models at stride 2");
  is(bsp_any_model_beats(true, 140001, 80, 2099., 1000.) && !bsp_any_model_beats(true, 140001, 80, 2100., 1000.), true, "models at stride 2, large");
  is(bsp_any_model_beats(true, 140000, 72, 2099., 1000.) && !bsp_any_model_beats(true, 140000, 72, 2100., 1000.), true, "models at stride 2, narrow");
  // pointwise layers: never before the specialised kernels, before the ring-tile kernel always
  BEATS(false, BSP_RIVAL_ROWS, 8, 1, 1, false, 100, 1000, 64, 64);
  BEATS(false, BSP_RIVAL_LDS, 8, 1, 1, false, 100, 1000, 64, 64);
  BEATS(true, BSP_RIVAL_TILE, 8, 1, 1, true, 1000000, 100000000, 64, 64);
  // block rows, pixels, channels in and out, 1x1
  FEW(true, 8, 64, 2048, 1000, true);                                     // 10.1 / 6.8
  FEW(false, 8, 28, 2048, 1000, true);
  FEW(false, 8, 65, 2048, 1000, true);
  FEW(false, 8, 64, 2056, 1000, true);
  FEW(true, 4, 17, 2048, 1000, true);                                     // 7.7 / 6.7
  FEW(false, 4, 33, 2048, 4096, true);                                    // 8.7 / 12.8
  FEW(false, 16, 52, 1864, 3346, true);                                   // 9.4 / 11.5
  FEW(true, 16, 61, 1656, 4406, true);                                    // 16.7 / 10.2
  FEW(true, 8, 64, 2048, 4096, true);                                     // 14.3 / 13.2
  FEW(true, 4, 49, 2048, 4096, false);                                    // a window
  // channels out, results: direct / through the image
  DIRECT(true, 32, 160000);                                               // 0.95, none slower
  DIRECT(false, 48, 192000);                                              // up to 1.09
  DIRECT(false, 48, 480000);                                              // 5.11 / 5.47
  DIRECT(true, 64, 400000);                                               // 0.96
  DIRECT(false, 64, 480000);                                              // up to 1.09
  DIRECT(true, 60, 160000);
  DIRECT(false, 66, 1000);                                                // channels come in fours
  // rival, matrix instructions, channels in and out, both models: the other / persistent, us
  TALL(true, BSP_RIVAL_ROWS, 1964952, 544, 336, 44422, 53418);            // 71 / 29
  TALL(true, BSP_RIVAL_ROWS, 2474304, 256, 256, 41416, 47991);            // 47 / 42
  TALL(true, BSP_RIVAL_ROWS, 2631888, 512, 512, 40516, 48351);            // 52 / 40
  TALL(true, BSP_RIVAL_ROWS, 1265376, 256, 512, 23586, 24452);            // 27 / 24
  TALL(false, BSP_RIVAL_ROWS, 66576, 256, 296, 11353, 5246);              // 10.4 / 12.7
  TALL(false, BSP_RIVAL_ROWS, 175770, 520, 64, 17696, 10246);             // 14.3 / 18.2
  TALL(false, BSP_RIVAL_ROWS, 2474304, 128, 256, 41416, 47991);
  TALL(true, BSP_RIVAL_ROWS, 20000, 136, 256, 1349, 1000);
  TALL(false, BSP_RIVAL_ROWS, 20000, 136, 256, 1350, 1000);
  TALL(false, BSP_RIVAL_ROWS, 19999, 136, 256, 1, 1000);                  // a full chip's opening is longer
  TALL(true, BSP_RIVAL_LDS, 1405404, 72, 344, 39535, 0);                  // 98 / 61
  TALL(true, BSP_RIVAL_LDS, 542490, 72, 432, 20220, 0);                   // 39 / 29
  TALL(false, BSP_RIVAL_LDS, 532824, 32, 64, 17086, 0);
  TALL(false, BSP_RIVAL_LDS, 542490, 72, 64, 20220, 0);
  TALL(false, BSP_RIVAL_LDS, 120000, 72, 432, 20220, 0);
  TALL(false, BSP_RIVAL_LDS, 542490, 136, 432, 20220, 0);
  TALL(false, BSP_RIVAL_BAND, 879285, 80, 192, 1, 1000);                  // 26 / 36
  TALL(false, BSP_RIVAL_TILE, 879285, 256, 192, 1, 1000);
  // 1x1 of up to 64 pixels, block rows, pixels, channels in and out: the others / pointwise
  PWFEW(true, 8, 1, 512, 4096);                                           // 4.4 / 4.1
  PWFEW(true, 8, 16, 64, 1000);                                           // 4.1 / 3.4
  PWFEW(true, 8, 49, 512, 2048);                                          // 5.0 / 4.4
  PWFEW(true, 8, 28, 1024, 1000);                                         // 1.23 times faster, and so on
  PWFEW(true, 8, 64, 1280, 4096);                                         // 1.43
  PWFEW(false, 8, 1, 1024, 1000);                                         // 0.93
  PWFEW(false, 8, 16, 1024, 1000);
  PWFEW(false, 8, 32, 2048, 256);                                         // 0.94
  PWFEW(true, 4, 1, 512, 1000);                                           // 1.28
  PWFEW(true, 4, 8, 1280, 1000);                                          // 1.06
  PWFEW(false, 4, 1, 2048, 256);                                          // 0.89
  PWFEW(true, 4, 1, 2048, 8192);                                          // 1.4 and up
  PWFEW(false, 4, 32, 1024, 256);                                         // 0.97
  PWFEW(true, 4, 32, 1024, 4096);                                         // 1.09
  PWFEW(false, 4, 32, 1288, 4096);
  PWFEW(true, 16, 8, 2048, 1000);                                         // 1.3 and up
  PWFEW(true, 16, 32, 512, 1000);                                         // 1.01
  PWFEW(false, 16, 32, 1024, 1000);                                       // 0.97
  PWFEW(true, 16, 32, 1024, 4096);                                        // 1.06
  PWFEW(false, 16, 8, 2056, 8192);
  PWFEW8(true, 256, 256);                                                 // 1.31
  PWFEW8(true, 512, 2048);                                                // 1.29
  PWFEW8(true, 1024, 1008);                                               // 1.07
  PWFEW8(false, 2048, 1008);                                              // 0.92
  PWFEW8(true, 2048, 4096);                                               // 0.99 to 1.31
  PWFEW8(false, 2064, 4096);
  // 1x1 of more than 64 pixels, int8, strips, steps, residual, rounds of 32 (past 8 steps 16) pixels: pointwise / streamed
  PWS(true, false, 8, 8, false, 100352 / 32 / 512.);                      // 256->128 on 100352 pixels 25.7 / 18.0
  PWS(true, false, 16, 2, true, 2 * 100352 / 32 / 512.);                  // 64->256 26.0 / 24.2
  PWS(true, false, 16, 2, true, 2 * 62720 / 32 / 512.);                   // 15.5 / 15.1
  PWS(false, false, 16, 2, true, 2 * 39168 / 32 / 512.);                  // 9.0 / 10.9
  PWS(false, false, 16, 2, true, 2 * 28224 / 32 / 512.);                  // 6.4 / 7.6
  PWS(true, false, 16, 2, false, 2 * 28224 / 32 / 512.);                  // 5.6 / 5.2
  PWS(false, false, 16, 2, false, 2 * 21632 / 32 / 512.);                 // 4.9 / 5.1
  PWS(false, false, 4, 2, false, 100352 / 32 / 512.);                     // 64->64 7.1 / 7.8
  PWS(false, false, 4, 7, false, 19881 / 32 / 512.);                      // 256->64 5.2 / 5.8
  PWS(true, false, 4, 7, false, 100352 / 32 / 512.);                      // 17.0 / 15.2
  PWS(true, false, 8, 7, false, 33000 / 32 / 512.);                       // 256->128 11.8 / 8.7
  PWS(false, false, 8, 7, false, 32000 / 32 / 512.);
  PWS(true, false, 32, 4, true, 4 * 8320 / 32 / 512.);                    // 128->512 8.1 / 6.5
  PWS(false, false, 32, 4, true, 4 * 8000 / 32 / 512.);                   // 0.96 to 0.99
  PWS(true, false, 16, 14, false, 18816 / 16 / 256.);                     // 512->256 17.9 / 14.1
  PWS(false, false, 16, 14, false, 16000 / 16 / 256.);                    // a third of them slower
  PWS(true, true, 16, 1, false, 2 * 25600 / 32 / 1024.);                  // 64->256 6.1 / 5.1
  PWS(false, true, 16, 1, false, 2 * 23232 / 32 / 1024.);                 // 4.8 / 5.1
  PWS(true, true, 32, 2, false, 4 * 14112 / 32 / 512.);                   // 128->512 6.9 / 5.6
  PWS(false, true, 32, 2, false, 4 * 11200 / 32 / 512.);                  // 5.0 / 5.3
  PWS(false, true, 32, 2, false, 4 * 6272 / 32 / 512.);                   // 4.4 / 4.5
  PWS(false, true, 8, 2, false, 42496 / 32 / 512.);                       // 128->128 5.6 / 6.0
  PWS(true, true, 8, 4, false, 100352 / 32 / 512.);                       // 256->128 13.7 / 11.2
  PWS(true, true, 8, 4, false, 42496 / 32 / 512.);                        // 7.6 / 7.4
  PWS(false, true, 8, 4, false, 31232 / 32 / 512.);                       // 6.1 / 6.5
  PWS(false, true, 32, 4, false, 4 * 11776 / 32 / 512.);                  // 256->512 5.9 / 6.2
  PWS(true, true, 32, 4, false, 4 * 13312 / 32 / 512.);                   // 7.4 / 6.4
  PWS(true, true, 16, 8, false, 2 * 18816 / 32 / 512.);                   // 512->256 10.1 / 7.7
  PWS(false, true, 16, 8, false, 2 * 14112 / 32 / 512.);                  // 7.0 / 7.3
  PWS(false, true, 4, 4, false, 100352 / 32 / 512.);                      // 256->64 8.9 / 9.7
  PWS(false, true, 16, 15, false, 100352 / 16 / 256.);
  // its workgroups that the chip holds
  is(bsp_pws_held(8, 84480) == 256, true, "512 channels in, eight strips, tiles of 32 pixels");
  is(bsp_pws_held(8, 81920) == 512, true, "half a CU's LDS");
  is(bsp_pws_held(8, 81936) == 256, true, "more than half a CU's LDS");
  is(bsp_pws_held(4, 14848) == 1024, true, "four waves");
  is(bsp_pws_held(16, 51200) == 256, true, "sixteen waves");
  // 3x3 at stride 1: strips, steps, pixels, channels in, rounds: the band or LDS-resident kernel / streamed
  BANDS(true, 2, 3, 16 * 147 * 147, 32, 2.89);                            // 27.2 / 14.4
  BANDS(true, 2, 3, 2 * 147 * 147, 32, 0.36);                             // 8.4 / 6.1
  BANDS(true, 4, 3, 16 * 147 * 147, 32, 5.78);                            // 29.6 / 19.1
  BANDS(true, 12, 6, 16 * 71 * 71, 80, 5.6);                              // 28.2 / 23.2
  BANDS(true, 12, 4, 4107, 48, 1);
  BANDS(false, 12, 4, 4107, 48, 0.35);                                    // 7.0 / 7.7
  BANDS(true, 12, 3, 4107, 48, 0.35);
  BANDS(true, 4, 5, 16 * 224 * 224, 64, 16.3);                            // 66.7 / 51.0
  BANDS(true, 8, 5, 16 * 112 * 112, 64, 12.3);                            // 31.2 / 29.5
  BANDS(true, 8, 6, 100000, 64, 4);
  BANDS(false, 8, 6, 100000, 64, 3.99);
  BANDS(false, 6, 5, 16 * 35 * 35, 64, 1.69);                             // 7.4 / 7.6
  BANDS(true, 4, 5, 4 * 56 * 56, 64, 0.29);                               // 5.9 / 5.2
  BANDS(true, 4, 5, 16 * 56 * 56, 64, 1.17);                              // 8.5 / 7.7
  BANDS(true, 4, 5, 32 * 48 * 48, 64, 1.5);                               // 8.9 / 8.3
  BANDS(false, 4, 5, 24 * 56 * 56, 64, 1.75);                             // 9.0 / 9.4
  BANDS(true, 4, 3, 24 * 56 * 56, 64, 1.75);
  BANDS(true, 4, 5, 24 * 56 * 56, 56, 1.75);
  BANDS(false, 8, 7, 6 * 56 * 56, 128, 1);                                // 11.1 / 11.9
  BANDS(true, 2, 3, 4000, 32, 0.2);
  BANDS(false, 2, 3, 3999, 32, 0.2);                                      // 0.98 and less
  // int8: slabs, window, pixels, channels out, matrix instructions: LDS-resident / any-shape, us
  LDS8(true, 1, 1, 6272, 256, 6272);                                      // 6.4 / 5.0
  LDS8(false, 1, 1, 100352, 256, 100352);                                 // 21 / 31
  LDS8(true, 4, 9, 1568, 512, 216000);                                    // 15.2 / 11.5
  LDS8(false, 2, 1, 360000, 16, 225000);                                  // 57 / 95
  LDS8(false, 2, 1, 360000, 32, 450000);                                  // 58 / 69
  LDS8(true, 2, 1, 360000, 48, 675000);                                   // 62 / 62
  LDS8(true, 2, 1, 90000, 16, 56250);                                     // 23 / 17
  LDS8(true, 2, 4, 134749, 32, 210550);                                   // 21 / 14
  LDS8(true, 5, 9, 18125, 192, 1120537);                                  // 41 / 35
  // int8: channels in and out, window, results: general / any-shape, us
  GEN8(true, 16, 16, 1, 109440);                                          // 3.2 / 4.0
  GEN8(true, 24, 40, 1, 265880);                                          // 3.3 / 4.0
  GEN8(true, 32, 16, 1, 1000000);
  GEN8(false, 32, 16, 1, 1000016);
  GEN8(true, 16, 592, 1, 67212720);                                       // 62 / 82
  GEN8(false, 16, 352, 1, 4066304);                                       // 10.1 / 7.8
  GEN8(false, 16, 24, 1, 6000000);
  GEN8(false, 24, 16, 1, 8000000);
  GEN8(true, 32, 432, 1, 36205920);                                       // 32 / 41
  GEN8(false, 32, 384, 1, 12000000);                                      // 16.8 / 16.2
  GEN8(false, 40, 16, 1, 1000);
  GEN8(false, 17, 16, 1, 1000);
  GEN8(false, 16, 16, 3, 1000);
  // pointwise tiles: lane tiles, strips a workgroup, whole lines; pixels, channels in and out, int8
  pw(2, 4, 0, 16 * 1225, 192, 64, false);                                 // 4.65 -> 4.31, four strips: 1228 waves
  pw(4, 4, 0, 16 * 1281, 192, 64, false);                                 // 1284
  pw(2, 8, 1, 8 * 196, 512, 512, false);                                  // 4.95 -> 4.51
  pw(2, 8, 0, 8 * 784, 256, 128, false);                                  // 4.26 -> 3.86
  pw(4, 8, 1, 32 * 196, 1024, 256, false);                                // 7.19 / 7.99: 1568
  pw(2, 4, 1, 2 * 324, 1536, 1504, true);                                 // 10.4 -> 6.3
  pw(1, 4, 0, 16 * 64, 2048, 192, false);                                 // 6.29 -> 5.36: 384
  pw(2, 4, 0, 16 * 64, 2048, 384, false);                                 // 6.52 / 7.09: 768
  pw(4, 8, 0, 19 * 400, 936, 136, false);                                 // 6.9 / 8.8: 27 MB staged
  pw(4, 8, 0, 5 * 784, 800, 272, false);                                  // 6.3 / 7.8
  pw(2, 4, 0, 31 * 144, 888, 232, false);                                 // 11.1 / 8.5
  pw(2, 4, 0, 2 * 1764, 848, 88, false);                                  // 6.0 / 6.7 as one lane tile of six strips
  pw(4, 8, 0, 17 * 121, 712, 664, false);                                 // 7.0 / 7.9 as whole lines: 42 strips
  pw(4, 8, 0, 8 * 1369, 688, 144, false);                                 // 8.8 / 9.4: 9 strips
  pw(4, 8, 1, 6 * 625, 648, 512, false);                                  // cold 9.0 -> 8.4 as whole lines
  pw(2, 8, 0, 5 * 441, 848, 504, false);                                  // 8.1 / 8.4
  pw(2, 4, 1, 3136, 64, 256, false);                                      // 3.27 -> 3.03: thin tiles by their number
  // lane tiles, bytes of a pixel, strips
  THIN(2, 4, 256, 1);
  THIN(1, 4, 512, 1);
  THIN(1, 4, 1024, 1);
  THIN(4, 4, 128, 1);
  THIN(4, 4, 256, 2);
  THIN(2, 4, 512, 2);
  THIN(2, 4, 768, 2);
  THIN(1, 4, 1024, 2);
  THIN(4, 4, 256, 3);
  THIN(2, 4, 512, 3);
  THIN(2, 4, 1024, 3);
  THIN(2, 2, 256, 1);
  THIN(1, 2, 512, 1);
  THIN(1, 1, 128, 1);
  // block rows, channels in and out, window, (chunk, tap) pairs, strips, results, FC of up to 256 rows: general / tiles, us
  F32(true, 16, 5, 125, 1, 8, 8, 318750, false);                          // 3.9 / 9.5
  F32(true, 16, 3, 323, 9, 21 * 9, 21, 9690000, false);                   // 31 / 60
  F32(false, 16, 1, 496, 25, 31 * 14, 31, 7336832, false);                // 51 / 23
  F32(false, 8, 8, 64, 9, 4 * 9, 4, 6400000, false);                      // many results, by vectors
  F32(true, 8, 8, 64, 9, 4 * 9, 4, 640000, false);
  F32(true, 8, 8, 64, 1, 4, 4, 6400000, false);
  F32(true, 8, 11, 118, 1, 12, 8, 138768, false);                         // 4.3 / 6.7
  F32(false, 8, 40, 84, 3, 58, 7, 111384, false);                         // 6.7 / 5.6
  F32(true, 8, 18, 11, 3, 11, 2, 77128, false);
  F32(false, 8, 20, 20, 3, 12, 2, 11581740, false);                       // 73 / 39
  F32(false, 16, 79, 180, 1, 120, 12, 10804500, false);                   // 165 / 51
  F32(false, 4, 43, 100, 1, 6 * 27, 27, 64600, false);                    // 5.6 / 5.3
  F32(true, 4, 1, 248, 3, 16 * 3, 16, 32946000, false);                   // 52 / 80
  F32(false, 8, 33, 236, 1, 30, 15, 18505568, false);                     // 63 / 42
  // the line itself: block rows; vectors up to 3e5, up to 1e6 and beyond; one by one up to 1e6 and beyond
  const int lines[3][6] = {{8, 5, 4, 1, 7, 6}, {4, 3, 2, 2, 5, 5}, {16, 7, 2, 1, 12, 6}};
  for (auto& l : lines)
    for (int k = 0; k < 5; ++k) {
      const int O = k < 3 ? 64 : 63, po = k == 0 ? 300000 : k == 1 || k == 3 ? 1000000 : 1000001;
      F32(true, l[0], 64, O, 1, 4 * l[1 + k], 4, po, false);
      F32(false, l[0], 64, O, 1, 4 * l[1 + k] + 1, 4, po, false);
    }
  F32(true, 4, 81, 4, 1, 4, 1, 19600, false);                             // 4.3 / 9.8
  F32(true, 4, 287, 4, 1, 8, 1, 338800, false);                           // 14 / 32
  F32(false, 4, 287, 4, 1, 9, 1, 338800, false);
  F32(true, 8, 5, 110, 1, 7, 7, 21120, true);                             // 3.2 / 6.2
  F32(false, 8, 64, 64, 1, 8, 4, 4096, true);
  // block rows, strips, steps, pixels, channels in, window: the others / three parts, us
  X3(true, 8, 4, 15, 100352, 64, 9);                                      // 55 / 36
  X3(true, 8, 32, 4, 6272, 128, 1);                                       // 15.2 / 11.3
  X3(true, 16, 21, 2, 50864, 40, 3);                                      // 31 / 21
  X3(false, 8, 48, 1, 24500, 8, 1);                                       // 23 / 28
  X3(true, 16, 41, 1, 100000, 24, 1);
  X3(false, 16, 1, 1, 57600, 88, 3);                                      // 6.8 / 24.3
  X3(true, 16, 1, 2, 57600, 88, 3);
  X3(true, 16, 1, 57, 1600, 256, 9);                                      // one strip, 16x4
  X3(false, 8, 1, 35, 1890, 1120, 1);                                     // 17.1 / 24.9
  X3(true, 8, 1, 30, 1890, 960, 1);
  X3(false, 4, 1, 26, 1152, 408, 3);                                      // 11.2 / 14.2
  X3(false, 4, 1, 126, 648, 448, 9);                                      // 28 / 45
  X3(false, 4, 2, 31, 100000, 136, 9);
  X3(true, 4, 2, 30, 100000, 136, 9);
  X3(false, 4, 4, 5, 4224, 32, 9);                                        // few products
  X3(false, 4, 3, 269, 150, 344, 25);                                     // 23 / 42
  X3(false, 4, 5, 105, 640, 400, 9);                                      // 18.2 / 22.6
  X3(true, 4, 37, 24, 7203, 104, 9);                                      // 1.5 times faster
  X3(false, 4, 16, 26, 240, 104, 9);
  X3(true, 4, 16, 26, 256, 104, 9);
  X3(false, 8, 7, 303, 384, 504, 25);                                     // 48 / 82
  X3(true, 8, 25, 101, 256, 504, 9);
  X3(false, 8, 25, 101, 240, 504, 9);
  X3(true, 8, 25, 100, 240, 504, 9);
  X3(true, 16, 7, 303, 384, 504, 25);                                     // 16x4 blocks unite nothing
  // what no number of pixels brings to that kernel gets no weights for it in its plan
  X3(false, 4, 1, 20, (int64_t)1 << 31, 64, 9);
  X3(true, 4, 3, 300, (int64_t)1 << 31, 64, 9);
  // the widths that a tile's search tries: those of every even cut, and few of them on the widest image
  for (int least : {4, 8})
    for (int64_t N = 1; N <= 3000; ++N) {
      std::vector<int> got, want;
      bsp_widths(N, least, [&](int cw) { got.push_back(cw); });
      for (int64_t nc = 1; nc <= (N + least - 1) / least; ++nc) {
        const int cw = (int)((N + nc - 1) / nc);
        if (cw <= 64 && (want.empty() || want.back() != cw)) want.push_back(cw);
      }
      is(got == want, true, "bsp_widths");
    }
  int tried = 0;
  bsp_widths(0x7FFFFFFF, 4, [&](int) { ++tried; });
  is(tried <= 61, true, "bsp_widths on the widest image");
  std::printf("%d\n", wrong);
}
"""


def test_timed_layers_go_to_the_faster_kernel(tmp_path):
    src = tmp_path / "rules.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "rules")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2407_09453_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    assert out.strip() == "0", out
