"""Where the kernel that streams bands past weights keeps what in LDS (csrc/bsp_bands_map.h), compiled for the host: for
every layer it takes, no two things share a byte and nothing lies past what the workgroup has."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "bsp_bands_map.h"
int main() {
  long layers = 0, doubled = 0, idle = 0, wrong = 0;
  std::vector<int> owner;
  for (int I = 8; I <= 128; I += 8)
    for (int O = 8; O <= 256; O += 8)
      for (int steps = 1; steps <= 7; ++steps)
        for (int N : {1, 16, 17, 33, 49, 500}) {
          BandsMap m{};
          const int nstrips = (O + 15) / 16;
          if (!bsp_bands_map(I, N, O, nstrips, steps, &m)) continue;
          ++layers;
          doubled += !m.single;
          long bad = m.lds > kBandsLds || m.resident * m.lds > kBandsLds || m.depth < steps;
          // 1, 2: patches; 3, 4: images; 5: biases
          owner.assign((size_t)(m.lds + 15) / 16, 0);
          auto take = [&](long at, int bytes, int who) {
            for (long b = at & ~15l; b < at + bytes; b += 16) {
              if (b < 0 || at + bytes > m.lds) {
                ++bad;
                return;
              }
              int& o = owner[(size_t)b / 16];
              if (o && o != who) ++bad;
              o = who;
            }
          };
          for (int buf = 0; buf < (m.single ? 1 : 2); ++buf) {
            for (int tid = 0; tid < 64 * m.waves; ++tid)
              for (int j = 0; j < kBandsPieces; ++j) {
                const int idx = tid + j * 64 * m.waves, px = idx / m.cpx, piece = idx % m.cpx, row = px / (m.cw + 2), col = px % (m.cw + 2);
                idle += !bsp_bands_some(idx, m.pieces);
                if (!bsp_bands_some(idx, m.pieces)) continue;
                const long at = row * m.rowpitch + col * m.pitch + piece * 16;
                if (at + 16 > m.patch) ++bad;
                take(buf * m.slot + at, 16, 1 + buf);
              }
            for (int pixel = 0; pixel < kBandsRows * m.cw; ++pixel) take(m.out_off + buf * m.oslot + (long)pixel * m.opitch, O * 2 + 8, 3 + buf);
          }
          for (int wave = 0; wave < m.waves; ++wave)
            for (int g = 0; g < 4; ++g) take(bsp_bands_bias((uint32_t)m.bias, wave, g), 16, 5);
          if (bad && wrong++ < 5) std::printf("I=%d O=%d steps=%d N=%d: %ld\n", I, O, steps, N, bad);
        }
  std::printf("%ld %ld %ld %ld\n", layers, doubled, idle, wrong);
}
"""


def test_nothing_in_lds_overlaps(tmp_path):
    src = tmp_path / "map.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "map")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2407_09453_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    layers, doubled, idle, wrong = (int(v) for v in out.splitlines()[-1].split())
    assert layers > 1000 and 0 < doubled < layers and idle > 0
    assert wrong == 0, out
