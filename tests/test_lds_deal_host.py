"""How the LDS-resident kernel deals tiles to workgroups (csrc/bsp_deal.h), compiled for the host: every tile goes to one workgroup of
every strip group, and the busiest workgroup has no more of them than the chip's size asks for."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "bsp_deal.h"
int main() {
  long cases = 0, eighths = 0, wrong = 0;
  for (int cus : {256, 304, 32, 1})
    for (int groups = 1; groups <= 70; ++groups)
      for (int ntiles : {1, 2, 7, 8, 9, 15, 16, 31, 33, 63, 64, 65, 255, 256, 257, 263, 1000, 2049}) {
        const LdsDeal d = bsp_lds_deal(ntiles, groups, cus);
        std::vector<int> dealt((size_t)ntiles * groups, 0);
        long most = 0, bad = d.tpx && d.nwg % 8;
        for (uint32_t bid = 0; bid < d.nwg; ++bid) {
          const uint32_t slot = bsp_lds_slot(d.tpx, bid);
          const int cidx = (int)(slot / groups), sg = (int)(slot % groups), end = bsp_lds_end(d.tpx, bid, ntiles);
          long mine = 0;
          for (int tile = bsp_lds_first(d.tpx, bid) + cidx; tile < end; tile += d.wg_per_group, ++mine) {
            if (tile < 0 || tile >= ntiles) {
              ++bad;
              break;
            }
            ++dealt[(size_t)tile * groups + sg];
            bad += d.tpx && tile / d.tpx != (int)(bid & 7u);
          }
          most = mine > most ? mine : most;
        }
        for (int n : dealt) bad += n != 1;
        const int slots = cus / groups < 1 ? 1 : cus / groups;
        bad += most != (ntiles + slots - 1) / slots;
        ++cases;
        eighths += d.tpx != 0;
        if (bad && wrong++ < 5) std::printf("cus=%d groups=%d tiles=%d: %ld\n", cus, groups, ntiles, bad);
      }
  std::printf("%ld %ld %ld\n", cases, eighths, wrong);
}
"""


def test_every_tile_is_dealt_once(tmp_path):
    src = tmp_path / "deal.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "deal")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2407_09453_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    cases, eighths, wrong = (int(v) for v in out.splitlines()[-1].split())
    assert eighths == 6 * 18 and cases == 4 * 70 * 18  # 1, 2, 4, 8, 16 and 32 groups on 256 CUs
    assert wrong == 0, out
