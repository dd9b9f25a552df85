// How the LDS-resident kernel (bsp_lds.hip) deals a layer's tiles to its workgroups (library private; plain C++, also compiled
// on the host by the tests).
//
// A workgroup owns a group of strips and walks tiles.  Consecutive workgroups go to the eight XCDs in turn.  Where the groups
// divide an XCD's 32 CUs, XCD x takes the x-th eighth of the tiles, in order, for all groups (bsp_tile.h: XCD); other numbers of
// groups would leave CUs idle so, and there a group's workgroups take every tile's share over the whole chip.
#ifndef BSP_DEAL_H
#define BSP_DEAL_H

#include <stdint.h>

struct LdsDeal {
  int64_t nwg;           // workgroups
  int32_t wg_per_group;  // workgroups sharing one strip group (an XCD's, where tpx is set)
  int32_t tpx;           // tiles of an XCD, or 0
};

constexpr LdsDeal bsp_lds_deal(int64_t ntiles, int groups, int cus) {
  auto least = [](int64_t a, int64_t b) { return a < b ? a : b; };
  if (32 % groups == 0 && cus == 256) {
    const int64_t tpx = (ntiles + 7) / 8, wgs = least(tpx, 32 / groups);
    return {8 * wgs * groups, (int32_t)wgs, (int32_t)tpx};
  }
  const int64_t slots = cus / groups < 1 ? 1 : cus / groups, wgs = least(ntiles, slots);
  return {wgs * groups, (int32_t)wgs, 0};
}

// Workgroup `bid`: slot = group + groups * its place among the group's workgroups; its first tile is that place after the first of
// its share, its others follow wg_per_group apart, before the share's end.
constexpr uint32_t bsp_lds_slot(int32_t tpx, uint32_t bid) { return tpx ? bid >> 3 : bid; }
constexpr int bsp_lds_first(int32_t tpx, uint32_t bid) { return (int)(bid & 7u) * tpx; }
constexpr int bsp_lds_end(int32_t tpx, uint32_t bid, int32_t ntiles) {
  const int end = bsp_lds_first(tpx, bid) + tpx;
  return tpx && end < ntiles ? end : ntiles;
}

#endif
