// CPU harness for the order in which the interpolation by tiles takes a tile's
// list (order_tiles in paper_1311_4120_amd/csrc/lists.h), built with the address
// and undefined-behaviour sanitizers by tests/test_tile_order.py: each tile's
// entries are the same ones in another order, the node-major index still finds
// each node's entries in the order of its tiles, and no point that a footprint
// of a group of 16 covers is left out of the group's products.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <tuple>

#include "lists.h"

using namespace jgb::lists;

int main() {
  std::mt19937 rng(5);
  const int bias = 512;
  const int sides[4][3] = {{48, 34, 40}, {34, 96, 22}, {16, 12, 20}, {512, 24, 30}};
  for (const auto& nf : sides)
    for (int w : {2, 5, 7, 12, 16}) {
      Geometry g{};
      bool nowrap = true;
      for (int a = 0; a < 3; ++a) {
        g.nf[a] = nf[a];
        g.T[a] = 8;
        g.nt[a] = (nf[a] + 7) / 8;
        g.w[a] = std::min(w, nf[a]);
        nowrap &= nf[a] >= 8 + g.w[a] - 1;
      }
      std::vector<Start> hdr(9000);
      for (Start& s : hdr)
        s = Start{(int)(rng() % nf[0]), (int)(rng() % nf[1]), (int)(rng() % nf[2]), 0};
      std::vector<int64_t> tcount, tgroup;
      std::vector<Entry> list;
      std::vector<int> nstart, npos, tneed;
      if (!gather_lists(g, nowrap, nowrap ? bias : 0, hdr, tcount, list, true, nstart, npos, 3).empty()) return 1;
      const std::vector<int> before = npos;
      std::vector<Entry> tlist(tcount.back()), serial(tcount.back());
      order_tiles(g, nowrap, nowrap ? bias : 0, tcount, list, tlist.data(), npos, tgroup, tneed, 3);
      std::vector<int> npos1 = before, need1;
      std::vector<int64_t> group1;
      order_tiles(g, nowrap, nowrap ? bias : 0, tcount, list, serial.data(), npos1, group1, need1, 1);
      if (npos1 != npos || need1 != tneed || group1 != tgroup) return 2;
      // every entry once, where the node-major index says
      std::vector<char> hit(tcount.back(), 0);
      for (size_t i = 0; i < npos.size(); ++i) {
        const Entry &o = list[before[i]], &n = tlist[npos[i]];
        if (o.node != n.node || o.code != n.code || hit[npos[i]]) return 3;
        hit[npos[i]] = 1;
      }
      for (int64_t t = 0; t + 1 < (int64_t)tcount.size(); ++t) {
        if (tgroup[t + 1] - tgroup[t] != (tcount[t + 1] - tcount[t] + 15) / 16) return 4;
        for (int64_t i = tcount[t]; i < tcount[t + 1]; ++i) {
          const int need = tneed[tgroup[t] + (i - tcount[t]) / 16], c = tlist[i].code;
          const int b = nowrap ? bias : 0;
          for (int x = 0; x < 8; ++x)
            for (int y = 0; y < 8; ++y) {
              int dx = x + b - (c & 1023), dy = y + b - ((c >> 10) & 1023);
              if (!nowrap) dx = (dx + nf[0]) % nf[0], dy = (dy + nf[1]) % nf[1];
              const bool covered = dx >= 0 && dx < g.w[0] && dy >= 0 && dy < g.w[1];
              if (covered && !(need >> (x + 8 * (y / 4)) & 1)) return 5;
            }
        }
      }
    }
  puts("ok");
  return 0;
}
