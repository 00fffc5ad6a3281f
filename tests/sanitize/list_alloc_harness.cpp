// CPU harness: order_tiles (lists.h) allocates nothing on its worker threads,
// where an exception would end the process instead of reaching the plan's
// caller.  Every allocation off the main thread fails here; the orders for one
// and for several threads are the same, also where most tiles are empty and one
// holds most entries.  Built by tests/test_tile_order_threads.py.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <thread>

#include "lists.h"

static std::thread::id main_thread;
static bool strict = false;

void* operator new(std::size_t n) {
  if (strict && std::this_thread::get_id() != main_thread) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

using namespace jgb::lists;

int main() {
  main_thread = std::this_thread::get_id();
  std::mt19937 rng(11);
  const int bias = 512;
  for (int shape = 0; shape < 3; ++shape) {
    Geometry g{};
    for (int a = 0; a < 3; ++a) {
      g.nf[a] = 64;
      g.T[a] = 8;
      g.nt[a] = 8;
      g.w[a] = 7;
    }
    // spread out; nearly all in one tile; too few for a second thread
    std::vector<Start> hdr(shape == 2 ? 50 : 30000);
    for (size_t j = 0; j < hdr.size(); ++j) {
      const bool one = shape == 1 && j % 100;
      hdr[j] = one ? Start{24, 25, 24, 0} : Start{(int)(rng() % 64), (int)(rng() % 64), (int)(rng() % 64), 0};
    }
    std::vector<int64_t> tcount, tgroup, group1;
    std::vector<Entry> list;
    std::vector<int> nstart, npos, tneed, need1;
    if (!gather_lists(g, true, bias, hdr, tcount, list, true, nstart, npos, 4).empty()) return 1;
    std::vector<int> npos1 = npos;
    std::vector<Entry> tlist(tcount.back()), serial(tcount.back());
    strict = true;
    order_tiles(g, true, bias, tcount, list, tlist.data(), npos, tgroup, tneed, 4);
    strict = false;
    order_tiles(g, true, bias, tcount, list, serial.data(), npos1, group1, need1, 1);
    if (npos != npos1 || tgroup != group1 || tneed != need1) return 2;
    for (size_t i = 0; i < tlist.size(); ++i)
      if (tlist[i].node != serial[i].node || tlist[i].code != serial[i].code) return 3;
  }
  puts("ok");
  return 0;
}
