// Host check of the pool's lookups from the place of the last answer (SlabPool::find, SlabPool::step), built with the
// sanitizers: whatever the order of the questions, the answers are those of a plain search; and a record tells the allocation
// that it holds from those that held it before.
// Usage: pool_lookups <first seed> <count>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "../../include/faastube.h"
#include "../../paper_2411_01830_amd/csrc/ft_pool.h"
using namespace ft;
#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d seed %llu\n", #c, __LINE__, (unsigned long long)seed); std::abort(); } } while (0)

int main(int argc, char **argv) {
  const uint64_t first = argc > 1 ? strtoull(argv[1], 0, 10) : 1, count = argc > 2 ? strtoull(argv[2], 0, 10) : 50;
  for (uint64_t seed = first; seed < first + count; ++seed) {
    std::mt19937_64 r(seed);
    auto U = [&](uint64_t a, uint64_t b) { return a + r() % (b - a + 1); };
    SlabPool pool(256);
    char *base = reinterpret_cast<char *>(0x7f0000000000ull);
    for (int s = 0; s < 3; ++s) CHECK(pool.add_segment(base + s * (1 << 20), 256 * U(1, 200)) == FT_OK);
    struct Live { uint64_t off, bytes; Allocation *al; uint64_t serial; };
    std::vector<Live> live, gone;
    for (int round = 0; round < 20; ++round) {
      for (int i = 0; i < 30; ++i) {
        uint64_t off, n = U(1, 3000);
        if (r() % 3 == 0 && !live.empty()) {
          const size_t k = U(0, live.size() - 1);
          CHECK(pool.free(live[k].off) == FT_OK);
          gone.push_back(live[k]);
          live.erase(live.begin() + (long)k);
        } else if (pool.alloc(n, &off) == FT_OK) {
          live.push_back(Live{off, (n + 255) / 256 * 256, pool.at(off), pool.at(off)->serial});
        }
      }
      std::sort(live.begin(), live.end(), [](const Live &a, const Live &b) { return a.off < b.off; });
      for (const Live &l : live) {
        const Allocation *al = pool.at(l.off);
        CHECK(al != nullptr && al == l.al && al->serial == l.serial && al->nslabs * 256 == l.bytes);
      }
      for (const Live &l : gone) CHECK(l.al->serial != l.serial);
      CHECK(pool.at(live.empty() ? 0 : live[0].off + 1) == nullptr);
      // one after another, all of them
      SlabPool::Place walk = pool.begin();
      for (size_t i = 1; i < live.size(); ++i) {
        const SlabPool::Entry *e = pool.step(&walk);
        CHECK(e != nullptr && e->start == live[i].off && e->al == live[i].al);
      }
      CHECK(pool.step(&walk) == nullptr && pool.step(&walk) == nullptr);
      SlabPool::Place near = pool.begin();
      uint64_t pos = 0;
      for (int q = 0; q < 200; ++q) {
        pos = r() % 3 ? pos + U(0, 900) : U(0, pool.total_bytes() + 500);  // mostly onwards, sometimes anywhere
        const uint64_t ext = U(1, 2000);
        size_t want = live.size();
        for (size_t i = 0; i < live.size(); ++i)
          if (pos >= live[i].off && pos < live[i].off + live[i].bytes && ext <= live[i].off + live[i].bytes - pos) want = i;
        const SlabPool::Entry *got = pool.find(pos, ext, &near);
        CHECK((got != nullptr) == (want < live.size()));
        if (got == nullptr) continue;
        CHECK(got->start == live[want].off && got->end == live[want].off + live[want].bytes && got->al == live[want].al);
        CHECK(got->dev == reinterpret_cast<uint64_t>(pool.ptr(got->start)));
        SlabPool::Place behind = near;
        const SlabPool::Entry *next = pool.step(&behind);
        CHECK((next != nullptr) == (want + 1 < live.size()) && (next == nullptr || next->start == live[want + 1].off));
      }
    }
  }
  std::printf("done %llu..%llu\n", (unsigned long long)first, (unsigned long long)(first + count - 1));
  return 0;
}
