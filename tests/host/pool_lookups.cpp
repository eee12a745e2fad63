// Host check of the pool's lookups from the place of the last answer (SlabPool::owner, SlabPool::at), built with the
// sanitizers: whatever the order of the questions, the answers are those of a plain search.
// Usage: pool_lookups <first seed> <count>
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
    struct Live { uint64_t off, bytes; };
    std::vector<Live> live;
    for (int round = 0; round < 20; ++round) {
      for (int i = 0; i < 30; ++i) {
        uint64_t off, n = U(1, 3000);
        if (r() % 3 == 0 && !live.empty()) {
          const size_t k = U(0, live.size() - 1);
          CHECK(pool.free(live[k].off) == FT_OK);
          live.erase(live.begin() + (long)k);
        } else if (pool.alloc(n, &off) == FT_OK) {
          live.push_back(Live{off, (n + 255) / 256 * 256});
        }
      }
      SlabPool::Place near = pool.begin(), near_at = pool.begin();
      uint64_t pos = 0;
      for (int q = 0; q < 200; ++q) {
        pos = r() % 3 ? pos + U(0, 900) : U(0, pool.total_bytes() + 500);  // mostly onwards, sometimes anywhere
        const uint64_t ext = U(1, 2000);
        const Live *want = nullptr;
        for (const Live &l : live)
          if (pos >= l.off && pos < l.off + l.bytes && ext <= l.off + l.bytes - pos) want = &l;
        uint64_t start = ~0ull;
        Allocation *got = pool.owner(pos, ext, &start, &near);
        CHECK((got != nullptr) == (want != nullptr));
        if (want) CHECK(start == want->off && got == pool.at(want->off) && got->nslabs * 256 == want->bytes);
        const uint64_t ask = want && r() % 2 ? want->off : pos;
        CHECK(pool.at(ask, &near_at) == pool.at(ask));
      }
    }
  }
  std::printf("done %llu..%llu\n", (unsigned long long)first, (unsigned long long)(first + count - 1));
  return 0;
}
