// The protocol by which the wavefronts of a workgroup share out batches of tickets (ft_batches.h), run by threads: every
// ticket is taken exactly once, every wavefront ends, each batch is taken in order, and a wavefront that is slow
// keeps nobody from the tickets behind its own.
// Usage: ticket_batches <first seed> <count>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>
#include "../../paper_2411_01830_amd/csrc/ft_batches.h"
using namespace ft;
#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d\n", #c, __LINE__); std::abort(); } } while (0)

struct Workgroup {
  std::atomic<uint64_t> taken;
  std::atomic<uint32_t> next;
  uint64_t add_taken() { return taken.fetch_add(1); }
  uint64_t word() { return taken.load(); }
  void set_word(uint64_t v) { taken.store(v); }
  uint32_t ahead() { return next.load(); }
  void set_ahead(uint32_t t) { next.store(t); }
  void pause() { std::this_thread::yield(); }
};

static void launch(uint32_t groups, uint32_t waves, uint32_t tickets, uint32_t slow) {
  const uint32_t round = groups * waves, batch = wave_batch(waves);
  CHECK(batch > 0 && batch + waves < 64);
  std::vector<Workgroup> wg(groups);
  std::vector<std::atomic<uint32_t>> hits(tickets);
  std::fprintf(stderr, "%u workgroups of %u, %u tickets, slow %u\n", groups, waves, tickets, slow);  // the last line names a case that hangs
  for (auto &h : hits) h = 0;
  std::atomic<uint32_t> counter{0}, done{0}, latest{0};
  std::atomic<bool> reset{false};
  for (uint32_t b = 0; b < groups; ++b) {
    wg[b].taken = batch;
    wg[b].next = round + b * batch;
  }
  std::vector<std::thread> ts;
  for (uint32_t b = 0; b < groups; ++b)
    for (uint32_t w = 0; w < waves; ++w)
      ts.emplace_back([&, b, w] {
        Workgroup &g = wg[b];
        uint32_t t = w * groups + b;
        bool draw = false;
        while (t < tickets) {
          if (draw) {
            uint32_t first = tickets;
            if (wave_counts(groups, waves, tickets)) {
              const uint32_t drawn = counter.fetch_add(1);
              first = round + (groups + drawn) * batch;
              if (drawn == wave_last_draw(groups, waves, tickets)) {
                CHECK(!reset.exchange(true));
                counter = 0;  // a draw after this would find a batch that was handed out already
              }
            }
            g.set_ahead(first);
          }
          hits[t].fetch_add(1);
          uint32_t was = latest.load();
          while (was < t && !latest.compare_exchange_weak(was, t)) {}
          if (t == slow) // until the others have nothing left to do but their own last tiles
            while (done.load() < groups * waves - 1) std::this_thread::yield();
          t = take_ticket(g, batch, tickets, &draw);
        }
        done.fetch_add(1);
      });
  for (auto &t : ts) t.join();
  for (auto &h : hits) CHECK(h == 1);
  CHECK(latest == tickets - 1);
  CHECK(counter == 0 && reset == wave_counts(groups, waves, tickets));
}

int main(int argc, char **argv) {
  const uint64_t first = argc > 1 ? strtoull(argv[1], 0, 10) : 1, count = argc > 2 ? strtoull(argv[2], 0, 10) : 50;
  for (uint64_t seed = first; seed < first + count; ++seed) {
    std::mt19937_64 r(seed);
    const uint32_t waves = 1u << (r() % 5), groups = 1 + r() % (waves > 8 ? 3 : 6);
    const uint32_t most = groups * waves;
    // around whole rounds and whole batches, and anything
    const uint32_t tickets = r() % 2 ? most + 1 + r() % 700 : most * (1 + r() % 4) + (uint32_t)(r() % 5) * wave_batch(waves) + r() % 3;
    if (!wave_shares(most, tickets)) continue;
    // no slow wavefront, one in the first round, or any; one that owes a draw has made it before its tile
    launch(groups, waves, tickets, seed % 3 == 0 ? ~0u : (uint32_t)(r() % (seed % 3 == 1 ? most : tickets)));
  }
  std::printf("done %llu..%llu\n", (unsigned long long)first, (unsigned long long)(first + count - 1));
  return 0;
}
