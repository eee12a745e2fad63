// Which launches of pieces write words to the host when they are done (ft_pieces.h: says_done), on a machine without a GPU, by
// tests/host/hip_stand_in.cpp: those of streams on which few jobs are in flight at once. And when the runtime is made to give back its records of launches.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/faastube.h"

extern "C" int stand_in_words(void);
extern "C" int stand_in_calls(const char *name);
extern "C" int stand_in_fail(const char *name, int nth);

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d\n", #c, __LINE__); std::abort(); } } while (0)

namespace {
constexpr uint64_t KiB = 1024, kRoom = 64 * KiB, kBig = 24 << 20;
char *g_dev;
ft_pool *g_pool;
ft_off_t g_src, g_dst, g_big[2];

ft_job_t submit(uint32_t i, void *stream, uint32_t flags = 0, bool big = false) {
  ft_desc d = {};
  d.rows = 1;
  d.row_bytes = big ? kBig : 40 * KiB;
  d.src_space = d.dst_space = FT_POOL;
  d.src = big ? g_big[0] : g_src + i * kRoom;
  d.dst = big ? g_big[1] : g_dst + i * kRoom;
  const uint32_t weight = 1;
  ft_job_t job = 0;
  CHECK(ft_submit_transfers(g_pool, &d, 1, &weight, 1, 256 * KiB, flags, stream, &job) == FT_OK);
  return job;
}

// n jobs submitted one behind the other and then waited for: how many of them had words.
int burst(uint32_t n, void *stream) {
  std::memset(g_dev + g_dst, 0, 32 * kRoom);
  const int before = stand_in_words();
  std::vector<ft_job_t> jobs;
  for (uint32_t i = 0; i < n; ++i) jobs.push_back(submit(i, stream));
  for (ft_job_t j : jobs) CHECK(ft_wait(g_pool, j) == FT_OK);
  for (uint32_t i = 0; i < n; ++i) CHECK(std::memcmp(g_dev + g_src + i * kRoom, g_dev + g_dst + i * kRoom, 40 * KiB) == 0);
  return stand_in_words() - before;
}
}  // namespace

int main() {
  const uint64_t bytes = 64 * kRoom + 2 * kBig;
  g_dev = static_cast<char *>(std::calloc(bytes, 1));
  for (uint64_t i = 0; i < bytes; ++i) g_dev[i] = (char)(i * 2654435761u >> 13);
  CHECK(ft_pool_create(&g_pool, g_dev, bytes, 4096, 0) == FT_OK);
  CHECK(ft_slab_alloc(g_pool, 32 * kRoom, &g_src) == FT_OK && ft_slab_alloc(g_pool, 32 * kRoom, &g_dst) == FT_OK);
  CHECK(ft_slab_alloc(g_pool, kBig, &g_big[0]) == FT_OK && ft_slab_alloc(g_pool, kBig, &g_big[1]) == FT_OK);
  hipStream_t a, b;
  CHECK(hipStreamCreate(&a) == hipSuccess && hipStreamCreate(&b) == hipSuccess);
  for (int k = 0; k < 3; ++k) CHECK(burst(1, a) == 1);
  for (uint32_t n : {2u, 3u, 4u})
    for (int k = 0; k < 2; ++k) CHECK(burst(n, a) == (int)n);
  CHECK(burst(5, a) == 4);  // the fifth is the first that the stream has not been known for
  for (int k = 0; k < 3; ++k) CHECK(burst(5, a) == 0);
  CHECK(burst(1, b) == 1);   // of another stream nothing is known yet
  CHECK(burst(32, a) == 0 && burst(32, a) == 0);
  CHECK(burst(1, a) == 0);   // a burst was before it
  for (int k = 0; k < 3; ++k) CHECK(burst(1, a) == 1);
  {  // a job on the stream that is not as short, and not waited for in its turn
    const ft_job_t j = submit(0, a, 0, true);
    CHECK(burst(3, a) == 3 && burst(4, a) == 3);
    CHECK(ft_wait(g_pool, j) == FT_OK);
    CHECK(burst(1, a) == 0 && burst(1, a) == 1);
  }
  {  // a long detached one is on the library's streams
    const ft_job_t j = submit(0, a, FT_DETACHED, true);
    CHECK(burst(4, a) == 4 && burst(1, a) == 1);
    CHECK(ft_wait(g_pool, j) == FT_OK && burst(1, a) == 1);
  }
  {  // one aligned tensor from the host: as pieces up to 128 KiB, and up to 256 where it is alone and not timed
    std::vector<char> host(300 * KiB + 64);
    const uint64_t at = (reinterpret_cast<uint64_t>(host.data()) + 15) / 16 * 16;
    CHECK(ft_host_window_add(g_pool, host.data(), host.size()) == FT_OK);
    const auto pieces = [&](uint64_t bytes, uint32_t n, uint32_t flags) {
      const int before = stand_in_calls("launch_pieces");
      std::vector<ft_job_t> jobs(n);
      for (ft_job_t &job : jobs) {
        ft_desc d = {};
        d.rows = 1;
        d.row_bytes = bytes;
        d.src_space = FT_HOST;
        d.dst_space = FT_POOL;
        d.src = at;
        d.dst = g_dst;
        const uint32_t weight = 1;
        for (char &c : host) c += 7;
        CHECK(ft_submit_transfers(g_pool, &d, 1, &weight, 1, 2048 * KiB, flags, b, &job) == FT_OK);
      }
      const int launches = stand_in_calls("launch_pieces") - before;
      for (ft_job_t job : jobs) CHECK(ft_wait(g_pool, job) == FT_OK);
      CHECK(std::memcmp(g_dev + g_dst, reinterpret_cast<char *>(at), bytes) == 0);
      return launches;
    };
    for (int k = 0; k < 2; ++k) CHECK(pieces(128 * KiB, 1, 0) == 1 && pieces(128 * KiB + 16, 1, 0) == 1 && pieces(256 * KiB, 1, 0) == 1 && pieces(256 * KiB + 16, 1, 0) == 0);
    CHECK(pieces(128 * KiB, 1, FT_TIMING) == 1 && pieces(128 * KiB + 16, 1, FT_TIMING) == 0 && pieces(256 * KiB, 1, FT_TIMING) == 0);
    CHECK(pieces(256 * KiB, 4, 0) == 1 && pieces(256 * KiB, 4, 0) == 0 && pieces(128 * KiB, 4, 0) == 4 && pieces(200 * KiB, 2, 0) == 0 && pieces(256 * KiB, 1, 0) == 0);
    CHECK(pieces(256 * KiB, 1, 0) == 1);
  }
  const int before = stand_in_words();
  CHECK(ft_wait(g_pool, submit(0, a, FT_DETACHED)) == FT_OK && stand_in_words() == before + 1);
  {  // more streams than are remembered: nothing is lost of those with unfinished jobs
    std::vector<hipStream_t> many(200);
    std::vector<ft_job_t> jobs;
    for (hipStream_t &s : many) {
      CHECK(hipStreamCreate(&s) == hipSuccess);
      jobs.push_back(submit(0, s));
      CHECK(ft_wait(g_pool, submit(1, s)) == FT_OK);
    }
    for (ft_job_t j : jobs) CHECK(ft_wait(g_pool, j) == FT_OK);
    for (int k = 0; k < 2; ++k)
      for (hipStream_t s : many) CHECK(burst(1, s) == 1);
    for (hipStream_t s : many) CHECK(hipStreamDestroy(s) == hipSuccess);
  }
  CHECK(ft_pool_destroy(g_pool) == FT_OK);
  {  // a launch that gives records back for every 2^20 jobs of all streams at most, each stream's share of them
    CHECK(ft_pool_create(&g_pool, g_dev, bytes, 4096, 0) == FT_OK);
    CHECK(ft_slab_alloc(g_pool, 32 * kRoom, &g_src) == FT_OK && ft_slab_alloc(g_pool, 32 * kRoom, &g_dst) == FT_OK);
    constexpr uint32_t kStreams = 64, kShare = (1u << 20) / kStreams;
    std::vector<hipStream_t> many(kStreams);
    const auto run = [&](hipStream_t s, uint32_t n) {
      const int before = stand_in_calls("launch_plain_fill");
      for (uint32_t i = 0; i < n; ++i) CHECK(ft_wait(g_pool, submit(0, s, i % 7 == 0 ? FT_TIMING : 0)) == FT_OK);
      return stand_in_calls("launch_plain_fill") - before;
    };
    for (hipStream_t &s : many) CHECK(hipStreamCreate(&s) == hipSuccess && run(s, 1) == 0);
    CHECK(run(many[3], kShare - 1) == 0 && run(many[3], 1) == 1 && run(many[3], kShare - 1) == 0);
    CHECK(stand_in_fail("launch_plain_fill", 1) == 0);  // one that fails is made up for by the next job
    ft_desc d = {};
    d.rows = 1;
    d.row_bytes = 40 * KiB;
    d.src_space = d.dst_space = FT_POOL;
    d.src = g_src;
    d.dst = g_dst;
    const uint32_t weight = 1;
    ft_job_t job = 0;
    CHECK(ft_submit_transfers(g_pool, &d, 1, &weight, 1, 256 * KiB, 0, many[3], &job) == FT_EHIP);
    CHECK(run(many[3], 1) == 1 && run(many[5], 1) == 0);
    for (hipStream_t s : many) CHECK(hipStreamDestroy(s) == hipSuccess);
    CHECK(ft_pool_destroy(g_pool) == FT_OK);
  }
  std::free(g_dev);
  std::printf("done_words done\n");
  return 0;
}
