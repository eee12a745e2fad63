// Batches of pageable sources that are launched in parts (ft_open.cpp), on a machine without a GPU: with tests/host/hip_stand_in.cpp the
// n-th launch or event fails, or none does. The job ends either way, its bytes are in place if it succeeds, and nothing stays busy.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/faastube.h"

extern "C" int stand_in_fail(const char *name, int nth);
extern "C" uint64_t stand_in_copied(void);
extern "C" int stand_in_calls(const char *name);

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d (%s, n %d)\n", #c, __LINE__, point, n); std::abort(); } } while (0)

// What an open job of 8 MiB uploads for its tables.
static uint64_t tables_of(uint32_t space, uint64_t chunk, uint32_t batch) {
  const char *point = "tables";
  const int n = (int)batch;
  const uint64_t bytes = 8 << 20;
  std::vector<char> src(bytes, 5), dev(2 * bytes);
  ft_pool *pool = nullptr;
  char *base = reinterpret_cast<char *>((reinterpret_cast<uint64_t>(dev.data()) + 4095) / 4096 * 4096);
  CHECK(ft_pool_create(&pool, base, bytes, 4096, 0) == FT_OK && ft_set_batch(pool, batch, 3) == FT_OK);
  CHECK((space == FT_HOST ? ft_host_window_add : ft_pageable_window_add)(pool, src.data(), bytes) == FT_OK);
  ft_off_t off;
  CHECK(ft_slab_alloc(pool, bytes, &off) == FT_OK);
  ft_desc d = {};
  d.rows = 1;
  d.row_bytes = bytes;
  d.src_space = space;
  d.dst_space = FT_POOL;
  d.src = reinterpret_cast<uint64_t>(src.data());
  d.dst = off;
  const uint32_t weight = 1;
  ft_job_t job;
  const uint64_t before = stand_in_copied();
  CHECK(ft_submit_transfers(pool, &d, 1, &weight, 1, chunk, FT_OPEN, nullptr, &job) == FT_OK && ft_wait(pool, job) == FT_OK);
  const uint64_t uploaded = stand_in_copied() - before;
  CHECK(std::memcmp(ft_pool_ptr(pool, off), src.data(), bytes) == 0);
  CHECK(ft_slab_free(pool, off) == FT_OK && ft_pool_destroy(pool) == FT_OK);
  return uploaded;
}

// Launches of an open job of 8 chunks of pinned memory and, of another function, one of pageable memory.
static int launches_beside(bool pageable, uint32_t batch) {
  const char *point = "launches";
  const int n = (int)batch;
  const uint64_t chunk = 2 << 20, bytes = 9 * chunk;
  std::vector<char> src(bytes, 5), dev(bytes + 4096);
  char *base = reinterpret_cast<char *>((reinterpret_cast<uint64_t>(dev.data()) + 4095) / 4096 * 4096);
  ft_pool *pool = nullptr;
  CHECK(ft_pool_create(&pool, base, bytes, 4096, 0) == FT_OK && ft_set_batch(pool, batch, 1) == FT_OK);
  CHECK(ft_host_window_add(pool, src.data(), 8 * chunk) == FT_OK && ft_pageable_window_add(pool, src.data() + 8 * chunk, chunk) == FT_OK);
  ft_off_t off;
  CHECK(ft_slab_alloc(pool, bytes, &off) == FT_OK);
  ft_desc d[2] = {};
  for (uint32_t f = 0; f < 2; ++f) {
    d[f].func = f;
    d[f].rows = 1;
    d[f].row_bytes = f == 0 ? 8 * chunk : chunk;
    d[f].src_space = f == 0 ? FT_HOST : FT_PAGEABLE;
    d[f].dst_space = FT_POOL;
    d[f].src = reinterpret_cast<uint64_t>(src.data()) + f * 8 * chunk;
    d[f].dst = off + f * 8 * chunk;
  }
  const uint32_t weights[2] = {1, 1};
  const int before = stand_in_calls("launch_copy");
  ft_job_t job;
  CHECK(ft_submit_transfers(pool, d, pageable ? 2 : 1, weights, pageable ? 2 : 1, chunk, FT_OPEN, nullptr, &job) == FT_OK && ft_wait(pool, job) == FT_OK);
  CHECK(std::memcmp(ft_pool_ptr(pool, off), src.data(), (pageable ? 9 : 8) * chunk) == 0);
  CHECK(ft_slab_free(pool, off) == FT_OK && ft_pool_destroy(pool) == FT_OK);
  return stand_in_calls("launch_copy") - before;
}

#define CHECK_TABLES(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d\n", #c, __LINE__); std::abort(); } } while (0)

int main() {
  // a ticket counter for every launch, 8 bytes in a table of whole 256: of a batch of chunks under 2 MiB one, whatever its sources
  for (uint64_t chunk : {4096ull, 64 * 1024ull, 1024 * 1024ull})
    for (uint32_t batch : {1u, 5u, 16u}) CHECK_TABLES(tables_of(FT_PAGEABLE, chunk, batch) == tables_of(FT_HOST, chunk, batch));
  for (uint32_t batch : {1u, 2u, 20u}) CHECK_TABLES(tables_of(FT_PAGEABLE, 2 << 20, batch) == tables_of(FT_HOST, 2 << 20, batch));
  // the batch with the staged chunk in parts, the others whole
  CHECK_TABLES(launches_beside(false, 3) == 3 && launches_beside(true, 3) == 3 + 2);
  const uint64_t MiB = 1 << 20, bytes = 7 * MiB + 12345;
  std::vector<char> src(2 * bytes);
  for (size_t i = 0; i < src.size(); ++i) src[i] = (char)(i * 2654435761u >> 13);
  for (const char *point : {"launch_copy", "hipEventRecord", "hipEventSynchronize", "hipEventCreateWithFlags", "hipStreamWaitEvent"})
    for (uint64_t chunk : {256 * 1024ull, 2ull * MiB})
      for (uint32_t depth : {1u, 3u})
        for (int n = 0; n < 14; ++n) {
          char *dev = static_cast<char *>(std::calloc(32, MiB));
          ft_pool *pool = nullptr;
          CHECK(ft_pool_create(&pool, dev, 32 * MiB, 4096, 0) == FT_OK);
          CHECK(ft_pageable_window_add(pool, src.data(), src.size()) == FT_OK);
          CHECK(ft_set_batch(pool, 5, depth) == FT_OK);
          ft_off_t off[2];
          ft_desc d[2] = {};
          for (uint32_t f = 0; f < 2; ++f) {
            CHECK(ft_slab_alloc(pool, bytes + 16, &off[f]) == FT_OK);
            d[f].func = f;
            d[f].rows = 1;
            d[f].row_bytes = bytes;
            d[f].src_space = FT_PAGEABLE;
            d[f].dst_space = FT_POOL;
            d[f].src = reinterpret_cast<uint64_t>(src.data() + f * bytes);
            d[f].dst = off[f] + 3 * f;
          }
          const uint32_t weights[2] = {1, 3};
          stand_in_fail(point, n);
          ft_job_t job = 0;
          int rc = ft_submit_transfers(pool, d, 2, weights, 2, chunk, FT_OPEN | FT_KEEP, nullptr, &job);
          CHECK(rc == FT_OK || rc == FT_EHIP);
          if (rc == FT_OK) {
            rc = ft_wait(pool, job);
            CHECK(rc == FT_OK || (rc == FT_EHIP && n != 0));
            uint64_t done[2], batches = 0, chunks = 2 * ((bytes + chunk - 1) / chunk);
            CHECK(ft_job_progress(pool, job, 0, done, 2, &batches) == FT_OK);
            if (rc == FT_OK) {
              CHECK(batches == (chunks + 4) / 5 && done[0] == bytes && done[1] == bytes);
              for (uint32_t f = 0; f < 2; ++f) CHECK(std::memcmp(static_cast<char *>(ft_pool_ptr(pool, off[f])) + 3 * f, src.data() + f * bytes, bytes) == 0);
            }
            CHECK(ft_job_release(pool, job) == FT_OK);
          }
          stand_in_fail(point, 0);
          for (uint32_t f = 0; f < 2; ++f) CHECK(ft_slab_free(pool, off[f]) == FT_OK);
          CHECK(ft_pool_destroy(pool) == FT_OK);
          std::free(dev);
        }
  std::printf("ring_parts done\n");
  return 0;
}
