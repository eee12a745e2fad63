// Batches of pageable sources that are launched in parts (ft_open.cpp), on a machine without a GPU: with tests/host/hip_stand_in.cpp the
// n-th launch or event fails, or none does. The job ends either way, its bytes are in place if it succeeds, and nothing stays busy.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/faastube.h"

extern "C" int stand_in_fail(const char *name, int nth);

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d (%s, n %d)\n", #c, __LINE__, point, n); std::abort(); } } while (0)

int main() {
  const uint64_t MiB = 1 << 20, bytes = 7 * MiB + 12345;
  std::vector<char> src(2 * bytes);
  for (size_t i = 0; i < src.size(); ++i) src[i] = (char)(i * 2654435761u >> 13);
  for (const char *point : {"launch_copy", "hipEventRecord", "hipEventSynchronize", "hipEventCreateWithFlags", "hipStreamWaitEvent"})
    for (uint64_t chunk : {256 * 1024ull, 1ull * MiB, 2ull * MiB})
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
