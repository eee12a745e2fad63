// Error paths of the library's host code, on a machine without a GPU: built with
// tests/host/hip_stand_in.cpp, which can make the n-th call of a runtime function (or of the kernel
// launch) fail. For every such point and n = 1, 2, ... a closed job on each launch route, an open
// job, a merge and a weight change are attempted. Whatever fails, the calls must return FT_OK or
// a negative code (never hang, never crash), nothing may stay busy afterwards (every allocation
// can be freed once the jobs that were accepted have been waited for), and the same jobs run
// again without a failure must put every byte where memcpy puts it.
// Usage: fault_paths
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/faastube.h"

extern "C" int stand_in_fail(const char *name, int nth);
extern "C" int stand_in_calls(const char *name);
extern "C" hipStream_t stand_in_stream(void);

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d (point %s, n %d)\n", #c, __LINE__, g_point, g_n); std::abort(); } } while (0)
static const char *g_point = "-";
static int g_n = 0;

static const uint64_t KiB = 1024, MiB = 1024 * 1024;

struct World {
  char *dev = nullptr, *host = nullptr;
  uint64_t pool_bytes = 64 * MiB, host_bytes = 32 * MiB;
  std::vector<char> expect, host_expect;
  std::vector<char> pageable, pageable_expect;  // ordinary host memory for the jobs that stage
  ft_pool *pool = nullptr;
  std::vector<ft_off_t> allocs;
};

static ft_off_t alloc(World &w, uint64_t n) {
  ft_off_t off = 0;
  CHECK(ft_slab_alloc(w.pool, n, &off) == FT_OK);
  w.allocs.push_back(off);
  return off;
}

// One job of `nfunc` functions moving `bytes` each host->pool (and pool->pool when mixed); its
// expected effect is written into w.expect only when `count` (the job was accepted).
struct JobSpec {
  std::vector<ft_desc> d;
  std::vector<uint32_t> wts;
};

static JobSpec make_job(World &w, uint32_t nfunc, uint64_t bytes, bool mixed, uint64_t salt) {
  JobSpec j;
  for (uint32_t f = 0; f < nfunc; ++f) {
    ft_desc d{};
    d.func = f;
    d.rows = 1;
    d.row_bytes = bytes + f * 16 + 3;
    d.src_pitch = d.dst_pitch = d.row_bytes;
    d.dst_space = FT_POOL;
    d.dst = alloc(w, d.row_bytes + 32) + 5;
    if (mixed && f % 2 == 1) {
      const ft_off_t s = alloc(w, d.row_bytes + 32);
      std::memcpy(w.dev + s, w.host + (salt * 4099 + f * 77) % (w.host_bytes / 2), d.row_bytes + 32);
      std::memcpy(w.expect.data() + s, w.dev + s, d.row_bytes + 32);
      d.src_space = FT_POOL;
      d.src = s + 1;
    } else {
      d.src_space = FT_HOST;
      d.src = reinterpret_cast<uint64_t>(w.host + (salt * 8191 + f * 131) % (w.host_bytes / 2));
    }
    j.d.push_back(d);
    j.wts.push_back(1 + f % 3);
  }
  return j;
}

// One job of n runs of `bytes` bytes or so, on both sides of one allocation each (so 300 of them cost two).
static JobSpec make_runs(World &w, int cls, uint32_t nfunc, uint32_t n, uint64_t bytes, uint64_t salt) {
  JobSpec j;
  const uint64_t step = bytes + 40;
  const ft_off_t a = alloc(w, n * step), b = cls == 2 ? alloc(w, n * step) : 0;
  char *host = w.host + (cls == 1 ? w.host_bytes / 2 + salt * 1 * MiB : salt * 8191);
  for (uint64_t i = 0; i < n * step; ++i)
    if (cls != 0) w.dev[a + i] = w.expect[a + i] = (char)(i * salt >> 5);
  for (uint32_t i = 0; i < n; ++i) {
    ft_desc d{};
    d.func = i % nfunc;
    d.rows = 1;
    d.row_bytes = bytes + i % 7;
    d.src_space = cls == 0 ? FT_HOST : FT_POOL;
    d.dst_space = cls == 1 ? FT_HOST : FT_POOL;
    d.src = cls == 0 ? reinterpret_cast<uint64_t>(host + i * step) : a + i * step + i % 3;
    d.dst = cls == 1 ? reinterpret_cast<uint64_t>(host + i * step) : (cls == 0 ? a : b) + i * step + i % 5;
    j.d.push_back(d);
  }
  for (uint32_t f = 0; f < nfunc; ++f) j.wts.push_back(1 + f % 3);
  return j;
}

static void expect_job(World &w, const JobSpec &j) {
  for (const ft_desc &d : j.d) {
    const char *src = d.src_space == FT_POOL ? w.expect.data() + d.src : reinterpret_cast<const char *>(d.src);
    char *dst = d.dst_space == FT_POOL ? w.expect.data() + d.dst : w.host_expect.data() + (d.dst - reinterpret_cast<uint64_t>(w.host));
    std::memmove(dst, src, d.row_bytes);
  }
}

// One pass over all kinds of job. inject: arm the failure before the pass.
static int pass(World &w, bool inject, const char *point, int n) {
  int failures = 0;
  std::vector<ft_job_t> to_wait, once;  // once: not kept, dead after a wait that succeeds
  auto outcome = [&](int rc, const JobSpec &j, ft_job_t id) {
    CHECK(rc <= 0);
    if (rc == FT_OK) {
      expect_job(w, j);
      to_wait.push_back(id);
    } else {
      failures += 1;
    }
  };
  if (inject) CHECK(stand_in_fail(point, n) == 0);
  // closed jobs: tables inside the launch, a counter pair, uploaded tables (two classes)
  for (int kind = 0; kind < 3; ++kind) {
    JobSpec j = make_job(w, kind == 2 ? 4 : 1, kind == 0 ? 20 * KiB : 3 * MiB, kind == 2, 11 + kind);
    ft_job_t id = 0;
    const int rj = ft_submit_transfers(w.pool, j.d.data(), (uint32_t)j.d.size(), j.wts.data(), (uint32_t)j.wts.size(),
                                       256 * KiB, FT_KEEP, nullptr, &id);
    outcome(rj, j, id);
  }
  // closed jobs as pieces: with the launch, uploaded; each link class, with and without a counter; rows; asked for their schedule
  for (int kind = 0; kind < 8; ++kind) {
    const int cls = kind < 3 ? 2 : kind % 2;
    JobSpec j = make_runs(w, cls, 1 + kind % 4, kind == 0 ? 20 : kind >= 5 ? 10 : 300, kind == 7 ? 100 : 3000, 3 + kind);
    if (kind == 2)
      for (ft_desc &d : j.d) {  // the same bytes as rows of 100
        d.rows = 30;
        d.row_bytes = 100;
        d.src_pitch = 100;
        d.dst_pitch = 101;
      }
    ft_job_t id = 0;
    const int rj = ft_submit_transfers(w.pool, j.d.data(), (uint32_t)j.d.size(), j.wts.data(), (uint32_t)j.wts.size(), 16 * KiB,
                                       kind % 3 == 1 ? FT_TIMING : kind == 6 ? FT_DETACHED : 0, nullptr, &id);
    if (kind == 2 && rj == FT_OK) {
      for (const ft_desc &d : j.d)
        for (uint64_t r = 0; r < d.rows; ++r) std::memcpy(w.expect.data() + d.dst + r * d.dst_pitch, w.expect.data() + d.src + r * d.src_pitch, d.row_bytes);
      to_wait.push_back(id);
      once.push_back(id);
      continue;
    }
    outcome(rj, j, id);
    if (rj == FT_OK && kind % 3 == 1) {
      uint64_t chunks = 0;
      std::vector<uint32_t> func(4096), chunk(4096);
      const int rs = ft_job_schedule(w.pool, id, cls, func.data(), chunk.data(), 4096, &chunks);
      CHECK(rs <= 0);
      if (rs != FT_OK) failures += 1;
      else CHECK(chunks > 0 && func[0] < j.wts.size() && chunk[0] == 0);
    } else if (rj == FT_OK) {
      once.push_back(id);
    }
  }
  // a closed job with pageable memory on both sides (a pinned buffer of its own, copies in ft_wait)
  {
    const uint64_t n = 100 * KiB + 7;
    const ft_off_t in = alloc(w, n + 16), out = alloc(w, n + 16);
    std::memcpy(w.dev + out, w.host + 12345, n);
    std::memcpy(w.expect.data() + out, w.dev + out, n);
    ft_desc d2[2] = {};
    d2[0].func = 0; d2[0].src_space = FT_PAGEABLE; d2[0].src = reinterpret_cast<uint64_t>(w.pageable.data() + 100);
    d2[0].dst_space = FT_POOL; d2[0].dst = in + 3; d2[0].row_bytes = n; d2[0].rows = 1;
    d2[1].func = 0; d2[1].src_space = FT_POOL; d2[1].src = out;
    d2[1].dst_space = FT_PAGEABLE; d2[1].dst = reinterpret_cast<uint64_t>(w.pageable.data() + 2 * MiB + 5); d2[1].row_bytes = n; d2[1].rows = 1;
    const uint32_t one = 1;
    ft_job_t id = 0;
    const int rj = ft_submit_transfers(w.pool, d2, 2, &one, 1, 64 * KiB, FT_KEEP, nullptr, &id);
    CHECK(rj <= 0);
    if (rj == FT_OK) {
      std::memcpy(w.expect.data() + in + 3, w.pageable.data() + 100, n);
      std::memcpy(w.pageable_expect.data() + 2 * MiB + 5, w.expect.data() + out, n);
      to_wait.push_back(id);
    } else {
      failures += 1;
    }
  }
  // an open job, a merge into it, a change of its weights
  JobSpec open = make_job(w, 3, 2 * MiB, true, 29);
  ft_job_t open_id = 0;
  int rc = ft_submit_transfers(w.pool, open.d.data(), (uint32_t)open.d.size(), open.wts.data(), (uint32_t)open.wts.size(),
                               128 * KiB, FT_OPEN | FT_KEEP, nullptr, &open_id);
  outcome(rc, open, open_id);
  if (rc == FT_OK) {
    JobSpec late = make_job(w, 2, 600 * KiB, false, 31);
    ft_job_t late_id = 0;
    int rm = ft_submit_merge(w.pool, open_id, late.d.data(), (uint32_t)late.d.size(), late.wts.data(), (uint32_t)late.wts.size(),
                             FT_KEEP, nullptr, &late_id);
    if (rm == FT_ECLOSED) {
      rm = ft_submit_transfers(w.pool, late.d.data(), (uint32_t)late.d.size(), late.wts.data(), (uint32_t)late.wts.size(), 128 * KiB,
                               FT_KEEP, nullptr, &late_id);
    }
    outcome(rm, late, late_id);
    const uint32_t nw[3] = {5, 1, 2};
    const int rr = ft_job_reweight(w.pool, open_id, nw, 3, nullptr, nullptr);
    CHECK(rr <= 0);
    if (rr != FT_OK) failures += 1;
  }
  stand_in_fail(point, 0);
  // every accepted job comes to an end; a wait may report the failure of a batch
  bool data_defined = true;
  for (ft_job_t id : to_wait) {
    const int rw = ft_wait(w.pool, id);
    CHECK(rw <= 0);
    if (rw != FT_OK) {
      failures += 1;
      data_defined = false;  // some chunks of that sequence were never moved
    }
    if (rw == FT_OK && std::find(once.begin(), once.end(), id) != once.end()) {
      CHECK(ft_wait(w.pool, id) == FT_EINVAL);
      continue;
    }
    const int rl = ft_job_release(w.pool, id);
    if (rl != FT_OK) std::fprintf(stderr, "release of job %llu -> %d (wait gave %d)\n", (unsigned long long)id, rl, rw);
    CHECK(rl == FT_OK);
  }
  // nothing is left busy
  for (ft_off_t off : w.allocs) CHECK(ft_slab_free(w.pool, off) == FT_OK);
  w.allocs.clear();
  uint64_t total = 0, live = 1;
  CHECK(ft_pool_usage(w.pool, &total, &live) == FT_OK && live == 0);
  if (data_defined) {
    CHECK(std::memcmp(w.dev, w.expect.data(), w.pool_bytes) == 0);
    CHECK(std::memcmp(w.host, w.host_expect.data(), w.host_bytes) == 0);
    CHECK(w.pageable == w.pageable_expect);
  } else {
    std::memcpy(w.expect.data(), w.dev, w.pool_bytes);  // start the next pass from what is there
    std::memcpy(w.host_expect.data(), w.host, w.host_bytes);
    w.pageable_expect = w.pageable;
  }
  return failures;
}

// A job by the copy engines launches no kernel, however long its tables.
static void copy_engines_alone(World &w) {
  std::vector<ft_desc> d(1000);
  ft_off_t src = 0, dst = 0;
  CHECK(ft_slab_alloc(w.pool, 1 * MiB, &src) == FT_OK && ft_slab_alloc(w.pool, 1 * MiB, &dst) == FT_OK);
  for (size_t i = 0; i < d.size(); ++i) {
    std::memset(&d[i], 0, sizeof(ft_desc));
    d[i].src_space = d[i].dst_space = FT_POOL;
    d[i].src = src + i * 1024;
    d[i].dst = dst + i * 1024;
    d[i].row_bytes = 700;
    d[i].rows = 1;
  }
  for (uint64_t i = 0; i < 1 * MiB; ++i) w.dev[src + i] = (char)(i * 97 >> 3);
  const uint32_t weight = 1;
  ft_job_t job = 0;
  CHECK(stand_in_fail("launch_copy", 1) == 0);
  CHECK(ft_submit_transfers(w.pool, d.data(), (uint32_t)d.size(), &weight, 1, 64 * KiB, FT_PATH_DMA, nullptr, &job) == FT_OK);
  CHECK(ft_wait(w.pool, job) == FT_OK);
  CHECK(stand_in_fail("launch_copy", 0) == 0);
  for (const ft_desc &x : d) CHECK(std::memcmp(w.dev + x.src, w.dev + x.dst, x.row_bytes) == 0);
  CHECK(ft_slab_free(w.pool, src) == FT_OK && ft_slab_free(w.pool, dst) == FT_OK);
  std::memcpy(w.expect.data(), w.dev, w.pool_bytes);
}

// More jobs at once than there are counters: those that find none take the general route, and the counters come back.
static void counters_run_out(World &w) {
  for (int round = 0; round < 2; ++round) {
    std::vector<ft_job_t> jobs;
    JobSpec j = make_runs(w, 0, 2, 4, 100 * KiB, 17);
    const int before = stand_in_calls("launch_copy"), pieces = stand_in_calls("launch_pieces");
    for (int i = 0; i < 300; ++i) {
      ft_job_t id = 0;
      CHECK(ft_submit_transfers(w.pool, j.d.data(), (uint32_t)j.d.size(), j.wts.data(), (uint32_t)j.wts.size(), 64 * KiB, 0, nullptr, &id) == FT_OK);
      jobs.push_back(id);
    }
    CHECK(stand_in_calls("launch_pieces") - pieces == 256 && stand_in_calls("launch_copy") - before == 44);
    for (ft_job_t id : jobs) CHECK(ft_wait(w.pool, id) == FT_OK);
    expect_job(w, j);
    for (ft_off_t off : w.allocs) CHECK(ft_slab_free(w.pool, off) == FT_OK);
    w.allocs.clear();
  }
  CHECK(std::memcmp(w.dev, w.expect.data(), w.pool_bytes) == 0);
}

// A job out of pageable memory that fails for want of a table buffer gives its pinned buffer back: the next attempt takes the same one.
static void pinned_buffer_comes_back(World &w) {
  JobSpec j = make_runs(w, 0, 1, 8000, 100, 23);  // tables beyond every buffer that is there
  for (size_t i = 0; i < j.d.size(); ++i) {
    j.d[i].src_space = FT_PAGEABLE;
    j.d[i].src = reinterpret_cast<uint64_t>(w.pageable.data() + i * 120);
  }
  const int before = stand_in_calls("hipHostMalloc");
  for (int i = 0; i < 5; ++i) {
    ft_job_t id = 0;
    CHECK(stand_in_fail("hipMalloc", 1) == 0);
    CHECK(ft_submit_transfers(w.pool, j.d.data(), (uint32_t)j.d.size(), j.wts.data(), 1, 2 * MiB, 0, nullptr, &id) == FT_EHIP);
  }
  CHECK(stand_in_fail("hipMalloc", 0) == 0);
  CHECK(stand_in_calls("hipHostMalloc") - before <= 1);
  for (ft_off_t off : w.allocs) CHECK(ft_slab_free(w.pool, off) == FT_OK);
  w.allocs.clear();
}

// A detached job leaves the caller's stream alone unless it is small enough to go along with its launch, whatever it is launched as.
static void detached_jobs(World &w) {
  hipStream_t mine;
  CHECK(hipStreamCreate(&mine) == hipSuccess);
  struct {
    int cls;
    uint32_t n;
    uint64_t bytes;
    bool on_mine, as_pieces;
  } cases[] = {{2, 20, 3000, true, true},   {2, 200, 3000, false, false}, {2, 300, 3000, false, false}, {0, 20, 3000, true, true}, {0, 20, 30000, true, true},
               {0, 300, 1000, false, false}, {1, 20, 30000, true, true},   {1, 300, 1000, false, false}, {0, 20, 100000, false, false}};
  for (auto &c : cases)
    for (uint32_t flags : {0u, (uint32_t)FT_DETACHED}) {
      JobSpec j = make_runs(w, c.cls, 2, c.n, c.bytes, 5);
      const int pieces = stand_in_calls("launch_pieces"), copies = stand_in_calls("launch_copy");
      ft_job_t id = 0;
      CHECK(ft_submit_transfers(w.pool, j.d.data(), (uint32_t)j.d.size(), j.wts.data(), (uint32_t)j.wts.size(), 64 * KiB, flags, mine, &id) == FT_OK);
      const bool on_mine = flags == 0 || c.on_mine, as_pieces = flags == 0 || c.as_pieces;
      CHECK((stand_in_stream() == mine) == on_mine);
      CHECK((stand_in_calls("launch_copy") == copies) == as_pieces && (as_pieces ? stand_in_calls("launch_pieces") > pieces : true));
      CHECK(ft_wait(w.pool, id) == FT_OK);
      expect_job(w, j);
      for (ft_off_t off : w.allocs) CHECK(ft_slab_free(w.pool, off) == FT_OK);
      w.allocs.clear();
    }
  CHECK(std::memcmp(w.dev, w.expect.data(), w.pool_bytes) == 0);
  CHECK(std::memcmp(w.host, w.host_expect.data(), w.host_bytes) == 0);
  CHECK(hipStreamDestroy(mine) == hipSuccess);
}

int main() {
  World w;
  CHECK(hipMalloc(reinterpret_cast<void **>(&w.dev), w.pool_bytes) == hipSuccess);
  CHECK(hipHostMalloc(reinterpret_cast<void **>(&w.host), w.host_bytes, 0) == hipSuccess);
  for (uint64_t i = 0; i < w.host_bytes; ++i) w.host[i] = (char)(i * 2654435761u >> 13);
  w.host_expect.assign(w.host, w.host + w.host_bytes);
  std::memset(w.dev, 0, w.pool_bytes);
  w.expect.assign(w.pool_bytes, 0);
  CHECK(ft_pool_create(&w.pool, w.dev, w.pool_bytes, 64 * KiB, 0) == FT_OK);
  CHECK(ft_host_window_add(w.pool, w.host, w.host_bytes) == FT_OK);
  w.pageable.assign(4 * MiB, 0);
  for (uint64_t i = 0; i < 1 * MiB; ++i) w.pageable[i] = (char)(i * 40503u >> 7);
  w.pageable_expect = w.pageable;
  CHECK(ft_pageable_window_add(w.pool, w.pageable.data(), w.pageable.size()) == FT_OK);
  CHECK(pass(w, false, "-", 0) == 0);  // also creates the per-device resources
  copy_engines_alone(w);
  counters_run_out(w);
  pinned_buffer_comes_back(w);
  detached_jobs(w);
  const char *points[] = {"hipMemcpyAsync", "hipEventRecord", "hipStreamWaitEvent", "hipEventCreateWithFlags",
                          "hipMalloc",      "hipHostMalloc",  "hipEventSynchronize", "launch_copy", "launch_pieces"};
  int hit = 0;
  for (const char *point : points)
    for (int n = 1; n <= 20; ++n) {
      g_point = point;
      g_n = n;
      const int failures = pass(w, true, point, n);
      hit += failures > 0;
      g_point = "-";
      CHECK(pass(w, false, "-", 0) == 0);  // and everything works again afterwards
    }
  std::fprintf(stderr, "%d of %d injected failures were met by a call\n", hit, (int)(sizeof(points) / sizeof(points[0])) * 20);
  CHECK(hit >= 60);
  CHECK(ft_pool_destroy(w.pool) == FT_OK);
  std::printf("fault_paths done\n");
  return 0;
}
