// Host check of what the wave kernel (one tile per wavefront) relies on, built with the sanitizers: the windows that a
// piece of a transfer is cut into (ft_windows.h, the kernel's own arithmetic) stay inside the piece and cover it, and
// a ticket decoded without a cursor - 64 table entries compared at a time - names the bytes and the descriptor that
// the general walk names, for every job that launch_code sends to that kernel.
// Usage: wave_tiles <first seed> <count>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "../../paper_2411_01830_amd/csrc/ft_plan.h"
#include "../../paper_2411_01830_amd/csrc/ft_windows.h"
using namespace ft;
static uint64_t g_seed;
#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "FAIL %s line %d seed %llu\n", #c, __LINE__, (unsigned long long)g_seed); std::abort(); } } while (0)

template <uint32_t W>
static void rows(uint32_t rb, uint64_t p, uint32_t take) {
  const uint32_t c0 = (uint32_t)(p % rb);
  const RowWindows w = row_windows<W>(rb, c0, take);
  std::vector<uint8_t> hit(take, 0);
  auto mark = [&](uint64_t row, uint64_t col, uint32_t n) {
    const uint64_t b = row * rb + col;
    CHECK(col + n <= rb && b >= c0 && b + n <= (uint64_t)c0 + take);
    for (uint32_t i = 0; i < n; ++i) hit[b - c0 + i] = 1;
  };
  for (uint32_t q = 0; q < w.count; ++q) {
    const RowCursor c = row_window<W>(w, q);
    mark(c.row, row_window_col<W>(w, c), W);
    if (q < 64) continue;
    RowCursor d = row_window<W>(w, q - 64);  // reached by the kernel's step of 64 windows as well
    row_window_next<W>(w, 64 / w.per_row, 64 % w.per_row * W, &d);
    CHECK(d.row == c.row && d.col == c.col);
  }
  CHECK(w.short_first < W && w.short_last < W && W <= 16);
  if (w.short_first) mark(0, c0, w.short_first);
  if (w.short_last) mark(w.more, 0, w.short_last);
  for (uint8_t h : hit) CHECK(h);
}

static void run(uint64_t dst, uint32_t n) {
  const RunWindows w = run_windows(dst, n);
  std::vector<uint8_t> hit(n, 0);
  for (uint32_t j = 0; j < w.count + 130; ++j) {  // lanes past the last window repeat it
    const uint32_t o = run_window_at(w, j);
    CHECK(o + 16 <= n);
    if (j > 0 && j + 1 < w.count) CHECK(((dst + o) & 15) == 0);
    for (uint32_t i = 0; i < 16; ++i) hit[o + i] = 1;
  }
  CHECK(w.count <= n / 16 + 2);
  for (uint8_t h : hit) CHECK(h);
}

static uint64_t n_tickets, n_jobs[128];

static int decode_all(ClassPlan &cp, uint64_t C, int cls, bool alone);

static void job(std::mt19937_64 &r) {
  auto U = [&](uint64_t a, uint64_t b) { return a + r() % (b - a + 1); };
  ClassPlan cp;
  const uint64_t Cs[] = {1024, 4096, 65536, 100000 / 16 * 16, 2u << 20};
  const uint64_t C = Cs[U(0, 4)];
  const uint32_t nf = (uint32_t)(r() % 4 == 0 ? U(1, 1024) : U(1, 9));
  const uint64_t scale = 1ull << U(6, 20);
  for (uint32_t f = 0; f < nf; ++f) {
    Func fn{};
    fn.desc_off = (uint32_t)cp.xfers.size();
    fn.ndesc = (uint32_t)(r() % 8 == 0 ? U(60, 140) : U(1, 7));
    if (r() % 64 == 0) fn.ndesc = 5000;
    for (uint32_t i = 0; i < fn.ndesc; ++i) {
      Xfer x{};
      x.rows = r() % 3 == 0 ? U(2, 60) : 1;
      x.row_bytes = x.rows > 1 ? U(16, 6000) : U(1, fn.ndesc > 1000 ? 300 : scale);
      x.src_pitch = x.dst_pitch = x.row_bytes + U(0, 99);
      x.stream_off = fn.stream_bytes;
      fn.stream_bytes += x.row_bytes * x.rows;
      cp.xfers.push_back(x);
    }
    fn.nchunks = (fn.stream_bytes + C - 1) / C;
    fn.func = f;
    fn.weight = (uint32_t)U(1, 8);
    cp.funcs.push_back(fn);
    cp.payload += fn.stream_bytes;
  }
  const int cls = (int)U(0, 5) < 4 ? FT_P2P : (int)U(FT_H2P, FT_P2H);
  decode_all(cp, C, cls, r() % 4 != 0);
}

// The launch code that a job gets, and every n-th ticket of it as the wave kernel decodes it against the general walk.
static int decode_all(ClassPlan &cp, uint64_t C, int cls, bool alone) {
  CHECK(build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);
  const int code = launch_code(cp, cls, C, false, alone);
  CHECK(launch_code(cp, cls, C, true, true) == cls && (cls == FT_P2P || launch_code(cp, cls, C, false, false) == cls));
  CHECK(code < kWaveTiles || (cls == FT_P2P) == ((code & (kWaveFromHost | kWaveToHost)) == 0));
  n_jobs[code] += 1;
  if (code < kWaveTiles) return code;
  uint64_t tile;
  uint32_t tpc;
  tile_shape(C, wave_tile(code, cp.payload), &tile, &tpc);
  std::vector<Skip> skips;
  uint64_t nt;
  build_skips(cp, C, tile, tpc, &skips, &nt);
  CHECK(nt < (1u << 31) && tile <= 16384 && wave_code_threads(code) != 0);
  const uint64_t wg = wave_workgroups(256, code, nt);
  CHECK(wg > 0 && wg <= nt && ((code & 15) != kWaveTiles || wg == nt) && wg * wave_code_threads(code) < (1ull << 32));
  const uint64_t stride = nt > 3000 ? nt / 3000 : 1;
  for (uint64_t t = 0; t < nt; t += stride, ++n_tickets) {
    // as the wave kernel decodes it
    uint32_t v = (uint32_t)t;
    for (size_t j0 = 0; j0 < skips.size(); j0 += 64) {
      uint32_t before = 0;
      for (size_t j = j0; j < j0 + 64 && j < skips.size(); ++j)
        if (skips[j].at <= t) {
          CHECK(skips[j].gap < 65536);
          v += (uint32_t)skips[j].gap;
          before += 1;
        }
      if (before < 64) break;
    }
    const uint32_t rank = v / tpc, ti = v - rank * tpc;
    uint32_t idx = 0;
    for (size_t j0 = 0; j0 < cp.phases.size() && idx == j0; j0 += 64)
      for (size_t j = j0; j < j0 + 64 && j < cp.phases.size(); ++j) idx += cp.phases[j].rank_base <= rank ? 1 : 0;
    const Phase &ph = cp.phases.at(idx - 1);
    const uint32_t rel = rank - (uint32_t)ph.rank_base, round = rel / ph.nslots;
    const Slot &sl = cp.slots.at(ph.slot_off + rel - round * ph.nslots);
    const uint64_t k = (uint64_t)(((uint32_t)ph.round_base + round) * sl.weight + sl.i);
    const Func &f = cp.funcs[sl.fl];
    const uint64_t b0 = k * C + ti * tile;
    uint32_t x = f.desc_off, nx = f.ndesc;
    while (nx > 1) {
      const uint32_t step = (nx + 63) / 64;
      uint32_t at = 0;
      for (uint32_t lane = 0; lane < 64; ++lane) at += lane * step < nx && cp.xfers[x + lane * step].stream_off <= b0 ? 1 : 0;
      at = (at - 1) * step;
      x += at;
      nx = step < nx - at ? step : nx - at;
    }
    // the general walk
    const uint64_t gv = ticket_to_tile(skips.data(), (uint32_t)skips.size(), t);
    const ChunkId id = decode_rank(cp.phases.data(), (uint32_t)cp.phases.size(), cp.slots.data(), gv / tpc);
    CHECK(gv == v && id.fl == sl.fl && id.k == k);
    CHECK(x == find_xfer(cp.xfers.data(), f.desc_off, f.desc_off + f.ndesc - 1, b0));
    CHECK(b0 < f.stream_bytes && cp.xfers[x].stream_off <= b0);
  }
  return code;
}

// A job for every rule of launch_code: what it says, and the tickets of it decoded.
static void each_rule() {
  const uint64_t KiB = 1 << 10, MiB = 1 << 20;
  struct Rule {
    int cls;
    bool alone;
    uint64_t bytes;  // of the whole job, in `pieces` descriptors of eight functions
    uint64_t pieces, row_bytes;  // row_bytes 0: contiguous
    uint64_t misaligned;
    int code;
  };
  const int S = kWaveStreams, F = kWaveFromHost, T = kWaveToHost;
  const Rule rules[] = {
      {FT_P2P, true, 10 * MiB, 64, 0, 0, kWaveTiles},
      {FT_P2P, false, 10 * MiB, 64, 0, 0, kWaveTiles},
      {FT_P2P, true, 30 * MiB, 64, 0, 0, kWaveOnePerUnit},
      {FT_P2P, false, 30 * MiB, 64, 0, 0, FT_P2P},
      {FT_P2P, true, 60 * MiB, 64, 0, 0, FT_P2P},
      {FT_P2P, true, 60 * MiB, 1, 0, 0, kWaveOnePerUnit},
      {FT_P2P, true, 60 * MiB, 64, 0, 3, kWaveOnePerUnit},
      {FT_P2P, false, 60 * MiB, 64, 0, 3, FT_P2P},
      {FT_P2P, true, 200 * MiB, 1, 0, 0, FT_P2P},
      {FT_P2P, true, 200 * MiB, 64, 0, 3, FT_P2P},
      {FT_P2P, true, 20 * MiB, 64, 300, 0, kWaveTwoPerUnit},
      {FT_P2P, true, 20 * MiB, 64, 5000, 0, kWaveOnePerUnit},
      {FT_P2P, false, 20 * MiB, 64, 5000, 0, kWaveTwoPerUnit},
      {FT_P2P, true, 200 * MiB, 64, 300, 0, kWaveTwoPerUnit | S},
      {FT_P2P, true, 200 * MiB, 64, 5000, 0, kWaveOnePerUnit | S},
      {FT_P2P, true, 200 * MiB, 64, 65536, 0, FT_P2P},
      {FT_P2P, false, 200 * MiB, 64, 300, 0, kWaveBeside | S},
      {FT_P2P, true, 10 * MiB, 64, 15, 0, FT_P2P},
      {FT_H2P, true, 100 * KiB, 3, 0, 0, kWaveTiles | F},
      {FT_P2H, true, 100 * KiB, 3, 0, 0, kWaveTiles | T},
      {FT_H2P, true, 2 * MiB, 600, 0, 0, kWaveLink | F},
      {FT_P2H, true, 2 * MiB, 600, 0, 0, kWaveLink | T},
      {FT_P2H, true, 2 * MiB, 300, 0, 0, FT_P2H},
      {FT_H2P, true, 2 * MiB, 8, 300, 0, kWaveLink | F},
      {FT_H2P, false, 2 * MiB, 600, 0, 0, FT_H2P},
  };
  for (const Rule &q : rules)
    for (uint64_t C : {64 * KiB, 2 * MiB}) {
      ClassPlan cp;
      const uint32_t nf = q.pieces < 8 ? 1 : 8;
      for (uint32_t f = 0; f < nf; ++f) {
        Func fn{};
        fn.desc_off = (uint32_t)cp.xfers.size();
        fn.func = f;
        fn.weight = 1 + f % 3;
        for (uint64_t i = f; i < q.pieces; i += nf, ++fn.ndesc) {
          Xfer x{};
          x.row_bytes = q.row_bytes ? q.row_bytes : q.bytes / q.pieces;
          x.rows = q.row_bytes ? q.bytes / q.pieces / q.row_bytes : 1;
          x.src_pitch = x.dst_pitch = x.row_bytes + 99;
          x.dst = q.misaligned;
          x.stream_off = fn.stream_bytes;
          fn.stream_bytes += x.row_bytes * x.rows;
          cp.xfers.push_back(x);
        }
        fn.nchunks = (fn.stream_bytes + C - 1) / C;
        cp.funcs.push_back(fn);
        cp.payload += fn.stream_bytes;
      }
      CHECK(decode_all(cp, C, q.cls, q.alone) == q.code);
    }
}

// A launch has fewer than 2^32 threads however much there is to move: pitched rows in the smallest chunks that the wave
// kernel takes, up to what fits the device's memory twice, alone and beside host-link traffic.
static void largest_launches() {
  for (uint64_t gib = 1; gib <= 144; gib *= 2)
    for (uint64_t C : {1024ull, 4096ull, 2ull << 20})
      for (uint64_t rb : {16ull, 2000ull, 5760ull, 60000ull})
        for (int alone = 0; alone < 2; ++alone) {
          ClassPlan cp;
          Func fn{};
          fn.weight = 1;
          while (fn.stream_bytes < gib << 30) {
            Xfer x{};
            x.row_bytes = rb;
            x.rows = (1ull << 30) / rb + 1;
            x.src_pitch = x.dst_pitch = rb + 16;
            x.stream_off = fn.stream_bytes;
            fn.stream_bytes += x.row_bytes * x.rows;
            cp.xfers.push_back(x);
          }
          fn.ndesc = (uint32_t)cp.xfers.size();
          fn.nchunks = cp.nchunks = (fn.stream_bytes + C - 1) / C;
          cp.payload = fn.stream_bytes;
          cp.funcs.push_back(fn);
          const int code = launch_code(cp, FT_P2P, C, false, alone != 0);
          CHECK(code >= kWaveTiles || C == 1024);
          if (code < kWaveTiles) continue;
          uint64_t tile;
          uint32_t tpc;
          tile_shape(C, wave_tile(code, cp.payload), &tile, &tpc);
          const uint64_t nt = cp.nchunks * tpc, wg = wave_workgroups(256, code, nt);
          CHECK(nt < (1ull << 31) && wg * wave_code_threads(code) < (1ull << 32));
        }
}

// Rows however far apart: what is sent to the wave kernel fits its 32-bit distances from a tile's first row to the end of its
// last, and rows of a few MiB apart are sent, as are jobs of up to 1024 functions.
static void far_rows() {
  for (uint64_t rb : {16ull, 17ull, 64ull, 100ull, 2000ull, 8191ull, 8208ull, 60000ull, 1ull << 20})
    for (uint64_t pitch = rb; pitch < 1ull << 34; pitch = pitch * 3 / 2 + 1)
      for (uint64_t C : {1024ull, 65536ull, 2ull << 20, 1ull << 29})
        for (int cls = 0; cls < FT_NCLASS; ++cls)
          for (uint32_t nf : {1u, 257u, 1024u, 1025u}) {
            ClassPlan cp;
            for (uint32_t f = 0; f < nf; ++f) {
              Func fn{};
              Xfer x{};
              x.row_bytes = rb;
              x.rows = 40;
              x.src_pitch = f % 2 ? rb : pitch;
              x.dst_pitch = f % 2 ? pitch : rb;
              fn.stream_bytes = rb * x.rows;
              fn.nchunks = (fn.stream_bytes + C - 1) / C;
              cp.nchunks += fn.nchunks;
              cp.payload += fn.stream_bytes;
              cp.xfers.push_back(x);
              cp.funcs.push_back(fn);
            }
            const int code = launch_code(cp, cls, C, false, true);
            if (cls == FT_P2P && cp.payload <= 16u << 20) CHECK((code >= kWaveTiles) == (nf <= 1024 && pitch <= 0xffffffffu / (8208 / rb + 3)));
            if (code < kWaveTiles) continue;
            uint64_t tile;
            uint32_t tpc;
            tile_shape(C, wave_tile(code, cp.payload), &tile, &tpc);
            CHECK(((tile + rb - 2) / rb + 1) * pitch + rb < 1ull << 32);
          }
}

int main(int argc, char **argv) {
  const uint64_t first = argc > 1 ? strtoull(argv[1], 0, 10) : 1, count = argc > 2 ? strtoull(argv[2], 0, 10) : 50;
  largest_launches();
  each_rule();
  for (int code : {kWaveTiles, kWaveTwoPerUnit, kWaveOnePerUnit, kWaveTwoPerUnit | kWaveStreams, kWaveOnePerUnit | kWaveStreams, kWaveBeside | kWaveStreams,
                   kWaveTiles | kWaveFromHost, kWaveTiles | kWaveToHost, kWaveLink | kWaveFromHost, kWaveLink | kWaveToHost, (int)FT_P2P, (int)FT_H2P, (int)FT_P2H})
    CHECK(n_jobs[code] > 0);
  far_rows();
  for (uint32_t d = 0; d < 16; ++d)
    for (uint32_t n = 16; n < 9000; n += n < 200 ? 1 : 61) run(d, n);
  for (g_seed = first; g_seed < first + count; ++g_seed) {
    std::mt19937_64 r(g_seed);
    auto U = [&](uint64_t a, uint64_t b) { return a + r() % (b - a + 1); };
    for (int i = 0; i < 3000; ++i) {
      const uint32_t rb = (uint32_t)(i % 97 == 0 ? (1u << 30) - U(1, 99) : U(16, i % 3 == 0 ? 40 : i % 3 == 1 ? 400 : 70000));
      const uint64_t p = i % 2 ? rb * U(0, 9) : i % 97 == 0 ? rb - U(1, 300) : U(0, 9ull * rb);
      rows<16>(rb, p, (uint32_t)U(1, i % 5 == 0 ? 40 : 16400));
      rows<4>((uint32_t)U(4, 15), U(0, 100000), (uint32_t)U(1, 3000));
      rows<1>((uint32_t)U(1, 3), U(0, 100000), (uint32_t)U(1, 3000));
    }
    for (int i = 0; i < 8; ++i) job(r);
  }
  std::printf("tickets %llu; jobs: own kernel %llu, a workgroup per tile %llu, two workgroups per unit %llu, one %llu, host link %llu\n",
              (unsigned long long)n_tickets, (unsigned long long)n_jobs[FT_P2P], (unsigned long long)n_jobs[kWaveTiles],
              (unsigned long long)n_jobs[kWaveTwoPerUnit], (unsigned long long)n_jobs[kWaveOnePerUnit], (unsigned long long)(n_jobs[kWaveLink | kWaveFromHost] + n_jobs[kWaveLink | kWaveToHost] + n_jobs[kWaveTiles | kWaveFromHost] + n_jobs[kWaveTiles | kWaveToHost]));
  std::printf("done %llu..%llu\n", (unsigned long long)first, (unsigned long long)(first + count - 1));
  return 0;
}
