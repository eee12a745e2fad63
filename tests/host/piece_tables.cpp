// A class written out as pieces (ft_pieces.h) against the general walk over its tables: the same bytes in the same order,
// and the kernels' tile and window arithmetic carried out here moves each byte to its place, touches nothing outside the
// ranges of the descriptors and keeps to the windows that the kernels hold in registers. Random jobs of runs and pitched rows
// of every width, pitch and alignment, one to thirty functions, chunks of 1 KiB and more.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../include/faastube.h"
#include "../../paper_2411_01830_amd/csrc/ft_pieces.h"
#include "../../paper_2411_01830_amd/csrc/ft_plan.h"

using namespace ft;

static uint64_t g_seed;
#define CHECK(x)                                                                                   \
  do {                                                                                             \
    if (!(x)) {                                                                                    \
      std::fprintf(stderr, "%s:%d seed %llu: %s\n", __FILE__, __LINE__, (unsigned long long)g_seed, #x); \
      std::exit(1);                                                                                \
    }                                                                                              \
  } while (0)

static uint64_t n_tiles, n_rows, n_parts, n_merged, n_edges;

static void move(uint64_t d, uint64_t s, uint32_t n) { std::memcpy(reinterpret_cast<void *>(d), reinterpret_cast<const void *>(s), n); }

static void move_run(uint64_t d, uint64_t s, uint32_t n, uint32_t tile, bool by_source) {
  if (n < 16) return move(d, s, n);
  const RunWindows w = run_windows(by_source ? s : d, n);
  CHECK(w.count <= (tile == kStreamTile ? 1024u : 512u));
  for (uint32_t j = 0; j < w.count; ++j) {
    const uint32_t at = run_window_at(w, j);
    CHECK(at + 16 <= n);
    move(d + at, s + at, 16);
  }
}

// the tiles of piece i, moved as the kernels do
static void move_piece(const PieceTables &t, uint32_t i, bool by_source) {
  const uint32_t ntiles = (i + 1 < t.n ? t.first[i + 1] : t.ntiles) - t.first[i];
  CHECK(ntiles > 0);
  uint64_t moved = 0;
  for (uint32_t no = 0; no < ntiles; ++no, ++n_tiles) {
    uint64_t d = t.at[i].dst, s = t.at[i].src;
    uint32_t row, begin, n;
    if (t.shape == nullptr || t.shape[i] == 0) {
      const uint64_t side = by_source ? s : d;
      run_tile(side, t.len[i], t.tile, no, &begin, &n);
      CHECK(n > 0 && n <= t.tile && begin + n <= t.len[i] && begin == moved);
      CHECK(no == 0 || (side + begin) % kPieceLine == 0);
      move_run(d + begin, s + begin, n, t.tile, by_source);
      moved += n;
      continue;
    }
    const PieceRows &r = t.shapes[t.shape[i] - 1];
    const PieceEdges &e = t.edges[i];
    if (!(r.per & kPartsOfRow)) {
      const RowWindows w = rows_tile(r, t.len[i], e, no, &row);
      n = w.more + 1;
      CHECK(row == moved && row + n <= t.len[i] && w.per_row == windows_of_row(r.row_bytes) && w.count <= 512 && w.count * 16 <= t.tile);
      for (uint32_t g = 0; g < w.count; ++g) {
        const RowCursor c = row_window<16>(w, g);
        const uint32_t col = row_window_col<16>(w, c);
        CHECK(c.row <= w.more && col + 16 <= (row + c.row + 1 == t.len[i] ? e.to : r.row_bytes) && col >= (row + c.row == 0 ? e.from : 0));
        // distances of 32 bits
        CHECK((uint64_t)c.row * r.src_pitch + col + 16 < 1ull << 32 && (uint64_t)c.row * r.dst_pitch + col + 16 < 1ull << 32);
        move(d + (uint64_t)(row + c.row) * r.dst_pitch + col, s + (uint64_t)(row + c.row) * r.src_pitch + col, 16);
      }
      CHECK(w.short_first < 16 && w.short_last < 16);
      move(d + (uint64_t)row * r.dst_pitch + w.c0, s + (uint64_t)row * r.src_pitch + w.c0, w.short_first);
      move(d + (uint64_t)(row + w.more) * r.dst_pitch, s + (uint64_t)(row + w.more) * r.src_pitch, w.short_last);
      n_edges += w.short_first != 0 || w.short_last != 0;
      moved += n;
      ++n_rows;
    } else {
      CHECK(e.from == 0 && e.to == r.row_bytes);
      row_part(r, no, &row, &begin, &n);
      CHECK(row < t.len[i] && n > 0 && n <= t.tile && begin + n <= r.row_bytes);
      CHECK((uint64_t)row * r.row_bytes + begin == moved);
      move_run(d + (uint64_t)row * r.dst_pitch + begin, s + (uint64_t)row * r.src_pitch + begin, n, t.tile, by_source);
      moved += n;
      ++n_parts;
    }
  }
  const PieceRows *r = t.shape != nullptr && t.shape[i] != 0 ? &t.shapes[t.shape[i] - 1] : nullptr;
  CHECK(moved == (r && (r->per & kPartsOfRow) ? (uint64_t)t.len[i] * r->row_bytes : t.len[i]));
}

struct Byte {
  uint64_t src, dst;
  bool operator==(const Byte &o) const { return src == o.src && dst == o.dst; }
};

static void bytes_of(std::vector<Byte> &out, const Xfer &x, uint64_t p, uint64_t n) {
  for (; n > 0; ++p, --n)
    out.push_back(Byte{x.src + p / x.row_bytes * x.src_pitch + p % x.row_bytes, x.dst + p / x.row_bytes * x.dst_pitch + p % x.row_bytes});
}

static void job(std::mt19937_64 &r) {
  auto U = [&](uint64_t a, uint64_t b) { return a + r() % (b - a + 1); };
  const uint64_t C = U(0, 3) == 0 ? 16 * U(64, 200) : 1024ull << U(0, 7);
  const uint32_t F = (uint32_t)(U(0, 3) == 0 ? 1 : U(0, 4) == 0 ? U(17, 30) : U(2, 9));
  const int kind = (int)U(0, 3);  // 0: runs, 1: also rows, 2: rows, 3: runs that touch each other
  std::vector<uint8_t> src(1 << 20), dst(1 << 20, 0xA5), want;
  for (size_t i = 0; i < src.size(); ++i) src[i] = (uint8_t)r();
  uint64_t sa = U(0, 200), da = U(0, 200);
  ClassPlan cp;
  for (uint32_t f = 0; f < F; ++f) {
    Func fn{};
    fn.desc_off = (uint32_t)cp.xfers.size();
    fn.func = f;
    fn.weight = (uint32_t)U(1, 9);
    const uint32_t nd = (uint32_t)U(1, F == 1 ? 60 : 6);
    for (uint32_t i = 0; i < nd; ++i) {
      Xfer x{};
      x.rows = kind == 2 || (kind == 1 && U(0, 1)) ? U(2, 40) : 1;
      x.row_bytes = x.rows == 1 ? U(1, U(0, 5) == 0 ? 20000 : 900) : U(16, U(0, 9) == 0 ? 11000 : U(0, 1) ? 40 : 400);
      if (x.rows > 1 && U(0, 9) == 0) {  // about a whole number of tiles
        x.row_bytes = (1024ull << U(0, 3)) * U(1, 3) - 20 + U(0, 40);
        x.rows = U(2, 5);
      }
      x.src_pitch = x.row_bytes + (x.rows > 1 ? U(0, 90) : 0);
      x.dst_pitch = x.row_bytes + (x.rows > 1 ? U(x.src_pitch == x.row_bytes ? 1 : 0, 90) : 0);
      const uint64_t es = (x.rows - 1) * x.src_pitch + x.row_bytes, ed = (x.rows - 1) * x.dst_pitch + x.row_bytes;
      if (sa + es > src.size() || da + ed > dst.size()) break;
      x.src = reinterpret_cast<uint64_t>(src.data()) + sa;
      x.dst = reinterpret_cast<uint64_t>(dst.data()) + da;
      sa += es + (kind == 3 ? 0 : U(0, 33));
      da += ed + (kind == 3 ? 0 : U(0, 33));
      x.stream_off = fn.stream_bytes;
      fn.stream_bytes += x.row_bytes * x.rows;
      cp.xfers.push_back(x);
      cp.pitched += x.rows > 1;
      ++fn.ndesc;
    }
    if (fn.ndesc == 0) continue;
    fn.nchunks = (fn.stream_bytes + C - 1) / C;
    cp.payload += fn.stream_bytes;
    cp.funcs.push_back(fn);
  }
  CHECK(build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);

  // the general walk, chunk by chunk
  std::vector<Byte> order;
  uint64_t places = 0;  // where it goes from one function to another
  uint32_t before = ~0u;
  for (uint64_t rank = 0; rank < cp.nchunks; ++rank) {
    const ChunkId id = decode_rank(cp.phases.data(), (uint32_t)cp.phases.size(), cp.slots.data(), rank);
    const Func &fn = cp.funcs[id.fl];
    places += id.fl != before;
    before = id.fl;
    uint64_t pos = id.k * C;
    const uint64_t end = pos + C < fn.stream_bytes ? pos + C : fn.stream_bytes;
    uint32_t x = find_xfer(cp.xfers.data(), fn.desc_off, fn.desc_off + fn.ndesc - 1, pos);
    while (pos < end) {
      const Xfer &X = cp.xfers[x++];
      const uint64_t q = pos - X.stream_off, left = X.row_bytes * X.rows - q, n = left < end - pos ? left : end - pos;
      bytes_of(order, X, q, n);
      pos += n;
    }
  }
  CHECK(order.size() == cp.payload);
  want = dst;
  for (const Byte &b : order) want[b.dst - reinterpret_cast<uint64_t>(dst.data())] = *reinterpret_cast<const uint8_t *>(b.src);

  for (int by_source = 0; by_source < 2; ++by_source)
    for (uint32_t tile : {1024u, 2048u, 8192u, kStreamTile}) {
      if (tile == kStreamTile && cp.pitched != 0) continue;
      const PieceRoom room = piece_room(cp, C, tile);
      if (room.pieces == 0) continue;
      if (cp.pitched == 0) CHECK(room.pieces == cp.xfers.size() + (cp.funcs.size() == 1 ? 0 : places));
      std::vector<uint32_t> words(piece_bytes(room) / 4);  // no more than that: the sanitizer sees a write beyond
      PieceTables t = piece_places(reinterpret_cast<char *>(words.data()), room);
      CHECK(build_pieces(cp, C, tile, by_source != 0, &t));
      CHECK(t.n > 0 && t.n <= room.pieces && t.nshapes <= room.shapes && t.tile == tile && t.first[0] == 0);
      std::vector<Byte> got;
      std::memset(dst.data(), 0xA5, dst.size());
      for (uint32_t i = 0; i < t.n; ++i) {
        Xfer x{};
        const PieceRows *r = t.shape != nullptr && t.shape[i] != 0 ? &t.shapes[t.shape[i] - 1] : nullptr;
        x.src = t.at[i].src;
        x.dst = t.at[i].dst;
        x.row_bytes = r ? r->row_bytes : t.len[i];
        x.src_pitch = r ? r->src_pitch : t.len[i];
        x.dst_pitch = r ? r->dst_pitch : t.len[i];
        if (r) bytes_of(got, x, t.edges[i].from, (t.len[i] - 1) * x.row_bytes + t.edges[i].to - t.edges[i].from);
        else bytes_of(got, x, 0, x.row_bytes);
        move_piece(t, i, by_source != 0);
      }
      CHECK(got == order);
      CHECK(dst == want);
      n_merged += t.n < cp.xfers.size();
    }
}

// A run beyond 2^30 bytes becomes several pieces, and no table entry is exceeded.
static void long_run() {
  ClassPlan cp;
  Func fn{};
  fn.weight = 1;
  fn.ndesc = 2;
  for (uint64_t n : {(5ull << 30) + 77, 3ull << 30}) {
    Xfer x{};
    x.src = 0x100000000000ull + fn.stream_bytes;
    x.dst = 0x200000000005ull + fn.stream_bytes;
    x.row_bytes = n;
    x.rows = 1;
    x.stream_off = fn.stream_bytes;
    fn.stream_bytes += n;
    cp.xfers.push_back(x);
  }
  fn.nchunks = (fn.stream_bytes + (2 << 20) - 1) / (2 << 20);
  cp.payload = fn.stream_bytes;
  cp.funcs.push_back(fn);
  CHECK(build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);
  const PieceRoom room = piece_room(cp, 2 << 20, 4096);
  CHECK(room.pieces >= 9 && room.shapes == 0);
  std::vector<uint32_t> words(piece_bytes(room) / 4);
  PieceTables t = piece_places(reinterpret_cast<char *>(words.data()), room);
  CHECK(build_pieces(cp, 2 << 20, 4096, false, &t));
  uint64_t at = 0;
  for (uint32_t i = 0; i < t.n; ++i) {
    CHECK(t.at[i].src == cp.xfers[0].src + at && t.at[i].dst == cp.xfers[0].dst + at && t.len[i] <= 1u << 30);
    at += t.len[i];
  }
  CHECK(at == cp.payload && t.n == 9);
}

// Tables on their way to the device, up to what 2^32 descriptors take: the parts follow each other and their tiles cover every byte once.
static void table_uploads() {
  CHECK(!tables_by_kernel(256) && !tables_by_kernel(16 * 1024 - 1) && tables_by_kernel(16 * 1024) && tables_by_kernel(1ull << 33));
  const uint64_t g = kLongestRun;
  for (uint64_t bytes : {(uint64_t)256, (uint64_t)16384, (uint64_t)393216, g - 256, g, g + 256, 4 * g - 256, 4 * g, 4 * g + 768, 256 * g + 512})
    for (uint64_t host : {(uint64_t)1 << 44, ((uint64_t)1 << 44) + 16, ((uint64_t)1 << 44) + 0xfffff000u}) {
      const uint64_t dev = (uint64_t)1 << 45;
      uint64_t at = 0, parts = 0;
      for (; at < bytes; ++parts) {
        const OneRun part(host + at, dev + at, bytes - at, piece_tile(FT_H2P, bytes), true);
        const PieceTables &t = part.tables;
        CHECK(t.n == 1 && pieces_go_along(t) && t.shape == nullptr && t.first[0] == 0 && t.at[0].src == host + at && t.at[0].dst == dev + at);
        CHECK(t.src0 == t.at[0].src && t.dst0 == t.at[0].dst && t.len[0] > 0 && t.len[0] <= kLongestRun && t.tile <= 4096);
        CHECK((uint64_t)piece_workgroups(FT_H2P, t.ntiles) * t.tile <= 256 * 1024);  // no more asked of host memory at once than fills the link
        uint64_t moved = 0;
        const uint32_t step = parts == 0 || t.ntiles < 1000 ? 1 : t.ntiles / 1000;
        for (uint32_t no = 0; no < t.ntiles; no += no + step < t.ntiles || no + 1 == t.ntiles ? step : t.ntiles - 1 - no) {
          uint32_t begin, n;
          run_tile(t.at[0].src, t.len[0], t.tile, no, &begin, &n);
          CHECK(n > 0 && n <= t.tile && (uint64_t)begin + n <= t.len[0] && (step > 1 || begin == moved));
          moved = (uint64_t)begin + n;
        }
        CHECK(moved == t.len[0]);
        at += t.len[0];
      }
      CHECK(at == bytes && parts == (bytes + kLongestRun - 1) / kLongestRun);
    }
}

// What no list of pieces is made for.
static void refused() {
  auto with = [](uint64_t rb, uint64_t rows, uint64_t pitch, uint64_t chunk, uint64_t more_chunks) {
    ClassPlan cp;
    Xfer x{};
    x.row_bytes = rb;
    x.rows = rows;
    x.src_pitch = x.dst_pitch = pitch;
    for (uint32_t f = 0; f < 2; ++f) {
      Func fn{};
      fn.weight = fn.ndesc = 1;
      fn.desc_off = f;
      fn.stream_bytes = rb * rows;
      fn.nchunks = (fn.stream_bytes + chunk - 1) / chunk;
      cp.xfers.push_back(x);
      cp.funcs.push_back(fn);
      cp.pitched += rows > 1;
    }
    CHECK(build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);
    PieceRoom room = piece_room(cp, chunk, 2048);
    if (more_chunks != 0) {
      cp.nchunks = more_chunks;
      return piece_room(cp, chunk, 2048).pieces != 0;
    }
    if (room.pieces == 0) return false;
    std::vector<uint32_t> words(piece_bytes(room) / 4);
    PieceTables t = piece_places(reinterpret_cast<char *>(words.data()), room);
    return build_pieces(cp, chunk, 2048, false, &t);
  };
  for (uint64_t chunk : {1024, 1 << 20}) {
    CHECK(with(16, 3, 20, chunk, 0) && !with(15, 3, 20, chunk, 0));
    CHECK(with(16, 3, ((1ull << 32) - 1) / 516, chunk, 0) && !with(16, 3, ((1ull << 32) - 1) / 516 + 1, chunk, 0));
  }
  CHECK(with(1000, 4000, 1000000, 1 << 20, 0) && !with(1000, 5000000, 1001, 1 << 22, 0) && !with(1ull << 33, 2, 1ull << 33, 1ull << 30, 0));
  CHECK(!with(16, 3, 20, 512, 0));
  CHECK(with(100, 1, 100, 1024, kMaxPieces - 2) && !with(100, 1, 100, 1024, kMaxPieces - 1));
}

// What a list would cost the host is known before it is written: `n` tensors of equal size, `total` MiB of `nf` functions in chunks of `chunk`
// KiB.
static void priced() {
  auto takes = [](int cls, uint32_t n, uint64_t total, uint32_t nf, uint64_t chunk, uint64_t shift, bool tables_fit, uint64_t dst_shift = 0) {
    ClassPlan cp;
    const uint64_t size = (total << 20) / n / 16 * 16;
    for (uint32_t f = 0; f < nf; ++f) {
      Func fn{};
      fn.func = f;
      fn.weight = 1;
      fn.desc_off = (uint32_t)cp.xfers.size();
      for (uint32_t i = f; i < n; i += nf) {
        Xfer x{};
        x.src = 0x100000000000ull + i * (size + 4096) + shift;
        x.dst = 0x200000000000ull + i * (size + 4096) + dst_shift;
        x.row_bytes = x.src_pitch = x.dst_pitch = size;
        x.rows = 1;
        x.stream_off = fn.stream_bytes;
        fn.stream_bytes += size;
        fn.ndesc += 1;
        cp.xfers.push_back(x);
      }
      fn.nchunks = (fn.stream_bytes + (chunk << 10) - 1) / (chunk << 10);
      cp.payload += fn.stream_bytes;
      cp.funcs.push_back(fn);
    }
    CHECK(build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);
    return job_pieces(cp, cls, chunk << 10, tables_fit).pieces != 0;
  };
  // few large tensors whose general tables travel along
  CHECK(takes(FT_P2P, 8, 64, 8, 2048, false, true) && takes(FT_P2P, 8, 64, 1, 8, false, true));
  CHECK(!takes(FT_P2P, 8, 64, 8, 64, false, true) && !takes(FT_P2P, 8, 64, 8, 8, false, true) && !takes(FT_P2P, 8, 16, 8, 8, false, true));
  CHECK(!takes(FT_P2P, 40, 60, 8, 8, true, true) && takes(FT_P2P, 40, 40, 4, 512, true, true));
  // uploaded: beside the copy kernel any number, beside the wave kernel what a launch could hold
  CHECK(takes(FT_P2P, 64, 64, 8, 8, false, false) && !takes(FT_P2P, 64, 64, 8, 8, true, false) && !takes(FT_P2P, 64, 32, 8, 64, false, false));
  CHECK(takes(FT_P2P, 1024, 16, 4, 256, false, false) && !takes(FT_P2P, 300, 16, 4, 16, false, false) &&
        takes(FT_P2P, 2048, 16, 4, 16, false, false));
  // beyond the cache: sides 4, 8 or 12 bytes apart; any others of short tensors, and to misaligned destinations in jobs that are not too large
  for (uint64_t shift = 0; shift <= 32; ++shift)
    for (uint64_t dst : {0, 1, 4, 8, 15, 16, 33})
      for (uint32_t n : {1u, 8u, 100u, 200u, 300u, 500u}) {
        const uint64_t total = n == 8 ? 300 : n == 300 ? 500 : n == 500 ? 260 : 140, apart = (shift ^ dst) & 15;
        const bool want = apart % 4 == 0 ? apart != 0 : n == 200 || n == 500 || (dst % 16 != 0 && n != 8);
        CHECK(takes(FT_P2P, n, total, n < 4 ? n : 4, 2048, shift, false, dst) == want);
      }
  CHECK(takes(FT_P2P, 1, 768, 1, 2048, 4, true) && !takes(FT_P2P, 1, 769, 1, 2048, 4, true) && takes(FT_P2P, 2, 1000, 1, 2048, 4, true));
  for (int cls : {(int)FT_H2P, (int)FT_P2H})
    CHECK(takes(cls, 64, 4, 4, 16, false, false) && !takes(cls, 64, 4, 4, 4, false, false) && takes(cls, 300, 60, 4, 64, false, false) &&
          !takes(cls, 300, 60, 4, 16, false, false) && !takes(cls, 8, 60, 4, 64, false, true) && takes(cls, 8, 16, 4, 256, false, true) &&
          takes(cls, 1000, 4, 4, 4, false, false) && !takes(cls, 1000, 16, 4, 4, false, false));
}

// Every tile is some workgroup's, no more than seven places from its own; and of tiles that repeat after 2, 4 or 8 every die (b % 8) has as
// many of one kind as of another in 64 workgroups.
static void tiles_over_dies() {
  for (uint32_t ntiles = 1; ntiles < 700; ++ntiles) {
    std::vector<uint32_t> seen(ntiles, 0), kinds(64, 0);
    for (uint32_t b = 0; b < ntiles; ++b) {
      const uint32_t t = tile_of_workgroup(b, ntiles);
      CHECK(t < ntiles && t / 8 == b / 8);
      seen[t] += 1;
      kinds[b % 8 * 8 + t % 8] += 1;
      if ((b + 1) % 64 == 0)
        for (uint32_t k : kinds) CHECK(k == (b + 1) / 64);
    }
    for (uint32_t s : seen) CHECK(s == 1);
  }
}

// Which launches keep compute units free for others: lists that go along with more tiles than 48 MiB has, no rows, nothing over the link.
static void units_kept_free() {
  PieceRows rows{};
  uint32_t shape = 1;
  for (int cls = 0; cls < 3; ++cls)
    for (uint32_t n : {1u, kRunsAlong, kRunsAlong + 1})
      for (uint32_t ntiles : {1u, 6144u, 6145u, 16384u}) {
        PieceTables t;
        t.n = n;
        t.ntiles = ntiles;
        t.tile = 8192;
        CHECK(piece_lds(cls, t) == 0);  // sides too far apart for a launch
        t.close = true;
        const uint32_t lds = piece_lds(cls, t);
        CHECK((lds != 0) == (cls == 2 && n <= kRunsAlong && ntiles > 6144) && (lds == 0 || (160u << 10) / lds == 8));
        t.shape = &shape;
        t.shapes = &rows;
        CHECK(piece_lds(cls, t) == 0);
      }
  PieceTables t;  // jobs of up to 20 MiB have small tiles, and not too many of them
  for (uint64_t payload : {10u << 20, 20u << 20, 48u << 20}) {
    t.n = kRunsAlong;
    t.close = true;
    t.ntiles = (uint32_t)(payload / piece_tile(FT_P2P, payload)) + (payload < 48u << 20 ? t.n : 0);
    CHECK(piece_lds(FT_P2P, t) == 0);
  }
  for (uint32_t n : {1u, kRunsAlong, kRunsAlong + 1, kMaxPieces})  // beyond 128 MiB six tiles on a unit, 24 MiB on 256, wherever the list lies
    for (bool close : {false, true}) {
      t.n = n;
      t.close = close;
      t.tile = piece_tile(FT_P2P, kCacheResidentBytes + 1);
      t.ntiles = kCacheResidentBytes / t.tile + 1;
      CHECK(t.tile == kStreamTile && (160u << 10) / piece_lds(FT_P2P, t) == 6);
    }
}

// The shares of functions whose tensors are misaligned, beyond 128 MiB: when workgroup b begins, each function has begun as many bytes as the order of the
// chunks gives it among the first b tiles, but for seven of them; and that is its weight's share to two chunks.
static void streaming_shares() {
  const uint64_t C = 1 << 20;
  const uint32_t weights[] = {1, 2, 5}, each = 4;
  ClassPlan cp;
  for (uint32_t f = 0; f < 3; ++f) {
    Func fn{};
    fn.func = f;
    fn.weight = weights[f];
    fn.desc_off = (uint32_t)cp.xfers.size();
    for (uint32_t i = 0; i < each; ++i) {
      Xfer x{};
      const uint64_t n = cp.xfers.size();
      x.row_bytes = x.src_pitch = x.dst_pitch = (weights[f] * 6ull << 20) + 1000 * f + 7 * i;
      x.src = 0x100000000000ull + n * (64 << 20) + 4 * n + 1;
      x.dst = 0x200000000000ull + n * (64 << 20) + 9;
      x.rows = 1;
      x.stream_off = fn.stream_bytes;
      fn.stream_bytes += x.row_bytes;
      fn.ndesc += 1;
      cp.xfers.push_back(x);
    }
    fn.nchunks = (fn.stream_bytes + C - 1) / C;
    cp.payload += fn.stream_bytes;
    cp.funcs.push_back(fn);
  }
  CHECK(cp.payload > kCacheResidentBytes && build_phases(cp.funcs, cp.phases, cp.slots, &cp.nchunks) == FT_OK);
  const PieceRoom room = job_pieces(cp, FT_P2P, C, false);
  CHECK(room.pieces != 0);
  std::vector<uint64_t> words(piece_bytes(room) / 8 + 1);
  PieceTables t = piece_places(reinterpret_cast<char *>(words.data()), room);
  CHECK(build_pieces(cp, C, piece_tile(FT_P2P, cp.payload), false, &t) && t.tile == kStreamTile);
  const auto begun = [&](bool turned) {  // bytes of each function begun before each workgroup
    std::vector<uint64_t> sums(3 * (t.ntiles + 1), 0);
    for (uint32_t b = 0; b < t.ntiles; ++b) {
      const uint32_t no = turned ? tile_of_workgroup(b, t.ntiles) : b;
      const uint32_t i = (uint32_t)(std::upper_bound(t.first, t.first + t.n, no) - t.first - 1);
      uint32_t begin, n;
      run_tile(t.at[i].dst, t.len[i], t.tile, no - t.first[i], &begin, &n);
      for (uint32_t f = 0; f < 3; ++f)
        sums[3 * b + 3 + f] = sums[3 * b + f] + ((t.at[i].dst - 0x200000000000ull) / (64 << 20) / each == f ? n : 0);
    }
    return sums;
  };
  const std::vector<uint64_t> kernel = begun(true), order = begun(false);
  for (uint32_t b = 0; b <= t.ntiles; ++b) {
    const uint64_t total = order[3 * b] + order[3 * b + 1] + order[3 * b + 2];
    for (uint32_t f = 0; f < 3; ++f) {
      const auto apart = [](uint64_t x, uint64_t y) { return x > y ? x - y : y - x; };
      CHECK(apart(kernel[3 * b + f], order[3 * b + f]) <= 7 * kStreamTile);
      if (total < cp.payload - (8 << 20)) CHECK(apart(8 * order[3 * b + f], weights[f] * total) <= 8 * 2 * C);  // (the streams end together)
    }
  }
  for (uint32_t f = 0; f < 3; ++f) CHECK(kernel[3 * t.ntiles + f] == cp.funcs[f].stream_bytes);
}

int main(int argc, char **argv) {
  const uint64_t first = argc > 1 ? strtoull(argv[1], 0, 10) : 1, count = argc > 2 ? strtoull(argv[2], 0, 10) : 50;
  refused();
  long_run();
  table_uploads();
  priced();
  tiles_over_dies();
  units_kept_free();
  streaming_shares();
  for (g_seed = first; g_seed < first + count; ++g_seed) {
    std::mt19937_64 r(g_seed);
    for (int i = 0; i < 6; ++i) job(r);
  }
  CHECK(n_rows > 0 && n_parts > 0 && n_merged > 0 && n_edges > 0);
  std::printf("tiles %llu, of rows %llu, of parts of rows %llu, lists with merged tensors %llu\n", (unsigned long long)n_tiles,
              (unsigned long long)n_rows, (unsigned long long)n_parts, (unsigned long long)n_merged);
  std::printf("done %llu..%llu\n", (unsigned long long)first, (unsigned long long)(first + count - 1));
  return 0;
}
