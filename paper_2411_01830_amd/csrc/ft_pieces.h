// A class of a job as the list of its pieces: what the proportional chunk order of Sec. 6.1 comes to when it is written
// out, for jobs in which that is short. A piece is a run of bytes that lie together on both sides, or whole rows of one
// pitched descriptor; pieces follow each other in the order of the chunks that they come from, and every piece is cut into
// tiles of its own. Tile t of the launch is found by the first tiles of the pieces, or of blocks of them, in the launch's arguments and then its bytes by
// one read, where the general tables (ft_tables.h) take five dependent reads and several divisions.
#pragma once
#include <stdint.h>

#include "ft_plan.h"
#include "ft_tables.h"
#include "ft_windows.h"

namespace ft {

struct PieceSides {
  uint64_t src, dst;
};

// What pieces of rows have beyond their sides (those of column 0 of their first row). Most jobs have few shapes.
struct PieceRows {
  uint32_t row_bytes, src_pitch, dst_pitch;
  uint32_t per;    // rows of a tile; or kPartsOfRow | tiles of a row
  uint32_t magic;  // g / windows of a row = mulhi(g, magic) or one less; 0: a row is one window (ft_windows.h)
  uint32_t part;   // bytes of a tile that is part of a row
};
constexpr uint32_t kPartsOfRow = 1u << 31;  // a piece of such rows has whole ones only
struct PieceEdges {
  uint32_t from, to;
};

// The tables as arrays of `n` entries each, in host memory.
struct PieceTables {
  PieceSides *at = nullptr;
  uint32_t *first = nullptr;    // the piece's first tile; ascending, no piece is without one
  uint32_t *len = nullptr;      // bytes of a run, rows of a piece of rows
  uint32_t *shape = nullptr;    // 0: a run; else 1 + index into the shapes. Null: all are runs
  PieceRows *shapes = nullptr;  // null if shape is, as is
  PieceEdges *edges = nullptr;  // of rows (of a run nothing): the first row from column `from`, the last one up to `to`
  uint32_t n = 0, nshapes = 0, ntiles = 0;
  uint32_t tile = 0;              // bytes of a tile, a power of two
  const char *packed = nullptr;   // where the device finds a list of runs (pack_pieces), if it does not go along
  uint64_t src0 = 0, dst0 = 0;    // addresses not above any side's,
  bool close = false;             // from which every side is less than 2^32 bytes away (said of few pieces only, of more by find_base)
};

// A run's tiles begin and end where this many bytes of the side that is dearer to cut (the destination; host memory where
// that is the source) do, so that no line is written by two wavefronts: shared lines cost a misaligned job 4-12 %.
constexpr uint32_t kPieceLine = 128;
// Tiles of a pool->pool job of runs that no cache holds.
constexpr uint32_t kStreamTile = 16384;
// Pieces of one job at most, and at most as many as travel with a launch, with as many shapes: kernel arguments end at 4 KiB, and
// hold sides as 32-bit distances from the lowest.
constexpr uint32_t kMaxPieces = 16384, kRunsAlong = 240, kRowsAlong = 140;
inline bool pieces_go_along(const PieceTables &t) {
  return t.close && (t.shape == nullptr ? t.n <= kRunsAlong : (t.n <= 64 && t.nshapes <= 64) || (t.n <= kRowsAlong && t.nshapes <= 16));
}

// An upper bound for the pieces of a class and their shapes, 0 if it is no job for them.
struct PieceRoom {
  uint64_t pieces = 0, shapes = 0;
};
PieceRoom piece_room(const ClassPlan &cp, uint64_t chunk_bytes, uint32_t tile);
// Bytes of the tables, and their places from `base` (a multiple of 8) on.
uint64_t piece_bytes(const PieceRoom &room);
PieceTables piece_places(char *base, const PieceRoom &room);
// Lists of runs that do not go along lie in memory as arrays one behind the other: where no side is 2 GiB or more away from the first
// piece's, sources and destinations as 32-bit distances from t's src0 and dst0, lengths, 12 bytes a piece; else PieceSides and lengths. What else
// the kernels need is in their arguments (the first tile of every kPieceBlock-th piece) or follows from the lengths.
constexpr uint32_t kPieceBlock = 64;  // a lane each
inline uint64_t packed_bytes(const PieceTables &t) { return (uint64_t)t.n * (t.close ? 12 : 20); }
// Says whether t's pieces are close, and from where.
void find_base(PieceTables *t);
// Writes t, whose base is known, to `to`.
void pack_pieces(const PieceTables &t, char *to);
// Fills t with the pieces of a class in its order, cut into tiles of `tile` bytes, a power of two from 1 to 8 KiB (of runs alone, pool->pool, 16).
// by_source: the source's lines are the ones not to be cut. False: there are rows that the kernels do not cover (under 16
// bytes, or so far apart that a tile's distances leave 32 bits).
bool build_pieces(const ClassPlan &cp, uint64_t chunk_bytes, uint32_t tile, bool by_source, PieceTables *t);

// Tiles of a run of len bytes, one of whose sides (the one not to be cut) begins at `side`.
FT_HD uint32_t run_tiles(uint64_t side, uint32_t len, uint32_t tile) { return (len + ((uint32_t)side & (kPieceLine - 1)) + tile - 1) / tile; }

// A run longer than this is several pieces: tiles are found by 32-bit arithmetic.
constexpr uint64_t kLongestRun = 1ull << 30;

// One run on its own, without a list: the tables are its members. The first kLongestRun bytes of it at most; a longer one is launched
// in several parts.
struct OneRun {
  PieceSides at;
  uint32_t first, len;
  PieceTables tables;
  OneRun(uint64_t src, uint64_t dst, uint64_t bytes, uint32_t tile, bool by_source) {
    at = PieceSides{src, dst};
    first = 0;
    len = (uint32_t)(bytes < kLongestRun ? bytes : kLongestRun);
    tables.at = &at;
    tables.first = &first;
    tables.len = &len;
    tables.n = 1;
    tables.tile = tile;
    tables.ntiles = run_tiles(by_source ? src : dst, len, tile);
    tables.src0 = src;
    tables.dst0 = dst;
    tables.close = true;
  }
  OneRun(const OneRun &) = delete;
  OneRun &operator=(const OneRun &) = delete;
};

// The room for a class of a job that is to be launched as pieces, none if it is not; and the tile. tables_fit: the general tables
// would travel with the launch. alone: the kernel is to say itself when it is done, and no other job's follows at once.
PieceRoom job_pieces(const ClassPlan &cp, int cls, uint64_t chunk_bytes, bool tables_fit, bool alone = false);
uint32_t piece_tile(int cls, uint64_t payload);
// Workgroups, of one wavefront each, of a launch of that many tiles; and whether they draw tiles beyond their first from a counter: those
// of one piece, which has no order to keep, are dealt out, unless their number would leave some wavefronts a round more than others.
uint32_t piece_workgroups(int cls, uint32_t ntiles);
inline bool piece_draws(int cls, const PieceTables &t) {
  const uint32_t workgroups = piece_workgroups(cls, t.ntiles);
  return workgroups < t.ntiles && (t.n > 1 || (workgroups & (workgroups - 1)) != 0);
}

// Whether a list that does not go along is read where the host wrote it, in pinned memory, and not uploaded first: no launch in front of the
// job's and no gap between the two, but every die has the list over the link for itself, 8 x 12 bytes a piece. Passes, us, uploaded -> in
// place, 4 functions: 260 pieces 33.1 -> 29.2, 520 38.0 -> 34.2, 1000 47.3 -> 44.9, 2000 67.8 -> 66.6, 4000 109.5 -> 110.4, 8000 196 -> 205. The
// kernel alone 4.2 -> 4.2, 5.7 (1000), 7.2 (2000), 10.8 (4000). Not over the host link, whose few wavefronts look for a piece for each
// of their tiles, behind the link's own reads (536 tensors of 10 KB from the host 138 -> 154).
inline bool pieces_read_in_place(int cls, uint64_t bytes) { return cls == FT_P2P && bytes <= 32u << 10; }

// Words in pinned memory, one for each wavefront of a launch, that say when its bytes are where they belong; none if null. An event bound to the
// dispatch fires some 2 us after the last store: the end of the kernel is gathered, the L2 of every die written back, a signal sent. A
// wavefront that has waited for its own stores can tell the host at once. Each word has a cache line for itself: sixteen of 4 bytes to a
// line, written one after the other while the host reads them, are dearer than the event (64 KiB pool->pool, 32 wavefronts, a pass, us: by the
// event 10.7, with 4-byte words 10.0, eight words a line 9.75, a line each 9.1; 1 MiB, 512 wavefronts: 10.8, 13.8, 10.7, 10.0).
struct DoneWords {
  uint64_t *words = nullptr;
  uint64_t value = 0;
};
constexpr uint32_t kDoneStride = 8;    // words from one that is used to the next
constexpr uint32_t kDoneWords = 640;   // of a launch: more of them cost what they save (1000 in 2 MiB 12.4, by the event 10.9)
// Over the host link wavefronts are few, so there the line lies where 1.4 us are 1 % of the job (32 tensors, 4 MiB, to the pool and back 166.0 -> 163.2).
// And only where few jobs are in flight on the stream at once (StreamJobs::burst): a written-through kernel ends 1 us later than it would, which a wait that ends
// 2 us earlier makes up for once and a burst pays for every job. Passes, us, n jobs of one tensor each submitted and then waited for, by events -> by words:
// pool->pool 512 KiB n = 2 15.6 -> 14.9, 3 20.2 -> 18.4, 5 29.2 -> 28.3, 6 33.9 -> 34.5, 8 42.7 -> 47, 32 166 -> 188; 1 MiB 4 24.9 -> 24.2, 5 29.5 -> 30.5; 64 KiB 4 24.7 -> 22.1,
// 32 170 -> 170; towards the host 16 KiB 4 25.5 -> 22.4, 256 KiB 4 34.8 -> 34.4, 8 61.3 -> 62.3, 1 MiB 2 49.2 -> 48.4, 4 89.9 -> 90.4; from the host 128 KiB 2 20.3 -> 20.0, 4 31.9 -> 33.2,
// 32 191 -> 219. Words for some of a burst alone are no better: of two of 512 KiB the first one's alone 16.5.
constexpr uint32_t most_words(int cls) { return cls == FT_H2P ? 2 : 4; }
inline bool says_done(int cls, uint64_t payload, uint32_t ntiles, uint32_t burst) {
  return piece_workgroups(cls, ntiles) <= kDoneWords && payload <= 8u << 20 && burst <= most_words(cls) && (cls == FT_P2P || burst == 1 || burst * payload <= 2u << 20);
}

// LDS that a workgroup asks for without using it, so that a compute unit of 160 KiB takes no more of them at once.
uint32_t piece_lds(int cls, const PieceTables &t);

// ---- what a tile covers: the arithmetic of the kernels, so that it can be checked without a GPU

// The tile of workgroup b where every tile has one. The eight dies take the workgroups in turn, b % 8 says which, and each begins its own in
// order as others of its end. A list whose tiles repeat after 2, 4 or 8 would give a die tiles of one kind only: dies with slow or long
// ones fall behind the others, and with them the function that they belong to. So the eight tiles of a group go to the dies one
// further round in every group; the last group, if it is not whole, is as it is. Two functions of equal weight, one of 8 KiB tensors at
// odd addresses and one of large tensors, chunks of 16 KiB, 60 MiB: in tile order one of them was ahead by up to 8 % of the payload,
// now 0.5 % (tickets from a counter: 2 %). One of 1 KiB tensors, chunks of 7 KiB, which is eight tiles a turn, 22 MiB: all large tiles on one
// die, 20.4 us, now 11.3.
FT_HD uint32_t tile_of_workgroup(uint32_t b, uint32_t ntiles) { return (b | 7) < ntiles ? (b & ~7u) | ((b + (b >> 3)) & 7) : b; }

// Bytes [begin, begin + n) of a run of len bytes, one of whose sides (the one not to be cut) begins at `side`.
FT_HD void run_tile(uint64_t side, uint32_t len, uint32_t tile, uint32_t no, uint32_t *begin, uint32_t *n) {
  const uint32_t before = (uint32_t)side & (kPieceLine - 1);
  const uint32_t b = no == 0 ? 0u : no * tile - before, e = (no + 1) * tile - before;
  *begin = b;
  *n = (e < len ? e : len) - b;
}

// Windows of a row, and the windows (ft_windows.h) of a tile of rows: those of rows [*r0, ...) of a piece of len rows.
FT_HD uint32_t windows_of_row(uint32_t row_bytes) { return row_bytes / 16 + (row_bytes % 16 != 0 ? 1u : 0u); }
FT_HD RowWindows rows_tile(const PieceRows &r, uint32_t len, const PieceEdges &e, uint32_t no, uint32_t *r0) {
  const uint32_t begin = no * r.per, n = len - begin < r.per ? len - begin : r.per;
  *r0 = begin;
  RowWindows w;
  w.c0 = begin == 0 ? e.from : 0u;
  w.more = n - 1;
  w.row_bytes = r.row_bytes;
  w.last_end = begin + n == len ? e.to : r.row_bytes;
  w.per_row = windows_of_row(r.row_bytes);
  w.magic = r.magic;
  const uint32_t first_len = (n == 1 ? w.last_end : r.row_bytes) - w.c0;
  w.short_first = first_len < 16 ? first_len : 0u;
  w.short_last = n != 1 && w.last_end < 16 ? w.last_end : 0u;
  w.first = w.short_first != 0 ? w.per_row : w.c0 / 16;
  const uint32_t last = w.last_end < 16 ? w.more * w.per_row : w.more * w.per_row + (w.last_end + 15) / 16;  // one past it
  w.count = last > w.first ? last - w.first : 0u;
  return w;
}

// A tile that is part of a row: n bytes from column *begin of row *row on.
FT_HD void row_part(const PieceRows &r, uint32_t no, uint32_t *row, uint32_t *begin, uint32_t *n) {
  const uint32_t parts = r.per & ~kPartsOfRow;
  *row = no / parts;
  *begin = (no - *row * parts) * r.part;
  *n = r.row_bytes - *begin < r.part ? r.row_bytes - *begin : r.part;
}

}  // namespace ft
