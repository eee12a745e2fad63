// Kernels for a class that is written out as pieces (ft_pieces.h): pool->pool a workgroup of one wavefront per tile, dispatched in
// the order of the pieces; over the host link few wavefronts, which draw their tiles (ft_link_piece_kernel).
//
// What bounds them is what bounds a launch of some MiB: the fetch of its arguments and instructions, the reads that lead
// from a tile's number to its bytes, one round trip for the bytes, and HBM or the last-level cache. So the tables are
// small (16 bytes a run in the launch itself, up to kRunsAlong runs; 12 in memory), a tile is found by one compare of 64
// entries and one record, and the code is a few hundred instructions. Pool->pool needs no counter and no persistent
// workgroups: the hardware starts the workgroups in order as others end.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstring>

#include "ft_kernels.h"
#include "ft_moves.h"
#include "ft_pieces.h"

namespace ft {

// Tables that travel with the launch: the first kernel argument. A launch call costs the host 4.1 us with some bytes of arguments and
// 5.8 us with 3 KiB, so there are several sizes.
template <uint32_t CAP, uint32_t SHAPES>
struct PieceArgs {
  static constexpr bool kRows = SHAPES != 0, kOne = CAP == 1, kSays = true;
  uint32_t n, tile, ntiles;
  uint64_t src0, dst0;
  struct {
    uint32_t src, dst;  // bytes from src0 and dst0
  } at[CAP];
  uint32_t first[CAP], len[CAP];
  uint32_t shape[kRows ? (CAP + 3) / 4 : 1];  // a byte each
  PieceEdges edges[kRows ? CAP : 1];
  PieceRows shapes[kRows ? SHAPES : 1];
};
// and lists of runs in memory (pack_pieces), with the first tile of every block of pieces: a wavefront has its tile's block from the
// arguments, and the block's entries, one a lane, are one read deep. (A search through all first tiles and then a record were three, each a trip
// over the link where the list is read in place: 1024 tensors, 15.6 MB, in place 9.5 us with 24 bytes a piece searched, 7.7 so; uploaded 6.2 either way.)
template <uint32_t BLOCKS, bool CLOSE>
struct PieceRefs {
  static constexpr bool kRows = false, kOne = false;
  static constexpr bool kSays = (BLOCKS / 4) * kPieceBlock < kDoneWords;  // launch_refs takes it for more pieces than a quarter, each at least a tile
  uint32_t n, tile, ntiles;
  uint64_t src0, dst0;
  const char *packed;
  uint32_t block[BLOCKS];
};

struct Piece {
  uint64_t src, dst;
  uint32_t len, tile_no;  // tile within the piece
  uint32_t tile;          // bytes of a tile
  PieceRows rows;         // row_bytes 0: a run
  PieceEdges edges;
};

__device__ __forceinline__ PieceRows read_shape(const FT_CONST PieceRows *shapes, uint32_t shape) {
  PieceRows r;
  r.row_bytes = 0;
  if (shape != 0) {
    const FT_CONST PieceRows &s = shapes[shape - 1];
    r.row_bytes = s.row_bytes;
    r.src_pitch = s.src_pitch;
    r.dst_pitch = s.dst_pitch;
    r.per = s.per;
    r.magic = s.magic;
    r.part = s.part;
  }
  return r;
}

template <int NT, uint32_t CAP, uint32_t SHAPES>
__device__ __forceinline__ Piece find_piece(const PieceArgs<CAP, SHAPES> &, uint32_t t, uint32_t lane) {
  const FT_CONST PieceArgs<CAP, SHAPES> &a =
      *reinterpret_cast<const FT_CONST PieceArgs<CAP, SHAPES> *>(reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()));
  uint32_t x = 0;
  if (CAP > 1) {
    uint32_t before = 0;  // every compare's load is on its way before the first is counted
#pragma unroll
    for (uint32_t j0 = 0; j0 < CAP; j0 += 64) {
      const uint32_t j = j0 + lane;
      before += wave_count(a.first[j < CAP ? j : 0u] <= t && j < a.n);
    }
    x = uniform32(before - 1);
  }
  Piece p;
  p.src = a.src0 + a.at[x].src;
  p.dst = a.dst0 + a.at[x].dst;
  p.len = a.len[x];
  p.tile_no = t - a.first[x];
  p.tile = a.tile;
  if (SHAPES != 0) {
    p.rows = read_shape(a.shapes, a.shape[x / 4] >> x % 4 * 8 & 255);
    p.edges.from = a.edges[x].from;
    p.edges.to = a.edges[x].to;
  }
  return p;
}

template <class T>
__device__ __forceinline__ const FT_CONST T *constant(const char *p) { return reinterpret_cast<const FT_CONST T *>(reinterpret_cast<uintptr_t>(p)); }

template <int NT, uint32_t BLOCKS, bool CLOSE>
__device__ __forceinline__ Piece find_piece(const PieceRefs<BLOCKS, CLOSE> &, uint32_t t, uint32_t lane) {
  typedef PieceRefs<BLOCKS, CLOSE> Refs;
  const FT_CONST Refs &r = *reinterpret_cast<const FT_CONST Refs *>(reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()));
  uint32_t before = 0;
#pragma unroll
  for (uint32_t j0 = 0; j0 < BLOCKS; j0 += 64) {
    const uint32_t j = j0 + lane;
    before += wave_count(r.block[j < BLOCKS ? j : 0u] <= t && j * kPieceBlock < r.n);
  }
  const uint32_t b = uniform32(before - 1), begin = b * kPieceBlock;
  const bool is = begin + lane < r.n;
  const uint32_t j = is ? begin + lane : begin;
  uint64_t src, dst;
  uint32_t len;
  if (CLOSE) {
    src = r.src0 + constant<uint32_t>(r.packed)[j];
    dst = r.dst0 + constant<uint32_t>(r.packed)[r.n + j];
    len = constant<uint32_t>(r.packed)[2 * r.n + j];
  } else {
    src = constant<PieceSides>(r.packed)[j].src;
    dst = constant<PieceSides>(r.packed)[j].dst;
    len = constant<uint32_t>(r.packed + r.n * sizeof(PieceSides))[j];
  }
  // the tiles of the block's pieces up to each, which say where each begins
  const uint32_t tiles = run_tiles(NT == kFromHost ? src : dst, len, r.tile);
  const uint32_t first = r.block[b] + wave_sums(is ? tiles : 0u) - tiles;
  const uint32_t x = uniform32(wave_count(is && first <= t) - 1);
  Piece p;
  p.src = of_lane64(src, x);
  p.dst = of_lane64(dst, x);
  p.len = of_lane32(len, x);
  p.tile_no = t - of_lane32(first, x);
  p.tile = r.tile;
  return p;
}

// n bytes of a run, at most 512 windows, streaming 1024.
template <int NT>
__device__ __forceinline__ void move_run(uint64_t d, uint64_t s, uint32_t n, uint32_t lane) {
  if (n < 16) {
    if (lane < n) st_off<uint8_t, NT == kThrough ? kThrough : 0>(d, lane, ld_off<uint8_t, 0>(s, lane));
    return;
  }
  const RunWindows w = run_windows(NT == kFromHost ? s : d, n);  // whole granules on the side that is dearer
  // no deeper than need be: a lane's load beyond the last window costs as much as any other
  if (w.count <= 128) wave_run_pass<NT, 2>(d, s, w, 0, lane);
  else if (w.count <= 256) wave_run_pass<NT, 4>(d, s, w, 0, lane);
  else if (NT != kStream || w.count <= 512) wave_run_pass<NT, 8>(d, s, w, 0, lane);
  else wave_run_pass<NT, 16>(d, s, w, 0, lane);
}

// Up to R * 64 windows of rows. All loads before the first store; a lane past the last window loads the first one and stores nothing.
template <int NT, uint32_t R>
__device__ __forceinline__ void move_windows(uint64_t d, uint64_t s, const PieceRows &r, const RowWindows &w, uint32_t lane) {
  u32x4_any v[R];
  uint32_t to[R];
#pragma unroll
  for (uint32_t i = 0; i < R; ++i) {
    const uint32_t g = lane + i * 64;
    const RowCursor c = row_window<16>(w, g < w.count ? g : 0u);
    const uint32_t col = row_window_col<16>(w, c);
    v[i] = ld_off<u32x4_any, NT>(s, c.row * r.src_pitch + col);
    to[i] = c.row * r.dst_pitch + col;
  }
#pragma unroll
  for (uint32_t i = 0; i < R; ++i)
    if (lane + i * 64 < w.count) st_off<u32x4_any, NT>(d, to[i], v[i]);
}

// The windows of a tile of rows, and the bytes of a part of its first or last row that is shorter than a window: these are loaded before
// and stored after them.
template <int NT>
__device__ __forceinline__ void move_rows(uint64_t d, uint64_t s, const PieceRows &r, const RowWindows &w, uint32_t lane) {
  // lanes 0 .. 15: the first part's bytes, lanes 16 .. 31: the last part's
  const bool edge = lane < 16 ? lane < w.short_first : lane - 16 < w.short_last;
  const uint32_t es = lane < 16 ? w.c0 + lane : w.more * r.src_pitch + (lane - 16), ed = lane < 16 ? w.c0 + lane : w.more * r.dst_pitch + (lane - 16);
  uint8_t eb = 0;
  if (edge) eb = ld_off<uint8_t, 0>(s, es);
  if (w.count <= 256) {
    if (w.count != 0) move_windows<NT, 4>(d, s, r, w, lane);
  } else {
    move_windows<NT, 8>(d, s, r, w, lane);
  }
  if (edge) st_off<uint8_t, NT == kThrough ? kThrough : 0>(d, ed, eb);
}

template <int NT, bool ROWS>
__device__ __forceinline__ void move_tile(const Piece &p, uint32_t lane) {
  uint64_t d = p.dst, s = p.src;
  uint32_t begin, n;
  if (ROWS && p.rows.row_bytes != 0) {
    const PieceRows &r = p.rows;
    uint32_t row;
    if (!(r.per & kPartsOfRow)) {
      const RowWindows w = rows_tile(r, p.len, p.edges, p.tile_no, &row);
      move_rows<NT>(d + (uint64_t)row * r.dst_pitch, s + (uint64_t)row * r.src_pitch, r, w, lane);
      return;
    }
    row_part(r, p.tile_no, &row, &begin, &n);
    row = uniform32(row);
    begin = uniform32(begin);
    d += (uint64_t)row * r.dst_pitch;
    s += (uint64_t)row * r.src_pitch;
  } else {
    run_tile(NT == kFromHost ? p.src : p.dst, p.len, p.tile, p.tile_no, &begin, &n);
  }
  move_run<NT>(d + begin, s + begin, n, lane);
}

// A wavefront's last words: what it stored is there for the device, the copy engines and the host. The wait is spelled out because the
// compiler does not count the stores of inline assembly.
template <int NT>
__device__ __forceinline__ void say_done(const DoneWords &done) {
  // kThrough's stores are of system scope, like the word; others are released to it here. (64 KiB pool->pool with that instead 9.6 a pass, so 9.25.)
  if (NT != kThrough) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (threadIdx.x == 0) __hip_atomic_store(done.words + kDoneStride * blockIdx.x, done.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// (no words, no argument for them)
template <int NT, class A, class... Done>
__global__ __launch_bounds__(64) void ft_piece_kernel(A args, Done... done) {
  static_assert((NT == kThrough) == (sizeof...(Done) == 1), "words, and stores to go with them");
  const uint32_t t = A::kOne ? blockIdx.x : tile_of_workgroup(blockIdx.x, args.ntiles);
  move_tile<NT, A::kRows>(find_piece<NT>(args, t, threadIdx.x), threadIdx.x);
  if constexpr (NT == kThrough) say_done<NT>(done...);
}

// The same over the host link, which has to be full but not crowded: 64 wavefronts with 4 KiB of loads from host memory each, one on
// a compute unit, or 48 (in short jobs 128) with 4 KiB of stores, and each goes on to further tiles. Time beyond what the link takes for
// the bytes, us: 4 MiB in 32 tensors from the host 2.5 (the class's own kernel, 64 workgroups of 16 KiB, 9.5), to the host 2.4 (6.5);
// 128 or 256 wavefronts from the host 5.8, four a workgroup 10, every tile at once 39.
//
// A wavefront's first two tiles are given, the others are drawn from the counter, in the order of the pieces (of one piece they are
// dealt out where all wavefronts get as many). A tile costs one draw, so the draws of a launch are as many as its tiles, and who
// has made the last one sets the counter back. (Where no wavefront has a second tile the answers are not looked at, and the counter may be any.) A tile's loads, the draw
// in front of them and the search for the next tile's piece are waited for together, and the next tile's loads follow the
// stores at once.
struct LinkTiles {
  unsigned long long *counter;
  uint32_t ntiles;
  DoneWords done;
};

template <int NT, class A>
__global__ __launch_bounds__(64) void ft_link_piece_kernel(A args, LinkTiles l) {
  // (its low half: tiles are numbered in 32 bits, and of a 64-bit answer the compiler would use the unwanted register for an address of
  // the loads, which then wait for the answer)
  typedef uint32_t FT_GLOBAL *CounterP;
  const CounterP counter = reinterpret_cast<CounterP>(reinterpret_cast<uintptr_t>(l.counter));
  const uint32_t lane = threadIdx.x;
  uint32_t t = blockIdx.x, next = t + gridDim.x;
  Piece p = find_piece<NT>(args, t, lane);
  while (t < l.ntiles) {
    uint32_t begin, n, drawn = 0;
    run_tile(NT == kFromHost ? p.src : p.dst, p.len, p.tile, p.tile_no, &begin, &n);
    const uint64_t d = p.dst + begin, s = p.src + begin;
    const RunWindows w = run_windows(NT == kFromHost ? s : d, n < 16 ? 16u : n);  // at most 256: tiles are of 4 KiB at most
    if (!A::kOne && lane == 0) drawn = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    u32x4_any v[4];
    if (n >= 16) wave_run_loads<NT, 4>(v, s, w, 0, lane);
    else if (lane < n) st_off<uint8_t, 0>(d, lane, ld_off<uint8_t, 0>(s, lane));
    p = find_piece<NT>(args, next < l.ntiles ? next : t, lane);  // (found again where there is no next)
    t = next;
    next += gridDim.x;
    if (!A::kOne) {
      drawn = uniform32(drawn);
      if (drawn == l.ntiles - 1 && lane == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      next = 2 * gridDim.x + drawn;
    }
    if (n >= 16) wave_run_stores<NT, 4>(v, d, w, 0, lane);
  }
  if (l.done.words != nullptr) say_done<NT>(l.done);
}

namespace {

struct Launch {
  int cls;
  uint32_t ntiles, lds;
  unsigned long long *counter;
  DoneWords done;
  hipStream_t stream;
  hipEvent_t ev_start, ev_stop;
};

template <class A>
hipError_t launch(const A &a, const Launch &l) {
  static_assert(sizeof(A) + sizeof(LinkTiles) <= 4096, "kernel arguments end at 4 KiB");
  const dim3 grid(piece_workgroups(l.cls, l.ntiles)), block(64);
  const LinkTiles tiles = {l.counter, l.ntiles, l.done};
  if (l.done.words != nullptr && (grid.x > kDoneWords || a.tile == kStreamTile)) return hipErrorInvalidValue;
  if (l.cls == 2 && l.done.words != nullptr) {
    if constexpr (!A::kSays) return hipErrorInvalidValue;
    else hipExtLaunchKernelGGL((ft_piece_kernel<kThrough, A, DoneWords>), grid, block, l.lds, l.stream, l.ev_start, l.ev_stop, 0, a, l.done);
  } else if (l.cls == 2 && a.tile == kStreamTile) {
    if constexpr (A::kRows) return hipErrorInvalidValue;
    else hipExtLaunchKernelGGL((ft_piece_kernel<kStream, A>), grid, block, l.lds, l.stream, l.ev_start, l.ev_stop, 0, a);
  } else if (l.cls == 2) hipExtLaunchKernelGGL((ft_piece_kernel<0, A>), grid, block, l.lds, l.stream, l.ev_start, l.ev_stop, 0, a);
  else if constexpr (A::kRows) return hipErrorInvalidValue;
  else if (l.cls == 0) hipExtLaunchKernelGGL((ft_link_piece_kernel<kFromHost, A>), grid, block, 0, l.stream, l.ev_start, l.ev_stop, 0, a, tiles);
  else hipExtLaunchKernelGGL((ft_link_piece_kernel<kToHost, A>), grid, block, 0, l.stream, l.ev_start, l.ev_stop, 0, a, tiles);
  return hipGetLastError();
}

template <uint32_t CAP, uint32_t SHAPES>
hipError_t launch_along(const PieceTables &t, const Launch &l) {
  if (t.n > CAP || t.nshapes > SHAPES) return hipErrorInvalidValue;
  PieceArgs<CAP, SHAPES> a;
  a.n = t.n;
  a.tile = t.tile;
  a.ntiles = t.ntiles;
  a.src0 = t.src0;
  a.dst0 = t.dst0;
  for (uint32_t i = 0; i < t.n; ++i) {
    a.at[i].src = (uint32_t)(t.at[i].src - t.src0);
    a.at[i].dst = (uint32_t)(t.at[i].dst - t.dst0);
  }
  std::memcpy(a.first, t.first, t.n * sizeof(uint32_t));
  std::memcpy(a.len, t.len, t.n * sizeof(uint32_t));
  if (SHAPES != 0) {
    uint8_t *shape = reinterpret_cast<uint8_t *>(a.shape);
    for (uint32_t i = 0; i < t.n; ++i) shape[i] = (uint8_t)t.shape[i];
    std::memcpy(static_cast<void *>(a.edges), t.edges, t.n * sizeof(PieceEdges));
    std::memcpy(static_cast<void *>(a.shapes), t.shapes, t.nshapes * sizeof(PieceRows));
  }
  return launch(a, l);
}

template <uint32_t BLOCKS, bool CLOSE>
hipError_t launch_refs(const PieceTables &t, const Launch &l) {
  if (t.n > BLOCKS * kPieceBlock) return hipErrorInvalidValue;
  static_assert(256 * kPieceBlock >= kMaxPieces, "a block for every piece");
  PieceRefs<BLOCKS, CLOSE> r;
  r.n = t.n;
  r.tile = t.tile;
  r.ntiles = t.ntiles;
  r.src0 = t.src0;
  r.dst0 = t.dst0;
  r.packed = t.packed;
  for (uint32_t b = 0; b * kPieceBlock < t.n; ++b) r.block[b] = t.first[b * kPieceBlock];
  return launch(r, l);
}

}  // namespace

hipError_t launch_pieces(const PieceTables &t, int cls, bool on_host, unsigned long long *counter, const DoneWords &done, hipStream_t stream,
                         hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (t.n == 0 || t.ntiles == 0 || cls < 0 || cls > 2 || (on_host && !pieces_go_along(t)) || (cls != 2 && t.tile > 4096) || t.tile > kStreamTile) return hipErrorInvalidValue;
  const Launch l = {cls, t.ntiles, piece_lds(cls, t), counter, done, stream, ev_start, ev_stop};
  const bool rows = t.shape != nullptr;
  if (!on_host) {
    if (rows || t.packed == nullptr) return hipErrorInvalidValue;
    if (t.n <= 16 * kPieceBlock) return t.close ? launch_refs<16, true>(t, l) : launch_refs<16, false>(t, l);
    if (t.n <= 64 * kPieceBlock) return t.close ? launch_refs<64, true>(t, l) : launch_refs<64, false>(t, l);
    return t.close ? launch_refs<256, true>(t, l) : launch_refs<256, false>(t, l);
  }
  if (rows) {
    if (t.n <= 16 && t.nshapes <= 16) return launch_along<16, 16>(t, l);
    if (t.n <= 64) return launch_along<64, 64>(t, l);
    return launch_along<kRowsAlong, 16>(t, l);
  }
  if (t.n == 1 && (cls == 2 || !piece_draws(cls, t))) return launch_along<1, 0>(t, l);
  if (t.n <= 16) return launch_along<16, 0>(t, l);
  if (t.n <= 48) return launch_along<48, 0>(t, l);
  if (t.n <= 128) return launch_along<128, 0>(t, l);
  return launch_along<kRunsAlong, 0>(t, l);
}

}  // namespace ft
