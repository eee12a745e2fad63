// ft_submit_static: the submit for callers that cannot allocate (code under HIP graph capture,
// tight serving loops, harnesses that forbid hipMalloc). It does what ft_submit_transfers does for
// a job of pinned-host and pool sides - same validation, same chunk order, same kernels - but
// takes nothing from the runtime: no device buffer, no pinned buffer, no event, no stream. What the
// kernels need beyond the caller's memory (the schedule tables and the ticket counter of each link
// class) lies in one fixed array in device memory that belongs to this library, and everything is
// launched on the caller's stream.
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "ft_guard.h"
#include "ft_internal.h"

namespace ft {

// Per link class: one 256-byte line with the ticket counter, then the class's tables.
constexpr uint64_t kStaticTableBytes = 64 * 1024;
constexpr uint64_t kStaticClassBytes = 256 + kStaticTableBytes;
constexpr uint64_t kScratchBytes = FT_NCLASS * kStaticClassBytes;  // 197 376 bytes per GPU, held until the process ends

// In host code this name is a stand-in for the device array, not its address: host code uses the
// pointer that hipGetSymbolAddress returns for the current device (static_scratch below).
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kScratchBytes];

struct StaticDevice {
  unsigned char *ptr = nullptr;  // this device's copy of `scratch`
  int cu_count = 0;
};

// The scratch array of device `device`, which must be current. Looked up once per device: every
// GPU holds its own copy of the array at its own address.
int static_scratch(ft_pool *p, int device, StaticDevice *out) {
  static std::mutex mu;
  static std::unordered_map<int, StaticDevice> table;
  std::lock_guard<std::mutex> lock(mu);
  auto it = table.find(device);
  if (it != table.end()) {
    *out = it->second;
    return FT_OK;
  }
  StaticDevice sd;
  FT_HIP(p, hipGetSymbolAddress(reinterpret_cast<void **>(&sd.ptr), HIP_SYMBOL(scratch)));
  FT_HIP(p, hipDeviceGetAttribute(&sd.cu_count, hipDeviceAttributeMultiprocessorCount, device));
  if (sd.ptr == nullptr || sd.cu_count <= 0) {
    p->hip_error = "ft_submit_static: no scratch array on this device";
    return FT_EHIP;
  }
  table[device] = sd;
  *out = sd;
  return FT_OK;
}

// Writes `nwords` 8-byte words that came with the launch to dst, and (zero != null) sets the
// class's counter line back to zero: the array keeps what the last call left in it.
__global__ __launch_bounds__(kInlineBytes / 8) void ft_scratch_put_kernel(uint64_t *dst, InlineBlob blob, uint32_t nwords,
                                                                          unsigned long long *zero) {
  const uint32_t i = threadIdx.x;
  if (i < nwords) dst[i] = blob.w[i];
  if (zero != nullptr && i < 2) zero[i] = 0ull;
}

// n bytes of tables (a multiple of 8) to the array at d, in pieces that travel with small launches, the first of which
// also clears the counter. On one stream these launches and the kernel behind them run one after another.
hipError_t put_words(char *d, const char *h, uint64_t n, unsigned long long *counter, hipStream_t stream) {
  InlineBlob piece;
  for (uint64_t at = 0; at < n; at += kInlineBytes) {
    const uint64_t m = n - at < kInlineBytes ? n - at : kInlineBytes;
    std::memcpy(piece.w, h + at, m);
    hipLaunchKernelGGL(ft_scratch_put_kernel, dim3(1), dim3(kInlineBytes / 8), 0, stream, reinterpret_cast<uint64_t *>(d + at), piece,
                       (uint32_t)(m / 8), at == 0 ? counter : nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

struct StaticClass {
  bool used = false;
  Layout lay;
  std::vector<Skip> skips;
  uint64_t ntickets = 0, tile_bytes = 0;
  uint32_t tiles_per_chunk = 0;
  int code = 0;
  // launched as pieces (ft_pieces.h): the tables at `words`
  PieceRoom room;
  PieceTables pieces;
  std::vector<uint64_t> words;
};

// What the class's tables would take with the descriptor table that the copy kernel proper needs and the wave kernel does
// without: the limit of this entry point does not depend on the kernel that a job happens to get. (A table with
// an entry per chunk alone can be left out, then the kernel searches; one with an entry per tile cannot.)
uint64_t tables_with_descriptor_table(const ClassPlan &cp, int c, bool with_p2p, uint64_t chunk_bytes) {
  uint64_t tile;
  uint32_t tiles_per_chunk;
  tile_shape(chunk_bytes, default_tile(c, with_p2p, mostly_short_rows(cp), cp.payload), &tile, &tiles_per_chunk);
  const Layout lay = layout_of(cp, 0, 1);
  const uint64_t entries = cp.nchunks * tiles_per_chunk + cp.funcs.size();
  const bool per_tile = tiles_per_chunk > 1 && cp.xfers.size() > 2 * cp.nchunks && entries <= kMaxChunkTable;
  const uint64_t skips = align_up(lay.chunks + entries * sizeof(uint32_t), 64);
  return per_tile ? align_up(skips + cp.funcs.size() * sizeof(Skip), 256) : lay.end;
}

}  // namespace ft

using namespace ft;

extern "C" int ft_submit_static(ft_pool *p, const ft_desc *descs, uint32_t ndesc, const uint32_t *weights,
                                uint32_t nfunc, uint64_t chunk_bytes, uint32_t flags, void *hip_stream) try {
  if (p == nullptr) return FT_EINVAL;
  if (flags & ~(uint32_t)FT_VALIDATE) return FT_EINVAL;
  std::lock_guard<std::mutex> lock(p->mu);
  SubmitPlan plan;
  int rc = plan_submit(p->slabs, p->windows, descs, ndesc, weights, nfunc, chunk_bytes, flags, &plan);
  if (rc != FT_OK) return rc;
  if (plan.has_pageable) return FT_EINVAL;  // pageable memory needs a pinned buffer, which would be an allocation
  const bool with_p2p = plan.cls[FT_P2P].nchunks > 0;
  StaticClass sc[FT_NCLASS];
  bool any = false;
  // every class is shaped and measured before anything is launched: all or nothing
  for (int c = 0; c < FT_NCLASS; ++c) {
    ClassPlan &cp = plan.cls[c];
    if (cp.nchunks == 0) continue;
    StaticClass &s = sc[c];
    s.used = any = true;
    if (c == FT_P2P) s.room = job_pieces(cp, c, chunk_bytes, false);  // (there is no counter pair here for the host link's)
    // Pieces that do not go along with their launch take a small launch for every 3 KiB of their list (pack_pieces), and so do the general tables: few tensors
    // in many chunks are shorter by these (20 tensors of 10 functions in chunks of 64 KiB, 40 MB: 18.4 us, by 640 pieces of 24 bytes 26.9), others by the list (100 of 64 KiB, 8 functions,
    // chunks of 32 KiB: 32.1 -> 27.6 a call; by 24 bytes a piece they would count as longer).
    const auto launches = [](uint64_t bytes) { return (bytes + kInlineBytes - 1) / kInlineBytes; };
    const Layout general = layout_of(cp, 0, 1);
    if (s.room.pieces != 0 && 12 * s.room.pieces <= kStaticTableBytes) {
      if (tables_with_descriptor_table(cp, c, with_p2p, chunk_bytes) > kStaticClassBytes) return FT_E2BIG;
      const auto shorter = [&](uint64_t bytes) { return bytes <= kStaticTableBytes && launches(bytes) < launches(general.end - general.phases); };
      const bool list = s.room.shapes == 0 && shorter(12 * s.room.pieces);  // (if its sides are close)
      if (list || s.room.shapes != 0 || s.room.pieces - cp.xfers.size() <= kRunsAlong) {  // (else they can't go along: nothing is written out)
        s.words.resize((piece_bytes(s.room) + 7) / 8);
        s.pieces = piece_places(reinterpret_cast<char *>(s.words.data()), s.room);
        if (build_pieces(cp, chunk_bytes, piece_tile(c, cp.payload), false, &s.pieces)) {
          if (pieces_go_along(s.pieces)) continue;
          if (list) find_base(&s.pieces);
          if (list && shorter(packed_bytes(s.pieces))) continue;
        }
        s.pieces = PieceTables();
      }
    }
    s.code = launch_code(cp, c, chunk_bytes, false, true);  // the classes run one after another
    if (s.code >= kWaveTiles) {
      tile_shape(chunk_bytes, wave_tile(s.code, cp.payload), &s.tile_bytes, &s.tiles_per_chunk);
      cp.chunk_desc.clear();
      cp.desc_per = 1;
      if (tables_with_descriptor_table(cp, c, with_p2p, chunk_bytes) > kStaticClassBytes) return FT_E2BIG;
    } else {
      tile_shape(chunk_bytes, default_tile(c, with_p2p, mostly_short_rows(cp), cp.payload), &s.tile_bytes, &s.tiles_per_chunk);
      build_chunk_table(cp, chunk_bytes, s.tile_bytes, s.tiles_per_chunk);
    }
    build_skips(cp, chunk_bytes, s.tile_bytes, s.tiles_per_chunk, &s.skips, &s.ntickets);
    s.lay = layout_of(cp, 0, 1);
    if (s.lay.end > kStaticClassBytes && cp.desc_per == 1) {
      // without the table of descriptors per chunk the decode searches the function's descriptors
      cp.chunk_desc.clear();
      s.lay = layout_of(cp, 0, 1);
    }
    if (s.lay.end > kStaticClassBytes) return FT_E2BIG;
  }
  if (!any) return FT_OK;
  DeviceGuard guard(p->device);
  StaticDevice sd;
  rc = static_scratch(p, p->device, &sd);
  if (rc != FT_OK) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  std::vector<char> h;
  InlineBlob piece;  // tables that go with their launch
  for (int c = 0; c < FT_NCLASS; ++c) {
    const StaticClass &s = sc[c];
    if (!s.used) continue;
    const ClassPlan &cp = plan.cls[c];
    char *d = reinterpret_cast<char *>(sd.ptr) + (uint64_t)c * kStaticClassBytes;
    if (s.pieces.n != 0) {
      const bool with_launch = pieces_go_along(s.pieces);
      PieceTables t = s.pieces;
      if (!with_launch) {
        h.assign(align_up(packed_bytes(t), 8), 0);
        pack_pieces(t, h.data());
        FT_HIP(p, put_words(d + 256, h.data(), h.size(), nullptr, stream));
        t.packed = d + 256;
      }
      FT_HIP(p, launch_pieces(t, c, with_launch, nullptr, DoneWords(), stream, nullptr, nullptr));
      continue;
    }
    uint64_t wg = s.code >= kWaveTiles ? wave_workgroups(sd.cu_count, s.code, s.ntickets)
                  : c == FT_P2P ? (uint64_t)sd.cu_count : (with_p2p || c == FT_P2H) ? 32u : 64u;
    if (wg > s.ntickets) wg = s.ntickets;
    const Layout small = inline_layout_of(cp);
    const bool single = cp.funcs.size() == 1 && cp.xfers.size() == 1;
    if (s.code >= kWaveTiles && !wave_draws(s.code, wg, s.ntickets, single) && small.end <= kInlineBytes) {
      // no counter and tables that fit the launch: nothing has to reach the array first (11 tensors, 18 MB: 11.0 -> 7.7 us
      // a call back to back, one tensor 10.5 -> 6.1: the small launch in front and the gap behind it are gone)
      ClassTable T{};
      fill_class_table(cp, small, reinterpret_cast<char *>(piece.w), nullptr, s.skips, s.ntickets, chunk_bytes, s.tile_bytes,
                       s.tiles_per_chunk, &T);
      T.single = single ? 1u : 0u;
      FT_HIP(p, launch_copy(T, s.code, (uint32_t)wg, stream, nullptr, nullptr, &piece));
      continue;
    }
    h.assign(s.lay.end, 0);
    ClassTable T{};
    fill_class_table(cp, s.lay, h.data(), d, s.skips, s.ntickets, chunk_bytes, s.tile_bytes, s.tiles_per_chunk, &T);
    // the counter line is not uploaded
    FT_HIP(p, put_words(d + s.lay.phases, h.data() + s.lay.phases, s.lay.end - s.lay.phases, T.ticket, stream));
    FT_HIP(p, launch_copy(T, s.code, (uint32_t)wg, stream, nullptr, nullptr));
  }
  return FT_OK;
}
FT_CATCH_ALL
