// Device helpers of the kernels that give every wavefront tiles of its own.
#pragma once
#include <hip/hip_runtime.h>

#include "ft_windows.h"

namespace ft {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The job's tables are written before the launch and never during it. Reading them
// through constant-address-space pointers lets uniform reads go through the scalar
// unit and its cache, which the streaming vector traffic does not evict.
#define FT_CONST __attribute__((address_space(4)))

// Every payload address (pool memory or pinned host memory) is a global-segment
// address. Saying so keeps the copies off the flat path, whose loads also count on
// the scalar/LDS wait counter and would serialise with the table reads.
#define FT_GLOBAL __attribute__((address_space(1)))

// How a routine reaches memory, its first template parameter NT: 0 ordinary loads and stores (data that
// is wanted in the caches); kStream nontemporal loads and stores (payload streaming through HBM once);
// kToHost nontemporal loads and stores that are written through to the fabric at once (the `sc1` bit)
// for destinations in host memory. A nontemporal or ordinary store to host memory stays in the L2 until
// that evicts it or the kernel ends: the tiny workload's pool->host kernel had every store issued after
// 260 us and then ended 80 us later, when the L2 had written its lines back over the link (50 GB/s);
// written through, the link carries them while the kernel runs (55 GB/s, what host->pool reaches on the
// same buffers). `sc0 sc1` measured 53.4 GB/s, `sc0 sc1 nt` 53.5. Towards HBM every other combination
// of the bits is slower than `nt` alone. (The stores are inline assembly, and the compiler does not keep the next
// instructions from writing a store's data registers before it has read them, which takes two wait states on this
// architecture: hence the s_nop behind each.) kFromHost: as kStream, for the wave kernels' sources in host memory.
// kThrough: ordinary loads, and stores of system scope (`sc0 sc1`), which the device, the copy engines and the host see once a wait for them is over: for
// kernels that say themselves when they are done.
constexpr int kStream = 1, kToHost = 2, kFromHost = 3, kThrough = 4;

// 16 bytes from any address (the hardware splits an access that straddles aligned granules).
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

// A value that is the same in every lane of the wavefront, moved to scalar registers: what
// is computed from it stays on the scalar unit and table reads indexed by it are scalar
// loads.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (uint64_t)hi << 32 | lo;
}

// What one lane has, the same one for all.
__device__ __forceinline__ uint32_t of_lane32(uint32_t v, uint32_t lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ uint64_t of_lane64(uint64_t v, uint32_t lane) {
  return (uint64_t)of_lane32((uint32_t)(v >> 32), lane) << 32 | of_lane32((uint32_t)v, lane);
}

// What each lane has, and all lanes before it.
__device__ __forceinline__ uint32_t wave_sums(uint32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // within a row of 16: from 1, 2, 4 and 8 lanes before
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // the last of a row to the row after it, of two rows to the two after them
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// How many of the 64 lanes say yes.
__device__ __forceinline__ uint32_t wave_count(bool yes) { return (uint32_t)__popcll(__ballot(yes)); }

// An address off a base that is the same in every lane: base in scalar registers, 32 bits of offset per lane.
// Loads are ordinary ones unless NT: the source has often just been written, and a piece's lines may be wanted
// again. Stores are nontemporal always. Against ordinary stores that is as good or better wherever it was
// measured (64 tensors, 34 MB: source in the last-level cache 12.6 -> 11.1 us, not there 18.7 -> 16.8); with
// nontemporal loads as well, what the cache holds is not served from it (34 MB 11.1 against 16.7 us), beyond its size
// they are the faster ones.
template <class V, int NT>
__device__ __forceinline__ V ld_off(uint64_t base, uint32_t off) {
  const V FT_GLOBAL *at = reinterpret_cast<const V FT_GLOBAL *>(reinterpret_cast<const char FT_GLOBAL *>(base) + off);
  return NT == kStream || NT == kFromHost ? __builtin_nontemporal_load(at) : *at;
}
template <class V, int NT>
__device__ __forceinline__ void st_off(uint64_t base, uint32_t off, V v) {
  if constexpr (NT == kThrough && sizeof(V) == 16) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(base + off), "v"(v) : "memory");
    return;
  }
  if (NT == kToHost && sizeof(V) == 16) {
    // Written through to the fabric at once, as st16 does. The whole address in vector registers: between a vector instruction
    // that writes a scalar register and a store that reads it there must be five wait states, which the compiler does not
    // see to for inline assembly.
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(base + off), "v"(v) : "memory");
    return;
  }
  if constexpr (NT == kThrough && sizeof(V) == 1) {
    asm volatile("global_store_byte %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(base + off), "v"((uint32_t)v) : "memory");
    return;
  }
  __builtin_nontemporal_store(v, reinterpret_cast<V FT_GLOBAL *>(reinterpret_cast<char FT_GLOBAL *>(base) + off));
}

// Up to R * 64 windows of a contiguous run, from window `blk` on, loaded and stored. All loads before the first store; no load is
// predicated (a lane past the last window repeats it and stores nothing).
template <int NT, uint32_t R>
__device__ __forceinline__ void wave_run_loads(u32x4_any (&v)[R], uint64_t s, const RunWindows &w, uint32_t blk, uint32_t lane) {
#pragma unroll
  for (uint32_t i = 0; i < R; ++i) v[i] = ld_off<u32x4_any, NT>(s, run_window_at(w, blk + lane + i * 64));
}
template <int NT, uint32_t R>
__device__ __forceinline__ void wave_run_stores(const u32x4_any (&v)[R], uint64_t d, const RunWindows &w, uint32_t blk, uint32_t lane) {
#pragma unroll
  for (uint32_t i = 0; i < R; ++i)
    if (blk + lane + i * 64 < w.count) st_off<u32x4_any, NT>(d, run_window_at(w, blk + lane + i * 64), v[i]);
}
template <int NT, uint32_t R>
__device__ __forceinline__ void wave_run_pass(uint64_t d, uint64_t s, const RunWindows &w, uint32_t blk, uint32_t lane) {
  u32x4_any v[R];
  wave_run_loads<NT, R>(v, s, w, blk, lane);
  wave_run_stores<NT, R>(v, d, w, blk, lane);
}

}  // namespace ft
