// kernels.h — gfx950 (CDNA4) kernels of the reshard library.
//
// The reshard moves bytes without arithmetic, so every kernel here is bound
// by HBM bandwidth; there is no matrix work and no MFMA.
//   k_prepare     one workgroup turns the plan into per-tile work: it
//                 compacts the block table into the sorted list of live
//                 blocks (wavefront prefix sums over block flags), resolves
//                 block-id ranges into list positions and scans the tile
//                 counts of every descriptor (wavefront prefix sums).
//   k_mark_pool   before it, the block flags of a pool too large for its LDS.
//   k_copy16      descriptor-driven copy in 16-byte chunks, 2 independent
//                 loads in flight per thread, non-temporal hints; a tile is
//                 512 consecutive chunks (8 KiB) of one descriptor.
//   k_copy_link   the same over the link to the host, on a narrow persistent
//                 grid with two tiles in flight per workgroup.
//   k_copy_linear contiguous bytes of the host buffer into a landing-ring slot.
//   k_copy_any    the same for lines that are not 16-byte aligned (odd column
//                 counts): unaligned 16-byte accesses on one side, the
//                 chunks of a line cut at the other side's boundaries.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "desc.h"

namespace atp {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((address_space(1))) global_u32x4;
typedef unsigned char __attribute__((address_space(1))) global_u8;

enum : int32_t { ERR_BAD_BLOCK = 1, ERR_LIVE_COUNT = 2 };

__device__ __forceinline__ uint32_t divq(uint32_t n, uint64_t magic) {
  return magic ? uint32_t(__umul64hi(uint64_t(n), magic)) : n;
}

// The same for a dividend past 32 bits whose quotient fits them.
__device__ __forceinline__ uint32_t divl(uint64_t n, uint64_t magic) {
  return uint32_t(magic ? __umul64hi(n, magic) : n);
}

__device__ __forceinline__ char *slot_base(uint32_t slot, char *b0, char *b1, char *b2) {
  return slot == BUF_IN ? b0 : (slot == BUF_OUT ? b1 : b2);
}

// Exclusive prefix sum over the 1024 threads of a workgroup (wave64 scans
// with lane shuffles, then one scan of the 16 wave totals).
template <typename T>
__device__ T block_exclusive_scan(T v, T *lds16, T *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  T x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) lds16[wave] = x;
  __syncthreads();
  if (wave == 0) {
    T w = lane < nw ? lds16[lane] : T(0);
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      T y = __shfl_up(w, d, 64);
      if (lane >= d) w += y;
    }
    if (lane < nw) lds16[lane] = w;
  }
  __syncthreads();
  T base = wave ? lds16[wave - 1] : T(0);
  *total = lds16[nw - 1];
  __syncthreads();
  return base + x - v;
}

struct PrepArgs {
  const Desc *plan_descs;  // the plan's descriptors, in pinned host memory (null: already in descs)
  Desc *descs;             // their device copies, block ranges resolved
  int32_t n_desc;
  int32_t kv;            // 1: compact the block table first
  int64_t *prefix;       // [n_desc + 1] tile prefix
  int32_t *err;          // error word, in pinned host memory
  const int32_t *table;  // block table, n_entries int32
  int64_t n_entries;
  uint64_t *mask;        // [ceil(n_blocks / 64)] live blocks of each group of 64 ids
  int32_t *rank;         // [ceil(n_blocks / 64)] live blocks before each group
  int32_t *live;         // [n_blocks] sorted live block ids
  int64_t n_blocks;
  int64_t expect_live;
};

// Live ids below b: the position in the live list where block b's would be.
__device__ __forceinline__ int64_t live_rank(const PrepArgs &a, int64_t b, int64_t total) {
  if (b <= 0) return 0;
  if (b >= a.n_blocks) return total;
  return a.rank[b >> 6] + __popcll(a.mask[b >> 6] & ((uint64_t(1) << (b & 63)) - 1));
}

// Block ids k_prepare takes at once: a byte each in LDS.
constexpr int kPrepWindow = 1 << 16;
constexpr int kPrepThreads = 1024;
constexpr int kPrepGroups = 8;  // groups of 64 ids in flight per wave

// Table entries [e, e + 1024 K), K loads in flight per thread: marks the ids
// below n (in LDS or in memory) and keeps the largest id seen.
template <int K, typename Flags>
__device__ __forceinline__ void mark_blocks(const PrepArgs &a, int64_t e, uint32_t n, Flags flag, int32_t *top) {
  int32_t v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t i = e + threadIdx.x + int64_t(k) * kPrepThreads;
    v[k] = a.table[i < a.n_entries ? i : a.n_entries - 1];
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    *top = v[k] > *top ? v[k] : *top;
    if (uint32_t(v[k]) < n) flag[uint32_t(v[k])] = 1;  // n is at most 2^31: no negative id is below it
  }
}

// The whole table: the widest batches first, then one as wide as the rest needs.
template <typename Flags>
__device__ __forceinline__ void mark_table(const PrepArgs &a, uint32_t n, Flags flag, int32_t *top) {
  constexpr int nt = kPrepThreads;
  int64_t e = 0;
  for (; a.n_entries - e >= int64_t(nt) * 16; e += int64_t(nt) * 16) mark_blocks<16>(a, e, n, flag, top);
  const int64_t rest = a.n_entries - e;
  if (rest > nt * 8)
    mark_blocks<16>(a, e, n, flag, top);
  else if (rest > nt * 4)
    mark_blocks<8>(a, e, n, flag, top);
  else if (rest > nt)
    mark_blocks<4>(a, e, n, flag, top);
  else if (rest > 0)
    mark_blocks<1>(a, e, n, flag, top);
}

// Flags of a pool beyond one window, a byte per id: the last quarter of the
// live list's room.  The list grows 4 bytes per live id from the front, so
// that after the ids below w it ends at most at 4 w, below the flags of the
// ids from w on.
__device__ __forceinline__ global_u8 *pool_flags(const PrepArgs &a) {
  return (global_u8 *)(reinterpret_cast<uint8_t *>(a.live) + 3 * flag_room(a.n_blocks));
}

// Before k_prepare where the pool is larger than one window: the flags, and
// the largest id of the table in rank[0].  One workgroup (a barrier lies
// between clearing and marking), in a kernel of its own so that the small
// pools' k_prepare stays small.
__global__ void __launch_bounds__(kPrepThreads) k_mark_pool(PrepArgs a) {
  __shared__ int32_t s_top;
  global_u8 *flags = pool_flags(a);
  if (threadIdx.x == 0) s_top = -1;
  for (int64_t i = threadIdx.x; i < flag_room(a.n_blocks) / 16; i += kPrepThreads)
    ((global_u32x4 *)flags)[i] = u32x4{0, 0, 0, 0};
  __syncthreads();
  int32_t top = -1;
  mark_table(a, uint32_t(a.n_blocks < (int64_t(1) << 31) ? a.n_blocks : int64_t(1) << 31), flags, &top);
  atomicMax(&s_top, top);
  __syncthreads();
  if (threadIdx.x == 0) a.rank[0] = s_top;
}

// One workgroup, bound by the latency of its loads and by what one CU moves.
// It reads few descriptors from the host's pinned copy and writes the error
// word there itself: a copy command before it and one at the call's end cost
// the stream a blit kernel each (2-4 us and the gaps beside them) and the
// host two more calls; a TP 4->3 KV move of 84 MB took 87 us a call
// with them and 83 without.
//
// The block table is read with up to 16 independent loads per thread; an
// id sets its byte in LDS (plain stores: neighbouring ids of an ordered
// table would queue up on the words of a bit mask, and random ids on the
// cache lines of flags in memory).  Each wave then turns 64 bytes into a
// mask with a ballot, one scan over the groups gives their ranks, and a wave
// writes the ids of a group to consecutive places.  A pool beyond kPrepWindow
// ids is marked in memory (k_mark_pool) in one pass over the table and taken window
// by window from there (a pass over the table per window took longer from about the third
// window on, and more the emptier the table is).
// MARKED: k_mark_pool has set the flags of the pool.
template <bool MARKED>
__global__ void __launch_bounds__(kPrepThreads) k_prepare(PrepArgs a) {
  __shared__ int64_t s64[16];
  __shared__ int32_t s32[16];
  __shared__ int32_t s_err;
  __shared__ __align__(16) uint8_t s_flag[kPrepWindow];
  __shared__ uint64_t s_mask[kPrepWindow / 64];
  __shared__ int32_t s_rank[kPrepWindow / 64];
  static_assert(kPrepWindow / 64 == kPrepThreads, "one group per thread in the scan");
  const int tid = threadIdx.x, nt = kPrepThreads, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_err = 0;
  // (the loops below read descs only after a barrier)
  constexpr int kDescLoads = 4;
  const int64_t words = a.plan_descs ? int64_t(a.n_desc) * int64_t(sizeof(Desc) / 16) : 0;
  for (int64_t i0 = tid; i0 < words; i0 += nt * kDescLoads) {
    u32x4 v[kDescLoads];
#pragma unroll
    for (int k = 0; k < kDescLoads; ++k) {
      const int64_t i = i0 + int64_t(k) * nt;
      v[k] = reinterpret_cast<const u32x4 *>(a.plan_descs)[i < words ? i : words - 1];
    }
#pragma unroll
    for (int k = 0; k < kDescLoads; ++k) {
      const int64_t i = i0 + int64_t(k) * nt;
      if (i < words) reinterpret_cast<u32x4 *>(a.descs)[i] = v[k];
    }
  }
  int64_t n_live = 0;
  if (a.kv) {
    int32_t top = -1;
    if (MARKED) top = a.rank[0];
    for (int64_t w0 = 0; w0 < a.n_blocks; w0 += kPrepWindow) {
      const int n = int(a.n_blocks - w0 < kPrepWindow ? a.n_blocks - w0 : kPrepWindow);
      const int groups = (n + 63) >> 6;
      if (!MARKED) {  // one window
        for (int i = tid; i < groups * 4; i += nt) reinterpret_cast<u32x4 *>(s_flag)[i] = u32x4{0, 0, 0, 0};
        __syncthreads();
        mark_table(a, uint32_t(n), s_flag, &top);
      } else {
        for (int i = tid; i < groups * 4; i += nt)
          reinterpret_cast<u32x4 *>(s_flag)[i] = ((const global_u32x4 *)(pool_flags(a) + w0))[i];
      }
      __syncthreads();
      for (int g = wave * kPrepGroups; g < groups; g += kPrepGroups * (nt >> 6)) {
        uint8_t f[kPrepGroups];
#pragma unroll
        for (int k = 0; k < kPrepGroups; ++k) f[k] = g + k < groups ? s_flag[(g + k) * 64 + lane] : 0;
#pragma unroll
        for (int k = 0; k < kPrepGroups; ++k) {
          const uint64_t m = __ballot(f[k] != 0);
          if (lane == k && g + k < groups) s_mask[g + k] = m;
        }
      }
      __syncthreads();
      int32_t tot;
      const uint64_t mine = tid < groups ? s_mask[tid] : 0;
      const int32_t r = int32_t(n_live) + block_exclusive_scan<int32_t>(__popcll(mine), s32, &tot);
      if (tid < groups) {
        s_rank[tid] = r;
        a.mask[(w0 >> 6) + tid] = mine;
        a.rank[(w0 >> 6) + tid] = r;
      }
      __syncthreads();
      for (int g = wave * kPrepGroups; g < groups; g += kPrepGroups * (nt >> 6)) {
        uint8_t f[kPrepGroups];
        int32_t at[kPrepGroups];
#pragma unroll
        for (int k = 0; k < kPrepGroups; ++k) {
          f[k] = g + k < groups ? s_flag[(g + k) * 64 + lane] : 0;
          at[k] = g + k < groups ? s_rank[g + k] : 0;
        }
#pragma unroll
        for (int k = 0; k < kPrepGroups; ++k) {
          const uint64_t m = __ballot(f[k] != 0);
          int32_t *to = a.live + __builtin_amdgcn_readfirstlane(at[k]);
          const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0));
          if (f[k]) to[below] = int32_t(w0) + (g + k) * 64 + lane;
        }
      }
      n_live += tot;
      __syncthreads();  // the next pass clears the flags this one still reads
    }
    if (top >= a.n_blocks) atomicOr(&s_err, ERR_BAD_BLOCK);
    if (tid == 0 && n_live != a.expect_live) atomicOr(&s_err, ERR_LIVE_COUNT);
  }
  __syncthreads();
  const bool bad = s_err != 0;
  // resolve block ranges, count tiles, scan
  int64_t per = (a.n_desc + nt - 1) / nt;
  int64_t d0 = tid * per, d1 = d0 + per < a.n_desc ? d0 + per : a.n_desc;
  int64_t sum = 0;
  for (int64_t d = d0; d < d1; ++d) {
    Desc &x = a.descs[d];
    if (x.flags & DF_BLOCKRANGE) {
      const int64_t b0 = x.o_begin, b1 = x.o_end;
      x.o_begin = live_rank(a, b0, n_live);
      x.o_end = b1 > b0 ? live_rank(a, b1, n_live) : x.o_begin;
      x.flags &= ~DF_BLOCKRANGE;
    }
    if (bad) x.o_end = x.o_begin;  // an invalid table moves nothing
    uint64_t lines = uint64_t(x.o_end - x.o_begin) * x.rows;
    const uint64_t tiles = (lines * x.cpl + tile_chunks(x.flags) - 1) / tile_chunks(x.flags);
    a.prefix[d] = int64_t(tiles);  // temporarily the count
    sum += int64_t(tiles);
  }
  int64_t tot;
  int64_t run = block_exclusive_scan<int64_t>(sum, s64, &tot);
  for (int64_t d = d0; d < d1; ++d) {
    int64_t c = a.prefix[d];
    a.prefix[d] = run;
    run += c;
  }
  if (tid == 0) {
    a.prefix[a.n_desc] = tot;
    *a.err = s_err;
    __threadfence_system();
  }
}

// Descriptor of tile t: the last d in [d0, d1) with prefix[d] <= t.
__device__ __forceinline__ int find_desc(const int64_t *__restrict__ prefix, int d0, int d1, int64_t t) {
  int lo = d0, hi = d1 - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

struct LineAddr {
  char *src, *dst;
};

// The live-block list and the descriptors are never written while a copy
// kernel runs, so a wave-uniform index may read them through the scalar
// cache (constant address space) instead of a per-lane vector load.
typedef const int32_t __attribute__((address_space(4))) *const_i32_p;

// Addresses of the first line of outer item `orel` of descriptor x.
// UNIFORM: `orel` is the same on every lane of the wave, and the block id
// comes in through a scalar load.
template <bool UNIFORM>
__device__ __forceinline__ LineAddr item_addr(const Desc &x, uint32_t orel, char *b0, char *b1, char *b2,
                                              const int32_t *__restrict__ live) {
  int64_t o = x.o_begin + orel;
  uint64_t id = 0;
  if (x.flags & (DF_SRC_IND | DF_DST_IND))
    id = UNIFORM ? uint64_t(((const_i32_p)(live))[o]) : uint64_t(live[o]);
  uint64_t si = (x.flags & DF_SRC_IND) ? id : uint64_t(orel);
  uint64_t di = (x.flags & DF_DST_IND) ? id : uint64_t(orel);
  char *sb = slot_base((x.flags >> DF_SRC_SHIFT) & 3, b0, b1, b2);
  char *db = slot_base((x.flags >> DF_DST_SHIFT) & 3, b0, b1, b2);
  LineAddr la;
  la.src = sb + x.src_off + si * x.src_ostride;
  la.dst = db + x.dst_off + di * x.dst_ostride;
  return la;
}

// Addresses of line `line` of descriptor x.
template <bool UNIFORM>
__device__ __forceinline__ LineAddr line_addr(const Desc &x, uint32_t line, char *b0, char *b1, char *b2,
                                              const int32_t *__restrict__ live) {
  const uint32_t orel = divq(line, x.magic_rows);
  const uint32_t r = line - orel * x.rows;
  LineAddr la = item_addr<UNIFORM>(x, orel, b0, b1, b2, live);
  la.src += uint64_t(r) * x.src_pitch;
  la.dst += uint64_t(r) * x.dst_pitch;
  return la;
}

// Streaming 16-byte accesses: nothing is read twice, so both sides carry
// the non-temporal hint by default.  The pointers are cast to the global
// address space, which keeps the accesses global_* rather than flat_*
// where the compiler cannot infer it.

__device__ __forceinline__ u32x4 load16(const u32x4 *p) {
#if ATP_NT_LOAD
  return __builtin_nontemporal_load((const global_u32x4 *)(p));
#else
  return *(const global_u32x4 *)(p);
#endif
}

__device__ __forceinline__ void store16(u32x4 *p, u32x4 v) {
#if ATP_NT_STORE
  __builtin_nontemporal_store(v, (global_u32x4 *)(p));
#else
  *(global_u32x4 *)(p) = v;
#endif
}

// First tile of this workgroup.  Workgroups are dealt round-robin to the
// 8 XCDs; with ATP_XCD_MAP each XCD gets a contiguous run of tiles instead
// of every 8th one.
__device__ __forceinline__ int64_t tile_of_block() {
#if ATP_XCD_MAP
  const uint32_t G = gridDim.x, b = blockIdx.x, q = G >> 3, r = G & 7, xcd = b & 7, i = b >> 3;
  return xcd < r ? int64_t(xcd) * (q + 1) + i : int64_t(r) * (q + 1) + int64_t(xcd - r) * q + i;
#else
  return blockIdx.x;
#endif
}

// Source and destination of this thread's U chunks of a tile, for lines of
// any alignment (ANY) or aligned ones.  The line is resolved once per
// wavefront when its 64 chunks share one (KV head runs), else the outer item
// when they share that (the tokens of a block in the token-major layout:
// with a block id per lane, each chunk waited for its id before its load:
// host reads of 268 MB into 256 B lines took 4.97 ms, now 4.78),
// else per lane.  Lanes past the tile's end get its last chunk.
template <int U, bool ANY>
__device__ __forceinline__ void tile_addr(const Desc &x, uint64_t cbase, uint64_t clast, char *b0, char *b1, char *b2,
                                          const int32_t *__restrict__ live, const char **sp, char **dp) {
  // an aligned descriptor has fewer than 2^32 chunks
  using C = typename std::conditional<ANY, uint64_t, uint32_t>::type;
  const C base = C(cbase), last = C(clast);
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const C g0r = base + k * kThreads + wv * 64;
    const C g0 = g0r < last ? g0r : last;
    const C gl = last - g0 > 63 ? g0 + 63 : last;
    const C cr = base + k * kThreads + threadIdx.x;
    const C c = cr < last ? cr : last;
    const uint32_t lf = divl(g0, x.magic_line), ll = divl(gl, x.magic_line);
    LineAddr la;
    uint32_t col;
    if (lf == ll) {
      la = line_addr<true>(x, lf, b0, b1, b2, live);
      col = uint32_t(c - C(lf) * x.cpl);
    } else {
      const uint32_t line = divl(c, x.magic_line);
      const uint32_t item = divq(lf, x.magic_rows);
      if (item == divq(ll, x.magic_rows)) {
        la = item_addr<true>(x, item, b0, b1, b2, live);
        la.src += uint64_t(line - item * x.rows) * x.src_pitch;
        la.dst += uint64_t(line - item * x.rows) * x.dst_pitch;
      } else {
        la = line_addr<false>(x, line, b0, b1, b2, live);
      }
      col = uint32_t(c - C(line) * x.cpl);
    }
    uint64_t off = uint64_t(col) * 16;  // a line may be just under 4 GiB long
    if (ANY) {
      const uint32_t h = uint32_t(uintptr_t((x.flags & DF_SRC_GRID) ? la.src : la.dst)) & 15;
      const uint64_t omax = uint64_t(x.run) - 16;
      off = off < h ? 0 : (off - h > omax ? omax : off - h);
    }
    sp[k] = la.src + off;
    dp[k] = la.dst + off;
  }
}

// Each tile resolves every address first (descriptor by value, block ids
// through scalar loads), then issues all of its loads, then all stores, so
// that no load waits behind another's address computation.  Lanes past the
// end of the tile load its last chunk again (a valid address) and store
// nothing: unconditional loads keep the compiler from waiting on each one.
// U chunks per thread: every descriptor of a launch has DF_WIDE exactly when
// U == kWideUnroll (the prepare kernel counted its tiles that way).
template <int U>
__global__ void __launch_bounds__(kThreads) k_copy16(const Desc *__restrict__ descs, const int64_t *__restrict__ prefix,
                                                     int d0, int d1, char *b0, char *b1, char *b2,
                                                     const int32_t *__restrict__ live) {
  constexpr int64_t kTile = int64_t(kThreads) * U;
  const int64_t T0 = prefix[d0], T1 = prefix[d1];
  for (int64_t t = T0 + tile_of_block(); t < T1; t += gridDim.x) {
    const int d = find_desc(prefix, d0, d1, t);
    const Desc x = descs[d];
    const uint32_t cpl = x.cpl;
    const uint64_t total = uint64_t(x.o_end - x.o_begin) * x.rows * cpl;
    const uint64_t cbase = uint64_t(t - prefix[d]) * kTile;
    const uint64_t clast = (cbase + kTile < total ? cbase + kTile : total) - 1;
    const uint32_t l0 = divq(uint32_t(cbase), x.magic_line);
    u32x4 v[U];
    if (l0 == divq(uint32_t(clast), x.magic_line)) {
      // the whole tile lies in one line: one address computation per tile
      const LineAddr la = line_addr<true>(x, l0, b0, b1, b2, live);
      const uint32_t col0 = uint32_t(cbase) - l0 * cpl;
      const uint32_t n = uint32_t(clast - cbase) + 1;
      const u32x4 *s = reinterpret_cast<const u32x4 *>(la.src) + col0;
      u32x4 *dd = reinterpret_cast<u32x4 *>(la.dst) + col0;
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t i = threadIdx.x + k * kThreads;
        v[k] = load16(s + (i < n ? i : n - 1));
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t i = threadIdx.x + k * kThreads;
        if (i < n) store16(dd + i, v[k]);
      }
      continue;
    }
    // several lines per tile
    const char *sp[U];
    char *dp[U];
    tile_addr<U, false>(x, cbase, clast, b0, b1, b2, live, sp, dp);
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = load16(reinterpret_cast<const u32x4 *>(sp[k]));
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (cbase + threadIdx.x + uint64_t(k) * kThreads <= clast) store16(reinterpret_cast<u32x4 *>(dp[k]), v[k]);
  }
}

// Lines that are not 16-byte aligned.  Unaligned 16-byte accesses are
// ordinary global memory operations here, so the bytes need no staging in
// LDS: a chunk starts at a 16-byte boundary of one side, which makes that
// side's accesses aligned, the other side is accessed wherever it falls, and
// the first and last chunk of a line are moved inwards so that all of their
// 16 bytes lie in the line (they repeat bytes of their neighbours, the same
// values).  The aligned side is the pinned host buffer of a host read
// (DF_SRC_GRID: a request that crosses a 64-byte line costs two PCIe reads)
// and the destination otherwise.  Tiles are consecutive chunks of one
// descriptor, as in k_copy16, so short lines share a workgroup: bound by the
// link or by HBM like the aligned ones.  Measured against one workgroup per
// line through LDS: host reads of 5 KB / 700 B / 344 B lines 19 / 2.8 / 1.5
// -> 57 / 56 / 54 GB/s; HBM copies of the same lines (read + write) 3.7 /
// 0.65 / 0.34 -> 4.8 / 3.2 / 2.7 TB/s at 306 / 124 / 71 MB.  Tiles of twice
// the width, and source boundaries for the HBM copies, were 0-9 % slower.
typedef u32x4 __attribute__((address_space(1), aligned(1))) global_u32x4_any;

__device__ __forceinline__ u32x4 load16_any(const char *p) {
  return __builtin_nontemporal_load((const global_u32x4_any *)(p));
}
__device__ __forceinline__ void store16_any(char *p, u32x4 v) {
  __builtin_nontemporal_store(v, (global_u32x4_any *)(p));
}

// Whether a launch is to go at half its rate: a word in pinned host memory,
// looked at every kCalmTiles tiles.  Each wave decides for itself.  (Only the
// CALM kernels look: the others' loops stay as they are without it.)
constexpr uint32_t kCalmTiles = 32;
template <bool CALM>
struct Calm {
  const int32_t *word;
  uint32_t n = 0;
  int32_t now = 0, seen = 0;

  __device__ __forceinline__ explicit Calm(const int32_t *w) : word(w) {}
  __device__ __forceinline__ bool poll() {
    if (!CALM) return false;
    if (n++ % kCalmTiles == 0) {
      now = seen;  // the read before this one: it has long arrived
      seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      if (n == 1) now = seen;
    }
    return now != 0;
  }
};

// Lines [c0, c1] shorter than one chunk, one per lane, byte by byte.
__device__ __forceinline__ void copy_short_lines(const Desc &x, uint64_t c0, uint64_t c1, char *b0, char *b1, char *b2,
                                                 const int32_t *__restrict__ live) {
  for (uint64_t c = c0 + threadIdx.x; c <= c1; c += kThreads) {
    const LineAddr la = line_addr<false>(x, uint32_t(c), b0, b1, b2, live);
    for (uint32_t i = 0; i < x.run; ++i) ((global_u8 *)la.dst)[i] = ((const global_u8 *)la.src)[i];
  }
}

template <bool CALM>
__global__ void __launch_bounds__(kThreads) k_copy_any(const Desc *__restrict__ descs,
                                                       const int64_t *__restrict__ prefix, int d0, int d1, char *b0,
                                                       char *b1, char *b2, const int32_t *__restrict__ live,
                                                       const int32_t *calm) {
  constexpr int U = kUnroll;
  Calm<CALM> slow(calm);
  const int64_t T0 = prefix[d0], T1 = prefix[d1];
  for (int64_t t = T0 + tile_of_block(); t < T1; t += gridDim.x) {
    const int d = find_desc(prefix, d0, d1, t);
    const Desc x = descs[d];
    const uint64_t total = uint64_t(x.o_end - x.o_begin) * x.rows * x.cpl;
    const uint64_t cbase = uint64_t(t - prefix[d]) * kTileChunks;
    const uint64_t clast = (cbase + kTileChunks < total ? cbase + kTileChunks : total) - 1;
    if (slow.poll()) __builtin_amdgcn_s_sleep(55);  // about the time a tile takes on 8 workgroups over the link
    if (x.run < 16) {
      copy_short_lines(x, cbase, clast, b0, b1, b2, live);
      continue;
    }
    const char *sp[U];
    char *dp[U];
    tile_addr<U, true>(x, cbase, clast, b0, b1, b2, live, sp, dp);
    u32x4 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = load16_any(sp[k]);
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (cbase + threadIdx.x + uint64_t(k) * kThreads <= clast) store16_any(dp[k], v[k]);
  }
}

// k_copy16 over the link to the host (inflow read from pinned memory,
// outbound bytes written to it), on a narrow persistent grid: a workgroup
// loads its next tile before it stores the one it has, so that the lookup of
// the next descriptor and of its addresses, slow beside an HBM-bound repack,
// does not leave the link without requests.  The two tiles in flight keep
// registers of their own (moving one into the other would wait for its
// loads).  The 40-layer TP 8->7 last rank's 374 MB came in at 48 GB/s beside
// its repack with one tile in flight on 32 workgroups, 57 with two on 20:
// the step took 7.33 ms and takes 6.63.  A calm launch keeps one tile in flight.
template <int U>
struct LinkTile {
  u32x4 v[U];
  char *dp[U];

  __device__ __forceinline__ void load(const Desc &x, int64_t tile, char *b0, char *b1, char *b2,
                                       const int32_t *__restrict__ live) {
    constexpr int64_t kTile = int64_t(kThreads) * U;
    const uint64_t total = uint64_t(x.o_end - x.o_begin) * x.rows * x.cpl;
    const uint64_t c0 = uint64_t(tile) * kTile, cl = (c0 + kTile < total ? c0 + kTile : total) - 1;
    const char *sp[U];
    tile_addr<U, false>(x, c0, cl, b0, b1, b2, live, sp, dp);
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = load16(reinterpret_cast<const u32x4 *>(sp[k]));
  }
  // every lane stores: those past the tile's end its last chunk once more
  // (a store under a condition would make the next load wait for all of it)
  __device__ __forceinline__ void store() const {
#pragma unroll
    for (int k = 0; k < U; ++k) store16(reinterpret_cast<u32x4 *>(dp[k]), v[k]);
  }
};

template <int U, bool CALM>
__global__ void __launch_bounds__(kThreads) k_copy_link(const Desc *__restrict__ descs,
                                                        const int64_t *__restrict__ prefix, int d0, int d1, char *b0,
                                                        char *b1, char *b2, const int32_t *__restrict__ live,
                                                        const int32_t *calm) {
  const int64_t T1 = prefix[d1];
  int64_t t = prefix[d0] + tile_of_block();
  if (t >= T1) return;
  int d = find_desc(prefix, d0, d1, t);
  Calm<CALM> one(calm);
  LinkTile<U> x, y;
  x.load(descs[d], t - prefix[d], b0, b1, b2, live);
  for (;;) {
    t += gridDim.x;
    if (t >= T1) return x.store();
    while (prefix[d + 1] <= t) ++d;  // a workgroup's tiles come in order
    if (one.poll()) {
      x.store();
      x.load(descs[d], t - prefix[d], b0, b1, b2, live);
      continue;
    }
    y.load(descs[d], t - prefix[d], b0, b1, b2, live);
    x.store();
    t += gridDim.x;
    if (t >= T1) return y.store();
    while (prefix[d + 1] <= t) ++d;
    x.load(descs[d], t - prefix[d], b0, b1, b2, live);
    y.store();
  }
}

// Contiguous bytes of the pinned inflow buffer into a landing-ring slot, at
// once: it needs no descriptor, so it does not wait for k_prepare.  Two tiles
// of a workgroup in flight, as in k_copy_link, on a grid as narrow.
struct LinearTile {
  u32x4 v[kUnroll];
  uint64_t at;

  __device__ __forceinline__ void load(const u32x4 *src, uint64_t tile, uint64_t n) {
    at = tile * kTileChunks + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const uint64_t i = at + uint64_t(k) * kThreads;
      v[k] = load16(src + (i < n ? i : n - 1));
    }
  }
  // lanes past the end store the last chunk once more
  __device__ __forceinline__ void store(u32x4 *dst, uint64_t n) const {
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const uint64_t i = at + uint64_t(k) * kThreads;
      store16(dst + (i < n ? i : n - 1), v[k]);
    }
  }
};

__global__ void __launch_bounds__(kThreads) k_copy_linear(const u32x4 *src, u32x4 *dst, uint64_t n) {
  const uint64_t T = (n + kTileChunks - 1) / kTileChunks;
  uint64_t t = blockIdx.x;
  if (t >= T) return;
  LinearTile x, y;
  x.load(src, t, n);
  for (;;) {
    t += gridDim.x;
    if (t >= T) return x.store(dst, n);
    y.load(src, t, n);
    x.store(dst, n);
    t += gridDim.x;
    if (t >= T) return y.store(dst, n);
    x.load(src, t, n);
    y.store(dst, n);
  }
}

}  // namespace atp
