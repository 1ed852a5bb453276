// desc.h — copy descriptors shared by the host planner and the gfx950
// kernels of the reshard library.
//
// A descriptor is one copy family (Sec. III-C: tasks on interval boundaries,
// lowered to bytes):
//   for every outer item o in [o_begin, o_end)
//     for every line t in [0, rows)
//       copy `run` bytes
//         from src_base + src_off + idx_src(o) * src_ostride + t * src_pitch
//         to   dst_base + dst_off + idx_dst(o) * dst_ostride + t * dst_pitch
// where idx(o) = o - o_begin on a direct side and live[o] (a physical KV
// block id from the compacted block table) on an indirect side.  Weight
// tensors use outer items = rows of the matrix; KV uses outer items = live
// blocks and lines = tokens (token-major) or one line per block.
#pragma once
#include <stdint.h>

namespace atp {

// base-pointer slots a descriptor reads from / writes to
enum : uint32_t { BUF_IN = 0, BUF_OUT = 1, BUF_STAGE = 2 };

enum : uint32_t {
  DF_SRC_SHIFT = 0,       // 2 bits: source buffer slot
  DF_DST_SHIFT = 2,       // 2 bits: destination buffer slot
  DF_SRC_IND = 1u << 4,   // source index through the live-block list
  DF_DST_IND = 1u << 5,   // destination index through the live-block list
  DF_BLOCKRANGE = 1u << 6,// [o_begin, o_end) are block ids; the prepare
                          // kernel rewrites them as live-list positions
  DF_ALIGNED = 1u << 7,   // every offset, pitch, stride and run is a
                          // multiple of 16: the 16-byte vector kernel
  DF_WIDE = 1u << 8,      // aligned, tiled kWideUnroll chunks per thread
  DF_SRC_GRID = 1u << 9,  // not aligned: chunks start at 16-byte boundaries
                          // of the source, not of the destination
};

// Launch shape of the vector kernel: 256 threads, ATP_UNROLL independent
// 16-byte chunks per thread per tile; one workgroup per tile.
#ifndef ATP_UNROLL
#define ATP_UNROLL 2
#endif
#ifndef ATP_NT_LOAD
#define ATP_NT_LOAD 1
#endif
#ifndef ATP_NT_STORE
#define ATP_NT_STORE 1
#endif
#ifndef ATP_XCD_MAP
#define ATP_XCD_MAP 1
#endif
constexpr int kThreads = 256;
constexpr int kUnroll = ATP_UNROLL;
constexpr int64_t kTileChunks = kThreads * kUnroll;
// Short aligned KV lines (a head of one block, 4 KiB or less) take tiles
// twice as wide, which keeps more bytes in flight per thread: the largest KV
// level of the 80-layer TP 8->7 reshard ran 5 % faster so, while the
// weights' long lines ran slower.
constexpr int kWideUnroll = 2 * ATP_UNROLL;
constexpr int64_t kWideTileChunks = kThreads * kWideUnroll;
constexpr uint64_t kWideMaxRun = 4096;
// 16-byte chunks per tile of a vector-kernel descriptor
constexpr int64_t tile_chunks(uint32_t flags) { return (flags & DF_WIDE) ? kWideTileChunks : kTileChunks; }
// Chunks per line of a descriptor.  A line that is not aligned is cut at the
// 16-byte boundaries of one side (DF_SRC_GRID), its first and last chunk
// overlapping their neighbours: at most ceil((run + 15) / 16) chunks,
// wherever the line starts.  A run shorter than one chunk is one chunk,
// copied byte by byte.
constexpr uint32_t line_chunks(uint64_t run, uint32_t flags) {
  return uint32_t((flags & DF_ALIGNED) ? run >> 4 : run < 16 ? 1 : (run + 30) >> 4);
}

// Bytes of a flag per block id, in whole groups of 64; the live-block list has
// room for four times as many.
constexpr int64_t flag_room(int64_t n_blocks) { return (n_blocks + 63) / 64 * 64; }

struct alignas(16) Desc {
  uint64_t src_off, dst_off;
  uint64_t src_pitch, dst_pitch;
  uint64_t src_ostride, dst_ostride;
  int64_t o_begin, o_end;
  uint32_t run, rows;
  uint32_t flags;
  uint32_t cpl;         // chunks per line (line_chunks)
  // exact division by a host-known divisor d >= 2: q = umulhi64(n, m) with
  // m = ceil(2^64 / d), for n * d < 2^64; m = 0 means d == 1
  uint64_t magic_line;  // divisor: cpl
  uint64_t magic_rows;  // divisor: rows
};

static_assert(sizeof(Desc) == 96, "descriptor layout");

}  // namespace atp
