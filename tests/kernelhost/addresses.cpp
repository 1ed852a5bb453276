// Prints the addresses the copy kernels compute for one tile of one copy
// family, from csrc/kernels.h compiled for the CPU (tests/test_kernel_addresses.py).
// argv: narrow | wide | any, then src_off dst_off src_pitch dst_pitch
// src_ostride dst_ostride items run rows flags tile.  One line per 16-byte
// chunk: source offset, destination offset.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "kernels.h"

using namespace atp;

static uint64_t magic_of(uint64_t d) {
  return d <= 1 ? 0 : uint64_t(((((unsigned __int128)1) << 64) + d - 1) / d);
}

template <int U, bool ANY>
static void tile(const Desc &x, uint64_t tile) {
  const uint64_t per = uint64_t(kThreads) * U;
  const uint64_t total = uint64_t(x.o_end - x.o_begin) * x.rows * x.cpl;
  const uint64_t c0 = tile * per, cl = (c0 + per < total ? c0 + per : total) - 1;
  for (int t = 0; t < kThreads; ++t) {
    threadIdx.x = uint32_t(t);
    const char *sp[U];
    char *dp[U];
    tile_addr<U, ANY>(x, c0, cl, nullptr, nullptr, nullptr, nullptr, sp, dp);
    for (int k = 0; k < U; ++k)
      if (c0 + t + uint64_t(k) * kThreads <= cl)
        printf("%llu %llu\n", (unsigned long long)uintptr_t(sp[k]), (unsigned long long)uintptr_t(dp[k]));
  }
}

int main(int argc, char **argv) {
  if (argc != 13) return 2;
  auto n = [&](int i) { return strtoull(argv[i], nullptr, 0); };
  Desc x{};
  x.src_off = n(2), x.dst_off = n(3), x.src_pitch = n(4), x.dst_pitch = n(5);
  x.src_ostride = n(6), x.dst_ostride = n(7), x.o_end = int64_t(n(8));
  x.run = uint32_t(n(9)), x.rows = uint32_t(n(10)), x.flags = uint32_t(n(11));
  x.flags |= (BUF_IN << DF_SRC_SHIFT) | (BUF_OUT << DF_DST_SHIFT);
  x.cpl = line_chunks(n(9), x.flags);
  x.magic_line = magic_of(x.cpl);
  x.magic_rows = magic_of(x.rows);
  if (!strcmp(argv[1], "narrow")) tile<kUnroll, false>(x, n(12));
  else if (!strcmp(argv[1], "wide")) tile<kWideUnroll, false>(x, n(12));
  else tile<kUnroll, true>(x, n(12));
  return 0;
}
