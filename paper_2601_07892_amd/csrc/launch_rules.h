// Rules by which the host picks a launch's shape from its sizes, and by which
// workgroups find their part of it: plain C++ (no HIP), so that they can be
// checked on the CPU.
#pragma once

#include <cstdint>

namespace sherry {

// Activation quantization: inputs of kStreamBytes and more are read past the
// caches (non-temporal).  Usually the operation before has just written the
// input.  Time with streaming against without, after a kernel that wrote x from
// one tensor, from two, and in place, and with x evicted (rows of 2048 .. 14336
// values): 12 MB +1%, +5%, +6%, -17%; 20 MB +2%, 0%, +14%, +2%; 32 MB -1%, -7%, +14%,
// -11%; 64 MB -5%, -8%, -3%, -4% (13.9 -> 12.9 us at 1953 x 8192); 96 MB -6%,
// -20%, -8%, -20%; 160 MB -23%, -26%, -10%, -8% (33.7 -> 25.4 us at 4882 x 8192).
constexpr int64_t kStreamBytes = int64_t(64) << 20;
constexpr bool quant_streams(int64_t rows, int64_t k) { return 4 * rows * k >= kStreamBytes; }

// Threads per row and float4 pieces per thread (0: two passes over the row) of
// the quantization of `rows` rows of up to k values.  512 threads past 8192
// values (1000 x 30000 51.7 -> 25 us, 64 x 14336 6.1 -> 4.7), except where the
// launch, one row per workgroup, would not fit the 2^32 - 1 threads of a grid.
struct QuantShape {
  int threads, pieces;
};
constexpr QuantShape quant_shape(int64_t rows, int64_t k) {
  if (k <= 8192) return {256, k <= 2048 ? 2 : k <= 4096 ? 4 : 8};
  if (rows * 512 > int64_t(UINT32_MAX)) return {256, k <= 16384 ? 16 : 0};
  return {512, k <= 16384 ? 8 : k <= 32768 ? 16 : 0};
}

}  // namespace sherry
