// Lane-interleaved units on the device: rewrites tiled units (as the host
// packer or sherry_ternarize_pack writes them) in the lane-interleaved
// layout that the matrix-core products read (defined in sherry.h).
#include "sherry_internal.h"

namespace sherry {
namespace {

// One wave per unit, four units per workgroup: the unit's rows go into LDS (one
// 16-byte and one 4-byte load per lane), then lane l = 16b + t gathers its 32
// codes and writes its own container.  Codes 4(2g + p) + c, c = 0..3, of the
// container are blocks 16p + 4b + c of row 16g + t: four codes side by side in
// both layouts, so a lane moves eight 20-bit fields, not 32 codes (bound by
// the launch and one trip to memory and back; with one wave per workgroup and
// code by code, the 7168 units of 4096 x 14336 took 10.4 us, now 5.4).
constexpr int kIlWaves = 4;

__global__ __launch_bounds__(64 * kIlWaves) void interleave_kernel(const uint8_t* __restrict__ tiled,
                                                                   uint8_t* __restrict__ il,
                                                                   int units) {
  __shared__ __attribute__((aligned(16))) uint32_t u32[kIlWaves][kUnitBytes / 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t unit = static_cast<int64_t>(blockIdx.x) * kIlWaves + wave;
  const size_t base = static_cast<size_t>(unit) * kUnitBytes;
  const bool live = unit < units;
  uint32_t* u = u32[wave];
  if (live) {
    reinterpret_cast<u32x4*>(u)[lane] = reinterpret_cast<const u32x4*>(tiled + base)[lane];
    u[kHeadBytes / 4 + lane] = reinterpret_cast<const uint32_t*>(tiled + base + kHeadBytes)[lane];
  }
  __syncthreads();
  if (!live) return;
  const int b = lane >> 4, t = lane & 15;
  uint32_t f[8];  // field 2g + p: row 16g + t, stream bits 20(4p + b) .. + 19
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int row = 16 * (j >> 1) + t;
    const int sp = 20 * (4 * (j & 1) + b), w = sp >> 5, s = sp & 31;
    // dwords 0-3 of a row are its head at 16*row, dword 4 the tail at 1024 +
    // 4*row; a field in dword 4 ends there (w + 1 = 5 is not part of it)
    auto word = [&](int q) { return u[q < 4 ? 4 * row + q : kHeadBytes / 4 + row]; };
    const uint64_t pair =
        static_cast<uint64_t>(word(w)) | static_cast<uint64_t>(word(w < 4 ? w + 1 : 4)) << 32;
    f[j] = static_cast<uint32_t>(pair >> s) & 0xfffffu;
  }
  // fields 20 bits apart, in five dwords
  const u32x4 head = {f[0] | f[1] << 20, f[1] >> 12 | f[2] << 8 | f[3] << 28,
                      f[3] >> 4 | f[4] << 16, f[4] >> 16 | f[5] << 4 | f[6] << 24};
  reinterpret_cast<u32x4*>(il + base)[lane] = head;
  reinterpret_cast<uint32_t*>(il + base + kHeadBytes)[lane] = f[6] >> 8 | f[7] << 12;
}

}  // namespace
}  // namespace sherry

using namespace sherry;

extern "C" int sherry_interleave(const uint8_t* tiled, uint8_t* il, int64_t n, int64_t k,
                                 void* stream) {
  if (!tiled || !il) return SHERRY_E_INVALID;
  if (sherry_packed_bytes(n, k) == 0) return SHERRY_E_SHAPE;
  if (tiled == il) return SHERRY_E_INVALID;
  if ((reinterpret_cast<uintptr_t>(tiled) & 15) || (reinterpret_cast<uintptr_t>(il) & 15))
    return SHERRY_E_ALIGN;
  const int64_t units = ceil_div(n, kTileRows) * ceil_div(k, kTileK);
  if (units > INT32_MAX) return SHERRY_E_SHAPE;
  return launch(interleave_kernel, dim3(static_cast<unsigned>(ceil_div(units, kIlWaves))), dim3(64 * kIlWaves),
                0, static_cast<hipStream_t>(stream), tiled, il, static_cast<int>(units));
}
