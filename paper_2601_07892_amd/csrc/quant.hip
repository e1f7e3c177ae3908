// Per-token int8 activation quantization on the device.
//
// The paper keeps activations in BF16 (weights-only setting, Limitations) but
// its engine accumulates in integers (Appendix A, online phase).  The integer
// inputs are produced here: s = absmax/127, q = clamp(rint(x/s), -127, 127).
// One workgroup per token row: 256 threads for rows of up to 8192 values, 512
// for longer ones (quant_shape).  Rows up to 32768 values are read once into
// registers; longer rows are read twice (absmax, then quantize).
//
// What bounds it: launch and memory latency at decode sizes, HBM (or the
// Infinity Cache, where the kernel before left the row there) at prefill sizes.
// A thread's loads go out back to back (the row's end through the range of a
// buffer resource, not a branch per load), and quant4 takes about 6 VALU
// operations per value (15 before).  Inputs out of cache, against the branches and
// 15 operations: 2048 x 14336 31.5 -> 25.8 us, 8192 x 4096 32.6 -> 28.4, 2048 x 3072
// 8.6 -> 8.1, 64 x 14336 6.1 -> 4.5 (in cache), 1000 x 30000 51.6 -> 28.2.
#include <type_traits>

#include "sherry_internal.h"

namespace sherry {
namespace {

template <int T>
__device__ __forceinline__ float block_max(float amax, float* part) {
  amax = wave_max_f32(amax);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = amax;
  __syncthreads();
  amax = part[0];
#pragma unroll
  for (int i = 1; i < T / 64; ++i) amax = fmaxf(amax, part[i]);
  return amax;
}

// One row x[0..k) -> q, *scale, by the whole workgroup of T threads.  NV > 0:
// rows of up to 4 NV T values, read once into registers (NV float4 per
// thread) and quantized from there; loads and stores past the row read zeros
// and are dropped.  NV = 0: any row length, two passes over the row (the
// second from cache).  AUX: the loads' cache policy.
template <int T, int NV, int AUX>
__device__ __forceinline__ void quantize_row(const float* x, int64_t k, int8_t* q, float* scale,
                                             float* part) {
  const float4* xr = reinterpret_cast<const float4*>(x);
  uint32_t* qr = reinterpret_cast<uint32_t*>(q);
  if constexpr (NV > 0) {
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(x), 0, static_cast<int>(k) * 4, kBufferWord3);
    const __amdgpu_buffer_rsrc_t rq =
        __builtin_amdgcn_make_buffer_rsrc(q, 0, static_cast<int>(k), kBufferWord3);
    u32x4 raw[NV];
#pragma unroll
    for (int e = 0; e < NV; ++e)
      raw[e] = __builtin_amdgcn_raw_buffer_load_b128(
          rx, 16 * (static_cast<int>(threadIdx.x) + e * T), 0, AUX);
    __builtin_amdgcn_sched_barrier(0);
    float4 v[NV];
    float amax = 0.0f;
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      v[e] = make_float4(__uint_as_float(raw[e].x), __uint_as_float(raw[e].y),
                         __uint_as_float(raw[e].z), __uint_as_float(raw[e].w));
      amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[e].x), fabsf(v[e].y)),
                               fmaxf(fabsf(v[e].z), fabsf(v[e].w))));
    }
    amax = block_max<T>(amax, part);
    const float s = amax / 127.0f;
    const float rs = 1.0f / s;
    // a wave whose whole piece lies past the row skips it: rounding zeros for
    // nothing costs many short rows 10-20% (16384 x 256 13.8 -> 12.0 us, 10236 x
    // 104 9.8 -> 8.6)
    const int first = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x));
#pragma unroll
    for (int e = 0; e < NV; ++e)
      if (4 * (first + e * T) < static_cast<int>(k))
        __builtin_amdgcn_raw_buffer_store_b32(
            (amax == 0.0f) ? 0u : quant4(v[e], s, rs), rq,
            4 * (static_cast<int>(threadIdx.x) + e * T), 0, 0);
    if (threadIdx.x == 0) *scale = (amax == 0.0f) ? 0.0f : s;
  } else {
    const int64_t k4 = k >> 2;
    float amax = 0.0f;
    for (int64_t i = threadIdx.x; i < k4; i += T) {
      const float4 v = xr[i];
      amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
    amax = block_max<T>(amax, part);
    if (amax == 0.0f) {
      for (int64_t i = threadIdx.x; i < k4; i += T) qr[i] = 0u;
      if (threadIdx.x == 0) *scale = 0.0f;
      return;
    }
    const float s = amax / 127.0f;
    const float rs = 1.0f / s;
    for (int64_t i = threadIdx.x; i < k4; i += T) qr[i] = quant4(xr[i], s, rs);
    if (threadIdx.x == 0) *scale = s;
  }
}

template <int T, int NV, int AUX>
__global__ __launch_bounds__(T) void quantize_rows_kernel(const float* __restrict__ x, int64_t k,
                                                          int8_t* __restrict__ q,
                                                          float* __restrict__ x_scale) {
  __shared__ float part[T / 64];
  const int64_t row = blockIdx.x;
  quantize_row<T, NV, AUX>(x + row * k, k, q + row * k, x_scale + row, part);
}

// Every row of every matrix of a descriptor array, one workgroup per row.
template <int T, int NV>
__global__ __launch_bounds__(T) void quantize_batched_kernel(
    const sherry_quant_desc* __restrict__ descs, int count) {
  __shared__ float part[T / 64];
  const int32_t blk = static_cast<int32_t>(blockIdx.x);
  // last descriptor with row_begin <= blk (a prefix: row_begin increases)
  const int lane = threadIdx.x & 63;
  int lo = 0;
  for (int base = 0; base < count; base += 64) {
    const int i = base + lane;
    const bool ok = i < count && as_global(descs)[i].row_begin <= blk;
    const int len = __popcll(__ballot(ok));
    lo = base + len - 1;
    if (len < 64) break;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const sherry_quant_desc& d = descs[lo];
  const int64_t row = blk - d.row_begin, k = d.k;
  quantize_row<T, NV, 0>(d.x + row * k, k, d.q + row * k, d.x_scale + row, part);
}

// Calls f(T, NV) with the workgroup for `rows` rows of up to k values.
template <class F>
int with_row_shape(int64_t rows, int64_t k, F f) {
  using std::integral_constant;
  const QuantShape q = quant_shape(rows, k);
  if (q.threads == 256) {
    switch (q.pieces) {
      case 2: return f(integral_constant<int, 256>{}, integral_constant<int, 2>{});
      case 4: return f(integral_constant<int, 256>{}, integral_constant<int, 4>{});
      case 8: return f(integral_constant<int, 256>{}, integral_constant<int, 8>{});
      case 16: return f(integral_constant<int, 256>{}, integral_constant<int, 16>{});
      default: return f(integral_constant<int, 256>{}, integral_constant<int, 0>{});
    }
  }
  switch (q.pieces) {
    case 8: return f(integral_constant<int, 512>{}, integral_constant<int, 8>{});
    case 16: return f(integral_constant<int, 512>{}, integral_constant<int, 16>{});
    default: return f(integral_constant<int, 512>{}, integral_constant<int, 0>{});
  }
}

}  // namespace

int launch_quantize(const float* x, int64_t m, int64_t k, int8_t* q, float* x_scale,
                    hipStream_t s) {
  return with_row_shape(m, k, [&](auto t, auto nv) {
    constexpr int T = decltype(t)::value, NV = decltype(nv)::value;
    const dim3 grid(static_cast<unsigned>(m)), block(T);
    // (two passes over a row: the second reads what the first left in the caches)
    if constexpr (NV > 0) {
      if (quant_streams(m, k))
        return launch(quantize_rows_kernel<T, NV, kLoadStream>, grid, block, 0, s, x, k, q, x_scale);
    }
    return launch(quantize_rows_kernel<T, NV, 0>, grid, block, 0, s, x, k, q, x_scale);
  });
}

int launch_quantize_batched(const sherry_quant_desc* descs, int count, int64_t total_rows,
                            int64_t max_k, hipStream_t s) {
  return with_row_shape(total_rows, max_k, [&](auto t, auto nv) {
    constexpr int T = decltype(t)::value, NV = decltype(nv)::value;
    const dim3 grid(static_cast<unsigned>(total_rows)), block(T);
    // (the inputs' size is not known here, rows times the longest row only a
    // bound: never read past the caches)
    return launch(quantize_batched_kernel<T, NV>, grid, block, 0, s, descs, count);
  });
}

}  // namespace sherry
