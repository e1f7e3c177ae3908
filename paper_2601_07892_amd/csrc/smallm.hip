// Products of up to 16 tokens on the matrix cores, with the weights in the
// registers they are loaded into (Eq. 2; grouped launches of small-M decode
// steps).
//
// Work mapping.  A workgroup is 4 waves; wave w owns 64-row tile 4g + w and
// the whole K of it (lane i = row i, as in the decode GEMV), streaming its
// units through a register ring and decoding each code through the 32-entry
// LDS table.  The 4 waves walk K in lockstep windows of 4 units: the
// activations of a window (16 token rows x 512 K values, int8) are staged in
// LDS by the whole workgroup, double-buffered, one window ahead.  (Four
// waves per workgroup rather than eight: twice the workgroups to balance the
// chip and half the waves held at each window barrier; 4% faster on a 3B
// step of 16 tokens.)
//
// What bounds it is the latency of each unit's chain (load, 32 table reads,
// MFMAs): at 3.6 waves per SIMD a 3B step of 16 tokens keeps LDS 57%, VALU
// 53% and the matrix cores 21% busy.  Windows of 4 rather than 8 units and
// table reads in batches of 8 codes on lane-interleaved units (72 registers)
// let six of their waves fit a SIMD: LLaMA-3.2-3B step at 16 tokens 118.4 ->
// 116.2 us, at 5 tokens 108 -> 101, on tiled units with per-group scales 171
// -> 166.
//
// Launches of few blocks (one layer's products) leave most of the chip idle
// while each wave walks its whole row: up to kSmFoldBlocks prepared blocks are
// run by four workgroups each, one tile per workgroup and a quarter of its K
// per wave (SmCfg<4>), the partial sums added through LDS.  Quantize and four
// launches of a LLaMA-3.2-3B layer, graph-launched: lane-interleaved at 12
// tokens 81 -> 47 us, tiled at 16 61 -> 46, with per-group scales 67 -> 54;
// an 8B layer at 6 tokens 110 -> 58.
//
// Every global load is issued on every path (past the end of a tile or of k
// it reads zeros through an empty or bounded resource), so the compiler's
// waits count exact numbers of loads instead of draining the queue; a
// drained queue before each unit cost a quarter of the throughput.
//
// Operands.  v_mfma_i32_32x32x32_i8 takes B[k][j] from lane j + 32h (k half
// h) and A[i][k] from lane i + 32h.  The four looked-up words of a 4-code
// chunk are B as they stand: lanes 0-31 give k half 0 = rows 0-31 of the
// tile, lanes 32-63 give k half 1 = rows 32-63, both over the same 16
// activations.  A row m (k half 0, lane m) and A row 16 + m (k half 1, lane
// 48 + m) carry token m's 16 activations of the chunk; every other lane's A
// stays zero.  So D[m][t] = x_m . w(row t) and D[16 + m][t] = x_m . w(row
// 32 + t): one MFMA per chunk serves 64 rows and 16 tokens, with no lane
// exchange of the weights.
//
// On lane-interleaved units (kIL) each 4-code chunk slot of a lane is the B
// operand of a v_mfma_i32_16x16x64_i8 over 16 rows and 64 weights instead;
// lane 16b + m reads token m's chunks b and 4 + b of the unit from the
// stage, an A operand that serves all four row groups (two 16-byte LDS reads
// per unit and lane), and D[m][t] of row group g lands in lane 16(m/4) + t.
#include "sherry_internal.h"

namespace sherry {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kSmWaves = 4;
constexpr int kSmThreads = 64 * kSmWaves;
constexpr int kSmTok = 16;                      // token rows staged
constexpr int kSmRing = 4;                      // units per wave in the register ring

// Staging geometry with each tile's K in S parts: a window is UPW units of
// every part (4 units of the whole row; 16 units, 4 of each part, with S = 4).
template <int S_>
struct SmCfg {
  static constexpr int S = S_;
  static constexpr int UPW = 4;                     // units per part and window
  static constexpr int kPart = UPW * kTileK;        // K values of a part's window
  static constexpr int kWinK = S * kPart;           // K values staged per token
  static constexpr int kRowStride = kWinK + 16;     // staged token row, padded
  static constexpr int kStageBytes = kSmTok * kRowStride;
  static constexpr int kWinPieces = kSmTok * kWinK / 16 / kSmThreads;  // per thread
  static_assert(UPW % kSmRing == 0, "ring slots repeat in every window");
  static_assert(S == 1 || kSmThreads * 16 * 4 <= 2 * kStageBytes, "the partial sums fit the stages");
};

// Table lookups of codes j0 .. j0 + 15 of a unit row (lane i = row i):
// wv[j] = the int8x4 weights of code j0 + j.
template <int j0, int... js>
__device__ __forceinline__ void sm_lookup(const uint32_t (&d)[5], const uint32_t* lut,
                                          uint32_t (&wv)[16], std::integer_sequence<int, js...>) {
  ((wv[js] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lut) +
                                                code_x4<j0 + js>(d))),
   ...);
}

// Row group g of a lane-interleaved unit: its two chunk slots.
template <int j0, int... js>
__device__ __forceinline__ void sm_lookup8(const uint32_t (&d)[5], const uint32_t* lut,
                                           uint32_t (&wv)[8], std::integer_sequence<int, js...>) {
  ((wv[js] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lut) +
                                                code_x4<j0 + js>(d))),
   ...);
}
template <int g>
__device__ __forceinline__ void sm_il_group(const uint32_t (&d)[5], const uint32_t* lut,
                                            const v4i (&xa)[2], v4i (&acc)[4]) {
  __builtin_amdgcn_sched_barrier(0);
  uint32_t wv[8];
  sm_lookup8<8 * g>(d, lut, wv, std::make_integer_sequence<int, 8>{});
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const v4i b = {static_cast<int>(wv[4 * p]), static_cast<int>(wv[4 * p + 1]),
                   static_cast<int>(wv[4 * p + 2]), static_cast<int>(wv[4 * p + 3])};
    acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[p], b, acc[g], 0, 0, 0);
  }
}

// Stage layout: token row t at t * kRowStride, its 16-byte piece p at 16p within
// it (part p / (kPart / 16), K offset 16p in that part's window); the 16-byte
// pad per row puts the lanes that read one piece of consecutive rows on
// different 4-bank groups.
//
// The window's activations for this thread: pieces i * kSmThreads + tid of the
// window, read through a resource over the m x k activations (rows past m read
// zeros).  Pieces are 16-byte loads when k % 16 == 0 (the activations are
// 16-byte aligned), else four word loads (k % 4 == 0).  A piece or word at or
// past its part's end or k is loaded from an offset outside the resource, so it
// reads zeros without touching memory and no load reaches into the next row;
// every load is issued on every path.
constexpr int kSmOutside = 0x40000000;  // past any m * k (m <= 16, k <= 2^18)

template <class G>
__device__ __forceinline__ void stage_load(u32x4 (&v)[G::kWinPieces], __amdgpu_buffer_rsrc_t rx,
                                           int k, int U, int w) {
  const bool wide = (k & 15) == 0;
#pragma unroll
  for (int i = 0; i < G::kWinPieces; ++i) {
    const int q = i * kSmThreads + static_cast<int>(threadIdx.x);
    const int t = q / (G::kWinK / 16), p = q % (G::kWinK / 16);
    const int part = p / (G::kPart / 16), o = 16 * (p % (G::kPart / 16)) + w * G::kPart;
    const int kk = part * U * kTileK + o;  // first K value of the piece
    const int end = G::S == 1 ? k : min(k, (part + 1) * U * kTileK);
    const int left = end - kk;             // K values of the part left from kk
    const int off = t * k + kk;
    if (wide) {
      v[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, left >= 16 ? off : kSmOutside, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rx, 4 * e < left ? off + 4 * e : kSmOutside,
                                                       0, 0);
    }
  }
}

template <class G>
__device__ __forceinline__ void stage_store(const u32x4 (&v)[G::kWinPieces], int8_t* st) {
#pragma unroll
  for (int i = 0; i < G::kWinPieces; ++i) {
    const int q = i * kSmThreads + static_cast<int>(threadIdx.x);
    const int t = q / (G::kWinK / 16), p = q % (G::kWinK / 16);
    *reinterpret_cast<u32x4*>(st + t * G::kRowStride + 16 * p) = v[i];
  }
}

// Barrier for LDS traffic only: outstanding global loads stay in flight.
__device__ __forceinline__ void sm_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct SmProblem {
  const uint8_t* w;
  const int8_t* x;
  const float* x_scale;
  float* y;
  int32_t* acc;
  int n, k, m;
  WScale ws;
  const float* gs;  // per-group scales [n][k/128], or nullptr
};

// One workgroup: tiles kSmWaves*g .. kSmWaves*g + kSmWaves - 1 of the
// problem (CFG::S == 1), or tile g, wave w the w-th part of its units
// (CFG::S == 4).  lds: the table (128 bytes), two stages, a zero row (the A
// operand of lanes that carry no token, read like a token row so that no
// lane branches) and the tokens' activation scales.
//
// kG: per-group scales (one per row and unit; k % 512 == 0 and p.gs 16-byte
// aligned, so that a lane reads four units' scales of its row at once).
// Each unit's MFMAs then run as one chain from zero into c[u & 1], and the
// unit is scaled one unit later (its chain has completed by then) into fp32
// accumulators: element e < 8 of a lane belongs to row l % 32 of the tile,
// e >= 8 to row l % 32 + 32, whose scales a lane-half swap of the loaded
// ones provides.
//
// kIL: lane-interleaved weights (sherry_pack_il; not with kG).  Lane 16b + t
// holds, as chunk slot (g, p), row 16g + t's weights of chunk 4p + b, the B
// operand of one v_mfma_i32_16x16x64_i8 over 16 rows and 64 weights; its A
// operand, token m = lane % 16's chunks b and 4 + b of the unit, is read once
// per unit and serves the four row groups.  D[m][t] lands in lane
// 16(m/4) + t, element m % 4 of accumulator g.
template <class CFG, bool kG, bool kIL = false>
__device__ __forceinline__ void sm_block(const SmProblem& p, int g, uint32_t* lut,
                                         int8_t* stages, int8_t* zrow, float* xs) {
  constexpr int S = CFG::S, UPW = CFG::UPW;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = (p.k + kTileK - 1) / kTileK;
  const int R = (p.n + kTileRows - 1) / kTileRows;
  const int r = S == 1 ? g * kSmWaves + wave : g;
  const bool live = r < R;
  // this wave's units of the tile: all, or part sp of S (whole chunks of four
  // with per-group scales, which are loaded for four units at once)
  const int sp = S == 1 ? 0 : wave;
  const int U = S == 1 ? C : (kG ? ((C + S - 1) / S + 3) & ~3 : (C + S - 1) / S);
  const int u0 = sp * U < C ? sp * U : C;
  const int Cn = live ? (u0 + U < C ? U : C - u0) : 0;  // (dead waves: none)
  const UnitRun tile{p.w + (int64_t(live ? r : 0) * C + (live ? u0 : 0)) * kUnitBytes, Cn};
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.x), 0, p.m * p.k, kBufferWord3);
  const int nwin = (U + UPW - 1) / UPW;

  // token of this lane's A operand (lanes 0-15 and 48-63; staged rows past m
  // are zero), or none
  const int tok = lane < 16 ? lane : (lane >= 48 ? lane - 48 : -1);

  // the scales and window 0 first, then the ring: the stage store waits for
  // the former only
  float xsv = 0.0f;
  if (tid < p.m) xsv = as_global(p.x_scale)[tid];
  u32x4 sv[CFG::kWinPieces];
  stage_load<CFG>(sv, rx, p.k, U, 0);
  __builtin_amdgcn_sched_barrier(0);
  uint32_t ring[kSmRing][5];
#pragma unroll
  for (int u = 0; u < kSmRing; ++u) {
    load_unit(ring[u], tile, u, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (tid < 32) lut[tid] = decode_word(tid);
  if (tid < CFG::kPart / 16) reinterpret_cast<u32x4*>(zrow)[tid] = u32x4{0u, 0u, 0u, 0u};
  if (tid < kSmTok) xs[tid] = xsv;
  stage_store<CFG>(sv, stages);
  sm_lds_barrier();  // window 0, the table, the zero row and the scales are ready

  // per-group scales: lane l reads row l of the tile, four units per load,
  // two chunks ahead; slo / shi hold the current chunk's scales of rows
  // l % 32 and l % 32 + 32, plo / phi the previous chunk's last ones
  const int grows =
      kG && live ? (p.n - r * kTileRows < kTileRows ? p.n - r * kTileRows : kTileRows) : 0;
  const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.gs) + int64_t(live ? r : 0) * kTileRows * C, 0, grows * C * 4,
      kBufferWord3);
  u32x4 gqa{}, gqb{};
  float slo[4] = {}, shi[4] = {}, plo = 0.0f, phi = 0.0f;
  float accf[16] = {};
  if constexpr (kG) {
    // (units past the part multiply nothing: their sums are not scaled)
    gqa = __builtin_amdgcn_raw_buffer_load_b128(gr, 4 * (lane * C + u0), 0, 0);
    gqb = __builtin_amdgcn_raw_buffer_load_b128(gr, 4 * (lane * C + u0 + 4), 0, 0);
  }

  static_assert(!(kG && kIL), "per-group scales: tiled units only");
  v16i c[2] = {v16i{}, v16i{}};
  v4i acc4[4] = {};  // kIL accumulators, one per row group
  for (int w = 0; w < nwin; ++w) {
    // the next window's activations are in flight during this one
    stage_load<CFG>(sv, rx, p.k, U, w + 1);
    // this lane's A row of the window
    const int8_t* arow =
        tok >= 0 ? stages + (w & 1) * CFG::kStageBytes + tok * CFG::kRowStride + sp * CFG::kPart : zrow;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
      const int j = w * UPW + u;  // unit of the part
      if constexpr (kG) {
        if (u % 4 == 0) {  // a new chunk of four units (issued on every path)
          plo = slo[3];
          phi = shi[3];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t own = gqa[e];
            const auto sw = __builtin_amdgcn_permlane32_swap(own, own, false, false);
            slo[e] = __uint_as_float(sw[0]);
            shi[e] = __uint_as_float(sw[1]);
          }
          gqa = gqb;
          gqb = __builtin_amdgcn_raw_buffer_load_b128(gr, 4 * (lane * C + u0 + j + 8), 0, 0);
        }
      }
      if (kIL && j < Cn) {
        // the unit's activation operands: token lane % 16 (rows past m are
        // zero in the stage), chunks b and 4 + b, b = lane / 16
        const int8_t* ar = stages + (w & 1) * CFG::kStageBytes + (lane & 15) * CFG::kRowStride +
                           sp * CFG::kPart + 16 * (8 * u + (lane >> 4));
        const v4i xa[2] = {*reinterpret_cast<const v4i*>(ar),
                           *reinterpret_cast<const v4i*>(ar + 64)};
        sm_il_group<0>(ring[u % kSmRing], lut, xa, acc4);
        sm_il_group<1>(ring[u % kSmRing], lut, xa, acc4);
        sm_il_group<2>(ring[u % kSmRing], lut, xa, acc4);
        sm_il_group<3>(ring[u % kSmRing], lut, xa, acc4);
      } else if (j < Cn) {
        // codes 16h .. 16h + 15: 16 table reads in flight, then 4 chunks
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          __builtin_amdgcn_sched_barrier(0);
          uint32_t wv[16];
          if (h == 0) sm_lookup<0>(ring[u % kSmRing], lut, wv, std::make_integer_sequence<int, 16>{});
          else sm_lookup<16>(ring[u % kSmRing], lut, wv, std::make_integer_sequence<int, 16>{});
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const v4i a = *reinterpret_cast<const v4i*>(arow + 16 * (8 * u + 4 * h + q));
            const v4i b = {static_cast<int>(wv[4 * q]), static_cast<int>(wv[4 * q + 1]),
                           static_cast<int>(wv[4 * q + 2]), static_cast<int>(wv[4 * q + 3])};
            if constexpr (kG) {
              const v16i cin = (h == 0 && q == 0) ? v16i{} : c[u & 1];
              c[u & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, cin, 0, 0, 0);
            } else {
              c[q & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c[q & 1], 0, 0, 0);
            }
          }
        }
      }
      if constexpr (kG) {
        if (j >= 1 && j <= Cn) {  // unit j - 1, in c[(u + 1) & 1]
          const float sl = (u % 4 == 0) ? plo : slo[(u + 3) % 4];
          const float sh = (u % 4 == 0) ? phi : shi[(u + 3) % 4];
#pragma unroll
          for (int e = 0; e < 16; ++e)
            accf[e] = __builtin_fmaf(static_cast<float>(c[(u + 1) & 1][e]), e < 8 ? sl : sh,
                                     accf[e]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      load_unit(ring[u % kSmRing], tile, j + kSmRing, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
    stage_store<CFG>(sv, stages + ((w + 1) & 1) * CFG::kStageBytes);
    sm_lds_barrier();
  }

  if constexpr (kG) {
    // the last unit, if the walk ended on it (in c[1]: UPW is even)
    if (Cn > 0 && Cn == nwin * UPW) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        accf[e] = __builtin_fmaf(static_cast<float>(c[1][e]), e < 8 ? slo[3] : shi[3], accf[e]);
    }
  }

  // the sums of this lane, element e (fp32 bits with kG): token i % 16 of tile
  // row (l % 32) + 32 (i / 16), i = 8(e/4) + 4(l/32) + e%4; kIL: token
  // 4(l / 16) + e%4 of tile row 16 (e/4) + l % 16
  auto sum = [&](int e) -> int32_t {
    if constexpr (kG) return __float_as_int(accf[e]);
    else if constexpr (kIL) return acc4[e >> 2][e & 3];
    else return c[0][e] + c[1][e];
  };
  constexpr int EN = 16 / S;  // elements this wave finishes: e0 .. e0 + EN - 1
  const int e0 = S == 1 ? 0 : EN * wave;
  int32_t v[EN];
  if constexpr (S == 1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = sum(e);
  } else {
    // the parts' sums through the stages (free after the last barrier), added
    // in order
    int32_t* red = reinterpret_cast<int32_t*>(stages);
#pragma unroll
    for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = sum(e);
    sm_lds_barrier();
#pragma unroll
    for (int e = 0; e < EN; ++e) {
      const int32_t* rp = red + (e0 + e) * 64 + lane;
      if constexpr (kG) {
        float f = __int_as_float(rp[0]);
#pragma unroll
        for (int q = 1; q < S; ++q) f += __int_as_float(rp[q * 16 * 64]);
        v[e] = __float_as_int(f);
      } else {
        v[e] = rp[0];
#pragma unroll
        for (int q = 1; q < S; ++q) v[e] += rp[q * 16 * 64];
      }
    }
  }

  // epilogue: the scales are fetched once, then every element is stored
  if (!live) return;
  // tile row and token of element e
  auto row_of = [&](int e) {
    return kIL ? 16 * (e >> 2) + (lane & 15) : (lane & 31) + 32 * (e >> 3);
  };
  auto tok_of = [&](int e) {
    return kIL ? 4 * (lane >> 4) + (e & 3) : (8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) & 15;
  };
  // the weight scales of this lane's rows (S = 4: the elements of a wave are
  // of one row)
  constexpr int NR = S > 1 ? 1 : kIL ? 4 : 2;
  float wsr[NR] = {};
  if constexpr (!kG) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int64_t row = int64_t(r) * kTileRows + row_of(e0 + i * (16 / (kIL ? 4 : 2)));
      wsr[i] = p.ws.at(row < p.n ? row : p.n - 1);
    }
  }
  // one wait for every load of the wave (the scales; the ring is drained), so
  // that no store below waits for the stores before it
  __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
  for (int e = 0; e < EN; ++e) {
    const int el = e0 + e;
    const int t = tok_of(el);
    const int64_t row = int64_t(r) * kTileRows + row_of(el);
    if (t < p.m && row < p.n) {
      const int64_t at = int64_t(t) * p.n + row;
      if constexpr (kG) {
        as_global_mut(p.y)[at] = __int_as_float(v[e]) * xs[t];
      } else {
        const float sc = xs[t] * wsr[S > 1 ? 0 : kIL ? e >> 2 : e >> 3];
        as_global_mut(p.y)[at] = static_cast<float>(v[e]) * sc;
        if (p.acc) as_global_mut(p.acc)[at] = v[e];
      }
    }
  }
}

// kGroups: some descriptor carries per-group scales (a kernel of its own,
// so that the other keeps its registers).  A prepared block is four tiles, one
// per wave; with S = 4 it is run by four workgroups, each of one tile with a
// quarter of its K per wave, or, where the rows are short, by one of them as with
// S = 1.
template <class CFG, bool kGroups, bool kIL>
constexpr int kSmPerSimd = CFG::S > 1 ? 2 : kIL ? 6 : kGroups ? 3 : 4;

template <class CFG, bool kGroups, bool kIL>
__global__ __launch_bounds__(kSmThreads) __attribute__((amdgpu_waves_per_eu((kSmPerSimd<CFG, kGroups, kIL>)))) void
smallm_batched_kernel(
    const sherry_gemm_desc* __restrict__ descs, int count) {
  __shared__ uint32_t lut[32];
  __shared__ __attribute__((aligned(16))) int8_t stages[2 * CFG::kStageBytes];
  __shared__ __attribute__((aligned(16))) int8_t zrow[CFG::kPart];
  __shared__ float xs[kSmTok];
  const int32_t blk = static_cast<int32_t>(blockIdx.x) / CFG::S;
  const int lo = find_block_desc(descs, count, blk);
  if (lo < 0) return;
  const sherry_gemm_desc& d = descs[lo];
  const SmProblem p{d.w, d.x, d.x_scale, d.y, d.acc, d.n, d.k, d.m,
                    WScale{d.w_scales, d.w_scale}, d.w_group_scales};
  if constexpr (CFG::S > 1) {
    const bool grp = kGroups && p.gs;
    if (!sm_splits((p.k + kTileK - 1) / kTileK, gridDim.x / CFG::S, grp)) {
      if (static_cast<int>(blockIdx.x) % CFG::S != sm_whole_sub(blk)) return;
      const int g = blk - d.block_begin;
      if (grp) sm_block<SmCfg<1>, kGroups>(p, g, lut, stages, zrow, xs);
      else sm_block<SmCfg<1>, false, kIL>(p, g, lut, stages, zrow, xs);
      return;
    }
  }
  // S = 4: tile 4 (blk - begin) + blockIdx % 4
  const int g = static_cast<int>(blockIdx.x) - d.block_begin * CFG::S;
  if (CFG::S > 1 && g * kTileRows >= p.n) return;
  if (kGroups && p.gs) sm_block<CFG, kGroups>(p, g, lut, stages, zrow, xs);
  else sm_block<CFG, false, kIL>(p, g, lut, stages, zrow, xs);
}

template <bool kGroups, bool kIL>
int launch_smallm(const sherry_gemm_desc* descs, int count, int64_t total_blocks, hipStream_t s) {
  if (total_blocks <= kSmFoldBlocks)
    return launch(smallm_batched_kernel<SmCfg<4>, kGroups, kIL>,
                  dim3(static_cast<unsigned>(total_blocks * 4)), dim3(kSmThreads), 0, s, descs, count);
  return launch(smallm_batched_kernel<SmCfg<1>, kGroups, kIL>,
                dim3(static_cast<unsigned>(total_blocks)), dim3(kSmThreads), 0, s, descs, count);
}

}  // namespace

int launch_smallm_il_batched(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                             hipStream_t s) {
  return launch_smallm<false, true>(descs, count, total_blocks, s);
}

int64_t smallm_blocks(int64_t n) { return ceil_div(ceil_div(n, kTileRows), kSmWaves); }

int launch_smallm_batched(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                          bool groups, hipStream_t s) {
  return groups ? launch_smallm<true, false>(descs, count, total_blocks, s)
                : launch_smallm<false, false>(descs, count, total_blocks, s);
}

}  // namespace sherry
