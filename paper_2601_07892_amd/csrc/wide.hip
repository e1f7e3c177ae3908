// Register-decoded int8-MFMA product (Eq. 2): the lone products of five and more
// tokens (but for long ones of short rows, sherry_gemm_kernel_for), and the
// grouped launches of more than 16 (with per-group scales whose rows the window
// kernel does not take, of more than four).
//
// Work mapping.  A wave owns one 64-row tile (or one of S parts of its K) and
// 32 MT tokens; a workgroup is W waves, W / S tiles.  Per container (64 rows x
// 128 weights, lane i = row i) a wave decodes its 32 codes per lane through
// the 32-entry LDS table; v_permlane32_swap pairs rows i and i + 32, so that
// each 16-byte operand holds one 32-row half in the MFMA layout (lane l: row
// l % 32, k half l / 32), and v_mfma_i32_32x32x32_i8 accumulates
// C[token][row].  The activations of a container's 128 K values arrive in LDS
// by DMA loads (buffer_load ... lds), three containers ahead.
//
// What bounds it.  Table reads, fragment reads and DMA writes load the LDS for
// (32 x 2 + 4 MT x 8 + 16 MT / W) cycles per wave and container, the MFMAs the
// matrix core for 256 MT: with 64 tokens per wave the LDS is as busy as the
// matrix cores of its four SIMDs, with 128 it is at 87%.  So long products run
// 128-token workgroups of four waves (230 registers per lane: two workgroups
// per CU, independent of each other, so that one's start and end hide behind
// the other's stream).  A container is taken in four slices of 32 K values,
// and everything a slice does is independent of its own MFMAs: the fragments
// of the next slice, the lane swap of the next slice's words, the lookups of
// the next container's previous group.  A scheduling group then places one LDS
// read and two or three VALU operations behind each MFMA; without it the
// compiler bunches them (8192 x 14336 x 4096: 407 us with, 421 without, the
// 8-wave 64-token kernel before 516).  Counters there: the matrix cores are
// busy 73% of the cycles, but the clock falls to 1.63-1.8 GHz under the load
// (2.41 GHz in a launch that leaves a quarter of the CUs idle).
//
// Shorter products are bound by one wave's chain (a container takes a lone
// wave about 0.55 us, mostly instruction issue: deeper rings of weights or
// stages changed nothing) and by about 5 us of launch, first loads, reduction
// and stores.  They run smaller workgroups with K split over more waves
// (wide_pick*, launch_rules.h).
#include <type_traits>

#include "sherry_internal.h"

namespace sherry {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kWdOutside = 0x7FFFFFF0;  // a buffer offset past any range: loads read zero
constexpr int kWdHead = 128 + 512 + 2048;  // table, x scales, weight scales
constexpr int kWdSW = 40;                  // words per token of an epilogue strip

// MT blocks of 32 tokens, K in S parts, W waves, EU waves per SIMD (the
// register budget).  RING weight containers per wave in registers; NST stages
// of one container's activations in LDS: the S parts' windows as S x TOK
// virtual rows of 128 bytes.
//
// GR: per-group weight scales, one per row and 128 weights, i.e. per unit:
// 1 with a 4-byte load per lane and unit (any row length), 4 with a 16-byte
// load per lane and four units (rows of whole, aligned 16-byte pieces; a
// quarter of the cache lines touched).
template <int MT_, int S_, int W_, int EU_, int GR_ = 0>
struct WdCfg {
  static constexpr int MT = MT_, S = S_, W = W_, EU = EU_, GR = GR_, RING = 4, NST = 4;
  static_assert(RING % NST == 0, "ring slots and stages repeat together");
  static constexpr int THREADS = 64 * W;
  static constexpr int TOK = 32 * MT;
  static constexpr int ROWS = TOK * S;
  static constexpr int STAGE = ROWS * kTileK;
  static constexpr int SPT = STAGE / 1024 / W;
  static constexpr int TILES = W / S;
  // workgroups per prepared block (8 tiles x 64 tokens) of a grouped launch
  static constexpr int PER = TOK > 64 ? 1 : 8 / TILES * (64 / TOK);
  // after the stream: the K parts' partial sums (RT token blocks at a time),
  // then two epilogue strips per wave
  static constexpr int RT = MT * W > 16 ? 16 / W : MT;
  static constexpr int RED = S > 1 ? W * RT * 32 * 256 : 0;
  static constexpr int STRIPS = W * 2 * 32 * kWdSW * 4;
  static constexpr int TAIL = RED > STRIPS ? RED : STRIPS;
  static constexpr int BODY = NST * STAGE > TAIL ? NST * STAGE : TAIL;
  static constexpr int LDS = kWdHead + BODY;
  static_assert(SPT >= 1 && SPT * 1024 * W == STAGE, "stage split");
  static_assert(TILES * kTileRows * 4 <= 2048 && TOK * 4 <= 512, "scales fit");
  static_assert(LDS <= 160 * 1024, "LDS");
};

struct WdProblem {
  const uint8_t* w;
  const int8_t* x;
  const float* x_scale;
  float* y;
  int32_t* acc;
  int n, k, m;
  WScale ws;
  const float* gs;  // per-group scales [n][ceil(k/128)]
};

// Waits until at most N vector-memory loads of this wave are outstanding
// (loads complete in issue order); the other counters are left alone.
// (a count past the field's 63 is only waited for more strictly)
constexpr int wd_cap(int n) { return n < 63 ? n : 63; }
template <int N>
__device__ __forceinline__ void wd_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  constexpr int kImm = (N & 15) | (7 << 4) | (15 << 8) | (((N >> 4) & 3) << 14);
  __builtin_amdgcn_s_waitcnt(static_cast<int16_t>(kImm));
}
// Waits for this wave's LDS reads and writes.
__device__ __forceinline__ void wd_wait_lgkm() {
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
}
// Workgroup barrier between stages.  A workgroup-scope release fence would
// also wait for every DMA in flight (they write LDS), so the ordering is
// explicit: the caller has waited for its own DMAs of the stage about to be
// read, every LDS read of the stage about to be overwritten has returned (its
// results fed MFMAs issued before this point), and the compiler moves no
// memory access across.
__device__ __forceinline__ void wd_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
// Barrier for LDS traffic only (outstanding stores stay in flight).
__device__ __forceinline__ void wd_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int j0, int... is>
__device__ __forceinline__ void wd_lookup8(const uint32_t (&d)[5], const uint32_t* lut,
                                           uint32_t (&wv)[32], std::integer_sequence<int, is...>) {
  ((wv[j0 + is] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lut) +
                                                     code_x4<j0 + is>(d))),
   ...);
}

// The 16-byte piece c of virtual row r sits at piece c ^ wd_swz(r) of its 128
// bytes: 16 lanes reading one piece of 16 consecutive rows then cover the 64
// banks once.
__device__ __forceinline__ int wd_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

template <int MT>
__device__ __forceinline__ void wd_read(v4i (&xv)[MT], const int8_t* p) {
#pragma unroll
  for (int tb = 0; tb < MT; ++tb) xv[tb] = *reinterpret_cast<const v4i*>(p + tb * 32 * kTileK);
}

// Pairs rows i and i + 32 of group s: words 8s..8s+3 become rows 0-31, words
// 8s+4..8s+7 rows 32-63, lane l holding K half l / 32.
template <int s>
__device__ __forceinline__ void wd_swap(uint32_t (&wv)[32]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r =
        __builtin_amdgcn_permlane32_swap(wv[8 * s + i], wv[8 * s + 4 + i], false, false);
    wv[8 * s + i] = r[0];
    wv[8 * s + 4 + i] = r[1];
  }
}

// Issue order of a slice of N MFMAs: behind each one LDS read (a fragment in
// the first half, lookups in the second) and its share of the 20 VALU
// operations.
template <int N, int i = 0>
__device__ __forceinline__ void wd_interleave() {
  if constexpr (i < N) {
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, i < N / 2 ? 1 : (8 + N / 2 - 1) / (N / 2), 0);
    __builtin_amdgcn_sched_group_barrier(0x2, (20 + N - 1) / N, 0);
    wd_interleave<N, i + 1>();
  }
}

// One slice: the MFMAs of group s; on the way the lookups of group l of the
// container in d, the fragments of the next slice (xn from pn) and the swap
// of the next slice's group.
// With kZero the sums start from zero.
template <int MT, int s, int l, bool kZero = false>
__device__ __forceinline__ void wd_slice(uint32_t (&wv)[32], const uint32_t (&d)[5],
                                         const uint32_t* lut, const v4i (&xv)[MT], v4i (&xn)[MT],
                                         const int8_t* pn, v16i (&c)[2][MT]) {
  __builtin_amdgcn_sched_barrier(0);
  const v4i wl = {static_cast<int>(wv[8 * s]), static_cast<int>(wv[8 * s + 1]),
                  static_cast<int>(wv[8 * s + 2]), static_cast<int>(wv[8 * s + 3])};
  const v4i wh = {static_cast<int>(wv[8 * s + 4]), static_cast<int>(wv[8 * s + 5]),
                  static_cast<int>(wv[8 * s + 6]), static_cast<int>(wv[8 * s + 7])};
  wd_read<MT>(xn, pn);
  wd_swap<(s + 1) % 4>(wv);
  wd_lookup8<8 * l>(d, lut, wv, std::make_integer_sequence<int, 8>{});
#pragma unroll
  for (int tb = 0; tb < MT; ++tb) {
    c[0][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xv[tb], wl, kZero ? v16i{} : c[0][tb], 0, 0, 0);
    c[1][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xv[tb], wh, kZero ? v16i{} : c[1][tb], 0, 0, 0);
  }
  wd_interleave<2 * MT>();
  __builtin_amdgcn_sched_barrier(0);
}

// Workgroup g of problem p: tiles TILES * g .. TILES * g + TILES - 1, wave w:
// tile w / S, part w % S of its units ([sp U, min((sp + 1) U, C)), U =
// ceil(C/S); units past a part's end read zeros and multiply zeros).
//
// Loads per unit, issued on every path in this order: two of weights (slice
// 1), SPT of DMA (after the barrier between slices 1 and 2, which makes the
// next unit's stage readable and the previous one's free).  So the number
// issued after any stage's last DMA is a constant, and the wait before each
// barrier an exact vmcnt.
template <class G>
__device__ __forceinline__ void wd_block(const WdProblem& p, int g, int8_t* lds) {
  constexpr int MT = G::MT, S = G::S, W = G::W;
  constexpr int D = G::NST - 1;
  // opaque, so that a caller's loop over blocks keeps no address of this
  // block in registers across it
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* lut = reinterpret_cast<uint32_t*>(lds);
  float* xsl = reinterpret_cast<float*>(lds + 128);
  float* wsl = reinterpret_cast<float*>(lds + 640);
  int8_t* const xs = lds + kWdHead;
  const int C = (p.k + kTileK - 1) / kTileK;
  const int R = (p.n + kTileRows - 1) / kTileRows;
  // (with 16-byte scale loads the parts are whole chunks of four units)
  const int U = G::GR == 4 ? ((C + S - 1) / S + 3) & ~3 : (C + S - 1) / S;
  const int r = g * G::TILES + wave / S;
  const int sp = wave % S;
  const int u0 = sp * U, u1 = (u0 + U < C) ? u0 + U : C;
  const bool live = r < R && u0 < u1;
  const UnitRun rs{p.w + (int64_t(r < R ? r : 0) * C + (live ? u0 : 0)) * kUnitBytes,
                   live ? u1 - u0 : 0};
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.x), 0, p.m * p.k, kBufferWord3);

  // DMA instruction i of this wave fills virtual rows 8 (W i + wave) + lane / 8
  // (eight rows of one window); pieces past the end of their part or past k
  // come from outside the buffer, as zeros, rows past m too
  const int o = 16 * ((lane & 7) ^ (lane >> 3) ^ (wave & 1));
  const int rowl = (lane >> 3) * p.k;
  int8_t* const xw = xs + 1024 * wave;
  auto dma = [&](int ch, int i) {
    const int vr = 8 * (W * i + wave);          // first virtual row of the instruction
    const int win = vr / G::TOK, t0 = vr % G::TOK;
    const int kb = win * U * kTileK;            // first K value of the window
    const int kend = (win + 1) * U < C ? (win + 1) * U * kTileK : p.k;
    const int off = rowl + (t0 * p.k + kb + ch * kTileK) + o;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rx, (lds_void*)(xw + (ch % G::NST) * G::STAGE + i * 1024 * W), 16,
        o + ch * kTileK < kend - kb ? off : kWdOutside, 0, 0, 0);
  };

  // reader: virtual row sp*TOK + 32tb + lane%32, piece 2s + lane/32
  int lo[4];
  {
    const int sw = wd_swz(lane & 31);
#pragma unroll
    for (int s = 0; s < 4; ++s)
      lo[s] = (sp * G::TOK + (lane & 31)) * kTileK + 16 * ((2 * s + (lane >> 5)) ^ sw);
  }

  // a k that is not a multiple of 16 leaves part of the next token's row in
  // the piece that holds K = k: cleared once that piece has landed (unit chl of
  // part sl)
  const int kr = p.k & 15;
  const int sl = (C - 1) / U, jl = (C - 1) - sl * U;
  const int chl = kr ? jl : -1;
  auto clear_tail = [&]() {
    const int pc = ((p.k & ~15) - (C - 1) * kTileK) / 16;
    const int nd = (16 - kr) / 4;
    int8_t* st = xs + (chl % G::NST) * G::STAGE;
    for (int e = tid; e < G::TOK * nd; e += G::THREADS) {
      const int vr = sl * G::TOK + e / nd, b = kr + 4 * (e % nd);
      *reinterpret_cast<uint32_t*>(st + vr * kTileK + 16 * (pc ^ wd_swz(vr)) + b) = 0;
    }
    wd_wait_lgkm();
    wd_barrier();
  };

  v16i c[2][MT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int tb = 0; tb < MT; ++tb) c[h][tb] = v16i{};

  // per-group: fp32 sums in unit order, and the scales of this lane's row
  // (lane i = row i of the tile; rows past n and units past the part read
  // zeros): slot u of gq holds the unit in flight at position u, the next
  // four come in while these are used
  typedef float v16f __attribute__((ext_vector_type(16)));
  constexpr int GM = G::GR ? MT : 1;
  v16f cf[2][GM];
  uint32_t gq[4];
  u32x4 gn;
  __amdgpu_buffer_rsrc_t grs;
  if constexpr (G::GR != 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int tb = 0; tb < MT; ++tb) cf[h][tb] = v16f{};
    const int rows = r < R ? p.n - r * kTileRows : 0;
    grs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(p.gs) + int64_t(r < R ? r : 0) * kTileRows * C, 0,
        (rows < kTileRows ? rows : kTileRows) * C * 4, kBufferWord3);
  }
  auto scale_off = [&](int unit) {
    return unit < u1 - u0 ? 4 * (lane * C + u0 + unit) : kWdOutside;
  };

  // the epilogue's scales, through LDS: loaded before anything else, since a
  // load between the stores would wait for every store before it
  float sxv = 0.0f, swv = 0.0f;
  if (tid < G::TOK) sxv = tid < p.m ? as_global(p.x_scale)[tid] : 0.0f;
  {
    const int row = g * G::TILES * kTileRows + tid;
    if (!G::GR && tid < G::TILES * kTileRows) swv = row < p.n ? p.ws.at(row) : 0.0f;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ch = 0; ch < D; ++ch)
#pragma unroll
    for (int i = 0; i < G::SPT; ++i) dma(ch, i);
  __builtin_amdgcn_sched_barrier(0);
  uint32_t ring[G::RING][5];
#pragma unroll
  for (int u = 0; u < G::RING; ++u) {
    load_unit(ring[u], rs, u, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (G::GR == 4) {
    const u32x4 g0 = __builtin_amdgcn_raw_buffer_load_b128(grs, scale_off(0), 0, 0);
    gn = __builtin_amdgcn_raw_buffer_load_b128(grs, scale_off(4), 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) gq[e] = g0[e];
  } else if constexpr (G::GR == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      gq[e] = __builtin_amdgcn_raw_buffer_load_b32(grs, scale_off(e), 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  constexpr int GP = G::GR == 4 ? 2 : G::GR == 1 ? 4 : 0;  // scale loads of the prologue
  if (tid < 32) lut[tid] = decode_word(tid);
  if (tid < G::TOK) xsl[tid] = sxv;
  if (!G::GR && tid < G::TILES * kTileRows) wsl[tid] = swv;
  wd_wait_vm<wd_cap((D - 1) * G::SPT + 2 * G::RING + GP)>();
  wd_wait_lgkm();
  wd_barrier();  // chunk 0, the table and the scales are ready
  if (chl == 0) clear_tail();

  uint32_t wv[32];
  wd_lookup8<0>(ring[0], lut, wv, std::make_integer_sequence<int, 8>{});
  wd_lookup8<8>(ring[0], lut, wv, std::make_integer_sequence<int, 8>{});
  wd_lookup8<16>(ring[0], lut, wv, std::make_integer_sequence<int, 8>{});
  // fragments are read one slice ahead, two with one token block
  constexpr int XD = MT <= 1 ? 2 : 1, XN = MT <= 1 ? 4 : 2;
  v4i xv[XN][MT];
  wd_read<MT>(xv[0], xs + lo[0]);
  if constexpr (XD == 2) wd_read<MT>(xv[1], xs + lo[1]);
  wd_swap<0>(wv);
  for (int j = 0; j < U; j += G::RING) {
#pragma unroll
    for (int u = 0; u < G::RING; ++u) {
      const int jj = j + u;
      if (u > 0 && jj >= U) break;
      const uint32_t (&dn)[5] = ring[(u + 1) % G::RING];
      const int8_t* st = xs + u % G::NST * G::STAGE;
      const int8_t* sn = xs + (u + 1) % G::NST * G::STAGE;
      wd_slice<MT, 0, 3, G::GR != 0>(wv, ring[u], lut, xv[0], xv[XD % XN], st + lo[XD], c);
      load_unit(ring[u], rs, jj + G::RING, lane);
      wd_slice<MT, 1, 0>(wv, dn, lut, xv[1], xv[(1 + XD) % XN], st + lo[1 + XD], c);
      // chunk jj + 1 has landed for every wave after this barrier, and every
      // wave is done with the stage of chunk jj - 1
      // (scale loads go out at the end of a unit: of every one, or, four units'
      // at once, of the last in a round)
      constexpr int LU = G::GR == 1 ? 3 : 2;  // loads per unit besides the DMA
      const int ge = G::GR == 4 && u < 2 ? 1 : 0;
      if (u < D - 1 && j == 0) {
        if (u == 0) wd_wait_vm<wd_cap((D - 2) * G::SPT + 2 * G::RING + GP + 2)>();
        else wd_wait_vm<wd_cap((D - 2) * G::SPT + 2 * G::RING + GP + 2 + LU)>();
      } else if (ge) {
        wd_wait_vm<wd_cap(LU * (D - 1) + (D - 2) * G::SPT + 1)>();
      } else {
        wd_wait_vm<wd_cap(LU * (D - 1) + (D - 2) * G::SPT)>();
      }
      wd_barrier();
      if (jj + 1 == chl) clear_tail();
#pragma unroll
      for (int i = 0; i < G::SPT; ++i) dma(jj + D, i);
      wd_slice<MT, 2, 1>(wv, dn, lut, xv[2 % XN], xv[(2 + XD) % XN],
                         XD == 2 ? sn + lo[0] : st + lo[3], c);
      wd_slice<MT, 3, 2>(wv, dn, lut, xv[3 % XN], xv[(3 + XD) % XN], sn + lo[XD - 1], c);
      if constexpr (G::GR != 0) {
        // rows lane % 32 and lane % 32 + 32
        const auto gr = __builtin_amdgcn_permlane32_swap(gq[u], gq[u], false, false);
#pragma unroll
        for (int tb = 0; tb < MT; ++tb)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float sc = __uint_as_float(h ? gr[1] : gr[0]);
#pragma unroll
            for (int e = 0; e < 16; ++e)
              cf[h][tb][e] = __builtin_fmaf(static_cast<float>(c[h][tb][e]), sc, cf[h][tb][e]);
          }
        if constexpr (G::GR == 1) {
          gq[u] = __builtin_amdgcn_raw_buffer_load_b32(grs, scale_off(jj + 4), 0, 0);
        } else if (u == 3) {
#pragma unroll
          for (int e = 0; e < 4; ++e) gq[e] = gn[e];
          gn = __builtin_amdgcn_raw_buffer_load_b128(grs, scale_off(jj + 5), 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  wd_wait_vm<0>();  // no DMA may land in the LDS after this point

  // part of the tile's sums that this wave finishes: all of them (S = 1), row
  // half h = sp (S = 2), or one half of the tokens of a row half (S = 4),
  // or a quarter (S = 8)
  constexpr int EN = S <= 2 ? 16 : 32 / S;            // elements per row half owned
  const int hs = S == 1 ? 0 : sp & 1;                 // first owned row half
  const int es = S <= 2 ? 0 : (sp >> 1) * EN;         // first owned element
  constexpr int HN = S == 1 ? 2 : 1;                  // owned row halves
  v16i f[HN][MT];  // owned sums (elements [0, EN)); fp32 bits with GR
  auto sum_bits = [&](int h, int tb, int e) {
    if constexpr (G::GR != 0) {
      const float v = cf[h][tb][e];  // (a bit cast of the element in place reads element 0)
      return __float_as_int(v);
    } else {
      return c[h][tb][e];
    }
  };
  if constexpr (S == 1) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int tb = 0; tb < MT; ++tb)
#pragma unroll
        for (int e = 0; e < 16; ++e) f[h][tb][e] = sum_bits(h, tb, e);
    wd_lds_barrier();  // every wave is done with the stages
  } else {
    int32_t* red = reinterpret_cast<int32_t*>(xs);
    constexpr int RT = G::RT;
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += RT) {
      wd_lds_barrier();
#pragma unroll
      for (int tb = 0; tb < RT; ++tb)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            red[(((wave * RT + tb) * 2 + h) * 16 + e) * 64 + lane] = sum_bits(h, t0 + tb, e);
      wd_lds_barrier();
      const int w0 = wave - sp;
#pragma unroll
      for (int tb = 0; tb < RT; ++tb)
#pragma unroll
        for (int e = 0; e < EN; ++e) {
          // the parts in order
          const int32_t* rp = red + (((w0 * RT + tb) * 2 + hs) * 16 + es + e) * 64 + lane;
          if constexpr (G::GR != 0) {
            float v = __int_as_float(rp[0]);
#pragma unroll
            for (int q = 1; q < S; ++q) v += __int_as_float(rp[q * RT * 2 * 16 * 64]);
            f[0][t0 + tb][e] = __float_as_int(v);
          } else {
            int32_t v = rp[0];
#pragma unroll
            for (int q = 1; q < S; ++q) v += rp[q * RT * 2 * 16 * 64];
            f[0][t0 + tb][e] = v;
          }
        }
    }
    wd_lds_barrier();
  }
  if (r >= R) return;

  // epilogue: lane holds C[token][row], row = 32h + lane % 32 of the tile,
  // token = 32tb + 8(e/4) + 4(lane/32) + e%4.  A block of 32 rows and the
  // owned tokens (TN of 32) goes through the wave's own LDS strip and comes
  // back as 16-byte pieces of four rows.  Two strips: the next block is
  // written while this one's reads are in flight.
  constexpr int TN = 2 * EN;       // tokens per block (16 elements: 32)
  constexpr int PN = TN / 8;       // pieces per lane
  constexpr int NB = HN * MT;      // blocks
  int32_t* strip = reinterpret_cast<int32_t*>(xs) + wave * 2 * 32 * kWdSW;
  const int c4 = lane & 7;
  const int tokb = 2 * es;         // first owned token of a 32-token block
  float swl[HN][4];
#pragma unroll
  for (int h = 0; h < HN; ++h)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      swl[h][u] = G::GR ? 0.0f : wsl[(wave / S) * kTileRows + 32 * (hs + h) + 4 * c4 + u];
  // y of one sum; the int32 sums themselves go to acc (not with GR)
  auto out = [&](int32_t v, float sx, float sw) {
    return G::GR ? __int_as_float(v) * sx : static_cast<float>(v) * (sx * sw);
  };
  int32_t* const acc_out = G::GR ? nullptr : p.acc;
  auto put = [&](int b) {
    int32_t* st = strip + (b & 1) * 32 * kWdSW;
#pragma unroll
    for (int e = 0; e < EN; ++e) {
      const int tl = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      st[tl * kWdSW + (lane & 31)] = f[b % HN][b / HN][e];
    }
  };
  const bool whole = p.m >= G::TOK && (r + 1) * kTileRows <= p.n && (p.n % 4 == 0) &&
                     (reinterpret_cast<uintptr_t>(p.y) % 16 == 0) &&
                     (!acc_out || reinterpret_cast<uintptr_t>(acc_out) % 16 == 0);
  const bool vec = (p.n % 4 == 0) && (reinterpret_cast<uintptr_t>(p.y) % 16 == 0) &&
                   (!acc_out || reinterpret_cast<uintptr_t>(acc_out) % 16 == 0);
  put(0);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int h = b % HN, tb = b / HN;
    __asm__ volatile("" ::: "memory");
    const int32_t* st = strip + (b & 1) * 32 * kWdSW;
    v4i v[PN];
    float sx[PN];
#pragma unroll
    for (int i = 0; i < PN; ++i) {
      const int tl = (lane >> 3) + 8 * i;
      v[i] = *reinterpret_cast<const v4i*>(st + tl * kWdSW + 4 * c4);
      sx[i] = xsl[32 * tb + tokb + tl];
    }
    __asm__ volatile("" ::: "memory");
    if (b + 1 < NB) put(b + 1);
    const int row = r * kTileRows + 32 * (hs + h) + 4 * c4;
    if (whole) {
      const int64_t at = int64_t(32 * tb + tokb + (lane >> 3)) * p.n + row;
      float* yp = as_global_mut(p.y) + at;
      int32_t* ap = as_global_mut(acc_out) + at;
#pragma unroll
      for (int i = 0; i < PN; ++i) {
        float4 o4;
        o4.x = out(v[i].x, sx[i], swl[h][0]);
        o4.y = out(v[i].y, sx[i], swl[h][1]);
        o4.z = out(v[i].z, sx[i], swl[h][2]);
        o4.w = out(v[i].w, sx[i], swl[h][3]);
        *reinterpret_cast<float4*>(yp + int64_t(8 * i) * p.n) = o4;
        if (acc_out) *reinterpret_cast<v4i*>(ap + int64_t(8 * i) * p.n) = v[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < PN; ++i) {
        const int tok = 32 * tb + tokb + (lane >> 3) + 8 * i;
        if (tok >= p.m || row >= p.n) continue;
        const int32_t vv[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        float o4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) o4[u] = out(vv[u], sx[i], swl[h][u]);
        float* yrow = as_global_mut(p.y) + int64_t(tok) * p.n + row;
        if (vec) {
          *reinterpret_cast<float4*>(yrow) = make_float4(o4[0], o4[1], o4[2], o4[3]);
          if (acc_out) *reinterpret_cast<v4i*>(as_global_mut(acc_out) + int64_t(tok) * p.n + row) = v[i];
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (row + u >= p.n) break;
            yrow[u] = o4[u];
            if (acc_out) as_global_mut(acc_out)[int64_t(tok) * p.n + row + u] = vv[u];
          }
        }
      }
    }
  }
}

// Token block t0 / TOK of a product.
template <class G>
__device__ __forceinline__ void wd_tokens(WdProblem& p, int64_t t0) {
  p.x += t0 * p.k;
  p.x_scale += t0;
  p.y += t0 * p.n;
  if (p.acc) p.acc += t0 * p.n;
  p.m = (p.m - t0 < G::TOK) ? static_cast<int>(p.m - t0) : G::TOK;
}

// grid: x = groups of TILES tiles, y = token blocks (wide_xcd_order: in eighths)
template <class G>
__global__ __launch_bounds__(G::THREADS) __attribute__((amdgpu_waves_per_eu(G::EU))) void wide_kernel(
    WdProblem p) {
  __shared__ __attribute__((aligned(16))) int8_t lds[G::LDS];
  const int groups = static_cast<int>(gridDim.x);
  int g = blockIdx.x, tb = blockIdx.y;
  if (wide_xcd_order(groups * G::TILES)) {
    const int b = xcd_block(tb * groups + g, groups * static_cast<int>(gridDim.y));
    tb = b / groups;
    g = b - tb * groups;
  }
  wd_tokens<G>(p, int64_t(tb) * G::TOK);
  wd_block<G>(p, g, lds);
}

// Grouped launch of 8 x 64 blocks, PER workgroups each (wide_run64).
template <class G>
__global__ __launch_bounds__(G::THREADS) __attribute__((amdgpu_waves_per_eu(G::EU))) void wide_batched_kernel(
    const sherry_gemm_desc* __restrict__ descs, int count) {
  __shared__ __attribute__((aligned(16))) int8_t lds[G::LDS];
  static_assert(G::TOK <= 64 || (G::TOK == 128 && G::TILES == 4 && G::PER == 1),
                "two prepared blocks, two workgroups");
  const int32_t blk = static_cast<int32_t>(blockIdx.x) / G::PER;
  const int lo = find_block_desc(descs, count, blk);
  if (lo < 0) return;
  const sherry_gemm_desc& d = descs[lo];
  const int R = (d.n + kTileRows - 1) / kTileRows;
  const WideRun run = wide_run64(G::TOK, G::TILES, blk - d.block_begin,
                                 static_cast<int>(blockIdx.x) % G::PER, d.m, R);
  if (run.reps == 0) return;
  WdProblem p{d.w, d.x, d.x_scale, d.y, d.acc, d.n, d.k, d.m, WScale{d.w_scales, d.w_scale}, nullptr};
  wd_tokens<G>(p, run.t0);
  for (int h = 0; h < run.reps; ++h) {
    if ((run.g + h) * G::TILES >= R) return;
    if (h) __syncthreads();  // the table, scales and strips are written again
    wd_block<G>(p, run.g + h, lds);
  }
}

// Grouped launch of 32-token prepared blocks (every m <= 32, or some product
// with per-group scales): 8 tiles x 32 tokens of a product without per-group
// scales, on G0 (wide_run32); 4 tiles x 32 tokens of one with them, on G1 (void:
// none), and its odd last token block on G1O where G1 has 64 tokens x two tiles
// (wide_run32_group).  PER workgroups share a block's parts.
template <class G0_, class G1_, int PER_, class G1O_ = void>
struct WdShort32 {
  using G0 = G0_;
  static constexpr bool kGroups = !std::is_same_v<G1_, void>, kOdd = !std::is_same_v<G1O_, void>;
  using GG = std::conditional_t<kGroups, G1_, G0>;
  using GO = std::conditional_t<kOdd, G1O_, GG>;
  static constexpr int PER = PER_;
  static constexpr int THREADS = G0::THREADS, EU = G0::EU < GG::EU ? G0::EU : GG::EU;
  static constexpr int LDS0 = G0::LDS > GG::LDS ? G0::LDS : GG::LDS;
  static constexpr int LDS = LDS0 > GO::LDS ? LDS0 : GO::LDS;
  static_assert(G0::TOK == 32 && G0::THREADS == GG::THREADS && G0::THREADS == GO::THREADS,
                "one block size");
  static_assert(8 / G0::TILES % PER == 0, "parts of a block");
  static_assert(!kGroups || (GG::TOK == 64 ? PER == 1 : 4 / GG::TILES % PER == 0),
                "parts of a block (64 tokens: one workgroup)");
  static_assert(kOdd == (kGroups && GG::TOK == 64 && GG::TILES == 2), "an odd token block's shape");
  static_assert(!kOdd || (GO::TOK == 32 && GO::TILES == 4), "a whole prepared block");
};

template <class G>
__device__ __forceinline__ void wd_run(WdProblem& p, const WideRun& run, int R, int8_t* lds) {
  wd_tokens<G>(p, run.t0);
  for (int h = 0; h < run.reps; ++h) {
    const int g = run.g + h * run.step;
    if (g * G::TILES >= R) return;
    if (h) __syncthreads();  // the table, scales and strips are written again
    wd_block<G>(p, g, lds);
  }
}

template <class B>
__global__ __launch_bounds__(B::THREADS) __attribute__((amdgpu_waves_per_eu(B::EU))) void wide_batched32_kernel(
    const sherry_gemm_desc* __restrict__ descs, int count) {
  using G0 = typename B::G0;
  using G1 = typename B::GG;
  constexpr int PER = B::PER;
  __shared__ __attribute__((aligned(16))) int8_t lds[B::LDS];
  const int32_t blk = static_cast<int32_t>(blockIdx.x) / PER;
  const int sub = static_cast<int>(blockIdx.x) % PER;
  const int lo = find_block_desc(descs, count, blk);
  if (lo < 0) return;
  const sherry_gemm_desc& d = descs[lo];
  const int R = (d.n + kTileRows - 1) / kTileRows;
  WdProblem p{d.w, d.x, d.x_scale, d.y, d.acc, d.n, d.k, d.m, WScale{d.w_scales, d.w_scale},
              d.w_group_scales};
  if constexpr (B::kGroups) {
    if (d.w_group_scales) {
      const WideRun run =
          wide_run32_group(G1::TOK, G1::TILES, PER, blk - d.block_begin, sub, d.m, R);
      if (run.reps == 0) return;
      p.acc = nullptr;
      if constexpr (B::kOdd) {
        if (run.odd) return wd_run<typename B::GO>(p, run, R, lds);
      }
      return wd_run<G1>(p, run, R, lds);
    }
  }
  const WideRun run = wide_run32(G0::TILES, PER, blk - d.block_begin, sub, d.m, R);
  if (run.reps == 0) return;
  wd_run<G0>(p, run, R, lds);
}

constexpr int64_t kWdMaxGridY = 32768;  // further token blocks go to further launches

template <class G>
int launch_wide_cfg(const WdProblem& p, hipStream_t s) {
  const int64_t R = ceil_div(p.n, kTileRows), TB = ceil_div(p.m, G::TOK);
  for (int64_t b0 = 0; b0 < TB; b0 += kWdMaxGridY) {
    const int64_t nb = TB - b0 < kWdMaxGridY ? TB - b0 : kWdMaxGridY, t0 = b0 * G::TOK;
    WdProblem q = p;
    q.x += t0 * p.k;
    q.x_scale += t0;
    q.y += t0 * p.n;
    if (q.acc) q.acc += t0 * p.n;
    q.m = static_cast<int>(p.m - t0);
    const int rc = launch(wide_kernel<G>,
                          dim3(static_cast<unsigned>(ceil_div(R, G::TILES)), static_cast<unsigned>(nb)),
                          dim3(G::THREADS), 0, s, q);
    if (rc != SHERRY_OK) return rc;
  }
  return SHERRY_OK;
}

// The shapes of a workgroup: tokens x tiles, K parts, waves.
using WdLong = WdCfg<4, 1, 4, 2>;    // 128 x 4
using WdMid = WdCfg<2, 1, 4, 3>;     // 64 x 4
using WdHalf = WdCfg<2, 2, 4, 2>;    // 64 x 2, K in 2
using WdQuarter = WdCfg<2, 4, 8, 2>; // 64 x 2, K in 4, eight waves
using WdShort = WdCfg<1, 4, 4, 2>;   // 32 x 1, K in 4
using WdTiny = WdCfg<1, 8, 8, 2>;    // 32 x 1, K in 8, eight waves
using WdPair = WdCfg<1, 2, 4, 3>;    // 32 x 2, K in 2 (grouped launches)
using WdThin = WdCfg<1, 1, 4, 4>;    // 32 x 4 (grouped launches)

template <class G>
constexpr bool wd_is(const WideCost& c) {
  return c.tokens == G::TOK && c.tiles == G::TILES && c.parts == G::S;
}
static_assert(wd_is<WdLong>(kWideCost[kWideLong]) && wd_is<WdMid>(kWideCost[kWideMid]) &&
                  wd_is<WdHalf>(kWideCost[kWideHalf]) && wd_is<WdQuarter>(kWideCost[kWideQuarter]) &&
                  wd_is<WdShort>(kWideCost[kWideShort]) && wd_is<WdTiny>(kWideCost[kWideTiny]) &&
                  wd_is<WdPair>(kWideCost[kWidePair]) && wd_is<WdThin>(kWideCost[kWideThin]),
              "the shapes that the cost model prices");

// The shapes with per-group scales: twice the accumulators (int32 sums of one
// unit, fp32 sums), and a conversion and an fma per unit and sum (128 VALU
// operations per 64 x 64 sums beside 16 MFMAs: with two waves per SIMD the
// VALU is what bounds them).
template <int GR>
using WdGrpMid = WdCfg<2, 1, 4, 2, GR>;  // 64 x 4
template <int GR>
using WdGrpHalf = WdCfg<2, 2, 4, 2, GR>;  // 64 x 2, K in 2
template <int GR>
using WdGrpPair = WdCfg<1, 2, 4, 3, GR>;  // 32 x 2, K in 2
template <int GR>
using WdGrpShort = WdCfg<1, 4, 4, 3, GR>;  // 32 x 1, K in 4
template <int GR>
using WdGrpTiny = WdCfg<1, 8, 8, 2, GR>;  // 32 x 1, K in 8, eight waves
template <int GR>
using WdGrpThin = WdCfg<1, 1, 4, 3, GR>;  // 32 x 4 (an odd token block beside 64 x 2)
static_assert(wd_is<WdGrpMid<1>>(kWideGroupCost[kWideMid]) &&
                  wd_is<WdGrpHalf<1>>(kWideGroupCost[kWideHalf]) &&
                  wd_is<WdGrpPair<1>>(kWideGroupCost[kWidePair]) &&
                  wd_is<WdGrpShort<1>>(kWideGroupCost[kWideShort]) &&
                  wd_is<WdGrpTiny<1>>(kWideGroupCost[kWideTiny]),
              "the shapes that the cost model prices");

template <int GR>
int launch_wide_group_gr(const WdProblem& p, hipStream_t s) {
  switch (wide_pick_group(p.m, p.n, p.k, GR == 4)) {
    case kWideMid: return launch_wide_cfg<WdGrpMid<GR>>(p, s);
    case kWideHalf: return launch_wide_cfg<WdGrpHalf<GR>>(p, s);
    case kWidePair: return launch_wide_cfg<WdGrpPair<GR>>(p, s);
    case kWideShort: return launch_wide_cfg<WdGrpShort<GR>>(p, s);
    default: return launch_wide_cfg<WdGrpTiny<GR>>(p, s);
  }
}

template <class G>
int launch_wide_batched_cfg(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                            hipStream_t s) {
  return launch(wide_batched_kernel<G>, dim3(static_cast<unsigned>(total_blocks * G::PER)),
                dim3(G::THREADS), 0, s, descs, count);
}
template <class G0, class G1, int PER, class G1O = void>
int launch_wide_batched32_cfg(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                              hipStream_t s) {
  return launch(wide_batched32_kernel<WdShort32<G0, G1, PER, G1O>>,
                dim3(static_cast<unsigned>(total_blocks * PER)), dim3(G0::THREADS), 0, s, descs,
                count);
}

}  // namespace

int launch_wide(const uint8_t* w, const int8_t* x, const float* x_scale, WScale ws, float* y,
                int32_t* acc, int64_t m, int64_t n, int64_t k, hipStream_t s) {
  const WdProblem p{w, x, x_scale, y, acc, static_cast<int>(n), static_cast<int>(k),
                    static_cast<int>(m), ws, nullptr};
  switch (wide_pick(m, n, k)) {
    case kWideLong: return launch_wide_cfg<WdLong>(p, s);
    case kWideMid: return launch_wide_cfg<WdMid>(p, s);
    case kWideHalf: return launch_wide_cfg<WdHalf>(p, s);
    case kWideQuarter: return launch_wide_cfg<WdQuarter>(p, s);
    case kWideShort: return launch_wide_cfg<WdShort>(p, s);
    default: return launch_wide_cfg<WdTiny>(p, s);
  }
}

int launch_wide_group(const uint8_t* w, const int8_t* x, const float* x_scale, const float* gs,
                      float* y, int32_t* acc, int64_t m, int64_t n, int64_t k, hipStream_t s) {
  if (acc) {
    // int32 totals from an unscaled launch (its y is overwritten below)
    const int rc = launch_wide(w, x, x_scale, WScale{nullptr, 1.0f}, y, acc, m, n, k, s);
    if (rc != SHERRY_OK) return rc;
  }
  const WdProblem p{w, x, x_scale, y, nullptr, static_cast<int>(n), static_cast<int>(k),
                    static_cast<int>(m), WScale{nullptr, 0.0f}, gs};
  const bool pieces = ceil_div(k, kTileK) % 4 == 0 && (reinterpret_cast<uintptr_t>(gs) & 15) == 0;
  return pieces ? launch_wide_group_gr<4>(p, s) : launch_wide_group_gr<1>(p, s);
}

int launch_wide_batched(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                        int max_m, bool groups, hipStream_t s) {
  if (groups) {
    // (a launch's products may have any row lengths: 4-byte scale loads)
    switch (wide_pick_batched_group(total_blocks, count, max_m)) {
      case kWideMid:
        return launch_wide_batched32_cfg<WdThin, WdGrpMid<1>, 1>(descs, count, total_blocks, s);
      case kWideHalf:
        return launch_wide_batched32_cfg<WdThin, WdGrpHalf<1>, 1, WdGrpThin<1>>(descs, count,
                                                                               total_blocks, s);
      case kWidePair:
        return launch_wide_batched32_cfg<WdThin, WdGrpPair<1>, 2>(descs, count, total_blocks, s);
      default:
        return launch_wide_batched32_cfg<WdPair, WdGrpShort<1>, 4>(descs, count, total_blocks, s);
    }
  }
  if (max_m <= 32) {
    switch (wide_pick_batched32(total_blocks)) {
      case kWideThin: return launch_wide_batched32_cfg<WdThin, void, 2>(descs, count, total_blocks, s);
      case kWidePair: return launch_wide_batched32_cfg<WdPair, void, 4>(descs, count, total_blocks, s);
      default: return launch_wide_batched32_cfg<WdShort, void, 8>(descs, count, total_blocks, s);
    }
  }
  switch (wide_pick_batched(total_blocks, max_m)) {
    case kWideLong: return launch_wide_batched_cfg<WdLong>(descs, count, total_blocks, s);
    case kWideMid: return launch_wide_batched_cfg<WdMid>(descs, count, total_blocks, s);
    case kWideHalf: return launch_wide_batched_cfg<WdHalf>(descs, count, total_blocks, s);
    default: return launch_wide_batched_cfg<WdShort>(descs, count, total_blocks, s);
  }
}

}  // namespace sherry
