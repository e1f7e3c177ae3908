// Register-decoded int8-MFMA product (Eq. 2): every lone product of five and
// more tokens, and the grouped launches of more than 32.
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
// and stores.  They run smaller workgroups with K split over more waves, as
// the cost model below picks.
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
template <int MT_, int S_, int W_, int EU_>
struct WdCfg {
  static constexpr int MT = MT_, S = S_, W = W_, EU = EU_, RING = 4, NST = 4;
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
// N + 2u outstanding loads (u a constant once unrolled)
template <int N>
__device__ __forceinline__ void wd_wait_first(int u) {
  switch (u) {
    case 0: wd_wait_vm<wd_cap(N)>(); break;
    case 1: wd_wait_vm<wd_cap(N + 2)>(); break;
    case 2: wd_wait_vm<wd_cap(N + 4)>(); break;
    case 3: wd_wait_vm<wd_cap(N + 6)>(); break;
    case 4: wd_wait_vm<wd_cap(N + 8)>(); break;
    default: wd_wait_vm<wd_cap(N + 10)>(); break;
  }
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
template <int MT, int s, int l>
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
    c[0][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xv[tb], wl, c[0][tb], 0, 0, 0);
    c[1][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xv[tb], wh, c[1][tb], 0, 0, 0);
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
  const int U = (C + S - 1) / S;
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

  // the epilogue's scales, through LDS: loaded before anything else, since a
  // load between the stores would wait for every store before it
  float sxv = 0.0f, swv = 0.0f;
  if (tid < G::TOK) sxv = tid < p.m ? as_global(p.x_scale)[tid] : 0.0f;
  {
    const int row = g * G::TILES * kTileRows + tid;
    if (tid < G::TILES * kTileRows) swv = row < p.n ? p.ws.at(row) : 0.0f;
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
  if (tid < 32) lut[tid] = decode_word(tid);
  if (tid < G::TOK) xsl[tid] = sxv;
  if (tid < G::TILES * kTileRows) wsl[tid] = swv;
  wd_wait_vm<wd_cap((D - 1) * G::SPT + 2 * G::RING)>();
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
      wd_slice<MT, 0, 3>(wv, ring[u], lut, xv[0], xv[XD % XN], st + lo[XD], c);
      load_unit(ring[u], rs, jj + G::RING, lane);
      wd_slice<MT, 1, 0>(wv, dn, lut, xv[1], xv[(1 + XD) % XN], st + lo[1 + XD], c);
      // chunk jj + 1 has landed for every wave after this barrier, and every
      // wave is done with the stage of chunk jj - 1
      if (u < D - 1 && j == 0) wd_wait_first<(D - 2) * G::SPT + 2 * G::RING + 2>(u);
      else wd_wait_vm<wd_cap(2 * (D - 1) + (D - 2) * G::SPT)>();
      wd_barrier();
      if (jj + 1 == chl) clear_tail();
#pragma unroll
      for (int i = 0; i < G::SPT; ++i) dma(jj + D, i);
      wd_slice<MT, 2, 1>(wv, dn, lut, xv[2 % XN], xv[(2 + XD) % XN],
                         XD == 2 ? sn + lo[0] : st + lo[3], c);
      wd_slice<MT, 3, 2>(wv, dn, lut, xv[3 % XN], xv[(3 + XD) % XN], sn + lo[XD - 1], c);
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
  v16i f[HN][MT];  // owned sums (elements [0, EN))
  if constexpr (S == 1) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int tb = 0; tb < MT; ++tb) f[h][tb] = c[h][tb];
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
            red[(((wave * RT + tb) * 2 + h) * 16 + e) * 64 + lane] = c[h][t0 + tb][e];
      wd_lds_barrier();
      const int w0 = wave - sp;
#pragma unroll
      for (int tb = 0; tb < RT; ++tb)
#pragma unroll
        for (int e = 0; e < EN; ++e) {
          int32_t v = 0;
#pragma unroll
          for (int q = 0; q < S; ++q)
            v += red[((((w0 + q) * RT + tb) * 2 + hs) * 16 + es + e) * 64 + lane];
          f[0][t0 + tb][e] = v;
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
      swl[h][u] = wsl[(wave / S) * kTileRows + 32 * (hs + h) + 4 * c4 + u];
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
                     (!p.acc || reinterpret_cast<uintptr_t>(p.acc) % 16 == 0);
  const bool vec = (p.n % 4 == 0) && (reinterpret_cast<uintptr_t>(p.y) % 16 == 0) &&
                   (!p.acc || reinterpret_cast<uintptr_t>(p.acc) % 16 == 0);
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
      int32_t* ap = as_global_mut(p.acc) + at;
#pragma unroll
      for (int i = 0; i < PN; ++i) {
        float4 o4;
        o4.x = static_cast<float>(v[i].x) * (sx[i] * swl[h][0]);
        o4.y = static_cast<float>(v[i].y) * (sx[i] * swl[h][1]);
        o4.z = static_cast<float>(v[i].z) * (sx[i] * swl[h][2]);
        o4.w = static_cast<float>(v[i].w) * (sx[i] * swl[h][3]);
        *reinterpret_cast<float4*>(yp + int64_t(8 * i) * p.n) = o4;
        if (p.acc) *reinterpret_cast<v4i*>(ap + int64_t(8 * i) * p.n) = v[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < PN; ++i) {
        const int tok = 32 * tb + tokb + (lane >> 3) + 8 * i;
        if (tok >= p.m || row >= p.n) continue;
        const int32_t vv[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        float o4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) o4[u] = static_cast<float>(vv[u]) * (sx[i] * swl[h][u]);
        float* yrow = as_global_mut(p.y) + int64_t(tok) * p.n + row;
        if (vec) {
          *reinterpret_cast<float4*>(yrow) = make_float4(o4[0], o4[1], o4[2], o4[3]);
          if (p.acc) *reinterpret_cast<v4i*>(as_global_mut(p.acc) + int64_t(tok) * p.n + row) = v[i];
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (row + u >= p.n) break;
            yrow[u] = o4[u];
            if (p.acc) as_global_mut(p.acc)[int64_t(tok) * p.n + row + u] = vv[u];
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

// grid: x = groups of TILES tiles, y = token blocks
template <class G>
__global__ __launch_bounds__(G::THREADS) __attribute__((amdgpu_waves_per_eu(G::EU))) void wide_kernel(
    WdProblem p) {
  __shared__ __attribute__((aligned(16))) int8_t lds[G::LDS];
  wd_tokens<G>(p, int64_t(blockIdx.y) * G::TOK);
  wd_block<G>(p, blockIdx.x, lds);
}

// Grouped launch.  A prepared block is 8 tiles x 64 tokens of its product
// (token blocks outermost); it is run by 8 / TILES x 64 / TOK workgroups, or,
// with 128-token blocks, every two prepared blocks of one tile group (an even
// and the next token block) by two workgroups of four tiles each.
template <class G>
__global__ __launch_bounds__(G::THREADS) __attribute__((amdgpu_waves_per_eu(G::EU))) void wide_batched_kernel(
    const sherry_gemm_desc* __restrict__ descs, int count) {
  __shared__ __attribute__((aligned(16))) int8_t lds[G::LDS];
  constexpr int PER = G::PER;
  const int32_t blk = static_cast<int32_t>(blockIdx.x) / PER;
  const int sub = static_cast<int>(blockIdx.x) % PER;
  const int lo = find_block_desc(descs, count, blk);
  if (lo < 0) return;
  const sherry_gemm_desc& d = descs[lo];
  const int lb = blk - d.block_begin;
  const int R = (d.n + kTileRows - 1) / kTileRows;
  const int gb = (R + 7) / 8;  // tile groups of a prepared block
  int g, reps = 1;
  int64_t t0;
  if constexpr (G::TOK <= 64) {
    constexpr int RPB = 8 / G::TILES;  // workgroups along the rows
    const int tb = lb / gb;
    t0 = int64_t(tb) * 64 + sub / RPB * G::TOK;
    g = (lb - tb * gb) * RPB + sub % RPB;
  } else {
    static_assert(G::TOK == 128 && G::TILES == 4 && PER == 1, "two prepared blocks, two workgroups");
    const int T = (d.m + 63) / 64;
    const int pairs = T / 2 * 2 * gb;  // blocks of the paired token blocks
    const bool paired = lb < pairs;
    const int q = paired ? lb : 2 * (lb - pairs);  // the last, odd token block: both
    reps = paired ? 1 : 2;                         // halves of its tiles
    const int pr = paired ? q / (2 * gb) : T / 2;
    g = paired ? q - pr * 2 * gb : q;
    t0 = int64_t(pr) * 128;
  }
  if (t0 >= d.m) return;
  WdProblem p{d.w, d.x, d.x_scale, d.y, d.acc, d.n, d.k, d.m, WScale{d.w_scales, d.w_scale}};
  wd_tokens<G>(p, t0);
  for (int h = 0; h < reps; ++h) {
    if ((g + h) * G::TILES >= R) return;
    if (h) __syncthreads();  // the table, scales and strips are written again
    wd_block<G>(p, g + h, lds);
  }
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

// Estimated time (us) of a launch on one of them: the busiest CU runs c
// workgroups of U units per wave; a lone workgroup takes fix + lat U, bound
// by one wave's chain, and c of them base + c (thr U + o).  Fitted to
// measured launches (m 37-8192, n 300-14336, k 128-14336), which it orders
// right or within 5% of the best.
struct WdCost {
  float fix, lat, base, thr, o;
};
constexpr WdCost kWdLong{8.2f, 0.68f, 5.0f, 0.64f, 7.7f}, kWdMid{6.0f, 0.54f, 5.0f, 0.45f, 1.7f},
    kWdHalf{6.0f, 0.575f, 5.0f, 0.50f, 2.0f}, kWdQuarter{7.5f, 0.83f, 5.0f, 0.80f, 5.2f},
    kWdShort{5.0f, 0.55f, 4.0f, 0.41f, 1.1f}, kWdTiny{5.3f, 0.83f, 4.0f, 0.78f, 3.06f};
template <class G>
float wd_estimate(const WdCost& c, int64_t workgroups, int64_t units) {
  const float U = static_cast<float>(ceil_div(units, G::S));
  const float per = static_cast<float>(ceil_div(workgroups, 256));
  const float one = c.fix + c.lat * U, many = c.base + per * (c.thr * U + c.o);
  return one > many ? one : many;
}

}  // namespace

int launch_wide(const uint8_t* w, const int8_t* x, const float* x_scale, WScale ws, float* y,
                int32_t* acc, int64_t m, int64_t n, int64_t k, hipStream_t s) {
  const WdProblem p{w, x, x_scale, y, acc, static_cast<int>(n), static_cast<int>(k),
                    static_cast<int>(m), ws};
  const int64_t R = ceil_div(n, kTileRows), C = ceil_div(k, kTileK);
  int best = 0;
  float t = 0.0f;
  auto offer = [&](int id, float e) {
    if (id == 0 || e < t) t = e, best = id;
  };
  auto blocks = [&](int64_t tiles, int64_t tok) { return ceil_div(R, tiles) * ceil_div(m, tok); };
  offer(0, wd_estimate<WdLong>(kWdLong, blocks(4, 128), C));
  offer(1, wd_estimate<WdMid>(kWdMid, blocks(4, 64), C));
  offer(2, wd_estimate<WdHalf>(kWdHalf, blocks(2, 64), C));
  offer(3, wd_estimate<WdQuarter>(kWdQuarter, blocks(2, 64), C));
  offer(4, wd_estimate<WdShort>(kWdShort, blocks(1, 32), C));
  offer(5, wd_estimate<WdTiny>(kWdTiny, blocks(1, 32), C));
  switch (best) {
    case 0: return launch_wide_cfg<WdLong>(p, s);
    case 1: return launch_wide_cfg<WdMid>(p, s);
    case 2: return launch_wide_cfg<WdHalf>(p, s);
    case 3: return launch_wide_cfg<WdQuarter>(p, s);
    case 4: return launch_wide_cfg<WdShort>(p, s);
    default: return launch_wide_cfg<WdTiny>(p, s);
  }
}

template <class G>
int launch_wide_batched_cfg(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                            hipStream_t s) {
  return launch(wide_batched_kernel<G>, dim3(static_cast<unsigned>(total_blocks * G::PER)),
                dim3(G::THREADS), 0, s, descs, count);
}

// Grouped launches of 64-token blocks: the workgroup shape by the number of
// blocks (the rows' lengths are not known here; 24 units stand for them).
int launch_wide_batched(const sherry_gemm_desc* descs, int count, int64_t total_blocks,
                        int max_m, hipStream_t s) {
  constexpr int64_t kUnits = 24;
  int best = 0;
  float t = 0.0f;
  auto offer = [&](int id, float e) {
    if (id == 0 || e < t) t = e, best = id;
  };
  // (64 tokens of a 128-token workgroup's are idle in an odd last block)
  const int64_t T = ceil_div(max_m, 64);
  offer(0, wd_estimate<WdLong>(kWdLong, ceil_div(total_blocks * ((T + 1) / 2 * 2), T), kUnits));
  offer(1, wd_estimate<WdMid>(kWdMid, total_blocks * WdMid::PER, kUnits));
  offer(2, wd_estimate<WdHalf>(kWdHalf, total_blocks * WdHalf::PER, kUnits));
  offer(4, wd_estimate<WdShort>(kWdShort, total_blocks * WdShort::PER, kUnits));
  switch (best) {
    case 0: return launch_wide_batched_cfg<WdLong>(descs, count, total_blocks, s);
    case 1: return launch_wide_batched_cfg<WdMid>(descs, count, total_blocks, s);
    case 2: return launch_wide_batched_cfg<WdHalf>(descs, count, total_blocks, s);
    default: return launch_wide_batched_cfg<WdShort>(descs, count, total_blocks, s);
  }
}

}  // namespace sherry
