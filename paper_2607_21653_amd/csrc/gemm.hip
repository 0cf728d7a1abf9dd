// GEMMs of the verify step on gfx950 MFMA: dense projections (QKV, O, router, LM head)
// and the grouped expert GEMMs of the top-K routed MoE (gate_up with a fused SwiGLU
// epilogue, down), in bf16 (v_mfma_f32_32x32x16_bf16) or fp8 e4m3 with f32 per-row x
// per-channel scales (v_mfma_f32_32x32x64_f8f6f4), f32 accumulation.
//
// Every operand is in the tiled layout of device_common.h (weights packed once at load;
// activations written tiled by their producers, rows padded to a multiple of 32; the token
// rows of gate_up row-major). Kernels, in the order of this file: weight streaming
// (stream_gemm_kernel: grouped, and few rows by many columns), LDS-tiled (lds_gemm_kernel:
// dense), few rows (qkv_few_kernel), big tiles (bigtile_gemm_kernel: dense;
// grouped_bigtile_kernel: grouped) and f32 (f32_gemm_kernel: everything of the f32 model);
// gemm_plan and moe_plan choose. Grouped launches run over a device-side tile table (expert,
// first row, end row) in padded expert order built by the permutation kernel, so the host
// never reads expert counts.
#include <math.h>

#include <algorithm>

#include "device_common.h"
#include "internal.h"

namespace molt {
namespace {

constexpr int kThreads = 256;
constexpr int kBN = 128;         // output columns per tile (gate_up: 64 gate + 64 up)
constexpr int kRowBytes = 128;   // K-slice, bytes

enum Mode { kDense = 0, kGateUp = 1, kDown = 2 };

// s_waitcnt immediate: vmcnt(0), expcnt(7) and lgkmcnt(15) (no wait on those two)
constexpr int kWaitVmcnt0 = (7 << 4) | (15 << 8);

struct GemmParams {
  const void* A;           // dense: [M, K] tiled; gate_up: token rows, row-major; down: h [R, K] tiled
  const void* B;           // tiled. dense: [N, K]; gate_up: [E, 2F, K]; down: [E, N, K]
  void* C;                 // dense: f32 [M, ldc]; gate_up: h tiled [R, F]; down: f32 [P, ldc]
  int M, N, K;             // N: output columns (gate_up: F)
  int ldc;
  const int4* tiles;       // grouped: {expert, row0, row1, -}
  const int32_t* n_tiles_live;   // grouped (device): entries of `tiles` in use; null: n_mtiles
  int n_mtiles, n_ntiles;
  const int32_t* perm;     // grouped: padded row -> pair (token * ktop + slot), -1 = padding;
                           // null (dense down mode): row r -> output row r
  int ktop;
  const float* a_scale;    // fp8: per A row (token for gate_up, padded row for down)
  const float* b_scale;    // fp8: [E, b_scale_ld]
  int b_scale_ld;
  int accumulate;          // dense: C += result
  int* queue;              // grouped fp8: per-XCD tile queues (zero at launch)
};

MOLT_DEV floatx16_t mfma(const bf16x8_t& a, const bf16x8_t& b, const floatx16_t& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
MOLT_DEV floatx16_t mfma(const int32x8_t& a, const int32x8_t& b, const floatx16_t& c) {
  // cbsz = blgp = 0: both operands fp8 e4m3; zero scale operands select the unscaled op
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}

// ---------------------------------------------------------------- grouped expert GEMM
// Expert GEMMs are HBM-bound at the verify step's row counts (tens of rows per expert):
// the weights must stream at full bandwidth and be read once. Workgroup = BM rows of one
// expert x 128 output columns; each of the 4 wavefronts owns 32 output columns (32 weight
// rows) and loads its weight fragments straight from global memory into MFMA operand
// registers, 4 K slices (128 bytes each) ahead; a weight element is used by exactly one
// wavefront, so weights never touch LDS. The BM activation rows, shared by the 4
// wavefronts, go through a double-buffered LDS ring: per slice each thread copies one
// 16-byte chunk of each 4 KB activation block, loaded two slices ahead into registers; one
// LDS-only barrier per slice (it does not wait for the weight loads in flight).
// Both operands are in the tiled layout, so every global load instruction reads 1 KB of
// one page (with row-major operands each instruction touched 32 rows, and the address
// translation requests, not HBM, set the pace) and every LDS fragment read is a
// contiguous 1 KB. Tiles start at multiples of 32 rows (padded expert order), so each
// 32-row block of A is one tile column of the tiled activation buffer.
// The grid is persistent (see stream_gemm_kernel) and, for the bf16 down GEMM when the K
// slices come in multiples of 4, chained: the last steps of a tile issue the first weight and activation
// loads of the workgroup's next tile into the slots where its prologue would put them, so
// a tile starts with its first 4 slices in flight or landed instead of waiting out a fresh
// HBM latency (an unchained tile carried a fixed cost of about a fifth of its time).
// Nothing after those loads waits for them before the next tile's first step: the
// epilogues use LDS-only barriers, and down reads its output rows' pair indices from LDS,
// copied there early in the tile.
struct Slice16 { int32x4_t c[4]; };   // one lane's 64 bytes of a 32-row x 128-byte tile

// Where one (m-tile, n-tile) pair of a grouped launch reads (all wavefront-uniform).
struct StreamTile {
  const uint8_t* b;     // the wavefront's 32 weight rows (gate_up: waves 0-1 gate, 2-3 up)
  const uint8_t* a;     // the tile's first 32-row activation block
  int a_last;           // its last 32-row block that holds rows (0 .. BM / 32 - 1)
  int rot;              // first K slice visited
  int expert, row0, row1, n0;
};

template <int MODE>
MOLT_DEV StreamTile stream_geometry(const GemmParams& p, int id, int nk, int wave) {
  StreamTile g;
  const int mt = id / p.n_ntiles, nt = id % p.n_ntiles;
  // through the constant address space: a scalar load (the table is read-only here), which
  // does not wait behind the vector stores of an epilogue
  typedef const __attribute__((address_space(4))) int32x4_t* ConstTile;
  int4 t = make_int4(0, 0, p.M, 0);                   // no table: one dense row tile
  if (p.tiles != nullptr) {
    const int32x4_t tv = *(ConstTile)(p.tiles + mt);
    t = make_int4(tv[0], tv[1], tv[2], tv[3]);
  }
  g.expert = t.x;
  g.row0 = t.y;                                       // a multiple of 32
  g.row1 = t.z;
  const long RB = long(nk) * kRowBytes;               // bytes per operand row
  long wrow;
  if (MODE == kGateUp) {
    g.n0 = nt * (kBN / 2);
    wrow = long(g.expert) * 2 * p.N + (wave < 2 ? g.n0 + 32 * wave : p.N + g.n0 + 32 * (wave - 2));
  } else {
    g.n0 = nt * kBN;
    // N is a multiple of 64: in a half column tile the last two wavefronts repeat the last rows
    // (their columns are not stored)
    wrow = long(g.expert) * p.N + min(g.n0 + 32 * wave, p.N - 32);
  }
  g.b = static_cast<const uint8_t*>(p.B) + wrow * RB;
  g.a = static_cast<const uint8_t*>(p.A) + long(g.row0) * RB;
  g.a_last = (((g.row1 - 1) & ~31) - g.row0) / 32;
  // K slices are visited in an order rotated by the column tile, so the workgroups of one
  // row tile (running side by side on one XCD) read different activation blocks at any
  // moment instead of all hitting the same L2 lines
  g.rot = int((long(nt) * nk) / p.n_ntiles);
  return g;
}

// Persistent grouped GEMM: the grid is what the chip holds at once (a multiple of 8, see
// run_stream). Workgroup b runs on XCD b % 8 and walks that XCD's contiguous eighth of the
// live (m-tile, n-tile) pairs, m-tile major, with the XCD's workgroup count as stride: the
// n-tiles of one row tile run side by side on one XCD, so its activation tile is read from
// HBM once and then hits that XCD's L2. Launching one workgroup per pair left the chip
// at 50-80% of its resident workgroups on average (dispatch gaps between short tiles).
// CHAIN requires K slices in multiples of 4 (the slot pattern then lines up across tiles).
// fp8 launches take each workgroup's later tiles from its XCD's queue instead (see below).
template <int BM, bool FP8, int MODE, bool CHAIN, bool ROWS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(BM <= 64 ? 3 : 2)))
void stream_gemm_kernel(GemmParams p) {
  static_assert(MODE == kGateUp || MODE == kDown, "grouped modes");
  static_assert(!ROWS || (MODE == kGateUp && !CHAIN), "row gather: gate_up");
  constexpr int MS = BM / 32;                        // 32-row MFMA tiles per wavefront
  constexpr int kElem = FP8 ? 1 : 2;
  // weight slices in flight per wavefront (each 4 KB slice of a wavefront's 32 weight rows
  // is 16 registers; 8 in flight measured slower than 4)
  constexpr int WD = 4;
  // activation staging: 2 buffers of MS 4 KB blocks; gate_up's epilogue reuses them, with
  // the space after them, as a BM x 128 f32 tile (2 * BM * 256 bytes)
  __shared__ __attribute__((aligned(16))) uint8_t smem[(MODE == kGateUp ? 4 : 2) * MS * 4096];
  uint8_t (*alds)[MS * 4096] = reinterpret_cast<uint8_t (*)[MS * 4096]>(smem);
  __shared__ int prow[MODE == kDown ? BM : 1];       // down: pair index of each tile row
  // down epilogue: the tile's outputs (BM x 128 f32; 128-row tiles in two 64-column passes)
  constexpr int kEpCols = BM == 128 ? 64 : 128;
  __shared__ __attribute__((aligned(16))) float dep[MODE == kDown ? BM * kEpCols : 1];
  const int total = (p.n_tiles_live != nullptr ? *p.n_tiles_live : p.n_mtiles) * p.n_ntiles;
  const int chunk = (total + 7) / 8;
  const int stride = gridDim.x / 8;
  const int first = (blockIdx.x % 8) * chunk;
  int k8 = blockIdx.x / 8;
  if (k8 >= chunk || first + k8 >= total) return;
  const int nk = int(long(p.K) * kElem / kRowBytes);  // 128-byte K slices
  const long RB = long(nk) * kRowBytes;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const unsigned boff = lane * 16u, aoff = threadIdx.x * 16u;
  auto slice = [&](const StreamTile& t, int kb) __attribute__((always_inline)) {
    const int k = min(kb, nk - 1) + t.rot;
    return long(k >= nk ? k - nk : k) * 4096;
  };
  // weights are read once per step: nontemporal loads
  auto wld = [&](Slice16& f, const StreamTile& t, int kb) __attribute__((always_inline)) {
    const uint8_t* src = t.b + slice(t, kb) + boff;
#pragma unroll
    for (int c = 0; c < 4; ++c) f.c[c] = __builtin_nontemporal_load(reinterpret_cast<const int32x4_t*>(src + 1024 * c));
  };
  // ROWS: thread t copies piece t % 8 (16 bytes) of row t / 8 of each 32-row block from the
  // token's row-major row (roff: its byte offset, set per tile), so each load instruction
  // reads 8 whole 128-byte row slices; in LDS the row's 8 pieces sit at piece ^ swz(row)
  // (conflict-free fragment reads and stores)
  long roff[ROWS ? MS : 1];
  const unsigned rsto = ROWS ? (threadIdx.x / 8) * 128 + ((threadIdx.x % 8) ^ ((threadIdx.x / 16) % 8)) * 16
                             : threadIdx.x * 16;
#define MOLT_GLOAD(ST, T, KB)                                                         \
  {                                                                                   \
    const long off_ = slice(T, KB);                                                   \
    if (ROWS) {                                                                       \
      _Pragma("unroll") for (int b_ = 0; b_ < MS; ++b_)                               \
          ST[b_] = *reinterpret_cast<const int32x4_t*>(static_cast<const uint8_t*>(p.A) + roff[b_ % (ROWS ? MS : 1)] + (off_ >> 5) + (threadIdx.x % 8) * 16); \
    } else {                                                                          \
      _Pragma("unroll") for (int b_ = 0; b_ < MS; ++b_)                               \
          ST[b_] = *reinterpret_cast<const int32x4_t*>((T).a + long(min(b_, (T).a_last)) * 32 * RB + off_ + aoff); \
    }                                                                                 \
  }
#define MOLT_SSTORE(ST, BUF)                                                          \
  {                                                                                   \
    _Pragma("unroll") for (int b_ = 0; b_ < MS; ++b_)                                 \
        *reinterpret_cast<int32x4_t*>(&alds[BUF][b_ * 4096 + rsto]) = ST[b_];         \
  }
  // ROWS fragment reads: lane l takes row l % 32, piece 4 (l / 32) + c for k-step c
  const unsigned rsw = (4 * (lane / 32)) ^ ((lane % 32 / 2) % 8);
  int32x4_t st0[MS], st1[MS];
  Slice16 wb[WD];
  floatx16_t acc[MS];
  StreamTile g = stream_geometry<MODE>(p, first + k8, nk, wave);
  StreamTile gn = g;
  bool more = false;
  bool primed = false;                               // g's first slices already loaded
  // fp8 launches take tiles from their XCD's queue: a workgroup's first tile is k8 as in the
  // static walk, each later one the next of the pool [stride, chunk), taken by thread 0 when
  // the tile enters its last K steps and passed on through LDS in the epilogue, so
  // workgroups that run faster take more tiles (the static walk left an XCD's workgroups
  // ending anywhere between half and all of the kernel's time). Their Zipf-hot tiles are
  // bound by the MFMAs and differ in cost; the bf16 launches are bound by HBM, where the
  // late workgroups still share the full bandwidth and the queue measured 0-5% slower.
  constexpr bool kDyn = FP8 && !CHAIN;
  const bool dyn = kDyn && p.queue != nullptr;
  __shared__ int s_grab;
  int grab = chunk;                                  // thread 0: the next tile (dyn)
  for (;;) {
    // down: the pair index of each of the tile's rows, loaded before the tile's own loads
    int pv = -1;
    if (MODE == kDown && threadIdx.x < BM && g.row0 + int(threadIdx.x) < g.row1)
      pv = p.perm != nullptr ? p.perm[g.row0 + threadIdx.x] : g.row0 + int(threadIdx.x);
    auto put_prow = [&]() __attribute__((always_inline)) {
      if (MODE == kDown && threadIdx.x < BM) prow[threadIdx.x] = pv;
    };
    if (!dyn) {
      const int kn = k8 + stride;
      more = kn < chunk && first + kn < total;
      // the next tile's table entry is read here, not after the epilogue
      if (more) gn = stream_geometry<MODE>(p, first + kn, nk, wave);
    }
    if (ROWS) {
      // rows past the tile's end (and padding rows) read token 0: their outputs are not stored
#pragma unroll
      for (int b_ = 0; b_ < MS; ++b_) {
        const int r = g.row0 + 32 * b_ + int(threadIdx.x / 8);
        const int pr = r < g.row1 ? p.perm[r] : -1;
        roff[b_ % (ROWS ? MS : 1)] = pr < 0 ? 0 : long(pr / p.ktop) * RB;
      }
    }
    if (!primed) {
      MOLT_GLOAD(st0, g, 0);
      MOLT_GLOAD(st1, g, 1);
#pragma unroll
      for (int s = 0; s < WD; ++s) wld(wb[s], g, s);
      // gate_up: every wavefront is done reading the last tile's epilogue tile from LDS
      if (MODE == kGateUp && k8 != int(blockIdx.x / 8)) lds_barrier();
      MOLT_SSTORE(st0, 0);
      MOLT_GLOAD(st0, g, 2);
      lds_barrier();
    }

#pragma unroll
    for (int i = 0; i < MS; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    // Step over slice k: LDS buffer U holds its activations, weight slot W its weights,
    // register slot ST_NEXT slice k + 1 (the other slot k + 2). It computes, refills W with
    // slice k + WD, stores slice k + 1 into buffer 1 - U (last read before the previous
    // barrier) and refills ST_NEXT with slice k + 3. In the last WD + 3 steps (TAIL = 1) a
    // refill past the end loads the next tile's slice (chained) or nothing: re-reading the
    // last slice instead cost the 12-slice down GEMM a third more weight loads. fp8: the
    // refills and the activation copy run at raised wave priority, so they issue ahead of
    // the other wavefronts' MFMAs (fp8 Zipf MoE layer 380 -> 370 us; bf16 unchanged).
#define MOLT_STEP(U, ST_NEXT, W, K, TAIL)                                                           \
  {                                                                                                  \
    const uint8_t* base_ = alds[U] + (ROWS ? (lane % 32) * 128 : lane * 16);                         \
    if (!FP8) {                                                                                      \
      _Pragma("unroll") for (int c = 0; c < 4; ++c) {                                                \
        const bf16x8_t bv = *reinterpret_cast<const bf16x8_t*>(&wb[W].c[c]);                         \
        const unsigned fo_ = ROWS ? ((rsw ^ c) * 16) : c * 1024;                                     \
        _Pragma("unroll") for (int i = 0; i < MS; ++i) acc[i] =                                      \
            mfma(*reinterpret_cast<const bf16x8_t*>(base_ + i * 4096 + fo_), bv, acc[i]);            \
      }                                                                                              \
    } else {                                                                                         \
      _Pragma("unroll") for (int c = 0; c < 2; ++c) {                                                \
        const int32x4_t w0 = wb[W].c[2 * c], w1 = wb[W].c[2 * c + 1];                                \
        const int32x8_t bv = int32x8_t{w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3]};     \
        const unsigned lo_ = ROWS ? ((rsw ^ (2 * c)) * 16) : 2 * c * 1024;                          \
        const unsigned hi_ = ROWS ? ((rsw ^ (2 * c + 1)) * 16) : (2 * c + 1) * 1024;                \
        _Pragma("unroll") for (int i = 0; i < MS; ++i) {                                             \
          const int32x4_t lo = *reinterpret_cast<const int32x4_t*>(base_ + i * 4096 + lo_);          \
          const int32x4_t hi = *reinterpret_cast<const int32x4_t*>(base_ + i * 4096 + hi_);          \
          acc[i] = mfma(int32x8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}, bv, acc[i]); \
        }                                                                                            \
      }                                                                                              \
    }                                                                                                \
    if (FP8) __builtin_amdgcn_s_setprio(3);                                                          \
    if (!(TAIL) || (K) + WD < nk) wld(wb[W], g, (K) + WD);                                           \
    else if (CHAIN && more) wld(wb[W], gn, (K) + WD - nk);                                           \
    MOLT_SSTORE(ST_NEXT, 1 - (U));                                                                   \
    if (!(TAIL) || (K) + 3 < nk) MOLT_GLOAD(ST_NEXT, g, (K) + 3)                                     \
    else if (CHAIN && more) MOLT_GLOAD(ST_NEXT, gn, (K) + 3 - nk)                                    \
    if (FP8) __builtin_amdgcn_s_setprio(0);                                                          \
    lds_barrier();                                                                                   \
  }
    static_assert(WD == 4, "the step sequence cycles through 4 weight slots");
    int kb = 0;
    for (; kb + WD + 3 < nk; kb += 4) {    // every refill of these 4 steps is in this tile
      MOLT_STEP(0, st1, 0, kb, 0);
      if (kb == 0) put_prow();             // waits for the row load, not for the step's own
      MOLT_STEP(1, st0, 1, kb + 1, 0);
      MOLT_STEP(0, st1, 2, kb + 2, 0);
      MOLT_STEP(1, st0, 3, kb + 3, 0);
    }
    if (kb == 0) {                         // no full 4 steps: a chained tile has had no
      if (primed) lds_barrier();           // barrier since the last tile's epilogue read prow
      put_prow();
    }
    if (dyn && threadIdx.x == 0) grab = stride + atomicAdd(p.queue + blockIdx.x % 8, 1);
    // the last 1..7 slices (kb % 4 == 0, so the slot pattern continues)
    if (kb < nk) MOLT_STEP(0, st1, 0, kb, 1);
    if (kb + 1 < nk) MOLT_STEP(1, st0, 1, kb + 1, 1);
    if (kb + 2 < nk) MOLT_STEP(0, st1, 2, kb + 2, 1);
    if (kb + 3 < nk) MOLT_STEP(1, st0, 3, kb + 3, 1);
    if (kb + 4 < nk) MOLT_STEP(0, st1, 0, kb + 4, 1);
    if (kb + 5 < nk) MOLT_STEP(1, st0, 1, kb + 5, 1);
    if (kb + 6 < nk) MOLT_STEP(0, st1, 2, kb + 6, 1);
#undef MOLT_STEP
    // published by the epilogue's first barrier, read after the tile
    if (dyn && threadIdx.x == 0) s_grab = grab;
    // accumulator element e of lane (lcol, lgrp) in tile i: row 32 i + 8 (e / 4) + 4 lgrp + e % 4
    int lcol = lane % 32, lgrp = lane / 32;
    // opaque per tile: the epilogue's address arithmetic stays here instead of being hoisted
    // out of the tile loop into registers held across the K steps (gate_up spilled them)
    asm volatile("" : "+v"(lcol), "+v"(lgrp));
    if (MODE == kGateUp) {
      // h = silu(gate) * up, bf16, tiled layout over padded rows. The accumulators go to LDS
      // as a BM x 128 tile (gate columns 0-63 from wavefronts 0-1, up columns 64-127 from
      // 2-3; the last step's barrier freed the staging buffers); then each thread finishes
      // 8 consecutive columns of a row per pass and writes them with one 16-byte store.
      float* ep = reinterpret_cast<float*>(smem);
#pragma unroll
      for (int i = 0; i < MS; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) ep[(32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4)) * 128 + 32 * wave + lcol] = acc[i][e];
      // fp8 scales of the thread's units (its 8 columns are the same in every unit) are all
      // loaded before the first store: a load issued after a store has to wait for it
      float sxv[MS];
      float4 swv[4];
      if (FP8) {
        const float* sw = p.b_scale + long(g.expert) * p.b_scale_ld + g.n0 + (threadIdx.x & 7) * 8;
        swv[0] = *reinterpret_cast<const float4*>(sw);
        swv[1] = *reinterpret_cast<const float4*>(sw + 4);
        swv[2] = *reinterpret_cast<const float4*>(sw + p.N);
        swv[3] = *reinterpret_cast<const float4*>(sw + p.N + 4);
        int pr[MS];
#pragma unroll
        for (int j = 0; j < MS; ++j) {
          const int grow = g.row0 + int((threadIdx.x + kThreads * j) >> 3);
          pr[j] = grow < g.row1 ? p.perm[grow] : 0;
        }
#pragma unroll
        for (int j = 0; j < MS; ++j) sxv[j] = p.a_scale[pr[j] / p.ktop];
      }
      lds_barrier();
      // the scales are in before the first store: with the stores behind per-unit branches the
      // compiler would otherwise wait for every earlier store before each unit's scale use
      // (s_waitcnt vmcnt(0), expcnt and lgkmcnt left open)
      if (FP8) __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      const long hrb = 2L * p.N;
#pragma unroll
      for (int j = 0; j < MS; ++j) {
        const int u = int(threadIdx.x) + kThreads * j;   // BM * 8 units of 8 columns
        const int r = u >> 3, cb = (u & 7) * 8;
        const int grow = g.row0 + r;
        if (grow >= g.row1) continue;
        const float4* gp = reinterpret_cast<const float4*>(ep + r * 128 + cb);
        const float4* up = reinterpret_cast<const float4*>(ep + r * 128 + 64 + cb);
        const float4 g0 = gp[0], g1 = gp[1], u0 = up[0], u1 = up[1];
        float gv[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        float uv[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        if (FP8) {
          const float sx = sxv[j];
          const float swg[8] = {swv[0].x, swv[0].y, swv[0].z, swv[0].w, swv[1].x, swv[1].y, swv[1].z, swv[1].w};
          const float swu[8] = {swv[2].x, swv[2].y, swv[2].z, swv[2].w, swv[3].x, swv[3].y, swv[3].z, swv[3].w};
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            gv[q] *= sx * swg[q];
            uv[q] *= sx * swu[q];
          }
        }
        uint32_t packed[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          packed[q] = uint32_t(f32_to_bf16(silu(gv[2 * q]) * uv[2 * q])) |
                      (uint32_t(f32_to_bf16(silu(gv[2 * q + 1]) * uv[2 * q + 1])) << 16);
        *reinterpret_cast<int32x4_t*>(static_cast<uint8_t*>(p.C) + tiled_offset(grow, 2L * (g.n0 + cb), hrb)) =
            int32x4_t{int(packed[0]), int(packed[1]), int(packed[2]), int(packed[3])};
      }
    } else {
      // per-pair expert output, f32, row = pair index (token * K + slot). Through LDS, so
      // that each thread writes 4 consecutive columns of a row with one 16-byte store.
      constexpr int kUnits = BM * kEpCols / 4;         // 4-column units per pass
      static_assert(kThreads % (kEpCols / 4) == 0, "a thread's columns are fixed per pass");
      // fp8: the thread's row and channel scales, all loaded before the first store
      float sxd[kUnits / kThreads];
      float4 swd[128 / kEpCols];
      if (FP8) {
        const int c4 = int(threadIdx.x % (kEpCols / 4)) * 4;
#pragma unroll
        for (int q = 0; q < 128 / kEpCols; ++q)
          swd[q] = *reinterpret_cast<const float4*>(p.b_scale + long(g.expert) * p.b_scale_ld + g.n0 + q * kEpCols + c4);
#pragma unroll
        for (int j = 0; j < kUnits / kThreads; ++j) {
          const int grow = g.row0 + int((threadIdx.x + kThreads * j) / (kEpCols / 4));
          sxd[j] = grow < g.row1 ? p.a_scale[grow] : 0.f;
        }
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);   // in before the first store (see gate_up)
      }
#pragma unroll
      for (int pass = 0; pass < 128 / kEpCols; ++pass) {
        const int c0 = pass * kEpCols;                 // first column of this pass
        if (32 * wave >= c0 && 32 * wave < c0 + kEpCols) {
#pragma unroll
          for (int i = 0; i < MS; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              dep[(32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4)) * kEpCols + 32 * wave - c0 + lcol] = acc[i][e];
        }
        lds_barrier();
        auto unit = [&](int j) __attribute__((always_inline)) {
          const int u = int(threadIdx.x) + kThreads * j;
          const int r = u / (kEpCols / 4), c4 = (u % (kEpCols / 4)) * 4;
          const int grow = g.row0 + r;
          if (grow >= g.row1 || g.n0 + c0 + c4 >= p.N) return;
          float4 v = *reinterpret_cast<const float4*>(dep + r * kEpCols + c4);
          const int c = g.n0 + c0 + c4;
          if (FP8) {
            const float sx = sxd[j];
            const float4 sw = swd[pass];
            v.x *= sx * sw.x;
            v.y *= sx * sw.y;
            v.z *= sx * sw.z;
            v.w *= sx * sw.w;
          }
          *reinterpret_cast<float4*>(static_cast<float*>(p.C) + long(prow[r]) * p.ldc + c) = v;
        };
        if constexpr (FP8) {
#pragma unroll
          for (int j = 0; j < kUnits / kThreads; ++j) unit(j);
        } else {
#pragma unroll 4
          for (int j = 0; j < kUnits / kThreads; ++j) unit(j);
        }
        if (pass + 1 < 128 / kEpCols) lds_barrier();
      }
    }
    if (dyn) {
      k8 = s_grab;
      if (k8 >= chunk || first + k8 >= total) break;
      g = stream_geometry<MODE>(p, first + k8, nk, wave);
      continue;
    }
    if (!more) break;
    k8 += stride;
    g = gn;
    primed = CHAIN;
  }
#undef MOLT_SSTORE
#undef MOLT_GLOAD
}

// Workgroups of `kernel` (`threads` each) resident on the whole device at once, rounded
// down to a multiple of 8 (>= 8).
template <typename K>
int resident_grid(K kernel, int threads = kThreads) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess)
    return 8;
  return (cus * per_cu) / 8 * 8 > 8 ? (cus * per_cu) / 8 * 8 : 8;
}

template <bool FP8, int MODE, bool CHAIN, bool ROWS = false>
hipError_t run_stream_k(GemmParams p, int tile_m, hipStream_t s) {
  // resident workgroups per kernel, queried once per process (one device model)
  static const int r32 = resident_grid(stream_gemm_kernel<32, FP8, MODE, CHAIN, ROWS>);
  static const int r64 = resident_grid(stream_gemm_kernel<64, FP8, MODE, CHAIN, ROWS>);
  static const int r128 = resident_grid(stream_gemm_kernel<128, FP8, MODE, CHAIN, ROWS>);
  const int pairs = (p.n_mtiles * p.n_ntiles + 7) / 8 * 8;   // upper bound of the live pairs
  const int cap = tile_m == 32 ? r32 : tile_m == 64 ? r64 : r128;
  const int grid = pairs < cap ? pairs : cap;
  if (tile_m == 32) stream_gemm_kernel<32, FP8, MODE, CHAIN, ROWS><<<grid, kThreads, 0, s>>>(p);
  else if (tile_m == 64) stream_gemm_kernel<64, FP8, MODE, CHAIN, ROWS><<<grid, kThreads, 0, s>>>(p);
  else stream_gemm_kernel<128, FP8, MODE, CHAIN, ROWS><<<grid, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

template <bool FP8, int MODE>
hipError_t run_stream(GemmParams p, int tile_m, hipStream_t s) {
  const long nk = long(p.K) * (FP8 ? 1 : 2) / kRowBytes;
  // chained in bf16 for down only: its 12-slice tiles gained (85 -> 82 us per launch at
  // T*K = 5120), gate_up's 32-slice tiles did not (159 -> 161 us)
  if constexpr (!FP8 && MODE == kDown)
    if (nk % 4 == 0) return run_stream_k<false, MODE, true>(p, tile_m, s);
  return run_stream_k<FP8, MODE, false, MODE == kGateUp>(p, tile_m, s);
}

// ---------------------------------------------------------------- LDS-tiled dense GEMM
// Dense projections of a few hundred rows: every weight tile feeds
// several row tiles and every activation tile many column tiles, so both operands are
// shared through LDS. Workgroup = BM x 128 outputs, wavefronts in a 2 x WN grid. Per
// 128-byte K slice the workgroup copies (BM/32 + 4) tiled 4 KB blocks (one 16-byte chunk
// per thread per block: coalesced 4 KB loads from one page) into a double-buffered LDS
// ring, loaded two slices ahead into registers; the tiled layout makes each wavefront's
// MFMA fragment a contiguous 1 KB LDS read (conflict-free, no padding). One barrier per
// slice. Split-K: split s covers slices [s * nk / S, (s + 1) * nk / S) and writes its
// partial sums to `part[s]`; a fixed-order reduction adds them (deterministic).
// Epilogue of the QKV projection with RoPE and the paged-KV write fused in (head_dim 128:
// output column tile nt is head nt; q heads, then k heads, then v heads).
struct RopeKv {
  const double2* table;     // [T][64] {cos, sin} of each token's position
  const int32_t* slot;      // [T] KV-cache slot of token t: block * 16 + position % 16, or -1
  int Hq, Hkv;
  uint16_t* q;              // [T, Hq, 128] bf16
  uint16_t* kc;             // [num_blocks, Hkv, 16, 128]
  uint16_t* vc;             // [num_blocks, Hkv, 128, 16]
};

template <int BM, bool ROPE, int WN, int DEPTH>
__global__ __launch_bounds__(128 * WN) void lds_gemm_kernel(GemmParams p, float* part, int splits,
                                                            RopeKv rk) {
  constexpr int NT = 128 * WN;                // 2 x WN wavefronts
  constexpr int AB = BM / 32;                 // activation row blocks
  constexpr int NB = AB + 4;                  // 4 KB blocks per slice (A then B)
  constexpr int CPT = NB * 256 / NT;          // 16-byte chunks per thread per slice
  constexpr int TM = BM / 64 > 0 ? BM / 64 : 1;   // 32-row MFMA tiles per wavefront
  constexpr int WROWS = 32 * TM;              // rows per wavefront
  constexpr int NJ = 4 / WN;                  // 32-column MFMA tiles per wavefront
  static_assert(BM == 64 || BM == 128, "BM");
  static_assert((NB * 256) % NT == 0, "chunks per thread");
  __shared__ __attribute__((aligned(16))) uint8_t lds[2][NB * 4096];

  const int total = p.n_mtiles * p.n_ntiles * splits;
  const int chunk = (total + 7) / 8;
  const int k8 = blockIdx.x / 8;
  const int id = (blockIdx.x % 8) * chunk + k8;   // XCD-contiguous; split, n-tile, m-tile
  if (k8 >= chunk || id >= total) return;
  const int mt = id % p.n_mtiles;
  const int nt = (id / p.n_mtiles) % p.n_ntiles;
  const int split = id / (p.n_mtiles * p.n_ntiles);
  const int row0 = mt * BM, n0 = nt * kBN;
  const long RB = long(p.K) * 2;
  const int nk = int(RB / kRowBytes);
  const int kb0 = int(long(nk) * split / splits), kb1 = int(long(nk) * (split + 1) / splits);
  // RoPE epilogue: this thread's row's KV-cache slot, read before the K loop (loaded at the
  // epilogue it would wait behind the table loads there)
  int my_slot = -1;
  if constexpr (ROPE) my_slot = rk.slot[min(row0 + int(threadIdx.x % BM), p.M - 1)];

  // chunk q = tid + NT u of a slice is 16-byte chunk q % 256 of block q / 256 (A blocks,
  // then B blocks; each a 4 KB tile, clamped into the padded operands); it lands at byte
  // 16 q of the slice's LDS buffer
  const uint8_t* src[CPT];
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int q = int(threadIdx.x) + NT * u, b = q / 256;
    const int last_a = (p.M - 1) & ~31, last_b = (p.N - 1) & ~31;
    const long r = b < AB ? min(row0 + 32 * b, last_a) : min(n0 + 32 * (b - AB), last_b);
    src[u] = static_cast<const uint8_t*>(b < AB ? p.A : p.B) + r * RB + (q % 256) * 16;
  }
  // register slots of DEPTH slices in flight (native vector type: HIP's int4 struct copied
  // into LDS made the compiler keep these arrays in scratch memory)
  int32x4_t st[DEPTH][CPT];
#define MOLT_GLOAD(ST, KB)                                                            \
  {                                                                                   \
    const long off_ = long(min((KB), kb1 - 1)) * 4096;                                \
    _Pragma("unroll") for (int b_ = 0; b_ < CPT; ++b_)                                \
        ST[b_] = *reinterpret_cast<const int32x4_t*>(src[b_] + off_);                 \
  }
#define MOLT_SSTORE(ST, BUF)                                                          \
  {                                                                                   \
    _Pragma("unroll") for (int b_ = 0; b_ < CPT; ++b_)                                \
        *reinterpret_cast<int32x4_t*>(&lds[BUF][(threadIdx.x + NT * b_) * 16]) = ST[b_]; \
  }
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int wm = wave / WN, wn = wave % WN;     // wavefront rows wm*WROWS.., cols wn*32*NJ..
  floatx16_t acc[TM][NJ];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll
  for (int j = 0; j < DEPTH; ++j) MOLT_GLOAD(st[j], kb0 + j);
  MOLT_SSTORE(st[0], 0);
  MOLT_GLOAD(st[0], kb0 + DEPTH);
  lds_barrier();
  // Step J (mod DEPTH) over slice k: LDS buffer k % 2 holds slice k, register slot
  // (J + 1) % DEPTH slice k + 1 (loaded DEPTH steps earlier). It computes, stores slice
  // k + 1 into the other buffer (last read before the previous barrier) and refills that
  // slot with slice k + 1 + DEPTH. Loads past the end re-read the last slice.
#define MOLT_STEP(J, K)                                                                           \
  {                                                                                                \
    const uint8_t* base_ = lds[(J) & 1];                                                           \
    _Pragma("unroll") for (int c = 0; c < 4; ++c) {                                                \
      bf16x8_t af[TM], bfr[NJ];                                                                    \
      _Pragma("unroll") for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(   \
          base_ + ((wm * WROWS) / 32 + i) * 4096 + c * 1024 + lane * 16);                          \
      _Pragma("unroll") for (int j = 0; j < NJ; ++j) bfr[j] = *reinterpret_cast<const bf16x8_t*>(  \
          base_ + (AB + wn * NJ + j) * 4096 + c * 1024 + lane * 16);                               \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                               \
          _Pragma("unroll") for (int j = 0; j < NJ; ++j) acc[i][j] = mfma(af[i], bfr[j], acc[i][j]); \
    }                                                                                              \
    MOLT_SSTORE(st[((J) + 1) % DEPTH], 1 - ((J) & 1));                                             \
    MOLT_GLOAD(st[((J) + 1) % DEPTH], (K) + 1 + DEPTH);                                            \
    lds_barrier();                                                                                 \
  }
  static_assert(DEPTH % 2 == 0, "LDS buffer parity follows the slot index");
  int kb = kb0;
  for (; kb + DEPTH - 1 < kb1; kb += DEPTH) {   // loads are clamped, never behind a branch
#pragma unroll
    for (int J = 0; J < DEPTH; ++J) MOLT_STEP(J, kb + J);
  }
#pragma unroll
  for (int J = 0; J < DEPTH - 1; ++J)
    if (kb + J < kb1) MOLT_STEP(J, kb + J);
#undef MOLT_STEP
#undef MOLT_SSTORE
#undef MOLT_GLOAD

  // acc[i][j][e]: row wm*WROWS + 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4,
  // col wn*32*NJ + 32 j + lane % 32
  const int lcol = lane % 32, lgrp = lane / 32;
  if constexpr (ROPE) {
    // The f32 tile goes through the (now idle) LDS ring so that each rotation pair (i, i + 64)
    // meets in one thread; the rotation is done in f64 with the step's cos/sin table. The
    // table entries and cache slots are fetched first, so their latency overlaps the exchange.
    // thread (pr, pi) rotates pair pi of rows pr + PR n, n < BM / PR, in groups of RG rows
    constexpr int PR = NT / 64;
    constexpr int RG = BM / PR < 16 ? BM / PR : 16;
    constexpr int NG = BM / (PR * RG);
    const int h = nt, pi = threadIdx.x % 64, pr = threadIdx.x / 64;
    const bool rotate = h < rk.Hq + rk.Hkv;
    double2 cs[RG];
    auto fetch = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < RG; ++n)
        cs[n] = rk.table[long(min(row0 + pr + PR * (RG * g + n), p.M - 1)) * 64 + pi];
    };
    __shared__ int s_slot[BM];
    if (rotate) fetch(0);
    if (threadIdx.x < BM) s_slot[threadIdx.x] = row0 + int(threadIdx.x) < p.M ? my_slot : -1;
    __syncthreads();
    float* ob = reinterpret_cast<float*>(&lds[0][0]);     // [BM][128]
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          ob[(wm * WROWS + 32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4)) * 128 + wn * 32 * NJ + 32 * j + lcol] =
              acc[i][j][e];
    __syncthreads();
    if (rotate) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g > 0) fetch(g);
        // all of the group's table entries in before its first store: with the stores behind
        // branches the compiler would otherwise wait for every earlier store at each row
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
        for (int n = 0; n < RG; ++n) {
          const int r = pr + PR * (RG * g + n), t = row0 + r;
          if (t >= p.M) break;
          const double a = ob[r * 128 + pi], c = ob[r * 128 + pi + 64];
          const uint16_t lo = f32_to_bf16(float(a * cs[n].x - c * cs[n].y));
          const uint16_t hi = f32_to_bf16(float(c * cs[n].x + a * cs[n].y));
          uint16_t* dst;
          if (h < rk.Hq) {
            dst = rk.q + (long(t) * rk.Hq + h) * 128;
          } else {
            const int sl = s_slot[r];
            if (sl < 0) continue;
            dst = rk.kc + ((long(sl >> 4) * rk.Hkv + (h - rk.Hq)) * 16 + (sl & 15)) * 128;
          }
          dst[pi] = lo;
          dst[pi + 64] = hi;
        }
      }
    } else {
      const int hk = h - rk.Hq - rk.Hkv;
      for (int w = threadIdx.x; w < BM * 128; w += NT) {
        const int r = w % BM, i = w / BM, sl = s_slot[r];
        if (sl < 0) continue;
        rk.vc[((long(sl >> 4) * rk.Hkv + hk) * 128 + i) * 16 + (sl & 15)] = f32_to_bf16(ob[r * 128 + i]);
      }
    }
    return;
  }
  float* out = splits > 1 ? part + long(split) * p.M * p.ldc : static_cast<float*>(p.C);
  if (!(splits == 1 && p.accumulate) && row0 + BM <= p.M && n0 + kBN <= p.N) {
    // whole tile: no bounds checks between the stores
    float* base = out + long(row0 + wm * WROWS + 4 * lgrp) * p.ldc + n0 + wn * 32 * NJ + lcol;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) base[long(32 * i + 8 * (e / 4) + (e % 4)) * p.ldc + 32 * j] = acc[i][j][e];
    return;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int c = n0 + wn * 32 * NJ + 32 * j + lcol;
    if (c >= p.N) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int grow = row0 + wm * WROWS + 32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4);
        if (grow >= p.M) continue;
        float* dst = out + long(grow) * p.ldc + c;
        *dst = (splits == 1 && p.accumulate) ? *dst + acc[i][j][e] : acc[i][j][e];
      }
  }
}

// ---------------------------------------------------------------- few-row QKV projection
// At up to 128 rows the QKV projection is the latency of its K walk: 40 column tiles x 32 slices,
// one after the other, on 40 workgroups (15 us at 5 rows for 21 MB of weights). Here a workgroup
// takes 32 columns of a head, the rotation pairs (i, i + 64) of 16 dims, x 32 AB rows, and its 8
// wavefronts split the K slices: at K = 2048 each has 4, all loaded at once straight into MFMA
// operand registers (weights and the tiled activations alike), so the walk is one memory latency;
// the 8 partial tiles meet in LDS and are added in wavefront order (deterministic). The epilogue
// has a rotation pair per thread. Measured (us, LDS-tiled / this): 5 rows 15.4 / 7.2, 48 rows
// 17.3 / 10.2, 80 rows 18.0 / 15.4; at 128 rows the layer gains 1 us, at 192 none, at 256 it loses 5.
constexpr int kFewWaves = 8;
constexpr int kFewSlices = 4;                 // slices of a wavefront in flight
constexpr int kFewRows = 128;

template <int AB>
__global__ __launch_bounds__(kFewWaves * kWave, 2) void qkv_few_kernel(GemmParams p, RopeKv rk) {
  __shared__ float red[kFewWaves][AB][1024];
  const int h = blockIdx.x / 4, i0 = 16 * (blockIdx.x % 4), row0 = 32 * AB * blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int nk = p.K / 64, l32 = lane % 32;
  const bool rotate = h < rk.Hq + rk.Hkv;
  // the thread's outputs: pair c (dims i0 + c, i0 + c + 64) of row r0 + 32 u
  const int c = threadIdx.x % 16, r0 = threadIdx.x / 16;
  double2 cs[AB];
  int slot[AB];
#pragma unroll
  for (int u = 0; u < AB; ++u) {
    const int t = min(row0 + r0 + 32 * u, p.M - 1);
    cs[u] = rotate ? rk.table[long(t) * 64 + i0 + c] : make_double2(1.0, 0.0);
    slot[u] = rk.slot[t];
  }
  // weight row of the lane: dim i0 + l (l < 16), then i0 + 64 + l - 16
  const int brow = h * 128 + i0 + (l32 < 16 ? l32 : 48 + l32);
  const long RB = 2L * p.K;
  const uint8_t* b = static_cast<const uint8_t*>(p.B) + tiled_offset(brow, 64 * (lane / 32), RB);
  const uint8_t* a[AB];
#pragma unroll
  for (int i = 0; i < AB; ++i) a[i] = static_cast<const uint8_t*>(p.A) + long(min(row0 + 32 * i, (p.M - 1) & ~31)) * RB + lane * 16;
  floatx16_t acc[AB];
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  auto walk = [&](auto& bv, auto& av, int kb, int n) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < n; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long off = long(kb + kFewWaves * s) * 4096 + q * 1024;
        bv[s][q] = __builtin_nontemporal_load(reinterpret_cast<const int32x4_t*>(b + off));
#pragma unroll
        for (int i = 0; i < AB; ++i) av[s][q][i] = *reinterpret_cast<const int32x4_t*>(a[i] + off);
      }
    __builtin_amdgcn_sched_barrier(0);        // all loads before the first MFMA waits for one
#pragma unroll
    for (int s = 0; s < n; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < AB; ++i)
          acc[i] = mfma(__builtin_bit_cast(bf16x8_t, av[s][q][i]), __builtin_bit_cast(bf16x8_t, bv[s][q]), acc[i]);
  };
  int32x4_t bv[kFewSlices][4], av[kFewSlices][4][AB];
  int kb = wave;
  for (; kb + kFewWaves * (kFewSlices - 1) < nk; kb += kFewWaves * kFewSlices) walk(bv, av, kb, kFewSlices);
  for (; kb < nk; kb += kFewWaves) walk(bv, av, kb, 1);
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][i][e * kWave + lane] = acc[i][e];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < AB; ++u) {
    // row r0 of block u sits at element 4 (r0 / 8) + r0 % 4 of lanes 32 (r0 / 4 % 2) + column
    const int at = (4 * (r0 / 8) + r0 % 4) * kWave + 32 * (r0 / 4 % 2) + c;
    float lo = red[0][u][at], hi = red[0][u][at + 16];
#pragma unroll
    for (int w = 1; w < kFewWaves; ++w) {
      lo += red[w][u][at];
      hi += red[w][u][at + 16];
    }
    const int t = row0 + r0 + 32 * u, sl = slot[u];
    if (t >= p.M) continue;
    if (rotate) {
      const double x = lo, y = hi;
      lo = float(x * cs[u].x - y * cs[u].y);
      hi = float(y * cs[u].x + x * cs[u].y);
    }
    uint16_t* dst;
    long step = 64;
    if (h < rk.Hq) {
      dst = rk.q + (long(t) * rk.Hq + h) * 128 + i0 + c;
    } else {
      if (sl < 0) continue;
      if (rotate) {
        dst = rk.kc + ((long(sl >> 4) * rk.Hkv + (h - rk.Hq)) * 16 + (sl & 15)) * 128 + i0 + c;
      } else {
        dst = rk.vc + ((long(sl >> 4) * rk.Hkv + (h - rk.Hq - rk.Hkv)) * 128 + i0 + c) * 16 + (sl & 15);
        step = 64 * 16;
      }
    }
    dst[0] = f32_to_bf16(lo);
    dst[step] = f32_to_bf16(hi);
  }
}

// ---------------------------------------------------------------- big-tile GEMM
// GEMMs with many rows and columns are bound by what the memory pipeline can hand the MFMAs,
// so their tile is sized for flops per loaded byte: 32 AB rows x 256 columns per workgroup
// (AB = 5: 101 flops per byte, where the 128 x 128 LDS-tiled kernel reaches 64). Wavefront w
// computes all rows of 64 columns, so the activation tile is shared by the four wavefronts
// and each weight column block belongs to one of them:
// * the AB activation blocks (tiled, 4 KB per K slice) go through a 4-stage LDS ring, copied
//   by the LDS-DMA form of the buffer load three slices ahead (each wavefront a quarter of
//   every block; it waits for its own copies and one barrier per slice publishes them);
// * the wavefront's 2 weight blocks are loaded straight into MFMA operand registers (the
//   tiled layout is the fragment layout) DEPTH slices ahead: they never touch LDS.
// Per 16-wide k step AB LDS fragments and 2 register fragments feed 2 AB MFMAs. The barrier
// sits before the last k step of a slice, so the next slice's first fragments are read
// behind that step's MFMAs. Loads past the last slice go through a resource of size 0: they
// move no data. The row tiles of one column tile are consecutive on one XCD, so its weights
// come from HBM once. Up to 4 blocks fit two workgroups on a CU (256 registers a wavefront,
// at 4 blocks with 2 weight slices in flight): one's loads and stores overlap the other's
// MFMAs, which made 128-row tiles the best per row (LM head, 640 x 151936 x 2048: 160 rows one
// a CU 401 us, 128 rows two a CU 360 us, one a CU 408 us; 192 rows 476 us).
constexpr int kBigBN = 256;
constexpr int kBigAStages = 4;
constexpr int kBigBLoads = 8;                  // weight loads per wavefront per slice
// weight slices in flight: what the registers hold (two wavefronts a SIMD up to 4 blocks)
template <int AB> constexpr int kBigDepth = AB == 3 ? 3 : AB == 4 ? 2 : 4;

// Buffer resource word 3 for raw byte-addressed loads (32-bit data format, no swizzle).
constexpr int kRawRsrcWord3 = 0x00020000;

MOLT_DEV __amdgpu_buffer_rsrc_t raw_rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, kRawRsrcWord3);
}

// Each lane copies the 16 bytes at voff + soff of the buffer into LDS at l + 16 * lane
// (l wave-uniform). The buffer form is a plain vector-memory instruction for the compiler's
// wait counting (the flat/global form makes it wait for every LDS read in flight).
MOLT_DEV void lds_dma16(__amdgpu_buffer_rsrc_t r, int voff, int soff, uint8_t* l) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)l, 16, voff, soff, 0, 0);
}

// acc[i][j] = rows 32 i .. of the activation tile x the wavefront's column block j over nk K
// slices. abase / avoff: each lane's source of its 16 bytes of every block's copy (wavefront w
// copies quarter w); bbase / bvoff: the lane's bytes of its weight blocks. ROWS: the activations
// are row-major rows; quarter w of a block is its rows 8 w .., and piece s of a row's 128 bytes
// holds piece s ^ (row / 2 % 8) (conflict-free fragment reads), which the caller's avoff picks.
// walk: nk rounded up to a multiple of DEPTH; every wavefront of the workgroup has to be given the
// same walk, it passes 1 + walk barriers. On return no copy is in flight; other wavefronts may still read the ring.
template <int AB, int DEPTH, bool ROWS = false>
MOLT_DEV void bigtile_loop(floatx16_t (&acc)[AB][2], uint8_t* ring, const void* abase, int abytes,
                           const int (&avoff)[AB], const void* bbase, int bbytes,
                           const int (&bvoff)[2], int nk, int walk, int wave, int lane) {
  constexpr int kStage = AB * 4096;
  auto issue_a = [&](int kb) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t ra = raw_rsrc(abase, kb < nk ? abytes : 0);
    uint8_t* dst = ring + (kb % kBigAStages) * kStage + wave * 1024;
#pragma unroll
    for (int j = 0; j < AB; ++j) lds_dma16(ra, avoff[j], kb * (ROWS ? kRowBytes : 4096), dst + j * 4096);
  };
  typedef bf16x8_t BSlice[4][2];   // [k step][column block]
  auto load_b = [&](int kb, BSlice& b) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rb = raw_rsrc(bbase, kb < nk ? bbytes : 0);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        b[c][j] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rb, bvoff[j] + c * 1024, kb * 4096, 0));
  };
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // activation fragments of one k step, two register sets
  bf16x8_t af[2][AB];
  const unsigned rsw = (4 * (lane / 32)) ^ ((lane % 32 / 2) % 8);
  const unsigned lbase = ROWS ? (lane % 32) * 128 : lane * 16;
  auto frag = [&](const uint8_t* stage, int c, int set) __attribute__((always_inline)) {
    const uint8_t* base = stage + lbase + (ROWS ? (rsw ^ c) * 16 : c * 1024);
#pragma unroll
    for (int i = 0; i < AB; ++i) af[set][i] = *reinterpret_cast<const bf16x8_t*>(base + i * 4096);
  };
  auto step = [&](int set, const bf16x8_t (&b)[2]) __attribute__((always_inline)) {
    // the scheduler would otherwise sink the next step's reads below these MFMAs
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma(af[set][i], b[j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);
  };
  BSlice bs[DEPTH];
  issue_a(0);
  issue_a(1);
  issue_a(2);
#pragma unroll
  for (int J = 0; J < DEPTH; ++J) load_b(J, bs[J]);
  // slice 0's activations are in (what follows them in the queue may be in flight)
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * AB + kBigBLoads * DEPTH) : "memory");
  frag(ring, 0, 0);
  // Per slice kb the vector-memory queue gets: activations kb + 3 (after the barrier), then
  // weights kb + depth (after the last MFMAs). The barrier of slice kb needs activations
  // kb + 1, issued in slice kb - 2; what may still be in flight behind them is at least
  // weights kb - 2 + depth, activations kb + 2 and weights kb - 1 + depth (exactly that from
  // slice 2 on, more before), so waiting for that many leaves it complete.
  static_assert(DEPTH >= 2, "the first barriers count two weight slices behind the copies");
  static_assert(2 * AB + kBigBLoads * DEPTH < 64, "vmcnt range");
  constexpr int kAWait = 2 * kBigBLoads + AB;
  auto body = [&](int kb, BSlice& b) __attribute__((always_inline)) {
    const uint8_t* base = ring + (kb % kBigAStages) * kStage;
    frag(base, 1, 1);
    step(0, b[0]);
    frag(base, 2, 0);
    step(1, b[1]);
    frag(base, 3, 1);
    step(0, b[2]);
    // this wavefront's copies of slice kb + 1 are done and all its reads of slice kb - 1's
    // stage have returned: after the barrier slice kb + 1 is complete for everyone and that
    // stage takes slice kb + 3
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kAWait) : "memory");
    issue_a(kb + 3);
    frag(ring + ((kb + 1) % kBigAStages) * kStage, 0, 0);
    step(1, b[3]);
    load_b(kb + DEPTH, b);
  };
  // `walk` slices in whole rounds of DEPTH (register sets are indexed statically): past the last
  // slice both operands are zeros and add nothing. (Exits between the slices of a round, and around the
  // loop, made the compiler move all accumulators at each of them, through scratch memory.)
  int kb = 0;
  do {
#pragma unroll
    for (int J = 0; J < DEPTH; ++J) body(kb + J, bs[J]);
    kb += DEPTH;
  } while (kb < walk);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Dense big-tile GEMM. Wavefront w takes column blocks 128 (w / 2) + 32 (w % 2) + {0, 64} of the
// tile: with ROPE a rotation pair (i, i + 64) of a head is then acc[.][0] and acc[.][1] of one
// lane. ROPE: the tile's two heads are rotated in registers (f64, the step's table), rounded to
// bf16 into the idle ring and written from there: q and K rows 16 bytes per store; V heads sit
// transposed in the ring, so that the lanes of a store are consecutive tokens of one dim. (With
// V read from rows and each token's cache slot from memory, the few V tiles alone took 40 us.)
enum BigEpilogue { kBigStore = 0, kBigAdd = 1, kBigRope = 2 };
template <int AB, int EPI>
__global__ __launch_bounds__(kThreads, AB <= 4 ? 2 : 1) void bigtile_gemm_kernel(GemmParams p, RopeKv rk) {
  constexpr bool ROPE = EPI == kBigRope;
  constexpr int BM = 32 * AB;
  // one LDS object (the compiler tells the ring's copies from other reads by their object):
  // the ring, then the cache slots of the tile's rows
  __shared__ __attribute__((aligned(16))) uint8_t ring[kBigAStages * AB * 4096 + (ROPE ? BM * 4 : 0)];
  const int total = p.n_mtiles * p.n_ntiles;
  const int chunk = (total + 7) / 8;
  const int k8 = blockIdx.x / 8;
  const int id = (blockIdx.x % 8) * chunk + k8;
  if (k8 >= chunk || id >= total) return;
  const int mt = id % p.n_mtiles, nt = id / p.n_mtiles;
  const int row0 = mt * BM, n0 = nt * kBigBN;
  const long RB = long(p.K) * 2;
  const int nk = int(RB / kRowBytes);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const int last_a = (p.M - 1) & ~31, last_b = (p.N - 1) & ~31;
  const int c0 = 128 * (wave >> 1) + 32 * (wave & 1);     // first column of block 0 in the tile
  // byte offsets relative to the activation matrix and to this tile's first weight row; row
  // blocks past the end re-read the last one (their results are never stored)
  int avoff[AB], bvoff[2];
#pragma unroll
  for (int j = 0; j < AB; ++j) avoff[j] = int(min(row0 + 32 * j, last_a) * RB) + wave * 1024 + lane * 16;
#pragma unroll
  for (int j = 0; j < 2; ++j) bvoff[j] = int((min(n0 + c0 + 64 * j, last_b) - n0) * RB) + lane * 16;
  floatx16_t acc[AB][2];
  bigtile_loop<AB, kBigDepth<AB>>(acc, ring, p.A, int(long(last_a + 32) * RB), avoff,
                      static_cast<const uint8_t*>(p.B) + long(n0) * RB,
                      int(long(min(n0 + kBigBN, last_b + 32) - n0) * RB), bvoff, nk,
                      (nk + kBigDepth<AB> - 1) / kBigDepth<AB> * kBigDepth<AB>, wave, lane);
  // acc[i][j][e]: row 32 i + 8 (e / 4) + 4 lgrp + e % 4, column c0 + 64 j + lcol
  const int lcol = lane % 32, lgrp = lane / 32;
  if constexpr (ROPE) {
    const int h = 2 * nt + (wave >> 1), nheads = rk.Hq + 2 * rk.Hkv;
    const int pi = 32 * (wave & 1) + lcol;
    // bf16 tile in the ring, one half per head: q and K [BM][128], V [128][BM]
    uint16_t* ob = reinterpret_cast<uint16_t*>(ring) + (wave >> 1) * BM * 128;
    int* s_slot = reinterpret_cast<int*>(ring + kBigAStages * AB * 4096);
    static_assert(2 * BM * 256 <= kBigAStages * AB * 4096, "the bf16 tile fits the ring");
    const bool rotate = h < rk.Hq + rk.Hkv;
    lds_barrier();                                        // every wavefront is done with the ring
    if (int(threadIdx.x) < BM) s_slot[threadIdx.x] = row0 + int(threadIdx.x) < p.M ? rk.slot[row0 + threadIdx.x] : -1;
#pragma unroll
    for (int i = 0; i < AB; ++i) {
      if (rotate) {
        double2 cs[16];
#pragma unroll
        for (int e = 0; e < 16; ++e)
          cs[e] = rk.table[long(min(row0 + 32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4), p.M - 1)) * 64 + pi];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const double a = acc[i][0][e], c = acc[i][1][e];
          uint16_t* o = ob + (32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4)) * 128 + pi;
          float lo = float(a * cs[e].x - c * cs[e].y), hi = float(c * cs[e].x + a * cs[e].y);
          // rounded to f32 first, as everywhere (the compiler would go from f64 to bf16 at once)
          asm("" : "+v"(lo), "+v"(hi));
          const uint32_t v = f32x2_to_bf16(lo, hi);
          o[0] = uint16_t(v);
          o[64] = uint16_t(v >> 16);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {                   // 4 consecutive rows of one dim
            *reinterpret_cast<uint2*>(ob + (pi + 64 * j) * BM + 32 * i + 8 * q + 4 * lgrp) =
                make_uint2(f32x2_to_bf16(acc[i][j][4 * q], acc[i][j][4 * q + 1]),
                           f32x2_to_bf16(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]));
          }
      }
    }
    lds_barrier();
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int hd = 2 * nt + hh;                         // workgroup-uniform
      if (hd >= nheads) break;
      const uint16_t* oh = reinterpret_cast<const uint16_t*>(ring) + hh * BM * 128;
      if (hd < rk.Hq + rk.Hkv) {
#pragma unroll 4
        for (int w = threadIdx.x; w < BM * 16; w += kThreads) {
          const int r = w / 16, ch = w % 16, t = row0 + r, sl = s_slot[r];
          if (t >= p.M || (hd >= rk.Hq && sl < 0)) continue;
          uint16_t* dst = hd < rk.Hq ? rk.q + (long(t) * rk.Hq + hd) * 128
                                     : rk.kc + ((long(sl >> 4) * rk.Hkv + (hd - rk.Hq)) * 16 + (sl & 15)) * 128;
          *reinterpret_cast<uint4*>(dst + 8 * ch) = *reinterpret_cast<const uint4*>(oh + r * 128 + 8 * ch);
        }
      } else {
        const int hk = hd - rk.Hq - rk.Hkv;
#pragma unroll 8
        for (int w = threadIdx.x; w < BM * 128; w += kThreads) {
          const int r = w % BM, i = w / BM, sl = s_slot[r];
          if (sl < 0) continue;
          rk.vc[((long(sl >> 4) * rk.Hkv + hk) * 128 + i) * 16 + (sl & 15)] = oh[w];
        }
      }
    }
    return;
  }
  float* C = static_cast<float*>(p.C);
  if (row0 + BM <= p.M && n0 + kBigBN <= p.N) {
    // whole tile (all but the last row and column tiles): no bounds checks between the stores
    // (the LM head: 451 -> 411 us; nontemporal stores measured 420 us); kBigAdd: 16 loads ahead of
    // their stores
    float* base = C + long(row0 + 4 * lgrp) * p.ldc + n0 + c0 + lcol;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < AB; ++i) {
        if (EPI == kBigAdd) {
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[i][j][e] += base[long(32 * i + 8 * (e / 4) + (e % 4)) * p.ldc + 64 * j];
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) base[long(32 * i + 8 * (e / 4) + (e % 4)) * p.ldc + 64 * j] = acc[i][j][e];
      }
    return;
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = n0 + c0 + 64 * j + lcol;
    if (col >= p.N) continue;
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int grow = row0 + 32 * i + 8 * (e / 4) + 4 * lgrp + (e % 4);
        if (grow >= p.M) continue;
        float* dst = C + long(grow) * p.ldc + col;
        *dst = EPI == kBigAdd ? *dst + acc[i][j][e] : acc[i][j][e];
      }
  }
}

template <int EPI>
hipError_t run_bigtile(GemmParams p, const RopeKv& rk, int ab, hipStream_t s) {
  p.n_mtiles = (p.M + 32 * ab - 1) / (32 * ab);
  p.n_ntiles = (p.N + kBigBN - 1) / kBigBN;
  const int grid = (p.n_mtiles * p.n_ntiles + 7) / 8 * 8;
  switch (ab) {
    case 2: bigtile_gemm_kernel<2, EPI><<<grid, kThreads, 0, s>>>(p, rk); break;
    case 3: bigtile_gemm_kernel<3, EPI><<<grid, kThreads, 0, s>>>(p, rk); break;
    case 4: bigtile_gemm_kernel<4, EPI><<<grid, kThreads, 0, s>>>(p, rk); break;
    case 5:
      if constexpr (EPI != kBigRope) {
        bigtile_gemm_kernel<5, EPI><<<grid, kThreads, 0, s>>>(p, rk);
        break;
      }
      [[fallthrough]];
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Grouped big-tile expert GEMM (bf16, experts of more than 128 rows): the tile table's tiles have
// up to 256 rows, the rows of an expert dealt out evenly; n-tiles of 256 weight rows. 8
// wavefronts, two halves of 4: each half takes half of the tile's 32-row blocks (its own part of
// the activation ring) against the same weight blocks, wavefront w of both the same columns, so
// the weights come from HBM once and meet in the CU's L1. (With one workgroup of 4 wavefronts per
// 128 rows, two a CU, an expert's two row tiles drifted apart by more than the 4 MB of an XCD's
// L2: the weights were read twice, 1.65 GB for 0.81.) gate_up: a wavefront holds the gate block
// and the up block of 32 columns, so SwiGLU happens in registers; the product goes through the
// ring to 16-byte stores. down: 64 columns per wavefront, stored from registers by buffer stores
// (rows past the tile's end get an offset out of range: no branch between the stores). The main
// loop is instantiated per number of blocks, so a part-filled tile costs its own blocks only. Each
// workgroup takes its first tile by its index and the next ones from its XCD's queue, then from
// the others' (tiles differ in cost, and so do the XCDs' shares).
constexpr int kGrpBlocks = 4;                  // 32-row blocks of a half, at most
constexpr int kGrpThreads = 512;
constexpr int kGrpRing = kBigAStages * kGrpBlocks * 4096;      // one half's ring
constexpr unsigned kNoRow = 0x80000000u;       // byte offset past every output row

struct GrpLds {                                // after the rings, in the same LDS object
  unsigned row[2][32 * kGrpBlocks];            // down: byte offset of the row's output
  int next;
};

// One half's share of a tile: rows [row0, row1) of the expert, AB blocks (none valid when row1 ==
// row0). Both halves pass the same barriers.
template <int AB, int MODE, bool ROWS>
MOLT_DEV void grouped_tile(const GemmParams& p, uint8_t* lds, int half, int expert, int row0, int row1,
                           int nt, int wave, int lane) {
  // the halves of a tile may have different AB: both walk nk rounded up to a multiple of 4
  constexpr int DEPTH = AB <= 2 ? 4 : 2;
  static_assert(4 % DEPTH == 0, "both halves pass the same number of barriers");
  // opaque per tile: the address arithmetic of the instances stays inside the tile loop instead
  // of being hoisted into registers held across it
  asm volatile("" : "+v"(lane));
  uint8_t* ring = lds + half * kGrpRing;
  unsigned* srow = reinterpret_cast<GrpLds*>(lds + 2 * kGrpRing)->row[half];
  const int tid = wave * kWave + lane;         // in the half
  const long RB = 2L * p.K;
  const int nk = int(RB / kRowBytes);
  const int lcol = lane % 32, lgrp = lane / 32;
  const int n0 = nt * (MODE == kGateUp ? 128 : kBigBN);
  // activations
  int avoff[AB];
  const uint8_t* abase = static_cast<const uint8_t*>(p.A);
  int abytes;
  if (ROWS) {
    // the lane's piece of row 8 wave + lane / 8 of each block, of that pair's token row; rows past
    // the end and padding rows read token 0 (their outputs are not stored)
    const int rr = 8 * wave + lane / 8;
#pragma unroll
    for (int j = 0; j < AB; ++j) {
      const int r = row0 + 32 * j + rr;
      const int pr = r < row1 ? p.perm[r] : -1;
      avoff[j] = (pr < 0 ? 0 : pr / p.ktop) * int(RB) + ((lane % 8) ^ ((rr / 2) % 8)) * 16;
    }
    abytes = p.M * int(RB);
  } else {
    abase += long(row0) * RB;
#pragma unroll
    for (int j = 0; j < AB; ++j) avoff[j] = j * 32 * int(RB) + wave * 1024 + lane * 16;
    abytes = AB * 32 * int(RB);
  }
  // weights: column block j of the wavefront (clamped into the expert's rows; not stored past them)
  const int rows_e = MODE == kGateUp ? 2 * p.N : p.N;
  int bcol[2], bvoff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    bcol[j] = MODE == kGateUp ? n0 + 32 * wave : n0 + 64 * wave + 32 * j;
    bvoff[j] = (min(bcol[j], p.N - 32) + (MODE == kGateUp ? j * p.N : 0)) * int(RB) + lane * 16;
  }
  if (MODE == kDown && tid < 32 * AB) {        // read after the main loop's barriers
    const int grow = row0 + tid;
    const int pr = grow < row1 ? p.perm[grow] : -1;
    srow[tid] = pr < 0 ? kNoRow : unsigned(pr) * unsigned(p.ldc) * 4u;
  }
  floatx16_t acc[AB][2];
  bigtile_loop<AB, DEPTH, ROWS>(acc, ring, abase, abytes, avoff,
                                static_cast<const uint8_t*>(p.B) + long(expert) * rows_e * RB,
                                rows_e * int(RB), bvoff, nk, (nk + 3) / 4 * 4, wave, lane);
  // acc[i][j][e]: row 32 i + 8 (e / 4) + 4 lgrp + e % 4, column bcol[j] + lcol
  lds_barrier();                               // everyone is done with the rings; the row table is in
  if (MODE == kGateUp) {
    uint16_t* ob = reinterpret_cast<uint16_t*>(ring);        // [32 AB][128] bf16
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        __builtin_amdgcn_sched_barrier(0);
        const int r = 32 * i + 8 * q + 4 * lgrp;
#pragma unroll
        for (int u = 0; u < 4; u += 2) {
          const uint32_t hv = f32x2_to_bf16(silu(acc[i][0][4 * q + u]) * acc[i][1][4 * q + u],
                                            silu(acc[i][0][4 * q + u + 1]) * acc[i][1][4 * q + u + 1]);
          ob[(r + u) * 128 + 32 * wave + lcol] = uint16_t(hv);
          ob[(r + u + 1) * 128 + 32 * wave + lcol] = uint16_t(hv >> 16);
        }
      }
    lds_barrier();
    const long hrb = 2L * p.N;
#pragma unroll
    for (int u = 0; u < 2 * AB; ++u) {
      const int w = tid + 256 * u, r = w / 16, cb = (w % 16) * 8;
      if (row0 + r < row1 && n0 + cb < p.N)
        *reinterpret_cast<int32x4_t*>(static_cast<uint8_t*>(p.C) + tiled_offset(row0 + r, 2L * (n0 + cb), hrb)) =
            *reinterpret_cast<const int32x4_t*>(ob + r * 128 + cb);
    }
  } else {
    // a wavefront past the last column (N is a multiple of 64): a resource of size 0
    const __amdgpu_buffer_rsrc_t rc = raw_rsrc(p.C, bcol[0] < p.N ? int(kNoRow - 1u) : 0);
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        __builtin_amdgcn_sched_barrier(0);                   // no more row entries in registers
        const uint4 ro = *reinterpret_cast<const uint4*>(srow + 32 * i + 8 * q + 4 * lgrp);
        const unsigned rof[4] = {ro.x, ro.y, ro.z, ro.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            // kNoRow plus a column stays past the resource's end
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][4 * q + u]), rc,
                                                  int(rof[u] + unsigned(lcol) * 4u), bcol[j] * 4, 0);
      }
  }
}

template <int MODE, bool ROWS>
__global__ __launch_bounds__(kGrpThreads, 2) void grouped_bigtile_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kGrpRing + sizeof(GrpLds)];
  GrpLds* sh = reinterpret_cast<GrpLds*>(lds + 2 * kGrpRing);
  const int total = *p.n_tiles_live * p.n_ntiles;
  const int chunk = (total + 7) / 8;
  const int stride = gridDim.x / 8;
  const int xcd = blockIdx.x % 8;
  const int w8 = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int half = w8 / 4, wave = w8 % 4;
  auto pool = [&](int x) { return min(chunk, total - x * chunk); };   // tiles of XCD x (may be <= 0)
  // the tile after XCD x's first `stride` ones that index k of its queue stands for; -1: past its end
  auto tile_of = [&](int x, int k) { return stride + k < pool(x) ? x * chunk + stride + k : -1; };
  auto steal = [&]() {
    for (int s = 1; s < 8; ++s) {
      const int x = (xcd + s) % 8;
      if (pool(x) <= stride) continue;          // all of it was given out by index
      const int t = tile_of(x, atomicAdd(p.queue + x, 1));
      if (t >= 0) return t;
    }
    return -1;
  };
  int id = int(blockIdx.x) / 8 < pool(xcd) ? xcd * chunk + int(blockIdx.x) / 8 : -1;
  for (;;) {
    // the next index of the own queue is asked for here and looked at after the tile
    const bool own = threadIdx.x == 0 && pool(xcd) > stride;
    int k = 0;
    if (own) k = atomicAdd(p.queue + xcd, 1);
    if (id >= 0) {
      const int mt = id / p.n_ntiles, nt = id % p.n_ntiles;
      typedef const __attribute__((address_space(4))) int32x4_t* ConstTile;
      const int32x4_t tv = *(ConstTile)(p.tiles + mt);
      const int blocks = (tv[2] - tv[1] + 31) / 32, b0 = (blocks + 1) / 2;
      // rows of this half; the second half of a one-block tile has none and reads the first's
      const int row0 = half == 0 ? tv[1] : blocks > b0 ? tv[1] + 32 * b0 : tv[1];
      const int row1 = half == 0 ? min(tv[1] + 32 * b0, tv[2]) : blocks > b0 ? tv[2] : tv[1];
      switch (half == 0 ? b0 : blocks - b0) {
        case 0:
        case 1: grouped_tile<1, MODE, ROWS>(p, lds, half, tv[0], row0, row1, nt, wave, lane); break;
        case 2: grouped_tile<2, MODE, ROWS>(p, lds, half, tv[0], row0, row1, nt, wave, lane); break;
        case 3: grouped_tile<3, MODE, ROWS>(p, lds, half, tv[0], row0, row1, nt, wave, lane); break;
        default: grouped_tile<4, MODE, ROWS>(p, lds, half, tv[0], row0, row1, nt, wave, lane); break;
      }
    }
    if (threadIdx.x == 0) {
      int t = own ? tile_of(xcd, k) : -1;
      if (t < 0) t = steal();
      sh->next = t;
    }
    // publishes `next`; everyone is done with the rings and the row table
    lds_barrier();
    id = __builtin_amdgcn_readfirstlane(sh->next);
    if (id < 0) break;
  }
}

template <int MODE, bool ROWS>
hipError_t run_grouped_big(GemmParams p, hipStream_t s) {
  static const int resident = resident_grid(grouped_bigtile_kernel<MODE, ROWS>, kGrpThreads);
  const int pairs = (p.n_mtiles * p.n_ntiles + 7) / 8 * 8;   // upper bound of the live pairs
  grouped_bigtile_kernel<MODE, ROWS><<<pairs < resident ? pairs : resident, kGrpThreads, 0, s>>>(p);
  return hipGetLastError();
}

// C (+)= sum over s of part[s], in split order
__global__ __launch_bounds__(kThreads) void splitk_reduce_kernel(const float* __restrict__ part,
                                                                 int splits, long n, float* __restrict__ C,
                                                                 int accumulate) {
  const long i = long(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= n) return;
  float v = accumulate ? C[i] : 0.f;
  for (int s = 0; s < splits; ++s) v += part[s * n + i];
  C[i] = v;
}

// ---------------------------------------------------------------- tiled-layout kernels
// pack: row-major [rows, RB bytes] -> tiled with rows padded to a multiple of 32 (padding
// rows zero); one thread per 16-byte chunk of the destination
__global__ __launch_bounds__(kThreads) void pack_tiled_kernel(const uint8_t* __restrict__ src,
                                                              uint8_t* __restrict__ dst, long rows,
                                                              long RB) {
  const long q = long(blockIdx.x) * kThreads + threadIdx.x;
  const long per_row = RB / 16;
  const long padded = (rows + 31) / 32 * 32;
  if (q >= padded * per_row) return;
  const long r = q / per_row, j = (q % per_row) * 16;
  int4 v = make_int4(0, 0, 0, 0);
  if (r < rows) v = *reinterpret_cast<const int4*>(src + r * RB + j);
  *reinterpret_cast<int4*>(dst + tiled_offset(r, j, RB)) = v;
}

// ---------------------------------------------------------------- f32 MFMA path
// The f32 model on v_mfma_f32_32x32x2_f32 (f32 products, f32 accumulation). Workgroup = one
// 32 x 32 output tile (gate_up: its gate and its up tile), 8 wavefronts that split the K
// slices (wavefront w takes slices w, w + 8, ...) and add their partial tiles through LDS in
// wavefront order (deterministic). The f32 decoder's calls have a few rows, so a launch is
// bound by its longest chain of loads and not by flops: with K = 256..512 every wavefront has
// at most two slices, their loads all in flight at once. A lane's 16-byte load of the tiled
// layout holds 4 consecutive k of its row, both operands alike, so element i of the 4 is the
// operand of one MFMA (k pair (4c + i, 16 + 4c + i) of the slice). gate_up reads the token
// rows through the permutation. One thread per output walking K element by element (the
// kernel before) took ~154 us per launch at K = 256..512 against 3-7 us (recompute of 16
// rows through 2 layers of the tiny decoder: 1755 -> 105 us, the attention kernel's share
// included).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kF32Waves = 8;

template <int MODE>
__global__ __launch_bounds__(kF32Waves * kWave) void f32_gemm_kernel(GemmParams p) {
  constexpr int NB = MODE == kGateUp ? 2 : 1;
  __shared__ float red[kF32Waves][NB][1024];
  const int mt = blockIdx.x % p.n_mtiles, nt = blockIdx.x / p.n_mtiles;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  int expert = 0, row0 = mt * 32, row1 = min(row0 + 32, p.M);
  if (MODE != kDense) {
    const int4 t = p.tiles[mt];
    if (t.x < 0) return;
    expert = t.x;
    row0 = t.y;                       // a multiple of 32: tiles are 32 rows of one expert
    row1 = t.z;
  }
  const long RB = 4L * p.K;
  const int nk = p.K / 32;
  // the lane's row of A: its own row of the tile, or that pair's token row (rows past the end
  // and padding rows read token 0; their outputs are not stored)
  long arow = row0 + lane % 32;
  if (MODE == kGateUp) {
    const int pr = arow < row1 ? p.perm[arow] : -1;
    arow = pr < 0 ? 0 : pr / p.ktop;
  }
  const uint8_t* a = static_cast<const uint8_t*>(p.A) + tiled_offset(arow, 64 * (lane / 32), RB);
  const long brow = long(expert) * (MODE == kGateUp ? 2L * p.N : MODE == kDown ? long(p.N) : 0L) + 32L * nt;
  const uint8_t* b[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) b[j] = static_cast<const uint8_t*>(p.B) + (brow + long(j) * p.N) * RB + lane * 16;
  floatx16_t acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
  for (int kb = wave; kb < nk; kb += kF32Waves) {
    f32x4 av[4], bv[NB][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      av[c] = *reinterpret_cast<const f32x4*>(a + kb * 4096L + c * 1024);
#pragma unroll
      for (int j = 0; j < NB; ++j) bv[j][c] = *reinterpret_cast<const f32x4*>(b[j] + kb * 4096L + c * 1024);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[c][i], bv[j][c][i], acc[j], 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][j][e * kWave + lane] = acc[j][e];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 1024 / (kF32Waves * kWave); ++u) {
    const int i = int(threadIdx.x) + kF32Waves * kWave * u;
    float v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v[j] = red[0][j][i];
#pragma unroll
      for (int w = 1; w < kF32Waves; ++w) v[j] += red[w][j][i];
    }
    // element e of lane l: row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
    const int e = i / kWave, l = i % kWave;
    const int grow = row0 + 8 * (e / 4) + 4 * (l / 32) + (e % 4), col = 32 * nt + l % 32;
    if (grow >= row1 || col >= p.N) continue;
    float* C = static_cast<float*>(p.C);
    if (MODE == kGateUp) {
      C[tiled_index(grow, col, p.N, 4)] = silu(v[0]) * v[NB - 1];
    } else {
      float* dst = C + (MODE == kDown ? long(p.perm[grow]) : long(grow)) * p.ldc + col;
      *dst = MODE == kDense && p.accumulate ? *dst + v[0] : v[0];
    }
  }
}

}  // namespace

// Row tiles of height h of one expert, on average: avg rows with the spread of T tokens that choose K of
// E experts alike (the share of experts past each multiple of h, linear over +-1.2 standard deviations).
static double expert_tiles(double avg, double share, int h) {
  const double width = 2.4 * sqrt(avg * std::max(0.0, 1.0 - share));
  if (width == 0.0) return ceil(avg / h);
  const long whole = std::max(0L, long((avg - 0.5 * width) / h));       // passed by every expert
  double n = 1.0 + double(whole);
  for (long j = whole + 1;; ++j) {
    const double p = (avg - double(j * h)) / width + 0.5;
    if (p <= 0.0) return n;
    n += std::min(p, 1.0);
  }
}

// Grouped expert GEMMs. Weight-streaming kernel: row tiles large enough that an expert of average
// load fits one (its weights are then streamed once), as small as that allows. From 120 rows per
// expert on average, where many experts need a second 128-row tile, the big-tile kernel may take bf16
// experts (us gate_up + down at d 2048, F 768, 128 experts top-8, streaming / big-tile: T = 4000
// 379 + 224 / 275 + 173, 2300 324 + 177 / 191 + 135, 1800 186 + 108 / 175 + 126, 1500 169 + 100 /
// 167 + 122). Its tiles are four times as large, so with few of them they leave the chip idle (E 8,
// top-2, 256 rows each, same d and F: 48 / 71). Either way a launch takes the longer of its rounds of
// tiles, each alone on its place of the chip (512 places / 256), and of all tiles' 128-byte K slices at
// the rate of a full chip; the constants (us) are fitted to both launches at 593 shapes (E 1..128, 120..4096
// rows, five d x F from 512 x 256 to 2048 x 6144): the choice costs 0.7% over the better kernel on
// average (big-tile from 120 rows on, without regard to the tiles: 16%). fp8 experts stay: their weights are
// half the bytes, and a version of the big-tile kernel in fp8 measured 125 + 95 against 131 + 93 at
// 2304 rows with skewed load.
MoePlan moe_plan(molt_dtype wdt, int T, int K, int E, int d, int F) {
  if (wdt == MOLT_F32) return {32, false};
  const long avg = (long(T) * K + E - 1) / E;
  const long lim = 1L << 31;           // 32-bit buffer offsets into each operand
  const MoePlan stream{avg <= 24 ? 32 : avg <= 56 ? 64 : 128, false};
  if (wdt != MOLT_BF16 || avg < 120 || 2L * T * d >= lim || 4L * T * K * d >= lim || 4L * F * d >= lim)
    return stream;
  const double share = double(K) / E;
  const double ms = E * expert_tiles(double(avg), share, 128), mb = E * expert_tiles(double(avg), share, 256);
  const double fill = 0.6 + 0.4 * std::min(1.0, double(avg) * E / mb / 256.0);   // a low tile's steps are shorter
  auto stream_us = [&](int nk, int nt) {
    return std::max(ceil(ms * nt / 512.0) * (8.0 + 0.5 * nk), ms * nt * (nk + 1.0) * 0.0038);
  };
  auto big_us = [&](int nk, int nt) {
    return std::max(ceil(mb * nt / 256.0) * (11.5 + 1.15 * fill * nk), mb * nt * (nk + 4.0) * 0.0084);
  };
  const int nkg = d / 64, nkd = F / 64;                // K slices of gate_up and of down
  const double ts = stream_us(nkg, F / 64) + stream_us(nkd, (d + 127) / 128);
  const double tb = big_us(nkg, (F + 127) / 128) + big_us(nkd, (d + 255) / 256);
  return tb < ts ? MoePlan{256, true} : stream;
}

// Plan of a dense bf16 GEMM: big tiles of 32 ab rows x 256 columns (ab > 0), or the LDS-tiled
// kernel with bm x 128 tiles and split-K. LDS-tiled: 128-row tiles when there are plenty of
// them, else 64 (and with the RoPE epilogue, whose rows take the big tiles long before); then the K
// range is halved while the grid is under one workgroup per CU, each split keeps >= 4 slices and the
// partial sums fit `part_elems` floats. Of 128-row tiles that leaves outputs of up to 128 columns and
// more than 65k rows (with the packing, us, 64 / 128 rows: 65500 x 128 x 2048 325 / 304, 66000 x 64 x
// 2048 318 / 315) and operands past 32-bit offsets.
// Between them the busiest CU decides: tiles per CU (rounded up) x the time of one tile, which
// was measured per 32 slices with the chip full (us): LDS-tiled 64 rows 11.5, 128 rows 20.5;
// big tiles of 64 rows 18, 96 rows 24, 128 rows 30, 160 rows 40; with the RoPE epilogue 64 rows 13
// and big tiles 20.5, 28.5, 33 (160 rows, 54, leave one workgroup a CU, with nothing to hide the epilogue
// behind: not used). The kernels both ways (us, LDS-tiled / big): 4000 x 5120 x 2048 135 / 87
// (160 rows), 4000 x 2048 x 4096 85 / 65 (128 rows), 2304 x 5120 x 2048 62 / 47 and 2304 x 2048
// x 4096 64 / 42 (96 rows), 640 x 5120 x 2048 25 / 21 (64 rows); 1024 x 2048 x 4096 26 / 32 and
// 640 x 2048 x 4096 29 / 30 stay LDS-tiled. QKV with RoPE at 4000 rows 138 / 98 (128 rows), at
// 2304 83 / 63 (96 rows), at 640 35 / 33 (64 rows).
GemmPlan gemm_plan(int M, int N, int K, long part_elems, bool rope) {
  constexpr long kCus = 256;
  GemmPlan g{128, 1, 0};
  const long nt = (N + kBN - 1) / kBN;
  if (rope || (M + 127) / 128 * nt < 512) g.bm = 64;
  const long wg = (M + g.bm - 1) / g.bm * nt;
  const int nk = int(2L * K / kRowBytes);
  long splits = 1;                       // without the limit of part_elems
  while (!rope && wg * splits < 256 && nk / (2 * splits) >= 4) splits *= 2;
  if (long(M + 31) * 2 * K < (1L << 31) && long(kBigBN) * 2 * K < (1L << 31)) {   // 32-bit buffer offsets
    constexpr double kTile[2][6] = {{0, 0, 18.0, 24.0, 30.0, 40.0}, {0, 0, 20.5, 28.5, 33.0}};
    const double lds_tile = rope ? 13.0 : g.bm == 64 ? 11.5 : 20.5;
    double best = double((wg * splits + kCus - 1) / kCus) * lds_tile / double(splits);
    for (int ab = 2; ab <= (rope ? 4 : 5); ++ab) {
      const long tiles = long((M + 32 * ab - 1) / (32 * ab)) * ((N + kBigBN - 1) / kBigBN);
      const double t = double((tiles + kCus - 1) / kCus) * kTile[rope][ab];
      if (t < best) { best = t; g.ab = ab; }
    }
    if (g.ab > 0) return g;
  }
  while (g.splits < splits && 2L * g.splits * M * N <= part_elems) g.splits *= 2;
  return g;
}

hipError_t launch_gemm(const void* A, const void* Bw, float* C, int M, int N, int K, molt_dtype dt,
                       bool accumulate, float* part, long part_elems, hipStream_t s,
                       int* splits_out) {
  if (splits_out) *splits_out = 1;
  GemmParams p{};
  p.A = A; p.B = Bw; p.C = C; p.M = M; p.N = N; p.K = K; p.ldc = N;
  p.accumulate = accumulate;
  if (dt == MOLT_F32) {
    p.n_mtiles = (M + 31) / 32;
    p.n_ntiles = (N + 31) / 32;
    f32_gemm_kernel<kDense><<<p.n_mtiles * p.n_ntiles, kF32Waves * kWave, 0, s>>>(p);
    return hipGetLastError();
  }
  if (dt == MOLT_BF16 && !accumulate && M <= 128 && N >= 8192 && N % kBN == 0) {
    // few rows and many columns (the draft head's LM head, one row per sequence): every
    // weight element is used by one row tile only, so the grouped GEMM's weight-streaming
    // kernel in down mode takes it as one "expert" holding all rows (no tile table: one row
    // tile, output row = input row); the 128 x 128 LDS kernel read the weights at about
    // half of HBM bandwidth
    p.tiles = nullptr; p.n_tiles_live = nullptr; p.perm = nullptr;
    p.n_mtiles = 1;
    p.n_ntiles = N / kBN;
    return run_stream<false, kDown>(p, M <= 32 ? 32 : M <= 64 ? 64 : 128, s);
  }
  const GemmPlan g = gemm_plan(M, N, K, part_elems);
  if (g.ab > 0)
    return accumulate ? run_bigtile<kBigAdd>(p, RopeKv{}, g.ab, s) : run_bigtile<kBigStore>(p, RopeKv{}, g.ab, s);
  p.n_mtiles = (M + g.bm - 1) / g.bm;
  p.n_ntiles = (N + kBN - 1) / kBN;
  const int grid = (p.n_mtiles * p.n_ntiles * g.splits + 7) / 8 * 8;
  // small grids (under two workgroups per CU): 8 wavefronts of 32 x 32 per tile, two per SIMD
  if (g.bm == 64) lds_gemm_kernel<64, false, 4, 2><<<grid, 512, 0, s>>>(p, part, g.splits, RopeKv{});
  else lds_gemm_kernel<128, false, 2, 2><<<grid, kThreads, 0, s>>>(p, part, g.splits, RopeKv{});
  if (g.splits > 1 && splits_out) {
    *splits_out = g.splits;         // the caller adds part[0 .. splits) (in order) into C
  } else if (g.splits > 1) {
    const long n = long(M) * N;
    splitk_reduce_kernel<<<(n + kThreads - 1) / kThreads, kThreads, 0, s>>>(part, g.splits, n, C,
                                                                             accumulate);
  }
  return hipGetLastError();
}

hipError_t launch_qkv_rope(const void* A, const void* Bw, int M, int K_in, int Hq, int Hkv,
                           const void* table, const int32_t* kv_slot, void* q_out, void* k_cache,
                           void* v_cache, hipStream_t s) {
  GemmParams p{};
  p.A = A; p.B = Bw; p.M = M; p.N = (Hq + 2 * Hkv) * 128; p.K = K_in; p.ldc = p.N;
  RopeKv rk{static_cast<const double2*>(table), kv_slot, Hq, Hkv, static_cast<uint16_t*>(q_out),
            static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache)};
  if (M <= kFewRows) {
    const int nt = 4 * (Hq + 2 * Hkv);
    if (M <= 32) qkv_few_kernel<1><<<dim3(nt, 1), kFewWaves * kWave, 0, s>>>(p, rk);
    else qkv_few_kernel<2><<<dim3(nt, (M + 63) / 64), kFewWaves * kWave, 0, s>>>(p, rk);
    return hipGetLastError();
  }
  const GemmPlan g = gemm_plan(M, p.N, K_in, 0, true);   // no split: the epilogue needs whole sums
  if (g.ab > 0) return run_bigtile<kBigRope>(p, rk, g.ab, s);
  p.n_mtiles = (M + 63) / 64;
  p.n_ntiles = Hq + 2 * Hkv;
  const int grid = (p.n_mtiles * p.n_ntiles + 7) / 8 * 8;
  lds_gemm_kernel<64, true, 4, 2><<<grid, 512, 0, s>>>(p, nullptr, 1, rk);
  return hipGetLastError();
}

hipError_t launch_moe_gate_up(const void* a, const float* a_scale, const int32_t* pperm, int K_top,
                              const void* w_gu, const float* s_gu, int T, int d, int F,
                              molt_dtype wdt, const int32_t* tiles, const int32_t* n_tiles,
                              int max_tiles, const MoePlan& plan, void* h, hipStream_t s) {
  GemmParams p{};
  p.M = T;
  p.n_tiles_live = n_tiles;
  p.A = a;
  p.B = w_gu; p.C = h; p.N = F; p.K = d; p.ldc = F;
  p.tiles = reinterpret_cast<const int4*>(tiles);
  p.n_mtiles = max_tiles;
  p.perm = pperm; p.ktop = K_top;
  p.a_scale = a_scale; p.b_scale = s_gu; p.b_scale_ld = 2 * F;
  if (wdt == MOLT_F32) {
    p.n_ntiles = F / 32;
    f32_gemm_kernel<kGateUp><<<max_tiles * p.n_ntiles, kF32Waves * kWave, 0, s>>>(p);
    return hipGetLastError();
  }
  p.queue = const_cast<int32_t*>(n_tiles) + 1;
  if (plan.big) {
    p.n_ntiles = (F + 127) / 128;
    return run_grouped_big<kGateUp, true>(p, s);
  }
  p.n_ntiles = F / (kBN / 2);
  if (wdt == MOLT_FP8_E4M3) return run_stream<true, kGateUp>(p, plan.tile_m, s);
  return run_stream<false, kGateUp>(p, plan.tile_m, s);
}

hipError_t launch_moe_down(const void* a, const float* a_scale, const int32_t* pperm,
                           const void* w_d, const float* s_d, int d, int F, molt_dtype wdt,
                           const int32_t* tiles, const int32_t* n_tiles, int max_tiles,
                           const MoePlan& plan, float* o, hipStream_t s) {
  GemmParams p{};
  p.n_tiles_live = n_tiles;
  p.A = a; p.B = w_d; p.C = o; p.N = d; p.K = F; p.ldc = d;
  p.tiles = reinterpret_cast<const int4*>(tiles);
  p.n_mtiles = max_tiles;
  p.perm = pperm;
  p.a_scale = a_scale; p.b_scale = s_d; p.b_scale_ld = d;
  if (wdt == MOLT_F32) {
    p.n_ntiles = d / 32;
    f32_gemm_kernel<kDown><<<max_tiles * p.n_ntiles, kF32Waves * kWave, 0, s>>>(p);
    return hipGetLastError();
  }
  p.queue = const_cast<int32_t*>(n_tiles) + 1 + kTileQueues;
  if (plan.big) {
    p.n_ntiles = (d + kBigBN - 1) / kBigBN;
    return run_grouped_big<kDown, false>(p, s);
  }
  p.n_ntiles = (d + kBN - 1) / kBN;
  if (wdt == MOLT_FP8_E4M3) return run_stream<true, kDown>(p, plan.tile_m, s);
  return run_stream<false, kDown>(p, plan.tile_m, s);
}

hipError_t launch_pack_tiled(const void* src, void* dst, long rows, long row_bytes, hipStream_t s) {
  const long chunks = (rows + 31) / 32 * 32 * (row_bytes / 16);
  if (chunks == 0) return hipSuccess;
  pack_tiled_kernel<<<(chunks + kThreads - 1) / kThreads, kThreads, 0, s>>>(
      static_cast<const uint8_t*>(src), static_cast<uint8_t*>(dst), rows, row_bytes);
  return hipGetLastError();
}

}  // namespace molt
