// The target model's LM head for the verify step (gfx950): the verify
// positions' logits, logits = hidden . weight^T, the forward that produces
// the target distributions of Eq. (1) (Sec. 2.2), with the softmax
// statistics of every (row, vocabulary tile) taken in the epilogue so that the
// acceptance never re-reads the logits for its normalisers (tiles of 128
// entries under lmh_low, 256 under lmh_tall).
//
// hidden [M, K] and weight [V, K] (one row per vocabulary entry, the linear
// layer's layout) are bf16 and both contiguous along K, so the operands of
// v_mfma_f32_16x16x32_bf16 are plain 16-byte row reads: lane l takes row
// l % 16, k = 8 (l / 16) .. +7 of a 16-row block, for the A (hidden) and the
// B (weight) operand alike, and holds C[4 (l / 16) + i][l % 16].
//
// 64-k slices of the hidden rows and the weight rows (one 128-byte cache line
// per row) stream through LDS by direct buffer -> LDS transfers; the 16-byte
// chunks of a row are swizzled so that the operand reads hit every bank.  Eight
// waves, one work-group per CU.  Two kernels, chosen by rows, rounds of
// work-groups and weight size (lmh_low_tiles):
//
//  - lmh_low (up to 192 rows): every row against 128 vocabulary entries, a deep
//    ring whose stream runs on from tile to tile.  Bound by the weights' stream
//    up to about 80 rows: 20 x 4096 x 32000 (262 MB) 41 us of GEMM, 72 x 8192 x
//    128256 (2.1 GB) 342 us, 6.2-6.4 TB/s.  With more rows every CU's own reads
//    of all of them (from L2, one 64-k slice per slice of weights) weigh in: 160
//    x 4096 x 32000 67.7 us for 262 MB of weights and 21 of logits, 4.2 TB/s,
//    with 256 CUs x 1.3 MB of hidden rows beside them.  What it took over
//    256-entry tiles of 64 or 128 rows (59 and 395 us at 20 and 72 rows): all
//    CUs busy on one vocabulary, the transfers' offsets out of the scalar unit
//    (descriptors rebuilt per transfer held the ring at 4.8 TB/s), each tile
//    starting at another k slice (lmh_first_slice), and the epilogue's
//    reductions on the vector ALU (12 -> 5 us a tile).
//  - lmh_tall: 64 RB rows x 256 entries (RB <= 6), 4 x 2 waves of 16 RB x 128.
//    Bound by the matrix cores and by what a slice's hand-over leaves idle, and
//    by the weights' latency where the vocabulary is short.  A wave keeps its
//    RB hidden operands in registers over a half slice and passes the weight
//    operands through two, so 384 x 256 fits 256 registers and 700 rows take
//    one round of work-groups: 716 x 4096 x 32000 with the acceptance 188 us,
//    against 223 for two rounds of 192-row tiles whose operands were read a
//    slice at a time (the products alone, without transfers, 120 of the GEMM);
//    92 MB of logits take 15 us of the epilogue.
#include "sv_internal.h"

#include <algorithm>
#include <type_traits>

namespace sv {
namespace {

#ifndef SV_LMH_LOW_NS
#define SV_LMH_LOW_NS 8
#endif
// Cache policy of the low tiles' weight transfers: non-temporal (2) keeps the
// weights, read once a call, from displacing the hidden rows and each other.
// GEMM and acceptance, us non-temporal / default, calls in a row: 20 rows x 4096
// x 32000 56.1 / 58.2, 80 x 8192 x 32000 101 / 117, 70 x 8192 x 128256 385 / 410;
// weights that stay in the Infinity Cache lose to it by less: 20 x 4096 x 9000
// 40.7 / 39.0 (46.0 / 46.7 when they come from HBM).
#ifndef SV_LMH_W_CPOL
#define SV_LMH_W_CPOL 2
#endif
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kWaves = 8;                 // two per SIMD, one work-group per compute unit
constexpr int kThreads = 64 * kWaves;
constexpr int kRowB = 128;                // bytes of one row's 64-k slice
constexpr int kLdsBytes = 160 * 1024;

template <int N>
__device__ __forceinline__ void lmh_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void lmh_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// 16-byte chunk c of LDS row r sits at chunk c ^ (r & 7): the 8 rows that 8
// consecutive lanes read (one chunk each) cover all the banks.
__device__ __forceinline__ int lmh_swz(int r) { return r & 7; }

// The decision kernel's inputs the row-statistics kernel would otherwise
// prepare (every work-group may take part; the grid can be smaller than B).
__device__ __forceinline__ void lmh_setup(const LmhParams& p) {
  for (int b = blockIdx.x; b < p.B; b += gridDim.x) {
    if (threadIdx.x < 2)
      reinterpret_cast<uint4*>(p.reqs + b)[threadIdx.x] = reinterpret_cast<const uint4*>(p.reqs_src + b)[threadIdx.x];
    if (threadIdx.x == 0) p.tickets[b] = 0;
  }
  for (int x = blockIdx.x * kThreads + threadIdx.x; x < p.nodes_n16; x += gridDim.x * kThreads)
    reinterpret_cast<uint4*>(p.nodes)[x] = reinterpret_cast<const uint4*>(p.nodes_src)[x];
}

// Tile `item` of the launch: the row tiles of one vocabulary tile are 8 items
// apart (one XCD of the round-robin dispatch) and within one window of 8 *
// m_tiles items, so they run together and share that tile's weight rows in
// the XCD's L2.
struct LmhTile {
  int m0, mrows, nt, n0, ncols;
};
template <int NT>
__device__ __forceinline__ LmhTile lmh_tile(const LmhParams& p, int item) {
  const int T = p.m_tiles;
  const int g = item / (8 * T), r8 = item % (8 * T);
  LmhTile t;
  t.nt = g * 8 + r8 % 8;
  t.m0 = (r8 / 8) * p.tile_rows;
  t.n0 = t.nt * NT;
  t.mrows = min(p.tile_rows, p.M - t.m0);
  t.ncols = min(NT, p.V - t.n0);          // <= 0 past the vocabulary
  return t;
}

// Each vocabulary tile starts its walk over K at another slice, 5 slices on
// from its neighbour's (K of whole slices only): rows a power of two apart
// read in step queue on the same memory channels.  GEMM and acceptance, us with
// steps of 0 / 1 / 3 / 5 slices: low tiles 20 x 4096 x 32000 71.2 / 54.9 / 56.2 /
// 56.1, 80 x 8192 x 32000 131.6 / 101.1 / 100.9 / 101.2, 70 x 8192 x 128256 477 /
// 383 / 381 / 385; tall 64 x 4096 x 50304 103.6 / 97.7 / 95.9 / 95.2, 380 179.7 /
// 175.7 / 186.5 / 183.2, 700 x 4096 x 32000 191 / 195 / 199 / 197.  Any step
// does for the low tiles; 5 shares no factor with 16, 32, 64 and 128 slices.
#ifndef SV_LMH_STAG
#define SV_LMH_STAG 5
#endif
__device__ __forceinline__ int lmh_first_slice(const LmhParams& p, int nt, int nk) {
  return p.K % 64 == 0 ? (nt * SV_LMH_STAG) % nk : 0;
}
// Buffer over `rows` rows of K bf16 at stride st elements, ending with the last
// row's last element: loads past it (rows of a partial tile, the second half
// of a K % 64 == 32 tail in the last row) read zeros.  The k offset goes into
// the vector offset, which the bounds check covers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t lmh_rows(const uint16_t* src, int rows, int64_t st, int K) {
  const int64_t bytes = rows > 0 ? ((int64_t)(rows - 1) * st + K) * 2 : 0;
  return __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, (uint32_t)bytes, 0x00020000);
}

// Epilogue of one tile.  The logits are stored (fp32, or rounded to bf16),
// and the statistics of each row over the tile's NT entries are taken on the
// stored values: the maximum, then the sum of exp(l - max) in fp64, lane
// sums in column-block order, then across the 16 lanes of a row, then across the WC waves of the row in wave order.  `red` holds
// WC * RA * 12 bytes of LDS that nothing else reads or writes meanwhile.
template <int RB, int CB, int WR, int WC, bool BF16OUT>
__device__ __forceinline__ void lmh_epilogue(const LmhParams& p, const LmhTile& t, f32x4 (&acc)[RB][CB], char* red,
                                             int wr, int wc, int lane) {
  constexpr int RA = 16 * RB * WR, NT = 16 * CB * WC;
  const int l16 = lane & 15, grp = lane >> 4;
  double* red_s = reinterpret_cast<double*>(red);                    // [WC][RA]
  float* red_m = reinterpret_cast<float*>(red + WC * RA * 8);        // [WC][RA]
  using OT = typename std::conditional<BF16OUT, uint16_t, float>::type;
  // this lane's byte offset from a row block's first row and column
  const int64_t lane_off = ((int64_t)(4 * grp) * p.o_st + 16 * CB * wc + l16) * (int64_t)sizeof(OT);
  const bool narrow = (13 * p.o_st + NT) * (int64_t)sizeof(OT) <= 0x7fffffff;   // uniform: 32-bit lane offsets
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row0 = 16 * (RB * wr + rb);
    const bool whole = narrow && t.ncols == NT && row0 + 16 <= t.mrows;          // wave-uniform
    OT* base = static_cast<OT*>(p.out) + (int64_t)(t.m0 + row0) * p.o_st + t.n0;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int col = 16 * CB * wc + 16 * cb + l16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = acc[rb][cb][i];
        OT st;
        if constexpr (BF16OUT) {
          const uint32_t u = __float_as_uint(v);
          st = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);   // round to nearest even
          v = __uint_as_float((uint32_t)st << 16);
        } else {
          st = v;
        }
        if (whole)
          *reinterpret_cast<OT*>(reinterpret_cast<char*>(base + i * p.o_st + 16 * cb) + (uint32_t)lane_off) = st;
        else if (row0 + 4 * grp + i < t.mrows && col < t.ncols)
          base[(int64_t)(4 * grp + i) * p.o_st + col] = st;
        acc[rb][cb][i] = col < t.ncols ? v : -INFINITY;
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // one row block at a time: bounded registers
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float m = acc[rb][0][i];
#pragma unroll
      for (int cb = 1; cb < CB; ++cb) m = fmaxf(m, acc[rb][cb][i]);
      m = max16(m);
      if (l16 == 0) red_m[wc * RA + 16 * (RB * wr + rb) + 4 * grp + i] = m;
      if (i == 3) __builtin_amdgcn_sched_barrier(0);
    }
  lmh_barrier();
  auto row_max = [&](int row) {
    float m = red_m[row];
#pragma unroll
    for (int x = 1; x < WC; ++x) m = fmaxf(m, red_m[x * RA + row]);
    return m;
  };
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * (RB * wr + rb) + 4 * grp + i;
      const float m = row_max(row);
      double sm = 0.0;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) sm += (double)exp_rel(acc[rb][cb][i], m);
      sm = sum16(sm);
      if (l16 == 0) red_s[wc * RA + row] = sm;
      if (i == 3) __builtin_amdgcn_sched_barrier(0);
    }
  lmh_barrier();
  for (int row = threadIdx.x; row < t.mrows; row += kThreads) {
    double sm = red_s[row];
#pragma unroll
    for (int x = 1; x < WC; ++x) sm += red_s[x * RA + row];
    p.tiles[(int64_t)(t.m0 + row) * p.ntiles + t.nt] = ChunkStat{sm, row_max(row), 0.f};
  }
}

// ---------------------------------------------------------------------------
// Low tiles: all of up to 192 rows x 128 vocabulary entries.
// ---------------------------------------------------------------------------
template <int RB, int WR>
struct LowGeo {
  static constexpr int WC = kWaves / WR, NT = kLmhNTLow, CB = NT / (16 * WC);
  static constexpr int RA = 16 * RB * WR;             // hidden rows
  static constexpr int STAGE = (RA + NT) * kRowB;
  static constexpr int RED = WC * RA * 12;
  static constexpr int FIT = (kLdsBytes - RED) / STAGE;
  static constexpr int NS = FIT < SV_LMH_LOW_NS ? FIT : SV_LMH_LOW_NS;   // ring stages
  static constexpr int XH = RA / 8;                   // 1 KB transfers of hidden rows per stage
  static constexpr int PH = (XH + kWaves - 1) / kWaves, FULLH = XH - (PH - 1) * kWaves;  // waves that issue PH, else PH - 1
  static constexpr int PW = NT / 8 / kWaves;          // transfers of weight rows per wave
  static_assert(NS >= 3, "ring depth");
};

template <int RB, int WR, bool BF16OUT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmh_low(LmhParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  using G = LowGeo<RB, WR>;
  constexpr int CB = G::CB, WC = G::WC, NS = G::NS;
  __shared__ __attribute__((aligned(1024))) char lds[NS * G::STAGE + G::RED];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / WC, wc = w % WC;
  const int l16 = lane & 15, grp = lane >> 4;

  // Transfer j of a matrix fills 1 KB: its LDS rows 8 j .. 8 j + 7, lane l
  // chunk l % 8 of row 8 j + l / 8; wave w issues transfers w, w + 8, ...
  const uint32_t lrow = (uint32_t)(8 * w + lane / 8), lchunk = (uint32_t)((lane % 8) ^ lmh_swz(lane / 8)) * 16u;
  uint32_t hoff[G::PH], woff[G::PW];
#pragma unroll
  for (int q = 0; q < G::PH; ++q) hoff[q] = (lrow + 64u * q) * (uint32_t)(p.h_st * 2) + lchunk;
#pragma unroll
  for (int q = 0; q < G::PW; ++q) woff[q] = (lrow + 64u * q) * (uint32_t)(p.w_st * 2) + lchunk;
  const bool fullh = w < G::FULLH;                    // wave-uniform
  const int nk = (p.K + 63) / 64;
  const __amdgpu_buffer_rsrc_t rh = lmh_rows(p.hidden, p.M, p.h_st, p.K);

  // The ring runs on over this work-group's tiles (blockIdx.x, + gridDim.x,
  // ...): the next tile's first slices are in flight during a tile's last
  // ones and its epilogue.  Past the last tile the weights' descriptor is
  // empty (zeros, no traffic); the hidden rows' transfers go on, up to NS - 1
  // slices of L2 hits that nothing reads, so that the counts stay the same.
  int ilt = blockIdx.x, it = 0, iks = lmh_first_slice(p, ilt, nk);   // tile, slice count and k slice to issue
  auto wrows = [&](int nt) {
    return lmh_rows(p.weight + (int64_t)nt * G::NT * p.w_st, min(G::NT, p.V - nt * G::NT), p.w_st, p.K);
  };
  __amdgpu_buffer_rsrc_t rw = wrows(ilt);
  auto issue = [&](int stage) {
    char* base = lds + stage * G::STAGE + w * 1024;
    const uint32_t koff = (uint32_t)iks * kRowB;
#pragma unroll
    for (int q = 0; q < G::PW; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void_t*)(base + G::RA * kRowB + q * 8192), 16, woff[q] + koff, 0,
                                               0, SV_LMH_W_CPOL);
#pragma unroll
    for (int q = 0; q < G::PH; ++q)
      if (q < G::PH - 1 || fullh)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rh, (lds_void_t*)(base + q * 8192), 16, hoff[q] + koff, 0, 0, 0);
    if (++iks == nk) iks = 0;
    if (++it == nk) {
      it = 0;
      ilt += gridDim.x;
      iks = lmh_first_slice(p, ilt, nk);
      rw = wrows(ilt);
    }
  };
  uint32_t ch[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) ch[h] = (uint32_t)(((4 * h + grp) ^ lmh_swz(l16)) * 16);
  const uint32_t abase = (uint32_t)(16 * RB * wr + l16) * kRowB;
  const uint32_t bbase = (uint32_t)(G::RA + 16 * CB * wc + l16) * kRowB;
#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue(st);
  lmh_setup(p);                     // its host reads fly beside the first slices
  int stage = 0;
  for (int nt = blockIdx.x; nt < p.ntiles; nt += gridDim.x) {
    f32x4 acc[RB][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < nk; ++t) {
      // this wave's transfers of the current slice have landed (the NS - 2
      // after it may still fly)
      if (fullh) lmh_wait_vm<(G::PH + G::PW) * (NS - 2)>();
      else lmh_wait_vm<(G::PH - 1 + G::PW) * (NS - 2)>();
      lmh_barrier();                // everyone's have; the stage read last is free
      issue(stage == 0 ? NS - 1 : stage - 1);
      const char* sb = lds + stage * G::STAGE;
      stage = stage + 1 == NS ? 0 : stage + 1;
      bf16x8 a[2][RB], b[2][CB];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) b[h][cb] = *reinterpret_cast<const bf16x8*>(sb + bbase + cb * 16 * kRowB + ch[h]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) a[h][rb] = *reinterpret_cast<const bf16x8*>(sb + abase + rb * 16 * kRowB + ch[h]);
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][rb], b[0][cb], acc[rb][cb], 0, 0, 0);
      // K % 64 == 32: the last k slice (no rotation then) holds 32 k only
      if (t + 1 < nk || p.K % 64 == 0) {              // wave-uniform
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][rb], b[1][cb], acc[rb][cb], 0, 0, 0);
      }
    }
    const LmhTile tile{0, p.M, nt, nt * G::NT, min(G::NT, p.V - nt * G::NT)};
    lmh_epilogue<RB, CB, WR, WC, BF16OUT>(p, tile, acc, lds + NS * G::STAGE, wr, wc, lane);
  }
#endif
}

// ---------------------------------------------------------------------------
// Tall tiles: up to 64 RB rows x 256 vocabulary entries, bound by the matrix
// cores.
// ---------------------------------------------------------------------------
template <int RB>
struct TallGeo {
  static constexpr int WR = 4, WC = 2, NT = kLmhNT, CB = NT / (16 * WC);
  static constexpr int RA = 16 * RB * WR;
  static constexpr int HST = RA * kRowB, WST = NT * kRowB;            // bytes of a slice of each matrix
  static constexpr int XH = RA / 8 / kWaves, XW = NT / 8 / kWaves;    // transfers per wave and slice
  // Slices in LDS: of the hidden rows (L2 hits) and of the weights (from HBM).
  // 64- and 128-row tiles run where the vocabulary has few of them, so each
  // compute unit's own latency shows: four and three of both, against two of
  // the hidden rows and three of the weights 190 rows x 8192 x 16000 118.6 us for
  // 134.2, 255 x 4096 x 1000 65.6 for 73.6 (weights from HBM; from the cache the
  // same).  Taller ones have room for two of the hidden rows, and three of the
  // weights up to 256 rows.
  static constexpr int NH = RB == 1 ? 4 : RB == 2 ? 3 : 2;
  static constexpr int NW = RB <= 2 ? NH : 2 * HST + 3 * WST <= kLdsBytes ? 3 : 2;
  static constexpr int FLY = (NH - 2) * XH + (NW - 2) * XW;           // transfers behind the next slice's
  static constexpr int LDS = NH * HST + NW * WST;
  static_assert(NH == NW || (NH == 2 && NW == 3), "the next slice's transfers are older than the FLY youngest");
  // A slice's transfers are issued after the barrier that frees their stages,
  // or spread over the column blocks behind it.  Together they start sooner
  // but hold the waves' next products back.  GEMM and acceptance, us together /
  // spread, one round of RB = 1 .. 6 (64, 128, 190, 255, 320 and 380 rows x 4096 x
  // 50304): 95.2 / 95.2, 109.2 / 110.5, 125.5 / 127.2, 137.8 / 141.0, 157 / 176,
  // 183 / 193; RB = 4 over two rounds (480 x 4096 x 32000) 141.0 / 138.4 and four
  // (960 rows) 278.6 / 277.0.
  static constexpr bool SPREAD = RB == 4;
  static_assert(RA % 64 == 0 && LDS <= kLdsBytes, "the slices fit LDS");
};

template <int RB, bool BF16OUT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmh_tall(LmhParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  using G = TallGeo<RB>;
  constexpr int CB = G::CB, WR = G::WR, WC = G::WC;
  __shared__ __attribute__((aligned(1024))) char lds[G::LDS];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / WC, wc = w % WC;
  const int l16 = lane & 15, grp = lane >> 4;
  const LmhTile it = lmh_tile<G::NT>(p, blockIdx.x);
  if (it.ncols <= 0 || it.mrows <= 0) {               // uniform
    lmh_setup(p);
    return;
  }
  const uint32_t lrow = (uint32_t)(8 * w + lane / 8), lchunk = (uint32_t)((lane % 8) ^ lmh_swz(lane / 8)) * 16u;
  const uint32_t hoff = lrow * (uint32_t)(p.h_st * 2) + lchunk, woff = lrow * (uint32_t)(p.w_st * 2) + lchunk;
  const int nk = (p.K + 63) / 64;
  const int k0 = lmh_first_slice(p, it.nt, nk);
  // Transfer q of slice t of a matrix into stage st.  Past the last slice the
  // descriptor is empty (zeros, no traffic), so that the transfer counts stay
  // the same.  The step between transfers is opaque: their offsets are formed
  // here and do not each hold a register through the loop.
  auto kbytes = [&](int t) { return (uint32_t)(t + k0 < nk ? t + k0 : t + k0 - nk) * kRowB; };
  auto xfer_h = [&](int st, int t, int q) {
    const __amdgpu_buffer_rsrc_t r = lmh_rows(p.hidden + it.m0 * p.h_st, t < nk ? it.mrows : 0, p.h_st, p.K);
    uint32_t step = 128u * (uint32_t)p.h_st;          // 64 rows
    asm volatile("" : "+s"(step));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(lds + st * G::HST + w * 1024 + q * 8192), 16,
                                             hoff + (q * step + kbytes(t)), 0, 0, 0);
  };
  auto xfer_w = [&](int st, int t, int q) {
    const __amdgpu_buffer_rsrc_t r = lmh_rows(p.weight + it.n0 * p.w_st, t < nk ? it.ncols : 0, p.w_st, p.K);
    uint32_t step = 128u * (uint32_t)p.w_st;
    asm volatile("" : "+s"(step));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (lds_void_t*)(lds + G::NH * G::HST + st * G::WST + w * 1024 + q * 8192), 16, woff + (q * step + kbytes(t)), 0, 0,
        0);
  };
  // LDS addresses of this lane's operands, by k half, in the stage being read
  // (updated as the walk changes stage)
  uint32_t aad[2], bad[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t c = (uint32_t)(((4 * h + grp) ^ lmh_swz(l16)) * 16);
    aad[h] = (uint32_t)(16 * RB * wr + l16) * kRowB + c;
    bad[h] = (uint32_t)(G::NH * G::HST) + (uint32_t)(16 * CB * wc + l16) * kRowB + c;
  }

  f32x4 acc[RB][CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 a[RB], b[2];
  auto lda = [&](int h, int rb) { return *reinterpret_cast<const bf16x8*>(lds + aad[h] + rb * 16 * kRowB); };
  auto ldb = [&](int h, int cb) { return *reinterpret_cast<const bf16x8*>(lds + bad[h] + cb * 16 * kRowB); };
#pragma unroll
  for (int st = 0; st < G::NW - 1; ++st) {
#pragma unroll
    for (int q = 0; q < G::XW; ++q) xfer_w(st, st, q);
    if (st < G::NH - 1)
#pragma unroll
      for (int q = 0; q < G::XH; ++q) xfer_h(st, st, q);
  }
  lmh_setup(p);                     // its host reads fly beside the first slices
  lmh_wait_vm<G::FLY>();
  lmh_barrier();
  b[0] = ldb(0, 0);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) a[rb] = lda(0, rb);
  // Half H (32 k) of a slice: the hidden rows' operands stay in registers, the
  // weight operands pass through two, each loaded one column block ahead; in
  // the last column block each hidden operand is replaced by the next half's
  // as its last product is issued (past the last slice: by what the ring
  // holds, never used).
  int hstage = 0, wstage = 0;       // the current slice's stages
  // During slice s (or, together, from the barrier that ends slice s - 1):
  // transfers h0 .. h1 of the hidden rows' slice s + NH - 1 and w0 .. w1 of the
  // weights' slice s + NW - 1, into the stages that slice s - 1 left.
  auto ahead = [&](int s, int h0, int h1, int w0, int w1) {
    const int hs = hstage == 0 ? G::NH - 1 : hstage - 1, ws = wstage == 0 ? G::NW - 1 : wstage - 1;
#pragma unroll
    for (int q = h0; q < h1; ++q) xfer_h(hs, s + G::NH - 1, q);
#pragma unroll
    for (int q = w0; q < w1; ++q) xfer_w(ws, s + G::NW - 1, q);
  };
  if constexpr (!G::SPREAD) ahead(0, 0, G::XH, 0, G::XW);
  auto half = [&](auto hc, int t) {
    constexpr int H = decltype(hc)::value;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if (H == 1 && cb + 1 == CB) {
        // Every operand of this slice has been read: the next slice has landed
        // (those after it may still fly), everyone is done with this one, and
        // later slices may overwrite it.
        lmh_wait_vm<G::FLY>();
        lmh_barrier();
        const int hstep = hstage + 1 == G::NH ? -(G::NH - 1) * G::HST : G::HST;
        const int wstep = wstage + 1 == G::NW ? -(G::NW - 1) * G::WST : G::WST;
        hstage = hstage + 1 == G::NH ? 0 : hstage + 1;
        wstage = wstage + 1 == G::NW ? 0 : wstage + 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          aad[h] += hstep;
          bad[h] += wstep;
        }
        if constexpr (!G::SPREAD) ahead(t + 1, 0, G::XH, 0, G::XW);
      } else if constexpr (G::SPREAD) {
        if (H == 0 && cb < G::XH) ahead(t, cb, cb + 1, 0, 0);
        if (H == 1 && cb < G::XW) ahead(t, 0, 0, cb, cb + 1);
      }
      b[(cb + 1) & 1] = cb + 1 < CB ? ldb(H, cb + 1) : ldb(1 - H, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], b[cb & 1], acc[rb][cb], 0, 0, 0);
        if (cb + 1 == CB) {
          a[rb] = lda(1 - H, rb);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert(CB % 2 == 0, "the weight operands alternate over two registers");
  for (int t = 0; t < p.K / 64; ++t) {
    half(std::integral_constant<int, 0>{}, t);
    half(std::integral_constant<int, 1>{}, t);
  }
  if (p.K % 64 != 0) half(std::integral_constant<int, 0>{}, nk - 1);   // the last slice holds 32 k only
  lmh_wait_vm<0>();
  lmh_barrier();                    // the ring is no longer read: reuse its LDS
  int elane = threadIdx.x & 63;     // opaque: keeps the epilogue's addresses out of the loop's registers
  asm volatile("" : "+v"(elane));
  lmh_epilogue<RB, CB, WR, WC, BF16OUT>(p, it, acc, lds, wr, wc, elane);
#endif
}

template <int RB, int WR>
hipError_t launch_low(const LmhParams& p, int cus, hipStream_t s) {
  const dim3 grid((unsigned)std::min(p.ntiles, std::max(cus, 1)));
  if (p.out_bf16) lmh_low<RB, WR, true><<<grid, dim3(kThreads), 0, s>>>(p);
  else lmh_low<RB, WR, false><<<grid, dim3(kThreads), 0, s>>>(p);
  return hipGetLastError();
}
template <int RB>
hipError_t launch_tall(const LmhParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(((p.ntiles + 7) / 8) * 8 * p.m_tiles));
  if (p.out_bf16) lmh_tall<RB, true><<<grid, dim3(kThreads), 0, s>>>(p);
  else lmh_tall<RB, false><<<grid, dim3(kThreads), 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_lmh(const LmhParams& p, int cus, hipStream_t s) {
  if (p.M < 1 || p.tile_rows < 1 || p.m_tiles != (p.M + p.tile_rows - 1) / p.tile_rows) return hipErrorInvalidValue;
  if (p.low_wr) {
    if (p.m_tiles != 1 || p.M > 16 * p.rb * p.low_wr) return hipErrorInvalidValue;
    switch (p.low_wr * 16 + p.rb) {
      case 16 + 1: return launch_low<1, 1>(p, cus, s);
      case 16 + 2: return launch_low<2, 1>(p, cus, s);
      case 16 + 3: return launch_low<3, 1>(p, cus, s);
      case 16 + 4: return launch_low<4, 1>(p, cus, s);
      case 16 + 5: return launch_low<5, 1>(p, cus, s);
      case 16 + 6: return launch_low<6, 1>(p, cus, s);
      case 32 + 4: return launch_low<4, 2>(p, cus, s);
      case 32 + 5: return launch_low<5, 2>(p, cus, s);
      case 32 + 6: return launch_low<6, 2>(p, cus, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (p.tile_rows > 64 * p.rb) return hipErrorInvalidValue;
  switch (p.rb) {
    case 1: return launch_tall<1>(p, s);
    case 2: return launch_tall<2>(p, s);
    case 3: return launch_tall<3>(p, s);
    case 4: return launch_tall<4>(p, s);
    case 5: return launch_tall<5>(p, s);
    case 6: return launch_tall<6>(p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sv
