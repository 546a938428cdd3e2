// The rules on sizes: how a batch's streams are cut into pieces, where the
// pieces are combined, whether a step runs on one stream or two, and the LM
// head's tiles.
// Plain host code, without the HIP runtime, so that the CPU tests compile it
// by itself.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <utility>
#include <vector>

namespace sv {

// Piece length for a stream of L >= 1 keys and a split of s >= 1 keys: the
// stream cut into ceil(L / s) equal parts, rounded up to 32 keys (a short
// trailing piece would leave its work-group idle most of the kernel while its
// partial costs the same).  Every piece but the last has this length.
inline int piece_len(int L, int64_t s) {
  const int64_t n0 = (L + s - 1) / s;
  return (int)(((L + n0 - 1) / n0 + 31) / 32 * 32);
}

// Longest piece when there are at least as many streams as slots
// (piece_lengths below).  A work-group streams about 30 keys per microsecond,
// so a 4096-key piece started first runs nearly as long as the whole kernel on
// a 128-request ragged batch (3200 keys per slot on average).  Measured there
// with run-time claims, attention alone: 2048-key pieces 158 us, 2560 150,
// 3072 146, 3328-3840 142-143, 4096 155 (and 155 without claims).
#ifndef SV_MAX_PIECE
#define SV_MAX_PIECE 3584
#endif
constexpr int64_t kMaxPiece = SV_MAX_PIECE;
constexpr int64_t kMaxSplit = 1 << 20;

// What the cut depends on, for the whole batch.
struct CutShape {
  int rows_max;        // query rows of the widest work item
  int kv_heads;
  int d;               // head dim
  int elem;            // bytes per K/V element
  int64_t slots;       // work-groups the device runs at once
  int64_t cus;         // compute units
};

// Largest partial block (rows x pieces x d x 4 bytes) of one split stream that
// the bf16 split kernel's last piece combines itself by default; above it the
// separate combine kernel spreads the work over the device.
constexpr int64_t kFuseMaxBytes = 64 << 10;
// Whether the bf16 split kernel combines its partials itself.  The last piece
// reads the block alone, after every other piece of the stream has finished:
// that pays only while other streams' items keep the device busy, so from half
// as many streams as slots on, and from three eighths on where the block is
// short (two pieces, or 6 KB).  Measured on one plan each, us fused minus
// separate over batches of equal and ragged lengths (64-16000 keys, d = 64 and
// 128; blocks over 64 KB left out), by streams on 512 slots:
//   rows     128           192            256            320            384
//   5    +0.5 .. +5.9   -1.8 .. +3.6   -2.2 .. +1.2   -4.0 .. +0.1   -4.4 .. -0.1
//   16   +2.9 .. +8.4   -1.1 .. +4.1   -0.8 .. +1.6   -1.1 .. +1.7   -4.9 .. -2.0
//   20   +2.1 .. +8.3   -1.5 .. +2.8   -1.3 .. +1.9   -3.9 .. +0.0   -4.8 .. -3.7
//   40   +0.9 .. +5.8   -2.1 .. +2.4   -3.6 .. +0.7   -2.7 .. -1.5   -6.0 .. -4.7
//   72   -1.1           -4.9 .. -1.1   -11.6 .. -2.9  -6.7 .. -6.1   -8.5
// At 192 streams the two-piece plans and the blocks of up to 6 KB are the ones
// at or below zero (-2.1 .. +0.7; 100-1000 keys in 5 KB blocks +1.2).  The ragged
// batch with more streams than slots (1024, the few split ones <= 55 KB): -5;
// few streams: 8 of 1000 keys in 8 pieces +5, 64 of 32K keys (295 KB) +6 to +14.
inline bool fuse_by_default(int64_t streams, int64_t slots, int64_t nseg_max, int64_t block_bytes) {
  return 2 * streams >= slots || (8 * streams >= 3 * slots && (nseg_max <= 2 || block_bytes <= 6 << 10));
}

// The estimates below were fitted to 1398 calls of uniform batches (8 to 256
// streams of 130 to 64000 keys, 5 to 72 rows, d = 64 and 128, bf16 and fp32,
// whole and in 2 to 512 pieces): 8 % RMS of the call's time beside a constant
// 9.5 us, and the plan of least estimate is 0.4 % slower than the best one
// measured on average, 14 % at worst (8 streams of 400 keys, 5 rows, d = 128:
// 18.2 against 16.0 us).

// Microseconds of one round of work-groups: its longest piece at a
// work-group's own rate, or the batch's K and V at the HBM rate; where the two
// are close both show (the fourth-power mean).  A bf16 work-group takes 26 ns
// a key at d = 128 and 17.5 at d = 64 whatever its rows, an fp32 one 78 and 42;
// two fp32 ones of several waves on a compute unit run at 0.6 of that each.
// (Paged caches stream up to a tenth slower; their plan is the packed one's, so
// that the outputs are the same bits.)
inline double round_us(const CutShape& c, int64_t longest, int64_t kv_keys, int64_t items) {
  double ns = c.elem == 4 ? (c.d == 64 ? 42.0 : 78.0) : (c.d == 64 ? 17.5 : 26.0);
  if (c.elem == 4 && c.rows_max > 16 && items > c.cus) ns *= 1.6;
  const double own = 1e-3 * ns * (double)longest, all = (double)kv_keys * (2.0 * c.d * c.elem) / 7.0e6;
  const double a = own * own, b = all * all;
  return std::sqrt(std::sqrt(a * a + b * b));
}
// Microseconds that cut streams cost beside it: the combine's launch, its
// waves (one per output row of the batch), the partial rows written and read,
// the walk over one row's pieces, and the further items (laid out and staged
// by the host, fetched by the device).  2 pieces a stream of 130 keys cost 3 us
// over 40 output rows, 8 over 8000 and 17 over 18000; 64000 keys of one stream
// in 63 / 125 / 250 / 500 pieces 43 / 37 / 43 / 66 us.  The combine inside
// the split kernel (batches of half a round of streams and more, blocks
// within kFuseMaxBytes) hides its start as far as the other streams cover it:
// over the separate one 1 us at 256 streams of 512 slots, 2 at 320, 4 from
// 384 on.
inline double cut_us(const CutShape& c, int64_t streams, int64_t items, int64_t out_rows, int64_t part_rows,
                     int64_t nseg_max) {
  const bool fused = c.elem == 2 && fuse_by_default(streams, c.slots, nseg_max, nseg_max * c.rows_max * c.d * 4) &&
                     2ll * c.rows_max * c.d * 4 <= kFuseMaxBytes;
  const double busy = fused ? std::min(std::max(3.0 * (double)streams / (double)c.slots - 1.25, 0.0), 1.0) : 0.0;
  return (3.4 + 0.35e-3 * (double)out_rows) * (1.0 - busy) + 0.4e-6 * (double)part_rows * (c.d * 4.0) +
         0.085 * (double)nseg_max + 0.0015 * (double)(items - streams);
}

// Keys per piece of each request's streams (every KV head and head group of
// a request has the same length).  `len[i]` = keys of request i, each the
// length of `mult[i]` streams, `out_rows[i]` = its (verify position, query
// head) rows.
//  - At least as many streams as slots: pieces of at most kMaxPiece keys
//    (above) and at least 40 * rows, so that the fp32 partials (rows x d x 4
//    bytes, written once and read once by the combine) stay a few percent of
//    the K/V bytes a piece streams; dispatched longest first, the items past
//    the first round claimed at run time.
//  - Fewer streams than slots: every work-group takes exactly one item (a
//    second, nearly empty round of items ran 7-27% slower).  One piece per
//    stream to start with, then repeatedly one more piece for the request
//    whose pieces are currently longest, while its streams' extra items still
//    fit the slots and its pieces keep 128 bytes per column (64 bf16 keys) and
//    2 * rows keys; of the plans on that path the one of the least estimated
//    time (round_us + cut_us) runs.  What a cut saves is the longest whole
//    stream's time beyond the longest piece's, and where every stream is short
//    that is less than the combine costs: 16 requests x 8 KV heads of 64 rows,
//    261 keys whole 15.6 us, cut in two 22.9, 1000 keys 33.0 / 31.7, 4000
//    101 / 66; 60 requests of 72 rows and 1000 keys (480 streams: only a few
//    have a slot for a second piece) 49 / 57.
// `coarse` (a caller's fixed scratch is too small for this): pieces of at
// least 40 * rows and 256 keys.
inline std::vector<int> piece_lengths(const std::vector<int>& len, const std::vector<int>& mult,
                                      const std::vector<int>& out_rows, const CutShape& c, bool coarse) {
  const int64_t slots = std::max<int64_t>(c.slots, 1);
  const size_t B = len.size();
  std::vector<int> out(B);
  int64_t streams = 0, kv_keys = 0, rows = 0;
  for (size_t i = 0; i < B; ++i) {
    streams += mult[i];
    kv_keys += (int64_t)len[i] * c.kv_heads;   // head groups of one KV head share its rows
    rows += out_rows[i];
  }
  if (streams >= slots) {
    for (size_t i = 0; i < B; ++i) out[i] = piece_len(len[i], std::max(kMaxPiece, 40 * (int64_t)c.rows_max));
    return out;
  }
  int64_t lo = coarse ? std::max<int64_t>(40 * (int64_t)c.rows_max, 256)
                      : std::max<int64_t>(2 * (int64_t)c.rows_max, 128 / c.elem);
  lo = std::min<int64_t>((lo + 31) / 32 * 32, kMaxSplit);
  std::vector<int64_t> n(B, 1);
  auto cur = [&](size_t i) { return ((int64_t)len[i] + n[i] - 1) / n[i]; };
  const int64_t longest = *std::max_element(len.begin(), len.end());
  double best = round_us(c, longest, kv_keys, streams);
  // what no cut plan undercuts: pieces of `lo` keys for no partial rows
  const bool cut = coarse || round_us(c, std::min(lo, longest), kv_keys, streams) +
                                     cut_us(c, streams, streams, rows, 0, 2) < best;
  // greedy: a max-heap of (current piece length, request)
  std::vector<std::pair<int64_t, size_t>> heap;
  heap.reserve(B);
  for (size_t i = 0; cut && i < B; ++i) heap.emplace_back(cur(i), i);
  std::make_heap(heap.begin(), heap.end());
  std::vector<size_t> steps;                 // the request of each further piece
  size_t best_steps = 0;
  int64_t total = streams, part_rows = 0, nseg_max = 1;
  while (!heap.empty()) {
    std::pop_heap(heap.begin(), heap.end());
    const size_t i = heap.back().second;
    heap.pop_back();
    // one more piece for request i: its pieces must stay >= lo keys, and its
    // streams' extra items must fit the remaining slots
    if (((int64_t)len[i] + n[i]) / (n[i] + 1) < lo || total + mult[i] > slots) break;
    part_rows += (n[i] == 1 ? 2 : 1) * (int64_t)out_rows[i];
    nseg_max = std::max(nseg_max, ++n[i]);
    total += mult[i];
    heap.emplace_back(cur(i), i);
    std::push_heap(heap.begin(), heap.end());
    steps.push_back(i);
    const double us = round_us(c, (heap.front().first + 31) / 32 * 32, kv_keys, total) +
                      cut_us(c, streams, total, rows, part_rows, nseg_max);
    if (coarse || us < best) {
      best = us;
      best_steps = steps.size();
    }
  }
  std::fill(n.begin(), n.end(), 1);
  for (size_t s = 0; s < best_steps; ++s) ++n[steps[s]];
  for (size_t i = 0; i < B; ++i) {
    const int64_t piece = (cur(i) + 31) / 32 * 32;            // equal 32-aligned pieces
    out[i] = (int)std::min<int64_t>(std::max<int64_t>(piece, 32), kMaxSplit);
  }
  return out;
}

// Whether a step's acceptance runs beside its attention on a second stream.
// The fork and join (event packets that both queues wait on, and their host
// calls) cost a step that runs ahead of the device about what hiding the
// shorter part saves once K/V and 1.2 times the logit bytes pass 165 MiB (the
// logits weigh more: acceptance streams slower, and its own chain of round
// trips is hidden too); a caller that waits for each step pays the host calls,
// 8 to 17 us, at any size.  752 steps on both, 2 to 128 requests, vocabularies
// of 5000 to 128256, us two streams minus one, mean (calls in a row / waited
// for), by MiB of K/V and of logits:
//   K/V        logits 1-4      4-16       16-48       48-120
//    32       +17 / +17    +17 / +17   +14 / +16    +6 / +14
//    64       +13 / +15    +12 / +15    +8 / +14    +1 / +12
//    96        +9 / +14     +7 / +14    +4 / +13    -3 / +11
//   128        +5 / +14     +2 / +13    -1 / +12    -5 / +10
//   160         0 / +14     -2 / +13    -4 / +12    -6 / +9
//   200        -5 / +14     -6 / +13    -7 / +12    -7 / +9
//   400        -6 / +13     -7 / +12    -7 / +12    -7 / +8
// Over 6896 steps drawn from mixed shapes (50 to 400 MiB by this measure, both
// tree rules, paged and packed, equal and ragged contexts, bf16 and fp32) its
// choice is 0.9 % slower in a row than the better of both on average; a model
// of all the sizes would still be 0.4 %.  What it leaves: 5 % of the one-stream
// steps over 60 MiB would be 8 % or more faster in a row on two (over half of them
// with 25 to 75 MiB of logits, or under the sequential rule; nearly all are
// slower on two when waited for).
inline bool overlap_pays(int64_t kv_bytes, int64_t logit_bytes) {
  return kv_bytes + logit_bytes + logit_bytes / 5 > (int64_t)165 << 20;
}

// The LM head's tiles.
constexpr int kLmhNT = 256;            // vocabulary entries per work-group and statistics tile: tall tiles
constexpr int kLmhNTLow = 128;         // and low ones
struct LmhGeometry {
  int32_t rb, low_wr, tile_rows, m_tiles, nt;   // 16-row blocks per wave, waves along the rows (0: tall), ...
};
// Whether M rows take the low tiles (every row at once against 128 vocabulary
// entries, one work-group per compute unit that runs on from tile to tile).
// Measured as low over tall tiles' time, weights from HBM (the cache between
// the calls full of other reads):
//  - up to one round of low tiles: tall ones leave half the compute units
//    without any.  V = 32000, K = 1024 to 8192: M = 20 0.89-0.82, 95 1.01-0.85,
//    190 1.02-0.94; V = 9000, M = 20 0.83-0.62, 125 1.01-0.92, 160 1.12-1.07.
//    Weights that stay in the Infinity Cache between calls (256 MB) favour the
//    tall tiles' cached loads beyond 64 rows: V = 32000, K = 1024, M = 95 1.07, K
//    = 2048, M = 95 1.13, 160 1.02, V = 16000, K = 4096, M = 125 1.08, 160 1.20;
//  - more rounds, fewer than two for each of the tall tiles': V = 78071, M =
//    20 0.87-0.84, 95 1.01-0.89, 190 1.07-1.02 (from the cache, K = 2048 on, 95
//    0.95-0.85, 190 0.98);
//  - two for each: their epilogues, and a last round that is partly empty, are
//    paid twice.  V = 50304, M = 20 1.00-0.98, 40 1.07, 95 1.18, 190 1.28.
//    Where every round is full and the weights are long they pay later: V =
//    128256, K = 4096, M = 40 0.97, 60 1.02, 95 1.08; K = 8192, M = 60 0.95,
//    95 0.94.
inline bool lmh_low_tiles(int M, int V, int K, int cus) {
  const int64_t tiles = ((int64_t)V + kLmhNTLow - 1) / kLmhNTLow;
  const int64_t rounds = (tiles + cus - 1) / cus;
  const int64_t tall_rounds = (((int64_t)V + kLmhNT - 1) / kLmhNT + cus - 1) / cus;
  const int64_t weight_mib = ((int64_t)V * K * 2) >> 20;
  if (2 * tiles <= cus) return M <= (weight_mib < 140 ? 64 : 128);
  if (rounds < 2 * tall_rounds) return M <= (weight_mib < 80 ? 64 : 192);
  if (K < 2048) return M <= 16;
  if (10 * tiles < 9 * rounds * cus) return M <= 24;
  return M <= (K >= 6144 ? 96 : K >= 4096 ? 48 : 24);
}
// Tile shape for M rows, V vocabulary entries and hidden width K: low tiles as
// above, or tall ones, which cost about RB + 3 a round of work-groups over the
// CUs (the products, and the prologue, epilogue and slice hand-overs; M = 240
// to 960 at V = 32000 within a few percent).  Rows past M read as zeros and
// cost no traffic, so the row tiles are balanced.
inline LmhGeometry lmh_geometry(int M, int V, int K, int cus) {
  LmhGeometry g{};
  if (lmh_low_tiles(M, V, K, cus)) {
    g.low_wr = M <= 96 ? 1 : 2;
    g.rb = (M + 16 * g.low_wr - 1) / (16 * g.low_wr);
    g.m_tiles = 1;
    g.nt = kLmhNTLow;
  } else {
    int64_t best = -1;
    for (int rb = 1; rb <= 6; ++rb) {
      const int64_t mt = (M + 64 * rb - 1) / (64 * rb);
      const int64_t groups = mt * (((int64_t)V + kLmhNT - 1) / kLmhNT);
      const int64_t cost = (groups + cus - 1) / cus * (rb + 3);
      if (best < 0 || cost < best) {
        best = cost;
        g.rb = rb;
        g.m_tiles = (int32_t)mt;
      }
    }
    g.nt = kLmhNT;
  }
  g.tile_rows = (M + g.m_tiles - 1) / g.m_tiles;
  return g;
}

}  // namespace sv
