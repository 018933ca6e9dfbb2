// plan.cpp -- host planner: segment descriptors -> per-row positions and the
// workgroup work list of one fused MSA launch.
//
// The paper dispatches every request segment to a group of CTAs inside a
// single kernel and gives each token its own "equivalent seq_len" through a
// precomputed array (Sec. 4.1).  Here:
//   1. rows: each packed query row gets its absolute position (its causal
//      limit is position + 1 keys);
//   2. tiles: consecutive rows of one sequence are packed into tiles of up to
//      tile_rows / G tokens (G = Hq / Hkv query heads share one KV head),
//      across segment gaps as long as the keys masked for the earlier rows
//      stay a small fraction of the tile's work.  tile_rows is 256 (one
//      workgroup per CU, each K/V step loaded once for 256 rows) when the
//      128-row tiling has full tiles and a long run of key steps per
//      workgroup slot, else 128 (two workgroups per CU: one's start-up and
//      tail overlap the other's work, and decode-heavy plans keep more key
//      streams in flight); it is 32 when no 128-row tile would hold more
//      than 32 rows (decode-like plans: the four waves of a workgroup then
//      split the tile's keys).  A 128-row plan of few short tiles runs as
//      items of up to 32 rows, in the same way;
//   3. units: tile x KV head, keys [0, max position in tile + 1);
//   4. key splits of 32-row tiles and items: the cut length is the shortest
//      whose pieces all fit one round of the workgroup slots, or, below 1024
//      keys, whose pieces (of 256 keys or more) have a CU each; units are left
//      whole where cutting gains less than a merge takes.  Other plans cut
//      units in step 6.  Split units are merged later by log-sum-exp;
//   5. order: (sequence, KV head) groups keep to one of the 8 XCDs (blockIdx
//      i runs on XCD i % 8) so tiles sharing K/V share one XCD's L2; groups
//      that would leave the XCDs uneven are spread over few of them.  Inside
//      each XCD, groups start in decreasing order of their longest chunk and
//      a group's chunks run back to back, longest first, so that no long
//      piece (a decode row over a long context) is left for the end;
//   6. workgroups: the launch is persistent, one workgroup per slot, each
//      with its own list of items; each XCD's queue is dealt out in order to
//      the least-loaded workgroup of that XCD, and a unit that would carry a
//      workgroup past the mean load is cut there.
#include "plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <queue>
#include <utility>

namespace msa {
namespace {

constexpr int kXcds = 8;
// 64-key steps per workgroup slot of the narrow tiling from which wide tiles
// pay: shorter plans gain more from two workgroups per CU (one's start-up and
// tail overlap the other's work) than from loading each K/V step once for 256
// rows.  Narrow against wide, us: head_dim 128, 75 steps 164 / 173, 109 steps
// 231 / 224, 200 steps 427 / 419, 290 steps 566 / 541; head_dim 64, whose steps
// are half as long, 160 steps 146 / 151, 185 steps 201 / 202.
constexpr double kWideMinStepsPerSlot = 96.0;
constexpr double kWideMinStepsPerSlot64 = 384.0;
constexpr int64_t kWideMinTiles64 = 1024;  // narrow tiles, head_dim 64
// ... and the share of the key steps' rows that hold queries: a decode row
// takes a whole workgroup's step however wide (45 of 60 sequences decoding:
// fill 0.82 1296 / 1313, 0.57 566 / 621; 24 of 32: 0.94 1645 / 1605)
constexpr double kWideMinFill = 0.9;
constexpr double kWasteFrac = 0.125;     // masked keys allowed per tile, relative
constexpr int64_t kMinSplitKeys = 1024;  // never split below this many keys
constexpr int64_t kMinSplitSteps = kMinSplitKeys / kKvStep;
constexpr int64_t kMinSplitKeysDecode = 256;  // the same for 32-row items with a CU each
constexpr int64_t kWholeKeysDecode = 768;     // 32-row items of up to this many keys stay whole
constexpr int64_t kMinTailSteps = kMinSplitSteps / 2;  // shortest remainder of a cut unit
// cost of starting and ending an item, in key steps: 7-9 us against 1.9 us a
// step (128- and 256-row tiles); small beside a streamed step of a 32-row tile
constexpr double kItemSteps = 4.0;
constexpr double kItemStepsDecode = 1.0;
// an XCD's load over the mean that still counts as even: for a group of more
// than half an XCD's share, and for a smaller one (spreading it gains less
// and costs as much L2)
constexpr double kHomeSlack = 0.03;
constexpr double kHomeSlackSmall = 0.15;
constexpr double kOneRoundFactor = 1.1;  // one piece per workgroup preferred up to this times the packed load
constexpr double kCutSlack = 0.02;       // a workgroup's load over the mean before a unit is cut

msa_status fail(std::string* err, msa_status st, const std::string& msg) {
  *err = msg;
  return st;
}

bool aligned8(int64_t x) { return x > 0 && (x % 8) == 0; }

struct Unit {
  int32_t seq, kv_head, row0, nrows, kv_hi;
};

}  // namespace

msa_status build_plan(const msa_shape* shape, const int32_t* seq_kv_len, const int32_t* seg_indptr,
                      const int32_t* seg_start, const int32_t* seg_len, const msa_plan_opts* opts,
                      HostPlan* out, std::string* err) {
  if (!shape || !out) return fail(err, MSA_ERR_INVALID_ARG, "shape and out must be non-null");
  const msa_shape& s = *shape;
  msa_plan_opts o{};
  if (opts) o = *opts;
  for (int i = 0; i < 5; ++i)
    if (o.reserved[i] != 0) return fail(err, MSA_ERR_INVALID_ARG, "opts.reserved must be zero");
  if (o.flags & ~(MSA_PLAN_HOST_ONLY | MSA_PLAN_NO_AUTO_SPLIT | MSA_PLAN_TILE_ROWS_128 |
                  MSA_PLAN_TILE_ROWS_256 | MSA_PLAN_TILE_ROWS_32 | MSA_PLAN_PRECISE_WEIGHTS))
    return fail(err, MSA_ERR_INVALID_ARG, "unknown opts.flags bits");
  const bool forced_width = (o.flags & (MSA_PLAN_TILE_ROWS_128 | MSA_PLAN_TILE_ROWS_256 | MSA_PLAN_TILE_ROWS_32)) != 0;
  {
    const int forced = !!(o.flags & MSA_PLAN_TILE_ROWS_128) + !!(o.flags & MSA_PLAN_TILE_ROWS_256) +
                       !!(o.flags & MSA_PLAN_TILE_ROWS_32);
    if (forced > 1)
      return fail(err, MSA_ERR_INVALID_ARG, "MSA_PLAN_TILE_ROWS_32, _128 and _256 are exclusive");
  }

  if (s.num_seqs < 0) return fail(err, MSA_ERR_INVALID_ARG, "num_seqs < 0");
  if (s.num_q_heads < 1 || s.num_kv_heads < 1)
    return fail(err, MSA_ERR_INVALID_ARG, "head counts must be >= 1");
  if (s.num_q_heads % s.num_kv_heads != 0)
    return fail(err, MSA_ERR_INVALID_ARG, "num_q_heads must be a multiple of num_kv_heads");
  const int32_t G = s.num_q_heads / s.num_kv_heads;
  if (G > kTileRowsWide) return fail(err, MSA_ERR_UNSUPPORTED, "num_q_heads / num_kv_heads > 256");
  if (G > kTileRowsNarrow && (o.flags & MSA_PLAN_TILE_ROWS_128))
    return fail(err, MSA_ERR_UNSUPPORTED, "128-row tiles need num_q_heads / num_kv_heads <= 128");
  if (G > kTileRowsDecode && (o.flags & MSA_PLAN_TILE_ROWS_32))
    return fail(err, MSA_ERR_UNSUPPORTED, "32-row tiles need num_q_heads / num_kv_heads <= 32");
  if (s.head_dim <= 0) return fail(err, MSA_ERR_INVALID_ARG, "head_dim <= 0");
  if (s.head_dim != 64 && s.head_dim != 128)
    return fail(err, MSA_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (s.block_size <= 0) return fail(err, MSA_ERR_INVALID_ARG, "block_size <= 0");
  if (s.block_size != kBlockSize) return fail(err, MSA_ERR_UNSUPPORTED, "block_size must be 16");
  if (s.max_blocks_per_seq < 0 || s.num_blocks < 0)
    return fail(err, MSA_ERR_INVALID_ARG, "max_blocks_per_seq and num_blocks must be >= 0");
  if (!std::isfinite(s.scale) || !(s.scale > 0.0f))
    return fail(err, MSA_ERR_INVALID_ARG, "scale must be finite and > 0");
  if (!aligned8(s.q_stride_tok) || !aligned8(s.q_stride_head) || !aligned8(s.o_stride_tok) ||
      !aligned8(s.o_stride_head) || !aligned8(s.k_stride_block) || !aligned8(s.k_stride_head) ||
      !aligned8(s.k_stride_tok) || !aligned8(s.v_stride_block) || !aligned8(s.v_stride_head) ||
      !aligned8(s.v_stride_dim))
    return fail(err, MSA_ERR_INVALID_ARG, "strides must be positive multiples of 8 elements");
  if (o.q_tile_tokens < 0 || o.q_tile_tokens > kTileRowsWide / G)
    return fail(err, MSA_ERR_INVALID_ARG, "q_tile_tokens must be in [0, tile_rows / (Hq/Hkv)]");
  if (o.kv_split_tokens < 0 || o.kv_split_tokens % kKvStep != 0)
    return fail(err, MSA_ERR_INVALID_ARG, "kv_split_tokens must be a non-negative multiple of 64");

  const int32_t B = s.num_seqs;
  if (B > 0 && (!seq_kv_len || !seg_indptr))
    return fail(err, MSA_ERR_INVALID_ARG, "seq_kv_len and seg_indptr must be non-null");
  if (B > 0 && seg_indptr[0] != 0) return fail(err, MSA_ERR_INVALID_ARG, "seg_indptr[0] != 0");
  for (int32_t b = 0; b < B; ++b)
    if (seg_indptr[b + 1] < seg_indptr[b])
      return fail(err, MSA_ERR_INVALID_ARG, "seg_indptr must be non-decreasing");
  const int64_t nseg = B > 0 ? seg_indptr[B] : 0;
  if (nseg > 0 && (!seg_start || !seg_len))
    return fail(err, MSA_ERR_INVALID_ARG, "seg_start and seg_len must be non-null");

  // 1. rows and their absolute positions
  HostPlan& P = *out;
  P = HostPlan{};
  P.shape = s;
  P.group = G;
  P.precise_weights = (o.flags & MSA_PLAN_PRECISE_WEIGHTS) != 0;
  std::vector<int64_t> seq_row0(B + 1, 0);
  std::vector<int32_t> seq_maxpos(B, -1);
  int64_t total = 0;
  const int64_t cap = (int64_t)s.max_blocks_per_seq * s.block_size;
  for (int32_t b = 0; b < B; ++b) {
    const int32_t L = seq_kv_len[b];
    if (L < 0 || L > cap)
      return fail(err, MSA_ERR_INVALID_ARG,
                  "seq_kv_len[" + std::to_string(b) + "] outside [0, max_blocks_per_seq*16]");
    int64_t prev_end = 0;
    seq_row0[b] = total;
    for (int32_t k = seg_indptr[b]; k < seg_indptr[b + 1]; ++k) {
      const int64_t st = seg_start[k], n = seg_len[k];
      if (n < 1) return fail(err, MSA_ERR_INVALID_ARG, "segment " + std::to_string(k) + " is empty");
      if (st < prev_end)
        return fail(err, MSA_ERR_INVALID_ARG,
                    "segment " + std::to_string(k) + " overlaps or is out of order");
      if (st + n > L)
        return fail(err, MSA_ERR_INVALID_ARG,
                    "segment " + std::to_string(k) + " extends past seq_kv_len");
      total += n;
      if (total >= ((int64_t)1 << 31)) return fail(err, MSA_ERR_INVALID_ARG, "total_q >= 2^31");
      prev_end = st + n;
      seq_maxpos[b] = (int32_t)(st + n - 1);
    }
  }
  seq_row0[B] = total;
  P.total_q = total;
  P.seq_blocks.resize((size_t)B);
  for (int32_t b = 0; b < B; ++b) P.seq_blocks[(size_t)b] = seq_maxpos[b] >= 0 ? seq_maxpos[b] / kBlockSize + 1 : 0;
  P.row_pos.resize((size_t)total);
  {
    int64_t r = 0;
    for (int32_t b = 0; b < B; ++b)
      for (int32_t k = seg_indptr[b]; k < seg_indptr[b + 1]; ++k)
        for (int32_t t = 0; t < seg_len[k]; ++t) P.row_pos[(size_t)r++] = seg_start[k] + t;
  }
  // 2. tiles of up to `tt` consecutive tokens of one sequence, packed
  // across segment gaps while the keys masked for the earlier rows stay a
  // small part of the tile's work; one unit per tile and KV head
  auto make_units = [&](int32_t tt) {
    std::vector<Unit> units;
    for (int32_t b = 0; b < B; ++b) {
      const int64_t lo = seq_row0[b], hi = seq_row0[b + 1];
      int64_t i = lo;
      while (i < hi) {
        const int64_t first = i;
        double useful = (double)P.row_pos[(size_t)i] + 1.0, waste = 0.0;
        int32_t cnt = 1;
        ++i;
        while (i < hi && cnt < tt) {
          const double step = (double)P.row_pos[(size_t)i] - (double)P.row_pos[(size_t)(i - 1)];
          const double nw = waste + cnt * step;
          const double nu = useful + (double)P.row_pos[(size_t)i] + 1.0;
          if (nw > kWasteFrac * nu && nw > (double)kKvStep * tt) break;
          waste = nw;
          useful = nu;
          ++cnt;
          ++i;
        }
        const int32_t kv_hi = P.row_pos[(size_t)(first + cnt - 1)] + 1;
        for (int32_t g = 0; g < s.num_kv_heads; ++g) units.push_back(Unit{b, g, (int32_t)first, cnt, kv_hi});
      }
    }
    return units;
  };

  // tile width: forced by a flag, else 32 rows when no 128-row tile would
  // hold more than 32 rows (decode-like plans), wide when the narrow tiling
  // has full tiles and enough work per workgroup slot (G > 128 needs wide
  // tiles), else narrow
  const int32_t narrow_tokens = G <= kTileRowsNarrow ? kTileRowsNarrow / G : 0;
  std::vector<Unit> narrow_units;
  {
    int32_t rows = kTileRowsNarrow;
    if (o.flags & MSA_PLAN_TILE_ROWS_256) {
      rows = kTileRowsWide;
    } else if (o.flags & MSA_PLAN_TILE_ROWS_32) {
      rows = kTileRowsDecode;
    } else if (!(o.flags & MSA_PLAN_TILE_ROWS_128)) {
      if (G > kTileRowsNarrow) {
        rows = kTileRowsWide;
      } else {
        narrow_units = make_units(narrow_tokens);
        double steps = 0, row_steps = 0;
        int64_t max_rows = 0;
        for (const Unit& u : narrow_units) {
          const double st = (double)((u.kv_hi + kKvStep - 1) / kKvStep);
          steps += st;
          row_steps += st * u.nrows;
          max_rows = std::max<int64_t>(max_rows, (int64_t)u.nrows * G);
        }
        // Units that are never cut take as long as the longest chain, and up to
        // one narrow unit per CU, a narrow step is the shorter (30K keys, d = 128:
        // 120 narrow units 365 us, 60 wide ones 596; past that, narrow units share
        // CUs: 264 narrow 615, 132 wide 611, 476 and 238 762 / 742).
        // The width decides which q_tile_tokens are accepted and how much
        // memory the pieces of a forced split length take, so plans with either
        // option widen by the 64-wide rule alone, at both head dimensions: a
        // rule tuned for speed must not move those limits.
        const bool given = o.q_tile_tokens > 0 || o.kv_split_tokens > 0;
        const bool late = given || s.head_dim == 64;
        if (!narrow_units.empty() && max_rows <= kTileRowsDecode)
          rows = kTileRowsDecode;
        else if (steps >= (late ? kWideMinStepsPerSlot64 : kWideMinStepsPerSlot) * 2.0 * kCUs &&
                 (given || row_steps >= kWideMinFill * steps * narrow_tokens) &&
                 (!late || (int64_t)narrow_units.size() >= kWideMinTiles64) &&
                 (!(o.flags & MSA_PLAN_NO_AUTO_SPLIT) || (int64_t)narrow_units.size() > kCUs))
          rows = kTileRowsWide;
      }
    }
    P.tile_rows = rows;
    P.tile_tokens = rows / G;
    if (o.q_tile_tokens > P.tile_tokens)
      return fail(err, MSA_ERR_INVALID_ARG, "q_tile_tokens must be in [0, tile_rows / (Hq/Hkv)]");
    if (o.q_tile_tokens > 0) P.tile_tokens = o.q_tile_tokens;
    P.item_rows = rows;
  }
  auto steps = [](int64_t keys) { return (keys + kKvStep - 1) / kKvStep; };
  // shortest 64-aligned length >= lo that cuts the units of more than `whole`
  // keys into at most `most` pieces, counting the uncut ones
  auto shortest_cut = [&](const std::vector<Unit>& us, int64_t lo, int64_t whole, int64_t most) {
    int64_t hi = lo;
    for (const Unit& u : us) hi = std::max(hi, steps(u.kv_hi) * kKvStep);
    while (lo < hi) {
      const int64_t mid = (lo / kKvStep + hi / kKvStep) / 2 * kKvStep;
      int64_t c = 0;
      for (const Unit& u : us) c += u.kv_hi > whole ? (u.kv_hi + mid - 1) / mid : 1;
      if (c <= most) hi = mid; else lo = mid + kKvStep;
    }
    return lo;
  };
  // Few short tiles: each 128-row tile runs as items of up to 32 rows whose
  // four waves split the keys, while such items have a CU each.  A call that
  // small lasts as long as its longest chain of key steps, and 128 keys of a
  // 32-row item take as long as 64 of a 128-row tile (two 64-token segments at
  // 512 keys, 8 tiles: 9.5 us as tiles, 6.2 us as 16 items; 56 tiles of a
  // 1.7K prompt 18.9 and 12.9 us).  Past one item per CU the chains queue up
  // and the K/V reads, no longer shared by 128 rows, cost more than they save
  // (192 tiles at 0.8K keys: 20.0 us, 20.2 us as 768 items; 344 tiles: 24.9
  // and 42 us); nor do long units pay, which tiles cut finer (58 tiles of up
  // to 28.9K keys: 93 us, 195 us as items).
  // Not with a forced split length: it cuts the items far past one per CU (32
  // tiles at 2K keys, 104 items, pieces of 64 keys: 1016 partials of tiles, 3296
  // of items, 64 and 208 MiB), and what a caller gets for it, the partials'
  // memory and whether they fit msa_forward_noalloc, is that of 128-row tiles.
  if (!forced_width && o.q_tile_tokens == 0 && o.kv_split_tokens == 0 && P.tile_rows == kTileRowsNarrow &&
      G <= kTileRowsDecode && (int64_t)narrow_units.size() < kCUs) {
    std::vector<Unit> items = make_units(kTileRowsDecode / G);
    if ((int64_t)items.size() < kCUs) {
      int64_t longest = 0, total_steps = 0;
      for (const Unit& u : narrow_units) {
        longest = std::max(longest, steps(u.kv_hi));
        total_steps += steps(u.kv_hi);
      }
      const int64_t tile_chain = std::min(longest, std::max<int64_t>(kMinSplitSteps, total_steps / kCUs));
      const int64_t item_chain =
          std::min(longest, shortest_cut(items, kMinSplitKeysDecode, kWholeKeysDecode, kCUs) / kKvStep);
      if (2 * item_chain <= 3 * tile_chain) {
        P.item_rows = kTileRowsDecode;
        P.tile_tokens = kTileRowsDecode / G;
        narrow_units.clear();
      }
    }
  }
  const int32_t tile_tokens = P.tile_tokens;
  const int64_t slots_total = (int64_t)kCUs * (P.tile_rows == kTileRowsWide ? 1 : 2);

  // slices of the cache write: each segment cut at cache-block boundaries
  {
    int64_t r = 0;
    for (int32_t b = 0; b < B; ++b)
      for (int32_t k = seg_indptr[b]; k < seg_indptr[b + 1]; ++k) {
        int32_t p = seg_start[k];
        const int32_t end = seg_start[k] + seg_len[k];
        while (p < end) {
          const int32_t stop = std::min(end, (p / kBlockSize + 1) * kBlockSize);
          P.append.push_back(AppendItem{(int32_t)r, b, p, stop - p});
          r += stop - p;
          p = stop;
        }
      }
  }

  // 3. units of the chosen width
  std::vector<Unit> units = narrow_units.empty() || tile_tokens != narrow_tokens ? make_units(tile_tokens)
                                                                                : std::move(narrow_units);
  const int32_t Hkv = s.num_kv_heads, d = s.head_dim;
  P.num_tiles = (int64_t)units.size();

  // 4. key splits decided by length alone: forced, or those of 32-row plans.
  // Other plans cut units where the workgroups' loads need it (step 6).
  const bool auto_split = o.kv_split_tokens == 0 && !(o.flags & MSA_PLAN_NO_AUTO_SPLIT);
  const bool cut_to_fit = auto_split && P.item_rows != kTileRowsDecode;
  int64_t split_keys = o.kv_split_tokens;  // 0: no split
  int64_t whole_keys = 0;  // units of up to this many keys are not split
  if (auto_split && P.item_rows == kTileRowsDecode && !units.empty() && (int64_t)units.size() <= slots_total) {
    // 32-row items (decode-like, bound by K/V streaming; the four waves of
    // a workgroup already split an item's keys): all pieces in one round
    // of the workgroup slots, the longest piece as short as possible, i.e.
    // the shortest 64-aligned piece length whose piece count fits the
    // slots (no split if the units alone exceed them)
    split_keys = shortest_cut(units, kKvStep, 0, slots_total);
    // Pieces below 1024 keys pay only while each has a CU to itself (8 heads
    // at 8K keys: 16.1 us in pieces of 1024 keys, 12.9 of 512, 12.2 of 256;
    // 58 units of up to 6.9K keys: 20.8 us in 228 pieces, 21.7 in 426), and
    // not for units whose chain is no longer than the merge launch takes.
    if (split_keys < kMinSplitKeys || P.tile_rows != kTileRowsDecode) {
      whole_keys = kWholeKeysDecode;
      split_keys = shortest_cut(units, kMinSplitKeysDecode, whole_keys, kCUs);
      if (P.tile_rows == kTileRowsDecode) split_keys = std::min(split_keys, kMinSplitKeys);
      int64_t longest = 0, kept = 0;  // of all units, of those that stay whole
      for (const Unit& u : units) {
        longest = std::max<int64_t>(longest, u.kv_hi);
        if (u.kv_hi <= whole_keys) kept = std::max<int64_t>(kept, u.kv_hi);
      }
      // (a merge launch takes as long as a chain of 500 keys: 216 items of up to
      // 1.7K keys 13.8 us in pieces of up to 1408, 12.9 whole.  Decode rows of up
      // to 1024 keys are cut only if the rows that stay whole are that much
      // shorter too: 64 items at d = 64, 9 of them 1024 keys long, take 8.7 us
      // whole and 9.5 cut beside rows of 650 keys, 8.7 and 7.7 beside 300.)
      int64_t rest = split_keys;
      if (P.tile_rows == kTileRowsDecode && longest <= kMinSplitKeys) rest = std::max(rest, kept);
      if (longest - rest < 2 * kMinSplitKeysDecode) split_keys = 0;
    }
  }
  // A chunk is a run of key steps of one unit that is handed to workgroups
  // whole or, if cuttable, piece by piece.
  struct Piece {
    int32_t unit, lo, hi, wg;
  };
  const double ov = P.item_rows == kTileRowsDecode ? kItemStepsDecode : kItemSteps;
  auto pcost = [&](const Piece& p) { return (double)steps(p.hi - p.lo) + ov; };
  std::vector<Piece> chunks;
  chunks.reserve(units.size());
  const int64_t ngroups = (int64_t)B * Hkv;
  auto group_of = [&](const Piece& p) {
    const Unit& u = units[(size_t)p.unit];
    return (size_t)((int64_t)u.seq * Hkv + u.kv_head);
  };
  std::vector<int32_t> gptr((size_t)ngroups + 1, 0);  // chunks of a group, counted here and placed below
  std::vector<double> gcost((size_t)ngroups, 0.0), gmax((size_t)ngroups, 0.0);
  double total_cost = 0;
  for (size_t ui = 0; ui < units.size(); ++ui) {
    const Unit& u = units[ui];
    int64_t chunk = u.kv_hi;
    if (split_keys > 0 && u.kv_hi > std::max(split_keys, whole_keys)) {  // equal 64-aligned chunks, the last one takes the remainder
      const int64_t nsplit = (u.kv_hi + split_keys - 1) / split_keys;
      chunk = steps((u.kv_hi + nsplit - 1) / nsplit) * kKvStep;
    }
    for (int64_t a = 0; a < u.kv_hi; a += chunk) {
      const Piece p{(int32_t)ui, (int32_t)a, (int32_t)std::min<int64_t>(u.kv_hi, a + chunk), -1};
      const size_t gi = group_of(p);
      const double c = pcost(p);
      chunks.push_back(p);
      ++gptr[gi + 1];
      gcost[gi] += c;
      gmax[gi] = std::max(gmax[gi], c);
      total_cost += c;
    }
  }

  // 5. XCDs: a group (sequence, KV head) keeps to one XCD, whose L2 then
  // holds its K/V, as long as that XCD's load stays within kHomeSlack of the
  // mean.  A group that fits nowhere (few or uneven groups) is spread over
  // the fewest XCDs that have room for it: 18 equal groups kept whole leave
  // XCDs with three groups beside XCDs with two (prompts of 10K tokens, 2 KV
  // heads: 2220 us whole, 1620 us spread).
  std::vector<int32_t> gchunk(chunks.size());  // chunk ids by group, longest first
  std::vector<int32_t> gorder;                 // groups by decreasing cost
  {
    for (int64_t gi = 0; gi < ngroups; ++gi) {
      if (gptr[(size_t)gi + 1] > 0) gorder.push_back((int32_t)gi);
      gptr[(size_t)gi + 1] += gptr[(size_t)gi];
    }
    std::vector<int32_t> at(gptr.begin(), gptr.end() - 1);
    for (size_t ci = chunks.size(); ci-- > 0;)  // backwards: a group's later tiles have more keys
      gchunk[(size_t)at[group_of(chunks[ci])]++] = (int32_t)ci;
    auto longer = [&](int32_t a, int32_t b) {
      return steps(chunks[(size_t)a].hi - chunks[(size_t)a].lo) > steps(chunks[(size_t)b].hi - chunks[(size_t)b].lo);
    };
    for (int32_t gi : gorder) {
      auto first = gchunk.begin() + gptr[(size_t)gi], last = gchunk.begin() + gptr[(size_t)gi + 1];
      if (!std::is_sorted(first, last, longer)) std::stable_sort(first, last, longer);
    }
  }
  std::stable_sort(gorder.begin(), gorder.end(),
                   [&](int32_t a, int32_t b) { return gcost[(size_t)a] > gcost[(size_t)b]; });
  const double mean = total_cost / kXcds;
  const double full = mean * (1.0 + kHomeSlack), full_small = mean * (1.0 + kHomeSlackSmall);
  std::vector<double> load(kXcds, 0.0);
  struct Part {  // a group's chunks on one XCD: first .. last of that XCD's list
    int32_t group;
    size_t first, last;
  };
  std::vector<std::vector<int32_t>> queue(kXcds);
  std::vector<std::vector<Part>> parts(kXcds);
  auto place = [&](int32_t gi, bool whole) {  // whole: not at all if it does not fit one XCD
    int by_load[kXcds];  // least loaded first, then lowest (std::stable_sort would allocate on every call)
    for (int x = 0; x < kXcds; ++x) {
      int i = x;
      for (; i > 0 && load[(size_t)x] < load[(size_t)by_load[i - 1]]; --i) by_load[i] = by_load[i - 1];
      by_load[i] = x;
    }
    if (whole && load[(size_t)by_load[0]] + gcost[(size_t)gi] > full_small) return false;
    int k = 1;
    if (!whole)
      for (double room = full - load[(size_t)by_load[0]]; k < kXcds && room < gcost[(size_t)gi];)
        room += full - load[(size_t)by_load[k++]];
    for (int i = 0; i < k; ++i) {
      const size_t n = queue[(size_t)by_load[i]].size();
      parts[(size_t)by_load[i]].push_back(Part{gi, n, n});
    }
    for (int32_t ci = gptr[(size_t)gi]; ci < gptr[(size_t)gi + 1]; ++ci) {
      int x = by_load[0];
      for (int i = 1; i < k; ++i)
        if (load[(size_t)by_load[i]] < load[(size_t)x]) x = by_load[i];
      load[(size_t)x] += pcost(chunks[(size_t)gchunk[(size_t)ci]]);
      queue[(size_t)x].push_back(gchunk[(size_t)ci]);
      ++parts[(size_t)x].back().last;
    }
    return true;
  };
  // small groups first, while they fit whole; the larger ones fill the rest
  std::vector<int32_t> later;
  for (int32_t gi : gorder)
    if (gcost[(size_t)gi] > 0.5 * mean || !place(gi, true)) later.push_back(gi);
  for (int32_t gi : later) place(gi, false);

  // 6. workgroups: one persistent workgroup per slot (256 for 256-row
  // tiles, one per CU; 512 otherwise, two per CU), fewer for small plans.
  // Workgroup i runs on XCD i % 8 and works through its own list of items,
  // so no workgroup waits for a dispatch between items.  Each XCD's chunks
  // go to the least-loaded workgroup of that XCD, groups by decreasing
  // longest chunk (then by id) and a group's chunks longest first, so that
  // the workgroups of an XCD work on the same groups at the same time and
  // share their K/V in that XCD's L2, and no long piece is left for the end.
  // A chunk that would fill a workgroup past the XCD's mean load is cut
  // there and its remainder goes back to the group's queue: a few cut units
  // even out the workgroups, where cutting every long unit sends more
  // partial results through the workspace (20 mixed sequences up to 4.6K,
  // 64 heads: 150 us with 512 of 944 units cut, 118 us with 240).
  const int wgs_per_xcd = (int)(slots_total / kXcds);
  // a cut adds at most two partials: all of them fit the workspace of msa_forward_noalloc
  int64_t cuts_left = (int64_t)(MSA_NOALLOC_WORKSPACE_BYTES / sizeof(float)) / slot_floats(d, P.tile_rows) / 2;
  std::vector<Piece> pieces;
  pieces.reserve(chunks.size() + (size_t)slots_total);
  std::vector<int32_t> unit_count(units.size(), 0);
  for (int x = 0; x < kXcds; ++x) {
    const auto& qx = queue[(size_t)x];
    if (qx.empty()) continue;
    auto& px = parts[(size_t)x];
    std::stable_sort(px.begin(), px.end(), [&](const Part& a, const Part& b) {
      const double ma = gmax[(size_t)a.group], mb = gmax[(size_t)b.group];
      return ma != mb ? ma > mb : a.group < b.group;
    });
    // capacity of a workgroup before a chunk is cut
    double capacity = 0.0;
    if (cut_to_fit) {
      auto pieces_at = [&](int64_t len) {
        int64_t c = 0;
        for (int32_t ci : qx) c += (steps(chunks[(size_t)ci].hi) + len - 1) / len;
        return c;
      };
      int64_t key_steps = 0, longest = kMinSplitSteps;
      for (int32_t ci : qx) {
        key_steps += steps(chunks[(size_t)ci].hi);
        longest = std::max(longest, steps(chunks[(size_t)ci].hi));
      }
      // the mean load, counting the items that cuts at that load would add
      double mean_load = load[(size_t)x] / wgs_per_xcd;
      if ((double)longest + ov > mean_load)
        for (int it = 0; it < 2; ++it) {
          const int64_t len = std::max<int64_t>(kMinSplitSteps, (int64_t)(mean_load - ov));
          const double items = std::min((double)pieces_at(len), (double)qx.size() + wgs_per_xcd);
          mean_load = ((double)key_steps + ov * items) / wgs_per_xcd;
        }
      // where no chunk has to be cut, a cut must also win back the merge launch
      capacity = mean_load * (1.0 + kCutSlack) + ((double)longest + ov > mean_load ? 1.0 : kItemSteps);
      // few chunks: the shortest length whose pieces take one workgroup
      // each, if that is no longer than packing them would take
      if ((int64_t)qx.size() <= wgs_per_xcd) {
        int64_t lo = kMinSplitSteps, hi = longest;
        while (lo < hi) {
          const int64_t mid = (lo + hi) / 2;
          if (pieces_at(mid) <= wgs_per_xcd) hi = mid; else lo = mid + 1;
        }
        if ((double)lo + ov <= kOneRoundFactor * capacity) capacity = (double)lo + ov;
      }
      capacity = std::max(capacity, kMinSplitSteps + ov);
    }
    typedef std::pair<double, int> Slot;  // (load, workgroup of this XCD): least loaded first, then lowest
    std::vector<Slot> slots;  // heap of the workgroups in use; pieces take the idle ones first, in turn
    slots.reserve((size_t)wgs_per_xcd);
    auto shorter = [&](const Piece& a, const Piece& b) { return a.hi - a.lo < b.hi - b.lo; };
    std::priority_queue<Piece, std::vector<Piece>, decltype(shorter)> tails(shorter);
    for (const Part& part : px) {
      for (size_t qi = part.first; qi < part.last || !tails.empty();) {
        // the longest of the group's remaining chunks and cut-off tails
        Piece p;
        if (qi < part.last && (tails.empty() || !shorter(chunks[(size_t)qx[qi]], tails.top()))) {
          p = chunks[(size_t)qx[qi++]];
        } else {
          p = tails.top();
          tails.pop();
        }
        Slot s0(0.0, (int)slots.size());
        if (s0.second == wgs_per_xcd) {
          std::pop_heap(slots.begin(), slots.end(), std::greater<Slot>());
          s0 = slots.back();
          slots.pop_back();
        }
        const int64_t n = steps(p.hi - p.lo);
        if (cut_to_fit && cuts_left > 0 && n > kMinSplitSteps && s0.first + (double)n + ov > capacity) {
          --cuts_left;
          const int64_t fit = (int64_t)(capacity - s0.first - ov);
          const int64_t take = std::min(std::max(fit, kMinTailSteps), n - kMinTailSteps);
          const int32_t mid = (int32_t)(p.lo + take * kKvStep);
          tails.push(Piece{p.unit, mid, p.hi, -1});
          p.hi = mid;
        }
        p.wg = s0.second * kXcds + x;
        pieces.push_back(p);
        ++unit_count[(size_t)p.unit];
        s0.first += pcost(p);
        slots.push_back(s0);
        std::push_heap(slots.begin(), slots.end(), std::greater<Slot>());
      }
    }
  }
  // workspace slots of the split units, in unit and key order
  std::vector<int32_t> unit_slot0(units.size(), -1);
  for (size_t ui = 0; ui < units.size(); ++ui) {
    const int32_t n = unit_count[ui];
    if (n < 2) continue;
    const Unit& u = units[ui];
    unit_slot0[ui] = (int32_t)P.num_slots;
    P.merge.push_back(MergeItem{u.seq, u.kv_head, u.row0, u.nrows, n, (int32_t)P.num_slots, 0, 0});
    P.max_splits = std::max<int64_t>(P.max_splits, n);
    P.max_merge_rows = std::max<int32_t>(P.max_merge_rows, u.nrows * G);
    P.num_slots += n;
  }
  P.workspace_bytes = P.num_slots * slot_floats(d, P.tile_rows) * (int64_t)sizeof(float);
  std::vector<int32_t> slot_lo((size_t)P.num_slots);  // first key of each slot's piece
  {
    std::vector<int32_t> filled(units.size(), 0);
    for (const Piece& p : pieces)
      if (unit_slot0[(size_t)p.unit] >= 0)
        slot_lo[(size_t)(unit_slot0[(size_t)p.unit] + filled[(size_t)p.unit]++)] = p.lo;
    for (const MergeItem& m : P.merge)
      std::sort(slot_lo.begin() + m.slot0, slot_lo.begin() + m.slot0 + m.nsplit);
  }
  // the items by workgroup, in run order; trailing workgroups with nothing to do are not launched
  int32_t launched = 0;
  for (const Piece& p : pieces) launched = std::max(launched, p.wg + 1);
  P.wg_ptr.assign((size_t)launched + 1, 0);
  for (const Piece& p : pieces) ++P.wg_ptr[(size_t)p.wg + 1];
  for (int32_t i = 0; i < launched; ++i) P.wg_ptr[(size_t)i + 1] += P.wg_ptr[(size_t)i];
  P.work.resize(pieces.size());
  {
    std::vector<int32_t> at(P.wg_ptr.begin(), P.wg_ptr.end() - 1);
    for (const Piece& p : pieces) {
      const Unit& u = units[(size_t)p.unit];
      int32_t slot = unit_slot0[(size_t)p.unit];
      if (slot >= 0) {
        const auto first = slot_lo.begin() + slot;
        slot += (int32_t)(std::lower_bound(first, first + unit_count[(size_t)p.unit], p.lo) - first);
      }
      P.work[(size_t)at[(size_t)p.wg]++] =
          WorkItem{u.seq, u.kv_head, u.row0, u.nrows, p.lo, p.hi, slot, p.wg};
    }
  }

  // figures
  const double hq = s.num_q_heads;
  for (int64_t r = 0; r < total; ++r) P.useful_flops += 4.0 * d * hq * ((double)P.row_pos[(size_t)r] + 1);
  const double qo_bytes = 2.0 * 2.0 * (double)total * hq * d;  // Q read + O write, bf16
  P.planned_bytes = qo_bytes;
  for (const WorkItem& w : P.work) {
    if (w.nrows == 0) continue;
    const double keys = (double)(w.kv_hi - w.kv_lo);
    P.planned_bytes += keys * d * 2.0 * 2.0;
    // waves whose 32 rows are all empty skip every step
    const double rows = (double)((w.nrows * G + 31) / 32 * 32);
    // 32-row tiles run 32-key half-steps, the others 64-key steps
    const int64_t gran = P.item_rows == kTileRowsDecode ? kKvStep / 2 : kKvStep;
    P.tile_flops += 4.0 * d * rows * (double)((w.kv_hi - w.kv_lo + gran - 1) / gran * gran);
  }
  P.min_bytes = qo_bytes;
  for (int32_t b = 0; b < B; ++b)
    if (seq_maxpos[b] >= 0) P.min_bytes += (double)(seq_maxpos[b] + 1) * d * 2.0 * 2.0 * Hkv;
  return MSA_OK;
}

}  // namespace msa
