// Work decomposition of a step: how many work-groups each launch runs and how
// the workspace is carved, a pure function of the shape (vp_shape). Kept apart
// from the ABI's validation code: these choices, with the kernels, set what
// the passes read and write.
#include <algorithm>

#include "vp_internal.h"

namespace vp {
namespace {
size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }
}  // namespace

// queries per sequence, and selection rows per query: one, or one per KV group
int queries(const vp_shape& s) { return s.n_queries > 1 ? s.n_queries : 1; }
int rows_per_query(const vp_shape& s) { return s.scope == VP_SCOPE_KV_GROUP ? s.n_kv_heads : 1; }
int rows_per_seq(const vp_shape& s) { return queries(s) * rows_per_query(s); }

// Parts of the one launch of both passes: one resident round of work-groups
// (resident_groups), so that none waits for a second one, shared by kPartWaves
// waves per part: a part's statistics and value partial are written once for
// four waves, where one wave per part and role left the select and merge
// launches 256 partials per head to read at one 30k-token sequence (per pass
// 61.8 -> 49.2 us there, 80.5 -> 76.5 at the ragged 16-sequence batch).
#ifndef VP_ONE_LAUNCH_TILES
#define VP_ONE_LAUNCH_TILES 1  // 32-row tiles per wave of the one launch, at least
#endif
#ifndef VP_LATER_TEXT_WAVES
#define VP_LATER_TEXT_WAVES 1024  // waves of a later layer's text pass with single-wave parts
#endif
// The visual and text passes in two launches (large caches) take three
// quarters of that, one wave each: 6 parts per KV head at the 64 x 32k batch, where 4, 5, 6,
// 7 and 8 parts measured 660, 631, 613.6, 618.5 and 616.5 us per step (the
// visual pass 265 / 238 / 222 / 226 / 225 us; the text pass 328.5 us at 4 parts
// and within 1 us of 325 us at 5 to 8).
#ifndef VP_TWO_LAUNCH_PARTS
#define VP_TWO_LAUNCH_PARTS 1536
#endif
#ifndef VP_MIN_TILES
#define VP_MIN_TILES 2  // 32-row tiles per context-pass part, at least
#endif

// Both context passes in one launch: saves a launch and overlaps the two
// passes' latency chains where the cache is small; kept apart otherwise, so
// the visual pass's logit writes stay out of the text pass's read stream.
// Two launches and one, us per step with four-wave parts: 8 x 9.1k tokens, 28/4 heads (9k
// tiles) 51.3 and 46.2, 16 ragged (25k) 70.3 and 68.8, 16 x 12k (24k) 85.7 and
// 85.5; past the line neither wins: 127.4 and 126.1 at 40k tiles, 132.0 and 126.9 at
// 52k (ragged), but 108.2 and 111.3 at 33k, 132.1 and 135.7 at 44k, 174.2 and 179.4 at
// 59k; the 64 x 32k batch (262k tiles) lost 100 us (one-wave parts).
#ifndef VP_DUAL_MAX_TILES
#define VP_DUAL_MAX_TILES 32768  // 32-row tiles over the batch and KV heads
#endif
bool use_dual(const vp_shape* s) {
  const int64_t tiles = static_cast<int64_t>(s->batch) * s->n_kv_heads * ((s->max_seq_len + 31) / 32);
  return tiles <= static_cast<int64_t>(VP_DUAL_MAX_TILES);
}

#ifndef VP_KEPT_WGS
#define VP_KEPT_WGS 2048  // kept-pass work-groups in one resident round (8 per CU)
#endif

#ifndef VP_MERGE_KEPT_WGS
#define VP_MERGE_KEPT_WGS 64  // kept-pass work-groups at most for the kept rows to be merged directly
#endif

#ifndef VP_SELECT_WGS
#define VP_SELECT_WGS 256  // target work-groups of the select launch: one per CU
#endif

Plan make_plan(const vp_shape& s) {
  Plan p{};
  // Context pass: parts of kPartWaves waves (one launch; small fp32 steps one wave) or one wave (two
  // launches). Tiles are dealt out cyclically, so every part sees the sequence's own mix of visual and text rows: consecutive
  // work-groups land on different XCDs, and contiguous chunks would hand whole
  // XCDs only visual (K) or only text (K + V) rows.
  const int64_t pairs = static_cast<int64_t>(s.batch) * s.n_kv_heads;
  const int64_t tiles = (s.max_seq_len + 31) / 32;
  const bool one_launch = use_dual(&s);
  p.waves = one_launch ? kPartWaves : 1;
  const int64_t min_tiles = one_launch ? kPartWaves * VP_ONE_LAUNCH_TILES : VP_MIN_TILES;
  auto capped = [&](int64_t n, int64_t least) {
    return static_cast<int>(std::max<int64_t>(1, std::min(n, (tiles + least - 1) / least)));
  };
  // A round is what is resident at a time. Parts are rounded down to one: a second
  // round of bf16 parts measured 1.09 to 1.12 times the step at 72 to 192 pairs. The exceptions:
  // * fp32 rows of 128 (one work-group per CU) with more than 32 pairs and two tiles per
  //   wave or more: two rounds. A batch's sequences differ in length, and with so few
  //   work-groups the CUs of the short ones stay idle in one round (16 x 28/4 heads
  //   x 3k to 10k tokens 103.6 and 94.3 us per step, 9 x 4k to 12k 85.1 and 75.1;
  //   of equal length 98.3 and 101.6 at 16 x 7k, 60.5 and 64.4 at 96 pairs x 2k). Fewer
  //   pairs or shorter sequences: one (4 x 11k 56.2 and 62.1, 48 pairs x 745 35.9 and 39.8).
  // * two parts where one per pair leaves a good part of the round, or of the second
  //   one, idle. bf16 above half a round, one and two parts: 125.2 and 121.4 us at
  //   264 pairs, 93.4 and 89.7 at 288, 104.4 and 103.0 at 504, but 105.8 and 109.0 at 384.
  //   Above one round: bf16 113.4 and 107.9 at 640, 110.4 and 103.7 at 768; fp32
  //   rows of 128 162.5 and 146.4 at 272, 191 and 179 at 384, but 137 and 151 at 416.
  const int64_t round = resident_groups(s.dtype, s.head_dim);
  const bool single_group = round == 256;  // one work-group per CU
  const bool two_rounds = single_group && pairs > 32 && pairs <= round && tiles >= 2 * kPartWaves * (2 * round / pairs);
  const bool two_parts =
      pairs > round ? 2 * pairs <= 3 * round
                    : !single_group && 2 * pairs > round && pairs < round && (4 * pairs < 3 * round || 8 * pairs >= 7 * round);
  const bool many_pairs = one_launch && pairs > 256;
  p.nparts = !one_launch ? capped((VP_TWO_LAUNCH_PARTS + pairs - 1) / pairs, min_tiles)
                         : capped(two_parts ? 2 : (two_rounds ? 2 * round : round) / pairs, min_tiles);
  // A later layer's text pass has the context pass's parts, but with many pairs
  // single-wave parts, one to four per pair: they balance the text rows alone
  // better (a later layer with four-wave parts and here: 68.1 and 64.8 us at 264
  // pairs, 56.0 and 50.9 at 288, 52.3 and 47.3 at 1024)
  p.text_waves = many_pairs ? 1 : p.waves;
  p.text_parts = many_pairs ? capped((VP_LATER_TEXT_WAVES + pairs - 1) / pairs, VP_MIN_TILES) : p.nparts;
  // fp32 steps whose tiles give at most one wave per CU: one tile per single-wave part
  // of both roles, so that no wave waits at the barrier of a part's merge (one head of 64:
  // 384 tokens 23.8 -> 22.7 us per step, 1800 24.7 -> 23.6; 28/4 heads of 128: 600
  // tokens 30.3 -> 29.7, 1.9k 31.0 -> 31.1; beyond, 304 tiles: 30.9 -> 34.0). fp32 only:
  // the smallest bf16 steps gained from four waves (384 tokens 22.8 -> 22.3 us).
  // A row capacity for kept rows beyond the cache's keeps four waves per part,
  // whose workspace is smaller.
  if (one_launch && s.dtype == VP_F32 && tiles <= 64 && pairs * tiles <= 256 && s.k_cap <= s.max_seq_len) {
    p.waves = p.text_waves = 1;
    p.nparts = p.text_parts = static_cast<int>(tiles);
  }
  // Kept pass: the fewest kept rows per work-group (32, 64, 128, ...) that
  // keep the launch within one resident round (VP_KEPT_WGS work-groups), so no
  // work-group waits for a second round (the 64 x 32k batch: 128 rows, 1792
  // work-groups; kept pass and merge 40.2 -> 35.9 us against 64 rows).
#ifdef VP_KEPT_SPLIT
  p.split = VP_KEPT_SPLIT;
#else
  {
    const int64_t heads = static_cast<int64_t>(s.batch) * s.n_kv_heads * queries(s);
    int64_t split = 32;
    while (split < s.k_cap && heads * ((s.k_cap + split - 1) / split) > VP_KEPT_WGS) split *= 2;
    p.split = static_cast<int>(split);
  }
#endif
  p.nsplit = (s.k_cap + p.split - 1) / p.split;
  // A later layer's kept work-groups share the launch of its text parts. Where a CU
  // holds one work-group they would wait for a whole CU to fall free: the parts
  // (the step's too, so that both give the same bits) are fewer by what they need,
  // if that is at most a quarter and no wave's chain of tiles gets longer (a later
  // layer of 4 x 3.3k tokens, 28/4 heads: 23.4 -> 17.5 us, 6 x 745, 32/8 heads: 19.6 -> 17.1; the steps
  // within 0.3 us). With two per CU the steps lose as much as the later layers
  // gain (2 x 3.6k tokens, 32/32 heads: 38.9 -> 40.5 and 23.6 -> 23.2 us).
  if (p.waves > 1 && single_group && !many_pairs) {
    const int64_t kept = (static_cast<int64_t>(queries(s)) * p.nsplit + kPartWaves - 1) / kPartWaves;
    const int64_t room = round / pairs - kept;
    auto chain = [&](int64_t parts) { return (tiles + kPartWaves * parts - 1) / (kPartWaves * parts); };
    if (p.nparts > room && 4 * room >= 3 * p.nparts && chain(room) == chain(p.nparts))
      p.nparts = p.text_parts = static_cast<int>(room);
  }
  // Single-wave parts also for a later layer's few text rows: where the four-wave
  // parts and the kept work-groups exceed a round and a wave has at most two tiles of
  // text (as the row capacities have it), the second round of short work-groups costs
  // more than the walk over the text; single-wave parts and the kept splits
  // share one round (a later layer of 16 x 300 text and 4000 visual tokens, 28/4 heads: 17.0
  // -> 14.1 us, 60 x 250 and 1000 21.2 -> 18.9, fp32 16 x 300 and 4000 35.7 -> 24.7; at
  // 2.4 to 2.8 tiles the four-wave parts are as fast).
  const int64_t kept_splits = static_cast<int64_t>(queries(s)) * p.nsplit;
  const int64_t text_tiles = s.max_seq_len > s.max_vis ? (s.max_seq_len - s.max_vis + 31) / 32 : 0;
  const int single_parts = capped((VP_LATER_TEXT_WAVES + pairs - 1) / pairs, VP_MIN_TILES);
  const bool few_text = p.waves > 1 && pairs > 16 && !many_pairs &&
                        pairs * (p.nparts + (kept_splits + kPartWaves - 1) / kPartWaves) > round &&
                        text_tiles <= 2 * kPartWaves * p.nparts && (single_parts + kept_splits) * pairs <= VP_KEPT_WGS;
  if (few_text) {
    p.text_waves = 1;
    p.text_parts = single_parts;
  }
  // A later layer (its own text rows, the anchor's kept list) launches its text
  // and kept passes together: with four-wave text parts, which fill a round by
  // themselves, when the kept splits are at most half a round of waves (text waves not
  // counted); with single-wave ones when both fit one resident round. The kept
  // work-groups then fill the text pass's tail (8 layers: 131.8 -> 98.6 us at the
  // 1-sequence batch, 381.9 -> 351.9 at the 72B-class loop); beyond one round
  // the text pass is split over two (the 64 x 32k batch: 3081 -> 3663 us).
  p.text_kept_one_launch =
      p.text_waves > 1 ? pairs * kept_splits <= VP_KEPT_WGS / 2 : (p.text_parts + kept_splits) * pairs <= VP_KEPT_WGS;
  // A step whose kept pass would be a handful of work-groups folds the kept
  // rows into the merge (their K and V rows read there): bf16 caches, every
  // text part and kept row in one batch per head.
  p.merge_kept = s.dtype == VP_BF16 &&
                 static_cast<int64_t>(p.nsplit) * queries(s) * s.n_kv_heads * s.batch <= VP_MERGE_KEPT_WGS &&
                 p.nparts <= merge_kept_max_parts(s.head_dim) && s.k_cap <= merge_kept_max_rows(s.head_dim);
  // per-head arrays hold one entry per query row (virtual head): T*Hq per sequence
  const size_t B = s.batch, Hq = static_cast<size_t>(s.n_q_heads) * queries(s), d = s.head_dim;
  p.zs_rows = ((s.max_seq_len + 31) / 32) * 32;
  p.zs_gp = queries(s) * (s.n_q_heads / s.n_kv_heads) <= 8 ? 8 : 16;
  const size_t rows = B * static_cast<size_t>(rows_per_seq(s));
  auto carve = [&] {
    size_t off = 0;
    p.zs = off;
    off = align256(off + B * static_cast<size_t>(s.n_kv_heads) * p.zs_rows * static_cast<size_t>(p.zs_gp) * 4);
    p.stats = off;
    const size_t part_slots = std::max(p.nparts, p.text_parts);
    off = align256(off + B * Hq * part_slots * 8 * 4);
    p.acc = off;
    off = align256(off + B * Hq * part_slots * d * 4);
    p.head = off;
    off = align256(off + B * Hq * 2 * 4);
    p.kstats = off;
    off = align256(off + B * Hq * p.nsplit * 2 * 4);
    p.kacc = off;
    off = align256(off + B * Hq * p.nsplit * d * 4);
    p.segtab = off;
    off = align256(off + B * kSegTableBytes);
    p.total = off;
  };
  carve();
  if (few_text && p.total > VP_STATIC_SCRATCH_BYTES) {
    // not where only the single-wave parts' partials take the step past the static scratch
    const Plan own = p;
    p.text_waves = p.waves;
    p.text_parts = p.nparts;
    p.text_kept_one_launch = pairs * kept_splits <= VP_KEPT_WGS / 2;
    carve();
    if (p.total > VP_STATIC_SCRATCH_BYTES) p = own;
  }
  // Select kernel: chunks of whole rounds (a round scores 1024 / lanes-per-token
  // visual ranks), enough rounds per chunk that the launch has about
  // VP_SELECT_WGS work-groups, so the spilled logits stream through many CUs.
  const int64_t tpr = select_tokens_per_round(s.n_kv_heads, rows_per_query(s));
  const int64_t want = static_cast<int64_t>(rows) * s.max_vis;
  int64_t rounds = (want + tpr * VP_SELECT_WGS - 1) / (tpr * VP_SELECT_WGS);
  if (rounds < 1) rounds = 1;
  const int64_t chunk = tpr * rounds;
  p.sel_chunks = static_cast<int>((s.max_vis + chunk - 1) / chunk);
  p.sel_chunk = p.sel_chunks == 1 ? s.max_vis : static_cast<int>(chunk);
  return p;
}

}  // namespace vp
