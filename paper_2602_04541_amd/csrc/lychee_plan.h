// How a launch is laid out: functions of sizes alone, in plain C++ (host, device and tests include them).
#pragma once

#include <stdint.h>

#ifdef __HIP__
#define LYCHEE_HD __host__ __device__
#else
#define LYCHEE_HD
#endif

namespace lychee {

// a / b for 0 <= a < 2^31 - b, 0 < b < 2^24, from `inv`, the reciprocal of b to one unit in its last place.  The
// product is off by at most 2^-22 of itself, so the remainder lies within 512 + b of zero, and what its
// quotient adds is at most one off.  (Unsigned up to there: q * b may pass 2^31.)  No branches.  u: what the
// caller does with a value that was computed in single precision.
template <typename U>
LYCHEE_HD inline int32_t quot_by(int32_t a, int32_t b, float inv, U u)
{
    uint32_t q = u((uint32_t)((float)a * inv));
    q += u((uint32_t)(int32_t)((float)(int32_t)((uint32_t)a - q * (uint32_t)b) * inv));
    const int32_t r = (int32_t)((uint32_t)a - q * (uint32_t)b);
    return (int32_t)(q + (r >= b ? 1u : 0u) - (r < 0 ? 1u : 0u));
}

// The generation of the layer launch after that of generation `gen`.  None is 0, also where the 32 bits wrap (30 hours
// of launches of 26 us): 0 is what a flag that nobody has written holds, and a threshold word that nobody has asked
// for (late_filter), and neither may pass for one of this launch.
constexpr uint32_t kFirstGeneration = 1;
LYCHEE_HD inline uint32_t next_generation(uint32_t gen) { return gen + 1u != 0u ? gen + 1u : kFirstGeneration; }

// Capacity, in entries, of one score row's candidate list.  A threshold unit aims at n = min(k, L)
// candidates plus six standard deviations of its sample (a few thousand at the usual sizes),
// and makes every row a candidate when L <= kDirectLen or L <= 2k.  A list that still
// overflows is not an error: the select unit then ranks the whole row itself.  Block-granular lists
// hold an entry for every block of 64 rows, the last, partial one included, each written at its place
// unasked: they must not overflow.
LYCHEE_HD inline int32_t list_row_entries(int32_t max_len, int32_t k, bool blocks)
{
    int64_t cap = 4ll * k;
    if (cap < (int64_t)k + 16384) cap = (int64_t)k + 16384;
    const int64_t per_64 = blocks ? ((int64_t)max_len + 63) / 64 : max_len / 64;
    if (cap < per_64) cap = per_64;
    const int64_t all = ((int64_t)max_len + 63) / 64 * 64;
    return (int32_t)(cap < all ? cap : all);
}

// The front units of a layer launch: workgroup w < n_front runs units w, w + n_front, ... before anything
// else, and takes pieces afterwards unless w < n_aside.
struct FrontPlan {
    int32_t n_front, n_aside;
};

// selects, copies, thresholds: how many units of each kind; gated: gather pieces of the launch wait for sets
// that its selects and copies write; r_blocks: blocks of 64 rows that the launch streams, by the sequences'
// lengths (a capacity far above the lengths says nothing about them).
//
// Pieces wait for thresholds and for gated sets, selects at the end of the grid (tail_selects) for pieces, and
// nothing else in a launch waits.  Workgroups are dealt to the XCDs in turn, every XCD starts its own in
// index order, and not all of them at once if the grid is larger than what fits the chip beside
// whatever else runs there.  So where something waits, the front units have workgroups to themselves,
// the lowest: those never wait, so that they end on every XCD whatever holds its other places; then
// the pieces, ahead of the selects on every XCD, do.
// (Copies dealt over the whole grid, whose workgroups then went on to gated gathers, needed every
// workgroup of the grid resident at once: the started ones would wait for copies of the others.)
// Fewer than eight workgroups are always resident together, and too few to set any aside.
// Copies alone (2 us) that nothing waits for are done on the way to the pieces.
//
// How many: one workgroup per unit, but never more than a quarter of the grid; and beyond a sixteenth of it
// (which a launch does not notice) only as many as run the units in turn, about 8 us each, in half of the
// time that the streaming takes (5.5 ns a block at 6 TB/s), since the pieces need the thresholds when
// they end.  On 512 workgroups, us a layer of the model loop with 32, 64 and 128 in front: 8 sequences of 16411 to 98304
// rows 142, 144, 152; 64 of 8192: 357, 271, 238; 64 of 16384: 435, 349, 360.  (By the cache's capacity, and on a
// sixteenth of the grid beside anything longer than 120 us, 64 sequences of 2000 to 5056 rows took 165 us in
// a cache of 65536 rows and 125 in one of 5056, and 64 of 8192 took 340 a layer.)
LYCHEE_HD inline FrontPlan front_plan(int32_t selects, int32_t copies, int32_t thresholds, bool gated, int32_t r_blocks,
                                      int32_t n_wg)
{
    const int32_t units = selects + copies + thresholds;
    if ((selects == 0 && thresholds == 0 && !gated) || n_wg < 8) return FrontPlan{units < n_wg ? units : n_wg, 0};
    const uint32_t turns = (uint32_t)r_blocks / (8000u * 2u * 2u / 11u);  // 8000 ns in half of 5.5 ns a block
    const int32_t few = n_wg / 16, most = n_wg / 4;
    int32_t front = units;
    if (turns > 1 && units > few) {
        front = (int32_t)(((uint32_t)units + turns - 1) / turns);
        front = front < few ? few : front;
    }
    front = front < most ? front : most;
    return FrontPlan{front, front};
}

// Workgroups at the end of a grid of n_wg that select the launch's own score rows, one each: `rows`, or 0
// (the workgroup that completes a segment then selects its set after its last piece).  They wait for the
// rows' pieces, which lie on lower workgroups: on every XCD those have started before one of these does.
// Selecting there begins when a row's last piece has counted itself in, beside the merge of its partials, which
// takes 4 us.  What it costs is the streaming that these workgroups would have done, rows / n_wg of 5.5 ns a
// block: up to 1/64 of it at any length, or up to 1/16 where that is no more than 1.5 us.  us a call, selected after the
// merge and at the end of the grid: two KV heads at 4K 20.4 and 16.4, four retrieval heads of eight KV heads at
// 32K 33.1 and 27.1, at 100K with k = 8192 70.6 and 63.8.
LYCHEE_HD inline int32_t tail_selects(int32_t rows, int32_t r_blocks, int32_t n_wg)
{
    if (n_wg < 64) return 0;
    return 64 * rows <= n_wg || (16 * rows <= n_wg && (int64_t)rows * r_blocks <= 256ll * n_wg) ? rows : 0;
}

// Whether a plain layer call under a probability rule selects in a second launch, a workgroup per row, instead of in
// its own.  r_blocks: blocks of 64 rows that the launch streams at most, by the cache's capacity.  A select with a rule takes up to 15 us, and of more rows than a quarter of the workgroups some complete
// several and select them in turn; a streaming of more than 32 blocks a workgroup hides that.  us a call
// in one launch and in two, Top-p, 64 sequences of four retrieval heads in three KV heads: of 1 to 1000 rows 68.6 and
// 63.8, 61 to 3001 (in 4096) 96 and 87.  (Not the faster side everywhere: 1000 to 3000 in 3000 91.5 and 98.)
LYCHEE_HD inline bool rules_apart(int32_t rows, int32_t r_blocks, int32_t n_wg)
{
    return 4 * rows > n_wg && r_blocks <= 32 * n_wg;
}

// The same where the cache's capacity does not bound the streaming (r_blocks above is by the capacity, which says
// nothing about what lies far below it): both launches are enqueued, the first one decides by the sequences'
// lengths, and the second returns at once if nothing is left to it (2 us).  r_blocks: what the n_wg streaming
// workgroups take; shortest: blocks of the shortest segment; both with the blocks that a segment counts beyond
// those it has.  Rows are selected in turn where a workgroup's run holds several segments, so: where it holds more
// than two of the shortest.  us a call selected by the first launch and by the second, Top-p, 64 sequences of three
// score rows in a cache of 65536 rows (blocks of a run over the shortest segment's): 2000 to 5000 rows (1.3) 118 and
// 133, 1000 to 3000 (1.7) 96 and 106, 500 to 2000 (2.3) 94 and 92, 61 to 3001 (5) 106 and 99, 61 to 12000 (11) 198 and
// 182.  When the rule was made also: 800 to 2400 (1.8) 96 and 104; 61 to 6000 (7) 130 and 131; 128 sequences of 300 to
// 1000 (4) 123 and 110, of 1000 to 3000 (3.4) 178 and 186; 256 of 61 to 1000 (12) 228 and 187.
LYCHEE_HD inline bool rows_in_turn(int32_t r_blocks, int32_t n_wg, int32_t shortest)
{
    return r_blocks > 2 * shortest * n_wg;
}

// Rows one threshold unit samples in one round of loads.
constexpr int32_t kAloneSample = 512;
// Whether a score row's threshold is taken by one unit from one round of loads (512 rows) instead of by four from
// 1024 to 4096.  r_blocks: blocks of 64 rows that the launch would stream if every sequence were as long as this one
// (what it does stream would take a sum over the batch in every unit; in a ragged batch a short row's
// threshold may so be taken by one unit behind a long streaming, from fewer samples, which costs the select up to
// what its registers hold).
// The four hand their keys to the one that ranks them through device memory: stores, a counter, loads, each of which takes about
// 2 us beside the streaming's first loads, and a piece of a short launch is done with its rows before the
// threshold is out.  From fewer samples the threshold lets more rows through for the same
// safety: with f of the n best among 512 rows, (f + 6 sqrt f + 6) / f times n.  So: where the streaming takes less
// than the hand-over (five blocks per workgroup), and what is let through (n, or L if no more are) still fits the
// select's registers with a tenth to spare.  us with four units and with one: layer calls of 16384 rows with one, three
// and five retrieval heads 20.7 and 20.0, 20.7 and 19.8, 22.7 and 22.2; of 32768, k = 2048, with one to five 24.0 and
// 21.9, 24.6 and 24.2, 25.2 and 25.3, 26.7 and 27.8, 26.8 and 27.6.  (So the line lies far out since pieces ask for
// the threshold ahead of their partials; eight layers of the model loop of 32768 with one retrieval head take 166 and
// 174, with three and five the same.)
LYCHEE_HD inline float threshold_target(float f, float margin) { return f + margin * __builtin_sqrtf(f) + 6.0f; }
LYCHEE_HD inline bool threshold_alone(int32_t n, int32_t L, int32_t r_blocks, int32_t n_wg, float margin, int32_t fits)
{
    if (r_blocks > 5 * n_wg) return false;
    const float per_sample = (float)L / (float)kAloneSample;
    return 10.0f * threshold_target((float)n / per_sample, margin) * per_sample <= 9.0f * (float)fits;
}

// Set entries per block of gather work, unless the caller chose it (blocks are dealt like blocks of 64
// streamed rows).  64 makes the fewest pieces, whose chains of latencies bound a short launch: the faster one
// for phased steps (12 layers of 1 to 64 sequences of 1K to 128K: 0.82 to 1.01 of the time with 48, 0.97 at
// most sizes) and for plain layer calls (one layer of the same: 0.98 on average).
constexpr int32_t kGatherRows = 64;
// In launches whose gathers follow a select of the same launch (deferred calls, layer-after-layer steps) they
// start late and should have more workgroups than as many streamed rows, but only where rows and not
// latencies fill the launch: beyond 12 blocks per workgroup, by the cache's capacity, and for the longest
// sequences.  Model loop, time with 64 over time with 48: two sequences (blocks per workgroup) at 48K (12) 0.98,
// 64K (16) 1.01; four at 16K (9) 0.98, 32K (18) 0.98; eight at 8K (9) 0.98, 16K (18) 1.00; 64 at 1K (9) 1.00, 3K (26)
// 1.04, 8K (72) 1.03; one sequence of three retrieval heads at 64K 1.00, 96K 0.98, 128K 1.01.  (When the rule was made
// 64K and more of two to eight sequences 1.05 to 1.11, 128K of 1 to 5 retrieval heads 0.95 to 1.08.)
LYCHEE_HD inline int32_t gather_block_rows(int32_t r_blocks, int32_t g_blocks, int32_t max_len, int32_t n_wg)
{
    return (int64_t)r_blocks + g_blocks > 12ll * n_wg || max_len >= 7 << 14 ? 48 : kGatherRows;
}

// How a phased step's merges are dealt: a unit merges all query heads of a KV head, its retrieval heads and then its
// sparse ones; or the heads of one of the two kinds; or one head.  kv_heads: KV heads over all sequences and layers;
// others: units of other kinds in the launch; slots: the most that a head can have.
//
// A unit is a chain of latencies, about 2.7 us, whether it merges one head or four of the same kind, and 2 us more
// for a second kind; four heads take another 3 us for every 48 slots beyond the first 48, one head 4 us for 190.
// Units are dealt to the workgroups in turn.  So: a head each where every head has a workgroup of its own; a kind
// each likewise (half of these units are empty in a dense step); else KV heads, of which none is empty and all have as
// much to do.  Heads again up to three rounds of them where they have more than two rounds of 48 slots.
// us of the merging launch with KV heads, kinds and heads, 8 KV heads of four query heads, one sequence: 8 layers of
// 4096 rows 7.1, 5.2, 4.9; 24 layers 7.4, 5.7, 7.8; 36 7.6, 8.1, 10.2; of 32768 (66 slots) 8 layers 7.8, 6.5, 6.4;
// 36 10.3, 10.7, 13.0, dense 10.4, 13.3, 13.0; of 65536 (130 slots) 24 layers 16.0, 14.5, 10.5; 44 17.5, 18.6, 14.7; 60
// 12.5, 11.7, 17.0, dense 14.6, 18.8, 17.2.  (Kinds in every step: 8 sequences of 8192, 36 layers, 31.4, dense 32.3, with
// KV heads 25.0 and 18.2; of one query head each 25.8 and 25.1, by the head 16.7 and 14.0.)
enum { kMergeKvHeads = 0, kMergeKinds = 1, kMergeHeads = 2 };
LYCHEE_HD inline int32_t merge_split(int32_t kv_heads, int32_t group, bool any_sparse, int32_t others, int32_t slots, int32_t n_wg)
{
    const int64_t heads = (int64_t)kv_heads * group;
    if (group == 1 || heads + others <= n_wg || (slots > 2 * 48 && heads <= 3ll * n_wg)) return kMergeHeads;
    return any_sparse && 2ll * kv_heads + others <= n_wg ? kMergeKinds : kMergeKvHeads;
}
LYCHEE_HD inline int32_t merge_parts(int32_t split, int32_t group)
{
    return split == kMergeHeads ? group : (split == kMergeKinds ? 2 : 1);
}
// Which of a KV head's query heads its part-th unit merges.  rmask: its retrieval heads.
LYCHEE_HD inline uint32_t merge_heads(int32_t split, int32_t part, uint32_t rmask, int32_t group)
{
    const uint32_t all = (1u << group) - 1u;
    if (split == kMergeHeads) return 1u << part;
    if (split == kMergeKinds) return (part != 0 ? ~rmask : rmask) & all;
    return all;
}

}  // namespace lychee
