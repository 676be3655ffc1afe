/* The library's layout functions behind C names, for tests/test_launch_plan.py. */
#include <cmath>

#include "lychee_plan.h"

extern "C" void front_plan(int32_t selects, int32_t copies, int32_t thresholds, int32_t gated, int32_t r_blocks, int32_t n_wg,
                           int32_t *out)
{
    const lychee::FrontPlan p = lychee::front_plan(selects, copies, thresholds, gated != 0, r_blocks, n_wg);
    out[0] = p.n_front;
    out[1] = p.n_aside;
}

extern "C" uint32_t first_generation() { return lychee::kFirstGeneration; }

extern "C" uint32_t next_generation(uint32_t gen) { return lychee::next_generation(gen); }

extern "C" int32_t list_row_entries(int32_t max_len, int32_t k, int32_t blocks)
{
    return lychee::list_row_entries(max_len, k, blocks != 0);
}

extern "C" int32_t gather_block_rows(int32_t r_blocks, int32_t g_blocks, int32_t max_len, int32_t n_wg)
{
    return lychee::gather_block_rows(r_blocks, g_blocks, max_len, n_wg);
}

extern "C" int32_t tail_selects(int32_t rows, int32_t r_blocks, int32_t n_wg)
{
    return lychee::tail_selects(rows, r_blocks, n_wg);
}

extern "C" int32_t rules_apart(int32_t rows, int32_t r_blocks, int32_t n_wg)
{
    return lychee::rules_apart(rows, r_blocks, n_wg);
}

extern "C" int32_t rows_in_turn(int32_t r_blocks, int32_t n_wg, int32_t shortest)
{
    return lychee::rows_in_turn(r_blocks, n_wg, shortest);
}

// (ulps: how far the reciprocal is off)
extern "C" int32_t quot(int32_t a, int32_t b, int32_t ulps)
{
    float inv = 1.0f / (float)b;
    if (ulps) inv = std::nextafter(inv, ulps > 0 ? 2.0f : 0.0f);
    return lychee::quot_by(a, b, inv, [](uint32_t v) { return v; });
}

extern "C" int32_t threshold_alone(int32_t n, int32_t L, int32_t r_blocks, int32_t n_wg, float margin, int32_t fits)
{
    return lychee::threshold_alone(n, L, r_blocks, n_wg, margin, fits);
}

extern "C" int32_t merge_split(int32_t kv_heads, int32_t group, int32_t any_sparse, int32_t others, int32_t slots, int32_t n_wg)
{
    return lychee::merge_split(kv_heads, group, any_sparse != 0, others, slots, n_wg);
}

extern "C" int32_t merge_parts(int32_t split, int32_t group) { return lychee::merge_parts(split, group); }

extern "C" uint32_t merge_heads(int32_t split, int32_t part, uint32_t rmask, int32_t group)
{
    return lychee::merge_heads(split, part, rmask, group);
}
