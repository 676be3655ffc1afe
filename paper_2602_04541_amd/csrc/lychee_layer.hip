// The single launch of one layer call (Alg. 1, one pass of the layer loop's per-head loop).
//
// A model that decodes layer after layer computes the next layer's query from this layer's
// output, so the layer's work cannot be pooled with other layers', and at 128K a layer is only
// about 30 microseconds of HBM time: every dependent launch (each costs a few microseconds of gap,
// a prologue and a tail) shows.  This kernel therefore runs the whole layer in ONE launch and
// hands results from workgroup to workgroup inside it:
//
//   front units  (the first workgroups, as many as front_plan says, before anything else; they wait for nothing)
//       S  the select of the PREVIOUS layer call (Eq. 2), left pending by that call: its set is
//          read again only by this layer's sparse heads (Sec. 3.1), so it runs beside this
//          layer's streaming instead of after the previous layer's; copies of the sets of KV
//          heads that keep theirs
//       T  the selection thresholds of this layer (a sample of each score row)
//   R pieces     Eq. 1 / o = A V over this layer's cache rows.  The threshold of a piece's score
//                row is computed by a T unit of the same launch, so the piece keeps its rows'
//                keys in LDS and filters them when it ends (by then the T unit, about half as
//                long as a piece, has published the threshold; a piece polls for it if not)
//   G pieces     Eq. 3 over the inherited set, on the last workgroups of the grid; a piece polls
//                until the front unit that writes its KV head's set has published it
//   combine      every piece writes its partial through to device memory and counts itself in;
//                the piece that completes a segment merges the segment's partials into `out` (a
//                segment of one piece writes `out` itself)
//   own select   in the build for calls that want their sets at once: the last workgroups of the grid
//                select, one score row each, as soon as the row's pieces have counted themselves in and
//                beside the merge that follows (tail_selects); where the rows are too many for that, the
//                workgroup that completed a segment selects its set after its last piece, or, under a
//                probability rule, the launch behind this one does (rules_apart, rows_in_turn)
//
// Waiting is safe because every XCD starts its workgroups in index order and every wait is for a kind of workgroup
// that comes earlier on all of them: pieces wait for front units, which never wait and have, where anything waits,
// the lowest indices to themselves (front_plan); selects at the end of the grid wait for pieces.  That holds for a
// launch by itself; launches of several streams that start at the same time share the places in an order that
// nothing here fixes.  Waits are bounded: one that gives up on a threshold or on a row costs time only.
// Partials cross from one XCD's L2 to another's without the agent-scope release fence (its
// write-back of the whole L2, executed by every workgroup, costs more than the layer): they are
// written with write-through stores, the writer waits until those have completed before it
// counts itself in, and the merging workgroup takes an acquire fence.  The sets are handed over
// the same way: written through, waited for, then flagged; but hundreds of workgroups read them, and an acquire
// fence invalidates the caches of its whole XCD, so they are read past the caches instead (gload_through; with
// a fence in every gathering workgroup a 32K layer of the model loop took 29.5 us, now 26.0).  The few that merge keep
// theirs: partials read past the caches, in loads of 8 bytes, made the 36-layer step at 128K 1748 us instead of 1690.
#include "lychee_internal.h"
#include "lychee_device.h"
#include "lychee_stream.h"
#include "lychee_select.h"

namespace lychee {
namespace {

struct SharedLayer {
    int32_t pre[kMaxBatch + 1];  // first block of every sequence in this workgroup's row space
    int32_t len[kMaxBatch];
    uint32_t scan[kWaves + 1];
    unsigned long long scan64[kWaves + 1];
    float fred[kWaves + 1];
    int32_t flag;
    int32_t role[2][4];            // per kind of piece: first workgroup, workgroups, segments per sequence, blocks
    uint32_t nb[2][kMaxBatch];     // per kind: blocks of one segment of every sequence
    int32_t extra[2];              // per kind: blocks that a segment counts beyond those it has
    int32_t run[3];                // the piece loop: next block of this workgroup's run, blocks per run, padded (2: `at` holds the only piece)
    __align__(16) int32_t at[12];  // the piece in hand: sequence, KV head, heads, blocks of the run; pieces of its segment, first and end row, slot; its blocks, its segment's
    FrontPlan front;               // who runs front units
    uint32_t gen;                  // the generation of this launch's flags
    int32_t closes;                // this workgroup was the last of its group to count in
};
template <bool kUnits>
union SharedRole {
    SharedAttn attn;     // a piece
    SharedCombine comb;  // the merge that follows a piece
    SharedSelect sel;    // a front unit, or the launch's own select
};
template <>
union SharedRole<false> {  // (the dense build selects nothing: a workgroup with less LDS is placed sooner)
    SharedAttn attn;
    SharedCombine comb;
};

__device__ __forceinline__ uint32_t load_agent(const uint32_t *p)
{
    return __hip_atomic_load((const LYCHEE_GLOBAL uint32_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(uint32_t *p, uint32_t v)
{
    __hip_atomic_store((LYCHEE_GLOBAL uint32_t *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every workgroup of a launch counts itself in once it has read the generation, among every kExitGroups-th
// workgroup; the last of a group counts the group in at its end (closes_launch), and the last of those advances the
// generation.  Whoever still runs then compares flags with the one it has read.  Returns what count_in_last
// makes of it.  (Counted on one word, each at its end, the 440 workgroups without a piece in a layer
// of 4K left together and held up the others' first rows, asked for just then, by 4 us; and the last workgroup's
// addition, 0.5 us, stood at the end of every launch.)
__device__ __forceinline__ uint32_t count_in(const LYCHEE_CONSTANT LayerLaunch *A, int w, uint32_t &gen)
{
    uint32_t at = kLineWords * (1 + w % kExitGroups);
    // (The generation has arrived; and the address is opaque: to an address that it knows to be the same in every lane the
    // compiler adds for the wavefront as a whole and waits for the answer on the spot.)
    asm volatile("" : "+v"(gen), "+v"(at) : : "memory");
    return __hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)A->exit_count + at, 1u, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool count_in_last(const LYCHEE_CONSTANT LayerLaunch *A, int w, int W, uint32_t before)
{
    if (before != (uint32_t)((W - 1 - w % kExitGroups) / kExitGroups)) return false;
    store_agent(A->exit_count + kLineWords * (1 + w % kExitGroups), 0u);  // as every launch finds it
    return true;
}
__device__ __forceinline__ void closes_launch(const LYCHEE_CONSTANT LayerLaunch *A, int W, uint32_t gen)
{
    const uint32_t groups = W < kExitGroups ? W : kExitGroups;
    const uint32_t before = __hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)A->exit_count, 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    if (before != groups - 1u) return;
    store_agent(A->exit_count, 0u);
    store_agent(A->gen, next_generation(gen));
}

// Blocks of 64 rows of all sequences of a batch, the same in every lane.
__device__ __forceinline__ int all_blocks(const int32_t *len, int batch)
{
    uint32_t n = 0;
    for (int b = fresh_tid() & 63; b < batch; b += 64) n += (uint32_t)(len[b] + kBlockRows - 1) / kBlockRows;
    return __builtin_amdgcn_readlane((int)wave_scan(n), 63);
}

// Whether the rows of this launch are left to the launch behind it (rows_in_turn).
__device__ __forceinline__ bool selects_apart(const SharedLayer &pool, int batch)
{
    uint32_t least = ~0u;
    for (int b = fresh_tid() & 63; b < batch; b += 64) least = min(least, pool.nb[0][b]);
    return rows_in_turn(uni(pool.role[0][3]), uni(pool.role[0][1]), uni((int)wave_min(least)));
}

// A front unit has written the set of (b, g), with write-through stores: once every wavefront's
// stores have completed the set is in device memory, and the flag says so.
__device__ __forceinline__ void publish_set(uint32_t *flag, uint32_t gen)
{
    wait_stores();
    __syncthreads();
    if (fresh_tid() == 0) store_agent(flag, gen);
}

// Before a gather piece reads (by gload_through) a set that a front unit of this launch writes.
__device__ __forceinline__ void await_set(ArgCommon &c, const uint32_t *flag, uint32_t gen, SharedLayer &pool)
{
    if (fresh_tid() == 0) {
        const int polls = c.wait_polls;
        int spin = 0;
        for (; spin < polls; ++spin) {
            if (load_agent(flag) == gen) break;
            __builtin_amdgcn_s_sleep(2);
        }
        if (spin == polls) atomicAdd(c.stats + 2, 1u);  // (the piece then reads whatever the array holds; entries are range-checked)
    }
    __syncthreads();
}

// Before a workgroup at the end of the grid selects a row: until the row's pieces have counted in all of its
// blocks.  Whether they have.  If it gives up it leaves the row, marked in the counter's highest bit, to the piece
// that completes it, whose workgroup then selects it: whatever the select reads and puts back to zero (the
// list and its counter, the pieces' log-sum-exps) is complete by then.  The counter goes back to zero here, or
// there.
constexpr uint32_t kNobodyWaits = 0x80000000u;
__device__ __forceinline__ bool await_rows(ArgCommon &c, uint32_t *counter, uint32_t blocks, SharedLayer &pool)
{
    if (fresh_tid() == 0) {
        const int polls = c.wait_polls;
        int spin = 0;
        for (; spin < polls; ++spin) {
            if (load_agent(counter) == blocks) break;
            __builtin_amdgcn_s_sleep(2);
        }
        if (spin == polls) {
            const uint32_t old = __hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)counter, kNobodyWaits, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            if (old == blocks) spin = -1;  // (just in time)
            else atomicAdd(c.stats + 2, 1u);
        }
        if (spin != polls) store_agent(counter, 0u);
        pool.flag = spin != polls;
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return uni(pool.flag) != 0;
}

// SELECTS: 0 no selection in the launch; 1 the select that an earlier call left pending; 2 the same with the
// probability rules; 3 this layer's own, by workgroups at the end of the grid or whoever completes a segment
// (nothing pends then: with one select in it every build keeps its registers).
template <bool COLLECT, int SELECTS>
__global__ __launch_bounds__(kThreads, 2) void lychee_layer_kernel(const LayerLaunch P)
{
    constexpr bool kNow = SELECTS == 3;
    __shared__ __align__(16) SharedRole<COLLECT> sh;
    SharedSelect &sel = reinterpret_cast<SharedSelect &>(sh);  // (never touched in the dense build)
    __shared__ uint32_t wanted[SELECTS == 3 ? kMaxBatch * kMaxKvHeads / 32 : 1];  // bit per score row: this workgroup selects its set
    __shared__ SharedLayer pool;
    // Both layer descriptors are staged in LDS, one word per thread, and read from there.  (The
    // kernel argument is never indexed with a run-time value: for `idx_src[g]` the compiler
    // emitted a scalar load whose base register held `argument + g` and whose offset register
    // held `7 g` - only their sum is a multiple of 4 -, and the scalar memory unit drops the
    // low bits of each, so that the load returned the halves of two neighbouring pointers.)
    __shared__ __align__(16) uint32_t desc_cur[kDescWords], desc_prev[kDescWords];
    const LYCHEE_CONSTANT LayerLaunch *A = arg_of<LayerLaunch>();
    ArgCommon &c = A->c;
    const int w = blockIdx.x;
    const int W = c.n_wg;
    const int tid = fresh_tid();
    // The second launch of a pair whose first one selected its rows itself: nothing is left to do, and as it
    // leaves no flags the generation may stay.
    if (SELECTS == 2 && A->apart != nullptr && uni(load_agent(A->apart)) == 0u) return;

    // The generation is only ever used by thread 0 (it sets, polls and advances the flags), which
    // keeps it in a register: the load is not waited for before its first use.
    uint32_t gen = tid == 0 ? load_agent(A->gen) : 0u;
    // (all loads before the first wait)
    int len = 0;
    uint32_t word_cur = 0, word_prev = 0;
    if (tid < c.batch) len = gload(c.lengths + tid);
    if (tid < kDescWords) {
        word_cur = reinterpret_cast<const LYCHEE_CONSTANT uint32_t *>(&A->cur)[tid];
        word_prev = reinterpret_cast<const LYCHEE_CONSTANT uint32_t *>(&A->prev)[tid];
    }
    if (SELECTS == 3)
        for (int i = tid; i < kMaxBatch * kMaxKvHeads / 32; i += kThreads) wanted[i] = 0;
    if (tid < c.batch) pool.len[tid] = clamp_len(len, c.max_len);
    if (tid < kDescWords) {
        desc_cur[tid] = word_cur;
        desc_prev[tid] = word_prev;
    }
    __syncthreads();
    const LayerDesc &cur = *reinterpret_cast<const LayerDesc *>(desc_cur);
    const LayerDesc &prev = *reinterpret_cast<const LayerDesc *>(desc_prev);
    const uint32_t *dw = desc_cur;

    // ------------------------------------------------------------------ front units
    FrontPlan front{A->front.n_front, A->front.n_aside};
    if (__builtin_expect(front.n_front < 0, 0))
        front = front_plan(A->n_selects, A->n_copies, A->n_thresholds, A->gate_mask != 0,
                           A->cur.n_rgroups * all_blocks(pool.len, c.batch), W);
    pool.front = front;  // (read again for the split; every thread writes the same, so that none waits for another's)
    if (w < front.n_front) {
        __builtin_amdgcn_s_setprio(3);  // (the launch waits for these; a streaming workgroup shares the CU)
        const int n_rp = A->has_prev ? prev.n_rgroups : 0;
        const int nS = SELECTS && !kNow ? c.batch * n_rp : 0;
        const LayerDesc &kept = kNow ? cur : prev;  // whose kept sets are copied
        const int n_keep = c.n_kv_heads - kept.n_rgroups;
        const int nC = (kNow || A->has_prev) && kept.copy_keep ? c.batch * n_keep : 0;
        const int nT = COLLECT && A->n_thresholds ? c.batch * cur.n_rgroups * kThrSplit : 0;
        for (int j = w; j < nS + nC + nT; j += front.n_front) {
            const LYCHEE_CONSTANT LayerLaunch *A = arg_of<LayerLaunch>();
            ArgCommon &c = A->c;
            if (j < nS) {
                const int b = j / n_rp;
                const int g = prev.rgroup[j % n_rp];
                if (SELECTS != 0 && !kNow) select_unit<SELECTS == 2>(c, prev, b, g, sel, pool);
                publish_set(A->set_flags + set_flag_at(b, g, c.n_kv_heads), gen);
            } else if (j < nS + nC) {
                const int u = j - nS;
                const int b = u / n_keep;
                int want = u % n_keep, g = 0;
                for (int gg = 0; gg < c.n_kv_heads; ++gg)
                    if (kept.rindex[gg] == 0xFF && want-- == 0) g = gg;
                copy_set_unit(c, kept, b, g);
                publish_set(A->set_flags + set_flag_at(b, g, c.n_kv_heads), gen);
            } else {
                // a score row's sample is dealt to kThrSplit units: one round of loads each
                const int u = (j - nS - nC) / kThrSplit;
                const int n_rc = cur.n_rgroups;
                const int b = u / n_rc, rgi = u % n_rc;
                const int64_t row = (int64_t)b * n_rc + rgi;
                unsigned long long *flag = A->thr_flags + row * (kLineWords / 2);
                ThrSplit split;
                split.sub = (j - nS - nC) % kThrSplit;
                split.n_sub = kThrSplit;
                split.keys = reinterpret_cast<uint32_t *>(cur.sel + row * c.sel_stride);  // (free until a select ranks this row whole)
                split.arrived = A->thr_arrived + row * kLineWords;
                switch (__builtin_popcount(cur.rmask[cur.rgroup[rgi]] & ((1u << c.group) - 1u))) {
                case 1: threshold_unit<1>(c, cur, b, rgi, sel, pool, flag, gen, split); break;
                case 2: threshold_unit<2>(c, cur, b, rgi, sel, pool, flag, gen, split); break;
                case 3: threshold_unit<3>(c, cur, b, rgi, sel, pool, flag, gen, split); break;
                default: threshold_unit<4>(c, cur, b, rgi, sel, pool, flag, gen, split); break;
                }
            }
            __syncthreads();
        }
        __builtin_amdgcn_s_setprio(0);
    }
    uint32_t counted = 0;
    if (tid == 0) counted = count_in(A, w, gen);  // (the answer is there before the first piece is found)

    // ------------------------------------------------------------------ the two row spaces
    // Per sequence: blocks of 64 cache rows per retrieval KV head, blocks of gathered rows per
    // sparse KV head.  The workgroups after the front ones are split between the two kinds.
    // Everything the piece loop needs afterwards is left in LDS and read again after every
    // piece: a piece wants every vector register, and whatever the schedule kept in registers
    // across it was spilled to scratch memory by all workgroups (a launch with a scratch
    // segment also starts its wavefronts more slowly).
    // (A single sequence needs no scans over the batch: every thread evaluates it for itself.)
    // Everything from here to the first piece's loads is a chain of latencies that every workgroup of the
    // launch goes through: a dozen divisions and as many LDS round trips took 3.4 us of a 20-us launch, and
    // a barrier a wavefront waits at in it costs more than the arithmetic between two of them.  So the
    // values that the first piece is found from stay in registers (`kd`, `next`), a single sequence's
    // run length has a closed form, and its piece follows from the workgroup's number alone.
    const bool single = c.batch == 1;
    struct Kind {
        int first, n_wg, segs, blocks, nb, extra;  // nb: of a single sequence's segment
    } kd, next;
    {
        const int n_rseg = A->has_cur ? (int)desc_u32(dw, offsetof(LayerDesc, n_rgroups)) : 0;
        const int n_gseg = A->has_cur ? (int)desc_u32(dw, offsetof(LayerDesc, n_sgroups)) : 0;
        uint32_t nb_r = 0, nb_g = 0;
        if (tid < c.batch || single) {
            const int L = pool.len[single ? 0 : tid];
            nb_r = n_rseg ? (uint32_t)((L + kBlockRows - 1) / kBlockRows) : 0u;
            nb_g = n_gseg ? (uint32_t)quot(gather_rows(c, L) + gather_block(c) - 1, gather_block(c)) : 0u;
        }
        // A run may cross segments, and every piece costs its start-up, merge and hand-over (about 8 us, a
        // block 1.2 to 1.7 us), so a segment counts kPieceBlocks blocks more than it has.
        // (64 sequences of 61 to 3001 rows: a run of equal blocks held up to nine short
        // segments, half the workgroups were done after 70 us and the last after 110.  Few segments of
        // a batch, us without and with: model loop of 8 x 2000-5000 rows, 4 layers, 125.5 and 121.4, of
        // 5 x 6000-24000 180.8 and 171.0; a layer call of 8 x 3000-8192 with one and two retrieval heads the same.)
        // Not the few gathers of a launch that selects its own rows: the blocks also weigh the split of the
        // grid, and there the streaming, which the select follows, should end first (8 x 3000-8192, four retrieval heads:
        // 32.8, with them 35.5, when a piece's fixed cost was higher.  It is no longer so: k = 256, 1024 and 2048 31.2,
        // 39.7 and 42.5, with them 30.3, 35.0 and 42.3; one retrieval head 22.7, 28.4 and 35.6, with them 21.7, 26.6
        // and 32.3.)  A single sequence's segments end with a run.
        const int extra_r = !single || 8 * n_rseg > W ? kPieceBlocks : 0;
        const int extra_g = (!single && !kNow) || 8 * n_gseg * c.batch > W ? kPieceBlocks : 0;
        nb_r += nb_r ? extra_r : 0;
        nb_g += nb_g ? extra_g : 0;
        unsigned long long tot64 = (unsigned long long)nb_r | ((unsigned long long)nb_g << 32);
        if (!single) (void)block_scan_pair(tot64, pool.scan64, tot64);
        // (the totals are the same in every lane: scalar arithmetic from here on)
        const int TR = uni((int)(uint32_t)tot64) * n_rseg;  // (below 2^31, checked before the launch)
        const int TG = uni((int)(uint32_t)(tot64 >> 32)) * n_gseg;
        const int first = uni(pool.front.n_aside);
        const int Wn = W - first - (kNow ? A->n_tail : 0);
        int W_R = 0, W_G = 0;
        if (Wn < 2) {  // a single workgroup does both kinds, one after the other
            W_R = TR > 0;
            W_G = TG > 0;
        } else if (TR > 0 && TG > 0) {
            // Gathers that wait for a select start late: by then every workgroup could have streamed
            // a = lead_blocks / Wn blocks.  Both kinds end together when a streaming workgroup takes u
            // blocks and a gathering one u - a:  TR / u + TG / (u - a) = Wn, the larger root of
            // Wn u^2 - (Wn a + TR + TG) u + TR a = 0.  Single precision is plenty (any split is a
            // valid one), and every workgroup evaluates the same operations on the same values, so
            // all agree on it.
            const float tr = (float)TR, tg = (float)TG, wn = (float)Wn;
            const float lead = A->has_prev && A->gate_mask != 0 ? (float)A->lead_blocks : 0.0f;
            const float inv_wn = __builtin_amdgcn_rcpf(wn);
            const float a = lead * inv_wn;
            const float half_b = 0.5f * (lead + tr + tg);
            float disc = half_b * half_b - tr * lead;
            disc = disc > 0.0f ? disc : 0.0f;
            const float u = (half_b + __builtin_amdgcn_sqrtf(disc)) * inv_wn;
            int wg = u - a > 0.0f ? (int)(tg * __builtin_amdgcn_rcpf(u - a) + 0.5f) : Wn;
            // a gather piece is a chain of latencies (flag, set entries, rows, merge) of about 10 us
            // whatever its size: few gather blocks get a workgroup each rather than a queue on two
            const int floor_wg = TG < (Wn >> 3) ? TG : Wn >> 3;
            wg = wg < floor_wg ? floor_wg : wg;
            // and the streaming keeps at least a third of the workgroups its share of the blocks would give it
            const int most = Wn - (int)(wn * tr * __builtin_amdgcn_rcpf(3.0f * (tr + tg)));
            wg = wg > most ? most : wg;
            W_G = uni(wg < 1 ? 1 : (wg > Wn - 1 ? Wn - 1 : wg));
            W_R = Wn - W_G;
        } else if (TG > 0) {
            W_G = Wn;
        } else if (TR > 0) {
            W_R = Wn;
        }
        if (tid == 0) {
            pool.role[0][0] = first;
            pool.role[0][1] = W_R;
            pool.role[0][2] = n_rseg;
            pool.role[0][3] = TR;
            pool.role[1][0] = Wn < 2 ? first : first + W_R;
            pool.role[1][1] = W_G;
            pool.role[1][2] = n_gseg;
            pool.role[1][3] = TG;
            pool.extra[0] = extra_r;
            pool.extra[1] = extra_g;
            pool.gen = gen;
            pool.closes = count_in_last(A, w, W, counted);
        }
        kd = Kind{first, W_R, n_rseg, TR, uni((int)nb_r), extra_r};
        next = Kind{Wn < 2 ? first : first + W_R, W_G, n_gseg, TG, uni((int)nb_g), extra_g};
        if (tid < c.batch) {
            pool.nb[0][tid] = nb_r;
            pool.nb[1][tid] = nb_g;
        }
    }

    for (int kind = 0; kind < 2; ++kind) {
        const bool gather = kind == 1;
        const int tid = fresh_tid();
        const LYCHEE_CONSTANT LayerLaunch *A = arg_of<LayerLaunch>();
        ArgCommon &c = A->c;
        auto head_at = [&](int gi) {  // KV head of a sequence's gi-th segment, and the query heads it works for
            return (int)desc_u8(dw, (gather ? offsetof(LayerDesc, sgroup) : offsetof(LayerDesc, rgroup)) + gi);
        };
        auto heads_of = [&](int g) {
            const uint32_t r = desc_u8(dw, offsetof(LayerDesc, rmask) + g);
            return (gather ? ~r : r) & ((1u << c.group) - 1u);
        };
        {
            const int wl = w - kd.first;
            const int role_n = kd.n_wg;
            if (role_n <= 0 || wl < 0 || wl >= role_n) {  // (uniform in the workgroup)
                kd = next;
                continue;
            }
            const int nseg = kd.segs;
            const uint32_t nb_mine = single ? (uint32_t)kd.nb : (tid < c.batch ? pool.nb[kind][tid] : 0u);

            // Equal contiguous runs of blocks; when the segments are few, every segment is padded to
            // a whole number of runs, so that each workgroup has exactly one piece (a second piece
            // costs a second start-up and merge, which a launch this short cannot level out).
            int share = quot_uni(kd.blocks + role_n - 1, role_n);
            int pad = 0;
            uint32_t mine = nseg * nb_mine;
            if (8 * nseg * c.batch <= role_n) {
                // (of the blocks the segments have: a single sequence's count none beyond them here)
                const int s_min = single ? share : quot_uni(kd.blocks - kd.extra * nseg * c.batch + role_n - 1, role_n);
                const int s_last = s_min + (s_min >= 16 ? s_min >> 3 : 1);
                if (single) {  // (the shortest run of which a segment takes no more than its part of the workgroups)
                    const int most = quot_uni(role_n, nseg);
                    const int s = quot_uni(kd.nb + most - 1, most);
                    if (s <= s_last) {
                        // the workgroup's one piece is run `ri` of segment `gi`: worked out here, read back below
                        share = s, pad = 2;
                        const int runs = quot_uni(kd.nb + s - 1, s);
                        mine = (uint32_t)(nseg * runs * s);
                        const int gi = quot_uni(wl, runs);
                        const int ri = wl - gi * runs;
                        if (gi < nseg) {
                            const int brows = gather ? gather_block(c) : kBlockRows;
                            const int len = pool.len[0];
                            const int seg_rows = gather ? gather_rows(c, len) : len;
                            const int r1 = (ri + 1) * s * brows;
                            const int g = head_at(gi);
                            const uint32_t hmask = heads_of(g);
                            if (tid == 0) {
                                pool.at[0] = 0;
                                pool.at[1] = g;
                                pool.at[2] = (int32_t)hmask;
                                pool.at[3] = s;
                                pool.at[4] = runs;
                                pool.at[5] = ri * s * brows;
                                pool.at[6] = r1 < seg_rows ? r1 : seg_rows;
                                pool.at[7] = ri;
                                pool.at[8] = kd.nb - ri * s < s ? kd.nb - ri * s : s;
                                pool.at[9] = kd.nb;
                            }
                        }
                    }
                } else {
                    const uint32_t nb_have = nb_mine - (nb_mine ? (uint32_t)kd.extra : 0u);
                    int s = s_min;
                    for (; s <= s_last; ++s) {
                        uint32_t need = nseg * (uint32_t)quot((int)nb_have + s - 1, s), all;
                        (void)block_scan(need, pool.scan, all);
                        if ((int)all <= role_n) break;
                    }
                    if (s <= s_last) {
                        share = s, pad = 1;
                        mine = nseg * (uint32_t)(quot((int)nb_have + s - 1, s) * s);
                    }
                }
            }
            uint32_t all;
            const uint32_t incl = single ? mine : block_scan(mine, pool.scan, all);
            if (tid < c.batch) pool.pre[tid + 1] = (int32_t)incl;
            if (tid == 0) {
                pool.pre[0] = 0;
                pool.run[0] = wl * share;  // the next block of this workgroup's run
                pool.run[1] = share;
                pool.run[2] = pad;
            }
        }
        __syncthreads();

        // One piece: where it lies, from the values in LDS alone.
        struct Piece {
            int b, g, len_b, r0, r1, slot, pieces, len, nb, next_seg;
            uint32_t hmask;
            bool ends, padding;
        };
        auto piece_at = [&](ArgCommon &c, int x, int x1, int share, int pad) {
            Piece pc;
            const int brows = gather ? gather_block(c) : kBlockRows;
            pc.b = uni(find_item(pool.pre, c.batch, x));
            pc.len_b = uni(pool.len[pc.b]);
            const int seg_rows = gather ? gather_rows(c, pc.len_b) : pc.len_b;
            const int nb = quot_uni(seg_rows + brows - 1, brows);
            const int nbv = pad ? quot_uni(nb + share - 1, share) * share : nb + uni(pool.extra[kind]);
            const int pre_b = uni(pool.pre[pc.b]);
            const int xo = x - pre_b;
            const int gi = quot_uni(xo, nbv);
            const int blk = xo - gi * nbv;
            pc.padding = blk >= nb;  // the run goes on in what a segment counts beyond its blocks
            const int seg_start = pre_b + gi * nbv;
            pc.next_seg = seg_start + nbv;
            int len = x1 - x;
            len = len < nb - blk ? len : nb - blk;
            pc.len = len;
            pc.nb = nb;
            pc.r0 = blk * brows;
            const int r1 = (blk + len) * brows;
            pc.r1 = r1 < seg_rows ? r1 : seg_rows;
            const int run0 = quot_uni(seg_start, share);
            pc.slot = quot_uni(x, share) - run0;
            pc.pieces = quot_uni(seg_start + nb - 1, share) - run0 + 1;
            pc.ends = blk + len == nb;
            pc.g = head_at(gi);
            pc.hmask = heads_of(pc.g);
            return pc;
        };

        for (;;) {
            const int tid = fresh_tid();
            const LYCHEE_CONSTANT LayerLaunch *A = arg_of<LayerLaunch>();
            ArgCommon &c = A->c;
            int x, x1, share, pad;
            auto where = [&]() {
                x = uni(pool.run[0]);
                share = uni(pool.run[1]);
                pad = uni(pool.run[2]);
                const int T = uni(pool.pre[c.batch]);
                x1 = (w - uni(pool.role[kind][0])) * share + share;
                x1 = x1 < T ? x1 : T;
            };
            where();
            if (x >= x1) break;
            {
                Piece pc;
                if (pad == 2) {
                    pc.b = 0;
                    pc.len_b = uni(pool.len[0]);
                    pc.g = uni(pool.at[1]);
                    pc.hmask = (uint32_t)uni(pool.at[2]);
                    pc.pieces = uni(pool.at[4]);
                    pc.r0 = uni(pool.at[5]);
                    pc.r1 = uni(pool.at[6]);
                    pc.slot = uni(pool.at[7]);
                    pc.ends = pc.slot == pc.pieces - 1;
                    pc.padding = false;
                } else {
                    pc = piece_at(c, x, x1, share, pad);
                }
                if (pc.padding) {  // (uniform) the next segment, if the run reaches it
                    if (pc.next_seg >= x1) break;
                    __syncthreads();
                    if (tid == 0) pool.run[0] = pc.next_seg;
                    __syncthreads();
                    continue;
                }
                if (pad != 2 && tid == 0) {  // (what follows the piece reads this instead of working it out again)
                    pool.at[0] = pc.b;
                    pool.at[1] = pc.g;
                    pool.at[2] = (int32_t)pc.hmask;
                    pool.at[3] = pc.len;
                    pool.at[4] = pc.pieces;
                    pool.at[8] = pc.len;
                    pool.at[9] = pc.nb;
                }
                auto nothing = []() {};
                const uint16_t *dq = desc_ptr<const uint16_t>(dw, offsetof(LayerDesc, q));
                const uint16_t *dk = desc_ptr<const uint16_t>(dw, offsetof(LayerDesc, k_cache));
                const uint16_t *dv = desc_ptr<const uint16_t>(dw, offsetof(LayerDesc, v_cache));
                float *d_part_o = desc_ptr<float>(dw, offsetof(LayerDesc, part_o));
                float *d_part_ml = desc_ptr<float>(dw, offsetof(LayerDesc, part_ml));
                int32_t *d_part_count = desc_ptr<int32_t>(dw, offsetof(LayerDesc, part_count));
                uint16_t *alone = pc.pieces == 1 ? desc_ptr<uint16_t>(dw, offsetof(LayerDesc, out)) : nullptr;
                const uint32_t my_gen = pool.gen;
                if (!gather) {
                    const int n_rseg = uni(pool.role[0][2]);
                    const int gi = (int)desc_u8(dw, offsetof(LayerDesc, rindex) + pc.g);
                    Emit em{};
                    if (COLLECT && desc_u32(dw, offsetof(LayerDesc, emit_sel))) {
                        const int64_t row = (int64_t)pc.b * n_rseg + gi;
                        em.list = desc_ptr<unsigned long long>(dw, offsetof(LayerDesc, list)) + row * c.list_row;
                        em.count = desc_ptr<int32_t>(dw, offsetof(LayerDesc, list_count)) + row * c.count_stride;
                        em.cap = c.list_row;
                        em.direct = c.block_shift != 0;
                        if (c.prob_rule != 0)
                            em.pool_ml = desc_ptr<float>(dw, offsetof(LayerDesc, part_pool)) + row * (2 * (int64_t)c.part_stride);
                        // rows that need no sample have their threshold at once (what the T unit would say)
                        const int n = budget_of(c, pc.len_b);
                        em.thr_known = needs_no_sample(n, pc.len_b);
                        em.thr = n == pc.len_b && c.prob_rule == 0 ? 0xFFFFFFFFu : 0u;
                        em.thr_flag = A->thr_flags + row * (kLineWords / 2);
                        em.gen = my_gen;
                        em.read_now = kNow;
                        em.timeouts = c.stats + 2;
                    }
                    dispatch_piece<false, true>(__builtin_popcount(pc.hmask), c, dq, dk, dv, nullptr, em, d_part_o, d_part_ml,
                                                d_part_count, alone, pc.b, pc.g, pc.hmask, pc.len_b, pc.r0, pc.r1, pc.slot, pc.ends,
                                                sh.attn, nothing);
                } else {
                    if ((A->gate_mask >> pc.g) & 1ull)
                        await_set(c, A->set_flags + set_flag_at(pc.b, pc.g, c.n_kv_heads), my_gen, pool);
                    const int32_t *idx_src = desc_ptr<const int32_t>(dw, offsetof(LayerDesc, idx_src) + 8 * (size_t)pc.g) +
                                             ((int64_t)pc.b * c.n_kv_heads + pc.g) * c.k;
                    dispatch_piece<true, true>(__builtin_popcount(pc.hmask), c, dq, dk, dv, idx_src, Emit{}, d_part_o, d_part_ml,
                                               d_part_count, alone, pc.b, pc.g, pc.hmask, pc.len_b, pc.r0, pc.r1, pc.slot, pc.ends,
                                               sh.attn, nothing);
                }
            }
            // The piece's partials are in device memory.  Count its blocks in; whoever completes the
            // segment merges its partials (slots 0 .. pieces-1 of every head of the segment).
            __syncthreads();
            A = arg_of<LayerLaunch>();
            ArgCommon &cc = A->c;
            where();
            const int b = uni(pool.at[0]), g = uni(pool.at[1]), pieces = uni(pool.at[4]);
            const uint32_t hmask = (uint32_t)uni(pool.at[2]);
            if (tid == 0) {
                int last = 1, selects = 1;
                const bool awaited = kNow && !gather && A->n_tail > 0;  // by the workgroup that selects the row
                if (pieces > 1 || awaited) {
                    uint32_t *counter = A->seg_count + (((int64_t)b * cc.n_kv_heads + g) * 2 + kind) * kLineWords;
                    const uint32_t mine = (uint32_t)pool.at[8];
                    const uint32_t old = __hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)counter, mine, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT);
                    last = (old & ~kNobodyWaits) + mine == (uint32_t)pool.at[9];
                    selects = !awaited || old >= kNobodyWaits;
                    if (last && selects) store_agent(counter, 0u);  // as every launch finds it
                }
                // 2: and the row's set is this workgroup's (every candidate of the row is in its list)
                pool.flag = !last ? 0 : (kNow && !gather && selects ? 2 : 1);
            }
            __syncthreads();
            // (only now: until the barrier a slower wavefront may still be reading where this piece lay, and
            // one that saw the next piece's place would merge, or not merge, another segment than the others)
            if (tid == 0) pool.run[0] = x + uni(pool.at[3]);
            if (pool.flag) {
                if (pieces > 1 || (kNow && pool.flag == 2)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                if (pieces > 1) switch (__builtin_popcount(hmask)) {
                case 1: combine_segment<1>(cc, cur, b, g, hmask, pieces, sh.comb); break;
                case 2: combine_segment<2>(cc, cur, b, g, hmask, pieces, sh.comb); break;
                case 3: combine_segment<3>(cc, cur, b, g, hmask, pieces, sh.comb); break;
                default: combine_segment<4>(cc, cur, b, g, hmask, pieces, sh.comb); break;
                }
                if (kNow && tid == 0 && pool.flag == 2) {
                    const int row = b * uni(pool.role[0][2]) + (int)desc_u8(dw, offsetof(LayerDesc, rindex) + g);
                    wanted[row >> 5] |= 1u << (row & 31);
                }
            }
            __syncthreads();
        }
        __syncthreads();  // (a workgroup that does both kinds sets up the second: every wavefront has read that the first is done)
        kd = Kind{uni(pool.role[1][0]), uni(pool.role[1][1]), uni(pool.role[1][2]), uni(pool.role[1][3]),
                  uni((int)pool.nb[1][0]), uni(pool.extra[1])};
    }

    // ------------------------------------------------------------------ this layer's own sets
    // The row of a workgroup at the end of the grid, or those of the segments that this one completed and that no
    // such workgroup waits for, after its last piece.  (Selected inside the piece loop they took registers from the
    // streaming, which spilled.)
    if (kNow) {
        __syncthreads();  // (a workgroup without pieces has passed no barrier since thread 0 left the roles)
        const LYCHEE_CONSTANT LayerLaunch *A = arg_of<LayerLaunch>();
        ArgCommon &c = A->c;
        const int n_rseg = uni(pool.role[0][2]);
        const int n_rows = c.batch * n_rseg;
        const int own = A->n_tail > 0 ? w - (W - A->n_tail) : -1;
        bool apart = false;
        if (A->apart != nullptr) {
            apart = selects_apart(pool, c.batch);
            if (w == 0 && tid == 0) store_agent(A->apart, apart ? 1u : 0u);
        }
        if (own >= 0) {
            if (tid == 0) wanted[own >> 5] = 1u << (own & 31);
            __syncthreads();
        }
        for (int i = 0; i < n_rows && !apart; i += 32) {
            for (uint32_t rows = uni(wanted[i >> 5]); rows != 0; rows &= rows - 1u) {
                const int row = i + __builtin_ctz(rows);
                const int b = row / n_rseg, g = cur.rgroup[row % n_rseg];
                if (own >= 0 && !await_rows(c, A->seg_count + ((int64_t)b * c.n_kv_heads + g) * 2 * kLineWords,
                                            (uint32_t)(pool.len[b] + kBlockRows - 1) / kBlockRows, pool))
                    break;
                select_unit<true>(c, cur, b, g, sel, pool, A->thr_flags + row * (kLineWords / 2), pool.gen);
                __syncthreads();
            }
        }
    }

    // ------------------------------------------------------------------ the generation moves on
    if (fresh_tid() == 0 && pool.closes) closes_launch(arg_of<LayerLaunch>(), W, pool.gen);
}

}  // namespace


hipError_t launch_layer(const LayerLaunch &plan, int build, hipStream_t stream)
{
    if (plan.c.n_wg < 1 || plan.c.n_wg > kMaxWg) return hipErrorInvalidValue;
    const dim3 grid(plan.c.n_wg), block(kThreads);
    switch (build) {
    case 0: hipLaunchKernelGGL((lychee_layer_kernel<false, 0>), grid, block, 0, stream, plan); break;
    case 1: hipLaunchKernelGGL((lychee_layer_kernel<true, 1>), grid, block, 0, stream, plan); break;
    case 2: hipLaunchKernelGGL((lychee_layer_kernel<true, 2>), grid, block, 0, stream, plan); break;
    default: hipLaunchKernelGGL((lychee_layer_kernel<true, 3>), grid, block, 0, stream, plan); break;
    }
    return hipGetLastError();
}

}  // namespace lychee
