// C, T, S and A units (included by lychee_units.hip and lychee_layer.hip): the log-sum-exp merge of partials, the
// sampled selection threshold, the exact select of Eq. 2 with the Ratio, Threshold and Top-p
// rules of Sec. 4.4.1, the set copies, and the cache append of Alg. 1.
#pragma once
#include "lychee_device.h"

namespace lychee {
namespace {

// ------------------------------------------------------------------------------ C
// out = (sum_s w_s o_s) / (sum_s w_s l_s),  w_s = 2^((m_s - M) log2(e)/sqrt(d)),  M = max_s m_s,
// over a head's partial slots in ascending order (a fixed summation tree), for all NH heads of a
// segment at once (in a layer launch by the workgroup that has just written the segment's last
// partial, in a phased step by a unit).
// It stands at the end of the layer's chain and is latency, not bytes: the partial outputs of up to
// kGrp * kU slots are asked for before anything else; meanwhile wavefront h turns head h's (m, l)
// pairs into weights (in LDS); then thread (head, group, column quad) sums its group's slots, and
// the groups are added in a fixed order.  (With every wavefront
// keeping every head's running maximum and fetching each weight through the LDS crossbar, 12
// exchanges per head and round and one more per slot, the merge took 6.0 us for 4 heads of 43
// slots, loads in the L2 or not.)
// SKIP: a slot of weight 0 adds nothing whatever it holds (a piece without a valid row re-reads some row
// in its place, and 0 times that row's infinity or NaN is NaN).  C units; in a layer launch such a slot
// shows in the output.
template <int NH, bool SKIP = false>
__device__ __forceinline__ void combine_segment(ArgCommon &c, const LayerDesc &p, int b, int g, uint32_t hmask,
                                                int count, SharedCombine &sh)
{
    constexpr int kGrp = NH == 1 ? 8 : (NH == 2 ? 4 : 2);  // slot groups of a head
    constexpr int kU = 24;                                 // slots a thread has in flight
    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int c4 = tid & 31;  // which 4 columns
    const int h = (tid >> 5) / kGrp;
    const int grp = (tid >> 5) % kGrp;
    // query head, within the group, of the i-th head of the segment
    auto head_of = [&](int i) {
        uint32_t mk = hmask;
#pragma unroll
        for (int j = 1; j < NH; ++j) mk = j <= i ? mk & (mk - 1) : mk;
        return (uint32_t)__builtin_ctz(mk);
    };
    // (addresses are the group's, the same in every lane, and 32-bit offsets from them)
    const int64_t row0 = (int64_t)b * c.n_q_heads + g * c.group;
    const char *po = reinterpret_cast<const char *>(uni(p.part_o + row0 * c.part_stride * kHeadDim));
    const uint32_t po_at = head_of(h < NH ? h : 0) * (uint32_t)c.part_stride * (kHeadDim * 4) + c4 * 16;
    float4 v[kU];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u % 4 == 0 && s0 + kGrp * u >= count) break;  // (uniform)
            const int s = s0 + kGrp * u + grp;
            v[u] = gload_f4(reinterpret_cast<const float *>(po + (po_at + (uint32_t)(s < count ? s : count - 1) * (kHeadDim * 4))));
        }
    };
    fetch(0);
    if (wave < NH) {
        const char *pm = reinterpret_cast<const char *>(uni(p.part_ml + row0 * c.part_stride * 2));
        const uint32_t pm_at = head_of(uni(wave)) * (uint32_t)c.part_stride * 8;
        float M = kMinusBig;
        // (four loads at a time: one by one, each waited for the one before it, 0.7 us each at the end of a 128K layer)
        for (int s0 = lane; s0 < count; s0 += 4 * 64) {
            float2 ml[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u > 0 && s0 - lane + 64 * u >= count) break;  // (uniform)
                ml[u] = gload_f2(reinterpret_cast<const float *>(pm + (pm_at + (uint32_t)min(s0 + 64 * u, count - 1) * 8)));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u > 0 && s0 - lane + 64 * u >= count) break;
                const int s = s0 + 64 * u;
                const float m = ml[u].y > 0.0f ? ml[u].x : kMinusBig;  // (a piece without a valid row leaves l = 0)
                if (s < count) {
                    sh.w[wave][s] = m;
                    sh.ls[wave][s] = ml[u].y > 0.0f ? ml[u].y : 0.0f;
                }
                M = fmaxf(M, m);
            }
        }
        M = wave_max_f(M);
        float l = 0.0f;
        for (int s = lane; s < count; s += 64) {
            const float ls = sh.ls[wave][s];
            const float w = ls > 0.0f ? fast_exp2((sh.w[wave][s] - M) * c.scale_log2e) : 0.0f;
            sh.w[wave][s] = w;
            l = fmaf(w, ls, l);
        }
        l = sum_halves32(sum_rows16(row16_sum(l)));
        if (lane == 0) sh.l[wave] = l;
    }
    __syncthreads();
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (h < NH) {
        for (int s0 = 0;;) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (u % 4 == 0 && s0 + kGrp * u >= count) break;
                const int s = s0 + kGrp * u + grp;
                const float w = s < count ? sh.w[h][s] : 0.0f;
                if (SKIP && !(w > 0.0f)) continue;
                acc.x = fmaf(w, v[u].x, acc.x);
                acc.y = fmaf(w, v[u].y, acc.y);
                acc.z = fmaf(w, v[u].z, acc.z);
                acc.w = fmaf(w, v[u].w, acc.w);
            }
            s0 += kGrp * kU;
            if (s0 >= count) break;
            fetch(s0);
        }
        reinterpret_cast<float4 *>(sh.red + (h * kGrp + grp) * kHeadDim)[c4] = acc;
    }
    __syncthreads();
    for (int i = tid; i < NH * kHeadDim; i += kThreads) {
        const int hh = i / kHeadDim, col = i % kHeadDim;
        float o = 0.0f;
#pragma unroll
        for (int j = 0; j < kGrp; ++j) o += sh.red[(hh * kGrp + j) * kHeadDim + col];
        const float l = sh.l[hh];
        gstore(p.out + (row0 + head_of(hh)) * kHeadDim + col, f32_to_bf16_rne(l > 0.0f ? o / l : 0.0f));
    }
    __syncthreads();
}

// ------------------------------------------------------------------------------ T and S
constexpr uint32_t kNoEntry = 0xFFFFFFFFu;
// (A key of 0 would be a NaN with every bit set, which no score is.  "No entry" needs no test of its
// own that way: a range [lo, hi] with lo >= 1 leaves it out, since 0 - lo wraps beyond hi - lo.
// Tested separately it was one lane mask per entry, kept from pass to pass and spilled.)
__device__ __forceinline__ uint32_t real_key(uint32_t key) { return key > 1u ? key : 1u; }
constexpr int kEntryBatch = 16;  // entries a thread loads before it looks at the first of them

// Among the counted bins, taken from the highest down, the one at which `need` entries are reached:
// its number, how many of its entries are needed, and how many it has.  Every thread sums eight
// neighbouring bins (two 16-byte reads); need must not exceed the count of all bins.
struct Bin {
    uint32_t bin, need, count;
};
__device__ __forceinline__ Bin find_bin(uint32_t need, SharedSelect &sh, int tid)
{
    static_assert(kBins == 8 * kThreads, "eight bins per thread");
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int first = kBins - 8 - 8 * tid;
    const uint4 lo4 = *reinterpret_cast<const uint4 *>(sh.hist + first);
    const uint4 hi4 = *reinterpret_cast<const uint4 *>(sh.hist + first + 4);
    const uint32_t c[8] = {hi4.w, hi4.z, hi4.y, hi4.x, lo4.w, lo4.z, lo4.y, lo4.x};
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += c[j];
    const uint32_t incl = wave_scan(sum);
    if (lane == 63) sh.wave_tot[wave] = incl;
    __syncthreads();
    uint32_t above = incl - sum;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) above += w < wave ? sh.wave_tot[w] : 0u;
    if (above < need && need <= above + sum) {  // one thread
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (above < need && need <= above + c[j]) {
                sh.found[0] = (uint32_t)(first + 7 - j);
                sh.found[1] = need - above;
                sh.found[2] = c[j];
            }
            above += c[j];
        }
    }
    __syncthreads();
    return Bin{uni(sh.found[0]), uni(sh.found[1]), uni(sh.found[2])};
}

// Values to a bin, as a power of two, of a level that splits a range whole.
__device__ __forceinline__ int level_shift(uint32_t range)
{
    return range >= (uint32_t)kBins ? 32 - __builtin_clz(range) - kBinBits : 0;
}

// The entries that pass `among` and whose value lies in [lo, hi], `count` of them, of which the
// `need` with the largest values are wanted.
struct Cut {
    uint32_t lo, hi, need, count;
};
// Narrows [lo, hi] around the need-th largest value until at most `few` entries are left in it, or
// all that are left are equal.  A level splits the range it is given evenly, 2^shift values to a bin
// (the last bin takes what lies beyond), not by fixed digits of the value: the candidates of
// a row lie within a few octaves, whose top digits are a few dozen different ones, and 64 lanes
// that count into the same few LDS words are served one after the other.
template <typename Entries, typename Val, typename Among>
__device__ __forceinline__ Cut narrow(const Entries &E, Cut cut, int shift, uint32_t few, Val val, Among among,
                                      SharedSelect &sh)
{
    const uint32_t lane = (uint32_t)E.tid & 63u;
    while (cut.hi != cut.lo && cut.count > few) {  // (uniform)
        const uint32_t range = cut.hi - cut.lo;
        uint4 *h4 = reinterpret_cast<uint4 *>(sh.hist);
        h4[E.tid] = h4[E.tid + kThreads] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        E.for_each([&](uint32_t key, uint32_t pos) {
            const uint32_t at = val(key, pos) - cut.lo;
            const bool in = among(key, pos) & (at <= range);
            atomicAdd(&sh.hist[in ? min(at >> shift, (uint32_t)kBins - 1u) : (uint32_t)kBins + lane], 1u);
        });
        __syncthreads();
        const Bin b = find_bin(cut.need, sh, E.tid);
        cut.lo += b.bin << shift;
        const uint32_t left = cut.hi - cut.lo, width = (1u << shift) - 1u;
        cut.hi = b.bin == (uint32_t)kBins - 1u || left < width ? cut.hi : cut.lo + width;
        cut.need = b.need;
        cut.count = b.count;
        shift = level_shift(cut.hi - cut.lo);
    }
    return cut;
}

template <int NH>
__device__ __forceinline__ void load_q(ArgCommon &c, const uint16_t *q, int b, int g, uint32_t hmask,
                                       uint4 (&qf)[NH])
{
    const int ch = fresh_tid() & 15;
    uint32_t mk = hmask;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int bit = __builtin_ctz(mk);
        mk &= mk - 1;
        qf[h] = gload_u4(q + ((int64_t)b * c.n_q_heads + g * c.group + bit) * kHeadDim + ch * 8);
    }
}

// Pooled scores of the 16 rows base .. base+15 of one KV head (rows past L-1 repeat row L-1);
// afterwards lane (rs, ch) with ch < 4 holds the score of row base + 4*ch + rs.
template <int NH>
__device__ __forceinline__ float tile_pooled_score(const uint4 (&kr)[4], const uint4 (&qf)[NH], float sel_mul)
{
    const int ch = fresh_tid() & 15;
    float mine = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float pooled = row_score(kr[j], qf[0]);
#pragma unroll
        for (int h = 1; h < NH; ++h) pooled += row_score(kr[j], qf[h]);
        mine = (ch == j) ? sel_value(pooled, sel_mul) : mine;
    }
    return mine;
}

// T unit of score row (b, rgi): the ordered key that a row's pooled score has to reach to
// become a candidate.  The key is the target-th largest of a sample of the row's scores, or the lower end
// of a range of keys that holds it and at most seven more, where target is the number of sampled rows expected among the top n = min(k, L)
// plus sel_margin (six, unless the caller changes it) standard deviations; the streamed rows
// that reach it are then very likely at least n and a few thousand more at most.  Whatever the sample yields, the select unit
// checks the candidate count and ranks the whole row itself when the list cannot be used.
// The sample is one row at a hashed offset inside each of 1024 to 4096 equal strata, as many as let 128
// sampled rows be expected among the top n: the threshold then lets through about 1.6 n rows,
// which a select of n = 4096 holds in registers.  (512 strata where one unit takes the threshold of a short
// launch for itself, see threshold_alone: more rows get through.)
//
// Latency bounds it (the row's streaming pieces wait for it at the end of their rows): one round
// of row loads, a hand-over (but for threshold_alone), one round of key loads, one level of bins (two or more where
// the target lies 16 octaves below the largest key).
// `publish` != nullptr (launches whose streaming runs beside this unit): the threshold goes, with
// the launch's generation `gen` in the upper half, into *publish by one 64-bit atomic store, which
// the row's pieces poll; the candidate counter is not touched (it is zero between uses, and the
// pieces may already be counting).
// `split` (launches whose streaming waits for the threshold): the row's sample is dealt to n_sub
// units, each of which reads its share of the rows in one round of loads and leaves the keys in
// device memory; the unit that arrives last ranks them.  Nobody waits for anybody.
constexpr int kSelRegs = 32;  // entries of a candidate list that a thread of the select keeps in registers
constexpr int kSampleRegs = kSampleTilesMax * 16 / kThreads;
constexpr int kThrNear = 8;  // sampled keys that the threshold may lie below the one that was aimed at
struct SampleEntries {  // the sample's keys, in registers (0: none)
    uint32_t key[kSampleRegs];
    int tid;
    int left;
    template <typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
#pragma unroll
        for (int e = 0; e < kSampleRegs; ++e) {
            if (e % 4 == 0 && e * kThreads >= left) break;  // (uniform)
            f(key[e], 0u);
        }
    }
};
struct ThrSplit {
    int sub = 0, n_sub = 1;
    uint32_t *keys = nullptr;     // [sample size] scratch of this score row
    uint32_t *arrived = nullptr;  // units of this row that have left their keys (zero between launches)
};
template <int NH, typename Pool>
__device__ __forceinline__ void threshold_unit(ArgCommon &c, const LayerDesc &p, int b, int rgi,
                                               SharedSelect &sh, Pool &pool, unsigned long long *publish = nullptr,
                                               uint32_t gen = 0, ThrSplit split = ThrSplit())
{
    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int rs = lane >> 4;
    const int ch = lane & 15;
    const int L = pool.len[b];  // staged by the kernel, clamped
    const int n = budget_of(c, L);
    const int64_t row = (int64_t)b * p.n_rgroups + rgi;
    auto emit = [&](uint32_t key) {
        if (tid != 0) return;
        if (publish != nullptr)
            __hip_atomic_store((LYCHEE_GLOBAL unsigned long long *)publish, ((unsigned long long)gen << 32) | key,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gstore(p.thr + row, key);  // (a later launch's select starts from it)
    };
    if (publish == nullptr && tid == 0) gstore(p.list_count + row * c.count_stride, (int32_t)0);
    if (split.sub == 0 && p.q_keep != nullptr && tid < c.group * (kHeadDim / 8)) {
        // the group's query rows (consecutive heads, 16 chunks of 16 bytes each)
        const int64_t at = ((int64_t)b * c.n_q_heads + p.rgroup[rgi] * c.group) * kHeadDim + tid * 8;
        *(LYCHEE_GLOBAL u32x4_t *)(p.q_keep + at) = *(const LYCHEE_GLOBAL u32x4_t *)(p.q + at);
    }
    if (needs_no_sample(n, L)) {
        // everything is selected anyway (no candidates wanted), or every row is a candidate
        // (a probability rule may keep fewer than everything: it still needs the candidates)
        if (split.sub == 0) emit(n == L && c.prob_rule == 0 ? 0xFFFFFFFFu : 0u);
        return;
    }
    // Short launches: the row's first unit takes one round of loads for itself
    if (split.n_sub > 1 && threshold_alone(n, L, c.batch * p.n_rgroups * ((L + kBlockRows - 1) / kBlockRows), c.n_wg, c.sel_margin,
                                           kThreads * kSelRegs)) {
        if (split.sub > 0) return;
        split = ThrSplit();
    }
    const bool alone = publish != nullptr && split.n_sub == 1;
    // 128 of the top n among the sample, if that takes no more rows than the sample may have; whole rounds
    // of loads of an undivided unit, which takes 2048 rows at most (eight rounds took it 50 us)
    const int most = L >= (1 << 16) && split.n_sub > 1 ? kSampleTilesMax : kSampleTilesMax / 2;
    const int enough = (int)(8.0f * (float)L / (float)n) & ~31;
    const int n_tiles = alone ? kAloneSample / 16 : enough > most ? most : (enough < kSampleTilesMin ? kSampleTilesMin : enough);
    const int n_sample = n_tiles * 16;
    const int g = p.rgroup[rgi];
    const uint32_t hmask = p.rmask[g] & ((1u << c.group) - 1u);
    uint4 qf[NH];
    load_q<NH>(c, p.q, b, g, hmask, qf);
    const uint16_t *kbase = p.k_cache + (int64_t)b * c.stride_b + (int64_t)g * c.stride_h;
    const float sel_mul = c.scale / (float)NH;

    constexpr int kBatch = 8;  // groups of 16 sampled rows a wavefront has in flight
    // One row at a hashed offset in each of n_sample equal strata of rows 0 .. L-2 (the newest
    // row may be being appended in this very launch).  Row by row, not tile by tile: scores
    // come in runs (a passage that matters is hundreds of consecutive rows), and a sample of
    // contiguous tiles would over- or under-count such runs far beyond its nominal deviation.
    const int stratum = quot_uni(L - 1, n_sample);  // >= 2
    const int t_lo = n_tiles * split.sub / split.n_sub, t_hi = n_tiles * (split.sub + 1) / split.n_sub;
    // (sample i of a row lies at i * stratum + umulhi(i * A + row * B, stratum); what is the same in a wavefront
    // is multiplied in scalar registers: two vector multiplications less per load, of 32 before the first is used)
    constexpr uint32_t kHashA = 2654435761u * 2246822519u, kHashB = 40503u * 2246822519u;
    const uint32_t h_lane = (uint32_t)rs * kHashA + (uint32_t)row * kHashB;
    const int p_lane = rs * stratum;
    for (int t0 = t_lo + uni(wave) * kBatch; t0 < t_hi; t0 += kWaves * kBatch) {
        uint4 kr[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int t = t0 + u < t_hi ? t0 + u : t_hi - 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = t * 16 + 4 * j;  // sample number, less rs
                const int pos = i * stratum + p_lane + (int)__umulhi(h_lane + (uint32_t)i * kHashA, (uint32_t)stratum);
                kr[u][j] = gload_u4(kbase + (int64_t)pos * c.stride_t + ch * 8);
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t key = ordered_key(tile_pooled_score<NH>(kr[u], qf, sel_mul));
            if (t0 + u < t_hi && ch < 4) {
                if (split.n_sub > 1)
                    gstore_through(split.keys + (t0 + u) * 16 + 4 * ch + rs, key);
                else
                    sh.samp[(t0 + u) * 16 + 4 * ch + rs] = key;
            }
        }
    }
    if (split.n_sub > 1) {
        // leave the keys, count this unit in; the last one to arrive goes on with all of them
        wait_stores();
        __syncthreads();
        if (tid == 0) {
            const uint32_t old = __hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)split.arrived, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            const bool last = old == (uint32_t)split.n_sub - 1u;
            if (last) __hip_atomic_store((LYCHEE_GLOBAL uint32_t *)split.arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh.found[0] = last;
        }
        __syncthreads();
        const bool last = sh.found[0] != 0;
        __syncthreads();
        if (!last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    } else {
        __syncthreads();
    }
    SampleEntries E;
    E.tid = tid;
    E.left = n_sample;
#pragma unroll
    for (int e = 0; e < kSampleRegs; ++e) {
        if (e % 4 == 0 && e * kThreads >= n_sample) break;
        const int i = e * kThreads + tid;
        const int at = i < n_sample ? i : n_sample - 1;
        const uint32_t key = split.n_sub > 1 ? gload(split.keys + at) : sh.samp[at];
        E.key[e] = i < n_sample ? real_key(key) : 0u;
    }
    const float f = (float)n_sample * (float)n / (float)L;
    const float want = threshold_target(f, c.sel_margin);
    const uint32_t target = want < 1.0f ? 1u : (want > (float)n_sample ? (uint32_t)n_sample : (uint32_t)want);
    uint32_t t_key = 0;
    if (target < (uint32_t)n_sample) {
        // The lower end of a narrow range of keys around the sample's target-th largest.  The first level's
        // bins, 128 to the octave, cover the 16 octaves below the largest key; what lies lower shares
        // the first bin.  So one level is normally enough.  (Over the range of all keys, four bins to the
        // octave, it took two or three, a microsecond each.)
        uint32_t top = 0;
#pragma unroll
        for (int e = 0; e < kSampleRegs; ++e) {
            if (e % 4 == 0 && e * kThreads >= n_sample) break;
            top = E.key[e] > top ? E.key[e] : top;
        }
        top = wave_max(top);
        if (lane == 0) sh.wave_tot[wave] = top;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) top = sh.wave_tot[w] > top ? sh.wave_tot[w] : top;
        top = uni(top);
        const uint32_t low = top > (16u << 23) ? top - (16u << 23) : 0u;
        auto all = [](uint32_t, uint32_t) { return true; };
        const uint32_t above = narrow(
            E, Cut{0u, top - low, target, (uint32_t)n_sample}, 16, (uint32_t)kThrNear,
            [low](uint32_t key, uint32_t) { return key > low ? key - low : 0u; }, all, sh).lo;
        t_key = low + above;
        if (above == 0 && low > 0)  // further down
            t_key = narrow(E, Cut{1u, low, target, (uint32_t)n_sample}, 32 - kBinBits, (uint32_t)kThrNear,
                           [low](uint32_t key, uint32_t) { return key < low ? key : low; }, all, sh).lo;
    }
    emit(t_key);
}

// Writes the pooled score of every row of (b, g) into sel[0 .. L): what the select unit falls
// back on when a row's candidate list is short of n entries or has overflowed.
template <int NH>
__device__ __forceinline__ void score_row_unit(ArgCommon &c, const LayerDesc &p, int b, int g, int L, float *sel)
{
    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int rs = lane >> 4;
    const int ch = lane & 15;
    const uint32_t hmask = p.rmask[g] & ((1u << c.group) - 1u);
    uint4 qf[NH];
    load_q<NH>(c, p.q, b, g, hmask, qf);
    const uint16_t *kbase = p.k_cache + (int64_t)b * c.stride_b + (int64_t)g * c.stride_h;
    const float sel_mul = c.scale / (float)NH;
    const int n_tiles = (L + 15) / 16;
    constexpr int kBatch = 4;
    for (int t0 = wave * kBatch; t0 < n_tiles; t0 += kWaves * kBatch) {
        uint4 kr[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int r = (t0 + u) * 16 + 4 * j + rs;
                r = r < L ? r : L - 1;
                kr[u][j] = gload_u4(kbase + (int64_t)r * c.stride_t + ch * 8);
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float v = tile_pooled_score<NH>(kr[u], qf, sel_mul);
            const int r = (t0 + u) * 16 + 4 * ch + rs;
            if (ch < 4 && r < L) gstore(sel + r, v);
        }
    }
}

// (key, ~position) as one number: larger keys first, then lower positions.
__device__ __forceinline__ unsigned long long ranked(uint32_t key, uint32_t pos)
{
    return ((unsigned long long)key << 32) | (uint32_t)~pos;
}

// Sources of (ordered key, position) entries.  for_each may also hand out "no entry": key 0, below
// every real key, and position kNoEntry.  keep_from leaves the entries from a cutoff on, whose
// positions for_kept hands out eight at a time (at least those of `count` positions from w0 on).  The visitors below fold everything that decides whether an entry counts
// into one flag, with bitwise operators, and let an entry that does not count go to a word of its
// lane's own: short-circuit conditions made the compiler keep a lane mask per entry and
// condition, spill them, and branch several times per entry.
struct RegEntries {           // up to kThreads * kSelRegs list entries, loaded once: beside a streaming
    uint32_t key[kSelRegs], pos[kSelRegs];  // launch every pass over memory costs a microsecond or two
    int tid;
    int left;                 // entries, uniform: whole groups of eight registers beyond them are skipped
    template <int kBatch = 8, typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
#pragma unroll
        for (int e = 0; e < kSelRegs; ++e) {
            if (e % 8 == 0 && e * kThreads >= left) break;
            f(key[e], pos[e]);
        }
    }
    __device__ __forceinline__ void keep_from(unsigned long long cutoff)
    {
#pragma unroll
        for (int e = 0; e < kSelRegs; ++e) {
            if (e % 8 == 0 && e * kThreads >= left) break;
            pos[e] = ranked(key[e], pos[e]) >= cutoff ? pos[e] : kNoEntry;  // (the keys are dead from here on)
        }
    }
    template <typename F>
    __device__ __forceinline__ void for_kept(uint32_t, uint32_t, F f) const
    {
#pragma unroll
        for (int e = 0; e < kSelRegs; e += 8) {
            if (e * kThreads >= left) break;
            uint32_t p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = pos[e + u];
            f(p);
        }
    }
};
struct ListEntries {          // a list too long to be held in LDS: read from memory on every pass
    const unsigned long long *list;
    int total;
    int tid;
    template <int kBatch = kEntryBatch, typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
        for (int i0 = 0; i0 < total; i0 += kBatch * kThreads) {
            const int left = total - i0;  // groups of eight registers beyond it are skipped (uniform)
            unsigned long long v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (u % 8 == 0 && u * kThreads >= left) break;
                const int i = i0 + u * kThreads + tid;
                v[u] = gload(list + (i < total ? i : total - 1));  // unconditional: the loads overlap
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (u % 8 == 0 && u * kThreads >= left) break;
                const bool ok = i0 + u * kThreads + tid < total;
                f(ok ? real_key((uint32_t)v[u]) : 0u, ok ? (uint32_t)(v[u] >> 32) : kNoEntry);
            }
        }
    }
    unsigned long long cutoff = 0;
    __device__ __forceinline__ void keep_from(unsigned long long cut) { cutoff = cut; }
    template <typename F>
    __device__ __forceinline__ void for_kept(uint32_t, uint32_t, F f) const
    {
        for (int i0 = 0; i0 < total; i0 += 8 * kThreads) {
            unsigned long long v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kThreads + tid;
                v[u] = gload(list + (i < total ? i : total - 1));
            }
            uint32_t p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t at = (uint32_t)(v[u] >> 32);
                const bool ok = (i0 + u * kThreads + tid < total) & (ranked(real_key((uint32_t)v[u]), at) >= cutoff);
                p[u] = ok ? at : kNoEntry;
            }
            f(p);
        }
    }
};
struct RowEntries {           // every row of the sequence, from its recomputed scores
    const float *sel;
    int total;
    int tid;
    template <int kBatch = 8, typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
        const int end = total;
        for (int i0 = tid; i0 < end; i0 += 8 * kThreads) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kThreads;
                v[u] = gload(sel + (i < end ? i : end - 1));
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kThreads;
                f(i < end ? real_key(ordered_key(v[u])) : 0u, i < end ? (uint32_t)i : kNoEntry);
            }
        }
    }
    unsigned long long cutoff = 0;
    __device__ __forceinline__ void keep_from(unsigned long long cut) { cutoff = cut; }
    template <typename F>
    __device__ __forceinline__ void for_kept(uint32_t w0, uint32_t count, F f) const
    {
        const int end = (int)(count < (uint32_t)total - w0 ? w0 + count : (uint32_t)total);
        for (int i0 = (int)w0 + tid; i0 < end; i0 += 8 * kThreads) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kThreads;
                v[u] = gload(sel + (i < end ? i : end - 1));
            }
            uint32_t p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kThreads;
                p[u] = ((i < end) & (ranked(real_key(ordered_key(v[u])), (uint32_t)i) >= cutoff)) ? (uint32_t)i : kNoEntry;
            }
            f(p);
        }
    }
};

// The smallest ranked() among the `need` largest of the entries in `cut`: the range of keys is
// narrowed until it holds at most kLastKeys entries, which are then ranked against one another;
// equal keys that are more than that are cut at a position found the same way.
template <typename Entries>
__device__ __forceinline__ unsigned long long cutoff_of(const Entries &E, Cut cut, int shift, int L, SharedSelect &sh)
{
    if (E.tid == 0) sh.n_last = 0;
    __syncthreads();  // (a list of kLastKeys entries or fewer goes straight to its use)
    cut = narrow(
        E, cut, shift, (uint32_t)kLastKeys, [](uint32_t key, uint32_t) { return key; },
        [](uint32_t, uint32_t) { return true; }, sh);
    if (cut.need == cut.count) return (unsigned long long)cut.lo << 32;
    if (cut.count > (uint32_t)kLastKeys) {
        const uint32_t key_cut = cut.lo;
        const Cut at = narrow(
            E, Cut{~(uint32_t)(L - 1), 0xFFFFFFFFu, cut.need, cut.count}, level_shift((uint32_t)(L - 1)), 0u,
            [](uint32_t, uint32_t pos) { return ~pos; }, [&](uint32_t key, uint32_t) { return key == key_cut; }, sh);
        return ((unsigned long long)key_cut << 32) | at.lo;
    }
    E.for_each([&](uint32_t key, uint32_t pos) {
        if (key - cut.lo <= cut.hi - cut.lo) sh.last[atomicAdd(&sh.n_last, 1u)] = ranked(key, pos);
    });
    __syncthreads();
    if ((uint32_t)E.tid < cut.count) {
        const unsigned long long mine = sh.last[E.tid];
        uint32_t above = 0;
        // (pairs, eight at a time: read one by one, each read waits for the one before it; what lies
        // past the last entry is not counted)
        for (uint32_t i0 = 0; i0 < cut.count; i0 += 16) {
            ulonglong2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = reinterpret_cast<const ulonglong2 *>(sh.last)[i0 / 2 + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                above += (uint32_t)((i0 + 2 * u < cut.count) & (v[u].x > mine));
                above += (uint32_t)((i0 + 2 * u + 1 < cut.count) & (v[u].y > mine));
            }
        }
        if (above + 1u == cut.need) sh.cutoff = mine;
    }
    __syncthreads();
    return sh.cutoff;
}

// Writes the positions of the kept entries to dst in ascending order: they are marked in an LDS bitmap,
// 131072 positions at a time, prefix sums over its words give every one its place, and each entry
// stages itself there.
template <typename Entries>
__device__ __forceinline__ void write_ordered(const Entries &E, int L, int32_t *dst, SharedSelect &sh)
{
    const int tid = E.tid;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    constexpr uint32_t kWindow = kMapWords * 32u;
    uint32_t base = 0;  // positions chosen in earlier windows
    for (uint32_t w0 = 0; w0 < (uint32_t)L; w0 += kWindow) {
        const uint32_t span = (uint32_t)L - w0 < kWindow ? (uint32_t)L - w0 : kWindow;
        // wavefront w owns words w << (6 + lg) .. of the window, 64 << lg of them
        const uint32_t per = (span + 32 * kThreads - 1) / (32 * kThreads);
        const int lg = per > 1 ? 32 - __builtin_clz(per - 1) : 0;
        const int rounds = 1 << lg;
        __syncthreads();
        for (int r = 0; r < rounds; ++r) sh.bits[r * kThreads + tid] = 0;
        __syncthreads();
        E.for_kept(w0, span, [&](const uint32_t (&pos)[8]) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t rel = pos[u] - w0;  // "no entry" lies outside every window
                atomicOr(&sh.bits[rel < span ? rel >> 5 : (uint32_t)(kMapWords + lane)], 1u << (rel & 31u));
            }
        });
        __syncthreads();
        const int first = (wave << (6 + lg)) + lane;
        uint32_t mine = 0;
        for (int r = 0; r < rounds; ++r) {
            const uint32_t c = (uint32_t)__builtin_popcount(sh.bits[first + r * 64]);
            const uint32_t incl = wave_scan(c);
            sh.before[first + r * 64] = (uint16_t)(mine + incl - c);  // (at most 1024 words of 32 before it)
            mine += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (lane == 0) sh.wave_tot[wave] = mine;
        __syncthreads();
        uint32_t at[kWaves], end = base;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            at[w] = end;
            end += sh.wave_tot[w];
        }
        // Staged in LDS and copied out with coalesced write-through stores: the set is in device
        // memory once the unit's stores have completed, whoever reads it next (a gather piece of
        // the same launch, on another XCD, past its caches).
        for (uint32_t c0 = base; c0 < end; c0 += (uint32_t)kStage) {
            E.for_kept(w0, span, [&](const uint32_t (&pos)[8]) {
                // (all lookups of a group before its first store: a lookup after a store waits for
                // it, the compiler cannot tell their LDS words apart)
                uint32_t put_at[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t rel = pos[u] - w0;
                    const uint32_t word_at = rel < span ? rel >> 5 : 0u;
                    const uint32_t word = sh.bits[word_at];
                    const uint32_t bit = 1u << (rel & 31u);
                    const uint32_t owner = word_at >> (6 + lg);
                    uint32_t place = owner == 0 ? at[0] : (owner == 1 ? at[1] : (owner == 2 ? at[2] : at[3]));
                    place += sh.before[word_at] + (uint32_t)__builtin_popcount(word & (bit - 1u)) - c0;
                    const bool put = (rel < span) & (place < (uint32_t)kStage);
                    put_at[u] = put ? place : (uint32_t)(kStage + lane);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) sh.stage[put_at[u]] = pos[u];
            });
            __syncthreads();
            const uint32_t m = end - c0 < (uint32_t)kStage ? end - c0 : (uint32_t)kStage;
            for (uint32_t i0 = 0; i0 < m; i0 += 8 * kThreads) {  // (eight reads, then eight stores)
                int32_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = (int32_t)sh.stage[i0 + u * kThreads + tid];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t i = i0 + u * kThreads + tid;
                    if (i < m) gstore_through(dst + c0 + i, v[u]);
                }
            }
            __syncthreads();
        }
        base = end;
    }
}

// Where the first level's bins begin and how wide they are (as a power of two).  Rows that were
// sampled hold keys from their threshold up: bins over the eight octaves above it, 256 to the
// octave.  Others (short rows, blocks, rows ranked whole): the range of all keys, four to the octave.
struct Level {
    uint32_t lo;
    int shift;
};
__device__ __forceinline__ Level first_level(uint32_t floor_key)
{
    return Level{floor_key > 1u ? floor_key : 1u, floor_key >= 0x80000000u ? 26 - kBinBits : 32 - kBinBits};
}

// Exact top-n of the `total` entries by key, ties to the lower position (Eq. 2), written to dst in
// ascending position order.
//
// One workgroup, a chain of LDS passes and barriers: latency bounds it.  6500 candidates, k = 4096, from
// the entries in registers to the last store: 9.6 us alone, 12.5 us beside a streaming launch.  (Three
// passes over fixed digits of the key, two more passes and a walk over the bitmap's bits took 17
// and 21 us, as long for 256 of 4096 rows, which takes 6.5 us now.)  Entries held in LDS as bin and
// position with the last bin's keys looked up again took 15 us, re-read from memory on every pass
// 15 to 20 us.
template <typename Entries>
__device__ __forceinline__ void select_from(Entries &E, uint32_t floor_key, int total, int n, int L, int32_t *dst,
                                            SharedSelect &sh)
{
    const Level lv = first_level(floor_key);
    E.keep_from(cutoff_of(E, Cut{lv.lo, 0xFFFFFFFFu, (uint32_t)n, (uint32_t)total}, lv.shift, L, sh));
    write_ordered(E, L, dst, sh);
}

// A unit of one layer (Alg. 1, "C.append(k, v)"): the decoded token's key and value rows become
// row L_b - 1 of every KV head's cache.  16 lanes move one 256-byte row.
__device__ __forceinline__ void append_unit(ArgCommon &c, const LayerDesc &p)
{
    const int ch = fresh_tid() & 15;
    const int n_rows = c.batch * c.n_kv_heads * 2;  // K rows, then V rows
    for (int r = fresh_tid() >> 4; r < n_rows; r += kThreads >> 4) {
        const int which = r / (c.batch * c.n_kv_heads);
        const int bg = r % (c.batch * c.n_kv_heads);
        const int b = bg / c.n_kv_heads, g = bg % c.n_kv_heads;
        const int L = clamp_len(gload(c.lengths + b), c.max_len);
        const uint16_t *src = (which ? p.v_new : p.k_new) + (int64_t)bg * kHeadDim + ch * 8;
        const uint16_t *dst = (which ? p.v_cache : p.k_cache) + (int64_t)b * c.stride_b +
                              (int64_t)g * c.stride_h + (int64_t)(L - 1) * c.stride_t + ch * 8;
        const uint4 v = gload_u4(src);
        *(LYCHEE_GLOBAL u32x4_t *)const_cast<uint16_t *>(dst) = u32x4_t{v.x, v.y, v.z, v.w};
    }
}

// ---- the probability rules of Sec. 4.4.1 (Threshold, Top-p): how many entries to keep
// The pooled logit an ordered key stands for.
__device__ __forceinline__ float key_score(uint32_t key)
{
    return __builtin_bit_cast(float, (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// Probability of a pooled logit under the softmax over the whole sequence, as a 40-bit
// fixed-point number: sums of these are integer sums, the same in any order.
constexpr float kMassOne = 1099511627776.0f;  // 2^40
__device__ __forceinline__ unsigned long long mass_of(uint32_t key, float lse)
{
    const float p = fast_exp2((key_score(key) - lse) * kLog2e);  // <= 1 up to rounding
    return (unsigned long long)(fminf(p, 1.0f) * kMassOne);
}

// In the histogram of probability mass per bin, from the highest bin down, the one at which `need` is
// reached, and what is still needed inside it; false when all the mass together does not reach it.
template <typename Pool>
__device__ __forceinline__ bool find_bin_mass(const unsigned long long *mass, unsigned long long need, Pool &pool,
                                              SharedSelect &sh, int tid, uint32_t &bin, unsigned long long &left)
{
    const int first = kBins - 8 - 8 * tid;
    unsigned long long c[8], sum = 0, total;
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += c[j] = mass[first + 7 - j];
    unsigned long long above = block_scan64(sum, pool.scan64, total) - sum;
    if (total < need) return false;  // (uniform)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (above < need && need <= above + c[j]) {  // one thread
            sh.found[0] = (uint32_t)(first + 7 - j);
            sh.cutoff = need - above;
        }
        above += c[j];
    }
    __syncthreads();
    bin = uni(sh.found[0]);
    left = sh.cutoff;
    __syncthreads();
    return true;
}

// Entries the rule keeps, before the clamp to [1, n]: Threshold counts the entries whose
// probability exceeds the parameter; Top-p finds, bin by bin, the key at which the
// probability mass of the descending order reaches the parameter (all entries with that key
// have the same mass, so a division says how many of them are needed).  `lse` is the
// log-sum-exp of the pooled logits of the whole sequence.  The entries hold at least the n best
// positions, and a rule that would go beyond them is capped at n anyway.
template <typename Entries, typename Pool>
__device__ __forceinline__ int rule_keeps(ArgCommon &c, const Entries &E, uint32_t floor_key, int n, float lse,
                                          SharedSelect &sh, Pool &pool)
{
    uint32_t want;
    if (c.prob_rule == 1) {
        const uint32_t cut = ordered_key(lse + __logf(c.prob_param));
        uint32_t mine = 0;
        E.template for_each<8>([&](uint32_t key, uint32_t pos) { mine += (uint32_t)(key > cut); });
        (void)block_scan(mine, pool.scan, want);
    } else {
        if (c.prob_param >= 1.0f) return n;  // all of the mass: everything, i.e. the cap
        unsigned long long *mh = sh.mass;
        unsigned long long need = (unsigned long long)((double)c.prob_param * (double)kMassOne);
        need = need < 1 ? 1 : need;
        // The range of keys is split into bins of mass as the select splits it into bins of entries, until the
        // bin where the mass is reached holds few entries, which are looked at one by one.
        const Level lv = first_level(floor_key);
        uint32_t lo = lv.lo, hi = 0xFFFFFFFFu, above;
        for (int shift = lv.shift;; shift = level_shift(hi - lo)) {
            for (int i = E.tid; i < kBins; i += kThreads) mh[i] = 0;
            if (E.tid == 0) sh.n_last = 0;
            __syncthreads();
            E.template for_each<8>([&](uint32_t key, uint32_t) {
                const uint32_t at = key - lo;
                if (at <= hi - lo) atomicAdd(&mh[min(at >> shift, (uint32_t)kBins - 1u)], mass_of(key, lse));
            });
            __syncthreads();
            uint32_t bin;
            if (!find_bin_mass(mh, need, pool, sh, E.tid, bin, need)) return n;  // not even all entries reach the mass: the cap decides
            lo += bin << shift;
            const uint32_t rest = hi - lo, width = (1u << shift) - 1u;
            hi = bin == (uint32_t)kBins - 1u || rest < width ? hi : lo + width;
            uint32_t mine = 0;
            E.template for_each<8>([&](uint32_t key, uint32_t) {
                mine += (uint32_t)(key > hi);
                if (key - lo <= hi - lo) {
                    const uint32_t at = atomicAdd(&sh.n_last, 1u);
                    if (at < (uint32_t)kLastKeys) sh.last[at] = key;
                }
            });
            (void)block_scan(mine, pool.scan, above);  // (its barriers publish the keys)
            const uint32_t in_bin = uni(sh.n_last);
            __syncthreads();  // (the next level, or the select that follows, counts in n_last anew)
            if (in_bin > (uint32_t)kLastKeys && hi != lo) continue;
            // the key at which the mass is reached; all entries with that key have the same mass
            if (in_bin > (uint32_t)kLastKeys) {  // (all equal)
                const unsigned long long each = mass_of(lo, lse);
                want = above + (uint32_t)((need + each - 1) / each);
                break;
            }
            if ((uint32_t)E.tid < in_bin) {
                const uint32_t key = (uint32_t)sh.last[E.tid];
                unsigned long long sum = 0;
                uint32_t larger = 0, equal = 0;
                for (uint32_t i = 0; i < in_bin; ++i) {
                    const uint32_t k = (uint32_t)sh.last[i];
                    sum += k > key ? mass_of(k, lse) : 0ull;
                    larger += (uint32_t)(k > key);
                    equal += (uint32_t)(k == key);
                }
                const unsigned long long each = mass_of(key, lse);
                if (sum < need && need <= sum + each * equal)  // (the same in every thread with this key)
                    sh.found[0] = above + larger + (uint32_t)((need - sum + each - 1) / each);
            }
            __syncthreads();
            want = uni(sh.found[0]);
            __syncthreads();
            break;
        }
    }
    return want < 1u ? 1 : (want > (uint32_t)n ? n : (int)want);
}

// Log-sum-exp of the pooled logits of score row `row`: the pieces' states, merged.
template <typename Pool>
__device__ __forceinline__ float pooled_lse(ArgCommon &c, const LayerDesc &p, int64_t row, int count,
                                            Pool &pool)
{
    const float *ml = p.part_pool + row * (2 * (int64_t)c.part_stride);
    float m_loc = kMinusBig;
    for (int s = fresh_tid(); s < count; s += kThreads) m_loc = fmaxf(m_loc, gload(ml + 2 * s));
    const float M = block_max(m_loc, pool.fred);
    float l_loc = 0.0f;
    for (int s = fresh_tid(); s < count; s += kThreads)
        l_loc = fmaf(fast_exp2((gload(ml + 2 * s) - M) * kLog2e), gload(ml + 2 * s + 1), l_loc);
    const float l = block_sum(l_loc, pool.fred);
    return M + __logf(l);
}

// The set of a KV head (b, g) whose group holds no retrieval head is handed on unchanged
// (Sec. 3.1): a verbatim copy.
__device__ __forceinline__ void copy_set_unit(ArgCommon &c, const LayerDesc &p, int b, int g)
{
    const int64_t bg = (int64_t)b * c.n_kv_heads + g;
    int32_t *dst = p.idx_out + bg * c.k;
    const int32_t *src = p.idx_src[g] + bg * c.k;
    for (int i = fresh_tid(); i < c.k; i += kThreads) gstore_through(dst + i, gload(src + i));
}

// S unit of KV head (b, g), whose group holds a retrieval head: the set the next layer's
// sparse heads of the group inherit.  PROB: the build that knows the probability rules (their
// 64-bit mass arithmetic over register-resident entries would cost the plain build registers).
// flag, gen: the row's threshold word and the generation, when the launch that streams the row
// also selects for it.
template <bool PROB, typename Pool>
__device__ __forceinline__ void select_unit(ArgCommon &c, const LayerDesc &p, int b, int g,
                                            SharedSelect &sh, Pool &pool, const unsigned long long *flag = nullptr,
                                            uint32_t gen = 0)
{
    const int64_t bg = (int64_t)b * c.n_kv_heads + g;
    int32_t *dst = p.idx_out + bg * c.k;
    const int rgi = p.rindex[g];
    const int len = pool.len[b];  // staged by the kernel, clamped
    const int L = units_of(c, len);  // what is ranked: positions, or blocks of positions
    const int n = budget_of(c, L);
    const bool by_prob = PROB && c.prob_rule != 0;
    if (n == L && !by_prob) {  // everything is selected
        for (int i = fresh_tid(); i < c.k; i += kThreads) gstore_through(dst + i, (int32_t)(i < L ? i : -1));
        if (fresh_tid() == 0 && c.block_shift == 0 && rgi != 0xFF)
            gstore(p.list_count + ((int64_t)b * p.n_rgroups + rgi) * c.count_stride, (int32_t)0);  // (nothing was collected; see below)
        return;
    }
    const int64_t row = (int64_t)b * p.n_rgroups + rgi;
    const unsigned long long *list = p.list + row * (int64_t)c.list_row;
    // The first entries are asked for before the list's length is known.
    const int tid = fresh_tid();
    constexpr int kHead = 8;
    unsigned long long head[kHead];
#pragma unroll
    for (int u = 0; u < kHead; ++u) {
        const int i = u * kThreads + tid;
        head[u] = gload(list + (i < c.list_row ? i : c.list_row - 1));
    }
    // block-granular: the streaming left every block's score at its place in the list
    const int total = c.block_shift ? L : gload(p.list_count + row * c.count_stride);
    // No entry lies below the row's threshold.  (A select of the launch that streamed the row takes it
    // from where the row's pieces did; rows whose pieces asked nobody may not have one there yet.)
    uint32_t floor_key = 0;
    if (c.block_shift == 0 && !needs_no_sample(n, len)) {
        if (flag != nullptr) {
            const unsigned long long v = __hip_atomic_load((const LYCHEE_GLOBAL unsigned long long *)flag, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT);
            floor_key = (uint32_t)(v >> 32) == gen ? (uint32_t)v : 0u;
        } else {
            floor_key = gload(p.thr + row);
        }
    }
    // The select is the counter's only reader: it leaves it at zero for the next launch that
    // collects into it (a launch whose streaming runs beside its threshold units has nobody who
    // could clear it first).  Every thread has read it before any thread gets past the barriers
    // that follow, so one thread may clear it then.
    const bool clear_count = c.block_shift == 0;
    float lse = 0.0f;
    if (by_prob) {
        // the pieces of this KV head's segment, counted by its first retrieval head
        const int h = g * c.group + __builtin_ctz((uint32_t)p.rmask[g]);
        int count = gload(p.part_count + (int64_t)b * c.n_q_heads + h);
        count = count < 0 ? 0 : (count > c.part_stride ? c.part_stride : count);
        lse = pooled_lse(c, p, row, count, pool);
    }
    int keep = n;  // what is selected in the end: n, or fewer under a probability rule
    const bool usable = total >= n && total <= c.list_row;
    if (PROB && by_prob && usable) {
        // (from memory, a few entries at a time: with the rules' 64-bit masses beside resident entries the
        // whole kernel spilled, and its threshold units took four times as long)
        ListEntries M;
        M.list = list, M.total = total, M.tid = tid;
        keep = rule_keeps(c, M, floor_key, n, lse, sh, pool);
    }
    if (usable && total <= kThreads * kSelRegs) {
        RegEntries E;
        E.tid = tid;
        E.left = total;
#pragma unroll
        for (int e = 0; e < kSelRegs; ++e) {
            if (e % 8 == 0 && e * kThreads >= total) break;  // (uniform)
            const int i = e * kThreads + tid;
            const unsigned long long v = e < kHead ? head[e] : gload(list + (i < total ? i : total - 1));
            E.key[e] = i < total ? real_key((uint32_t)v) : 0u;
            E.pos[e] = i < total ? (uint32_t)(v >> 32) : kNoEntry;
        }
        select_from(E, floor_key, total, keep, L, dst, sh);
    } else if (usable) {
        ListEntries M;
        M.list = list, M.total = total, M.tid = tid;
        select_from(M, floor_key, total, keep, L, dst, sh);
    } else {
        // too few candidates reached the threshold, or too many for the list: rank the row
        // (token-granular only: a block list is always complete)
        if (fresh_tid() == 0) (void)__hip_atomic_fetch_add((LYCHEE_GLOBAL uint32_t *)c.stats + (total < n ? 0 : 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        float *sel = p.sel + row * c.sel_stride;
        switch (__builtin_popcount(p.rmask[g] & ((1u << c.group) - 1u))) {
        case 1: score_row_unit<1>(c, p, b, g, len, sel); break;
        case 2: score_row_unit<2>(c, p, b, g, len, sel); break;
        case 3: score_row_unit<3>(c, p, b, g, len, sel); break;
        default: score_row_unit<4>(c, p, b, g, len, sel); break;
        }
        __threadfence();
        __syncthreads();  // the scores are read back by other threads of the workgroup
        RowEntries M;
        M.sel = sel, M.total = len, M.tid = tid;
        if (PROB && by_prob) keep = rule_keeps(c, M, 0u, n, lse, sh, pool);
        select_from(M, 0u, len, keep, L, dst, sh);
    }
    for (int i = keep + fresh_tid(); i < c.k; i += kThreads) gstore_through(dst + i, (int32_t)-1);
    if (clear_count && fresh_tid() == 0) gstore(p.list_count + row * c.count_stride, (int32_t)0);
}


}  // namespace
}  // namespace lychee
