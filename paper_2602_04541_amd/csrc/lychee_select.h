// C, T, S and A units (included by lychee_units.hip and lychee_layer.hip): the log-sum-exp merge of partials, the
// sampled selection threshold, the exact radix select of Eq. 2 with the Ratio, Threshold and Top-p
// rules of Sec. 4.4.1, the set copies, and the cache append of Alg. 1.
#pragma once
#include "lychee_device.h"

namespace lychee {
namespace {

// ------------------------------------------------------------------------------ C
// out = (sum_s w_s o_s) / (sum_s w_s l_s),  w_s = 2^((m_s - M) log2(e)/sqrt(d)),  M = max_s m_s,
// over the head's partial slots in ascending order (a fixed summation tree).
// `known_count` >= 0: the number of partial slots, known to the caller; else it is read from part_count.
template <typename Pool>
__device__ __forceinline__ void combine_unit(const Common &c, const LayerDesc &p, int bh, SharedCombine &sh,
                                             Pool &pool, int known_count = -1)
{
    int count = known_count >= 0 ? known_count : gload(p.part_count + bh);
    count = count < 0 ? 0 : (count > c.part_stride ? c.part_stride : count);
    const float *ml = p.part_ml + (int64_t)bh * c.part_stride * 2;
    const float *po = p.part_o + (int64_t)bh * c.part_stride * kHeadDim;
    float m_loc = kMinusBig;
    for (int s = threadIdx.x; s < count; s += kThreads)
        if (gload(ml + 2 * s + 1) > 0.0f) m_loc = fmaxf(m_loc, gload(ml + 2 * s));
    const float M = block_max(m_loc, pool.fred);
    float l_loc = 0.0f;
    for (int s = threadIdx.x; s < count; s += kThreads) {
        const float ls = gload(ml + 2 * s + 1);
        const float w = ls > 0.0f ? fast_exp2((gload(ml + 2 * s) - M) * c.scale_log2e) : 0.0f;
        sh.w[0][s] = w;
        l_loc = fmaf(w, ls, l_loc);
    }
    const float lsum = block_sum(l_loc, pool.fred);  // also publishes sh.w
    constexpr int kLanes = kThreads / 32;  // interleaved slot subsets
    const int lane8 = threadIdx.x >> 5;
    const int c4 = threadIdx.x & 31;       // which 4 columns
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = lane8; s0 < count; s0 += 8 * kLanes) {
        // 8 slots per thread and round, all loads issued before the first use
        float wv[8];
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int s = s0 + kLanes * u;
            wv[u] = s < count ? sh.w[0][s] : 0.0f;
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (wv[u] > 0.0f) v[u] = gload_f4(po + (int64_t)s * kHeadDim + c4 * 4);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            acc.x = fmaf(wv[u], v[u].x, acc.x);
            acc.y = fmaf(wv[u], v[u].y, acc.y);
            acc.z = fmaf(wv[u], v[u].z, acc.z);
            acc.w = fmaf(wv[u], v[u].w, acc.w);
        }
    }
    reinterpret_cast<float4 *>(sh.red + lane8 * kHeadDim)[c4] = acc;
    __syncthreads();
    if (threadIdx.x < kHeadDim) {
        float o = 0.0f;
#pragma unroll
        for (int i = 0; i < kLanes; ++i) o += sh.red[i * kHeadDim + threadIdx.x];
        const float r = lsum > 0.0f ? o / lsum : 0.0f;
        gstore(p.out + (int64_t)bh * kHeadDim + threadIdx.x, f32_to_bf16_rne(r));
    }
    __syncthreads();
}

// The same merge for all NH heads of a segment at once, by the workgroup that has just written the
// segment's last partial.  It stands at the end of the layer's chain and is latency, not bytes: the
// partial outputs of up to kGrp * kU slots are asked for before anything else; meanwhile wavefront
// h turns head h's (m, l) pairs into weights (in LDS); then thread (head, group, column quad)
// sums its group's slots, and the groups are added in a fixed order.  (With every wavefront
// keeping every head's running maximum and fetching each weight through the LDS crossbar, 12
// exchanges per head and round and one more per slot, the merge took 6.0 us for 4 heads of 43
// slots, loads in the L2 or not.)
template <int NH>
__device__ __forceinline__ void combine_segment(const Common &c, const LayerDesc &p, int b, int g, uint32_t hmask,
                                                int count, SharedCombine &sh)
{
    constexpr int kGrp = NH == 1 ? 8 : (NH == 2 ? 4 : 2);  // slot groups of a head
    constexpr int kU = 16;                                 // slots a thread has in flight
    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int c4 = tid & 31;  // which 4 columns
    const int h = (tid >> 5) / kGrp;
    const int grp = (tid >> 5) % kGrp;
    // (sequence, head) row of the i-th head of the segment
    auto row_of = [&](int i) {
        uint32_t mk = hmask;
#pragma unroll
        for (int j = 1; j < NH; ++j) mk = j <= i ? mk & (mk - 1) : mk;
        return (int64_t)b * c.n_q_heads + g * c.group + __builtin_ctz(mk);
    };
    const float *po = p.part_o + row_of(h < NH ? h : 0) * c.part_stride * kHeadDim + c4 * 4;
    float4 v[kU];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u % 4 == 0 && s0 + kGrp * u >= count) break;  // (uniform)
            const int s = s0 + kGrp * u + grp;
            v[u] = gload_f4(po + (int64_t)(s < count ? s : count - 1) * kHeadDim);
        }
    };
    fetch(0);
    if (wave < NH) {
        const float *pm = p.part_ml + row_of(wave) * c.part_stride * 2;
        float M = kMinusBig;
        for (int s = lane; s < count; s += 64) {
            const float2 ml = gload_f2(pm + 2 * s);
            const float m = ml.y > 0.0f ? ml.x : kMinusBig;  // (a piece without a valid row leaves l = 0)
            sh.w[wave][s] = m;
            sh.ls[wave][s] = ml.y > 0.0f ? ml.y : 0.0f;
            M = fmaxf(M, m);
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
        gstore(p.out + row_of(hh) * kHeadDim + col, f32_to_bf16_rne(l > 0.0f ? o / l : 0.0f));
    }
    __syncthreads();
}

// ------------------------------------------------------------------------------ T and S
constexpr uint32_t kNoEntry = 0xFFFFFFFFu;
// (A key of 0 would be a NaN with every bit set, which no score is.  "No entry" needs no test of its
// own that way: a range [lo, hi] with lo >= 1 leaves it out, since 0 - lo wraps beyond hi - lo.
// Tested separately it was one lane mask per entry, kept from pass to pass and spilled.)
__device__ __forceinline__ uint32_t real_key(uint32_t key) { return key > 1u ? key : 1u; }
constexpr int kEntryBatch = 32;  // entries a thread loads before it looks at the first of them

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
__device__ __forceinline__ void load_q(const Common &c, const uint16_t *q, int b, int g, uint32_t hmask,
                                       uint4 (&qf)[NH])
{
    const int ch = threadIdx.x & 15;
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
    const int ch = threadIdx.x & 15;
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
// become a candidate.  The key is the target-th largest of a sample of the row's scores,
// to 22 bits, where target is the number of sampled rows expected among the top n = min(k, L)
// plus sel_margin (six, unless the caller changes it) standard deviations; the streamed rows
// that reach it are then very likely at least n and a few thousand more at most.  Whatever the sample yields, the select unit
// checks the candidate count and ranks the whole row itself when the list cannot be used.
// The sample is one row at a hashed offset inside each of 1024 to 4096 equal strata: 2048 and more
// for long rows, fewer where 64 sampled rows are expected among the top n all the same.
//
// Latency bounds it (the row's streaming pieces wait for it at the end of their rows): one round
// of row loads, a hand-over, one round of key loads, two levels of bins.
// `publish` != nullptr (launches whose streaming runs beside this unit): the threshold goes, with
// the launch's generation `gen` in the upper half, into *publish by one 64-bit atomic store, which
// the row's pieces poll; the candidate counter is not touched (it is zero between uses, and the
// pieces may already be counting).
// `split` (launches whose streaming waits for the threshold): the row's sample is dealt to n_sub
// units, each of which reads its share of the rows in one round of loads and leaves the keys in
// device memory; the unit that arrives last ranks them.  Nobody waits for anybody.
constexpr int kSampleRegs = kSampleTilesMax * 16 / kThreads;
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
__device__ __forceinline__ void threshold_unit(const Common &c, const LayerDesc &p, int b, int rgi,
                                               SharedSelect &sh, Pool &pool, unsigned long long *publish = nullptr,
                                               uint32_t gen = 0, const ThrSplit split = ThrSplit())
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
        gstore(p.thr + row, key);  // (the row's select starts from it)
    };
    if (publish == nullptr && tid == 0) gstore(p.list_count + row, (int32_t)0);
    if (split.sub == 0 && p.q_keep != nullptr && tid < c.group * (kHeadDim / 8)) {
        // the group's query rows (consecutive heads, 16 chunks of 16 bytes each)
        const int64_t at = ((int64_t)b * c.n_q_heads + p.rgroup[rgi] * c.group) * kHeadDim + tid * 8;
        *(LYCHEE_GLOBAL u32x4_t *)(p.q_keep + at) = *(const LYCHEE_GLOBAL u32x4_t *)(p.q + at);
    }
    if (n == L || L <= kDirectLen || 2 * (int64_t)n >= L) {
        // everything is selected anyway (no candidates wanted), or every row is a candidate
        // (a probability rule may keep fewer than everything: it still needs the candidates)
        if (split.sub == 0) emit(n == L && c.prob_rule == 0 ? 0xFFFFFFFFu : 0u);
        return;
    }
    int n_tiles = L / 1024;
    n_tiles = n_tiles < kSampleTilesMin ? kSampleTilesMin : (n_tiles > kSampleTilesMax ? kSampleTilesMax : n_tiles);
    const int enough = (int)(4.0f * (float)L / (float)n) + 1;  // tiles of 16 rows that hold 64 of the top n
    n_tiles = enough < n_tiles ? (enough > kSampleTilesFew ? enough : kSampleTilesFew) : n_tiles;
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
    const int stratum = (L - 1) / n_sample;  // >= 2
    const int t_lo = n_tiles * split.sub / split.n_sub, t_hi = n_tiles * (split.sub + 1) / split.n_sub;
    for (int t0 = t_lo + wave * kBatch; t0 < t_hi; t0 += kWaves * kBatch) {
        uint4 kr[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int t = t0 + u < t_hi ? t0 + u : t_hi - 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = t * 16 + 4 * j + rs;  // sample number
                const uint32_t hsh = ((uint32_t)i * 2654435761u + (uint32_t)row * 40503u) * 2246822519u;
                const int pos = i * stratum + (int)__umulhi(hsh, (uint32_t)stratum);
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
    const float want = f + c.sel_margin * sqrtf(f) + 6.0f;
    const uint32_t target = want < 1.0f ? 1u : (want > (float)n_sample ? (uint32_t)n_sample : (uint32_t)want);
    uint32_t t_key = 0;
    if (target < (uint32_t)n_sample) {
        // the lower end of a narrow range of keys around the sample's target-th largest
        t_key = narrow(
            E, Cut{1u, 0xFFFFFFFFu, target, (uint32_t)n_sample}, 32 - kBinBits, 2u, [](uint32_t key, uint32_t) { return key; },
            [](uint32_t, uint32_t) { return true; }, sh).lo;
    }
    emit(t_key);
}

// Writes the pooled score of every row of (b, g) into sel[0 .. L): what the select unit falls
// back on when a row's candidate list is short of n entries or has overflowed.
template <int NH>
__device__ __forceinline__ void score_row_unit(const Common &c, const LayerDesc &p, int b, int g, int L, float *sel)
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

// The three sources of (ordered key, position) entries the select unit ranks.  for_each may
// also hand out "no entry": key 0, below every real key, and position kNoEntry; for_window
// hands out at least the entries of `count` positions from w0 on.  The visitors below fold
// everything that decides whether an entry counts into one flag, with bitwise operators, and
// guard a single LDS operation with it: short-circuit conditions made the compiler keep a lane
// mask per entry and condition, spill them, and branch several times per entry.
constexpr int kSelRegs = 40;     // entries one thread keeps in registers
constexpr int kSelHead = 8;      // and those of them that it asks for first
struct RegEntries {           // up to kThreads * kSelRegs list entries, loaded once: beside a streaming
    uint32_t key[kSelRegs], pos[kSelRegs];  // launch every pass over memory costs a microsecond or two
    int tid;
    int left;                 // entries, uniform: whole groups of eight registers beyond them are skipped
    unsigned long long head[kSelHead];
    // The first entries of a list with room for `cap`, asked for before its length is known.
    __device__ __forceinline__ void load_head(const unsigned long long *list, int cap, int tid_)
    {
        tid = tid_;
#pragma unroll
        for (int e = 0; e < kSelHead; ++e) {
            const int i = e * kThreads + tid;
            head[e] = gload(list + (i < cap ? i : cap - 1));
        }
    }
    __device__ __forceinline__ void load(const unsigned long long *list, int total)
    {
        left = total;
#pragma unroll
        for (int e = 0; e < kSelRegs; ++e) {
            if (e % 8 == 0 && e * kThreads >= left) break;
            const int i = e * kThreads + tid;
            const unsigned long long v = e < kSelHead ? head[e] : gload(list + (i < total ? i : total - 1));
            key[e] = i < total ? real_key((uint32_t)v) : 0u;
            pos[e] = i < total ? (uint32_t)(v >> 32) : kNoEntry;
        }
    }
    template <int kBatch = 8, typename F>
    __device__ __forceinline__ void for_each(F f) const
    {
#pragma unroll
        for (int e = 0; e < kSelRegs; ++e) {
            if (e % 8 == 0 && e * kThreads >= left) break;
            f(key[e], pos[e]);
        }
    }
    template <typename F>
    __device__ __forceinline__ void for_window(uint32_t, uint32_t, F f) const { for_each(f); }
};
struct ListEntries {          // a longer list, read from memory on every pass
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
    template <typename F>
    __device__ __forceinline__ void for_window(uint32_t, uint32_t, F f) const { for_each(f); }
};
struct RowEntries {           // every row of the sequence, from its recomputed scores
    const float *sel;
    int total;
    int tid;
    template <typename F>
    __device__ __forceinline__ void for_window(uint32_t w0, uint32_t count, F f) const
    {
        const int end = (int)(count < (uint32_t)total - w0 ? w0 + count : (uint32_t)total);
        for (int i0 = (int)w0 + tid; i0 < end; i0 += 8 * kThreads) {
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
    template <int kBatch = 8, typename F>
    __device__ __forceinline__ void for_each(F f) const { for_window(0u, (uint32_t)total, f); }
};

// Exact top-n of the `total` entries by key, ties to the lower position (Eq. 2), written to dst in
// ascending position order.  The entries may come in any order.  The range of keys is narrowed
// around the n-th largest until it holds at most kFewKeys entries, which are then ranked against
// one another by (key, position); equal keys that are more than that are cut at a position found
// the same way.  The chosen positions are marked in an LDS bitmap, 131072 positions at a
// time; a prefix sum over its words gives every chosen position its place, and each entry
// writes itself there.
//
// One workgroup, a chain of LDS passes and barriers: latency bounds it.  Counting by fixed digits,
// three passes always, with the positions read back by walking the bitmap's bits, took 15.7 us
// from the loads to the last store for any row (7500 candidates, k = 4096: see the figures at
// select_unit).
template <typename Entries, typename Pool>
__device__ __forceinline__ void select_from(const Entries &E, uint32_t floor_key, int total, int n, int L,
                                            int32_t *dst, SharedSelect &sh, Pool &pool)
{
    const int tid = E.tid;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    if (tid == 0) sh.n_few = 0;
    __syncthreads();  // (a list of kFewKeys entries or fewer goes straight to its use)
    // Rows that were sampled hold keys from their threshold up: the first level covers the eight
    // octaves above it, 256 bins each.  Others (short rows, blocks, rows ranked whole) start from
    // the range of all keys, four bins to the octave.
    const uint32_t lo = floor_key > 1u ? floor_key : 1u;
    const Cut cut = narrow(
        E, Cut{lo, 0xFFFFFFFFu, (uint32_t)n, (uint32_t)total}, lo >= 0x80000000u ? 26 - kBinBits : 32 - kBinBits,
        (uint32_t)kFewKeys, [](uint32_t key, uint32_t) { return key; }, [](uint32_t, uint32_t) { return true; }, sh);
    const bool all = cut.need == cut.count;  // everything in the range is chosen
    uint32_t my_few = kNoEntry;              // the position this thread ranked, if it is chosen
    uint32_t pos_cut = 0;                    // entries of equal keys are chosen up to this position
    bool by_pos = false;
    if (!all && cut.count <= (uint32_t)kFewKeys) {
        E.for_each([&](uint32_t key, uint32_t pos) {
            const bool in = key - cut.lo <= cut.hi - cut.lo;
            if (in) sh.few[atomicAdd(&sh.n_few, 1u)] = ((unsigned long long)key << 32) | (uint32_t)~pos;
        });
        __syncthreads();
        if ((uint32_t)tid < cut.count) {
            const unsigned long long mine = sh.few[tid];
            uint32_t before = 0;
            // (pairs, eight at a time: read one by one, each read waits for the one before it; what lies
            // past the last entry is not counted)
            for (uint32_t i0 = 0; i0 < cut.count; i0 += 16) {
                ulonglong2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = reinterpret_cast<const ulonglong2 *>(sh.few)[i0 / 2 + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    before += (uint32_t)((i0 + 2 * u < cut.count) & (v[u].x > mine));
                    before += (uint32_t)((i0 + 2 * u + 1 < cut.count) & (v[u].y > mine));
                }
            }
            if (before < cut.need) my_few = ~(uint32_t)mine;
        }
    } else if (!all) {
        by_pos = true;
        const Cut at = narrow(
            E, Cut{~(uint32_t)(L - 1), 0xFFFFFFFFu, cut.need, cut.count}, level_shift((uint32_t)(L - 1)), 0u, [](uint32_t, uint32_t pos) { return ~pos; },
            [&](uint32_t key, uint32_t) { return key == cut.lo; }, sh);
        pos_cut = ~at.lo;
    }
    constexpr uint32_t kWindow = kMapWords * 32u;
    uint32_t base = 0;  // positions chosen in earlier windows
    for (uint32_t w0 = 0; w0 < (uint32_t)L; w0 += kWindow) {
        const uint32_t span = (uint32_t)L - w0 < kWindow ? (uint32_t)L - w0 : kWindow;
        const int rounds = (int)(span + 32 * kThreads - 1) / (32 * kThreads);  // words of a wavefront's share / 64
        __syncthreads();
        for (int r = 0; r < rounds; ++r) sh.map[r * kThreads + tid] = make_uint2(0, 0);
        __syncthreads();
        E.for_window(w0, span, [&](uint32_t key, uint32_t pos) {
            const uint32_t rel = pos - w0;  // "no entry" lies outside every window
            const bool in = key - cut.lo <= cut.hi - cut.lo;
            const bool take = ((key > cut.hi) | (in & (all | (by_pos & (pos <= pos_cut))))) & (rel < span);
            atomicOr(&sh.map[take ? rel >> 5 : (uint32_t)(kMapWords + lane)].x, 1u << (rel & 31u));
        });
        if (my_few - w0 < span) atomicOr(&sh.map[(my_few - w0) >> 5].x, 1u << ((my_few - w0) & 31u));
        __syncthreads();
        // wavefront w counts words w * rounds * 64 .. of the window, then gives each its place
        const uint2 *share = sh.map + wave * rounds * 64 + lane;
        uint32_t cnt = 0;
        for (int r = 0; r < rounds; ++r) cnt += (uint32_t)__builtin_popcount(share[r * 64].x);
        cnt = wave_scan(cnt);
        if (lane == 63) sh.wave_tot[wave] = cnt;
        __syncthreads();
        uint32_t at0 = base, tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            at0 += w < wave ? sh.wave_tot[w] : 0u;
            tot += sh.wave_tot[w];
        }
        for (int r = 0; r < rounds; ++r) {
            const uint32_t c = (uint32_t)__builtin_popcount(share[r * 64].x);
            const uint32_t incl = wave_scan(c);
            sh.map[wave * rounds * 64 + lane + r * 64].y = at0 + incl - c;
            at0 += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        __syncthreads();
        // The positions are put in order in LDS, kStage at a time, and copied out with coalesced
        // write-through stores: the set is in device memory once the unit's stores have
        // completed, whoever reads it next (a gather piece of the same launch, on another XCD,
        // after an acquire).
        constexpr uint32_t kStage = (uint32_t)(sizeof(sh.samp) / sizeof(sh.samp[0])) - 64u;
        const uint32_t end = base + tot;
        for (uint32_t c0 = base; c0 < end; c0 += kStage) {
            E.for_window(w0, span, [&](uint32_t, uint32_t pos) {
                const uint32_t rel = pos - w0;
                const uint2 word = sh.map[rel < span ? rel >> 5 : 0];
                const uint32_t bit = 1u << (rel & 31u);
                const uint32_t at = word.y + (uint32_t)__builtin_popcount(word.x & (bit - 1u)) - c0;
                const bool put = (rel < span) & ((word.x & bit) != 0) & (at < kStage);
                sh.samp[put ? at : kStage + (uint32_t)lane] = pos;
            });
            __syncthreads();
            const uint32_t m = end - c0 < kStage ? end - c0 : kStage;
            for (uint32_t i = tid; i < m; i += kThreads) gstore_through(dst + c0 + i, (int32_t)sh.samp[i]);
            __syncthreads();
        }
        base = end;
    }
}

// A unit of one layer (Alg. 1, "C.append(k, v)"): the decoded token's key and value rows become
// row L_b - 1 of every KV head's cache.  16 lanes move one 256-byte row.
__device__ __forceinline__ void append_unit(const Common &c, const LayerDesc &p)
{
    const int ch = threadIdx.x & 15;
    const int n_rows = c.batch * c.n_kv_heads * 2;  // K rows, then V rows
    for (int r = threadIdx.x >> 4; r < n_rows; r += kThreads >> 4) {
        const int which = r / (c.batch * c.n_kv_heads);
        const int bg = r % (c.batch * c.n_kv_heads);
        const int b = bg / c.n_kv_heads, g = bg % c.n_kv_heads;
        const int L = clamp_len(c.lengths[b], c.max_len);
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

// In a histogram of probability mass per digit, finds the highest digit d at which the mass
// of the digits >= d reaches `need`; returns d and what is still needed inside d, or digit
// 0xFFFFFFFF when all the mass together does not reach it.
template <int kBins, typename Pool>
__device__ __forceinline__ void find_digit_mass(const unsigned long long *hist, unsigned long long need,
                                                Pool &pool, uint32_t &digit, unsigned long long &rest)
{
    constexpr int per = kBins / kThreads;
    unsigned long long mine[per], sum = 0;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        mine[j] = hist[kBins - 1 - (threadIdx.x * per + j)];  // bins taken from the top
        sum += mine[j];
    }
    unsigned long long total;
    unsigned long long above = block_scan64(sum, pool.scan64, total) - sum;
    if (threadIdx.x == 0) {
        pool.scan64[kWaves] = 0xFFFFFFFFull << 32;  // "not reached"
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < per; ++j) {
        if (above < need && need <= above + mine[j]) {
            // digit in the high word, the remaining need (< 2^41) cannot be packed with it: two words
            pool.scan64[kWaves] = (unsigned long long)(uint32_t)(kBins - 1 - (threadIdx.x * per + j)) << 32;
            pool.scan64[kWaves - 1] = need - above;
        }
        above += mine[j];
    }
    __syncthreads();
    digit = (uint32_t)(pool.scan64[kWaves] >> 32);
    rest = pool.scan64[kWaves - 1];
    __syncthreads();
}

// Entries the rule keeps, before the clamp to [1, n]: Threshold counts the entries whose
// probability exceeds the parameter; Top-p finds, digit by digit, the key at which the
// probability mass of the descending order reaches the parameter (all entries with that key
// have the same mass, so a division says how many of them are needed).  `lse` is the
// log-sum-exp of the pooled logits of the whole sequence.  The entries hold at least the n best
// positions, and a rule that would go beyond them is capped at n anyway.
template <typename Entries, typename Pool>
__device__ __forceinline__ int rule_keeps(const Common &c, const Entries &E, int n, float lse, SharedSelect &sh,
                                          Pool &pool)
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
        uint32_t prefix = 0, prefix_mask = 0;
        bool reached = true;
#pragma unroll
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
            const int n_bins = pass == 0 ? 4096 : 1024;
            const uint32_t digit_mask = (uint32_t)n_bins - 1u;
            for (int i = threadIdx.x; i < n_bins; i += kThreads) mh[i] = 0;
            __syncthreads();
            E.template for_each<8>([&](uint32_t key, uint32_t pos) {
                const bool in = (key != 0u) & ((key & prefix_mask) == prefix);
                if (in) atomicAdd(&mh[(key >> shift) & digit_mask], mass_of(key, lse));
            });
            __syncthreads();
            uint32_t digit;
            unsigned long long left;
            if (pass == 0)
                find_digit_mass<4096, Pool>(mh, need, pool, digit, left);
            else
                find_digit_mass<1024, Pool>(mh, need, pool, digit, left);
            if (digit == 0xFFFFFFFFu) {  // (uniform) not even all entries reach the mass: the cap decides
                reached = false;
                break;
            }
            prefix |= digit << shift;
            prefix_mask |= digit_mask << shift;
            need = left;
        }
        if (!reached) return n;
        const unsigned long long each = mass_of(prefix, lse);  // > 0: its digit held mass
        const uint32_t of_last = (uint32_t)((need + each - 1) / each);
        uint32_t mine = 0;
        E.template for_each<8>([&](uint32_t key, uint32_t pos) { mine += (uint32_t)(key > prefix); });
        uint32_t above;
        (void)block_scan(mine, pool.scan, above);
        want = above + of_last;
    }
    return want < 1u ? 1 : (want > (uint32_t)n ? n : (int)want);
}

// Log-sum-exp of the pooled logits of score row `row`: the pieces' states, merged.
template <typename Pool>
__device__ __forceinline__ float pooled_lse(const Common &c, const LayerDesc &p, int64_t row, int count,
                                            Pool &pool)
{
    const float *ml = p.part_pool + row * (2 * (int64_t)c.part_stride);
    float m_loc = kMinusBig;
    for (int s = threadIdx.x; s < count; s += kThreads) m_loc = fmaxf(m_loc, gload(ml + 2 * s));
    const float M = block_max(m_loc, pool.fred);
    float l_loc = 0.0f;
    for (int s = threadIdx.x; s < count; s += kThreads)
        l_loc = fmaf(fast_exp2((gload(ml + 2 * s) - M) * kLog2e), gload(ml + 2 * s + 1), l_loc);
    const float l = block_sum(l_loc, pool.fred);
    return M + __logf(l);
}

// The set of a KV head (b, g) whose group holds no retrieval head is handed on unchanged
// (Sec. 3.1): a verbatim copy.
__device__ __forceinline__ void copy_set_unit(const Common &c, const LayerDesc &p, int b, int g)
{
    const int64_t bg = (int64_t)b * c.n_kv_heads + g;
    int32_t *dst = p.idx_out + bg * c.k;
    const int32_t *src = p.idx_src[g] + bg * c.k;
    for (int i = threadIdx.x; i < c.k; i += kThreads) gstore_through(dst + i, gload(src + i));
}

// S unit of KV head (b, g), whose group holds a retrieval head: the set the next layer's
// sparse heads of the group inherit.  PROB: the build that knows the probability rules (their
// 64-bit mass arithmetic over register-resident entries would cost the plain build registers).
template <bool PROB, typename Pool>
__device__ __forceinline__ void select_unit(const Common &c, const LayerDesc &p, int b, int g,
                                            SharedSelect &sh, Pool &pool)
{
    const int64_t bg = (int64_t)b * c.n_kv_heads + g;
    int32_t *dst = p.idx_out + bg * c.k;
    const int rgi = p.rindex[g];
    const int len = pool.len[b];  // staged by the kernel, clamped
    const int L = units_of(c, len);  // what is ranked: positions, or blocks of positions
    const int n = budget_of(c, L);
    const bool by_prob = PROB && c.prob_rule != 0;
    if (n == L && !by_prob) {  // everything is selected
        for (int i = threadIdx.x; i < c.k; i += kThreads) gstore_through(dst + i, (int32_t)(i < L ? i : -1));
        if (threadIdx.x == 0 && c.block_shift == 0 && rgi != 0xFF)
            gstore(p.list_count + ((int64_t)b * p.n_rgroups + rgi), (int32_t)0);  // (nothing was collected; see below)
        return;
    }
    const int64_t row = (int64_t)b * p.n_rgroups + rgi;
    const unsigned long long *list = p.list + row * (int64_t)c.list_row;
    RegEntries E;
    E.load_head(list, c.list_row, fresh_tid());
    // block-granular: the streaming left every block's score at its place in the list
    const int total = c.block_shift ? L : gload(p.list_count + row);
    const uint32_t floor_key = c.block_shift ? 0u : gload(p.thr + row);  // no entry lies below it
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
    if (total >= n && total <= kThreads * kSelRegs && total <= c.list_row) {
        E.load(list, total);
        if (PROB && by_prob) keep = rule_keeps(c, E, n, lse, sh, pool);
        select_from(E, floor_key, total, keep, L, dst, sh, pool);
    } else if (total >= n && total <= c.list_row) {
        const ListEntries M{list, total, fresh_tid()};
        if (PROB && by_prob) keep = rule_keeps(c, M, n, lse, sh, pool);
        select_from(M, floor_key, total, keep, L, dst, sh, pool);
    } else {
        // too few candidates reached the threshold, or too many for the list: rank the row
        // (token-granular only: a block list is always complete)
        if (threadIdx.x == 0) atomicAdd(c.stats + (total < n ? 0 : 1), 1u);
        float *sel = p.sel + row * c.sel_stride;
        switch (__builtin_popcount(p.rmask[g] & ((1u << c.group) - 1u))) {
        case 1: score_row_unit<1>(c, p, b, g, len, sel); break;
        case 2: score_row_unit<2>(c, p, b, g, len, sel); break;
        case 3: score_row_unit<3>(c, p, b, g, len, sel); break;
        default: score_row_unit<4>(c, p, b, g, len, sel); break;
        }
        __threadfence();
        __syncthreads();  // the scores are read back by other threads of the workgroup
        const RowEntries M{sel, len, fresh_tid()};
        if (PROB && by_prob) keep = rule_keeps(c, M, n, lse, sh, pool);
        select_from(M, 0u, len, keep, L, dst, sh, pool);
    }
    for (int i = keep + threadIdx.x; i < c.k; i += kThreads) gstore_through(dst + i, (int32_t)-1);
    if (clear_count && threadIdx.x == 0) gstore(p.list_count + row, (int32_t)0);
}


}  // namespace
}  // namespace lychee
