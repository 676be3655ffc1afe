// Device-side building blocks of the work-unit kernels (included by lychee_units.hip and lychee_layer.hip):
// the LDS layout of a workgroup, global-memory accessors, the bf16 dot product, wavefront and
// workgroup reductions and scans.
#pragma once
#include "lychee_internal.h"

namespace lychee {
namespace {

// ------------------------------------------------------------------------------ LDS layout
struct SharedAttn {
    int32_t idx_s[kIdxChunk];
    float red_o[kWaves * kMaxGroup * kHeadDim];
    float red_ml[kWaves * kMaxGroup * 2];
    float pool_ml[kWaves * 2];
    union {
        unsigned long long cand[kWaves][kCandBuf];  // per wavefront: candidates not yet flushed
        uint32_t keys[kKeyBuf];                     // or: the ordered keys of the piece's last kKeyBuf rows,
    };                                              //     filtered once the row's threshold is known
    int32_t cand_left[kWaves];                  // what each wavefront still holds when a piece ends
    int32_t cand_base;                          // where the workgroup's last candidates go
};
constexpr int kBinBits = 11;               // a level of the select splits its range of keys into 2048 bins
constexpr int kBins = 1 << kBinBits;
constexpr int kLastKeys = 64;              // so few entries are ranked against one another, one per thread
constexpr int kMapWords = 4096;            // words of the position bitmap: a window of 131072 positions
constexpr int kStage = 8192;               // positions put in order in LDS at a time
// (hist, bits and stage end in a word per lane where entries that do not count go: a store to a word
// of its own costs less than a branch around the store for every entry)
struct SharedSelect {
    union {
        uint32_t hist[kBins + 64];         // entries per bin
        uint32_t bits[kMapWords + 64];     // ordered write: the chosen positions of a window
    };
    uint16_t before[kMapWords];            //   positions chosen before a word, within its wavefront's share
    union {
        uint32_t samp[kSampleTilesMax * 16];  // ordered keys of the threshold sample
        uint32_t stage[kStage + 64];          // staged positions
        unsigned long long mass[kBins];       // probability mass per bin (Top-p)
    };
    __align__(16) unsigned long long last[kLastKeys];  // (key, ~position) of the entries around the last place
    unsigned long long cutoff;
    uint32_t n_last;
    uint32_t wave_tot[kWaves];
    uint32_t found[3];
};
struct SharedCombine {
    float w[kMaxGroup][kMaxWg];   // per head: a slot's running maximum, then its weight
    float ls[kMaxGroup][kMaxWg];  // and its sum of exp
    float red[(kThreads / 32) * kHeadDim];
    float l[kMaxGroup];
};
union SharedUnit {
    SharedSelect sel;
    SharedCombine comb;
};
struct SharedPool {
    int32_t ipre[kMaxItems + 1];         // first pooled block of every (layer, sequence) item
    int32_t len[kMaxBatch];
    uint32_t scan[kWaves + 1];
    unsigned long long scan64[kWaves + 1];
};
struct SharedSmall {
    int32_t upre[4][kMaxLayers + 1];     // first small unit of every layer, per unit kind
    int32_t len[kMaxBatch];
    uint32_t scan[kWaves + 1];
    unsigned long long scan64[kWaves + 1];
    float fred[kWaves + 1];
};

// ------------------------------------------------------------------------------ primitives
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                           __builtin_bit_cast(bf16x2_t, b), acc, false);
}

template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float x)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xF, 0xF, false));
}

// (lanes without a source lane, or outside the row mask, get 0)
template <int kCtrl, int kRowMask = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRowMask, 0xF, false);
}

// Sum over the 16 lanes of a DPP row; every lane of the row ends with the same bits.
__device__ __forceinline__ float row16_sum(float x)
{
    x += dpp_f32<0xB1>(x);   // quad_perm [1,0,3,2]  : lane ^ 1
    x += dpp_f32<0x4E>(x);   // quad_perm [2,3,0,1]  : lane ^ 2
    x += dpp_f32<0x141>(x);  // row_half_mirror      : the other quad of the 8-lane half
    x += dpp_f32<0x140>(x);  // row_mirror           : the other half of the 16-lane row
    return x;
}

// x + (x of the lane 16 lanes away) and the same for 32 lanes, as x + __shfl_xor(x, 16 / 32) give
// them (bit for bit: one addition of the same two numbers), without the LDS crossbar: gfx950's row
// swaps are plain vector instructions.  v_permlane16_swap(a, b) exchanges the odd rows of 16 lanes of a
// with the even rows of b, v_permlane32_swap(a, b) the upper half of a with the lower half of b; with
// a = b = x the two results hold the even (lower) parts of x everywhere and the odd (upper) parts
// everywhere.
__device__ __forceinline__ float sum_rows16(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float sum_halves32(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
// The same sums of several numbers at once: a's over each pair of rows in the even rows, b's in the odd ones; then,
// of two such, a's (four rows), b's, c's and d's in rows 0 to 3.  One swap and one addition for two numbers
// instead of a copy, a swap and an addition for each.
__device__ __forceinline__ float sum_rows16_pair(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float sum_halves32_pair(float ab, float cd)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, ab), __builtin_bit_cast(uint32_t, cd), false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float max_rows16(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float max_halves32(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// Smallest and largest of a wavefront's 64 values, in every lane.
__device__ __forceinline__ uint32_t wave_min(uint32_t x)
{
    x = min(x, dpp_u32<0xB1>(x));
    x = min(x, dpp_u32<0x4E>(x));
    x = min(x, dpp_u32<0x141>(x));
    x = min(x, dpp_u32<0x140>(x));
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = min((uint32_t)r[0], (uint32_t)r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return min((uint32_t)h[0], (uint32_t)h[1]);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) { return ~wave_min(~x); }

// Inclusive prefix sum over the 64 lanes of a wavefront, by row shifts and row broadcasts (plain
// vector instructions; six exchanges through the LDS crossbar take about ten times as long).
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    x += dpp_u32<0x111>(x);  // row_shr 1, 2, 4, 8: prefix sums inside every row of 16 lanes
    x += dpp_u32<0x112>(x);
    x += dpp_u32<0x114>(x);
    x += dpp_u32<0x118>(x);
    x += dpp_u32<0x142, 0xA>(x);  // row_bcast15: the row before, into rows 1 and 3
    x += dpp_u32<0x143, 0xC>(x);  // row_bcast31: the first half, into rows 2 and 3
    return x;
}

__device__ __forceinline__ float wave_max_f(float x)
{
    x = fmaxf(x, dpp_f32<0xB1>(x));
    x = fmaxf(x, dpp_f32<0x4E>(x));
    x = fmaxf(x, dpp_f32<0x141>(x));
    x = fmaxf(x, dpp_f32<0x140>(x));
    return max_halves32(max_rows16(x));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __builtin_bit_cast(float, u & 0xFFFF0000u); }

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x)
{
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The kernel arguments are read through a pointer of their own address space (scalar loads, from the scalar
// cache after the first), and every unit of work starts from a pointer that is opaque to the compiler
// (arg_of).  Read through the kernel's parameter, a few dozen of the fields and what derives from them were
// loaded once at the top, kept across every unit and spilled: 220 scalar registers in lanes of vector
// registers, whose reads and writes made up a third of the instructions between two units.
#define LYCHEE_CONSTANT __attribute__((address_space(4)))
typedef const LYCHEE_CONSTANT Common ArgCommon;
template <typename T>
__device__ __forceinline__ const LYCHEE_CONSTANT T *arg_of()
{
    const LYCHEE_CONSTANT T *p = (const LYCHEE_CONSTANT T *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// Every buffer the units touch is device global memory, but most pointers reach the kernel
// through the descriptor table, where the compiler can no longer see that.  Generic-address
// ("flat") accesses make it wait for *all* outstanding loads before each use, which breaks the
// load pipeline of the streaming loop; so every access goes through these casts.
#define LYCHEE_GLOBAL __attribute__((address_space(1)))
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ T gload(const T *p)
{
    return *(const LYCHEE_GLOBAL T *)p;
}
template <typename T>
__device__ __forceinline__ void gstore(T *p, T v)
{
    *(LYCHEE_GLOBAL T *)p = v;
}
// Write-through store: the value goes through the XCD's L2 to device memory, and the store counts
// as outstanding (vmcnt) until it is there.  A workgroup on another XCD that learns, through an
// agent-scope atomic issued after wait_stores(), that the data exists reads it after an acquire
// fence, or past the caches (gload_through).  This is what lets a workgroup hand a partial result to another one in the same launch
// without the agent-scope release fence, whose write-back of the whole L2 costs tens of
// microseconds when hundreds of workgroups execute it.
__device__ __forceinline__ void gstore_through(float *p, float v)
{
    __hip_atomic_store((LYCHEE_GLOBAL float *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore_through(int32_t *p, int32_t v)
{
    __hip_atomic_store((LYCHEE_GLOBAL int32_t *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore_through(uint32_t *p, uint32_t v)
{
    __hip_atomic_store((LYCHEE_GLOBAL uint32_t *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore_through(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store((LYCHEE_GLOBAL unsigned long long *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore_through(float *p, float2 v)  // (8-byte aligned)
{
    gstore_through(reinterpret_cast<unsigned long long *>(p),
                   (unsigned long long)__builtin_bit_cast(uint32_t, v.x) | ((unsigned long long)__builtin_bit_cast(uint32_t, v.y) << 32));
}
__device__ __forceinline__ void gstore_f2(float *p, float2 v) { *(LYCHEE_GLOBAL f32x2_t *)p = f32x2_t{v.x, v.y}; }
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Reads what another workgroup of the launch has written through, without an acquire fence (whose invalidation of the
// caches takes 0.2 us and hits the whole XCD).
__device__ __forceinline__ int32_t gload_through(const int32_t *p)
{
    return __hip_atomic_load((const LYCHEE_GLOBAL int32_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float4 gload_f4(const float *p)
{
    const f32x4_t r = *(const LYCHEE_GLOBAL f32x4_t *)p;
    return make_float4(r.x, r.y, r.z, r.w);
}
__device__ __forceinline__ float2 gload_f2(const float *p)
{
    const f32x2_t r = *(const LYCHEE_GLOBAL f32x2_t *)p;
    return make_float2(r.x, r.y);
}
__device__ __forceinline__ uint4 gload_u4(const void *p)
{
    const u32x4_t r = *(const LYCHEE_GLOBAL u32x4_t *)p;
    return make_uint4(r.x, r.y, r.z, r.w);
}

// 16-byte streaming load: cache rows are read once per step and never again.
__device__ __forceinline__ uint4 load_stream16(const uint16_t *p)
{
    const u32x4_t r = __builtin_nontemporal_load((const LYCHEE_GLOBAL u32x4_t *)p);
    return make_uint4(r.x, r.y, r.z, r.w);
}

__device__ __forceinline__ uint32_t ordered_key(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ int clamp_len(int L, int max_len) { return L < 1 ? 1 : (L > max_len ? max_len : L); }

// Selectable units of a sequence of L rows: its positions, or its blocks of 64 positions
// (the last one may be short) in the block-granular variant (App. C).
__device__ __forceinline__ int units_of(ArgCommon &c, int L)
{
    return (L + (1 << c.block_shift) - 1) >> c.block_shift;
}

// Units selected for a sequence of L units: Eq. 2's fixed budget, min(k, L), or under the
// Ratio rule (Sec. 4.4.1: a budget proportional to the sequence length) the rounded-up share
// keep_ppm / 10^6 of L, at least 1 and at most the fixed budget.
__device__ __forceinline__ int budget_of(ArgCommon &c, int L)
{
    int n = c.k < L ? c.k : L;
    if (c.keep_ppm > 0) {
        long long r = ((long long)L * c.keep_ppm + 999999) / 1000000;
        r = r < 1 ? 1 : r;
        n = r < n ? (int)r : n;
    }
    return n;
}

// A score row of L positions of which n are selected whose threshold follows from the sizes: everything
// is selected, or every row is a candidate.
__device__ __forceinline__ bool needs_no_sample(int n, int L)
{
    return n == L || L <= kDirectLen || 2 * (int64_t)n >= L;
}

// Fields of a layer descriptor staged in LDS as 32-bit words.  The values are the same in
// every lane; reading them back through readfirstlane tells the compiler so (scalar registers,
// scalar address arithmetic in the streaming loop).
constexpr int kDescWords = (int)(sizeof(LayerDesc) / 4);
static_assert(sizeof(LayerDesc) % 4 == 0 && kDescWords <= kThreads, "one word per thread");

// The thread's index, opaque to the compiler where it is taken: what is computed from it stays inside
// the unit that asks (left visible, every unit's per-thread LDS and list addresses were computed
// once, at the top of the kernel, kept across everything and spilled).
__device__ __forceinline__ int fresh_tid()
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return (int)t;
}

// A value that is the same in every lane, said so to the compiler (a scalar register).
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T *uni(T *p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T *>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
                                 ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32));
}
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ uint32_t desc_u32(const uint32_t *dw, size_t off)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)dw[off / 4]);
}
__device__ __forceinline__ uint32_t desc_u8(const uint32_t *dw, size_t off)
{
    return (desc_u32(dw, off & ~(size_t)3) >> (8 * (off & 3))) & 0xFFu;
}
template <typename T>
__device__ __forceinline__ T *desc_ptr(const uint32_t *dw, size_t off)
{
    const uint64_t lo = desc_u32(dw, off), hi = desc_u32(dw, off + 4);
    return reinterpret_cast<T *>(lo | (hi << 32));
}

// a / b (quot_by).  A workgroup divides a dozen times before its first load; the compiler's 32-bit division is about
// 25 dependent instructions.
__device__ __forceinline__ int quot(int a, int b)
{
    return quot_by(a, b, __builtin_amdgcn_rcpf((float)b), [](uint32_t v) { return v; });
}
// The same of values that are the same in every lane: scalar arithmetic but for the product.
__device__ __forceinline__ int quot_uni(int a, int b)
{
    return quot_by(a, b, __builtin_amdgcn_rcpf((float)b), [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); });
}

// Largest i in [0, n) with pre[i] <= x, for a non-decreasing pre[0..n] with pre[0] <= x < pre[n].
__device__ __forceinline__ int find_item(const int32_t *pre, int n, int x)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Rows a sparse KV head gathers for a sequence of L cache rows (set entries that are -1 or
// name rows past L are skipped one by one), and how many of them make one pooled block.
__device__ __forceinline__ int gather_rows(ArgCommon &c, int L)
{
    const int units = units_of(c, L);
    return (c.k < units ? c.k : units) << c.block_shift;
}
__device__ __forceinline__ int gather_block(ArgCommon &c)
{
    return c.block_shift ? (1 << c.block_shift) : c.g_block_rows;  // whole blocks stream like R rows
}

// Inclusive prefix sum over the 256 threads of the workgroup; `total` = sum of all.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wave_tot, uint32_t &total)
{
    const int tid = fresh_tid();
    const int wave = tid >> 6;
    const uint32_t x = wave_scan(v);
    __syncthreads();  // wave_tot may still be read by the previous call
    if ((tid & 63) == 63) wave_tot[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t t = wave_tot[w];
        before += (w < wave) ? t : 0u;
        all += t;
    }
    total = all;
    return x + before;
}

// The same for two 32-bit counts packed in 64 bits (neither may overflow).
__device__ __forceinline__ unsigned long long block_scan_pair(unsigned long long v, unsigned long long *wave_tot,
                                                              unsigned long long &total)
{
    const int tid = fresh_tid();
    const int wave = tid >> 6;
    const unsigned long long x = (unsigned long long)wave_scan((uint32_t)v) |
                                 ((unsigned long long)wave_scan((uint32_t)(v >> 32)) << 32);
    __syncthreads();
    if ((tid & 63) == 63) wave_tot[wave] = x;
    __syncthreads();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const unsigned long long t = wave_tot[w];
        before += (w < wave) ? t : 0ull;
        all += t;
    }
    total = all;
    return x + before;
}

// The same for 64-bit numbers.
__device__ __forceinline__ unsigned long long block_scan64(unsigned long long v, unsigned long long *wave_tot,
                                                           unsigned long long &total)
{
    const int tid = fresh_tid();
    const int lane = tid & 63;
    const int wave = tid >> 6;
    unsigned long long x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    __syncthreads();
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const unsigned long long t = wave_tot[w];
        before += (w < wave) ? t : 0ull;
        all += t;
    }
    total = all;
    return x + before;
}

__device__ __forceinline__ float block_max(float v, float *scratch)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d));
    __syncthreads();
    if ((fresh_tid() & 63) == 0) scratch[fresh_tid() >> 6] = v;
    __syncthreads();
    float r = scratch[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r = fmaxf(r, scratch[w]);
    return r;
}

__device__ __forceinline__ float block_sum(float v, float *scratch)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    __syncthreads();
    if ((fresh_tid() & 63) == 0) scratch[fresh_tid() >> 6] = v;
    __syncthreads();
    float r = scratch[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r += scratch[w];
    return r;
}



}  // namespace
}  // namespace lychee
