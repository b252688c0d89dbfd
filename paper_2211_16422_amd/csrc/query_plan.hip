// Query planning around the one-shot search kernels: candidate windows,
// query order, tiles, and after them the narrow tiles and the results.
//
// Queries are ordered by the middle of their window (first row + last row),
// which is their (charge, precursor m/z) order (either end alone is not: the
// open windows of every precursor near a charge's edge share it), and cut
// into tiles; a tile's candidates are
// the union of its windows. Only the tiles' shape depends on the order
// (results are merged per query by (distance, library index)), so the order
// inside a bucket of neighbouring rows is left open and a counting sort over
// kBuckets equal runs of library rows does: one atomic per query, whose
// return value is also the query's place in its bucket. Queries without
// candidates go last (one atomic per wave: a cascade's open stage can have
// tens of thousands of them). Up to kSmallPlan queries, one workgroup does
// everything in one launch with a bitonic sort in LDS.
//
// A stable radix sort of (charge, m/z) keys took 27 launches and 100 us (64
// queries) to 230 us (100,000) here; this takes one or five.
#include <algorithm>

#include "internal.h"
#include "window_search.h"

namespace homs {
namespace {

constexpr int kThreads = 256;
constexpr int kBuckets = 16384;
constexpr int kSmallThreads = 1024;
constexpr int kSmallPlan = 512;   // queries of the one-workgroup plan

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kThreads - 1) / kThreads); }

struct PlanArgs {
    int64_t nq;
    const double* q_pmz;
    const int8_t* q_charge;
    bool use_charge;
    int32_t kind;
    double value;
    const double* lib_pmz;
    const uint32_t* charge_first;
    int64_t nlib;
    int tile;
    uint32_t words;
    const uint32_t* q_hv;  // rows of the fp4 query constants (NULL: not wanted)
    QueryPlan w;
};

__device__ __forceinline__ void query_window(const PlanArgs& a, int64_t q, int64_t* lo, int64_t* hi)
{
    const double pmz = a.q_pmz[q];
    const double tol = tolerance_da(pmz, a.kind, a.value);
    int64_t r_lo, r_hi;
    charge_run(a.charge_first, a.use_charge ? a.q_charge[q] : (int8_t)0, &r_lo, &r_hi);
    window_bounds(a.lib_pmz, r_lo, r_hi, __dsub_rn(pmz, tol), __dadd_rn(pmz, tol), lo, hi);
}

// fp4 constant of query q by one wave (search_mfma.hip states the form)
__device__ __forceinline__ void query_offset(const PlanArgs& a, int64_t q)
{
    const int l = threadIdx.x & 63;
    const uint32_t* row = a.q_hv + (size_t)q * a.words;
    int s = 0;
    for (uint32_t i = l; i < a.words; i += 64) s += fp4_word_weight(row[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (l == 0) a.w.qoff[q] = s + (int)(21 * a.words * 8);  // 21D/4
}

// one wave: the union of tile t's windows, the sum of their sizes and the
// largest; at(i) is the query in place i of the order
template <class At>
__device__ __forceinline__ void tile_shape(const PlanArgs& a, int64_t t, At at)
{
    const int l = threadIdx.x & 63;
    int64_t mn = INT64_MAX, mx = 0, sum = 0, big = 0;
    const int64_t end = min((t + 1) * (int64_t)a.tile, a.nq);
    for (int64_t i = t * a.tile + l; i < end; i += 64) {
        const uint32_t q = at(i);
        const int64_t lo = a.w.lo[q], hi = a.w.hi[q];
        if (hi > lo) {
            mn = min(mn, lo);
            mx = max(mx, hi);
            sum += hi - lo;
            big = max(big, hi - lo);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, (int64_t)__shfl_xor((long long)mn, o));
        mx = max(mx, (int64_t)__shfl_xor((long long)mx, o));
        sum += (int64_t)__shfl_xor((long long)sum, o);
        big = max(big, (int64_t)__shfl_xor((long long)big, o));
    }
    if (l == 0) {
        a.w.tile_lo[t] = mx == 0 ? 0 : mn;
        a.w.tile_hi[t] = mx;
        a.w.tile_sum[t] = sum;
        a.w.tile_max[t] = big;
    }
}

// ---- up to kSmallPlan queries: workgroup 0 plans, the others compute the
// fp4 query constants (kSmallThreads / 64 queries each)
__global__ __launch_bounds__(kSmallThreads) void plan_small_kernel(PlanArgs a)
{
    __shared__ uint64_t s_key[kSmallPlan];
    if (blockIdx.x > 0) {
        const int64_t q = (int64_t)(blockIdx.x - 1) * (kSmallThreads / 64) + (threadIdx.x >> 6);
        if (q < a.nq) query_offset(a, q);
        return;
    }
    const int n = (int)a.nq;
    int np = 64;
    while (np < n) np <<= 1;
    for (int i = threadIdx.x; i < np; i += kSmallThreads) {
        uint64_t key = ~0ull;
        if (i < n) {
            int64_t lo, hi;
            query_window(a, i, &lo, &hi);
            a.w.lo[i] = lo;
            a.w.hi[i] = hi;
            a.w.keys[i] = ~0ull;
            key = ((uint64_t)(hi > lo ? (uint32_t)(lo + hi) : 0xFFFFFFFFu) << 32) | (uint32_t)i;
        }
        s_key[i] = key;
    }
    for (int size = 2; size <= np; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < np / 2; t += kSmallThreads) {
                const int i = 2 * t - (t & (stride - 1)), j = i + stride;
                const uint64_t x = s_key[i], y = s_key[j];
                if ((x > y) == ((i & size) == 0)) {
                    s_key[i] = y;
                    s_key[j] = x;
                }
            }
        }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kSmallThreads) a.w.qperm[i] = (uint32_t)s_key[i];
    for (int t = threadIdx.x >> 6; t * a.tile < n; t += kSmallThreads / 64)
        tile_shape(a, t, [&](int64_t i) { return (uint32_t)s_key[i]; });
}

// ---- any number of queries, five launches

// buckets cleared, fp4 query constants (one wave per query)
__global__ __launch_bounds__(kThreads) void plan_init_kernel(PlanArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t <= kBuckets) a.w.hist[t] = 0;
    if (a.q_hv && t / 64 < a.nq) query_offset(a, t / 64);
}

// one-wave workgroups: the searches' scattered loads spread over all the
// compute units
__global__ __launch_bounds__(64) void plan_bounds_kernel(PlanArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const bool in = q < a.nq;
    int64_t lo = 0, hi = 0;
    if (in) {
        query_window(a, q, &lo, &hi);
        a.w.lo[q] = lo;
        a.w.hi[q] = hi;
        a.w.keys[q] = ~0ull;
    }
    // queries without candidates: the wave's first takes places for all
    const uint64_t none = __ballot(in && hi <= lo);
    const int l = threadIdx.x & 63;
    if (none) {
        const int first = __ffsll((unsigned long long)none) - 1;
        uint32_t base = 0;
        if (l == first) base = atomicAdd(a.w.hist + kBuckets, (uint32_t)__popcll(none));
        base = __shfl(base, first);
        if ((none >> l) & 1) {
            a.w.bucket[q] = kBuckets;
            a.w.place[q] = base + (uint32_t)__popcll(none & ((1ull << l) - 1));
        }
    }
    if (in && hi > lo) {
        const uint32_t b = (uint32_t)((uint64_t)(lo + hi) * kBuckets / (2 * (uint64_t)a.nlib + 1));
        a.w.bucket[q] = b;
        a.w.place[q] = atomicAdd(a.w.hist + b, 1u);
    }
}

// one workgroup: bucket starts (exclusive prefix sums)
__global__ __launch_bounds__(kSmallThreads) void plan_starts_kernel(PlanArgs a)
{
    constexpr int kPer = kBuckets / kSmallThreads;
    __shared__ uint32_t s_wave[kSmallThreads / 64];
    const int t = threadIdx.x, l = t & 63;
    uint4 v[kPer / 4];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
        v[i] = ((const uint4*)a.w.hist)[t * (kPer / 4) + i];
        sum += v[i].x + v[i].y + v[i].z + v[i].w;
    }
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (l >= o) inc += y;
    }
    if (l == 63) s_wave[t >> 6] = inc;
    __syncthreads();
    uint32_t run = inc - sum, total = 0;
    for (int i = 0; i < kSmallThreads / 64; ++i) {
        if (i < (t >> 6)) run += s_wave[i];
        total += s_wave[i];
    }
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
        uint4 o;
        o.x = run;
        o.y = o.x + v[i].x;
        o.z = o.y + v[i].y;
        o.w = o.z + v[i].z;
        run = o.w + v[i].w;
        ((uint4*)a.w.hist)[t * (kPer / 4) + i] = o;
    }
    if (t == 0) a.w.hist[kBuckets] = total;  // queries without candidates follow
}

__global__ __launch_bounds__(kThreads) void plan_order_kernel(PlanArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (q < a.nq) a.w.qperm[a.w.hist[a.w.bucket[q]] + a.w.place[q]] = (uint32_t)q;
}

__global__ __launch_bounds__(kThreads) void plan_tiles_kernel(PlanArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (t * a.tile < a.nq) tile_shape(a, t, [&](int64_t i) { return a.w.qperm[i]; });
}

}  // namespace

namespace {
size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
}  // namespace

size_t query_plan_bytes(int64_t nq, int tile)
{
    const int64_t nt = (nq + tile - 1) / tile;
    return 3 * al(nq * 8) + 4 * al(nq * 4) + 4 * al(nt * 8) + al((kBuckets + 1) * 4);
}

QueryPlan query_plan_carve(void* base, int64_t nq, int tile)
{
    const int64_t nt = (nq + tile - 1) / tile;
    char* p = (char*)base;
    auto take = [&](size_t bytes) {
        void* r = p;
        p += al(bytes);
        return r;
    };
    QueryPlan w{};
    w.lo = (int64_t*)take(nq * 8);
    w.hi = (int64_t*)take(nq * 8);
    w.keys = (uint64_t*)take(nq * 8);
    w.qperm = (uint32_t*)take(nq * 4);
    w.qoff = (int32_t*)take(nq * 4);
    w.bucket = (uint32_t*)take(nq * 4);
    w.place = (uint32_t*)take(nq * 4);
    w.tile_lo = (int64_t*)take(nt * 8);
    w.tile_hi = (int64_t*)take(nt * 8);
    w.tile_sum = (int64_t*)take(nt * 8);
    w.tile_max = (int64_t*)take(nt * 8);
    w.hist = (uint32_t*)take((kBuckets + 1) * 4);
    return w;
}

hipError_t launch_query_plan(const homs_ctx* c, int64_t nq, const double* q_pmz,
                             const int8_t* q_charge, int32_t kind, double value,
                             const uint32_t* q_hv, int tile, const QueryPlan& w, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    const PlanArgs a{nq,         q_pmz, q_charge, c->p.charge_match != 0, kind, value, c->lib.pmz,
                     c->lib.charge_first, c->lib.n, tile, c->words, q_hv, w};
    if (nq <= kSmallPlan) {
        const int64_t per = kSmallThreads / 64;
        plan_small_kernel<<<(uint32_t)(1 + (q_hv ? (nq + per - 1) / per : 0)), kSmallThreads, 0,
                            s>>>(a);
        return hipGetLastError();
    }
    plan_init_kernel<<<blocks_for(std::max<int64_t>(kBuckets + 1, q_hv ? nq * 64 : 0)), kThreads,
                       0, s>>>(a);
    plan_bounds_kernel<<<(uint32_t)((nq + 63) / 64), 64, 0, s>>>(a);
    plan_starts_kernel<<<1, kSmallThreads, 0, s>>>(a);
    plan_order_kernel<<<blocks_for(nq), kThreads, 0, s>>>(a);
    const int64_t nt = (nq + tile - 1) / tile;
    plan_tiles_kernel<<<(uint32_t)((nt + 3) / 4), kThreads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace homs
