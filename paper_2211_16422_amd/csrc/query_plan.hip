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
constexpr int kSums = 64, kSumStride = 8;  // the call's pairs in parts, a cache line each

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kThreads - 1) / kThreads); }

// Narrow tiles. A tile kernel multiplies a tile's whole union of windows with
// all its queries; where every window is a small part of the union (standard
// searches of a few dozen candidates), finish_kernel scans each window on its
// own instead, one wave per two queries, with XOR and population counts (the
// same distances). A tile is narrow when ratio x the sum of its windows is at
// most union x tile, and its windows leave the waves evenly loaded and are not
// too many pairs.
// The ratios are where both ways took the same time (D = 8,192): fp4, 256-query
// tiles: 100,000 queries over 2M rows, scan 1.76 ms at +-50 ppm against 2.25 ms
// of tiles at 75 and 100 (windows of 1/36 of the union at the crossing);
// fp8 there 6.0 / 10.8 ms at 200 / 400 ppm against 5.1 / 5.3; small tiles:
// 2,000 queries, scan 0.43 / 1.55 ms at 200 / 1,000 ppm against 0.70. At D = 512
// 9,000 queries over 2,000,000 rows cross at windows of 1/30 of the union (fp4:
// 500 rows 0.16 ms by scan and 0.40 by tiles, 2,400 rows 0.72 and 0.52), at D =
// 32,768 over 300,000 rows fp8 at more than 1/18 (500 rows 3.0 and 2.1 ms).
// Popcount crosses at the shares and numbers of pairs below; windows above 1/3 of
// the union are never the faster by scan (D = 8,192, 100,000 queries over 400,000
// rows: 400 rows 4.8 ms by scan and 2.8 by tiles).
int64_t narrow_ratio10(int32_t engine, int tile)  // in tenths
{
    if (engine == HOMS_ENGINE_POPCOUNT) return 30;
    if (engine == HOMS_ENGINE_MFMA_F4) return tile == 256 ? 360 : 920;
    return tile == 256 ? 180 : 480;
}
// Largest window of a narrow tile: few queries are few waves, which a tile
// kernel's chunks would beat on long windows (a wave scans its two queries of
// 1,800 rows of D = 8,192 for 0.9 ms).
int64_t narrow_max(int64_t nq) { return std::min<int64_t>(2048, 64 + nq / 4); }
// Most pairs of a call whose tiles may be narrow. 256-query matrix-core tiles take
// over from the scan at these (D = 8,192, 2,000,000 rows, windows of 1,800: 9,000
// queries fp4 2.6 ms where a few tiles were narrow and 1.8 by tiles, 16,000 fp8 4.9
// and 3.9). It is the call's windows that count: near a limit for each tile a part
// of the tiles would be narrow, and the call waits for both ways (100,000 popcount
// queries of 60,000 rows, windows of 55, D = 1,024: 154 us by scan, 170 by tiles, 232
// so; 6,000 fp4, 909 of 2,000,000, D = 8,192: 0.95 ms by scan, 1.07 so).
int64_t narrow_pairs(int64_t nq, int32_t engine, uint32_t words, int tile)
{
    if (engine == HOMS_ENGINE_POPCOUNT)
        return words >= 128  ? 20000000
               : words >= 64 ? 30000000
               : words >= 32 ? 8000000
                             : 3000000;
    if (tile != 256 || words < 128) return INT64_MAX;
    return nq * (engine == HOMS_ENGINE_MFMA_F4 ? 1024 : 1536);
}
// Popcount: a scan fetches the row of every pair, and the tiles of long rows take
// a time of their own (chains of scalar loads), so that scans of some million pairs
// are the faster. Beyond, the windows' share of the union decides. Milliseconds by
// scan and by tiles, 20,000 queries over 400,000 rows, windows of 550 / 900 rows (1/10
// and 1/6.7, 11M and 18M pairs): D = 512 0.26 / 0.40 and 0.23 / 0.23, 1,024 0.27 / 0.41
// and 0.34 / 0.35, 2,048 0.36 / 0.55 and 0.58 / 0.60, 8,192 1.6 / 2.6 and 2.3 / 2.3;
// 100,000 over 1,600,000, 300 / 550 rows (1/15 and 1/8.5, 30M and 55M): D = 512 0.65 /
// 1.05 and 0.69 / 0.74, 1,024 0.66 / 1.07 and 1.07 / 1.11, 2,048 0.90 / 1.51 and 1.85 /
// 1.94, 8,192 4.4 / 8.1 and 6.6 / 6.8.
int64_t narrow_far10(int32_t engine, uint32_t words)
{
    if (engine != HOMS_ENGINE_POPCOUNT) return 0;
    return words >= 512 ? 120 : words >= 256 ? 100 : words >= 32 ? 80 : 130;
}

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
    int64_t narrow_ratio10, narrow_far10, narrow_max, narrow_pairs;
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

// one wave: the union of tile t's windows and whether the tile is narrow;
// at(i) is the query in place i of the order, total the call's pairs
template <class At>
__device__ __forceinline__ void tile_shape(const PlanArgs& a, int64_t t, int64_t total, At at)
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
        // a narrow tile keeps no rows for the tile kernels
        const int64_t pairs = 10 * (mx - mn) * a.tile;
        const bool narrow = big <= a.narrow_max && sum * a.narrow_ratio10 <= pairs &&
                            (total <= a.narrow_pairs ||
                             (a.narrow_far10 > 0 && sum * a.narrow_far10 <= pairs));
        a.w.tile_narrow[t] = narrow || mx == 0 ? 1 : 0;
        a.w.tile_lo[t] = narrow || mx == 0 ? 0 : mn;
        a.w.tile_hi[t] = narrow ? 0 : mx;
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
        // (few queries: windows of up to narrow_max rows are always few pairs)
        tile_shape(a, t, 0, [&](int64_t i) { return (uint32_t)s_key[i]; });
}

// ---- any number of queries, five launches

// buckets and sums cleared, fp4 query constants (one wave per query)
__global__ __launch_bounds__(kThreads) void plan_init_kernel(PlanArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t <= kBuckets) a.w.hist[t] = 0;
    if (t < kSums) a.w.pairs[t * kSumStride] = 0;
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
    int64_t pairs = hi - lo;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pairs += (int64_t)__shfl_xor((long long)pairs, o);
    if (threadIdx.x == 0)
        atomicAdd((unsigned long long*)a.w.pairs + blockIdx.x % kSums * kSumStride,
                  (unsigned long long)pairs);
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
    if (t * a.tile >= a.nq) return;
    int64_t total = (int64_t)a.w.pairs[(threadIdx.x & 63) * kSumStride];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += (int64_t)__shfl_xor((long long)total, o);
    tile_shape(a, t, total, [&](int64_t i) { return a.w.qperm[i]; });
}

// ---- after the search: the results of every query, and the narrow tiles

// one wave: the best (distance, library index) of rows [lo, hi) for one query
// row; 16 lanes per library row (contiguous 256-byte reads), eight rows a step.
// Bound by fetching the rows: 20,001 queries of 17 rows of 1 KB on average
// take 72 us (4.8 TB/s) where their 256-query tiles took 1,394 us.
__device__ __forceinline__ uint64_t scan_window(uint32_t words, const uint32_t* __restrict__ qrow,
                                                int64_t lo, int64_t hi,
                                                const uint32_t* __restrict__ lib_hv,
                                                const uint32_t* __restrict__ lib_orig)
{
    const int l = threadIdx.x & 63, g = l >> 4, li = l & 15;
    const uint32_t nc = words / 4;  // 16-byte pieces per row
    const uint4* qp = (const uint4*)qrow;
    uint64_t best = ~0ull;
    for (int64_t base = lo; base < hi; base += 8) {
        // rows past the end repeat the last one
        const int64_t ra = min(base + g, hi - 1), rb = min(base + 4 + g, hi - 1);
        const uint4* pa = (const uint4*)(lib_hv + (size_t)ra * words);
        const uint4* pb = (const uint4*)(lib_hv + (size_t)rb * words);
        const uint32_t oa = lib_orig[ra], ob = lib_orig[rb];
        uint32_t da = 0, db = 0;
#pragma unroll 4
        for (uint32_t c = li; c < nc; c += 16) {
            const uint4 q = qp[c], x = pa[c], y = pb[c];
            da += __builtin_popcount(q.x ^ x.x) + __builtin_popcount(q.y ^ x.y) +
                  __builtin_popcount(q.z ^ x.z) + __builtin_popcount(q.w ^ x.w);
            db += __builtin_popcount(q.x ^ y.x) + __builtin_popcount(q.y ^ y.y) +
                  __builtin_popcount(q.z ^ y.z) + __builtin_popcount(q.w ^ y.w);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            da += __shfl_xor(da, o);
            db += __shfl_xor(db, o);
        }
        const uint64_t ka = ((uint64_t)da << 32) | oa, kb = ((uint64_t)db << 32) | ob;
        best = min(best, min(ka, kb));
    }
    best = min(best, (uint64_t)__shfl_xor(best, 16));
    return min(best, (uint64_t)__shfl_xor(best, 32));
}

// one wave per kPerWave places of the order (of one tile)
constexpr int kPerWave = 2;
constexpr int64_t kPieceQueries = (int64_t)1 << 26;  // of one launch
__global__ __launch_bounds__(kThreads) void finish_kernel(PlanArgs a,
    const uint32_t* __restrict__ q_hv, const uint32_t* __restrict__ lib_hv,
    const uint32_t* __restrict__ lib_orig, int64_t* __restrict__ out_idx,
    int32_t* __restrict__ out_dist)
{
    const int64_t p0 =
        ((int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)) * kPerWave;
    const int l = threadIdx.x & 63;
    if (p0 >= a.nq) return;
    const int n = (int)min((int64_t)kPerWave, a.nq - p0);
    const uint32_t mine = l < n ? a.w.qperm[p0 + l] : 0u;
    uint64_t key = ~0ull;
    if (a.w.tile_narrow[p0 / a.tile]) {  // wave-uniform
        for (int i = 0; i < n; ++i) {
            const uint32_t q = __builtin_amdgcn_readlane(mine, i);
            const int64_t lo = a.w.lo[q], hi = a.w.hi[q];
            if (hi <= lo) continue;
            const uint64_t k =
                scan_window(a.words, q_hv + (size_t)q * a.words, lo, hi, lib_hv, lib_orig);
            if (l == i) key = k;
        }
    } else if (l < n) {
        key = a.w.keys[mine];
    }
    if (l < n) {
        out_idx[mine] = key == ~0ull ? -1 : (int64_t)(uint32_t)key;
        out_dist[mine] = key == ~0ull ? -1 : (int32_t)(key >> 32);
    }
}

}  // namespace

namespace {
size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
}  // namespace

size_t query_plan_bytes(int64_t nq, int tile)
{
    const int64_t nt = (nq + tile - 1) / tile;
    return 3 * al(nq * 8) + 4 * al(nq * 4) + 2 * al(nt * 8) + al(nt * 4) + al((kBuckets + 1) * 4) +
           al(kSums * kSumStride * 8);
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
    w.tile_narrow = (uint32_t*)take(nt * 4);
    w.hist = (uint32_t*)take((kBuckets + 1) * 4);
    w.pairs = (uint64_t*)take(kSums * kSumStride * 8);
    return w;
}

hipError_t launch_query_plan(const homs_ctx* c, int64_t nq, const double* q_pmz,
                             const int8_t* q_charge, int32_t kind, double value, int32_t engine,
                             const uint32_t* q_hv, int tile, const QueryPlan& w, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    if (engine != HOMS_ENGINE_MFMA_F4) q_hv = nullptr;  // no constants wanted
    const PlanArgs a{nq,          q_pmz,
                     q_charge,    c->p.charge_match != 0,
                     kind,        value,
                     c->lib.pmz,  c->lib.charge_first,
                     c->lib.n,    tile,
                     narrow_ratio10(engine, tile),
                     narrow_far10(engine, c->words),
                     narrow_max(nq),
                     narrow_pairs(nq, engine, c->words, tile),
                     c->words,    q_hv,
                     w};
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

hipError_t launch_finish(const homs_ctx* c, int64_t nq, const uint32_t* q_hv, int tile,
                         const QueryPlan& w, int64_t* out_idx, int32_t* out_dist, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    PlanArgs a{};
    a.tile = tile;
    a.words = c->words;
    a.w = w;
    const int64_t per = kPerWave * (kThreads / 64);
    // 32 threads a query: a grid holds less than 2^32. Each launch takes whole
    // tiles of the order.
    static_assert(kPieceQueries % 256 == 0 && kPieceQueries * 32 < (int64_t)1 << 32, "");
    for (int64_t p = 0; p < nq; p += kPieceQueries) {
        a.nq = std::min(kPieceQueries, nq - p);
        a.w.qperm = w.qperm + p;
        a.w.tile_narrow = w.tile_narrow + p / tile;
        finish_kernel<<<(uint32_t)((a.nq + per - 1) / per), kThreads, 0, s>>>(
            a, q_hv, c->lib.hv, c->lib.orig, out_idx, out_dist);
    }
    return hipGetLastError();
}

}  // namespace homs
