// Batched search of a mixed query stream (narrow ppm and open Da windows,
// Table 1) in one persistent launch.
//
// A batch mixes windows of a few dozen candidates with windows of a million.
// Queries are split by window size: a "wide" query (more than
// cfg.narrow_max candidates) goes into 256-query tiles that share one
// candidate range, scored with the XOR + popcount tile code of the plain
// search; a "narrow" query is scored by one wave with one candidate row per
// lane. Both kinds become work items of queues: (wide tile, row chunk) pairs,
// then groups of narrow queries. A persistent grid of workgroups pulls items
// with atomic counters until every queue is empty, so every wave reaches the
// exit.
//
// The wide items are kept in patches of 8 adjacent tiles x 4 adjacent chunks
// on absolute chunk boundaries, and each of the eight XCDs (each with its own
// L2; workgroup i runs on XCD i mod 8) has a queue of every eighth patch, so
// the 32 workgroups of an XCD read the same few chunks together. A workgroup
// whose queue is empty goes on with the next one. With one queue in (tile,
// chunk) order every tile fetched its rows again from memory: 50,000 queries
// (15,000 wide) of 1,000,000 rows, D = 8,192: 9.70 ms so, 8.49 ms in patches
// (0.13 ms of that is planning done in parallel instead of by one workgroup).
//
// Everything between the inputs and the outputs is device work with a fixed
// launch shape (no host synchronisation, no memset or copy nodes, no library
// sort), so the whole batch can be captured once in a hipGraph and replayed:
//   window bounds -> bucket histogram (and key reset) -> scan -> scatter
//   (counting sort by (wide/narrow, charge, precursor bucket)) -> tiles ->
//   plan -> persistent search -> finalize.

#include "mfma_direct.h"
#include "popcount_tile.h"

namespace homs {
namespace {

constexpr int kThreads = 256;
constexpr int kScanBlock = 1024;          // elements per first-level scan block
constexpr int kCharges = 16;              // charges 0..15 get buckets; others clamp
constexpr int kPmzBuckets = 8192;         // precursor buckets of cfg width each
constexpr int kClassBuckets = kCharges * kPmzBuckets;
constexpr int kBuckets = 2 * kClassBuckets;  // wide first, then narrow

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kThreads - 1) / kThreads); }

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// bucket of every query: (narrow?, charge, floor(pmz / width)), clamped; and
// its empty result key
__global__ void bucket_kernel(int64_t nq, const double* __restrict__ q_pmz,
                              const int8_t* __restrict__ q_charge, bool use_charge,
                              const int64_t* __restrict__ lo, const int64_t* __restrict__ hi,
                              uint32_t narrow_max, double inv_width,
                              uint32_t* __restrict__ bucket, uint32_t* __restrict__ hist,
                              uint64_t* __restrict__ keys)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    keys[q] = ~0ull;
    const bool narrow = (hi[q] - lo[q]) <= (int64_t)narrow_max;
    int c = use_charge ? (int)q_charge[q] : 0;
    c = c < 0 ? 0 : (c >= kCharges ? kCharges - 1 : c);
    const double x = q_pmz[q] * inv_width;
    int p = (x >= 0.0) ? (x < (double)(kPmzBuckets - 1) ? (int)x : kPmzBuckets - 1) : 0;
    const uint32_t bkt = (narrow ? kClassBuckets : 0) + (uint32_t)(c * kPmzBuckets + p);
    bucket[q] = bkt;
    atomicAdd(hist + bkt, 1u);
}

// exclusive scan, level 1: each block scans kScanBlock entries in place, four
// a thread, and records its total
__global__ __launch_bounds__(kThreads) void scan_blocks_kernel(uint32_t* __restrict__ a,
                                                               uint32_t* __restrict__ block_sums)
{
    static_assert(kScanBlock == 4 * kThreads && kBuckets % kScanBlock == 0, "whole blocks");
    __shared__ uint32_t s_wave[kThreads / 64];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint4* const p = (uint4*)(a + (int64_t)blockIdx.x * kScanBlock) + threadIdx.x;
    const uint4 v = *p;
    const uint32_t sum = v.x + v.y + v.z + v.w;
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (l >= o) inc += y;
    }
    if (l == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t run = inc - sum, total = 0;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) {
        if (i < w) run += s_wave[i];
        total += s_wave[i];
    }
    *p = make_uint4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// level 2: each block adds the totals of the blocks before it
__global__ __launch_bounds__(kThreads) void scan_add_kernel(uint32_t* __restrict__ a,
                                                            const uint32_t* __restrict__ block_sums)
{
    static_assert(kBuckets / kScanBlock <= kThreads, "one total a thread");
    __shared__ uint32_t s_wave[kThreads / 64];
    uint32_t x = threadIdx.x < blockIdx.x ? block_sums[threadIdx.x] : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = x;
    __syncthreads();
    x = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    uint4* const p = (uint4*)(a + (int64_t)blockIdx.x * kScanBlock) + threadIdx.x;
    uint4 v = *p;
    v.x += x;
    v.y += x;
    v.z += x;
    v.w += x;
    *p = v;
}

// counting-sort scatter; the order inside a bucket is arbitrary and results
// do not depend on it (keys merge with atomicMin)
__global__ void scatter_kernel(int64_t nq, const uint32_t* __restrict__ bucket,
                               uint32_t* __restrict__ cursor, uint32_t* __restrict__ order)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const uint32_t pos = atomicAdd(cursor + bucket[q], 1u);
    order[pos] = (uint32_t)q;
}

constexpr uint32_t kXcds = 8;
constexpr int64_t kPatchTiles = 8;
constexpr uint32_t kPatchChunks = 4;
constexpr uint32_t kPatchItems = (uint32_t)kPatchTiles * kPatchChunks;

struct Plan {
    uint32_t n_wide;        // wide queries occupy order[0, n_wide)
    uint32_t groups;        // groups of kPatchTiles wide tiles
    uint32_t patches;       // patches of all groups
    uint32_t narrow_items;  // groups of narrow queries
    uint32_t next[kXcds];   // queue heads: the wide items of patches y, y + 8, ...
    uint32_t next_narrow;   // and the narrow ones
};
// a group's first patch and first chunk
struct Group {
    uint32_t patch, chunk;
};

// One wave per tile: the union of its queries' windows. After the scatter, the
// cursor of the last wide bucket has advanced to the first narrow position,
// i.e. to the number of wide queries.
__global__ __launch_bounds__(kThreads) void tiles_kernel(
    const uint32_t* __restrict__ cursor, const uint32_t* __restrict__ order,
    const int64_t* __restrict__ lo, const int64_t* __restrict__ hi, int64_t max_tiles,
    int64_t* __restrict__ tile_lo, int64_t* __restrict__ tile_hi)
{
    const int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (t >= max_tiles) return;
    const int64_t n_wide = cursor[kClassBuckets - 1];
    const int64_t end = min((t + 1) * (int64_t)popc::kTile, n_wide);
    int64_t mn = INT64_MAX, mx = 0;
    for (int64_t i = t * popc::kTile + (threadIdx.x & 63); i < end; i += 64) {
        const uint32_t q = order[i];
        if (hi[q] > lo[q]) {
            mn = min(mn, lo[q]);
            mx = max(mx, hi[q]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, (int64_t)__shfl_xor((long long)mn, o));
        mx = max(mx, (int64_t)__shfl_xor((long long)mx, o));
    }
    if ((threadIdx.x & 63) == 0) {
        tile_lo[t] = mn == INT64_MAX ? 0 : mn;
        tile_hi[t] = mx;
    }
}

// One workgroup: the groups' chunk ranges, the prefix of their patches, and
// the queue heads.
__global__ __launch_bounds__(1024) void plan_kernel(
    int64_t nq, const uint32_t* __restrict__ cursor, uint32_t chunk_rows, uint32_t narrow_group,
    const int64_t* __restrict__ tile_lo, const int64_t* __restrict__ tile_hi,
    Group* __restrict__ group, Plan* __restrict__ plan)
{
    __shared__ uint32_t s_part[1024];
    const uint32_t n_wide = cursor[kClassBuckets - 1];
    const int64_t n_tiles = ((int64_t)n_wide + popc::kTile - 1) / popc::kTile;
    const int64_t n_groups = (n_tiles + kPatchTiles - 1) / kPatchTiles;
    // contiguous groups per thread
    const int64_t per = (n_groups + blockDim.x - 1) / blockDim.x;
    const int64_t g0 = min(threadIdx.x * per, n_groups), g1 = min(g0 + per, n_groups);
    uint32_t part = 0;
    for (int64_t g = g0; g < g1; ++g) {
        int64_t mn = INT64_MAX, mx = 0;
        for (int64_t t = g * kPatchTiles; t < min((g + 1) * kPatchTiles, n_tiles); ++t)
            if (tile_hi[t] > tile_lo[t]) {
                mn = min(mn, tile_lo[t]);
                mx = max(mx, tile_hi[t]);
            }
        if (mn == INT64_MAX) mn = mx = 0;
        const uint32_t c0 = (uint32_t)(mn / chunk_rows);
        const uint32_t n = mx > mn ? (uint32_t)((mx + chunk_rows - 1) / chunk_rows) - c0 : 0u;
        const uint32_t patches = (n + kPatchChunks - 1) / kPatchChunks;
        group[g] = {patches, c0};
        part += patches;
    }
    s_part[threadIdx.x] = part;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {  // inclusive prefix of the threads' sums
        const uint32_t v = (int)threadIdx.x >= o ? s_part[threadIdx.x - o] : 0u;
        __syncthreads();
        s_part[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = s_part[threadIdx.x] - part;
    for (int64_t g = g0; g < g1; ++g) {
        const uint32_t n = group[g].patch;
        group[g].patch = run;
        run += n;
    }
    if (threadIdx.x < kXcds) plan->next[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        const uint32_t n_narrow = (uint32_t)(nq - n_wide);
        plan->n_wide = n_wide;
        plan->groups = (uint32_t)n_groups;
        plan->patches = s_part[1023];
        plan->narrow_items = (n_narrow + narrow_group - 1) / narrow_group;
        plan->next_narrow = 0;
    }
}

// ENGINE 0: popcount tiles, 256 threads; ENGINE 2 / 3: fp8 / fp4 matrix-core
// tiles (mfd::tile_rows), 512 threads. Narrow queries are spread over the waves.
template <int ENGINE>
__global__ __launch_bounds__(ENGINE == 0 ? popc::kTile : mfd::kThreads) void
persistent_search_kernel(uint32_t words, const uint32_t* __restrict__ q_hv,
                         const uint32_t* __restrict__ order, const int64_t* __restrict__ lo,
                         const int64_t* __restrict__ hi, int64_t nq,
                         const int64_t* __restrict__ tile_lo, const int64_t* __restrict__ tile_hi,
                         const Group* __restrict__ group, uint32_t chunk_rows,
                         uint32_t narrow_group, Plan* __restrict__ plan,
                         const uint32_t* __restrict__ lib_hv,
                         const uint32_t* __restrict__ lib_orig, const int32_t* __restrict__ qoff,
                         const float* __restrict__ rowk, uint64_t* __restrict__ keys)
{
    static_assert(popc::kTile == mfd::kQueries, "all engines use 256-query tiles");
    constexpr int kFormat = ENGINE == HOMS_ENGINE_MFMA_F4 ? 4 : 0;  // f8f6f4 element format
    __shared__ uint32_t s_item, s_drained;
    const uint32_t n_wide = plan->n_wide, n_groups = plan->groups, patches = plan->patches;
    const uint32_t n_tiles = (n_wide + popc::kTile - 1) / popc::kTile;
    const uint32_t waves = blockDim.x >> 6;
    // the next item of a queue, the same for the whole workgroup
    auto pull = [&](uint32_t* head) -> uint32_t {
        if (threadIdx.x == 0) s_item = atomicAdd(head, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        return item;
    };
    // wide items of queue y
    auto wide = [&](uint32_t y) { return (patches + kXcds - 1 - y) / kXcds * kPatchItems; };
    // queues found empty, bit kXcds the narrow one, in one look at their heads: a
    // compute unit holds one workgroup of the matrix-core tiles, and those of the
    // grid beyond 256 start when the others are done (a pull each, nine in turn, for
    // 768 of them made 4,183 queries of 54,000 rows 212 us where 186 do)
    if (threadIdx.x < 64) {
        bool empty = false;
        if (threadIdx.x <= kXcds) {
            const uint32_t y = threadIdx.x;
            const uint32_t head =
                __hip_atomic_load(y < kXcds ? &plan->next[y] : &plan->next_narrow,
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            empty = head >= (y < kXcds ? wide(y) : plan->narrow_items);
        }
        const uint64_t found = __ballot(empty);
        if (threadIdx.x == 0) s_drained = (uint32_t)found;
    }
    __syncthreads();
    const uint32_t drained = __builtin_amdgcn_readfirstlane(s_drained);
    // wide items: this XCD's queue first, then the others in turn; every
    // workgroup leaves a queue once its head has passed its items
    for (uint32_t i = 0; i < kXcds; ++i) {
        const uint32_t y = (blockIdx.x + i) % kXcds;
        if (drained >> y & 1) continue;  // uniform
        const uint32_t items = wide(y);
        for (;;) {
            const uint32_t item = pull(&plan->next[y]);
            if (item >= items) break;
            const uint32_t patch = item / kPatchItems * kXcds + y, local = item % kPatchItems;
            // largest group whose first patch <= patch
            uint32_t l = 0, r = n_groups - 1;
            while (l < r) {
                const uint32_t m = (l + r + 1) >> 1;
                if (group[m].patch <= patch)
                    l = m;
                else
                    r = m - 1;
            }
            const uint32_t tile = l * (uint32_t)kPatchTiles + local / kPatchChunks;
            if (tile >= n_tiles) continue;
            const int64_t c0 = (int64_t)(group[l].chunk + (patch - group[l].patch) * kPatchChunks +
                                         local % kPatchChunks) * chunk_rows;
            const int64_t a = max(c0, tile_lo[tile]);
            const int64_t b = min(c0 + (int64_t)chunk_rows, tile_hi[tile]);
            if (a >= b) continue;
            if constexpr (ENGINE == 0)
                popc::popcount_tile_rows(words, (int64_t)n_wide, q_hv, order, lo, hi, tile,
                                         (uint32_t)a, (uint32_t)b, lib_hv, lib_orig, keys);
            else
                mfd::tile_rows<kFormat>(words, (int64_t)n_wide, q_hv, order, lo, hi, tile,
                                        (uint32_t)a, (uint32_t)b, lib_hv, lib_orig, qoff, rowk,
                                        keys);
        }
    }
    if (drained >> kXcds & 1) return;  // uniform
    for (;;) {
        const uint32_t item = pull(&plan->next_narrow);
        if (item >= plan->narrow_items) break;  // uniform: every wave of every workgroup exits here
        const int64_t first = (int64_t)n_wide + (int64_t)item * narrow_group;
        const int64_t last = min(first + (int64_t)narrow_group, nq);
        for (int64_t p = first + (threadIdx.x >> 6); p < last; p += waves) {
            const uint32_t qi = order[p];
            if (hi[qi] > lo[qi])
                popc::window_rows_wave(words, qi, q_hv, (uint32_t)lo[qi], (uint32_t)hi[qi], lib_hv,
                                       lib_orig, keys);
        }
    }
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t batched_scratch_bytes(int64_t nq)
{
    const int64_t max_tiles = (nq + popc::kTile - 1) / popc::kTile + 1;
    const int64_t scan_blocks = (kBuckets + kScanBlock - 1) / kScanBlock;
    return 2 * al(nq * 8) + al(nq * 8) + 2 * al(nq * 4) + al(kBuckets * 4) +
           al(scan_blocks * 4) + 2 * al(max_tiles * 8) + al(max_tiles * sizeof(Group)) + al(nq * 4) +
           al(sizeof(Plan));
}

hipError_t launch_search_batched(const homs_ctx* c, const BatchedConfig& cfg, void* scratch,
                                 int64_t nq, const uint32_t* q_hv, const double* q_pmz,
                                 const int8_t* q_charge, const int8_t* kinds,
                                 const double* values, int64_t* out_idx, int32_t* out_dist,
                                 hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    const int64_t max_tiles = (nq + popc::kTile - 1) / popc::kTile + 1;
    const int64_t scan_blocks = (kBuckets + kScanBlock - 1) / kScanBlock;
    char* p = (char*)scratch;
    int64_t* lo = (int64_t*)p;
    p += al(nq * 8);
    int64_t* hi = (int64_t*)p;
    p += al(nq * 8);
    uint64_t* keys = (uint64_t*)p;
    p += al(nq * 8);
    uint32_t* bucket = (uint32_t*)p;
    p += al(nq * 4);
    uint32_t* order = (uint32_t*)p;
    p += al(nq * 4);
    uint32_t* hist = (uint32_t*)p;  // counts, then bucket starts, then cursors
    p += al(kBuckets * 4);
    uint32_t* sums = (uint32_t*)p;
    p += al(scan_blocks * 4);
    int64_t* tile_lo = (int64_t*)p;
    p += al(max_tiles * 8);
    int64_t* tile_hi = (int64_t*)p;
    p += al(max_tiles * 8);
    Group* group = (Group*)p;  // at most one per tile
    p += al(max_tiles * sizeof(Group));
    int32_t* qoff = (int32_t*)p;  // per-query constants of the fp4 engine
    p += al(nq * 4);
    Plan* plan = (Plan*)p;

    hipError_t e = launch_window_bounds(c, nq, q_pmz, q_charge, HOMS_TOL_DA, 0.0, kinds, values,
                                        lo, hi, s);
    if (e != hipSuccess) return e;
    fill_u32_kernel<<<blocks_for(kBuckets), kThreads, 0, s>>>(hist, kBuckets, 0u);
    bucket_kernel<<<blocks_for(nq), kThreads, 0, s>>>(nq, q_pmz, q_charge, c->p.charge_match != 0,
                                                      lo, hi, cfg.narrow_max,
                                                      1.0 / cfg.bucket_da, bucket, hist, keys);
    scan_blocks_kernel<<<(uint32_t)scan_blocks, kThreads, 0, s>>>(hist, sums);
    scan_add_kernel<<<(uint32_t)scan_blocks, kThreads, 0, s>>>(hist, sums);
    scatter_kernel<<<blocks_for(nq), kThreads, 0, s>>>(nq, bucket, hist, order);
    tiles_kernel<<<(uint32_t)((max_tiles + 3) / 4), kThreads, 0, s>>>(hist, order, lo, hi,
                                                                      max_tiles, tile_lo, tile_hi);
    plan_kernel<<<1, 1024, 0, s>>>(nq, hist, cfg.chunk_rows, cfg.narrow_group, tile_lo, tile_hi,
                                   group, plan);
    if (cfg.engine == HOMS_ENGINE_MFMA_F8) {
        persistent_search_kernel<HOMS_ENGINE_MFMA_F8><<<cfg.grid, mfd::kThreads, 0, s>>>(
            c->words, q_hv, order, lo, hi, nq, tile_lo, tile_hi, group,
            cfg.chunk_rows, cfg.narrow_group, plan, c->lib.hv, c->lib.orig, nullptr, nullptr,
            keys);
    } else if (cfg.engine == HOMS_ENGINE_MFMA_F4) {
        e = launch_fp4_query_offsets(c, nq, q_hv, qoff, s);
        if (e != hipSuccess) return e;
        persistent_search_kernel<HOMS_ENGINE_MFMA_F4><<<cfg.grid, mfd::kThreads, 0, s>>>(
            c->words, q_hv, order, lo, hi, nq, tile_lo, tile_hi, group,
            cfg.chunk_rows, cfg.narrow_group, plan, c->lib.hv, c->lib.orig, qoff, c->lib.rowk,
            keys);
    } else {
        persistent_search_kernel<HOMS_ENGINE_POPCOUNT><<<cfg.grid, popc::kTile, 0, s>>>(
            c->words, q_hv, order, lo, hi, nq, tile_lo, tile_hi, group,
            cfg.chunk_rows, cfg.narrow_group, plan, c->lib.hv, c->lib.orig, nullptr, nullptr,
            keys);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_finalize(nq, keys, out_idx, out_dist, s);
}

}  // namespace homs
