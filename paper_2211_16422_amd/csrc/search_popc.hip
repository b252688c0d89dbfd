// Open-window Hamming top-1 search with XOR + population count (Section 3.4;
// the bit-packed representation and popcount similarity of Section 4.1).
//
// Work decomposition. Queries are ordered by (charge, precursor m/z) and cut
// into tiles of 256; neighbouring queries share almost all of their
// candidates, so a tile's candidates are one contiguous range of the sorted
// library (the union of its queries' windows, a few rows wider than any one
// window). The range is cut into chunks of up to kChunk rows; one workgroup of
// four waves handles one (tile, chunk) pair, every lane owning one query.
//
// Inner loop. A wave walks its chunk kRefs rows at a time. For each block of
// kWords words of the packed vectors the lane loads that slice of its own
// query into VGPRs, and every reference row slice is fetched with scalar
// loads (the row index is wave-uniform, so one s_load_dwordx16 feeds all 64
// queries of the wave through SGPR operands). Each 32-bit word then costs
// exactly two VALU instructions per (query, reference) pair: v_xor_b32 and
// v_bcnt_u32_b32 (population count with accumulate) into a per-reference
// accumulator. The wave's four-wave workgroup walks the same rows, so the
// scalar cache serves one fetch of a row to all 256 queries of the tile, and
// a vector load of one word per line brings the next block's rows into L2
// ahead of the scalar loads (with the XCD map of the launch, 2,001 queries
// over 200,000 rows: 3.98 -> 3.11 ms, later 2.6 ms with the window-middle
// query order).
// Scalar loads are software-pipelined two rows ahead: without it every row
// waits out a full scalar-load round trip and the kernel sits near 70% of
// the VALU issue rate; with it, above 90%.
//
// Selection. After a block's distances are complete each lane keeps the
// lexicographic minimum of (distance, library index) over rows inside its
// own window [lo, hi); the lane's minimum is merged into the query's 64-bit
// key (distance << 32 | library index) with one global atomicMin.
#include "launch_pieces.h"
#include "popcount_tile.h"

namespace homs {
namespace {

using namespace popc;

__global__ __launch_bounds__(kTile) void search_popcount_kernel(
    uint32_t words, int64_t nq, const uint32_t* __restrict__ q_hv,
    const uint32_t* __restrict__ qperm, const int64_t* __restrict__ lo,
    const int64_t* __restrict__ hi, const int64_t* __restrict__ tile_lo,
    const int64_t* __restrict__ tile_hi, const uint32_t* __restrict__ lib_hv,
    const uint32_t* __restrict__ lib_orig, uint32_t tile0, uint32_t n_tiles, uint32_t round0,
    int64_t chunk, uint64_t* __restrict__ keys)
{
    // workgroup i runs on XCD i mod 8, which takes chunks c = i mod 8 and,
    // chunk after chunk, every tile, so that a chunk's rows come into one L2
    // once and serve all the tiles there; this launch: n_tiles tiles from tile0
    // on, rounds of eight chunks from round0 on
    const uint32_t wg = blockIdx.x;
    const uint32_t tile = tile0 + (wg / 8) % n_tiles;
    const int64_t c0 = ((int64_t)(round0 + (wg / 8) / n_tiles) * 8 + wg % 8) * chunk;
    const int64_t a = max(c0, tile_lo[tile]), b = min(c0 + chunk, tile_hi[tile]);
    if (a >= b) return;  // the chunk holds none of the tile's candidates
    popcount_tile_rows(words, nq, q_hv, qperm, lo, hi, tile, (uint32_t)a, (uint32_t)b, lib_hv,
                       lib_orig, keys);
}

__global__ void tile_bounds_kernel(int64_t nq, int64_t n_tiles, int tile,
                                   const uint32_t* __restrict__ qperm,
                                   const int64_t* __restrict__ lo, const int64_t* __restrict__ hi,
                                   int64_t* __restrict__ tile_lo, int64_t* __restrict__ tile_hi)
{
    // one wave per tile: lanes stride over its queries, then a wave reduction
    const int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (t >= n_tiles) return;  // wave-uniform
    int64_t mn = INT64_MAX, mx = 0;
    const int64_t end = min((t + 1) * (int64_t)tile, nq);
    for (int64_t i = t * tile + l; i < end; i += 64) {
        const uint32_t q = qperm[i];
        const int64_t a = lo[q], b = hi[q];
        if (b > a) {
            mn = min(mn, a);
            mx = max(mx, b);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, (int64_t)__shfl_xor((long long)mn, off));
        mx = max(mx, (int64_t)__shfl_xor((long long)mx, off));
    }
    if (l == 0) {
        if (mn == INT64_MAX) mn = mx = 0;
        tile_lo[t] = mn;
        tile_hi[t] = mx;
    }
}

}  // namespace

int search_popcount_tile() { return kTile; }

hipError_t launch_tile_bounds(int64_t nq, const uint32_t* qperm, const int64_t* lo,
                              const int64_t* hi, int tile, int64_t* tile_lo, int64_t* tile_hi,
                              hipStream_t s)
{
    const int64_t n_tiles = (nq + tile - 1) / tile;
    if (n_tiles <= 0) return hipSuccess;
    tile_bounds_kernel<<<(uint32_t)((n_tiles + 3) / 4), 256, 0, s>>>(nq, n_tiles, tile, qperm, lo,
                                                                     hi, tile_lo, tile_hi);
    return hipGetLastError();
}

hipError_t launch_search_popcount(const homs_ctx* c, int64_t nq, const uint32_t* q_hv,
                                  const uint32_t* qperm, const int64_t* lo, const int64_t* hi,
                                  const int64_t* tile_lo, const int64_t* tile_hi,
                                  uint64_t* keys, int32_t kind, double value, hipStream_t s)
{
    const int64_t n_tiles = (nq + kTile - 1) / kTile;
    if (n_tiles <= 0 || c->lib.n <= 0) return hipSuccess;
    // Enough (tile, chunk) items to fill the chip evenly (2,001 queries,
    // 200,000 rows, D = 8,192: 4.03 ms with 2,048-row chunks, 3.11 ms so). A
    // chunk is a chain of scalar loads (2,048 rows of D = 8,192: 7 ms), which
    // windows of a few thousand rows wait for (9,000 queries +-2.75 Da of
    // 2,000,000 rows 12.3 ms with chunks of 2,048 rows, 10.0 with 1,024). The
    // shortest windows are scanned instead and leave hardly an item here, but
    // each workgroup costs its dispatch (6,000 queries +-5 ppm of 2,000,000 rows,
    // D = 2,048: 41 us in all, 63 with chunks of 512 rows).
    const double da = kind == HOMS_TOL_PPM ? value / 1000.0 : value;  // near 1,000 Da
    int64_t chunk = da <= 0.15 ? kChunk : kChunk / 2;
    while (chunk > 64 && n_tiles * ((c->lib.n + chunk - 1) / chunk) < 16384) chunk /= 2;
    // whole rounds of 8 chunks, so every XCD's sequence is complete
    const int64_t n_rounds = ((c->lib.n + chunk - 1) / chunk + 7) / 8;
    in_pieces(n_tiles, n_rounds, kTile, [&](int64_t t, int64_t tiles, int64_t r, int64_t rounds) {
        search_popcount_kernel<<<(uint32_t)(tiles * rounds * 8), kTile, 0, s>>>(
            c->words, nq, q_hv, qperm, lo, hi, tile_lo, tile_hi, c->lib.hv, c->lib.orig,
            (uint32_t)t, (uint32_t)tiles, (uint32_t)r, chunk, keys);
    });
    return hipGetLastError();
}

}  // namespace homs
