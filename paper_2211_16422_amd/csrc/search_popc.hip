// Open-window Hamming top-1 search with XOR + population count (Section 3.4;
// the bit-packed representation and popcount similarity of Section 4.1).
//
// Work decomposition. Queries are ordered by (charge, precursor m/z) and cut
// into tiles of 256; neighbouring queries share almost all of their
// candidates, so a tile's candidates are one contiguous range of the sorted
// library (the union of its queries' windows, a few rows wider than any one
// window). The range is cut into chunks of up to kChunk rows; one workgroup of
// four waves handles the (tile, chunk) pairs of a chunk and up to eight tiles,
// one after the other, every lane owning one query of a tile.
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
// over 200,000 rows: 3.98 -> 3.11 ms, later 2.7 ms with the window-middle
// query order and 2.3 with an odd number of tiles per turn).
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
    const uint32_t* __restrict__ lib_orig, uint32_t n_tiles, uint32_t slots, uint32_t per,
    uint32_t slot0, uint32_t n_slots, uint32_t round0, uint32_t chunk,
    uint64_t* __restrict__ keys)
{
    // workgroup i runs on XCD i mod 8, which takes chunks c = i mod 8 and, chunk
    // after chunk, every slot of tiles, so that a chunk's rows come into one L2
    // once and serve all the tiles there; this launch: n_slots slots from slot0
    // on, rounds of eight chunks from round0 on. Slot x: tiles x, x + slots, ...
    const uint32_t wg = blockIdx.x;
    const uint32_t slot = slot0 + (wg / 8) % n_slots;
    const int64_t c0 = ((int64_t)(round0 + (wg / 8) / n_slots) * 8 + wg % 8) * chunk;
    const uint32_t l = threadIdx.x & 63;
    int64_t a = 0, b = 0;  // lane l: the slot's tile l
    const uint32_t mine = slot + l * slots;
    if (l < per && mine < n_tiles) {
        const int64_t t_lo = tile_lo[mine], t_hi = tile_hi[mine];
        a = max(c0, t_lo);
        b = min(c0 + chunk, t_hi);
    }
    // the tiles with candidates in the chunk: short windows leave one or none
    for (uint64_t todo = __ballot(a < b); todo; todo &= todo - 1) {
        const int i = __builtin_ctzll(todo);
        popcount_tile_rows(words, nq, q_hv, qperm, lo, hi, slot + (uint32_t)i * slots,
                           (uint32_t)__builtin_amdgcn_readlane((int)a, i),
                           (uint32_t)__builtin_amdgcn_readlane((int)b, i), lib_hv, lib_orig, keys);
    }
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
                                  uint64_t* keys, hipStream_t s)
{
    const int64_t n_tiles = (nq + kTile - 1) / kTile;
    if (n_tiles <= 0 || c->lib.n <= 0) return hipSuccess;
    // A chunk is a chain of scalar loads (256 rows of D = 8,192: 0.9 ms), and the
    // items that hold candidates should be many more than the 1,800 workgroups
    // the chip has room for (20,000 queries +-8.25 Da of 400,000 rows, D = 8,192:
    // 5.1 ms with 1,024 rows, 2.7 with 256; 2,001 queries +-500 Da of 200,000 rows,
    // D = 8,192: 4.0 ms with 2,048, 2.3 with 64). But each workgroup costs its
    // dispatch, 0.3 ns and more, and where windows are short hardly an item holds
    // candidates: a workgroup takes eight of a chunk's items, of tiles far from
    // each other (100,000 queries of 2,000,000 rows, D = 1,024: +-0.1 Da 1.27 ms with
    // a workgroup for each item, 0.51 so; +-1.65 Da 2.62 and 1.74, with chunks of 512
    // rows 2.28 and 1.79). Where all of them do, the rows are at hand (20,000
    // queries +-500 Da of 60,000 rows, D = 8,192: 5.65 and 5.59 ms).
    int64_t chunk = 256, per = 8;
    while (chunk < kChunk && n_tiles * (c->lib.n / chunk) > (per << 21)) chunk *= 2;
    while (chunk > 64 && n_tiles * ((c->lib.n + chunk - 1) / chunk) < 16384) chunk /= 2;
    const int64_t n_chunks = (c->lib.n + chunk - 1) / chunk;
    while (per > 1 && (n_tiles + per - 1) / per * n_chunks < 8192) per /= 2;
    // An odd number of slots, if need be with an empty one: where one or two of a
    // chunk's hold candidates, these come to the same few compute units of an XCD
    // turn after turn if the turns are 2, 4, 8 or 16 long (4,000 queries, 16 tiles,
    // +-1.65 Da of 2,000,000 rows, D = 8,192: 16.0 ms, 7.2 with an empty tile; 1,000
    // queries +-5 Da 22.6 and 7.1). Few workgroups run all at once (1,000 queries of
    // 60,000 rows, +-50 Da: 0.36 ms, 0.42 with an empty tile).
    int64_t slots = (n_tiles + per - 1) / per;
    if (slots * n_chunks >= 4096) slots |= 1;
    // whole rounds of 8 chunks, so every XCD's sequence is complete
    const int64_t n_rounds = (n_chunks + 7) / 8;
    in_pieces(slots, n_rounds, kTile, [&](int64_t t, int64_t count, int64_t r, int64_t rounds) {
        search_popcount_kernel<<<(uint32_t)(count * rounds * 8), kTile, 0, s>>>(
            c->words, nq, q_hv, qperm, lo, hi, tile_lo, tile_hi, c->lib.hv, c->lib.orig,
            (uint32_t)n_tiles, (uint32_t)slots, (uint32_t)per, (uint32_t)t, (uint32_t)count,
            (uint32_t)r, (uint32_t)chunk, keys);
    });
    return hipGetLastError();
}

}  // namespace homs
