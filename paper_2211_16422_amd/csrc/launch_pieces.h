// Launches of more workgroups than one grid may hold. A dispatch counts its
// threads in 32 bits, and HIP refuses a grid of 2^32 threads or more: 100,000
// queries of 45,000,000 library rows are 8.6M workgroups of 512 threads, most
// of which find no candidates. Such a launch is made in pieces. Plain C++, so
// that the arithmetic can be checked on the host.
#pragma once
#include <stdint.h>

namespace homs {

// most workgroups of one launch: whole rounds of the eight XCDs, so that
// workgroup i of every piece runs on XCD i mod 8
constexpr int64_t most_workgroups(int threads) { return 0xFFFFFFFFll / threads / 8 * 8; }

// go(first, count) for the workgroups [0, n) of `threads` threads each
template <class F>
void in_pieces(int64_t n, int threads, F&& go)
{
    const int64_t most = most_workgroups(threads);
    for (int64_t first = 0; first < n; first += most)
        go(first, n - first < most ? n - first : most);
}

// go(tile, tiles, round, rounds) for kernels of one workgroup per tile and
// chunk of the library, eight chunks (one for each XCD) a round
template <class F>
void in_pieces(int64_t n_tiles, int64_t n_rounds, int threads, F&& go)
{
    const int64_t pairs = most_workgroups(threads) / 8;
    const int64_t tiles = n_tiles < pairs ? n_tiles : pairs;
    const int64_t rounds = tiles > 0 ? pairs / tiles : 1;
    for (int64_t t = 0; t < n_tiles; t += tiles)
        for (int64_t r = 0; r < n_rounds; r += rounds)
            go(t, n_tiles - t < tiles ? n_tiles - t : tiles, r,
               n_rounds - r < rounds ? n_rounds - r : rounds);
}

}  // namespace homs
