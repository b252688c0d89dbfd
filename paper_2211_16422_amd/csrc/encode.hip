// Eq. 1 encoding (Section 3.3) on gfx950.
//
// One group of D/128 consecutive lanes encodes one spectrum; lane w owns the
// 128 components 128w .. 128w+127 (one uint4 of the packed row). For every
// peak (bin i, level j) the lane loads its uint4 of F_i (a coalesced 16-byte
// load: the group reads the whole 1 KiB row at D = 8192) and of L_j, binds
// them with XOR (bit 0 = +1, so the bipolar product is XOR) and adds the
// 128 resulting bits into bit-sliced counters: plane k holds bit k of the
// number of -1 components seen so far. Peaks are taken eight at a time: the
// 16 row loads of a group are issued together (the kernel waits on gathered
// rows, so loads in flight set its speed), and the eight bound rows enter the
// counters through a carry-save tree of full adders on the three low planes
// (the Harley-Seal scheme: planes 0, 1 and 2 take the ones, twos and fours,
// one carry of weight 8 ripples into the planes above): 21 + 2(P - 3)
// operations per word for eight peaks (27 at P = 6) where a ripple of half
// adders takes 2P per peak (96). The last, partial group is masked. The bipolar sum is I = n - 2c
// (n peaks, c components equal to -1), so the binarised bit (1 unless I > 0)
// is c >= ceil(n/2), evaluated on the planes with a bit-sliced comparison
// against that constant.
//
// The random-projection baseline of Section 4.2 weights bin i's random row by
// w = level + 1 instead of binding it with a level vector: S = W - 2c with
// W = sum of the weights and c the weighted count of -1 components, added to
// the planes as w's binary digits (the row's bits enter plane k for every
// set bit k of w); the bit is c >= ceil(W/2) again.
//
// Step-function encoding (the generated ID_LEVEL tables, spectra below 64
// peaks, calls of many spectra). Gathering F_i reads 1 KB per
// peak at D = 8192 and bounds the kernel above; but the generated tables are
// flips along a random order, so the bits follow from counting alone.
// Component d is flipped by the peak's position iff its flip rank t_d is
// below k_i = floor(alpha i / (f - 1)), and by its level iff j >= u_d. With
// the peaks in ascending k, the e peaks with k <= t_d do not flip it, so for
// every component of one class (u, c0 = F_0 xor L_0 at d) the count depends
// on e alone:
//     count = tot_u + e - 2 pre_u(e),   tot_u = #{j < u}, pre_u(e) = #{first e, j < u},
// and the bit (count >= ceil(n/2), or count <= floor(n/2) where c0 = 1) is a
// step function of t_d with few steps. One wave per spectrum, a lane per e,
// collects the bits of all classes in one word per lane (per level one ballot
// and two sign bits); where a lane's word differs from its neighbour's, a
// class steps at that peak's k, and the step is one toggled bit: word s of the
// slot where the class's components with t_d >= k begin (slots: codebook.h).
// 32 spectra share the slots, one bit each, so one running XOR over the slots
// gives every component's bit of 32 spectra, and output word w of all of them
// is a gather of 32 slots and a 32 x 32 bit transpose. A class's slots start
// from the value the running XOR brings (a toggle where its first bit differs
// from the previous class's last).
#include <algorithm>
#include <type_traits>

#include "bits.h"
#include "codebook.h"
#include "internal.h"
#include "launch_pieces.h"

namespace homs {
namespace {

constexpr int kStepSpectra = 32;   // spectra per workgroup
constexpr int kStepPeaks = 63;     // most peaks of a spectrum (n + 1 lanes)
constexpr uint32_t kStepSlots = 16384;  // most slots (64 KB of LDS)
constexpr int64_t kStepWords = (int64_t)3 << 18;  // least words of output
constexpr int kStepThreads = 512;

struct StepArgs {
    const uint32_t* start;
    const uint16_t* source;
    const uint16_t* first_off;
    uint32_t classes, slots, alpha, words;
    uint32_t chunk;  // slots per thread of the running XOR (odd: distinct banks)
    int64_t first;   // spectrum of workgroup 0
    int64_t n, n_bins;
    uint32_t n_levels;
    const int64_t* off;
    const int32_t* bin;
    const uint8_t* level;
    const uint32_t* slot;  // output row of each spectrum (NULL: its own index)
    uint32_t* out;
    uint32_t* err;
};

template <int NT>
__global__ __launch_bounds__(NT) void encode_step_kernel(StepArgs a)
{
    constexpr int NW = NT / 64;
    extern __shared__ uint32_t s_slot[];  // [chunk * NT]
    __shared__ uint32_t s_sort[NW][64];
    __shared__ uint32_t s_wave[NW];
    __shared__ uint32_t s_row[kStepSpectra];  // output row, ~0: not this kernel's
    const int t = threadIdx.x, l = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t s0 = a.first + (int64_t)blockIdx.x * kStepSpectra;
    for (uint32_t i = t; i < a.chunk * NT; i += NT) s_slot[i] = 0;
    __syncthreads();

    for (int s = w; s < kStepSpectra; s += NW) {
        const int64_t sp = s0 + s;
        const int64_t b0 = sp < a.n ? a.off[sp] : 0;
        // (offsets that descend hold no peaks, here as on the general path)
        const int64_t np = sp < a.n ? max(a.off[sp + 1] - b0, (int64_t)0) : -1;
        if (l == 0)
            s_row[s] = np < 0 || np > kStepPeaks ? ~0u : a.slot ? a.slot[sp] : (uint32_t)sp;
        if (np < 0 || np > kStepPeaks) continue;  // wave-uniform
        // a lane per peak, as k << 8 | level; one out of range is left out
        uint32_t peak = ~0u;
        bool ok = false;
        if (l < np) {
            const int32_t b = a.bin[b0 + l];
            const uint32_t j = a.level[b0 + l];
            ok = b >= 0 && (int64_t)b < a.n_bins && j < a.n_levels;
            // floor of an exact quotient: the product is below 2^40 and the
            // divisor below 2^24, so rounding cannot reach the next integer
            const double den = a.n_bins > 1 ? (double)(a.n_bins - 1) : 1.0;
            const uint32_t k = (uint32_t)floor((double)((uint64_t)a.alpha * (uint32_t)b) / den);
            if (ok) peak = (k << 8) | j;
        }
        const int n = __popcll(__ballot(ok));
        if (n < np && l == 0) atomicOr(a.err, kErrRange);
        // ascending k (spectra come in ascending bins; peaks left out go last)
        const uint32_t after = __shfl_down(peak, 1);
        if (__ballot(l < 63 && (peak >> 8) > (after >> 8))) {
            int rank = 0;
            for (int i = 0; i < (int)np; ++i) {
                const uint32_t x = __builtin_amdgcn_readlane(peak, i);
                rank += (x < peak || (x == peak && i < l)) ? 1 : 0;
            }
            if (l < np) s_sort[w][rank] = peak;
            __builtin_amdgcn_wave_barrier();
            if (l < np) peak = s_sort[w][l];
            __builtin_amdgcn_wave_barrier();
        }
        // lane e stands for the components that the first e peaks do not flip:
        // flip ranks from the k of peak e - 1 on
        const uint32_t k_prev = __shfl_up(peak, 1) >> 8;
        const uint32_t j = peak & 255u;
        const int half = (n + 1) / 2, low = n / 2;
        // Class c = 2 (u - 1) + c0 at bit 2 Q - 1 - c. A sign bit enters the
        // word from the right: set where count < half (c0 = 0), or count >
        // floor(n/2) (c0 = 1), so the finished word is inverted.
        uint32_t word = 0;
#pragma unroll 4
        for (uint32_t u = 1; u <= a.n_levels; ++u) {
            const uint64_t below = __ballot(l < n && j < u);
            const int tot = __popcll(below);
            const int pre = (int)__builtin_amdgcn_mbcnt_hi(
                (uint32_t)(below >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)below, 0u));
            const int v = l - 2 * pre;  // count - tot
            word = __builtin_amdgcn_alignbit(word, (uint32_t)(v + (tot - half)), 31);
            word = __builtin_amdgcn_alignbit(word, (uint32_t)((low - tot) - v), 31);
        }
        word = ~word & (a.classes < 32 ? (1u << a.classes) - 1 : ~0u);
        const uint32_t prev = __shfl_up(word, 1);
        uint32_t steps = l >= 1 && l <= n ? word ^ prev : 0u;
        const uint16_t* at = a.first_off + (size_t)(steps ? k_prev : 0u) * a.classes;
        while (__ballot(steps != 0)) {  // four steps of a lane at a time, their loads together
            uint32_t slot[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                slot[i] = ~0u;
                if (steps) {
                    slot[i] = at[a.classes - 1 - (uint32_t)__builtin_ctz(steps)];
                    steps &= steps - 1;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (slot[i] != ~0u) atomicXor(s_slot + slot[i], 1u << s);
        }
        // a class whose first bit (e = 0) differs from the last (e = n) before
        const uint32_t first = __builtin_amdgcn_readlane(word, 0);
        const uint32_t last = __builtin_amdgcn_readlane(word, n);
        const uint32_t firsts = first ^ (last >> 1);
        if (l < (int)a.classes && ((firsts >> (a.classes - 1 - l)) & 1u))
            atomicXor(s_slot + a.start[l], 1u << s);
    }
    __syncthreads();

    // running XOR over the slots: each thread its run, then the runs before it
    uint32_t* mine = s_slot + t * a.chunk;
    uint32_t run = 0;
    for (uint32_t i = 0; i < a.chunk; ++i) run ^= mine[i];
    uint32_t inc = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (l >= o) inc ^= y;
    }
    if (l == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t acc = inc ^ run;
    for (int i = 0; i < w; ++i) acc ^= s_wave[i];
    for (uint32_t i = 0; i < a.chunk; ++i) {
        acc ^= mine[i];
        mine[i] = acc;
    }
    __syncthreads();

    // output word x of the 32 spectra: slots of its 32 components, transposed
    for (uint32_t x = t; x < a.words; x += NT) {
        uint32_t v[32];
        const uint4* src = (const uint4*)(a.source + x * 32);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 p = src[q];
            const uint32_t pw[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[8 * q + 2 * i] = s_slot[pw[i] & 0xFFFFu];
                v[8 * q + 2 * i + 1] = s_slot[pw[i] >> 16];
            }
        }
        transpose32(v);
#pragma unroll
        for (int s = 0; s < kStepSpectra; ++s)
            if (s_row[s] != ~0u) a.out[(size_t)s_row[s] * a.words + x] = v[s];
    }
}

struct U4 {
    uint32_t v[4];
};

// one bit-sliced full adder: a + b + c = sum + 2 carry in every bit position
// (carry = majority, one bitfield select)
__device__ __forceinline__ void full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t& sum,
                                         uint32_t& carry)
{
    const uint32_t u = a ^ b;
    sum = u ^ c;
    carry = (u & c) | (~u & a);
}

// add eight 0/1 slices to the counters (P >= 4): the low three planes act as
// carry-save accumulators of weight 1, 2 and 4 and the carry of weight 8
// ripples from plane 3 up, so the count is sum_k plane_k 2^k after every group
template <int P>
__device__ __forceinline__ void add_eight(U4 (&c)[P], const U4 (&x)[8])
{
    static_assert(P >= 4, "the carry-save tree needs planes 0..3");
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t ta, tb, fa, fb, y;
        full_add(c[0].v[e], x[0].v[e], x[1].v[e], c[0].v[e], ta);
        full_add(c[0].v[e], x[2].v[e], x[3].v[e], c[0].v[e], tb);
        full_add(c[1].v[e], ta, tb, c[1].v[e], fa);
        full_add(c[0].v[e], x[4].v[e], x[5].v[e], c[0].v[e], ta);
        full_add(c[0].v[e], x[6].v[e], x[7].v[e], c[0].v[e], tb);
        full_add(c[1].v[e], ta, tb, c[1].v[e], fb);
        full_add(c[2].v[e], fa, fb, c[2].v[e], y);
#pragma unroll
        for (int k = 3; k < P; ++k) {
            const uint32_t carry = c[k].v[e] & y;
            c[k].v[e] ^= y;
            y = carry;
        }
    }
}

// bit-sliced (count >= t) for a constant t < 2^P
template <int P>
__device__ __forceinline__ U4 at_least(const U4 (&c)[P], uint32_t t)
{
    U4 gt, eq;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        gt.v[e] = 0u;
        eq.v[e] = ~0u;
    }
#pragma unroll
    for (int k = P - 1; k >= 0; --k) {
        const bool tk = (t >> k) & 1u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (tk) {
                eq.v[e] &= c[k].v[e];
            } else {
                gt.v[e] |= eq.v[e] & c[k].v[e];
                eq.v[e] &= ~c[k].v[e];
            }
        }
    }
    U4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r.v[e] = gt.v[e] | eq.v[e];
    return r;
}

// adds the peaks [a, b) to the counters and the number of those in range to n_ok
template <int P>
__device__ __forceinline__ void count_peaks(U4 (&c)[P], uint32_t& n_ok,
                                            const uint4* __restrict__ id,
                                            const uint4* __restrict__ lv, uint32_t w4,
                                            uint32_t lane, int64_t a, int64_t b,
                                            const int32_t* __restrict__ bin,
                                            const uint8_t* __restrict__ level, int64_t n_bins,
                                            uint32_t n_levels, uint32_t* __restrict__ err)
{
    bool bad = false;
    // one group of eight peaks from p on; with `partial`, the slots from b on
    // re-read peak b - 1 and are masked off. A peak out of range adds nothing
    // and is not counted (row 0 is loaded in its place and masked off).
    auto group = [&](int64_t p, bool partial) {
        U4 x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool present = !partial || p + i < b;
            const int64_t q = present ? p + i : b - 1;
            const int32_t bi = bin[q];
            const uint32_t lj = level[q];
            const bool in_range = bi >= 0 && (int64_t)bi < n_bins && lj < n_levels;
            const bool ok = present && in_range;
            const uint4 f = id[(ok ? (size_t)bi : 0) * w4 + lane];
            const uint4 l = lv[(ok ? (size_t)lj : 0) * w4 + lane];
            const uint32_t m = ok ? ~0u : 0u;
            x[i].v[0] = (f.x ^ l.x) & m;
            x[i].v[1] = (f.y ^ l.y) & m;
            x[i].v[2] = (f.z ^ l.z) & m;
            x[i].v[3] = (f.w ^ l.w) & m;
            n_ok += ok ? 1u : 0u;
            bad |= present && !in_range;
        }
        add_eight<P>(c, x);
    };
    int64_t p = a;
    for (; p + 8 <= b; p += 8) group(p, false);
    if (p < b) group(p, true);
    if (bad && lane == 0) atomicOr(err, kErrRange);
}

template <int P>
__device__ __forceinline__ void clear(U4 (&c)[P])
{
#pragma unroll
    for (int k = 0; k < P; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) c[k].v[e] = 0u;
}

template <int P>
__device__ __forceinline__ U4 encode_one(const uint4* __restrict__ id, const uint4* __restrict__ lv,
                                         uint32_t w4, uint32_t lane, int64_t a, int64_t b,
                                         const int32_t* __restrict__ bin,
                                         const uint8_t* __restrict__ level, int64_t n_bins,
                                         uint32_t n_levels, uint32_t* __restrict__ err)
{
    U4 c[P];
    clear<P>(c);
    uint32_t n_ok = 0;
    count_peaks<P>(c, n_ok, id, lv, w4, lane, a, b, bin, level, n_bins, n_levels, err);
    return at_least<P>(c, (n_ok + 1u) / 2u);
}

// add x * w to the counters: x enters plane k for every set bit k of w
template <int P>
__device__ __forceinline__ void add_weighted(U4 (&c)[P], const U4& x, uint32_t w)
{
#pragma unroll
    for (int k0 = 0; k0 < 9; ++k0) {  // w <= 256
        if (!((w >> k0) & 1u)) continue;  // uniform over the lane group
        U4 y = x;
#pragma unroll
        for (int k = k0; k < P; ++k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t carry = c[k].v[e] & y.v[e];
                c[k].v[e] ^= y.v[e];
                y.v[e] = carry;
            }
        }
    }
}

template <int P>
__device__ __forceinline__ U4 encode_one_lsh(const uint4* __restrict__ id, uint32_t w4,
                                             uint32_t lane, int64_t a, int64_t b,
                                             const int32_t* __restrict__ bin,
                                             const uint8_t* __restrict__ level, int64_t n_bins,
                                             uint32_t n_levels, uint32_t* __restrict__ err)
{
    U4 c[P];
    clear<P>(c);
    uint32_t W = 0;
    for (int64_t p = a; p < b; ++p) {
        const int32_t bi = bin[p];
        const uint32_t lj = level[p];
        if (bi < 0 || (int64_t)bi >= n_bins || lj >= n_levels) {
            if (lane == 0) atomicOr(err, kErrRange);
            continue;
        }
        const uint4 f = id[(size_t)bi * w4 + lane];
        U4 x;
        x.v[0] = f.x;
        x.v[1] = f.y;
        x.v[2] = f.z;
        x.v[3] = f.w;
        add_weighted<P>(c, x, lj + 1u);
        W += lj + 1u;
    }
    return at_least<P>(c, (W + 1u) / 2u);
}

// Spectra of the general path by size class: kClass 0 below 64 peaks, 1 from
// 64 to 255, 2 from 256 on (wider counters). The launches write disjoint
// spectra; splitting keeps the register count, and so the occupancy, of the
// common case independent of the counters that larger spectra need. A
// workgroup looks at `look` consecutive spectra (at most kLook), lists those
// of its class and encodes them, D/128 lanes each: a launch that finds none of
// its class costs one look at the offsets (400,001 spectra, two launches that
// found none: 186 us when every lane group started for its own spectrum).
constexpr int kLook = 256;
__device__ __forceinline__ int size_class(int64_t np) { return np < 64 ? 0 : np < 256 ? 1 : 2; }

struct EncodeArgs {
    const uint4* id;
    const uint4* lv;
    uint32_t w4, per_block;  // lanes per spectrum, spectra a workgroup encodes at once
    int look;
    int64_t n;
    const int64_t* off;
    const int32_t* bin;
    const uint8_t* level;
    int64_t n_bins;
    uint32_t n_levels;
    const uint32_t* slot;
    uint4* out;
    uint32_t* err;
};

template <int kClass, bool kLsh>
__global__ __launch_bounds__(256) void encode_kernel(EncodeArgs x)
{
    __shared__ int s_found[kLook];
    __shared__ int s_count;
    const int64_t s0 = (int64_t)blockIdx.x * x.look;
    const uint32_t t = threadIdx.x;
    if (t == 0) s_count = 0;
    __syncthreads();
    for (int i = (int)t; i < x.look; i += blockDim.x)
        if (s0 + i < x.n && size_class(x.off[s0 + i + 1] - x.off[s0 + i]) == kClass)
            s_found[atomicAdd(&s_count, 1)] = i;
    __syncthreads();
    const uint32_t sub = t / x.w4;
    const uint32_t lane = t - sub * x.w4;
    if (sub >= x.per_block) return;
    for (int f = (int)sub; f < s_count; f += (int)x.per_block) {
        const int64_t s = s0 + s_found[f];
        const int64_t a = x.off[s], b = x.off[s + 1];
        auto one = [&](auto planes) {
            constexpr int P = decltype(planes)::value;
            if constexpr (kLsh)
                return encode_one_lsh<P>(x.id, x.w4, lane, a, b, x.bin, x.level, x.n_bins,
                                         x.n_levels, x.err);
            else
                return encode_one<P>(x.id, x.lv, x.w4, lane, a, b, x.bin, x.level, x.n_bins,
                                     x.n_levels, x.err);
        };
        U4 r;
        // planes for the largest count: np, or (lsh) np * 256
        if constexpr (kClass == 0)
            r = one(std::integral_constant<int, kLsh ? 14 : 6>{});
        else if constexpr (kClass == 1)
            r = one(std::integral_constant<int, kLsh ? 16 : 8>{});
        else if (!kLsh && b - a < 65536)
            r = one(std::integral_constant<int, 16>{});
        else
            r = one(std::integral_constant<int, 32>{});
        const int64_t row = x.slot ? (int64_t)x.slot[s] : s;
        x.out[(size_t)row * x.w4 + lane] = make_uint4(r.v[0], r.v[1], r.v[2], r.v[3]);
    }
}

// Few spectra: a workgroup each. Its groups of D/128 lanes take a share of the
// peaks each and add their counters up in LDS, in a tree: a share is a chain
// of one or two rounds of (bin, row) loads where a whole spectrum is six, and
// the chains are what a call of few spectra takes. One launch for all size
// classes (spectra of 256 peaks and more by the first group alone).
// Measured per call (top 50, then 150 peaks; the three launches by size class
// in brackets): 64 spectra at D = 8,192 8.5 (13.8) and 8.9 (33.7) us, 512 8.4
// (15.0) and 13.3 (50.7), 1,024 15.7 (17.6) and 24.4 (52.9); 2,048 27.8 (22.0)
// and 40.1 (60.3); at D = 2,048 1,024 11.3 (14.0) and 14.5 (36.1).
constexpr int kFewPlanes = 8;
constexpr int64_t kFewSpectra = 1024;
__global__ __launch_bounds__(256) void encode_few_kernel(EncodeArgs x)
{
    __shared__ uint4 s_c[kFewPlanes][256];
    __shared__ uint32_t s_ok[256];
    const int64_t s = blockIdx.x;
    const uint32_t t = threadIdx.x, sub = t / x.w4, lane = t - sub * x.w4;
    const int64_t a = x.off[s], b = x.off[s + 1], np = b - a;
    const int64_t row = x.slot ? (int64_t)x.slot[s] : s;
    U4 r;
    if (np >= 256) {  // uniform
        if (sub != 0) return;
        r = np < 65536 ? encode_one<16>(x.id, x.lv, x.w4, lane, a, b, x.bin, x.level, x.n_bins,
                                        x.n_levels, x.err)
                       : encode_one<32>(x.id, x.lv, x.w4, lane, a, b, x.bin, x.level, x.n_bins,
                                        x.n_levels, x.err);
    } else {
        const int64_t share = (np + x.per_block - 1) / x.per_block;
        const int64_t p0 = min(a + (int64_t)sub * share, b), p1 = min(p0 + share, b);
        U4 c[kFewPlanes];
        clear<kFewPlanes>(c);
        uint32_t n_ok = 0;
        count_peaks<kFewPlanes>(c, n_ok, x.id, x.lv, x.w4, lane, p0, p1, x.bin, x.level, x.n_bins,
                                x.n_levels, x.err);
        for (uint32_t m = x.per_block; m > 1; m = (m + 1) / 2) {  // groups left
            const uint32_t h = (m + 1) / 2;
            if (sub >= h && sub < m) {
#pragma unroll
                for (int k = 0; k < kFewPlanes; ++k)
                    s_c[k][t] = make_uint4(c[k].v[0], c[k].v[1], c[k].v[2], c[k].v[3]);
                s_ok[t] = n_ok;
            }
            __syncthreads();
            if (sub + h < m) {
                const uint32_t o = t + h * x.w4;
                U4 carry;
#pragma unroll
                for (int e = 0; e < 4; ++e) carry.v[e] = 0u;
#pragma unroll
                for (int k = 0; k < kFewPlanes; ++k) {
                    const uint4 y4 = s_c[k][o];
                    const uint32_t y[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t v = c[k].v[e] ^ y[e];
                        const uint32_t up = (c[k].v[e] & y[e]) | (v & carry.v[e]);
                        c[k].v[e] = v ^ carry.v[e];
                        carry.v[e] = up;
                    }
                }
                n_ok += s_ok[o];
            }
            // the groups that wrote are done, those that read write elsewhere
        }
        if (sub != 0) return;
        r = at_least<kFewPlanes>(c, (n_ok + 1u) / 2u);
    }
    x.out[(size_t)row * x.w4 + lane] = make_uint4(r.v[0], r.v[1], r.v[2], r.v[3]);
}

}  // namespace

bool step_encode_takes(const homs_params& p)
{
    // two bits of class per level in one word, and the slots in LDS
    return p.encoding == HOMS_ENCODING_ID_LEVEL && p.n_levels <= 16 &&
           p.id_flips + 2 * p.n_levels <= kStepSlots;
}

hipError_t launch_encode(const homs_ctx* c, int64_t n, const int64_t* off, const int32_t* bin,
                         const uint8_t* level, const uint32_t* slot, uint32_t* out,
                         hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // The step-function kernel needs 32 spectra per workgroup to fill the
    // chip, and saves row bytes: it wins from about 3,000 spectra at D = 8,192
    // (D = 8,192: 4,000 spectra 34 against 42 us, 400,000 0.45 against 2.25
    // ms; D = 2,048: 400,000 0.41 against 0.60 ms).
    const bool step = c->step.classes > 0 && n * (int64_t)c->words >= kStepWords;
    if (step) {
        const StepEncode& st = c->step;
        const uint32_t chunk = ((st.slots + kStepThreads - 1) / kStepThreads) | 1u;
        in_pieces((n + kStepSpectra - 1) / kStepSpectra, kStepThreads,
                  [&](int64_t first, int64_t count) {
            const StepArgs a{st.start, st.source, st.first_off, st.classes,
                             st.slots, st.alpha,  c->words,     chunk,
                             first * kStepSpectra, n, c->n_bins, c->p.n_levels,
                             off,      bin,       level,        slot,
                             out,      c->d_err};
            encode_step_kernel<kStepThreads>
                <<<(uint32_t)count, kStepThreads, (size_t)chunk * kStepThreads * 4, s>>>(a);
        });
    }
    const uint32_t w4 = c->words / 4;  // lanes per spectrum
    const uint32_t per_block = 256u / w4;
    auto go = [&](auto kern, int64_t look) {
        const EncodeArgs x{reinterpret_cast<const uint4*>(c->d_id),
                           reinterpret_cast<const uint4*>(c->d_level),
                           w4, per_block, (int)look, n, off, bin, level, c->n_bins,
                           c->p.n_levels, slot, reinterpret_cast<uint4*>(out), c->d_err};
        kern<<<(uint32_t)((n + look - 1) / look), per_block * w4, 0, s>>>(x);
    };
    // the common class by the spectra a workgroup encodes at once; the others
    // look further once there are thousands of workgroups
    const int64_t near = per_block, far = std::min<int64_t>(kLook, std::max(near, n / 2048));
    if (c->p.encoding == HOMS_ENCODING_LSH) {
        go(encode_kernel<0, true>, near);
        go(encode_kernel<1, true>, far);
        go(encode_kernel<2, true>, far);
        return hipGetLastError();
    }
    if (!step && n <= kFewSpectra) {
        go(encode_few_kernel, 1);
        return hipGetLastError();
    }
    if (!step) go(encode_kernel<0, false>, near);
    go(encode_kernel<1, false>, far);
    go(encode_kernel<2, false>, far);
    return hipGetLastError();
}

}  // namespace homs
