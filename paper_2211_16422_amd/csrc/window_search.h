// Candidate windows (Section 3.4) in the sorted library, and the fp4 form's
// class weights: device code shared by the planning and library kernels.
#pragma once

#include "internal.h"

namespace homs {

// tolerance in Da, or ppm of the precursor m/z: (pmz * v) / 1e6
__device__ __forceinline__ double tolerance_da(double pmz, int32_t kind, double v)
{
    return (kind == HOMS_TOL_DA) ? v : __ddiv_rn(__dmul_rn(pmz, v), 1.0e6);
}

// The rows [*lo, *hi) of a charge's run [r_lo, r_hi) of the sorted library
// with lo_b <= pmz <= hi_b: a query's candidates. Both searches run together,
// each with three pivots a round whose loads are in flight at once: a search
// is a chain of dependent loads, and 2^20 rows take 10 rounds of six loads
// where two binary searches over all charges took 42 of two.
__device__ __forceinline__ void window_bounds(const double* __restrict__ pmz, int64_t r_lo,
                                              int64_t r_hi, double lo_b, double hi_b, int64_t* lo,
                                              int64_t* hi)
{
    int64_t l0 = r_lo, r0 = r_hi, l1 = r_lo, r1 = r_hi;
    while (l0 < r0 || l1 < r1) {
        int64_t p0[3], p1[3];
        double m0[3], m1[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            p0[i] = l0 + (((r0 - l0) * (i + 1)) >> 2);
            p1[i] = l1 + (((r1 - l1) * (i + 1)) >> 2);
            // a finished search (l == r, maybe the end) re-reads the other's rows
            m0[i] = pmz[l0 < r0 ? p0[i] : p1[i]];
            m1[i] = pmz[l1 < r1 ? p1[i] : p0[i]];
        }
        // rows before a bound come first
        if (l0 < r0) {
            if (!(m0[0] < lo_b)) {
                r0 = p0[0];
            } else if (!(m0[1] < lo_b)) {
                l0 = p0[0] + 1;
                r0 = p0[1];
            } else if (!(m0[2] < lo_b)) {
                l0 = p0[1] + 1;
                r0 = p0[2];
            } else {
                l0 = p0[2] + 1;
            }
        }
        if (l1 < r1) {
            if (!(m1[0] <= hi_b)) {
                r1 = p1[0];
            } else if (!(m1[1] <= hi_b)) {
                l1 = p1[0] + 1;
                r1 = p1[1];
            } else if (!(m1[2] <= hi_b)) {
                l1 = p1[1] + 1;
                r1 = p1[2];
            } else {
                l1 = p1[2] + 1;
            }
        }
    }
    *lo = l0;
    *hi = l1 < l0 ? l0 : l1;  // NaN precursor or negative tolerance: empty
}

// a charge's run in the table of run starts (first[c + 128], 257 entries)
__device__ __forceinline__ void charge_run(const uint32_t* __restrict__ first, int8_t c,
                                           int64_t* lo, int64_t* hi)
{
    *lo = first ? first[(int)c + 128] : 0;  // no table: an empty library
    *hi = first ? first[(int)c + 129] : 0;
}

// 10 |x|_0 + 6 |x|_1 + 2 |x|_2 of one packed word, |x|_m its set bits at
// components of class m (component mod 4): the terms of the fp4 form's
// constants
__device__ __forceinline__ int fp4_word_weight(uint32_t w)
{
    return 10 * __builtin_popcount(w & 0x11111111u) + 6 * __builtin_popcount(w & 0x22222222u) +
           2 * __builtin_popcount(w & 0x44444444u);
}

}  // namespace homs
