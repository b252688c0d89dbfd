// bf16 matrix-core GEMM used by the learned shortlist:
//     C[m][n] = alpha * sum_k A[m][k] * B[n][k]   (+ epilogue)
// with K contiguous in both operands ("NT"), fp32 accumulation on
// v_mfma_f32_32x32x16_bf16 in ascending k. Either operand may be a packed bit
// matrix (bit 0 = +1, bit 1 = -1: the bipolar hypervectors), expanded to
// +-1.0 in registers right before the matrix instruction, so the hypervectors
// are never written out as bf16. K must be a multiple of 32; M and N are
// arbitrary (loads clamp, stores mask).
//
// A workgroup of WM x WN waves, each owning TR x TC tiles of 32 x 32, walks K
// in stages of KS = 64 (32 when K is no multiple of 64). A stage's rows move
// into one of three LDS buffers by direct global-to-LDS loads, two stages
// ahead of their use; one barrier per stage publishes the landed stage and
// frees the one before it. bf16 rows: the 16-byte piece p of row r sits at
// position p ^ f(r) (mfma_direct.h's swizzle), so that the 16 rows a
// quarter-wave reads together fall in 16 bank groups. Bit rows: word j of the
// stage of all rows, then word j + 1 (consecutive lanes read consecutive
// words).
//
// Operand layout of 32x32x16 bf16 (checked on gfx950): lane l supplies row
// (l % 32) and the 8 consecutive k of group (l / 32); accumulator register r
// of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
#pragma once

#include <type_traits>

#include "internal.h"

namespace homs {
namespace gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

enum Epi : int {
    kBias = 1,       // + bias[n]
    kRelu = 2,       // max(., 0)
    kMask = 4,       // * (mask[m][n] > 0), mask fp32 with C's layout
    kStoreF32 = 8,   // C (fp32, ldc)
    kStoreBf16 = 16, // Cb (bf16, ldcb)
    kReluBf16 = 32,  // ReLU applied to the bf16 stores only (C keeps the pre-activation)
    kStoreT = 64     // Ct: the bf16 result transposed ([n][m], ldct)
};

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    // round to nearest even; inputs here are finite
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// An operand: bf16 rows (ld in elements) or packed bit rows (ld in words).
struct Bf16 {
    static constexpr bool kBits = false;
    const uint16_t* p;
    int ld;
};
struct Bits {
    static constexpr bool kBits = true;
    const uint32_t* p;
    int ld;
};

// s_waitcnt immediate: vmcnt(n), expcnt and lgkmcnt left at their maxima
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70 | 0xF00; }

// One side of a workgroup's stage: R rows of an operand, NW waves.
template <class Op, int R, int KS, int NW>
struct Side {
    static constexpr int kRow = KS * 2;                // bf16: bytes of a row and stage
    static constexpr int kP = kRow / 16;               // 16-byte pieces of it
    static constexpr int kRPB = 16 / kP;               // rows between repeats of the banks
    static constexpr int kBytes = Op::kBits ? R * KS / 8 : R * kRow;
    static constexpr int kInstr = Op::kBits ? (R / 64) * (KS / 32) : R * kRow / 1024;
    static constexpr int kPerWave = (kInstr + NW - 1) / NW;
    static_assert(R % 64 == 0, "whole load instructions");
    uint32_t voff[kPerWave];  // this lane's byte offsets from the stage's first word
    uint32_t dst[kPerWave];   // LDS offsets, wave-uniform

    // rows past the operand's last one repeat it; waves past the last
    // instruction repeat that one (same bytes to the same place), so every
    // wave waits for the same number of loads
    __device__ __forceinline__ void init(const Op& op, int row0, int rows, int w, int l)
    {
#pragma unroll
        for (int x = 0; x < kPerWave; ++x) {
            const int i = min(w + x * NW, kInstr - 1);
            if constexpr (Op::kBits) {
                const int j = i / (R / 64), row = i % (R / 64) * 64 + l;
                voff[x] = (uint32_t)(min(row, rows - 1 - row0) * op.ld + j) * 4u;
                dst[x] = (uint32_t)i * 256u;
            } else {
                const int row = i * (64 / kP) + l / kP;
                const int piece = (l % kP) ^ ((row / kRPB) % kP);
                voff[x] = (uint32_t)(min(row, rows - 1 - row0) * op.ld + piece * 8) * 2u;
                dst[x] = (uint32_t)i * 1024u;
            }
        }
    }
    // bytes from one stage of a row to the next
    static constexpr uint32_t kStep = Op::kBits ? KS / 8 : kRow;
    __device__ __forceinline__ static const char* start(const Op& op, int row0)
    {
        return (const char*)(op.p + (size_t)row0 * op.ld);
    }
    // the stage at `base` (wave-uniform) into the LDS bytes at `lds`
    __device__ __forceinline__ void issue(const char* base, uint32_t lds) const
    {
#pragma unroll
        for (int x = 0; x < kPerWave; ++x) {
            const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds + dst[x]);
            if constexpr (Op::kBits)
                asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1"
                             :
                             : "v"(voff[x]), "s"(base), "s"(m0)
                             : "memory", "m0");
            else
                asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                             :
                             : "v"(voff[x]), "s"(base), "s"(m0)
                             : "memory", "m0");
        }
    }
};

// 8 bits (the low byte of b) -> eight +-1.0 in bf16: the sign bit of value i
// is bit i. Even bits stay, odd bits move up 16 places less one, so one shift
// brings a pair's bits to the two sign positions of a dword.
__device__ __forceinline__ bf16x8 expand8(uint32_t b, uint32_t sel, uint32_t one)
{
    const uint32_t y = (b & 0x55u) | ((b & 0xAAu) << 15);
    union {
        uint32_t d[4];
        bf16x8 v;
    } o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t x = y << (15 - 2 * j);
        // one operation (not inline asm: the compiler must count the wait states
        // between this write and the matrix instruction)
        o.d[j] = (sel & x) | (~sel & one);
    }
    return o.v;
}

// the operands of T 32-row tiles for one 16-wide k step of a stage in LDS
template <class Op, int R, int KS, int T>
struct Reader {
    uint32_t words[T];
    typename std::conditional<Op::kBits, uint32_t, bf16x8>::type all[KS / (Op::kBits ? 32 : 16)][T];
    // a whole stage's operands (fetch), then those of one k step (take)
    __device__ __forceinline__ void fetch(const uint8_t* lds, int row, int h)
    {
#pragma unroll
        for (int x = 0; x < KS / (Op::kBits ? 32 : 16); ++x)
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if constexpr (Op::kBits) {
                    all[x][i] = *(const uint32_t*)(lds + (x * R + row + i * 32) * 4) >> (8 * h);
                } else {
                    using S = Side<Op, R, KS, 1>;
                    const int piece = (2 * x + h) ^ ((row / S::kRPB) % S::kP);
                    all[x][i] = *(const bf16x8*)(lds + (row + i * 32) * S::kRow + piece * 16);
                }
            }
    }
    __device__ __forceinline__ void take(int kk, uint32_t sel, uint32_t one, bf16x8 (&out)[T])
    {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if constexpr (Op::kBits)
                out[i] = expand8((kk & 1) ? all[kk >> 1][i] >> 16 : all[kk >> 1][i], sel, one);
            else
                out[i] = all[kk][i];
        }
    }
    // row: this lane's row of tile 0 (tiles are 32 rows apart)
    __device__ __forceinline__ void read(const uint8_t* lds, int row, int kk, int h, uint32_t sel,
                                         uint32_t one, bf16x8 (&out)[T])
    {
        if constexpr (Op::kBits) {
            if ((kk & 1) == 0) {
#pragma unroll
                for (int i = 0; i < T; ++i)
                    words[i] = *(const uint32_t*)(lds + ((kk >> 1) * R + row + i * 32) * 4) >>
                               (8 * h);
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
                out[i] = expand8((kk & 1) ? words[i] >> 16 : words[i], sel, one);
        } else {
            using S = Side<Op, R, KS, 1>;
            const int piece = (2 * kk + h) ^ ((row / S::kRPB) % S::kP);
#pragma unroll
            for (int i = 0; i < T; ++i)
                out[i] = *(const bf16x8*)(lds + (row + i * 32) * S::kRow + piece * 16);
        }
    }
};

struct Out {
    float alpha = 1.f;
    const float* bias = nullptr;
    const float* mask = nullptr;
    float* C = nullptr;
    int ldc = 0;
    uint16_t* Cb = nullptr;
    int ldcb = 0;
    uint16_t* Ct = nullptr;
    int ldct = 0;
    // `batch` products of one shape in one launch: operand and C offsets from
    // one to the next, in elements
    int batch = 1;
    int64_t nextA = 0, nextB = 0, nextC = 0;
};

template <int EPI, class OpA, class OpB, int WM, int WN, int TR, int TC, int KS>
__global__ __launch_bounds__(64 * WM * WN, (TR * TC > 4 ? 2 : 3)) void gemm_nt_kernel(
    int M, int N, int K, OpA A, OpB B, Out o)
{
    constexpr int NW = WM * WN, kTM = WM * TR * 32, kTN = WN * TC * 32, kBufs = 3;
    using SideA = Side<OpA, kTM, KS, NW>;
    using SideB = Side<OpB, kTN, KS, NW>;
    constexpr int kLoads = SideA::kPerWave + SideB::kPerWave;
    constexpr int kStage = SideA::kBytes + SideB::kBytes;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kBufs][kStage];
    const int t = threadIdx.x, l = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wr = w % WM, wn = w / WM, h = l >> 5;
    // Workgroups go to the eight XCDs in turn: a run of consecutive tiles,
    // which share A rows, is dealt to one XCD, whose L2 then holds them.
    A.p += blockIdx.y * o.nextA;
    B.p += blockIdx.y * o.nextB;
    o.C += blockIdx.y * o.nextC;
    const int nb = (N + kTN - 1) / kTN, total = (int)gridDim.x;
    const int per = (total + 7) / 8, rest = total % 8 == 0 ? 8 : total % 8;
    const int x = (int)blockIdx.x % 8, y = (int)blockIdx.x / 8;
    const int tile = x < rest ? x * per + y : rest * per + (x - rest) * (per - 1) + y;
    const int m0 = tile / nb * kTM, n0 = tile % nb * kTN;

    SideA sa;
    SideB sb;
    sa.init(A, m0, M, w, l);
    sb.init(B, n0, N, w, l);
    uint32_t sel = 0x80008000u, one = 0x3F803F80u;
    if constexpr (OpA::kBits || OpB::kBits) asm volatile("" : "+v"(sel), "+v"(one));

    const int nk = K / KS;
    // The next stage into buffer `to`; stages past the end re-read the last one
    // into a buffer that is not read.
    const char *fa = SideA::start(A, m0), *fb = SideB::start(B, n0);
    int ahead = nk - 1;  // stages after the one at fa, fb
    auto issue = [&](int to) {
        const uint32_t at = (uint32_t)(uintptr_t)&lds[to][0];
        sa.issue(fa, at);
        sb.issue(fb, at + SideA::kBytes);
        const bool more = ahead > 0;
        fa += more ? SideA::kStep : 0;
        fb += more ? SideB::kStep : 0;
        --ahead;
    };
    f32x16 acc[TR][TC];
#pragma unroll
    for (int i = 0; i < TR; ++i)
#pragma unroll
        for (int j = 0; j < TC; ++j) acc[i][j] = f32x16{0};

    const int rowA = wr * TR * 32 + (l & 31), rowB = wn * TC * 32 + (l & 31);
    Reader<OpA, kTM, KS, TR> ra;
    Reader<OpB, kTN, KS, TC> rb;
    // A stage, in buffer `b` (a constant: the loop is unrolled over the buffers,
    // so that no address is worked out per stage; with one wave per SIMD all
    // that a stage does besides its matrix instructions adds to its time.
    // N = 1,024, K = 8,192, bits: 300 rows 51.6 -> 44.9 us, 2,048 rows 61 ->
    // 55 us with the reads below, 8,000 rows 154 -> 146 us in all; neither
    // more buffers (6) nor k split over two sets of waves gave anything)
    auto stage = [&](auto buf) {
        constexpr int b = decltype(buf)::value;
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kLoads));  // this wave's loads of the stage
        __syncthreads();  // everyone's; the stage before is fully read
        issue((b + 2) % kBufs);
        const uint8_t* pa = &lds[b][0];
        const uint8_t* pb = pa + SideA::kBytes;
        // few matrix instructions a stage: all its LDS reads first, so that
        // their latency is waited for once
        constexpr bool kFirst = TR * TC <= 2;
        if constexpr (kFirst) {
            ra.fetch(pa, rowA, h);
            rb.fetch(pb, rowB, h);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int kk = 0; kk < KS / 16; ++kk) {
            bf16x8 av[TR], bv[TC];
            if constexpr (kFirst) {
                ra.take(kk, sel, one, av);
                rb.take(kk, sel, one, bv);
            } else {
                ra.read(pa, rowA, kk, h, sel, one, av);
                rb.read(pb, rowB, kk, h, sel, one, bv);
            }
#pragma unroll
            for (int i = 0; i < TR; ++i)
#pragma unroll
                for (int j = 0; j < TC; ++j)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    };
    issue(0);
    issue(1);
    for (int s = 0; s < nk; s += 3) {
        stage(std::integral_constant<int, 0>{});
        if (s + 1 < nk) stage(std::integral_constant<int, 1>{});
        if (s + 2 < nk) stage(std::integral_constant<int, 2>{});
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // the re-reads land before the LDS is released

#pragma unroll
    for (int i = 0; i < TR; ++i)
#pragma unroll
        for (int j = 0; j < TC; ++j) {
            const int n = n0 + wn * TC * 32 + j * 32 + (l & 31);
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int mr = m0 + wr * TR * 32 + i * 32 + 8 * rg + 4 * h;
                uint32_t tb[4];
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int m = mr + r4;
                    tb[r4] = 0;
                    if (m >= M || n >= N) continue;
                    float v = o.alpha * acc[i][j][4 * rg + r4];
                    if (EPI & kBias) v += o.bias[n];
                    if (EPI & kRelu) v = v > 0.f ? v : 0.f;
                    if (EPI & kMask) v = o.mask[(size_t)m * o.ldc + n] > 0.f ? v : 0.f;
                    if (EPI & kStoreF32) o.C[(size_t)m * o.ldc + n] = v;
                    if (EPI & (kStoreBf16 | kStoreT)) {
                        const uint16_t b = to_bf16((EPI & kReluBf16) && v < 0.f ? 0.f : v);
                        if (EPI & kStoreBf16) o.Cb[(size_t)m * o.ldcb + n] = b;
                        tb[r4] = b;
                    }
                }
                if (EPI & kStoreT) {  // four consecutive m of one n (M and ldct multiples of 4)
                    if (mr < M && n < N)
                        *(uint2*)(o.Ct + (size_t)n * o.ldct + mr) =
                            make_uint2(tb[0] | (tb[1] << 16), tb[2] | (tb[3] << 16));
                }
            }
        }
}

template <int EPI, int WM, int WN, int TR, int TC, class OpA, class OpB>
inline hipError_t gemm_tile(hipStream_t s, int M, int N, int K, OpA A, OpB B, const Out& o)
{
    const int64_t tm = WM * TR * 32, tn = WN * TC * 32;
    const int64_t grid = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
    if (grid > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
    if (K % 64 == 0)
        gemm_nt_kernel<EPI, OpA, OpB, WM, WN, TR, TC, 64>
            <<<dim3((unsigned)grid, (unsigned)o.batch), 64 * WM * WN, 0, s>>>(M, N, K, A, B, o);
    else
        gemm_nt_kernel<EPI, OpA, OpB, WM, WN, TR, TC, 32>
            <<<dim3((unsigned)grid, (unsigned)o.batch), 64 * WM * WN, 0, s>>>(M, N, K, A, B, o);
    return hipGetLastError();
}

template <int EPI, class OpA, class OpB>
inline hipError_t gemm_nt(hipStream_t s, int M, int N, int K, OpA A, OpB B, const Out& o)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K % 32 != 0 || (!OpA::kBits && A.ld % 8 != 0) || (!OpB::kBits && B.ld % 8 != 0))
        return hipErrorInvalidValue;
    if ((EPI & kStoreT) && (M % 4 != 0 || o.ldct % 4 != 0)) return hipErrorInvalidValue;
    auto tiles = [&](int64_t tm, int64_t tn) { return ((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
    // The largest tile that still gives every compute unit work: the larger
    // ones read less LDS per matrix instruction, the smaller ones keep more
    // waves in flight. With bits for A, a wave of 32 x 64 expands each A
    // operand for two matrix instructions. Measured (N = 1,024, K = 8,192,
    // bits): M = 50,001: 256 x 128 0.88 ms in all, 128 x 128 0.92, 64 x 64
    // 1.48; M = 4,096: 0.140, 0.101, 0.104 (64 x 128), 0.109 (64 x 64).
    if (tiles(256, 128) >= 512) return gemm_tile<EPI, 4, 2, 2, 2>(s, M, N, K, A, B, o);
    if (tiles(128, 128) >= 256) return gemm_tile<EPI, 2, 2, 2, 2>(s, M, N, K, A, B, o);
    if constexpr (OpA::kBits)
        if (tiles(64, 128) >= 256) return gemm_tile<EPI, 2, 2, 1, 2>(s, M, N, K, A, B, o);
    return gemm_tile<EPI, 2, 2, 1, 1>(s, M, N, K, A, B, o);
}

}  // namespace gemm
}  // namespace homs
