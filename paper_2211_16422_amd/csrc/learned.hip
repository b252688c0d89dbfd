// Learned shortlist: a small MLP embeds hypervectors into unit vectors,
// trained on the GPU on (query, exact top-1) pairs produced by the search
// itself; at query time it proposes the k best-scoring candidates of each
// window, which are rescored exactly by Hamming distance. Queries whose
// shortlist cannot be formed reliably fall back to the exhaustive search.
//
// Network: x (bipolar hypervector, D) -> a1 = W1 x + b1 -> h = ReLU(a1) (H)
// -> z = W2 h + b2 (E) -> e = z / sqrt(z.z + eps). Weights are fp32 masters
// with bf16 copies for the matrix-core GEMMs (fp32 accumulation). Loss:
// InfoNCE over a batch of B pairs with in-batch negatives, temperature tau.
// Optimizer: Adam (beta1 0.9, beta2 0.999, eps 1e-8).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "bits.h"
#include "gemm_bf16.h"
#include "learned.h"

namespace homs {
namespace {

using gemm::to_bf16;
constexpr int kThreads = 256;
constexpr float kEpsNorm = 1e-12f;

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kThreads - 1) / kThreads); }

// Packed rows of one training batch, both towers stacked: X [M2][words] and
// its bit transpose XT [words * 32][M2 / 32] (bit i of word j of row d is bit d
// of X row 32 j + i), the operands of the forward product and of the first
// layer's weight gradient. Row r < B is query r, row B + r reference r: rows
// of q_hv / r_hv themselves, or (sel) q_hv[q_rows[perm[step] * B + r]] and
// r_hv[r_rows[...]]. The first workgroups transpose: a thread turns one
// 32 x 32 block of bits in registers, and 4 x 16 blocks go through LDS so that
// the transposed rows are written 64 bytes at a time (in 16-byte pieces this
// kernel took 19 us of a 2,048 x 8,192 batch); the others copy rows.
struct PackArgs {
    const uint32_t* q_hv;
    const uint32_t* r_hv;
    RowSelect sel;  // q_rows == nullptr: rows as they are
};

__global__ __launch_bounds__(64) void pack_batch_kernel(int B, uint32_t words, PackArgs a,
                                                        int transposers, uint32_t* __restrict__ X,
                                                        uint32_t* __restrict__ XT)
{
    __shared__ uint32_t tile[4 * 32][17];
    const int M2 = 2 * B, mws = M2 / 32;
    auto source = [&](int r) {
        const bool ref = r >= B;
        int64_t src = ref ? r - B : r;
        if (a.sel.q_rows)
            src = (ref ? a.sel.r_rows : a.sel.q_rows)[(int64_t)a.sel.perm[a.sel.step] * B + src];
        return (ref ? a.r_hv : a.q_hv) + src * words;
    };
    if ((int)blockIdx.x >= transposers) {  // one row per workgroup
        const int r = (int)blockIdx.x - transposers;
        const uint32_t* src = source(r);
        for (uint32_t i = threadIdx.x; i < words; i += 64) X[(size_t)r * words + i] = src[i];
        return;
    }
    const int bx = (int)blockIdx.x % (int)(words / 4), by = (int)blockIdx.x / (int)(words / 4);
    const int c = threadIdx.x & 3, g = threadIdx.x >> 2;
    const int mw = by * 16 + g;
    if (mw < mws) {
        uint32_t v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = source(mw * 32 + i)[bx * 4 + c];
        transpose32(v);
#pragma unroll
        for (int i = 0; i < 32; ++i) tile[c * 32 + i][g] = v[i];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 4 * 32 * 16; i += 64) {
        const int d = i >> 4, j = i & 15;
        if (by * 16 + j < mws) XT[((size_t)bx * 128 + d) * mws + by * 16 + j] = tile[d][j];
    }
}

// bf16 [R][C] -> bf16 [C][R], 32 x 32 tiles through LDS; up to two matrices
// in one launch (tiles of the first, then of the second)
struct Transpose {
    int R, C;
    const uint16_t* in;
    uint16_t* out;
    __host__ __device__ int tiles() const { return ((R + 31) / 32) * ((C + 31) / 32); }
};
__global__ void transpose_bf16_kernel(Transpose a, Transpose b)
{
    __shared__ uint16_t tile[32][33];
    int at = (int)blockIdx.x;
    const bool second = at >= a.tiles();
    const Transpose x = second ? b : a;
    if (second) at -= a.tiles();
    const int across = (x.C + 31) / 32;
    const int c0 = at % across * 32, r0 = at / across * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: 8 rows per pass
    for (int i = ty; i < 32; i += 8) {
        const int r = r0 + i, c = c0 + tx;
        tile[i][tx] = (r < x.R && c < x.C) ? x.in[(size_t)r * x.C + c] : (uint16_t)0;
    }
    __syncthreads();
    for (int i = ty; i < 32; i += 8) {
        const int c = c0 + i, r = r0 + tx;
        if (c < x.C && r < x.R) x.out[(size_t)c * x.R + r] = tile[tx][i];
    }
}
inline void transpose(hipStream_t s, Transpose a, Transpose b = {0, 0, nullptr, nullptr})
{
    transpose_bf16_kernel<<<(unsigned)(a.tiles() + b.tiles()), 256, 0, s>>>(a, b);
}

// unit embedding rows: e = z / sqrt(z.z + eps); one wave per row. With eb8,
// the scoring embeddings: eb8 = E4M3 code of kScoreScale e and eb = that
// value / kScoreScale (exact in bf16); otherwise eb = bf16(e).
__global__ void normalize_kernel(int64_t M, int E, const float* __restrict__ z,
                                 float* __restrict__ e, uint16_t* __restrict__ eb,
                                 float* __restrict__ s, float* __restrict__ out_f32,
                                 uint8_t* __restrict__ eb8 = nullptr)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (row >= M) return;
    const float* zr = z + row * E;
    float ss = 0.f;
    for (int j = l; j < E; j += 64) ss += zr[j] * zr[j];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    const float sc = sqrtf(ss + kEpsNorm);
    for (int j = l; j < E; j += 64) {
        const float v = zr[j] / sc;
        if (e) e[row * E + j] = v;
        if (eb8) {
            const uint32_t c = to_e4m3(v * kScoreScale);
            eb8[row * E + j] = (uint8_t)c;
            if (eb) eb[row * E + j] = to_bf16(from_e4m3(c) * (1.f / kScoreScale));
        } else if (eb) {
            eb[row * E + j] = to_bf16(v);
        }
        if (out_f32) out_f32[row * E + j] = v;
    }
    if (s && l == 0) s[row] = sc;
}

// InfoNCE over logits S [B][B] (already divided by tau): per row softmax,
// row_loss = (logsumexp - S_ii) / B (summed by colsum_final_kernel: an atomic
// per row on one address took longer than the rows), dS = (P - I) / B stored
// as bf16. One workgroup per row.
__global__ void info_nce_kernel(int B, const float* __restrict__ S, uint16_t* __restrict__ dS,
                                float* __restrict__ row_loss)
{
    extern __shared__ float row[];  // the row's logits, read once
    __shared__ float red[kThreads / 64];
    const int i = blockIdx.x;
    float mx = -INFINITY;
    for (int j = threadIdx.x; j < B; j += kThreads) {
        row[j] = S[(size_t)i * B + j];
        mx = fmaxf(mx, row[j]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float sum = 0.f;
    for (int j = threadIdx.x; j < B; j += kThreads) sum += __expf(row[j] - mx);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    sum = red[0] + red[1] + red[2] + red[3];
    for (int j = threadIdx.x; j < B; j += kThreads) {
        const float p = __expf(row[j] - mx) / sum;
        const float g = (p - (j == i ? 1.f : 0.f)) / (float)B;
        dS[(size_t)i * B + j] = to_bf16(g);
    }
    if (threadIdx.x == 0) row_loss[i] = (logf(sum) + mx - row[i]) / (float)B;
}

// dz = (dE - e (e.dE)) / s, one wave per row; fp32 and bf16 copies
__global__ void normalize_backward_kernel(int64_t M, int E, const float* __restrict__ e,
                                          const float* __restrict__ s,
                                          const float* __restrict__ dE, float* __restrict__ dz,
                                          uint16_t* __restrict__ dzb)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (row >= M) return;
    float dot = 0.f;
    for (int j = l; j < E; j += 64) dot += e[row * E + j] * dE[row * E + j];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
    const float sc = s[row];
    for (int j = l; j < E; j += 64) {
        const float v = (dE[row * E + j] - e[row * E + j] * dot) / sc;
        dz[row * E + j] = v;
        dzb[row * E + j] = to_bf16(v);
    }
}

// column sums of two fp32 matrices of M rows (Na and Nb columns) in two
// deterministic passes: partial sums of kColRows-row slabs (grid.y = slab),
// then the slabs in order; sums keep their order, with the loads of 16 rows
// in flight. The second pass also sums the batch's loss.
constexpr int kColRows = 128;

__global__ void colsum_partial_kernel(int M, int Na, int Nb, const float* __restrict__ a,
                                      const float* __restrict__ b, float* __restrict__ part)
{
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= Na + Nb) return;
    const float* col = n < Na ? a + n : b + (n - Na);
    const int ld = n < Na ? Na : Nb;
    const int m0 = blockIdx.y * kColRows, m1 = min(m0 + kColRows, M);
    float acc = 0.f;
#pragma unroll 16
    for (int m = m0; m < m1; ++m) acc += col[(size_t)m * ld];
    part[(size_t)blockIdx.y * (Na + Nb) + n] = acc;
}

__global__ void colsum_final_kernel(int P, int Na, int Nb, const float* __restrict__ part,
                                    float* __restrict__ out_a, float* __restrict__ out_b, int B,
                                    const float* __restrict__ row_loss, float* __restrict__ loss)
{
    if (blockIdx.x + 1 == gridDim.x) {  // the last one-wave workgroup: the batch's loss
        float sum = 0.f;
        for (int i = threadIdx.x; i < B; i += 64) sum += row_loss[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (threadIdx.x == 0) *loss = sum;
        return;
    }
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= Na + Nb) return;
    float acc = 0.f;
#pragma unroll 16
    for (int p = 0; p < P; ++p) acc += part[(size_t)p * (Na + Nb) + n];
    (n < Na ? out_a[n] : out_b[n - Na]) = acc;
}

inline void colsums(int M, int Na, int Nb, const float* a, const float* b, float* part,
                    float* out_a, float* out_b, int B, const float* row_loss, float* loss,
                    hipStream_t s)
{
    const int P = (M + kColRows - 1) / kColRows;
    const unsigned blocks = (unsigned)((Na + Nb + 63) / 64);
    colsum_partial_kernel<<<dim3(blocks, (unsigned)P), 64, 0, s>>>(M, Na, Nb, a, b, part);
    colsum_final_kernel<<<blocks + 1, 64, 0, s>>>(P, Na, Nb, part, out_a, out_b, B, row_loss,
                                                  loss);
}

// Adam over the four parameter arrays, four elements per thread (every
// array's size is a multiple of 4); wb: the bf16 copy
struct AdamArray {
    float* w;
    const float* g;
    float* m;
    float* v;
    uint16_t* wb;
    int64_t quads;
};
struct AdamArrays {
    AdamArray a[4];
};
__global__ __launch_bounds__(kThreads) void adam_kernel(AdamArrays all, float lr, float c1,
                                                        float c2)
{
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const AdamArray& p = all.a[k];
        if (i < p.quads) {
            const float4 g4 = ((const float4*)p.g)[i];
            float4 m4 = ((float4*)p.m)[i], v4 = ((float4*)p.v)[i], w4 = ((float4*)p.w)[i];
            uint32_t b[4];
            auto one = [&](float gi, float& m, float& v, float& w, uint32_t& bf) {
                const float mi = 0.9f * m + 0.1f * gi;
                const float vi = 0.999f * v + 0.001f * gi * gi;
                m = mi;
                v = vi;
                w = w - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
                bf = to_bf16(w);
            };
            one(g4.x, m4.x, v4.x, w4.x, b[0]);
            one(g4.y, m4.y, v4.y, w4.y, b[1]);
            one(g4.z, m4.z, v4.z, w4.z, b[2]);
            one(g4.w, m4.w, v4.w, w4.w, b[3]);
            ((float4*)p.m)[i] = m4;
            ((float4*)p.v)[i] = v4;
            ((float4*)p.w)[i] = w4;
            if (p.wb) ((uint2*)p.wb)[i] = make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
            return;
        }
        i -= p.quads;
    }
}

__global__ void to_bf16_kernel(int64_t n, const float* __restrict__ a, uint16_t* __restrict__ b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = to_bf16(a[i]);
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

// ---------------------------------------------------------------------------
// model lifetime and weights

void model_free(homs_model* m)
{
    for (void* p : {(void*)m->W1, (void*)m->b1, (void*)m->W2, (void*)m->b2, (void*)m->mW1,
                    (void*)m->vW1, (void*)m->mb1, (void*)m->vb1, (void*)m->mW2, (void*)m->vW2,
                    (void*)m->mb2, (void*)m->vb2, (void*)m->W1h, (void*)m->W2h, (void*)m->W2Th,
                    (void*)m->gW1, (void*)m->gb1, (void*)m->gW2, (void*)m->gb2, m->train_ws,
                    m->emb_ws, (void*)m->lib_emb, (void*)m->lib_emb8, (void*)m->loss_scratch})
        if (p) (void)hipFree(p);
}

hipError_t model_alloc(homs_model* m)
{
    const size_t n1 = (size_t)m->H * m->D, n2 = (size_t)m->E * m->H;
    hipError_t e = hipSuccess;
    auto A = [&](void** p, size_t bytes) {
        if (e == hipSuccess) e = dev_malloc(p, bytes);
        if (e == hipSuccess) e = hipMemset(*p, 0, bytes);
    };
    A((void**)&m->W1, n1 * 4);
    A((void**)&m->b1, m->H * 4);
    A((void**)&m->W2, n2 * 4);
    A((void**)&m->b2, m->E * 4);
    A((void**)&m->mW1, n1 * 4);
    A((void**)&m->vW1, n1 * 4);
    A((void**)&m->mb1, m->H * 4);
    A((void**)&m->vb1, m->H * 4);
    A((void**)&m->mW2, n2 * 4);
    A((void**)&m->vW2, n2 * 4);
    A((void**)&m->mb2, m->E * 4);
    A((void**)&m->vb2, m->E * 4);
    A((void**)&m->W1h, n1 * 2);
    A((void**)&m->W2h, n2 * 2);
    A((void**)&m->W2Th, n2 * 2);
    A((void**)&m->gW1, n1 * 4);
    A((void**)&m->gb1, m->H * 4);
    A((void**)&m->gW2, n2 * 4);
    A((void**)&m->gb2, m->E * 4);
    A((void**)&m->loss_scratch, 256);
    return e;
}

// bf16 copies of the weights (and W2 transposed) from the fp32 masters
hipError_t model_refresh_bf16(homs_model* m, hipStream_t s)
{
    const int64_t n1 = (int64_t)m->H * m->D, n2 = (int64_t)m->E * m->H;
    to_bf16_kernel<<<blocks_for(n1), kThreads, 0, s>>>(n1, m->W1, m->W1h);
    to_bf16_kernel<<<blocks_for(n2), kThreads, 0, s>>>(n2, m->W2, m->W2h);
    transpose(s, {m->E, m->H, m->W2h, m->W2Th});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// embedding inference: n packed rows -> unit embeddings (fp32 and/or bf16)

size_t embed_ws_bytes(const homs_model* m, int64_t rows)
{
    return al(rows * m->H * 2) + al(rows * m->E * 4);
}

hipError_t model_embed(homs_model* m, int64_t n, const uint32_t* hv, float* out_f32,
                       uint16_t* out_bf16, uint8_t* out_fp8, hipStream_t s)
{
    const int64_t rows = std::min<int64_t>(n, kEmbedBatch);
    if (n <= 0) return hipSuccess;
    const size_t need = embed_ws_bytes(m, rows);
    if (m->emb_ws_bytes < need) {
        hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        if (m->emb_ws) (void)hipFree(m->emb_ws);
        m->emb_ws = nullptr;
        m->emb_ws_bytes = 0;
        e = dev_malloc(&m->emb_ws, need);
        if (e != hipSuccess) return e;
        m->emb_ws_bytes = need;
    }
    uint16_t* hb = (uint16_t*)m->emb_ws;
    float* z = (float*)((char*)m->emb_ws + al(rows * m->H * 2));
    const int words = m->D / 32;
    for (int64_t r0 = 0; r0 < n; r0 += rows) {
        const int64_t nr = std::min(rows, n - r0);
        using namespace gemm;
        Out h;
        h.bias = m->b1;
        h.Cb = hb;
        h.ldcb = m->H;
        hipError_t e = gemm_nt<kBias | kStoreBf16 | kReluBf16>(
            s, (int)nr, m->H, m->D, Bits{hv + r0 * words, words}, Bf16{m->W1h, m->D}, h);
        if (e != hipSuccess) return e;
        Out zo;
        zo.bias = m->b2;
        zo.C = z;
        zo.ldc = m->E;
        e = gemm_nt<kBias | kStoreF32>(s, (int)nr, m->E, m->H, Bf16{hb, m->H},
                                       Bf16{m->W2h, m->H}, zo);
        if (e != hipSuccess) return e;
        normalize_kernel<<<(uint32_t)((nr + 3) / 4), 256, 0, s>>>(
            nr, m->E, z, nullptr, out_bf16 ? out_bf16 + r0 * m->E : nullptr, nullptr,
            out_f32 ? out_f32 + r0 * m->E : nullptr, out_fp8 ? out_fp8 + r0 * m->E : nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// one training step (forward, loss, backward; Adam when `update`)

size_t train_ws_bytes(const homs_model* m, int B)
{
    const size_t M2 = 2 * (size_t)B, D = m->D, H = m->H, E = m->E;
    return 2 * al(M2 * D / 8) + al(M2 * H * 4) + 2 * al(M2 * H * 2) + 3 * al(M2 * E * 4) +
           al(M2 * E * 2) + al(M2 * 4) + al(E * M2 * 2) + al((size_t)B * B * 4) +
           2 * al((size_t)B * B * 2) + al(M2 * E * 4) + al(M2 * E * 2) + al(E * M2 * 2) +
           al(M2 * H * 4) + al(H * M2 * 2) +
           al(((M2 + kColRows - 1) / kColRows) * (H + E) * 4) + al((size_t)B * 4);
}

hipError_t model_step(homs_model* m, int B, const uint32_t* q_hv, const uint32_t* r_hv, float tau,
                      float lr, bool update, float* loss, hipStream_t s, const RowSelect* sel)
{
    const int M2 = 2 * B, D = m->D, H = m->H, E = m->E;
    const uint32_t words = (uint32_t)(D / 32);
    const size_t need = train_ws_bytes(m, B);
    if (m->train_ws_bytes < need) {
        hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        if (m->train_ws) (void)hipFree(m->train_ws);
        m->train_ws = nullptr;
        m->train_ws_bytes = 0;
        e = dev_malloc(&m->train_ws, need);
        if (e != hipSuccess) return e;
        m->train_ws_bytes = need;
    }
    char* p = (char*)m->train_ws;
    auto take = [&](size_t bytes) {
        void* r = p;
        p += al(bytes);
        return r;
    };
    uint32_t* X = (uint32_t*)take((size_t)M2 * D / 8);
    uint32_t* XT = (uint32_t*)take((size_t)M2 * D / 8);
    float* a1 = (float*)take((size_t)M2 * H * 4);
    uint16_t* hb = (uint16_t*)take((size_t)M2 * H * 2);
    uint16_t* hT = (uint16_t*)take((size_t)M2 * H * 2);
    float* z = (float*)take((size_t)M2 * E * 4);
    float* e = (float*)take((size_t)M2 * E * 4);
    float* dz = (float*)take((size_t)M2 * E * 4);
    uint16_t* eb = (uint16_t*)take((size_t)M2 * E * 2);
    float* sc = (float*)take((size_t)M2 * 4);
    uint16_t* eT = (uint16_t*)take((size_t)E * M2 * 2);
    float* S = (float*)take((size_t)B * B * 4);
    uint16_t* dS = (uint16_t*)take((size_t)B * B * 2);
    uint16_t* dST = (uint16_t*)take((size_t)B * B * 2);
    float* dE = (float*)take((size_t)M2 * E * 4);
    uint16_t* dzb = (uint16_t*)take((size_t)M2 * E * 2);
    uint16_t* dzT = (uint16_t*)take((size_t)E * M2 * 2);
    float* da1 = (float*)take((size_t)M2 * H * 4);
    uint16_t* da1T = (uint16_t*)take((size_t)H * M2 * 2);
    float* colpart = (float*)take((size_t)((M2 + kColRows - 1) / kColRows) * (H + E) * 4);
    float* row_loss = (float*)take((size_t)B * 4);

    using namespace gemm;
    hipError_t err = hipSuccess;
#define STEP(x)                              \
    do {                                     \
        err = (x);                           \
        if (err != hipSuccess) return err;   \
    } while (0)
    // forward, both towers stacked: rows [0, B) queries, [B, 2B) references
    const PackArgs pack{q_hv, r_hv, sel ? *sel : RowSelect{nullptr, nullptr, nullptr, 0}};
    const int transposers = (int)(words / 4) * ((M2 / 32 + 15) / 16);
    pack_batch_kernel<<<(unsigned)(transposers + M2), 64, 0, s>>>(B, words, pack, transposers, X,
                                                                  XT);
    {
        Out o;
        o.bias = m->b1;
        o.C = a1;
        o.ldc = H;
        o.Cb = hb;
        o.ldcb = H;
        o.Ct = hT;
        o.ldct = M2;
        STEP(gemm_nt<kBias | kStoreF32 | kStoreBf16 | kReluBf16 | kStoreT>(
            s, M2, H, D, Bits{X, (int)words}, Bf16{m->W1h, D}, o));
    }
    {
        Out o;
        o.bias = m->b2;
        o.C = z;
        o.ldc = E;
        STEP(gemm_nt<kBias | kStoreF32>(s, M2, E, H, Bf16{hb, H}, Bf16{m->W2h, H}, o));
    }
    normalize_kernel<<<(uint32_t)((M2 + 3) / 4), 256, 0, s>>>(M2, E, z, e, eb, sc, nullptr);
    // logits and loss
    {
        Out o;
        o.alpha = 1.f / tau;
        o.C = S;
        o.ldc = B;
        STEP(gemm_nt<kStoreF32>(s, B, B, E, Bf16{eb, E}, Bf16{eb + (size_t)B * E, E}, o));
    }
    info_nce_kernel<<<B, kThreads, (size_t)B * 4, s>>>(B, S, dS, row_loss);
    // dE_q = dS E_r / tau, dE_r = dS^T E_q / tau (B operands are E^T slices)
    transpose(s, {B, B, dS, dST}, {M2, E, eb, eT});
    {
        Out o;
        o.alpha = 1.f / tau;
        o.C = dE;
        o.ldc = E;
        o.batch = 2;
        o.nextA = dST - dS;
        o.nextB = -B;
        o.nextC = (int64_t)B * E;
        STEP(gemm_nt<kStoreF32>(s, B, E, B, Bf16{dS, B}, Bf16{eT + B, M2}, o));
    }
    normalize_backward_kernel<<<(uint32_t)((M2 + 3) / 4), 256, 0, s>>>(M2, E, e, sc, dE, dz, dzb);
    transpose(s, {M2, E, dzb, dzT});
    {  // dW2 = dz^T h
        Out o;
        o.C = m->gW2;
        o.ldc = H;
        STEP(gemm_nt<kStoreF32>(s, E, H, M2, Bf16{dzT, M2}, Bf16{hT, M2}, o));
    }
    {  // da1 = (dz W2) * [a1 > 0]
        Out o;
        o.mask = a1;
        o.C = da1;
        o.ldc = H;
        o.Ct = da1T;
        o.ldct = M2;
        STEP(gemm_nt<kMask | kStoreF32 | kStoreT>(s, M2, H, E, Bf16{dzb, E}, Bf16{m->W2Th, E}, o));
    }
    colsums(M2, E, H, dz, da1, colpart, m->gb2, m->gb1, B, row_loss, loss, s);
    {  // dW1 = da1^T X
        Out o;
        o.C = m->gW1;
        o.ldc = D;
        STEP(gemm_nt<kStoreF32>(s, H, D, M2, Bf16{da1T, M2}, Bits{XT, M2 / 32}, o));
    }
    STEP(hipGetLastError());
    if (!update) return hipSuccess;
    m->step += 1;
    const float c1 = 1.f - powf(0.9f, (float)m->step), c2 = 1.f - powf(0.999f, (float)m->step);
    AdamArrays all{{{m->W1, m->gW1, m->mW1, m->vW1, m->W1h, (int64_t)H * D / 4},
                    {m->W2, m->gW2, m->mW2, m->vW2, m->W2h, (int64_t)E * H / 4},
                    {m->b1, m->gb1, m->mb1, m->vb1, nullptr, H / 4},
                    {m->b2, m->gb2, m->mb2, m->vb2, nullptr, E / 4}}};
    int64_t quads = 0;
    for (const AdamArray& p : all.a) quads += p.quads;
    adam_kernel<<<blocks_for(quads), kThreads, 0, s>>>(all, lr, c1, c2);
    transpose(s, {E, H, m->W2h, m->W2Th});
#undef STEP
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// training schedule over (query, reference) pairs

namespace {

// output k (0-based) of the SplitMix64 stream started at `seed` (Steele, Lea,
// Flood, OOPSLA 2014): the state after k + 1 increments of the golden gamma,
// through the generator's output mix
__device__ __forceinline__ uint64_t splitmix64_output(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// pair k -> key = sorted library row of its reference (2^32 - 1 when the
// index is outside the library), value = k; counts the valid pairs
__global__ void pair_keys_kernel(int64_t n, const int64_t* __restrict__ target,
                                 const uint32_t* __restrict__ slot, int64_t nlib,
                                 uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                 unsigned long long* __restrict__ n_valid)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = k < n;
    const int64_t t = in ? target[k] : -1;
    const bool valid = t >= 0 && t < nlib;
    if (in) {
        keys[k] = valid ? (uint64_t)slot[t] : 0xFFFFFFFFull;
        vals[k] = (uint32_t)k;
    }
    const uint64_t m = __ballot(valid);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(n_valid, (unsigned long long)__popcll(m));
}

// ordered pair j -> its query row and its reference's sorted library row
__global__ void pair_rows_kernel(int64_t n, const uint64_t* __restrict__ keys,
                                 const uint32_t* __restrict__ vals, uint32_t* __restrict__ q_rows,
                                 uint32_t* __restrict__ r_rows)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    q_rows[j] = vals[j];
    r_rows[j] = (uint32_t)keys[j];
}

// batch b of epoch e -> key = SplitMix64 output e * nb + b, value = b
__global__ void epoch_keys_kernel(int64_t nb, int64_t epoch, uint64_t seed,
                                  uint64_t* __restrict__ keys, uint32_t* __restrict__ vals)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    keys[b] = splitmix64_output(seed, (uint64_t)(epoch * nb + b));
    vals[b] = (uint32_t)b;
}

}  // namespace

hipError_t model_train(homs_model* m, int64_t n, const uint32_t* q_hv, const int64_t* target,
                       int epochs, int B, float lr, float tau, uint64_t seed, float* losses,
                       int64_t* steps_out, hipStream_t s)
{
    *steps_out = 0;
    const homs_ctx* c = m->ctx;
    const int64_t cap = n > 1 ? n : 1;
    const size_t sort_tmp = radix_sort_temp_bytes(cap);
    const size_t need = 2 * al((size_t)cap * 8) + 4 * al((size_t)cap * 4) + al(sort_tmp) + al(8);
    char* base = nullptr;
    hipError_t e = dev_malloc((void**)&base, need);
    if (e != hipSuccess) return e;
    char* p = base;
    auto take = [&](size_t bytes) {
        void* r = p;
        p += al(bytes);
        return r;
    };
    uint64_t* ka = (uint64_t*)take((size_t)cap * 8);
    uint64_t* kb = (uint64_t*)take((size_t)cap * 8);
    uint32_t* va = (uint32_t*)take((size_t)cap * 4);
    uint32_t* vb = (uint32_t*)take((size_t)cap * 4);
    uint32_t* q_rows = (uint32_t*)take((size_t)cap * 4);
    uint32_t* r_rows = (uint32_t*)take((size_t)cap * 4);
    void* tmp = take(sort_tmp);
    unsigned long long* d_valid = (unsigned long long*)take(8);
    unsigned long long n_valid = 0;
    int64_t nb = 0;
    bool alt = false;

    e = hipMemsetAsync(d_valid, 0, 8, s);
    if (e == hipSuccess && n > 0) {
        pair_keys_kernel<<<blocks_for(n), kThreads, 0, s>>>(n, target, c->lib.slot, c->lib.n, ka,
                                                            va, d_valid);
        // stable: pairs of one reference keep their input order
        e = radix_sort_pairs(n, ka, kb, va, vb, 0, 32, tmp, s, &alt);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&n_valid, d_valid, 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) {
        nb = (int64_t)n_valid / B;
        if (nb > 0) {
            // invalid pairs sorted last; the last partial batch is dropped
            pair_rows_kernel<<<blocks_for(nb * B), kThreads, 0, s>>>(
                nb * B, alt ? kb : ka, alt ? vb : va, q_rows, r_rows);
            e = hipGetLastError();
        }
    }
    for (int ep = 0; ep < epochs && e == hipSuccess && nb > 0; ++ep) {
        epoch_keys_kernel<<<blocks_for(nb), kThreads, 0, s>>>(nb, ep, seed, ka, va);
        e = radix_sort_pairs(nb, ka, kb, va, vb, 0, 64, tmp, s, &alt);
        const uint32_t* perm = alt ? vb : va;
        for (int64_t j = 0; j < nb && e == hipSuccess; ++j) {
            const RowSelect sel{q_rows, r_rows, perm, j};
            e = model_step(m, B, q_hv, c->lib.hv, tau, lr, true,
                           losses ? losses + (int64_t)ep * nb + j : m->loss_scratch, s, &sel);
        }
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(base);
    if (e == hipSuccess) *steps_out = (int64_t)epochs * nb;
    return e;
}

}  // namespace homs
