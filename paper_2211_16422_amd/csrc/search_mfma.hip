// Open-window Hamming top-1 search on matrix cores (the precision form).
//
// With bit 0 standing for +1 and bit 1 for -1, the Hamming distance of two
// D-component vectors is H = (D - <x, y>) / 2 (the bipolar reading of
// Section 3.3 with the Hamming similarity of Section 3.4), and <x, y> over a
// window of candidates is a dense matrix product. Every partial sum is an
// integer of magnitude at most D <= 32768, exactly representable in int32 and
// in fp32 (int8 works on +-64 components: 4096 times the same integers), so
// every engine reproduces the popcount distances bit for bit.
//
// Two kernels: mfma_direct_kernel for calls of thousands of queries and
// mfma_stream_kernel, below it, for fewer. What follows is the first.
//
// Work decomposition (every engine): a workgroup takes one tile of 256
// m/z-ordered queries and one chunk of its candidate rows, in blocks of 256
// library rows (the M dimension). Eight waves form a 2 x 4 grid; each owns a
// 128-row x 64-query accumulator tile (4 x 2 tiles of 32 x 32) in
// registers, so two waves share every SIMD and one wave's bit expansion
// overlaps the other's matrix instructions.
//
// Data movement (mfma_direct.h): the packed bits of a block's rows and of the
// tile's queries move into LDS in stages of 1,024 components by direct
// global-to-LDS loads, one stage ahead of their use; each wave reads its
// operand words from LDS and expands them in registers between the matrix
// instructions of the step before, with one shift and one bit insert per 4 components
// (int8 +-64, fp8 +-1.0) or per 8 (fp4, asymmetric on the library side).
//
// Epilogue per block: distance = (Q - dot) / 2 (Q = D, or the fp4 form's
// per-query constant), masked by each query's own window and the chunk end,
// folded into a per-lane 64-bit running minimum of (distance << 32 | library
// index); lanes l and l+32 hold the same query columns and are merged with a
// shuffle before one atomicMin per query.
#include <algorithm>
#include <cmath>

#include "internal.h"
#include "launch_pieces.h"
#include "mfma_direct.h"
#include "window_search.h"

namespace homs {
namespace {

// XCD-aware work map of the direct kernels. Workgroups are handed
// to the eight XCDs in turn (workgroup i to XCD i mod 8), and each XCD has its
// own L2. Work items are (query tile, library chunk) pairs on absolute chunk
// boundaries; they are grouped into patches of adjacent tiles x adjacent
// chunks (8 x 4 where there are that many), and consecutive patches go to
// consecutive XCDs, so the 32 workgroups an XCD runs side by side share 4
// chunks of library rows and 8 tiles of query rows (about 3 MB per 256-row
// step) in their L2. The patches of a window's share are few (200 for 16,003
// queries of 600,002 rows with 2,048-row chunks), so their sizes also decide
// how evenly the XCDs are loaded: 16,003 queries 8.44 ms with 4 x 8 patches
// and 2,048-row chunks, 7.89 ms with 8 x 4 and 1,024; 100,000 queries of
// 2,000,000 rows 157.0 ms with 4 x 8 and 4,096, 152.3 ms with 8 x 4 and 2,048
// (152.2 with 8 x 2, which is 2% slower at 8,000 to 16,000 queries).
constexpr int kXcds = 8;
struct WorkMap {
  uint32_t n_tiles, n_chunks, chunk;          // chunk: library rows per item
  uint32_t patch_tiles, patch_chunks;         // items of a patch
  uint32_t chunk_patches, patches;            // patches along the library, in all
  uint32_t items;                             // kXcds rounds of whole patches
  uint32_t first;                             // item of workgroup 0
  bool listed;                                // the workgroups list their items
};

// wave layout of the one-shot kernels
using DirectLayout = mfd::Layout8;

template <int F>
__global__ __launch_bounds__(DirectLayout::kThreads, 1) void mfma_direct_kernel(
    uint32_t words,
    int64_t nq,
    const uint32_t* __restrict__ q_hv, const uint32_t* __restrict__ qperm,
    const int64_t* __restrict__ lo, const int64_t* __restrict__ hi,
    const int64_t* __restrict__ tlo, const int64_t* __restrict__ thi,
    const uint32_t* __restrict__ lib, const uint32_t* __restrict__ orig,
    const int32_t* __restrict__ qoff, const float* __restrict__ rowk,
    uint64_t* __restrict__ keys, WorkMap map)
{
  // the rows [*a, *b) of an item (none: a >= b)
  auto rows_of = [&](uint32_t item, uint32_t* tile, int64_t* a, int64_t* b) {
    const uint32_t per = map.patch_tiles * map.patch_chunks;
    const uint32_t slot = item / kXcds;  // position in its XCD's sequence
    const uint32_t patch = (slot / per) * kXcds + item % kXcds;
    const uint32_t local = slot % per;
    *tile = (patch / map.chunk_patches) * map.patch_tiles + local / map.patch_chunks;
    const uint32_t cidx =
        (patch % map.chunk_patches) * map.patch_chunks + local % map.patch_chunks;
    *a = *b = 0;
    if (patch >= map.patches || *tile >= map.n_tiles || cidx >= map.n_chunks) return;
    const int64_t c0 = (int64_t)cidx * map.chunk;
    *a = max(c0, tlo[*tile]);
    *b = min(c0 + map.chunk, thi[*tile]);
  };
  // One item per workgroup, or (listed) items blockIdx.x, + gridDim.x, ...: each
  // thread looks at one, and those with candidates are listed.
  __shared__ uint32_t s_items[DirectLayout::kThreads], s_n;
  const uint32_t mine = map.first + blockIdx.x;
  const uint64_t end = map.listed ? map.items : (uint64_t)mine + 1;
  for (uint64_t i0 = mine; i0 < end; i0 += (uint64_t)gridDim.x * DirectLayout::kThreads) {
    uint32_t n = 1;
    if (map.listed) {
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      const uint64_t item = i0 + (uint64_t)threadIdx.x * gridDim.x;
      uint32_t tile;
      int64_t a = 0, b = 0;
      if (item < map.items) rows_of((uint32_t)item, &tile, &a, &b);
      if (a < b) s_items[atomicAdd(&s_n, 1u)] = (uint32_t)item;
      __syncthreads();
      n = s_n;
    }
    for (uint32_t k = 0; k < n; ++k) {
      uint32_t tile;
      int64_t a, b;
      rows_of(map.listed ? __builtin_amdgcn_readfirstlane(s_items[k]) : mine, &tile, &a, &b);
      if (a < b)
        mfd::tile_rows<F, DirectLayout>(words, nq, q_hv, qperm, lo, hi, tile, (uint32_t)a,
                                        (uint32_t)b, lib, orig, qoff, rowk, keys);
    }
    __syncthreads();  // the list is read
  }
}

// ---- few queries ------------------------------------------------------------
// A call of few queries is bound by reading the library rows, and a tile of
// 256 queries would mostly multiply padding. Tiles of 32 TQ queries instead:
// the workgroup keeps the packed bits of its queries in LDS for the whole
// chunk (row stride D/8 + 16 bytes, so the 16 rows a quarter-wave reads
// together fall in 16 distinct bank groups), and each of its eight waves
// streams its own 32-row blocks of the library straight into registers, two
// stages of kSG 16-byte loads ahead, with no barrier after the start. The
// operands are expanded as in mfma_direct.h. The dot products, the row order
// inside a block and the result keys are those of tile_rows.
//
// Measured (D = 8,192, fp4): 64 queries over 400,000 rows 0.65 ms with the
// 256-query kernel and 4,096-row chunks, 0.14 ms so; 4 queries over 2M rows
// (1.6 GB of candidates) 0.31 ms per call. Without the one atomic per
// workgroup (one per wave and query, unconditional) the first took 0.3 ms.
constexpr int kStreamThreads = 512, kStreamWaves = kStreamThreads / 64;
constexpr uint32_t kStreamBlock = 32;  // library rows per wave step

template <int F, int TQ, int kSG>
__device__ __forceinline__ void stream_rows(uint32_t words, int64_t nq,
    const uint32_t* __restrict__ q_hv, const uint32_t* __restrict__ qperm,
    const int64_t* __restrict__ lo, const int64_t* __restrict__ hi, int64_t tile, uint32_t a,
    uint32_t b, const uint32_t* __restrict__ lib, const uint32_t* __restrict__ orig,
    const int32_t* __restrict__ qoff, const float* __restrict__ rowk,
    uint64_t* __restrict__ keys)
{
  using mfd::v16f;
  using mfd::v16i;
  using mfd::v4i;
  using mfd::v8i;
  constexpr int NQ = 32 * TQ;
  extern __shared__ __attribute__((aligned(16))) char s_query[];
  __shared__ unsigned long long s_best[NQ];
  const int t = threadIdx.x, l = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t r31 = l & 31, h = l >> 5;
  const uint32_t D = words * 32, stride = words * 4 + 16, pieces = words / 4;

  if (t < NQ) s_best[t] = ~0ull;
  for (uint32_t i = t; i < NQ * pieces; i += kStreamThreads) {
    const uint32_t r = i / pieces, p = i % pieces;
    const int64_t qs = tile * NQ + r;
    const uint32_t qi = qperm[qs < nq ? qs : nq - 1];
    *(uint4*)(s_query + r * stride + p * 16) =
        *(const uint4*)(q_hv + (size_t)qi * words + p * 4);
  }
  uint32_t qlo[TQ], qhi[TQ], qid[TQ];
  int Q[TQ];
  uint64_t bk[TQ];
  bool qok[TQ];
  float need[TQ];
#pragma unroll
  for (int j = 0; j < TQ; ++j) {
    const int64_t qs = tile * NQ + j * 32 + r31;
    qok[j] = qs < nq;
    qid[j] = qperm[qok[j] ? qs : nq - 1];
    qlo[j] = qok[j] ? (uint32_t)lo[qid[j]] : 0u;
    qhi[j] = qok[j] ? (uint32_t)hi[qid[j]] : 0u;
    Q[j] = F == mfd::kFmtF4 ? qoff[qid[j]] : (int)D;
    bk[j] = ~0ull;
    const uint64_t k0 = qok[j] ? keys[qid[j]] : 0ull;
    need[j] = !qok[j] ? INFINITY
              : k0 == ~0ull ? -INFINITY
                            : (float)(Q[j] - 2 * (int)(uint32_t)(k0 >> 32));
  }
  __syncthreads();

  // This wave's blocks: every kStreamWaves-th of the 32-row blocks meeting
  // [a, b), on absolute multiples of 32. Rows of a block outside [a, b) lie
  // outside every window of the tile (a chunk's ends are multiples of 32).
  const uint32_t first = a / kStreamBlock + w, end = (b + kStreamBlock - 1) / kStreamBlock;
  const uint32_t SPB = words / (8 * kSG);  // stages per block
  const uint32_t total =
      first < end ? (end - first + kStreamWaves - 1) / kStreamWaves * SPB : 0;
  uint32_t sel = 0x80808080u, one = F == mfd::kFmtI8 ? 0x40404040u : 0x38383838u;
  mfd::Fp4Consts k4{0x11111111u, 0x22222222u, 0x44444444u, 0x88888888u, 0x66666666u};
  if constexpr (F != mfd::kFmtF4)
    asm volatile("" : "+v"(sel), "+v"(one));
  else
    asm volatile("" : "+v"(k4.c11), "+v"(k4.c22), "+v"(k4.c44), "+v"(k4.c88), "+v"(k4.c66));

  // the loads' cursor (past the end it stays on the last stage)
  uint32_t l_blk = first, l_sp = 0;
  auto load = [&](uint4 (&buf)[kSG]) {
    const uint32_t row = min(l_blk * kStreamBlock + r31, b - 1u);
    const uint32_t* p = lib + (size_t)row * words + l_sp * (kSG * 8) + h * 4;
#pragma unroll
    for (int g = 0; g < kSG; ++g) buf[g] = *(const uint4*)(p + g * 8);
    if (++l_sp == SPB) {
      if (l_blk + kStreamWaves < end) {
        l_blk += kStreamWaves;
        l_sp = 0;
      } else {
        l_sp = SPB - 1;
      }
    }
  };
  using Acc = typename std::conditional<F == mfd::kFmtI8, v16i, v16f>::type;
  Acc acc[TQ];
  uint32_t blk = first, sp = 0;
  auto stage = [&](uint4 (&buf)[kSG]) {
    if (sp == 0) {
#pragma unroll
      for (int j = 0; j < TQ; ++j) acc[j] = Acc{0};
    }
    const char* qb = s_query + r31 * stride + (sp * (2 * kSG) + h) * 16;
    uint4 cur[kSG];
#pragma unroll
    for (int g = 0; g < kSG; ++g) cur[g] = buf[g];
#pragma unroll
    for (int g = 0; g < kSG; ++g) {
      uint4 cb[TQ];
#pragma unroll
      for (int j = 0; j < TQ; ++j) cb[j] = *(const uint4*)(qb + j * 32 * stride + g * 32);
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        const uint32_t x = st == 0   ? cur[g].x
                           : st == 1 ? cur[g].y
                           : st == 2 ? cur[g].z
                                     : cur[g].w;
        v8i av;
        if constexpr (F == mfd::kFmtF4)
          av = mfd::expand_fp4(x, k4);
        else
          av = mfd::expand_pm1(x, sel, one);
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
          const uint32_t y = st == 0 ? cb[j].x : st == 1 ? cb[j].y : st == 2 ? cb[j].z : cb[j].w;
          v8i bv;
          if constexpr (F == mfd::kFmtF4)
            bv = mfd::expand_fp4(y, k4);
          else
            bv = mfd::expand_pm1(y, sel, one);
          if constexpr (F == mfd::kFmtI8) {
            const v4i a0 = {av[0], av[1], av[2], av[3]}, a1 = {av[4], av[5], av[6], av[7]};
            const v4i b0 = {bv[0], bv[1], bv[2], bv[3]}, b1 = {bv[4], bv[5], bv[6], bv[7]};
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, acc[j], 0, 0, 0);
          } else {
            acc[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[j], F, F, 0, 0,
                                                                     0, 0);
          }
        }
      }
    }
    if (++sp < SPB) return;

    // The block's results. Accumulator register r of tile j holds row
    // base + 8 (r / 4) + 4 h + r % 4 and query column j.
    sp = 0;
    const uint32_t base = blk * kStreamBlock;
    blk += kStreamWaves;
    if constexpr (F == mfd::kFmtF4) {  // t = <x, y> - K(row)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const float4 k = *(const float4*)(rowk + base + 8 * rg + 4 * h);
        const float kv[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
          for (int j = 0; j < TQ; ++j) acc[j][4 * rg + r4] -= kv[r4];
      }
    }
    bool inner = base >= a && base + kStreamBlock <= b;
#pragma unroll
    for (int j = 0; j < TQ; ++j)
      inner = inner && (!qok[j] || (qlo[j] <= base && base + kStreamBlock <= qhi[j]));
    const bool all_in = __ballot(!inner) == 0;
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
      // the largest dot product among the lane's candidates; only one that
      // reaches the query's best so far looks up library indices
      float m = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t g = base + 8 * (r >> 2) + 4 * h + (r & 3);
        const bool in = all_in || (g >= qlo[j] && g < qhi[j]);
        m = fmaxf(m, in ? mfd::dot_of(acc[j], r) : -INFINITY);
      }
      if (m != -INFINITY && m >= need[j]) {
        uint32_t o_min = ~0u;
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const uint4 o4 = *(const uint4*)(orig + base + 8 * rg + 4 * h);
          const uint32_t ov[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const uint32_t g = base + 8 * rg + 4 * h + r4;
            const bool in = all_in || (g >= qlo[j] && g < qhi[j]);
            if (in && mfd::dot_of(acc[j], 4 * rg + r4) == m) o_min = min(o_min, ov[r4]);
          }
        }
        const uint32_t d = (uint32_t)(Q[j] - (int)m) >> 1;
        const uint64_t key = ((uint64_t)d << 32) | o_min;
        bk[j] = key < bk[j] ? key : bk[j];
        need[j] = m;
      }
    }
  };

  // Two stages of loads in flight in two named register sets, each refilled
  // right after its stage has taken its words
  uint4 b0[kSG], b1[kSG];
  if (total) {
    load(b0);
    load(b1);
  }
  for (uint32_t s = 0; s < total; s += 2) {
    stage(b0);
    load(b0);
    if (s + 1 < total) {
      stage(b1);
      load(b1);
    }
  }
  // One atomic per workgroup and query, and only where it still lowers the
  // result: thousands of them meet on the few lines of a small call's keys
  // (a value read too early, or from a stale line, is only too large).
#pragma unroll
  for (int j = 0; j < TQ; ++j)
    if (bk[j] != ~0ull) atomicMin(s_best + j * 32 + r31, (unsigned long long)bk[j]);
  __syncthreads();
  if (t < NQ && s_best[t] != ~0ull) {
    uint64_t* key = keys + qperm[tile * NQ + t];
    if (s_best[t] < *(volatile uint64_t*)key) atomicMin((unsigned long long*)key, s_best[t]);
  }
}

template <int F, int TQ>
__global__ __launch_bounds__(kStreamThreads, 4) void mfma_stream_kernel(uint32_t words,
    int64_t nq, const uint32_t* __restrict__ q_hv, const uint32_t* __restrict__ qperm,
    const int64_t* __restrict__ lo, const int64_t* __restrict__ hi,
    const int64_t* __restrict__ tlo, const int64_t* __restrict__ thi,
    const uint32_t* __restrict__ lib, const uint32_t* __restrict__ orig,
    const int32_t* __restrict__ qoff, const float* __restrict__ rowk,
    uint64_t* __restrict__ keys, uint32_t n_tiles, uint32_t round0, uint32_t chunk)
{
  // XCD x (workgroup i runs on XCD i mod 8) takes chunks x, x + 8, ... and,
  // chunk after chunk, every tile: a chunk's rows come into one L2 once (this
  // launch: from round round0 of eight chunks on)
  const uint32_t wg = blockIdx.x, slot = wg / kXcds;
  const uint32_t tile = slot % n_tiles;
  const int64_t c0 = ((int64_t)(round0 + slot / n_tiles) * kXcds + wg % kXcds) * chunk;
  const int64_t a = max(c0, tlo[tile]), b = min(c0 + chunk, thi[tile]);
  if (a >= b) return;
  if (words % 32 == 0)
    stream_rows<F, TQ, 4>(words, nq, q_hv, qperm, lo, hi, tile, (uint32_t)a, (uint32_t)b, lib,
                          orig, qoff, rowk, keys);
  else
    stream_rows<F, TQ, 2>(words, nq, q_hv, qperm, lo, hi, tile, (uint32_t)a, (uint32_t)b, lib,
                          orig, qoff, rowk, keys);
}

// the class weights of a packed row: the fp4 form's per-row constant K (and,
// plus 21D/4, its per-query constant Q); one wave per row
__device__ __forceinline__ int fp4_class_weight(const uint32_t* __restrict__ row, uint32_t words)
{
  const int l = threadIdx.x & 63;
  int s = 0;
  for (uint32_t i = l; i < words; i += 64) s += fp4_word_weight(row[i]);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  return s;
}

__global__ __launch_bounds__(256) void fp4_query_offsets_kernel(int64_t nq, uint32_t words,
    const uint32_t* __restrict__ q_hv, int32_t* __restrict__ qoff)
{
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= nq) return;
  const int s = fp4_class_weight(q_hv + (size_t)q * words, words);
  if ((threadIdx.x & 63) == 0) qoff[q] = s + (int)(21 * words * 8);  // 21D/4
}

// the per-row constants, n rows, then `pad` zeros: four rows a wave, 16 bytes a
// lane and row, so that four loads are in flight (400,001 rows, D = 8,192:
// 153 -> 77 us, 5.3 TB/s)
constexpr int kConstRows = 4;
__global__ __launch_bounds__(256) void fp4_row_consts_kernel(int64_t n, int64_t pad, uint32_t words,
    const uint32_t* __restrict__ hv, float* __restrict__ rowk)
{
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kConstRows;
  if (r0 >= n + pad) return;
  const uint32_t l = threadIdx.x & 63, w4 = words / 4;
  int s[kConstRows] = {};
  if (r0 < n)
    for (uint32_t c = l; c < w4; c += 64) {
      uint4 v[kConstRows];
#pragma unroll
      for (int k = 0; k < kConstRows; ++k)
        v[k] = *(const uint4*)(hv + (size_t)min(r0 + k, n - 1) * words + c * 4);
#pragma unroll
      for (int k = 0; k < kConstRows; ++k)
        s[k] += fp4_word_weight(v[k].x) + fp4_word_weight(v[k].y) + fp4_word_weight(v[k].z) +
                fp4_word_weight(v[k].w);
    }
#pragma unroll
  for (int k = 0; k < kConstRows; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o);
    if (l == 0 && r0 + k < n + pad) rowk[r0 + k] = r0 + k < n ? (float)s[k] : 0.f;
  }
}

// Library rows per workgroup: the largest power of two up to `most`, and at
// least 256, that makes `items` (tile, chunk) items, of which a window's share
// holds candidates; fewer leave compute units idle (16,003 queries, 600,002
// rows, D = 8,192, 8 x 4 patches: 8.19 ms with 16,384 items, 7.89 ms with
// 24,576, 7.91 ms with 49,152).
constexpr int64_t kMfChunk = 2048;
constexpr int64_t kMfItems = 24576;
int64_t chunk_rows(int64_t n_tiles, int64_t n, int64_t most, int64_t items, int64_t least = 256)
{
    int64_t chunk = most;
    while (chunk > least && n_tiles * ((n + chunk - 1) / chunk) < items) chunk /= 2;
    return chunk;
}

// The stream kernel's rows per workgroup (a multiple of its 32-row blocks).
// 512 of its workgroups run at once. Up to four tiles, whose windows cover most
// of the library, they are made to fit that many one or two rounds: a
// workgroup starts by filling LDS with its queries, and a round that is
// nearly empty costs as much as a full one (400,000 rows, D = 8,192, against
// powers of two: 64 queries 0.135 against 0.167 ms, 16 0.113 against 0.131,
// 200 0.30 against 0.40). More tiles cover less of the library each, and
// more, smaller items even that out (1,000 queries 0.557 ms with 1,024 rows,
// 0.585 with 512; of 120,000 rows 0.223 with 512, 0.247 with 256 and 0.274
// with 1,600).
int64_t stream_chunk(int64_t n_tiles, int64_t n)
{
    if (n_tiles <= 4) {
        const int64_t wgs = n_tiles == 1 ? 512 : 1024;
        const int64_t rows = (n * n_tiles + wgs - 1) / wgs;
        return std::min<int64_t>(1600, std::max<int64_t>(256, (rows + 31) / 32 * 32));
    }
    return n_tiles < 32 ? chunk_rows(n_tiles, n, 2048, 3072) : chunk_rows(n_tiles, n, 8192, 8192);
}

}  // namespace

// Queries per tile. Up to a few thousand queries the streaming kernel's small
// tiles win: less padding, and tighter unions of windows (measured at 200,000
// to 800,000 rows, D = 8,192, both kernels with their best chunks: 64 queries
// 0.18 against 0.39 ms, 1,000 0.86 against 0.92, 4,000 0.85 against 0.92 and
// 3.30 against 3.22, 8,000 1.60 against 1.65). Above D = 8,192 its LDS leaves
// one workgroup per compute unit, or tiles of 32 only (D = 16,384: 200
// queries 0.25 against 0.41 ms, 2,000 1.26 against 1.02). Tiles of 32 are also
// the better ones where a row is short, so that reading it once per tile
// costs little (D = 1,536, 200 queries 0.13 against 0.19 ms; D = 8,192, 300
// queries 0.67 against 0.55).
int search_mfma_tile(const homs_ctx* c, int64_t nq)
{
    const bool wide = c->words > 256;
    if (nq > (wide ? 1024 : 4096)) return mfd::kQueries;
    return wide || nq <= 32 || (c->words <= 64 && nq <= 512) ? 32 : 64;
}
int64_t search_mfma_row_pad() { return mfd::kRows; }

hipError_t launch_fp4_row_consts(int64_t n, uint32_t words, const uint32_t* hv, float* rowk,
                                 hipStream_t s)
{
  const int64_t pad = mfd::kRows;  // the epilogue reads whole groups past the last row
  if (n + pad <= 0) return hipSuccess;
  const int64_t per = 4 * kConstRows;  // rows of a workgroup
  fp4_row_consts_kernel<<<(uint32_t)((n + pad + per - 1) / per), 256, 0, s>>>(n, pad, words, hv,
                                                                             rowk);
  return hipGetLastError();
}

hipError_t launch_fp4_query_offsets(const homs_ctx* c, int64_t nq, const uint32_t* q_hv,
                                    int32_t* qoff, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    fp4_query_offsets_kernel<<<(uint32_t)((nq + 3) / 4), 256, 0, s>>>(nq, c->words, q_hv, qoff);
    return hipGetLastError();
}

hipError_t launch_search_mfma(const homs_ctx* c, int fmt, int64_t nq, const uint32_t* q_hv,
                              const uint32_t* qperm, const int64_t* lo, const int64_t* hi,
                              const int64_t* tile_lo, const int64_t* tile_hi, const int32_t* qoff,
                              uint64_t* keys, int32_t kind, double value, hipStream_t s)
{
    if (nq <= 0 || c->lib.n <= 0) return hipSuccess;
    const int tile = search_mfma_tile(c, nq);
    const int64_t n_tiles = (nq + tile - 1) / tile;
    const bool f4 = fmt == 2;
    if (tile != mfd::kQueries) {
        const int64_t ch = stream_chunk(n_tiles, c->lib.n);
        const int64_t n_rounds = ((c->lib.n + ch - 1) / ch + kXcds - 1) / kXcds;
        const size_t lds = (size_t)tile * (c->words * 4 + 16);
        auto go = [&](auto kern) {  // a few tiles: a piece holds them all
            in_pieces(n_tiles, n_rounds, kStreamThreads,
                      [&](int64_t, int64_t, int64_t r, int64_t rounds) {
                kern<<<(uint32_t)(n_tiles * rounds * kXcds), kStreamThreads, lds, s>>>(
                    c->words, nq, q_hv, qperm, lo, hi, tile_lo, tile_hi, c->lib.hv, c->lib.orig,
                    f4 ? qoff : nullptr, f4 ? c->lib.rowk : nullptr, keys, (uint32_t)n_tiles,
                    (uint32_t)r, (uint32_t)ch);
            });
        };
        if (tile == 32) {
            if (fmt == 0) go(mfma_stream_kernel<mfd::kFmtI8, 1>);
            else if (fmt == 1) go(mfma_stream_kernel<mfd::kFmtF8, 1>);
            else go(mfma_stream_kernel<mfd::kFmtF4, 1>);
        } else {
            if (fmt == 0) go(mfma_stream_kernel<mfd::kFmtI8, 2>);
            else if (fmt == 1) go(mfma_stream_kernel<mfd::kFmtF8, 2>);
            else go(mfma_stream_kernel<mfd::kFmtF4, 2>);
        }
        return hipGetLastError();
    }
    // a block of short rows is done before its queries are loaded (D = 512, 6,000
    // queries of 400,000 rows, +-500 Da: 0.71 ms with 256-row chunks, 0.55 so)
    const int64_t chunk = chunk_rows(n_tiles, c->lib.n, kMfChunk, kMfItems,
                                     std::max<int64_t>(256, 16384 / c->words));
    const int64_t n_chunks = (c->lib.n + chunk - 1) / chunk;
    WorkMap m;
    m.n_tiles = (uint32_t)n_tiles;
    m.n_chunks = (uint32_t)n_chunks;
    m.chunk = (uint32_t)chunk;
    m.patch_tiles = (uint32_t)std::min<int64_t>(8, n_tiles);
    m.patch_chunks = n_tiles * n_chunks >= 32 * 64 ? 4 : 1;
    const int64_t tile_groups = (n_tiles + m.patch_tiles - 1) / m.patch_tiles;
    m.chunk_patches = (uint32_t)((n_chunks + m.patch_chunks - 1) / m.patch_chunks);
    // Short windows lie along a diagonal: a group of tiles has its candidates in
    // a patch or two, `step` patches further along the library than the group
    // before, chunk_patches + step patches on in the sequence dealt to the XCDs.
    // An even distance would leave half of the XCDs idle (100,000 queries of
    // 400,000 rows, +-3.3 Da: 1.85 ms; 1.23 with one empty patch more a group).
    const double step = ((double)n_chunks / m.patch_chunks) / ((double)n_tiles / m.patch_tiles);
    const double turn = std::fmod(m.chunk_patches + step, 2.0);
    if (step < 4.0 && (turn < 0.2 || turn > 1.8)) m.chunk_patches += 1;
    const int64_t patches = tile_groups * m.chunk_patches;
    // whole rounds of kXcds patches, so every XCD's sequence is complete
    const int64_t blocks =
        (patches + kXcds - 1) / kXcds * kXcds * m.patch_tiles * m.patch_chunks;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
    m.patches = (uint32_t)patches;
    m.items = (uint32_t)blocks;
    // A workgroup of an item without candidates costs 2 ns of dispatch: with
    // windows of a few dozen rows hardly any item has some (20,001 queries of
    // 1,000,000 rows: 39,000 items, 84 us of nothing else). A fixed grid whose
    // workgroups first list their items with candidates, one item a thread,
    // passes over them in 5 us; where most items hold work, one workgroup each
    // is the better balanced. 100,000 queries of 2,000,000 rows with 1,024, 4,096 and
    // 65,536 workgroups and one for each of the 382,000 items: D = 8,192, +-1.4 Da 3.0,
    // 2.8, 3.0 and 4.2 ms, +-3 Da 3.7, 3.4, 3.8 and 4.7, +-500 Da 170.5 (4,096), 157.8
    // and 155.0; D = 512, +-3 Da 0.86, 0.78, 1.07 and 2.24; 30,000 of 400,000 rows, D =
    // 512, +-1.4 Da 0.17, 0.19, 0.34 and 0.34. Against one each, 4,096 take 0.96 and 0.87
    // of the time at +-25 Da, D = 8,192 and 512, 0.97 and 0.88 at +-50, 1.00 and 0.91 at
    // +-100 and 1.02 and 0.97 at +-500 (6,000 to 60,000 queries of 60,000 to 1,000,000
    // rows).
    // Few items are listed by 1,024 in 10 us less (6,000 queries +-0.5 Da of 400,000
    // rows, D = 2,048: 78 us, 89 with 4,096), but many or long ones keep those waiting
    // for each other (30,000 +-1.4 Da of 900,000 rows, D = 512: 364 us, 265 with 4,096;
    // 4,000 +-5 Da of 200,000 rows, D = 32,768: 1.36 ms, 1.16).
    const double da = kind == HOMS_TOL_PPM ? value / 1000.0 : value;  // near 1,000 Da
    const bool many = (da > 1.0 && (c->words >= 256 || blocks > 32768)) ||
                      (da > 0.1 && blocks > 65536);
    const int64_t most_groups = da > 50.0 ? INT64_MAX : many ? 4096 : 1024;
    m.listed = blocks > most_groups;
    auto go = [&](auto kern) {
        in_pieces(m.listed ? most_groups : blocks, DirectLayout::kThreads,
                  [&](int64_t first, int64_t count) {
            m.first = (uint32_t)first;
            kern<<<(uint32_t)count, DirectLayout::kThreads, 0, s>>>(
                c->words, nq, q_hv, qperm, lo, hi, tile_lo, tile_hi, c->lib.hv, c->lib.orig,
                f4 ? qoff : nullptr, f4 ? c->lib.rowk : nullptr, keys, m);
        });
    };
    if (fmt == 0) go(mfma_direct_kernel<mfd::kFmtI8>);
    else if (fmt == 1) go(mfma_direct_kernel<mfd::kFmtF8>);
    else go(mfma_direct_kernel<mfd::kFmtF4>);
    return hipGetLastError();
}

}  // namespace homs
