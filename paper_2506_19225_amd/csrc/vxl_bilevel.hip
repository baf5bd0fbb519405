// Bi-level KV decoding, the integer / bandwidth-bound steps: per-chunk mean keys, relevance
// scores + top-k selection (by rank), and the dense/sparse gather into the mixed KV.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "vxl_internal.h"

namespace vxl {

namespace {

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const uint16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

// 16 bytes that are read once (NT: not kept in the caches)
template <bool NT>
__device__ __forceinline__ uint4 load16(const uint4* p) {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    if constexpr (NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)p));
    else return *p;
}
// 16 bytes that the caches need not keep (NT)
template <bool NT>
__device__ __forceinline__ void store16(uint4* p, uint4 v) {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (u32x4*)p);
    else *p = v;
}

// ------------------------------------------------------------------------------------------
// kbar[g, c, :] = mean of the dense key rows of chunk c.  One block per (chunk, kv head).
// A thread owns one 16-byte column piece and the rows rg, rg + RG, ... of the chunk, which it
// sums in row order in four (512 threads: two) independent accumulators; all partial sums are then added in a
// fixed tree.  The summation tree depends only on the values and their offsets inside the chunk, not on the
// number of threads: two chunks with equal contents get bit-identical means, hence exactly tied scores, also
// in different layouts.  Bound by HBM when large, otherwise by a block's chain of round
// trips: the last rows of a thread are requested together as well (114 chunks of 128 to 1,024 tokens, one
// by one -> so, 25.6 -> 24.1 us with the selection).  How many threads, and whether past the caches: launch_summaries.
// ------------------------------------------------------------------------------------------
// qbar[b, g, :] = mean over the T query tokens and the query heads of KV head g of Qd[b, t, h, :].
// Up to kMeanLoads tokens: one block per (b, g), a thread owns one 16-byte column piece of one head and adds its T tokens in
// token order; the heads of the group are then added in head order.  (Eight loads of a thread in flight here and below:
// sixteen take 82 to 98 registers, which leave the chunks of the launch five or four waves per SIMD instead of eight, 256
// chunks 18.5 -> 19.8 us; streamed past the caches four are as good as eight and steadier, 640 chunks 35.4 -> 34.6.)
constexpr int kMeanLoads = 8;

template <typename T, int D, int THREADS>
__device__ __forceinline__ void query_mean_block(const T* __restrict__ Qd, float* __restrict__ qbar, int b, int g,
                                                 int T_q, int n_q_heads, int n_kv_heads, float* hsum /*[group][D]*/) {
    constexpr int EPC = 16 / (int)sizeof(T);
    constexpr int PPR = D / EPC;
    const int group = n_q_heads / n_kv_heads, tid = threadIdx.x;
    const T* qb = Qd + (size_t)b * T_q * n_q_heads * D;
    const int row_pieces = n_q_heads * PPR;
    for (int p = tid; p < group * PPR; p += THREADS) {
        const int gp = g * group * PPR + p;                    // piece index inside a token's [Hq*D] row
        float acc[EPC];
#pragma unroll
        for (int i = 0; i < EPC; ++i) acc[i] = 0.f;
        uint4 v[kMeanLoads];
#pragma unroll
        for (int u = 0; u < kMeanLoads; ++u)                   // (clamped rows are not added below)
            v[u] = ((const uint4*)qb)[(size_t)min(u, T_q - 1) * row_pieces + gp];
#pragma unroll
        for (int u = 0; u < kMeanLoads; ++u) {
            if (u < T_q) {
                const T* e = (const T*)&v[u];
#pragma unroll
                for (int i = 0; i < EPC; ++i) acc[i] += ld(e + i);
            }
        }
#pragma unroll
        for (int i = 0; i < EPC; ++i) hsum[p * EPC + i] = acc[i];
    }
    __syncthreads();
    for (int dd = tid; dd < D; dd += THREADS) {
        float a = 0.f;
        for (int hg = 0; hg < group; ++hg) a += hsum[hg * D + dd];
        qbar[((size_t)b * n_kv_heads + g) * D + dd] = a / (float)(T_q * group);
    }
}

// The same for more tokens, one block per (b, g, four pieces of a row), begun before the chunks: a thread owns one piece of
// one head and every tg_n-th token; the tg_n sums of a piece are added in order, then the heads of the group.  A chain of
// round trips: with all tokens of a piece in one thread, 128 tokens took eight, behind the chunks of the launch (28 heads on
// four, D = 128, with the selection: 64 chunks of 256 tokens 17.3 -> 11.3 us, 256 chunks 28.2 -> 20.6, 640 40.1 -> 35.5;
// 8 of 128 tokens 14.0 -> 8.3; 64 tokens 10.1 -> 8.0, 32 8.4 -> 7.6, 16 7.6 -> 7.5).
constexpr int kMeanPieces = 4, kMeanTokens = kMeanLoads;      // pieces of a block; tokens up to which one block takes a row
constexpr int kMeanThreads = 256;                             // threads of a block that own a piece and tokens of it

template <typename T, int D, int THREADS>
__device__ __forceinline__ void query_mean_part(const T* __restrict__ Qd, float* __restrict__ qbar, int b, int g, int first,
                                                int T_q, int n_q_heads, int n_kv_heads, float* sums /*[tg_n][group][COLS]*/) {
    constexpr int EPC = 16 / (int)sizeof(T);
    constexpr int PPR = D / EPC, COLS = kMeanPieces * EPC;
    const int group = n_q_heads / n_kv_heads, tid = threadIdx.x, n = group * kMeanPieces;
    // token groups, this thread's (as many from 512 threads as from 256: a query's mean does not depend on the layout)
    const int tg_n = max(1, min(kMeanThreads / n, (T_q + kMeanLoads - 1) / kMeanLoads)), tg = tid / n;
    const T* qb = Qd + (size_t)b * T_q * n_q_heads * D;
    const int row_pieces = n_q_heads * PPR;
    if (tg < tg_n) {
        for (int p = tid - tg * n; p < n; p += THREADS) {
            const int gp = (g * group + p / kMeanPieces) * PPR + first + p % kMeanPieces;     // piece inside a token's [Hq*D] row
            float acc[EPC];
#pragma unroll
            for (int i = 0; i < EPC; ++i) acc[i] = 0.f;
            for (int t0 = tg; t0 < T_q; t0 += kMeanLoads * tg_n) {
                uint4 v[kMeanLoads];
#pragma unroll
                for (int u = 0; u < kMeanLoads; ++u)                   // (clamped rows are not added below)
                    v[u] = ((const uint4*)qb)[(size_t)min(t0 + u * tg_n, T_q - 1) * row_pieces + gp];
#pragma unroll
                for (int u = 0; u < kMeanLoads; ++u) {
                    if (t0 + u * tg_n < T_q) {
                        const T* e = (const T*)&v[u];
#pragma unroll
                        for (int i = 0; i < EPC; ++i) acc[i] += ld(e + i);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < EPC; ++i) sums[(tg * n + p) * EPC + i] = acc[i];
        }
    }
    __syncthreads();
    if (tg_n > 1) {                                           // (in one step with the heads, by COLS threads: 0.3 to 1.9 us more)
        for (int e = tid; e < n * EPC; e += THREADS) {
            float a = sums[e];
            for (int k = 1; k < tg_n; ++k) a += sums[k * n * EPC + e];
            sums[e] = a;
        }
        __syncthreads();
    }
    for (int dd = tid; dd < COLS; dd += THREADS) {
        float a = 0.f;
        for (int hg = 0; hg < group; ++hg) a += sums[hg * COLS + dd];
        qbar[((size_t)b * n_kv_heads + g) * D + first * EPC + dd] = a / (float)(T_q * group);
    }
}

// The first n_mean blocks (more than kMeanTokens tokens), or those behind the chunks, form the mean queries, the others
// summarise a chunk each: both feed the scoring kernel, one launch serves both.
template <typename T, int D, int THREADS, bool NT>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(NT ? 4 : 8, NT ? 4 : 8))) void chunk_summarize_kernel(const T* __restrict__ K,
                                                              const int32_t* __restrict__ bounds,
                                                              float* __restrict__ kbar, long long kv_head_u4,
                                                              long long kv_tok_u4,   // K strides, 16-byte units
                                                              int n_chunks, int n_mean, const T* __restrict__ Qd,
                                                              float* __restrict__ qbar, int T_q, int n_q_heads,
                                                              int n_kv_heads) {
    constexpr int EPC = 16 / (int)sizeof(T);        // elements per 16-byte piece
    constexpr int PPR = D / EPC;                    // pieces per row
    constexpr int RG = THREADS / PPR;               // row groups
    constexpr int U = THREADS == 512 && !NT ? 8 : 4;      // rows that a thread requests together
    // Partial sums of the rows of equal place mod CHAINS, which is the same for either number of threads: a thread has A
    // of them, and they are added in the same tree.
    constexpr int A = THREADS == 512 ? 2 : 4, CHAINS = A * RG, GROUPS = CHAINS / 4;
    constexpr int KEPT = THREADS == 512 ? CHAINS : GROUPS;      // (256 threads: a thread adds the four of its group)
    extern __shared__ float dyn[];                  // for the query blocks: [group][D], or four pieces per head and group of tokens
    __shared__ float part[KEPT][D];
    if ((int)blockIdx.x < n_mean) {
        constexpr int PARTS = PPR / kMeanPieces;
        query_mean_part<T, D, THREADS>(Qd, qbar, blockIdx.x / PARTS, blockIdx.y, blockIdx.x % PARTS * kMeanPieces, T_q,
                                       n_q_heads, n_kv_heads, dyn);
        return;
    }
    const int c = blockIdx.x - n_mean, g = blockIdx.y;
    if (c >= n_chunks) {
        query_mean_block<T, D, THREADS>(Qd, qbar, c - n_chunks, g, T_q, n_q_heads, n_kv_heads, dyn);
        return;
    }
    const int piece = threadIdx.x % PPR, rg = threadIdx.x / PPR;
    const int lo = bounds[c], hi = bounds[c + 1];
    const uint4* base = (const uint4*)K + (size_t)g * kv_head_u4 + piece;
    float acc[A][EPC];
#pragma unroll
    for (int u = 0; u < A; ++u)
#pragma unroll
        for (int i = 0; i < EPC; ++i) acc[u][i] = 0.f;
    int r = lo + rg;
    for (; r + (U - 1) * RG < hi; r += U * RG) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load16<NT>(base + (size_t)(r + u * RG) * kv_tok_u4);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T* e = (const T*)&v[u];
#pragma unroll
            for (int i = 0; i < EPC; ++i) acc[u % A][i] += ld(e + i);
        }
    }
    if (r < hi) {                                             // the last rows, requested together as well (a repeated one is not added)
        uint4 v[U - 1];
#pragma unroll
        for (int u = 0; u < U - 1; ++u) v[u] = load16<NT>(base + (size_t)min(r + u * RG, hi - 1) * kv_tok_u4);
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (r + u * RG < hi) {
                const T* e = (const T*)&v[u];
#pragma unroll
                for (int i = 0; i < EPC; ++i) acc[u % A][i] += ld(e + i);
            }
    }
#pragma unroll
    for (int i = 0; i < EPC; ++i) {
        if constexpr (A == 4) {
            part[rg][piece * EPC + i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
        } else {
            part[rg][piece * EPC + i] = acc[0][i];
            part[rg + RG][piece * EPC + i] = acc[1][i];
        }
    }
    __syncthreads();
    if (threadIdx.x < D) {
        auto group = [&](int i) __attribute__((always_inline)) {
            if constexpr (A == 4) return part[i][threadIdx.x];
            else return (part[i][threadIdx.x] + part[i + GROUPS][threadIdx.x]) +
                        (part[i + 2 * GROUPS][threadIdx.x] + part[i + 3 * GROUPS][threadIdx.x]);
        };
        float q[4];
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) q[i & 3] = i < 4 ? group(i) : q[i & 3] + group(i);
        const float s = (q[0] + q[1]) + (q[2] + q[3]);
        kbar[((size_t)g * n_chunks + c) * D + threadIdx.x] = s / (float)(hi - lo);
    }
}

// ------------------------------------------------------------------------------------------
// Relevance score of one chunk, formed by 16 neighbouring lanes: lane p takes the 16-byte pieces
// p, p + 16, ... of the flattened (kv head, d) range (256 contiguous bytes per step), in that
// order, and the sixteen partial dot products are added in a fixed tree.  A chunk's score thus
// depends on nothing but its mean keys, whichever kernel computes it: equal chunks tie exactly.
// Latency bound (2 KiB per chunk): the pieces of U steps of both operands are requested before the
// first multiply-add (U changes no bit).  Every lane of the group returns the score.
// ------------------------------------------------------------------------------------------
constexpr int kScoreLanes = 16;

template <int D, int U = 8>
__device__ __forceinline__ float chunk_score(const float* __restrict__ qbar_b, const float* __restrict__ kbar,
                                             int c, int n_kv_heads, int n_chunks, int p) {
    constexpr int PPH = D / 4;                                // 16-byte pieces per KV head
    const int n_pieces = n_kv_heads * PPH;
    const float4* q4 = (const float4*)qbar_b;
    const float4* k4 = (const float4*)kbar + (size_t)c * PPH;
    const size_t head_skip = (size_t)(n_chunks - 1) * PPH;    // from piece index to its place in kbar[g][c]
    float a = 0.f;
    for (int base = p; base < n_pieces; base += U * kScoreLanes) {
        float4 kv[U], qv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(base + u * kScoreLanes, n_pieces - 1);     // (clamped pieces are not added)
            kv[u] = k4[e + (e / PPH) * head_skip];
            qv[u] = q4[e];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = base + u * kScoreLanes < n_pieces;
            const float t = fmaf(qv[u].w, kv[u].w, fmaf(qv[u].z, kv[u].z, fmaf(qv[u].y, kv[u].y, fmaf(qv[u].x, kv[u].x, a))));
            a = in ? t : a;
        }
    }
#pragma unroll
    for (int o = 1; o < kScoreLanes; o <<= 1) a += __shfl_xor(a, o);
    return a;
}

// ------------------------------------------------------------------------------------------
// Selection by rank: chunk c's place in the order (score descending, ties to the lower chunk id)
// is the number of chunks before it.  Score and id are packed into one 64-bit key -- the score's
// bits mapped so that unsigned order is float order (-0 counts as 0), the id complemented -- so
// the order is total and one comparison decides; the ranks are a permutation whatever the scores
// hold.  C^2 comparisons, but spread over many waves with no barrier between them: a wave ranks 64
// chunks (one per lane) against its slice of the keys, read from LDS two at a time by broadcast.
// One block counting for all chunks took 50 us at 640 chunks and 8.3 at 256; 64 chunks per block
// with the keys cut over eight waves: 4.8 and 4.6, most of it the launch.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long rank_key(float s, int c) {
    uint32_t u = __float_as_uint(s + 0.f);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)u << 32) | (uint32_t)~c;
}

// Keys of the slice [lo, hi) (both even) of `keys` (LDS) that come before `mine`.
__device__ __forceinline__ int count_before(const unsigned long long* keys, int lo, int hi, unsigned long long mine) {
    int n = 0;
#pragma unroll 4
    for (int o = lo; o < hi; o += 2) {
        const ulonglong2 k2 = *(const ulonglong2*)(keys + o);
        n += (k2.x > mine ? 1 : 0) + (k2.y > mine ? 1 : 0);
    }
    return n;
}

// Called by a whole block of WAVES waves: ranks the chunks [64 * group0, 64 * (group0 + GROUPS)) of
// the n_chunks whose keys lie in LDS (padded to an even count with 0, which precedes nothing) and
// writes their places in topk_idx / dense_mask of query b.  The WAVES / GROUPS waves of a group of
// 64 chunks share the keys; `part` holds WAVES * 64 ints.
template <int WAVES, int GROUPS>
__device__ __forceinline__ void rank_select(const unsigned long long* keys, int* part, int n_chunks, int group0, int k,
                                            int b, int32_t* __restrict__ topk_idx, uint8_t* __restrict__ dense_mask) {
    constexpr int SL = WAVES / GROUPS;                        // slices of the keys
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int grp = wave % GROUPS, sl = wave / GROUPS;
    const int c = (group0 + grp) * 64 + lane;
    const int n2 = (n_chunks + 1) & ~1;
    const int len = ((n2 / 2 + SL - 1) / SL) * 2;
    const unsigned long long mine = keys[min(c, n_chunks - 1)];
    part[(sl * GROUPS + grp) * 64 + lane] = count_before(keys, min(sl * len, n2), min((sl + 1) * len, n2), mine);
    __syncthreads();
    if (sl == 0 && c < n_chunks) {
        int rank = 0;
#pragma unroll
        for (int i = 0; i < SL; ++i) rank += part[(i * GROUPS + grp) * 64 + lane];
        if (rank < k) topk_idx[(size_t)b * k + rank] = c;
        dense_mask[(size_t)b * n_chunks + c] = (uint8_t)(rank < k ? 1 : 0);
    }
}

// The scores alone, 16 chunks per block (grid: chunk groups x queries).
template <int D>
__global__ __launch_bounds__(256) void chunk_score_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar,
                                                          int n_kv_heads, int n_chunks, float scale,
                                                          float* __restrict__ scores) {
    const int b = blockIdx.y, p = threadIdx.x % kScoreLanes;
    const int c = blockIdx.x * (256 / kScoreLanes) + threadIdx.x / kScoreLanes;
    const float a = chunk_score<D>(qbar + (size_t)b * n_kv_heads * D, kbar, min(c, n_chunks - 1), n_kv_heads, n_chunks, p);
    if (p == 0 && c < n_chunks) scores[(size_t)b * n_chunks + c] = a * (scale / (float)n_kv_heads);
}

// Scores and selection of up to fused_chunks() chunks in one block per query: a launch less, at the
// price of one compute unit reading all mean keys of a query (2 KiB per chunk at four KV heads):
// 4.1 us at 64 chunks (9.6 with 256 threads and one load at a time), against 4.7 for each of the
// two launches of the separate form.
// A block has threads for no more chunks than there are (16, 32 or 64 at once: starting 16 waves costs more
// than a few chunks take) and requests no more steps than a row has (two up to 32 pieces, otherwise eight).
// us of the whole call with the mean keys there, one form of 16 waves and eight steps -> so: two KV heads,
// D = 64, 4 chunks 6.5 -> 4.8, 19 chunks 6.5 -> 5.0, 64 chunks 6.6 -> 5.3, 128 chunks 8.6 -> 6.0; four KV heads,
// D = 128, 4 chunks 6.5 -> 5.2, 32 chunks 6.5 -> 5.7.
// The line is what one compute unit reads in the time of a launch: 128 chunks, of short rows (512 bytes a chunk) 192 (two
// KV heads, D = 64, with their mean keys: 150 chunks 11.6 -> 8.4 us, eight queries over 200 chunks still 11.4 -> 9.7, but
// 256 chunks of 512 tokens 14.2 -> 14.9; rows of 2 KiB: 130 chunks 11.2 -> 12.4, 200 chunks 11.0 -> 15.4).
constexpr int kShortSteps = 2;                                // steps of a row of up to 32 pieces
constexpr int fused_chunks(int steps) { return steps == kShortSteps ? 192 : 128; }

template <int D, int THREADS, int U>
__global__ __launch_bounds__(THREADS) void score_topk_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar, int n_kv_heads, int n_chunks, int k, float scale,
    int32_t* __restrict__ topk_idx, uint8_t* __restrict__ dense_mask, float* __restrict__ scores) {
    constexpr int AT_ONCE = THREADS / kScoreLanes, MAX = AT_ONCE < 64 ? AT_ONCE : (fused_chunks(U) + 127) / 128 * 128;
    constexpr int GROUPS = (MAX + 63) / 64;
    __shared__ __attribute__((aligned(16))) unsigned long long keys[MAX];
    __shared__ int part[THREADS];
    const int b = blockIdx.x, tid = threadIdx.x, p = tid % kScoreLanes;
#pragma unroll
    for (int base = 0; base < MAX; base += AT_ONCE) {
        const int c = base + tid / kScoreLanes;
        if (base >= n_chunks) break;                          // (uniform)
        const float a = chunk_score<D, U>(qbar + (size_t)b * n_kv_heads * D, kbar, min(c, n_chunks - 1), n_kv_heads,
                                          n_chunks, p) * (scale / (float)n_kv_heads);
        if (p == 0) {
            if (c < n_chunks && scores) scores[(size_t)b * n_chunks + c] = a;
            keys[c] = c < n_chunks ? rank_key(a, c) : 0ull;
        }
    }
    __syncthreads();
    rank_select<THREADS / 64, GROUPS>(keys, part, n_chunks, 0, k, b, topk_idx, dense_mask);
}

// Selection alone, from scores some other kernel has written: 64 chunks per block (grid: chunk
// groups x queries), every block holding the keys of all chunks (at most 32 KiB).
__global__ __launch_bounds__(512) void topk_from_scores_kernel(const float* __restrict__ scores, int n_chunks,
                                                               int k, int32_t* __restrict__ topk_idx,
                                                               uint8_t* __restrict__ dense_mask) {
    extern __shared__ __attribute__((aligned(16))) unsigned long long keys_dyn[];   // [n_chunks, padded to even]
    __shared__ int part[512];
    const int b = blockIdx.y;
    for (int c = threadIdx.x; c < ((n_chunks + 1) & ~1); c += 512)
        keys_dyn[c] = c < n_chunks ? rank_key(scores[(size_t)b * n_chunks + c], c) : 0ull;
    __syncthreads();
    rank_select<8, 1>(keys_dyn, part, n_chunks, blockIdx.x, k, b, topk_idx, dense_mask);
}

// ------------------------------------------------------------------------------------------
// Pooled sparse KVs: chunk c (len rows) is cut into cnt = soff[c+1] - soff[c] consecutive groups,
// group m = rows [floor(m*len/cnt), floor((m+1)*len/cnt)); pooled row soff[c] + m is the mean of
// the group's rows, K and V alike.  LPR lanes per pooled row (a 16-byte piece each), fp32 sums in
// row order, one division, one rounding to the storage dtype.
// Bound by HBM (dense K and V once), as long as enough loads are in flight: four rows of K and of V
// are requested before the first addition, the last two or one of a group by themselves (a whole four
// with repeated rows made groups of one row 10 % slower than one row at a time), a result is stored as
// one piece, and the chunk of a row is found by two or three probes of its LPR lanes instead of a
// chain of halvings.  Eight waves per SIMD: the compiler would widen all rows of a batch first (90
// registers).  K and V of 131,328 tokens (303 MB in and out): 64.5 us with one row at a time and stores
// of two bytes, 61.4 so; 16,384 groups of one row of four heads, D = 128: 18.7 -> 17.6 (repeated rows 20.4).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void st_round(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_round(uint16_t* p, float v) {
    const uint32_t b = __float_as_uint(v);
    const uint32_t up = b + 0x7fffu + ((b >> 16) & 1u);
    *p = (b & 0x7fffffffu) > 0x7f800000u ? 0x7fc0 : (uint16_t)(up >> 16);
}

template <typename T, int D, bool NT>
__global__ __launch_bounds__(256, 8) void pool_sparse_kernel(const T* __restrict__ K, const T* __restrict__ V,
                                                          const int32_t* __restrict__ bounds,
                                                          const int32_t* __restrict__ soff, int n_chunks,
                                                          long long kv_head_u4, long long kv_tok_u4,
                                                          int s_total, T* __restrict__ Ksp,
                                                          T* __restrict__ Vsp) {
    constexpr int EPC = 16 / (int)sizeof(T);        // elements per 16-byte piece
    constexpr int LPR = D / EPC;                    // lanes per row
    constexpr int ROWS = 256 / LPR;
    const int r = blockIdx.x * ROWS + threadIdx.x / LPR, part = threadIdx.x % LPR, g = blockIdx.y;
    if (r >= s_total) return;                       // (all lanes of the row)
    int c = 0;                                      // last chunk with soff[c] <= r: it lies in [c, c + span)
    for (int span = n_chunks; span > 1;) {
        const int step = (span + LPR - 1) / LPR;
        const unsigned long long hit = __ballot(part * step < span && soff[min(c + part * step, n_chunks)] <= r);
        const int last = __popcll((hit >> (threadIdx.x & 63 & ~(LPR - 1))) & ((1ull << LPR) - 1)) - 1;   // (soff ascends, soff[c] <= r)
        c += last * step;
        span = min(step, span - last * step);
    }
    const long long len = bounds[c + 1] - bounds[c], cnt = soff[c + 1] - soff[c], m = r - soff[c];
    const int lo = bounds[c] + (int)((m * len) / cnt), hi = bounds[c] + (int)(((m + 1) * len) / cnt);
    float ak[EPC], av[EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) ak[i] = av[i] = 0.f;
    const size_t first = (size_t)g * kv_head_u4 + (size_t)lo * kv_tok_u4 + part;   // (K, V strides in 16-byte units)
    const uint4 *kp = (const uint4*)K + first, *vp = (const uint4*)V + first;
    auto rows = [&](auto n) __attribute__((always_inline)) {   // the loads of n rows, then their additions
        constexpr int N = decltype(n)::value;
        uint4 kq[N], vq[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            kq[u] = load16<NT>(kp + u * kv_tok_u4);
            vq[u] = load16<NT>(vp + u * kv_tok_u4);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const T* ke = (const T*)&kq[u];
            const T* ve = (const T*)&vq[u];
#pragma unroll
            for (int i = 0; i < EPC; ++i) { ak[i] += ld(ke + i); av[i] += ld(ve + i); }
        }
        kp += N * kv_tok_u4;
        vp += N * kv_tok_u4;
    };
    int left = hi - lo;
#pragma unroll 1
    for (; left >= 4; left -= 4) rows(std::integral_constant<int, 4>{});
    if (left & 2) rows(std::integral_constant<int, 2>{});
    if (left & 1) rows(std::integral_constant<int, 1>{});
    const float n = (float)(hi - lo);
    __attribute__((aligned(16))) T ko[EPC], vo[EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) { st_round(ko + i, ak[i] / n); st_round(vo + i, av[i] / n); }
    const size_t out = ((size_t)g * s_total + r) * LPR + part;
    ((uint4*)Ksp)[out] = *(const uint4*)ko;
    ((uint4*)Vsp)[out] = *(const uint4*)vo;
}

// ------------------------------------------------------------------------------------------
// Gather, one launch.  Every block first forms, in LDS, the exclusive scan of the rows every chunk
// of its query contributes (its length if dense, its sparse-row count otherwise) and where they come from --
// C <= 4096 entries, a few hundred nanoseconds, cheaper than a launch of its own -- and then copies its
// share of the mixed rows: a group of LPR lanes per row (all KV heads, K and V, 16-byte
// accesses), the chunk of a row found by a few probes of its lanes in the scanned offsets.  A block handles
// `groups` consecutive passes of 256 / LPR rows (chosen by the host so that small gathers still
// fill the chip and large ones amortise the scan).  The first block of a query writes mix_len; a query whose
// mixed set does not fit l_cap gets mix_len = -(rows needed) and none of its rows is copied.
// Small calls are a chain of memory round trips: mask, bounds and offsets of a chunk are requested together and
// the rows find them in LDS (one after the other, and again per row -> so, with the decode: three questions on a
// 16k prompt 23.0 -> 22.2 us, 1,000 chunks 34.9 -> 32.7).  Bound by HBM when large.  A head's two loads and two stores follow one another, at
// eight waves per SIMD; FOUR (exactly four KV heads): the pieces of all heads are requested before the first store, at
// four waves per SIMD (the line is at launch_gather).  835 MB in and out, eight mixed sets of 25k rows: 158 us one head
// after the other, 140 us (6.0 TB/s) at four heads together; with eight waves per SIMD 148.
// ONCE, buffers that could exceed the on-package cache: the queries of a batch take turns (block id = block of the query *
// batch + query), so that K and V stay in that cache for all of them, and a query whose rows, times the batch, are more
// than kPastCaches stores them past it (the line is at launch_gather).  By its rows, since the host knows the capacity
// only: with the decode, rows stored past the cache by capacity -> so, eight sets of 5,344 rows in buffers for 30,000
// 87.9 -> 75.5 us, of 8,320 rows 128.1 -> 109.0, one of 36,096 in 100,000 64.7 -> 57.5; full sets unchanged.
// With Kmix == nullptr nothing is copied at all: the call only writes mix_len and src_idx (the row
// map the in-place decode reads the dense and sparse rows through).
// ------------------------------------------------------------------------------------------
constexpr long long kPastCaches = 160ll << 20;
// Chunks up to which a block keeps where a chunk's rows come from in LDS beside the offsets: more would leave room for
// fewer than the eight blocks per compute unit that the heads one after the other run at (FOUR, at four, always does).
// Beyond, a row asks memory for it.  Eight queries, one head, 3,000 chunks of 40 tokens 55.0 -> 42.3 us, three, two heads
// of D = 64, 4,096 of 40, 2,000 dense 74.9 -> 56.7; one query, one head, 4,096 of 32 22.3 -> 23.0.
constexpr int kTableChunks = 2500;

template <int ROW_BYTES, bool FOUR, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FOUR ? 4 : 8, FOUR ? 4 : 8))) void gather_kernel(
    const uint4* __restrict__ K, const uint4* __restrict__ V, const uint8_t* __restrict__ dense_mask,
    const int32_t* __restrict__ bounds, const int32_t* __restrict__ soff, const int32_t* __restrict__ sidx,
    int n_chunks, int n_prefix, long long kv_head_u4, long long kv_tok_u4,   // K, V strides in 16-byte units
    int n_kv_heads, int l_cap, int groups, uint4* __restrict__ Kmix,
    uint4* __restrict__ Vmix, int32_t* __restrict__ mix_len, int32_t* __restrict__ src_idx,
    const uint4* __restrict__ Ksp, const uint4* __restrict__ Vsp, int s_total, int batch) {
    constexpr int LPR = ROW_BYTES / 16;                       // lanes per row
    constexpr int ROWS = 256 / LPR;                           // rows per pass
    extern __shared__ int off[];                              // [n_chunks] first mixed row of every chunk, top bit: dense; then
    int* from = off + n_chunks;                               // (table) [n_chunks] its first token, or -1 - its first kept row
    const bool table = FOUR || n_chunks <= kTableChunks;
    constexpr int DENSE = INT32_MIN;
    __shared__ int wave_tot[4][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = ONCE ? blockIdx.x % batch : blockIdx.y, block = ONCE ? blockIdx.x / batch : blockIdx.x;
    const uint8_t* mask = dense_mask + (size_t)b * n_chunks;
    int len = n_prefix;                                       // rows of the chunks so far
    // The rows every chunk contributes, four 256-chunk passes at a time: their loads are all requested before the
    // first scan and do not wait for the mask (one memory round trip and one barrier per 1,024 chunks).
    for (int base4 = 0; base4 < n_chunks; base4 += 1024) {
        int rows[4], inc[4], flag[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = base4 + u * 256 + tid;
            rows[u] = flag[u] = 0;
            if (c < n_chunks) {
                const int lo = bounds[c], hi = bounds[c + 1], s_lo = soff[c], s_hi = soff[c + 1];
                const bool dense = mask[c] != 0;
                rows[u] = dense ? hi - lo : s_hi - s_lo;
                flag[u] = dense ? DENSE : 0;
                if (table) from[c] = dense ? lo : -1 - s_lo;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (base4 + u * 256 >= n_chunks) break;           // (uniform)
            inc[u] = rows[u];                                 // inclusive scan inside the wave
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(inc[u], o);
                if (lane >= o) inc[u] += t;
            }
            if (lane == 63) wave_tot[u][wave] = inc[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (base4 + u * 256 >= n_chunks) break;
            const int c = base4 + u * 256 + tid;
            int before = len;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int t = wave_tot[u][w];
                before += w < wave ? t : 0;
                len += t;
            }
            if (c < n_chunks) off[c] = (before + inc[u] - rows[u]) | flag[u];
        }
        __syncthreads();                                      // off is there; wave_tot may be written again
    }
    // a mixed set that does not fit l_cap is reported, not truncated: minus the rows it needs
    if (block == 0 && tid == 0) mix_len[b] = len <= l_cap ? len : -len;
    if (len > l_cap) return;
    const bool past = ONCE && 2ll * batch * n_kv_heads * len * ROW_BYTES > kPastCaches;
    const int part = tid % LPR;
    for (int gi = 0; gi < groups; ++gi) {
        const int r = (block * groups + gi) * ROWS + tid / LPR;
        if (r >= len) break;                                  // (rows ascend with gi; the lanes of a row together)
        int src;                                              // token id, or -1 - pooled row
        if (r < n_prefix) {
            src = r;
        } else {
            int c = 0;                                        // last chunk with off[c] <= r: it lies in [c, c + span)
            for (int span = n_chunks; span > 1;) {
                const int step = (span + LPR - 1) / LPR;
                const unsigned long long hit = __ballot(part * step < span && (off[min(c + part * step, n_chunks - 1)] & ~DENSE) <= r);
                const int last = __popcll((hit >> (lane & ~(LPR - 1))) & ((1ull << LPR) - 1)) - 1;
                c += last * step;
                span = min(step, span - last * step);
            }
            const int at = off[c], o = r - (at & ~DENSE);
            const int first = table ? from[c] : at < 0 ? bounds[c] : -1 - soff[c];
            if (first >= 0) src = first + o;
            else src = Ksp ? first - o : sidx[-1 - first + o];
        }
        if (src_idx && part == 0) src_idx[(size_t)b * l_cap + r] = src;
        if (!Kmix) continue;                                  // index-only call: no rows are copied
        const uint4* ks = src >= 0 ? K : Ksp;
        const uint4* vs = src >= 0 ? V : Vsp;
        // the pooled rows are dense [Hkv, S_total, D]; K and V have the caller's strides
        const size_t head_u4 = src >= 0 ? (size_t)kv_head_u4 : (size_t)s_total * LPR;
        const size_t row_u4 = src >= 0 ? (size_t)src * kv_tok_u4 : (size_t)(-1 - src) * LPR;
        const size_t s_off = row_u4 + part, d_off = ((size_t)b * n_kv_heads * l_cap + r) * LPR + part;
        const size_t d_head = (size_t)l_cap * LPR;
        if constexpr (FOUR) {
            uint4 kq[4], vq[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                kq[g] = ks[s_off + g * head_u4];
                vq[g] = vs[s_off + g * head_u4];
            }
            auto store = [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    store16<nt>(Kmix + d_off + g * d_head, kq[g]);
                    store16<nt>(Vmix + d_off + g * d_head, vq[g]);
                }
            };
            if (past) store(std::true_type{}); else store(std::false_type{});
        } else {
            auto copy = [&](auto nt) __attribute__((always_inline)) {
                for (int g = 0; g < n_kv_heads; ++g) {
                    const uint4 kq = ks[s_off + g * head_u4], vq = vs[s_off + g * head_u4];
                    store16<nt>(Kmix + d_off + g * d_head, kq);
                    store16<nt>(Vmix + d_off + g * d_head, vq);
                }
            };
            if (past) copy(std::true_type{}); else copy(std::false_type{});
        }
    }
}

// ------------------------------------------------------------------------------------------
// Gather for several queries at once: a row is read once and written to every mixed set that takes it, where the kernel
// above reads it for each of them (the line is at shared_gather).  A block takes 256 / LPR tokens (prefix rows go to all
// queries, a chunk's rows to those that have it dense) or, behind all of those, as many kept or pooled rows (to those that
// have it sparse), of HEADS KV heads (grid.y).  A block whose rows nobody takes ends when it has the masks: sets that leave
// their buffers nearly empty are mostly such blocks.  The others request their rows and then form, in LDS, where every chunk
// begins in every query's mixed set: a wave per query, scans of 64 chunks, from lengths that all its threads have requested
// at once.
// Bound by the writes.  With all scans before the search, and head counts other than two and four one head after the other ->
// so, us, inputs not in the caches: D = 128, 16 heads, three sets of 6,702 rows in buffers for 19,044 64.0 -> 58.3, four
// heads, eight full sets of 52,648 of 64,428 tokens (863 MB) 212 -> 207; D = 64, eight heads,
// four sets of 2,388 rows in buffers for 33,642 19.0 -> 13.2.
// ------------------------------------------------------------------------------------------
constexpr int kSharedQueries = 32;

template <int ROW_BYTES, int HEADS>                           // HEADS: KV heads whose pieces are in flight together
__global__ __launch_bounds__(256) void gather_shared_kernel(
    const uint4* __restrict__ K, const uint4* __restrict__ V, const uint8_t* __restrict__ dense_mask,
    const int32_t* __restrict__ bounds, const int32_t* __restrict__ soff, const int32_t* __restrict__ sidx,
    int n_chunks, int n_prefix, int n_tokens, int s_total, long long kv_head_u4, long long kv_tok_u4,
    int n_kv_heads, int l_cap, int batch, uint4* __restrict__ Kmix, uint4* __restrict__ Vmix,
    int32_t* __restrict__ mix_len, int32_t* __restrict__ src_idx, const uint4* __restrict__ Ksp, const uint4* __restrict__ Vsp) {
    constexpr int LPR = ROW_BYTES / 16, ROWS = 256 / LPR;     // lanes per row, rows per pass
    constexpr int DENSE = INT32_MIN;
    extern __shared__ int off[];                              // [batch][n_chunks] first mixed row, top bit: dense; then
    int* lo = off + batch * n_chunks;                         // [n_chunks] first token and
    int* so = lo + n_chunks;                                  // [n_chunks] first kept row of every chunk
    __shared__ int lens[kSharedQueries];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, part = tid % LPR;
    for (int c = tid; c < n_chunks; c += 256) { lo[c] = bounds[c]; so[c] = soff[c]; }
    for (int e = tid; e < batch * n_chunks; e += 256) off[e] = dense_mask[e] != 0 ? DENSE : 0;
    __syncthreads();
    const int token_blocks = (n_tokens + ROWS - 1) / ROWS;
    const bool tokens = (int)blockIdx.x < token_blocks;
    const int r = (tokens ? blockIdx.x : blockIdx.x - token_blocks) * ROWS + tid / LPR;      // token, or kept row
    const int* first = tokens ? lo : so;
    int c = -1, o = r;                                        // its chunk (none: the prefix) and place in it
    unsigned takes = 0;                                       // queries that take the row
    if (r < (tokens ? n_tokens : s_total)) {
        takes = ~0u >> (32 - batch);
        if (!tokens || r >= n_prefix) {
            c = 0;                                            // last chunk with first[c] <= r: it lies in [c, c + span)
            for (int span = n_chunks; span > 1;) {
                const int step = (span + LPR - 1) / LPR;
                const unsigned long long hit = __ballot(part * step < span && first[min(c + part * step, n_chunks - 1)] <= r);
                const int last = __popcll((hit >> (lane & ~(LPR - 1))) & ((1ull << LPR) - 1)) - 1;
                c += last * step;
                span = min(step, span - last * step);
            }
            o = r - first[c];
            takes = 0;
            for (int b0 = 0; b0 < batch; b0 += LPR) {             // (a lane of the row per query)
                const unsigned long long hit = __ballot(b0 + part < batch && (off[(b0 + part) * n_chunks + c] < 0) == tokens);
                takes |= (unsigned)((hit >> (lane & ~(LPR - 1))) & ((1ull << LPR) - 1)) << b0;
            }
        }
    }
    // (the first block writes the lengths)
    if (!__syncthreads_or(takes != 0) && (blockIdx.x != 0 || blockIdx.y != 0)) return;
    const int g0 = blockIdx.y * HEADS;
    int src = 0;                                              // token id, or -1 - pooled row
    uint4 kq[HEADS], vq[HEADS];
    if (takes) {                                              // (requested before the scans, which they do not need)
        src = tokens ? r : Ksp ? -1 - r : sidx[r];
        const uint4* ks = src >= 0 ? K : Ksp;
        const uint4* vs = src >= 0 ? V : Vsp;
        const size_t head_u4 = src >= 0 ? (size_t)kv_head_u4 : (size_t)s_total * LPR;
        const size_t s_off = (src >= 0 ? (size_t)src * kv_tok_u4 : (size_t)(-1 - src) * LPR) + part;
#pragma unroll
        for (int g = 0; g < HEADS; ++g) {
            kq[g] = ks[s_off + (g0 + g) * head_u4];
            vq[g] = vs[s_off + (g0 + g) * head_u4];
        }
    }
    for (int b = wave; b < batch; b += 4) {
        int len = n_prefix;
        for (int base = 0; base < n_chunks; base += 64) {
            const int c = base + lane;
            int flag = 0, rows = 0;
            if (c < n_chunks) {
                flag = off[b * n_chunks + c];
                const int* first = flag ? lo : so;
                rows = (c + 1 < n_chunks ? first[c + 1] : flag ? n_tokens : s_total) - first[c];
            }
            int inc = rows;
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(inc, o);
                if (lane >= o) inc += t;
            }
            if (c < n_chunks) off[b * n_chunks + c] = (len + inc - rows) | flag;
            len += __shfl(inc, 63);
        }
        if (lane == 0) {
            lens[b] = len;
            // a mixed set that does not fit l_cap is reported, not truncated: minus the rows it needs
            if (blockIdx.x == 0 && blockIdx.y == 0) mix_len[b] = len <= l_cap ? len : -len;
        }
    }
    __syncthreads();
    unsigned fits = 0;                                        // queries that get rows
    bool past = false;
    for (int b = 0; b < batch; ++b) {
        if (lens[b] <= l_cap) fits |= 1u << b;
        past |= lens[b] <= l_cap && 2ll * batch * n_kv_heads * lens[b] * ROW_BYTES > kPastCaches;
    }
    takes &= fits;
    const size_t d_head = (size_t)l_cap * LPR;
    for (unsigned left = takes; left; left &= left - 1) {
        const int b = __builtin_ctz(left);
        const int row = c >= 0 ? (off[b * n_chunks + c] & ~DENSE) + o : o;
        if (src_idx && part == 0 && g0 == 0) src_idx[(size_t)b * l_cap + row] = src;
        const size_t d_off = ((size_t)b * n_kv_heads * l_cap + row) * LPR + part + g0 * d_head;
        auto store = [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < HEADS; ++g) {
                store16<nt>(Kmix + d_off + g * d_head, kq[g]);
                store16<nt>(Vmix + d_off + g * d_head, vq[g]);
            }
        };
        if (past) store(std::true_type{}); else store(std::false_type{});
    }
}

}  // namespace

// kbar (n_chunks blocks per KV head; skipped when do_chunks is false) and qbar (batch blocks per KV
// head) in one launch.
vxl_status launch_summaries(const vxl_layout* L, const vxl_attn_desc* d, const void* K, float* kbar,
                            bool do_chunks, const void* Qd, int batch, int T, float* qbar, hipStream_t s) {
    const int nc = do_chunks ? L->n_chunks : 0;
    const TokStrides ts = tok_strides(d, L->n_tokens);
    const long long epc = d->dtype == VXL_BF16 ? 8 : 4;       // elements per 16 bytes
    // 512 threads per chunk and KV head where there are few of them, long ones of rows of 256 bytes and more: a block is
    // a chain of round trips (28 heads, D = 128, 256 -> 512 threads: 20 chunks of 1,000 tokens 16.0 -> 10.9 us with the
    // selection, 60 of 700 17.8 -> 14.8; but 64 of 256 10.1 -> 11.1, and 160 of 1,000, 640 blocks, 36.8 -> 41.0), eight
    // rows of a thread at once instead of four unless they are streamed (those 20 chunks 11.4 -> 10.1; 100 of 1,200,
    // streamed, 28.3 -> 28.8; 256 threads: 64 of 256 28.3 -> 28.7 with the rest of a query).
    // Keys beyond 96 MB are streamed past the caches: 164,096 tokens 45.5 -> 40.0; six layers in turn, 104 MB 28.1 -> 24.0,
    // two 23.7 -> 23.3.  Of fewer the on-package cache holds two or three layers, which is then the faster source for a
    // caller that scores so many: 79 MB, two layers in turn 18.6 -> 19.4, 42 MB 13.2 -> 13.7, 17 MB 10.1 -> 10.7; a stack
    // of more finds none of them there and would be streamed sooner (79 MB, six in turn 22.1 -> 20.1).
    // (The choice depends on layout and descriptor alone: means that a caller keeps are those of every later call.)
    const long long elem = d->dtype == VXL_BF16 ? 2 : 4, row = d->head_dim * elem;
    const bool wide = row >= 256 && (long long)L->n_chunks * d->n_kv_heads <= 512 &&
                      (long long)L->n_tokens * row >= 19ll * 256 * 16 * L->n_chunks;
    const bool once = L->n_tokens * (row * d->n_kv_heads) > (96 << 20);
    const int pieces = d->head_dim / (int)epc, n_mean = T > kMeanTokens ? batch * (pieces / kMeanPieces) : 0;
    const int group = d->n_q_heads / d->n_kv_heads;
    const dim3 grid(nc + (n_mean ? n_mean : batch), d->n_kv_heads);
    const size_t smem = (size_t)(n_mean ? std::max(kMeanThreads, group * kMeanPieces) * (int)epc : group * d->head_dim) * sizeof(float);
#define VXL_LAUNCH_AS(T_, D, THREADS, NT)                                                                        \
    hipLaunchKernelGGL((chunk_summarize_kernel<T_, D, THREADS, NT>), grid, dim3(THREADS), smem, s, (const T_*)K,  \
                       L->d_bounds, kbar, ts.kh / epc, ts.kt / epc, nc, n_mean, (const T_*)Qd, qbar, T,     \
                       d->n_q_heads, d->n_kv_heads)
#define VXL_LAUNCH(T_, D)                                                                                        \
    do {                                                                                                         \
        if (wide) { if (once) VXL_LAUNCH_AS(T_, D, 512, true); else VXL_LAUNCH_AS(T_, D, 512, false); }          \
        else { if (once) VXL_LAUNCH_AS(T_, D, 256, true); else VXL_LAUNCH_AS(T_, D, 256, false); }               \
    } while (0)
    if (d->dtype == VXL_F32) { if (d->head_dim == 64) VXL_LAUNCH(float, 64); else VXL_LAUNCH(float, 128); }
    else { if (d->head_dim == 64) VXL_LAUNCH(uint16_t, 64); else VXL_LAUNCH(uint16_t, 128); }
#undef VXL_LAUNCH
#undef VXL_LAUNCH_AS
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

vxl_status launch_score_topk(const vxl_layout* L, const vxl_attn_desc* d, float scale, int batch, int k,
                             const float* qbar, const float* kbar, int32_t* topk_idx, uint8_t* dense_mask,
                             float* scores, float* scores_ws, hipStream_t s) {
    // One block per query reads all its mean keys through one compute unit, so beyond fused_chunks()
    // chunks the scores are formed by 16 chunks per block and the selection reads them back.
    const bool short_rows = d->n_kv_heads * d->head_dim <= kShortSteps * kScoreLanes * 4;
    if (L->n_chunks > fused_chunks(short_rows ? kShortSteps : 8)) {
        float* sc = scores ? scores : scores_ws;
        const dim3 grid((L->n_chunks + 256 / kScoreLanes - 1) / (256 / kScoreLanes), batch);
        if (d->head_dim == 64)
            hipLaunchKernelGGL((chunk_score_kernel<64>), grid, dim3(256), 0, s, qbar, kbar, d->n_kv_heads,
                               L->n_chunks, scale, sc);
        else
            hipLaunchKernelGGL((chunk_score_kernel<128>), grid, dim3(256), 0, s, qbar, kbar, d->n_kv_heads,
                               L->n_chunks, scale, sc);
        VXL_HIP_TRY(hipGetLastError());
        return launch_topk_from_scores(L, sc, batch, k, topk_idx, dense_mask, s);
    }
#define VXL_LAUNCH(D, THREADS, U)                                                                              \
    hipLaunchKernelGGL((score_topk_kernel<D, THREADS, U>), dim3(batch), dim3(THREADS), 0, s, qbar, kbar,         \
                       d->n_kv_heads, L->n_chunks, k, scale, topk_idx, dense_mask, scores)
#define VXL_BY_CHUNKS(D, U)                                                                                     \
    do {                                                                                                        \
        if (L->n_chunks <= 256 / kScoreLanes) VXL_LAUNCH(D, 256, U);                                            \
        else if (L->n_chunks <= 512 / kScoreLanes) VXL_LAUNCH(D, 512, U);                                       \
        else VXL_LAUNCH(D, 1024, U);                                                                            \
    } while (0)
    if (d->head_dim == 64) { if (short_rows) VXL_BY_CHUNKS(64, kShortSteps); else VXL_BY_CHUNKS(64, 8); }
    else { if (short_rows) VXL_BY_CHUNKS(128, kShortSteps); else VXL_BY_CHUNKS(128, 8); }
#undef VXL_BY_CHUNKS
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

vxl_status launch_topk_from_scores(const vxl_layout* L, const float* scores, int batch, int k,
                                   int32_t* topk_idx, uint8_t* dense_mask, hipStream_t s) {
    const size_t smem = (size_t)((L->n_chunks + 1) & ~1) * sizeof(unsigned long long);
    hipLaunchKernelGGL(topk_from_scores_kernel, dim3((L->n_chunks + 63) / 64, batch), dim3(512), smem, s, scores,
                       L->n_chunks, k, topk_idx, dense_mask);
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

vxl_status launch_pool_sparse(const vxl_layout* L, const vxl_attn_desc* d, const void* K, const void* V,
                              void* Ksp, void* Vsp, hipStream_t s) {
    if (L->s_total == 0) return VXL_OK;
    const int epc = d->dtype == VXL_BF16 ? 8 : 4;
    const int rows = 256 / (d->head_dim / epc);
    const dim3 grid((L->s_total + rows - 1) / rows, d->n_kv_heads), block(256);
    const TokStrides ts = tok_strides(d, L->n_tokens);
    // K and V that the 256 MB of the on-package cache do not hold are streamed past it (131,328 tokens, 269 MB, with
    // the in-place decode behind it 123 -> 116 us; but 66,000 tokens, 136 MB, whose rows the decode then reads from
    // there, 113 -> 122).
    const bool once = 2ll * L->n_tokens * d->n_kv_heads * d->head_dim * (16 / epc) > (256ll << 20);
#define VXL_LAUNCH(T, D)                                                                                       \
    do {                                                                                                       \
        hipLaunchKernelGGL((once ? pool_sparse_kernel<T, D, true> : pool_sparse_kernel<T, D, false>), grid, block, 0, s, \
                           (const T*)K, (const T*)V, L->d_bounds, L->d_soff, L->n_chunks, ts.kh / epc, ts.kt / epc, \
                           L->s_total, (T*)Ksp, (T*)Vsp);                                                      \
    } while (0)
    if (d->dtype == VXL_F32) { if (d->head_dim == 64) VXL_LAUNCH(float, 64); else VXL_LAUNCH(float, 128); }
    else { if (d->head_dim == 64) VXL_LAUNCH(uint16_t, 64); else VXL_LAUNCH(uint16_t, 128); }
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

static long long shared_gather_blocks(int row_bytes, int n_tokens, int s_total) {
    const int rows = 256 / (row_bytes / 16);
    return ((long long)n_tokens + rows - 1) / rows + (s_total + rows - 1) / rows;
}

// Several queries that take most rows more than once read each row once.  By the sets' capacity (the host does not know their
// lengths): 45 MB together, two rows per token, 128 blocks of rows per set, chunks x queries few enough for a block's scans,
// and, with more than 16 queries, K and V of 20 MB (below, the caches serve the repeated reads: 28 queries, 2,124 tokens 26.2 ->
// 32.4 us; beyond, 80 random calls 1.28x).  Read per query -> once, us, inputs not in the caches, with the decode behind
// it: eight queries of 35,410 rows of 64,512 tokens 245 -> 231, of 52,648 of 64,428 371 -> 336; D = 64, 16 heads, 16 of 14,694 of 37,016
// 482 -> 377; one head, 8 of 13,262 of 44,901 40.2 -> 33.9; buffers nearly empty, eight heads, three sets of 1,064 rows for
// 5,328 22.8 -> 22.7, D = 64, four of 2,388 for 33,642 56.0 -> 34.0.  Over 450 random calls of 1 to 16 heads, of which two thirds
// leave a third to nearly all of their buffers empty, 1.21; at worst D = 64, sixteen sets of 490 rows for 4,285 20.1 -> 23.0.
static bool shared_gather(const vxl_attn_desc* d, int n_tokens, int s_total, int n_chunks, int batch, int l_cap) {
    const int row_bytes = d->head_dim * (d->dtype == VXL_BF16 ? 2 : 4);
    const long long kv = 2ll * n_tokens * d->n_kv_heads * row_bytes;
    return batch > 1 && batch <= (kv < 20000000ll ? 16 : kSharedQueries) && (long long)batch * n_chunks <= 1024 &&
           shared_gather_blocks(row_bytes, n_tokens, s_total) <= kMaxGridX &&
           2ll * batch * d->n_kv_heads * l_cap * row_bytes >= 45000000ll && (long long)batch * l_cap >= 2ll * n_tokens &&
           l_cap >= 128 * (256 / (row_bytes / 16));
}

// Test hook (vxl_debug.h): whether a gather of these sizes is the one that reads a row once for all queries.
extern "C" int vxl_debug_gather_shared(const vxl_attn_desc* d, int n_tokens, int n_sparse, int n_chunks, int batch, int l_cap) {
    return shared_gather(d, n_tokens, n_sparse, n_chunks, batch, l_cap);
}

vxl_status launch_gather(const vxl_layout* L, const vxl_attn_desc* d, const void* K, const void* V,
                         const void* Ksp, const void* Vsp, const uint8_t* dense_mask, int batch, void* Kmix,
                         void* Vmix, int l_cap, int32_t* mix_len, int32_t* src_idx, hipStream_t s) {
    const int row_bytes = d->head_dim * (d->dtype == VXL_BF16 ? 2 : 4);
    // Exactly four heads go together: one head after the other waits for its own loads four times, which small calls
    // spend most of their time on, and it keeps fewer bytes in flight.  Over 96 sizes of one to eight queries with
    // buffers in turn 1.05x, with the same buffers every time 1.01x.  One head after the other -> together, us:
    // D = 128, bf16, one query of 4,128 rows 10.1 -> 8.1, of 2,368 rows 7.2 -> 5.9; eight of 6,912 rows 51.6 -> 45.1;
    // at worst (20 to 50 MB of mixed rows in HBM) 13.4 -> 13.8 and, D = 64, 12.9 -> 13.7.  Other head counts in
    // groups of four lose up to 18 %: eight heads, D = 128, 987 MB 347 -> 377; sixteen, D = 64, 1,958 MB 602 -> 725.
    const TokStrides ts = tok_strides(d, L->n_tokens);
    const long long epc = d->dtype == VXL_BF16 ? 8 : 4;
    if (Kmix && shared_gather(d, L->n_tokens, L->s_total, L->n_chunks, batch, l_cap)) {
        const unsigned shared_blocks = (unsigned)shared_gather_blocks(row_bytes, L->n_tokens, L->s_total);
        const size_t lds = (size_t)(batch + 2) * L->n_chunks * sizeof(int);
#define VXL_LAUNCH_AS(RB, HEADS)                                                                                        \
    hipLaunchKernelGGL((gather_shared_kernel<RB, HEADS>), dim3(shared_blocks, d->n_kv_heads / HEADS), dim3(256), lds, s,              \
                       (const uint4*)K, (const uint4*)V, dense_mask, L->d_bounds, L->d_soff, L->d_sidx, L->n_chunks,     \
                       L->n_prefix, L->n_tokens, L->s_total, ts.kh / epc, ts.kt / epc, d->n_kv_heads, l_cap, batch,      \
                       (uint4*)Kmix, (uint4*)Vmix, mix_len, src_idx, (const uint4*)Ksp, (const uint4*)Vsp)
#define VXL_LAUNCH(RB)                                                                                                  \
    do {                                                                                                                \
        if (d->n_kv_heads % 4 == 0) VXL_LAUNCH_AS(RB, 4);                                                               \
        else if (d->n_kv_heads % 2 == 0) VXL_LAUNCH_AS(RB, 2);                                                           \
        else VXL_LAUNCH_AS(RB, 1);                                                                                      \
    } while (0)
        if (row_bytes == 128) VXL_LAUNCH(128);
        else if (row_bytes == 256) VXL_LAUNCH(256);
        else VXL_LAUNCH(512);
#undef VXL_LAUNCH
#undef VXL_LAUNCH_AS
        VXL_HIP_TRY(hipGetLastError());
        return VXL_OK;
    }
    const bool four = Kmix && d->n_kv_heads == 4;
    const size_t smem = (size_t)L->n_chunks * (four || L->n_chunks <= kTableChunks ? 2 : 1) * sizeof(int);
    // Mixed sets that would push K and V out of the 256 MB of the on-package cache go past it, queries in turn (here by the
    // capacity, in the kernel by the rows).  With the
    // decode behind it, us: eight queries of 388 MB over 131,328 tokens 228 -> 200, of 344 MB 182 -> 175, of 418 MB on a
    // ragged prompt 250 -> 246; three of 190 MB 119.7 -> 118; one of 336 MB 206 -> 203; but three of 146 MB 103.8 -> 106,
    // one of 134 MB 86 -> 91 (the decode then reads the mixed rows from that cache).
    const bool once = Kmix && 2ll * batch * d->n_kv_heads * l_cap * row_bytes > kPastCaches;
#define VXL_LAUNCH_AS(RB, FOUR, ONCE)                                                              \
    hipLaunchKernelGGL((gather_kernel<RB, FOUR, ONCE>), ONCE ? dim3(blocks * batch) : dim3(blocks, batch), dim3(256), smem, \
                       s, (const uint4*)K, (const uint4*)V, dense_mask, L->d_bounds, L->d_soff, L->d_sidx,  \
                       L->n_chunks, L->n_prefix, ts.kh / epc, ts.kt / epc, d->n_kv_heads, l_cap, groups,    \
                       (uint4*)Kmix, (uint4*)Vmix, mix_len, src_idx, (const uint4*)Ksp, (const uint4*)Vsp,  \
                       L->s_total, batch)
#define VXL_LAUNCH(RB)                                                                             \
    do {                                                                                           \
        constexpr int rows = 256 / (RB / 16);                                                      \
        const long passes = (l_cap + rows - 1) / rows;                                             \
        const int groups = (int)std::max<long>(1, std::min<long>(8, passes * batch / 512));        \
        const unsigned blocks = (unsigned)((passes + groups - 1) / groups);                        \
        if (four) { if (once) VXL_LAUNCH_AS(RB, true, true); else VXL_LAUNCH_AS(RB, true, false); } \
        else { if (once) VXL_LAUNCH_AS(RB, false, true); else VXL_LAUNCH_AS(RB, false, false); }   \
    } while (0)
    if (row_bytes == 128) VXL_LAUNCH(128);
    else if (row_bytes == 256) VXL_LAUNCH(256);
    else VXL_LAUNCH(512);
#undef VXL_LAUNCH
#undef VXL_LAUNCH_AS
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

}  // namespace vxl
