// Softmax attention-mass relevance score (the second reading of the attention-score relevance
// oracle of "Bi-level KVs Decoding"): score[b, c] = mean over (t, h) of the softmax probability
// mass that query token t of head h puts on the dense keys of chunk c, the softmax running over
// ALL tokens (prefix and every chunk).
//
// One pass over the dense keys.  The token range is cut into items (the prefix and every chunk,
// each in pieces of at most kMassPiece keys; table built with the layout).  A workgroup owns one
// (item, KV head, row tile) and produces for each of its stacked query rows, those of all queries one
// after the other, rho = (b*T + t)*G + hg, the pair (m, l): m = a reference logit of the item in base-2 units (no logit of the
// item lies more than 2^30 above it in the exp2 domain), l = sum over the item's keys of
// 2^(logit2 - m).  Two small kernels then combine the items of a row (M = max m,
// L = sum l*2^(m-M)) and add up, per chunk, l*2^(m-M)/L over the rows; both use fixed summation
// orders, so equal inputs give equal scores.  The selection is the same as in the mean-logit mode.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "vxl_internal.h"
#include "vxl_mfma.h"

namespace vxl {

namespace {

__device__ __forceinline__ float ldf(const float* p) { return *p; }
__device__ __forceinline__ float ldf(const uint16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

constexpr float kMassGrow = 1073741824.f;             // 2^30: a lane's sum over a tile from which its row's reference is raised
constexpr int kMassRowTile = 128;                     // stacked query rows per workgroup (4 waves x 32)

// bf16, matrix cores: S^T = K.Q^T per 64-key tile, running (m, l) per query column.
// Bound by the exponentials of a tile (a multiply-add, an exponential and an addition per logit,
// as many issue slots as the matrix instructions take), once the keys come from L2: the row tiles
// of one (item, KV head) are neighbours in the launch order of one XCD (workgroups go to the eight
// XCDs in turn), so that HBM delivers a key once and not once per row tile.  An item's reference is the
// largest logit of its first tile; another maximum is formed only when a tile's sum says that the reference no longer
// fits (`kMassGrow`).  (The logit of the first key instead saves up to 1 %, 173.1 -> 171.2 us at the largest size below, but rounds the
// exponents that count: the error against float64 grew by up to 12 %, to 2.7e-7 where first keys lie 19 octaves below.)  The tiles come by direct loads into two stages, the next one in flight while a tile
// is worked on (through registers the compiler placed the loads behind the arithmetic), four waves per SIMD.
// The queries of a batch score the same keys, so their rows are stacked too (eight queries of 7 rows over
// 164,096 keys, a launch of row tiles per query 206 us, so 46; of 427 rows over 36,000 keys 167 -> 150).
// Where a launch has enough workgroups, CHAIN, one takes several short items in turn and loads its
// queries once.  The whole score and selection, loads behind the arithmetic -> so, us: 448 rows x 4 heads
// over 131,328 keys in 256 chunks 91.7 -> 80.0; 896 rows over 164,096 keys in 640 chunks 217 -> 173 (an item
// per workgroup 186); 56 rows over 131,328 keys 42.9 -> 34.9; 7 rows over 164,096 keys 48.3 -> 40.2.
// Two row blocks per wave (half the operand reads, three waves per SIMD): 79.9 and 182, and slower on
// small calls; a third stage at three waves per SIMD 85 and 204.
template <int D, bool CHAIN, bool ONCE>
__global__ __launch_bounds__(256, 4) void mass_partial_kernel(
    const uint16_t* __restrict__ Qd, const uint16_t* __restrict__ K, const MassItem* __restrict__ items,
    float* __restrict__ part_m, float* __restrict__ part_l, int T_q, int n_q_heads, int n_kv_heads, int group,
    long long kv_head, long long kv_tok, int n_items, int per_wg, int batch, float scale) {   // K strides in elements
    constexpr int TILE = kKeyTile * D;                // elements of one unpadded K tile
    constexpr int PPR = D / 8, RPI = 64 / PPR;        // 16-byte pieces per row, rows per load instruction (1 KiB)
    constexpr int IPW = kKeyTile / RPI / 4;           // load instructions per wave and tile
    __shared__ __attribute__((aligned(16))) uint16_t Ks[2][TILE];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&Ks[0][0];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup id -> (unit = (items, KV head), row tile): id = (unit / 8 * n_rt + rt) * 8 + unit % 8
    const int n_rows = group * T_q, all_rows = batch * n_rows, n_rt = (all_rows + kMassRowTile - 1) / kMassRowTile;
    const unsigned id = folded_id(), xcd = id % kXcds, seq = id / kXcds;
    const unsigned unit = seq / n_rt * kXcds + xcd;
    const int rt = seq % n_rt, g = unit % n_kv_heads;
    int item = unit / n_kv_heads * per_wg;
    if (item >= n_items) return;
    const int item_end = CHAIN ? min(item + per_wg, n_items) : item + 1;
    const int wrow0 = rt * kMassRowTile + wave * 32;
    const bool wave_active = wrow0 < all_rows;          // waves without rows only help with the loads

    const char* kbase = (const char*)(K + (size_t)g * kv_head);
    const uint32_t row_bytes = (uint32_t)kv_tok * 2;
    const int r_in = lane / PPR, pp = lane % PPR;
    uint32_t koff[IPW];                               // row and (swizzled) piece of this lane in a full tile
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
        const int row = (wave + i * 4) * RPI + r_in;
        koff[i] = (uint32_t)row * row_bytes + (pp ^ ((row / (16 / PPR)) & (PPR - 1))) * 16;
    }
    // The tile of the keys [key0, key_end) -> stage; rows past the last key repeat it (their scores are masked).
    auto issue = [&](int key0, int key_end, int stage) __attribute__((always_inline)) {
        const int rlim = min(kKeyTile - 1, key_end - 1 - key0);
        const char* kb = kbase + (size_t)key0 * row_bytes;
        const uint32_t st = lds_base + (uint32_t)stage * (TILE * 2);
        if (rlim == kKeyTile - 1) {
#pragma unroll
            for (int i = 0; i < IPW; ++i) dma16_as<ONCE>(kb, koff[i], st + (wave + i * 4) * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < IPW; ++i) {
                const int row = (wave + i * 4) * RPI + r_in;
                dma16(kb, koff[i] - (uint32_t)(row - min(row, rlim)) * row_bytes, st + (wave + i * 4) * 1024);
            }
        }
    };
    int k_lo = items[item].key_lo, k_hi = items[item].key_hi;
    issue(k_lo, k_hi, 0);
    bf16x8 qreg[1][D / 16];
    size_t part_row;                                  // place of this lane's row in the results of item 0
    {
        const int row = min(wrow0 + l32, all_rows - 1);       // (query b, token t, head in group hg), hg fastest
        part_row = (((size_t)(row / n_rows) * n_kv_heads + g) * n_items) * n_rows + row % n_rows;
        const uint4* src = (const uint4*)(Qd + ((size_t)(row / group) * n_q_heads + g * group + row % group) * D);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qreg[0][ks] = __builtin_bit_cast(bf16x8, src[ks * 2 + hi]);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {             // complete here: no load the compiler knows of is in flight below
            typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
            asm volatile("" :: "v"(__builtin_bit_cast(u32x4, qreg[0][ks])));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    float m_run = 0.f, l_run = 0.f;
    const float c2 = scale * kLog2e;
    int key0 = k_lo;                                  // first key of the tile at hand

    // one tile; false behind the last tile of the last item
    auto step = [&](auto stage) __attribute__((always_inline)) {
        const bool item_ends = key0 + kKeyTile >= k_hi;
        int nk_lo = 0, nk_hi = 0;
        if (CHAIN && item_ends && item + 1 < item_end) {
            nk_lo = items[item + 1].key_lo;
            nk_hi = items[item + 1].key_hi;
        }
        wait_vmcnt<0>();                              // this wave's part of the tile has landed ...
        __builtin_amdgcn_s_barrier();                 // ... and everyone's; the other stage is free
        if (!item_ends) issue(key0 + kKeyTile, k_hi, stage ^ 1);
        else if (CHAIN && item + 1 < item_end) issue(nk_lo, nk_hi, stage ^ 1);
        if (wave_active) {
            f32x16 s[1][2];
            qk_tile_ahead<D, 1>(Ks[stage], qreg, l32, hi, s);
            if (key0 + kKeyTile > k_hi) {
                const int lim = k_hi - key0 - 1;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        s[0][kb][r] = acc_key(kb, r, hi) <= lim ? s[0][kb][r] : -INFINITY;
            }
            auto row_max = [&]() __attribute__((always_inline)) {     // (every tile holds at least one valid key)
                float mx = s[0][0][0];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[0][kb][r]);
                return fmaxf(mx, __shfl_xor(mx, 32));
            };
            if (key0 == k_lo) { m_run = row_max(); l_run = 0.f; }
            auto exp_sum = [&](float mc) __attribute__((always_inline)) {
                float sum[4];
#pragma unroll
                for (int r = 0; r < 32; r += 8) {
                    float e[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) e[i] = fmaf(s[0][(r + i) >> 4][(r + i) & 15], c2, -mc);
#pragma unroll
                    for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_exp2f(e[i]);
#pragma unroll
                    for (int i = 0; i < 8; ++i) sum[i & 3] = r + i < 4 ? e[i] : sum[i & 3] + e[i];
                }
                return (sum[0] + sum[1]) + (sum[2] + sum[3]);
            };
            // (a sum that is too large or not a number; a row, both its lanes, decides for itself: the rows of a
            // wave may belong to several queries, whose scores do not depend on one another)
            float sum = exp_sum(m_run * c2);
            const uint64_t lanes = __builtin_amdgcn_ballot_w64(!(sum <= kMassGrow));
            if (lanes != 0) {
                const bool row_grows = (((uint32_t)lanes | (uint32_t)(lanes >> 32)) >> l32 & 1) != 0;
                const float mx = row_max();
                const float m_new = row_grows ? fmaxf(m_run, mx) : m_run;
                l_run *= row_grows ? __builtin_amdgcn_exp2f((m_run - m_new) * c2) : 1.f;
                m_run = m_new;
                sum = exp_sum(m_run * c2);
            }
            l_run += sum;
            if (item_ends) {
                const float l_tot = l_run + __shfl_xor(l_run, 32);
                if (wrow0 + l32 < all_rows && hi == 0) {
                    const size_t idx = part_row + (size_t)item * n_rows;
                    part_m[idx] = m_run * c2;
                    part_l[idx] = l_tot;
                }
            }
        }
        if (!item_ends) { key0 += kKeyTile; return true; }
        if (!CHAIN) return false;
        k_lo = key0 = nk_lo;
        k_hi = nk_hi;
        return ++item < item_end;
    };
    if constexpr (CHAIN) while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {}
    else for (int stage = 0; step(stage); stage ^= 1) {}
}

__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Vector-ALU form (fp32 arithmetic): one wavefront per query row, a lane per key.  Serves the F32
// storage dtype and, for BF16, an on-device cross-check of the matrix-core kernel.
template <typename T, int D>
__global__ __launch_bounds__(256) void mass_partial_simple_kernel(
    const T* __restrict__ Qd, const T* __restrict__ K, const MassItem* __restrict__ items,
    float* __restrict__ part_m, float* __restrict__ part_l, int T_q, int n_q_heads, int n_kv_heads, int group,
    long long kv_head, long long kv_tok, int n_items, float scale) {   // K strides in elements
    __shared__ float q_lds[4][D];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int item = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    const int n_rows = group * T_q;
    const int k_lo = items[item].key_lo, k_hi = items[item].key_hi;
    const float c2 = scale * kLog2e;
    const T* kbase = K + (size_t)g * kv_head;
    for (int rho = wave; rho < n_rows; rho += 4) {
        const int t = rho / group, hg = rho % group;
        const T* qrow = Qd + (((size_t)b * T_q + t) * n_q_heads + g * group + hg) * D;
#pragma unroll
        for (int x = 0; x < D / 64; ++x) q_lds[wave][lane + 64 * x] = ldf(qrow + lane + 64 * x);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        float m = -INFINITY, l = 0.f;
        for (int base = k_lo; base < k_hi; base += 64) {
            const int j = base + lane;
            const bool valid = j < k_hi;
            float s = -INFINITY;
            if (valid) {
                const T* kp = kbase + (size_t)j * kv_tok;
                float a = 0.f;
#pragma unroll 8
                for (int d = 0; d < D; ++d) a = fmaf(q_lds[wave][d], ldf(kp + d), a);
                s = a * c2;
            }
            const float m_new = fmaxf(m, wave_max(s));
            const float p = valid ? exp2f(s - m_new) : 0.f;
            l = l * exp2f(m - m_new) + wave_sum(p);
            m = m_new;
        }
        if (lane == 0) {
            const size_t idx = (((size_t)b * n_kv_heads + g) * n_items + item) * (size_t)n_rows + rho;
            part_m[idx] = m;
            part_l[idx] = l;
        }
        __builtin_amdgcn_wave_barrier();               // q_lds[wave] is rewritten by the next row
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Per stacked row (b, g, rho): M = max over the items of m, 1/L with L = sum l * 2^(m - M).  A block
// handles 32 consecutive rows of one (b, g): thread (ig, r) folds the items ig, ig + GROUPS, ... of
// row r into a running (M, L), U items at a time whose loads are all requested first (coalesced
// over the rows); then the maximum over the GROUPS partial pairs of a row, and their sum in group
// order -- a fixed summation order without a chain of exponentials.  Bound by latency: few rows, up
// to hundreds of items each.  Per launch, 448 rows x 4 heads, items taken one by one by eight groups
// and folded pair by pair -> so: 8 items 2.5 -> 2.1 us, 64 items 3.7 -> 2.5, 257 items 8.2 -> 3.8.
template <int GROUPS, int U>
__global__ __launch_bounds__(32 * GROUPS) void mass_rowstat_kernel(const float* __restrict__ part_m,
                                                                   const float* __restrict__ part_l,
                                                                   float* __restrict__ row_m,
                                                                   float* __restrict__ row_il, int n_items,
                                                                   int n_rows) {
    __shared__ float sm[GROUPS][32], sl[GROUPS][32];
    const int r = threadIdx.x & 31, ig = threadIdx.x >> 5;
    const int rho = blockIdx.x * 32 + r;
    const size_t bg = blockIdx.y;
    float M = -INFINITY, L = 0.f;
    if (rho < n_rows) {
        const size_t base = bg * n_items * n_rows + rho;
        for (int it = ig; it < n_items; it += U * GROUPS) {
            float m[U], l[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t idx = base + (size_t)min(it + u * GROUPS, n_items - 1) * n_rows;
                m[u] = part_m[idx];
                l[u] = part_l[idx];
            }
            float Mn = M;
#pragma unroll
            for (int u = 0; u < U; ++u) Mn = fmaxf(Mn, m[u]);  // (a clamped item is one of the row's: the maximum stands)
            L *= exp2f(M - Mn);                                // (M = -inf: L = 0 and 2^-inf = 0)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (it + u * GROUPS < n_items) L += l[u] * exp2f(m[u] - Mn);
            M = Mn;
        }
    }
    sm[ig][r] = M;
    sl[ig][r] = L;
    __syncthreads();
    if (ig == 0 && rho < n_rows) {
        float Mr = M;
#pragma unroll
        for (int k = 1; k < GROUPS; ++k) Mr = fmaxf(Mr, sm[k][r]);
        float Lr = L * exp2f(M - Mr);
#pragma unroll
        for (int k = 1; k < GROUPS; ++k) Lr += sl[k][r] * exp2f(sm[k][r] - Mr);   // (a group without items: 0 * 2^-inf)
        row_m[bg * n_rows + rho] = Mr;
        row_il[bg * n_rows + rho] = 1.f / Lr;
    }
}

// One block per (chunk c, query b): score = (1 / (T * Hq)) * sum over the stacked rows of all KV
// heads of [sum over the items of c of l * 2^(m - M_row)] / L_row.  A thread adds its rows
// r = tid, tid + blockDim.x, ... in that order; the partial sums are added in a fixed tree.
// Latency bound (a chain of loads per row): 512 threads where a chunk has more than 256 rows
// (1,792 rows, 256 chunks: 6.6 us with 256 threads, 4.8 with 512).
constexpr int kChunkThreads = 512;

__global__ __launch_bounds__(kChunkThreads) void mass_chunk_kernel(const float* __restrict__ part_m,
                                                         const float* __restrict__ part_l,
                                                         const float* __restrict__ row_m,
                                                         const float* __restrict__ row_il,
                                                         const int32_t* __restrict__ item_off,
                                                         float* __restrict__ scores, int n_items, int n_rows,
                                                         int n_kv_heads, int n_chunks, float inv_count) {
    __shared__ float wsum[kChunkThreads / 64];
    const int c = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int i0 = item_off[c], i1 = item_off[c + 1];
    const int total = n_kv_heads * n_rows;
    float acc = 0.f;
    for (int r = tid; r < total; r += (int)blockDim.x) {
        const int g = r / n_rows, rho = r % n_rows;
        const size_t bg = (size_t)b * n_kv_heads + g;
        const float M = row_m[bg * n_rows + rho];
        float a = 0.f;
        for (int it = i0; it < i1; ++it) {
            const size_t idx = (bg * n_items + it) * (size_t)n_rows + rho;
            a = fmaf(part_l[idx], exp2f(part_m[idx] - M), a);
        }
        acc = fmaf(a, row_il[bg * n_rows + rho], acc);
    }
    acc = wave_sum(acc);
    if ((tid & 63) == 0) wsum[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        float total_sum = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
        if (blockDim.x > 256) total_sum += (wsum[4] + wsum[5]) + (wsum[6] + wsum[7]);
        scores[(size_t)b * n_chunks + c] = total_sum * inv_count;
    }
}

}  // namespace

MassPlan mass_plan(const vxl_layout* L, const vxl_attn_desc* d, int batch, int T) {
    MassPlan p{};
    const size_t rows = (size_t)(d->n_q_heads / d->n_kv_heads) * T;
    const size_t bg = (size_t)batch * d->n_kv_heads;
    size_t off = 0;
    p.part_m = off;  off += align_up(bg * L->n_mass_items * rows * sizeof(float), 256);
    p.part_l = off;  off += align_up(bg * L->n_mass_items * rows * sizeof(float), 256);
    p.row_m = off;   off += align_up(bg * rows * sizeof(float), 256);
    p.row_il = off;  off += align_up(bg * rows * sizeof(float), 256);
    p.scores = off;  off += align_up((size_t)batch * std::max(1, L->n_chunks) * sizeof(float), 256);
    p.total = off;
    return p;
}

// Items that a workgroup takes one after the other: up to some 16 tiles of keys, while the launch keeps 2,048
// workgroups (twice what the chip holds).
static int mass_items_per_workgroup(const vxl_layout* L, long long workgroups) {
    const long long tiles = std::max<long long>(1, (long long)L->n_tokens / kKeyTile / L->n_mass_items);
    return (int)std::max<long long>(1, std::min((16 + tiles - 1) / tiles, workgroups / 2048));
}

vxl_status launch_score_mass(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Qd,
                             int batch, int T, const void* K, float* scores, void* ws, bool force_simple,
                             hipStream_t s) {
    const MassPlan p = mass_plan(L, d, batch, T);
    float* part_m = (float*)((char*)ws + p.part_m);
    float* part_l = (float*)((char*)ws + p.part_l);
    float* row_m = (float*)((char*)ws + p.row_m);
    float* row_il = (float*)((char*)ws + p.row_il);
    const int group = d->n_q_heads / d->n_kv_heads;
    const int n_rows = group * T;
    const int n_items = L->n_mass_items;
    const TokStrides ts = tok_strides(d, L->n_tokens);
    if (d->dtype == VXL_BF16 && !force_simple) {
        const long long all_rows = (long long)batch * n_rows, n_rt = (all_rows + kMassRowTile - 1) / kMassRowTile;
        // One row tile reads a key once: keys that the eight L2s (32 MB) do not hold are streamed past the caches
        // (164,096 tokens, 7 rows 45.2 -> 41.7 us, 84 rows 49.7 -> 45.5; 77,056 tokens, 126 rows 31.9 -> 30.7; but two
        // row tiles and more 83.4 -> 87.3, and 4 MB 15.7 -> 16.0).
        const bool once = n_rt == 1 && 2ll * L->n_tokens * d->n_kv_heads * d->head_dim > (32 << 20);
        const int per_wg = once ? 1 : mass_items_per_workgroup(L, n_items * d->n_kv_heads * n_rt);
        const long long units = (long long)((n_items + per_wg - 1) / per_wg) * d->n_kv_heads;
        const dim3 grid = folded_grid((units + kXcds - 1) / kXcds * kXcds * n_rt);
#define VXL_LAUNCH_AS(D, CHAIN, ONCE)                                                                   \
    hipLaunchKernelGGL((mass_partial_kernel<D, CHAIN, ONCE>), grid, dim3(256), 0, s, (const uint16_t*)Qd, \
                       (const uint16_t*)K, L->d_mass_items, part_m, part_l, T, d->n_q_heads,            \
                       d->n_kv_heads, group, ts.kh, ts.kt, n_items, per_wg, batch, scale)
#define VXL_LAUNCH(D)                                                                                   \
    do {                                                                                                \
        if (once) VXL_LAUNCH_AS(D, false, true);                                                        \
        else if (per_wg > 1) VXL_LAUNCH_AS(D, true, false);                                             \
        else VXL_LAUNCH_AS(D, false, false);                                                            \
    } while (0)
        if (d->head_dim == 64) VXL_LAUNCH(64); else VXL_LAUNCH(128);
#undef VXL_LAUNCH_AS
#undef VXL_LAUNCH
    } else {
        const dim3 grid(n_items, d->n_kv_heads, batch);
#define VXL_LAUNCH(T_, D)                                                                               \
    hipLaunchKernelGGL((mass_partial_simple_kernel<T_, D>), grid, dim3(256), 0, s, (const T_*)Qd,       \
                       (const T_*)K, L->d_mass_items, part_m, part_l, T, d->n_q_heads, d->n_kv_heads,   \
                       group, ts.kh, ts.kt, n_items, scale)
        if (d->dtype == VXL_F32) { if (d->head_dim == 64) VXL_LAUNCH(float, 64); else VXL_LAUNCH(float, 128); }
        else { if (d->head_dim == 64) VXL_LAUNCH(uint16_t, 64); else VXL_LAUNCH(uint16_t, 128); }
#undef VXL_LAUNCH
    }
    VXL_HIP_TRY(hipGetLastError());
    const dim3 stat_grid((n_rows + 31) / 32, batch * d->n_kv_heads);
    // Up to 16 items eight groups hold them in one batch; more loads per thread or groups only cost there
    // (1 row, 8 items: 2.1 us, with sixteen groups of four loads 2.5).  Sixteen groups of four up to a few
    // hundred items (1 row, 64 items 2.6 against 3.2 with 32 groups; 448 rows, 257 items 3.8 against 4.0),
    // 32 groups beyond (1 row, 641 items 6.9 against 9.2; 896 rows x 8 heads 7.1 against 7.9).
    if (n_items > 512)
        hipLaunchKernelGGL((mass_rowstat_kernel<32, 4>), stat_grid, dim3(32 * 32), 0, s, part_m, part_l, row_m, row_il,
                           n_items, n_rows);
    else if (n_items > 16)
        hipLaunchKernelGGL((mass_rowstat_kernel<16, 4>), stat_grid, dim3(32 * 16), 0, s, part_m, part_l, row_m, row_il,
                           n_items, n_rows);
    else
        hipLaunchKernelGGL((mass_rowstat_kernel<8, 2>), stat_grid, dim3(32 * 8), 0, s, part_m, part_l, row_m, row_il,
                           n_items, n_rows);
    VXL_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(mass_chunk_kernel, dim3(L->n_chunks, batch),
                       dim3(d->n_kv_heads * n_rows > 256 ? kChunkThreads : 256), 0, s, part_m, part_l, row_m,
                       row_il, L->d_mass_off, scores, n_items, n_rows, d->n_kv_heads, L->n_chunks,
                       1.f / ((float)T * (float)d->n_q_heads));
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

}  // namespace vxl
