// fp32 storage: pre-filling and decode attention on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation -- the 1e-5 tolerance of this storage
// type rules out bf16 operands), softmax with expf.
//
// fp32 is the type of small prompts, whose calls are bound by latency: rows are few and the serial
// walk over the keys is the call.  A wave therefore takes 16 stacked query rows (rho = t * G + head
// in group, so that short chunks and small groups still fill a block) and only a slice of the keys;
// the waves of a workgroup share the keys of a block and are merged through LDS.  Operands come
// straight from global memory into registers in an order that both products can use as it is:
//   S^T = K.Q^T    A: lane (i = lane % 16, j = lane / 16) holds K[key i][16*s + 4*j + e], B: Q[row i]
//                  of the same pieces, one instruction per element e of a 16-byte piece;
//                  result register r of a lane: key 4*j + r, row i
//   O^T = V^T.P^T  step r takes the keys {4*j + r}: B is the lane's own probability, A the lane's
//                  V[key 4*j + r][64*blk + 4*i + e], again one instruction per element of a piece;
//                  result register r' of (blk, e): O[row i][64*blk + 16*j + 4*r' + e]
// so there is no transposition, no LDS and no cross-lane traffic but the row maximum, and every
// load is 16 bytes per lane (64 contiguous bytes per key row for K, 256 for V).  At D = 64 the K pieces of
// the next tile are requested before the softmax of the current one; at D = 128 a tile requests its own
// (a wave has few tiles, and one tile's pieces more cost registers and a wait at the end: pre-filling of 1,335
// tokens, 8 query heads on 4 KV heads, 44.0 us ahead, 42.8 so).
//
// A wave that owns one query row and adds one key at a time took, at 576 tokens, two heads and
// D = 64, 51 us for the pre-filling and 95 us for 8 query tokens over 352 mixed rows; these kernels
// take 8.6 and 10.3.
#include <math.h>

#include <algorithm>

#include "vxl_internal.h"
#include "vxl_mfma.h"

namespace vxl {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kF32Rows = 16;         // stacked query rows per block
constexpr int kF32Band = 128;        // query tokens per entry of the pre-filling's work list
constexpr int kDecodeKB = 2;         // blocks of 16 keys per tile of the decode

// Rows of a contiguous pair of buffers: slot = row.
struct RowsPlain {
    const float *k, *v;
    int d;
    __device__ __forceinline__ int entry(int slot) const { return slot; }
    __device__ __forceinline__ const float* krow(int e) const { return k + (size_t)e * d; }
    __device__ __forceinline__ const float* vrow(int e) const { return v + (size_t)e * d; }
};
// Pre-filling: history slots through the layout's slot table, then the segment's own tokens.
struct RowsSegment {
    const float *k, *v;
    const int32_t* tile_src;
    int ctx, own0;                   // history slots; token of slot ctx
    long long tok;                   // elements between rows
    __device__ __forceinline__ int entry(int slot) const {
        const int h = tile_src[min(slot, max(ctx - 1, 0))];
        return slot < ctx ? h : own0 + slot - ctx;
    }
    __device__ __forceinline__ const float* krow(int e) const { return k + (size_t)e * tok; }
    __device__ __forceinline__ const float* vrow(int e) const { return v + (size_t)e * tok; }
};
// In-place decode: entry e >= 0 is token e, e < 0 row -1 - e of the sparse buffers.
struct RowsMapped {
    const float *k, *v, *ksp, *vsp;
    const int32_t* src;
    int d;
    long long tok;
    __device__ __forceinline__ int entry(int slot) const { return src[slot]; }
    __device__ __forceinline__ const float* krow(int e) const { return e >= 0 ? k + (size_t)e * tok : ksp + (size_t)~e * d; }
    __device__ __forceinline__ const float* vrow(int e) const { return e >= 0 ? v + (size_t)e * tok : vsp + (size_t)~e * d; }
};

template <int D>
__device__ __forceinline__ void load_q_f32(const float* qrow, float4 (&q)[D / 16]) {
    const int j = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) q[s] = *(const float4*)(qrow + 16 * s + 4 * j);
}

// One wave: 16 query rows (pieces in q) over the slots [lo, hi); slots beyond `lim` (per lane: the
// lane's own row) are masked.  m, l: running maximum and this lane's share of the running sum.
template <int D, int KB, typename Rows>
__device__ __forceinline__ void attend_tiles(const Rows& rows, const float4 (&q)[D / 16], int lo, int hi, int lim,
                                             float scale, float& m, float& l, f32x4 (&o)[D / 16]) {
    constexpr int TILE = 16 * KB;                             // keys per tile
    const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
    if (lo >= hi) return;
    float4 k[KB][D / 16], v[KB][4][D / 64];
    int ent[KB];
    auto entries = [&](int t, int (&e)[KB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) e[kb] = rows.entry(min(t + kb * 16 + i, hi - 1));
    };
    auto load_k = [&](const int (&e)[KB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const float* p = rows.krow(e[kb]) + 4 * j;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) k[kb][s] = *(const float4*)(p + 16 * s);
        }
    };
    entries(lo, ent);
    if (D == 64) load_k(ent);
    for (int t = lo; t < hi; t += TILE) {
        int next[KB];
        if (D == 128) load_k(ent);
        entries(min(t + TILE, hi - 1), next);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float* p = rows.vrow(__shfl(ent[kb], 4 * j + r)) + 4 * i;
#pragma unroll
                for (int b = 0; b < D / 64; ++b) v[kb][r][b] = *(const float4*)(p + 64 * b);
            }
        f32x4 s[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < D / 16; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    s[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(((const float*)&k[kb][x])[e], ((const float*)&q[x])[e],
                                                                 s[kb], 0, 0, 0);
        if (D == 64) load_k(next);                            // (the last tile fetches its last row again)
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int slot = t + kb * 16 + 4 * j + r;
                s[kb][r] = slot < hi && slot <= lim ? s[kb][r] * scale : -INFINITY;
                mx = fmaxf(mx, s[kb][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        const float ref = m_new == -INFINITY ? 0.f : m_new;  // (no visible key yet)
        const float alpha = expf(m - ref);
        m = m_new;
        float sum = 0.f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[kb][r] = expf(s[kb][r] - ref);
                sum += s[kb][r];
            }
        l = l * alpha + sum;
#pragma unroll
        for (int x = 0; x < D / 16; ++x) o[x] *= alpha;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < D / 16; ++x)
                    o[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(((const float*)&v[kb][r][x / 4])[x % 4], s[kb][r], o[x],
                                                                0, 0, 0);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) ent[kb] = next[kb];
    }
}

// The same row by row, a key per lane for the scores and a column per lane for O, over the slots a row sees
// and no others.
template <int D, typename Rows, typename QRow>
__device__ __forceinline__ void attend_rows(const Rows& rows, QRow q_row, int lo, int hi, int lim, float scale, float& m,
                                            float& l, f32x4 (&o)[D / 16]) {
    const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
#pragma unroll 1
    for (int row = 0; row < kF32Rows; ++row) {
        const int last = min(hi - 1, __builtin_amdgcn_readlane(lim, row));
        const float* qp = q_row(row);
        float m_row = -INFINITY, l_row = 0.f, acc[D / 64];
#pragma unroll
        for (int x = 0; x < D / 64; ++x) acc[x] = 0.f;
#pragma unroll 1
        for (int t = lo; t <= last; t += 64) {
            const int ent = rows.entry(min(t + lane, last));
            const float* kp = rows.krow(ent);
            float s = 0.f;
#pragma unroll 1
            for (int d = 0; d < D; d += 4) {
                const float4 qd = *(const float4*)(qp + d), kd = *(const float4*)(kp + d);
                s = fmaf(qd.w, kd.w, fmaf(qd.z, kd.z, fmaf(qd.y, kd.y, fmaf(qd.x, kd.x, s))));
            }
            s = t + lane <= last ? s * scale : -INFINITY;
            float m_new = s, sum;
#pragma unroll
            for (int x = 32; x > 0; x >>= 1) m_new = fmaxf(m_new, __shfl_xor(m_new, x));
            m_new = fmaxf(m_new, m_row);
            const float ref = m_new == -INFINITY ? 0.f : m_new, alpha = expf(m_row - ref), p = expf(s - ref);
            sum = p;
#pragma unroll
            for (int x = 32; x > 0; x >>= 1) sum += __shfl_xor(sum, x);
            l_row = l_row * alpha + sum;
            m_row = m_new;
#pragma unroll
            for (int x = 0; x < D / 64; ++x) acc[x] *= alpha;
#pragma unroll 1
            for (int key = 0; key <= min(63, last - t); ++key) {
                const float* vp = rows.vrow(__shfl(ent, key)) + lane;
                const float pk = __shfl(p, key);
#pragma unroll
                for (int x = 0; x < D / 64; ++x) acc[x] = fmaf(pk, vp[64 * x], acc[x]);
            }
        }
        if (i == row) {
            m = m_row;
            l = j == 0 ? l_row : 0.f;
        }
#pragma unroll
        for (int x = 0; x < D / 16; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = __shfl(acc[x / 4], 16 * j + 4 * r + x % 4);
                if (i == row) o[x][r] = v;
            }
    }
}

// A row's result depends on nothing but the slots it sees.  In a tile, a slot that a row does not see (beyond
// its limit, or the repetitions behind the last slot) enters the product as 0 * V, which is 0 only while V is
// finite; a result that is not finite is therefore formed again without the tiles, in a loop so small that the
// tiles keep their registers (without check and loop -> with them, 4 KV heads: D = 128, eight queries of two
// rows over 390 keys 14.1 -> 14.6 us; D = 64, pre-filling of 847 tokens 9.7 -> 9.9).  q_row(row): the Q row.
template <int D, int KB, typename Rows, typename QRow>
__device__ __forceinline__ void attend_f32(const Rows& rows, QRow q_row, int lo, int hi, int lim, float scale, float& m,
                                           float& l, f32x4 (&o)[D / 16]) {
    float4 q[D / 16];
    load_q_f32<D>(q_row(threadIdx.x & 15), q);
    attend_tiles<D, KB>(rows, q, lo, hi, lim, scale, m, l, o);
    float z = 0.f;                                            // stays 0, or NaN
#pragma unroll
    for (int x = 0; x < D / 16; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(o[x][r], 0.f, z);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != z) != 0, 0))
        attend_rows<D>(rows, q_row, lo, hi, lim, scale, m, l, o);
}

// LSE of a row that sees a key: like its O not a number if all its logits are -inf or one is NaN or +inf.
__device__ __forceinline__ float lse_f32(float m, float l) { return l > 0.f ? m + logf(l) : NAN; }

// The waves of one block of rows, merged in wave order through LDS: every wave leaves its (m, l, O),
// then thread `tid` of `n_thr` forms the elements tid, tid + n_thr, ... of the 16 x D block and hands
// them, four neighbouring d at a time, to store(row, d, float4 O, float lse).  A block that sees no key at
// all (`some` false) has O = 0 and LSE = -inf.  RAW: store(row, d, sum of O, (reference, sum)), for a later merge.
template <int D, int W, bool RAW = false>
struct MergeF32 {
    static constexpr int ROW = D + 4;                         // (padded: 16 rows in distinct banks)
    static constexpr int FLOATS = W * (kF32Rows * ROW + 2 * kF32Rows);
    template <typename Store>
    static __device__ __forceinline__ void run(float* lds, int w, int tid, int n_thr, float m, float l,
                                               const f32x4 (&o)[D / 16], bool some, Store store) {
        const int lane = threadIdx.x & 63, i = lane & 15, j = lane >> 4;
        float* stat = lds + W * kF32Rows * ROW;               // [W][16][2]
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (j == 0) { stat[(w * kF32Rows + i) * 2] = m; stat[(w * kF32Rows + i) * 2 + 1] = l; }
        float* dst = lds + (w * kF32Rows + i) * ROW + 16 * j;
#pragma unroll
        for (int b = 0; b < D / 64; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *(float4*)(dst + 64 * b + 4 * r) = make_float4(o[b * 4][r], o[b * 4 + 1][r], o[b * 4 + 2][r], o[b * 4 + 3][r]);
        __syncthreads();
        for (int e = tid; e < kF32Rows * D / 4; e += n_thr) {
            const int row = e / (D / 4), d = (e % (D / 4)) * 4;
            float M = -INFINITY;
#pragma unroll
            for (int x = 0; x < W; ++x) M = fmaxf(M, stat[(x * kF32Rows + row) * 2]);
            const float ref = M == -INFINITY ? 0.f : M;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            float L = 0.f;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const float f = expf(stat[(x * kF32Rows + row) * 2] - ref);
                const float4 p = *(const float4*)(lds + (x * kF32Rows + row) * ROW + d);
                L = fmaf(f, stat[(x * kF32Rows + row) * 2 + 1], L);
                a.x = fmaf(f, p.x, a.x); a.y = fmaf(f, p.y, a.y); a.z = fmaf(f, p.z, a.z); a.w = fmaf(f, p.w, a.w);
            }
            if constexpr (RAW) {
                store(row, d, a, make_float2(M, L));
            } else {
                const float inv = some ? 1.f / L : 0.f;
                store(row, d, make_float4(a.x * inv, a.y * inv, a.z * inv, a.w * inv), some ? lse_f32(M, L) : -INFINITY);
            }
        }
    }
};

// Pre-filling.  grid: bands of 128 tokens of the work list, heaviest first, x row blocks of the longest band x KV heads;
// LONG_FIRST: row blocks x bands x heads in one dimension (folded_grid).  The four waves of a workgroup share the keys of a block: loads go unhidden while few waves
// are in flight (one wave per block from 4 blocks per compute unit on -> four waves, 8 heads on 4 KV heads, us: D = 64,
// 2,064 tokens 53.1 -> 31.3, 20,064 tokens 876 -> 733; D = 128 92.2 -> 59.3 and 1,731 -> 1,565).
// LONG_FIRST, more blocks than compute units: a workgroup's walk over the keys is long against the call, so the long ones
// begin first: the last row blocks of all bands and heads, and so on (bands, then row blocks from the first on, then
// heads 56.0 -> 51.6 us at 2,064 tokens, D = 128; 26.0 -> 22.6 at 864); and tiles of 16 keys, since a wave's share is a
// whole number of tiles and 32 leave more waves waiting (21.7 -> 19.9 at 1,264 tokens, D = 64; D = 128, 2,064 tokens 59.3
// -> 56.1).  Otherwise all run at once, spread evenly in the plain order, and a tile is a round trip: 2 heads on one KV
// head, 576 tokens, D = 64, 8.1 us against 8.5, 4 heads on two, 877 tokens 12.7 against 14.9.
// Blocks that no band has are not launched: 2,064 tokens in chunks of 50, D = 64, 28.4 -> 22.4.
// Matrix pipes 30 % busy at 2,064 tokens, D = 128.
template <int D, bool LONG_FIRST>
__global__ __launch_bounds__(256, LONG_FIRST ? 3 : 2) void prefill_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, float* __restrict__ O,
    float* __restrict__ LSE, const Segment* __restrict__ segs, const WorkItem* __restrict__ work,
    const int32_t* __restrict__ tile_src, int n_work, int blocks, int n_tokens, int n_kv_heads, int group, float scale, long long q_head,
    long long q_tok, long long kv_head, long long kv_tok) {
    constexpr int BAND = kF32Band, KS = 4, KB = LONG_FIRST ? 1 : 2, TILE = 16 * KB;
    __shared__ __attribute__((aligned(16))) float lds[MergeF32<D, KS>::FLOATS];
    const int lane = threadIdx.x & 63, i = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned band = blockIdx.x, block = blockIdx.y, g = blockIdx.z;
    if constexpr (LONG_FIRST) {
        const unsigned id = folded_id(), at = id / n_kv_heads;
        g = id % n_kv_heads;
        band = at % n_work;
        block = blocks - 1 - at / n_work;
        if (at / n_work >= (unsigned)blocks) return;
    }
    const WorkItem wi = work[band];
    const Segment sg = segs[wi.seg];
    const int t0 = wi.m_tile * BAND;
    const int rows_band = min(BAND, sg.q_len - t0) * group;
    const int rho0 = block * kF32Rows;
    if (rho0 >= rows_band) return;
    const int rho = min(rho0 + i, rows_band - 1);
    const int t = t0 + rho / group;
    auto q_row = [&](int row) __attribute__((always_inline)) {
        const int r = min(rho0 + row, rows_band - 1);
        return Q + (size_t)(g * group + r % group) * q_head + (size_t)(sg.q_start + t0 + r / group) * q_tok;
    };

    const RowsSegment rows{K + (size_t)g * kv_head, V + (size_t)g * kv_head, tile_src, sg.ctx_len,
                           sg.q_start - sg.back, kv_tok};
    const int n_keys = sg.ctx_len + sg.back + t0 + (min(rho0 + kF32Rows, rows_band) - 1) / group + 1;
    const int per = ((n_keys + TILE - 1) / TILE + KS - 1) / KS * TILE;
    const int lo = wave * per, hi = min(lo + per, n_keys);
    float m = -INFINITY, l = 0.f;
    f32x4 o[D / 16];
#pragma unroll
    for (int x = 0; x < D / 16; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    attend_f32<D, KB>(rows, q_row, lo, hi, sg.ctx_len + sg.back + t, scale, m, l, o);

    auto store = [&](int row, int d, float4 val, float lse) __attribute__((always_inline)) {
        const int rr = rho0 + row;
        if (rr >= rows_band) return;
        const int tt = sg.q_start + t0 + rr / group, hh = g * group + rr % group;
        *(float4*)(O + (size_t)hh * q_head + (size_t)tt * q_tok + d) = val;
        if (LSE && d == 0) LSE[(size_t)hh * n_tokens + tt] = lse;
    };
    MergeF32<D, KS>::run(lds, wave, threadIdx.x, 256, m, l, o, true, store);
}

// Decode over the mixed KV set, gathered (rows of Kmix / Vmix) or in place (MAPPED, rows of K / V /
// Ksp / Vsp through src_idx).  grid: key splits x row blocks x KV heads x queries, in one dimension (folded_grid);
// all W waves of the workgroup share the keys of its split.  One split: the workgroup writes the results, no scratch
// memory.  SPLIT: it writes the sum of O, the reference and the sum of every row, and decode_f32_merge_kernel the
// results.  Bound by the matrix instruction (a 32-key tile takes a SIMD 0.9 us at D = 64, 1.7 at D = 128), so a long
// mixed set on few row blocks wants many compute units: the line is at decode_f32_plan.
template <int D, bool SPLIT> struct DecodeF32 {
    static constexpr int W = SPLIT ? 4 : D == 64 ? 16 : 8;    // (registers: 96 / 192 for operands and output)
    static constexpr int THREADS = 64 * W, WAVES_PER_SIMD = SPLIT ? 2 : W / 4;
    static constexpr int LDS_BYTES = MergeF32<D, W>::FLOATS * 4;
};
template <int D, bool MAPPED, bool SPLIT>
__global__ __launch_bounds__((DecodeF32<D, SPLIT>::THREADS), (DecodeF32<D, SPLIT>::WAVES_PER_SIMD)) void decode_f32_kernel(
    const float* __restrict__ Qd, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ Ksp, const float* __restrict__ Vsp, const int32_t* __restrict__ src_idx,
    float* __restrict__ O, float* __restrict__ LSE, const int32_t* __restrict__ mix_len, int T_q, int n_q_heads,
    int n_kv_heads, int group, int batch, int l_cap, int s_total, long long kv_head, long long kv_tok, float scale,
    int n_split, float* __restrict__ part_o, float2* __restrict__ part_ml) {
    constexpr int W = DecodeF32<D, SPLIT>::W;
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_rows = T_q * group;
    const unsigned blocks = (n_rows + kF32Rows - 1) / kF32Rows, id = folded_id();
    const unsigned split = SPLIT ? id % n_split : 0, rest = SPLIT ? id / n_split : id, unit = rest / blocks;
    const int rho0 = rest % blocks * kF32Rows, g = unit % n_kv_heads, b = unit / n_kv_heads;
    if (b >= batch) return;
    auto q_row = [&](int row) __attribute__((always_inline)) {
        const int r = min(rho0 + row, n_rows - 1);
        return Qd + (((size_t)b * T_q + r / group) * n_q_heads + g * group + r % group) * D;
    };
    const int n_keys = min(max(mix_len[b], 0), l_cap);

    // (dealt out by the length, over the waves of all splits)
    constexpr int TILE = 16 * kDecodeKB;
    const int n_w = SPLIT ? n_split * W : W;
    const int per = ((n_keys + TILE - 1) / TILE + n_w - 1) / n_w * TILE;
    const int lo = min((int)(split * W + wave) * per, n_keys), hi = min(lo + per, n_keys);
    float m = -INFINITY, l = 0.f;
    f32x4 o[D / 16];
#pragma unroll
    for (int x = 0; x < D / 16; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (MAPPED) {
        const RowsMapped rows{K + (size_t)g * kv_head, V + (size_t)g * kv_head, Ksp + (size_t)g * s_total * D,
                              Vsp + (size_t)g * s_total * D, src_idx + (size_t)b * l_cap, D, kv_tok};
        attend_f32<D, kDecodeKB>(rows, q_row, lo, hi, n_keys, scale, m, l, o);
    } else {
        const size_t off = ((size_t)b * n_kv_heads + g) * (size_t)l_cap * D;
        attend_f32<D, kDecodeKB>(RowsPlain{K + off, V + off, D}, q_row, lo, hi, n_keys, scale, m, l, o);
    }
    if constexpr (SPLIT) {
        const size_t part = (((size_t)b * n_kv_heads + g) * n_split + split) * n_rows + rho0;
        MergeF32<D, W, true>::run(lds_f, wave, threadIdx.x, 64 * W, m, l, o, true, [&](int row, int d, float4 val, float2 ml)
                                  __attribute__((always_inline)) {
            if (rho0 + row >= n_rows) return;
            *(float4*)(part_o + (part + row) * D + d) = val;
            if (d == 0) part_ml[part + row] = ml;
        });
    } else {
        MergeF32<D, W>::run(lds_f, wave, threadIdx.x, 64 * W, m, l, o, n_keys > 0, [&](int row, int d, float4 val, float lse)
                            __attribute__((always_inline)) {
            const int rr = rho0 + row;
            if (rr >= n_rows) return;
            const size_t dst = ((size_t)b * T_q + rr / group) * n_q_heads + g * group + rr % group;
            *(float4*)(O + dst * D + d) = val;
            if (LSE && d == 0) LSE[dst] = lse;
        });
    }
}

// The merge of the splits, one workgroup per query row: SG groups of D / 4 lanes take every SG-th split, U of them
// requested together, and are folded through LDS; the order depends on the split index alone.  A split that a row
// has no key in holds reference -inf and sums of 0.
template <int D>
__global__ __launch_bounds__(256) void decode_f32_merge_kernel(const float* __restrict__ part_o,
                                                               const float2* __restrict__ part_ml, float* __restrict__ O,
                                                               float* __restrict__ LSE, const int32_t* __restrict__ mix_len,
                                                               int T_q, int n_q_heads, int n_kv_heads, int group, int n_split) {
    constexpr int NV = D / 4, SG = 256 / NV, U = 4;
    __shared__ __attribute__((aligned(16))) float red[SG][D];
    __shared__ float2 stat[SG];
    const int n_rows = T_q * group, sg = threadIdx.x / NV, d = threadIdx.x % NV * 4;
    const int rho = blockIdx.x % n_rows, g = blockIdx.x / n_rows % n_kv_heads, b = blockIdx.x / n_rows / n_kv_heads;
    const size_t base = ((size_t)b * n_kv_heads + g) * n_split * n_rows + rho;
    float M = -INFINITY, L = 0.f;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = sg; s0 < n_split; s0 += U * SG) {
        float2 ml[U];
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {                         // (behind the last split its own values again, not counted)
            const size_t at = base + (size_t)min(s0 + u * SG, n_split - 1) * n_rows;
            ml[u] = part_ml[at];
            v[u] = *(const float4*)(part_o + at * D + d);
        }
        float m_new = M;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u * SG < n_split) m_new = fmaxf(m_new, ml[u].x);
        const float ref = m_new == -INFINITY ? 0.f : m_new, f0 = expf(M - ref);
        M = m_new;
        L *= f0;
        a.x *= f0; a.y *= f0; a.z *= f0; a.w *= f0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u * SG < n_split) {
                const float f = expf(ml[u].x - ref);
                L = fmaf(f, ml[u].y, L);
                a.x = fmaf(f, v[u].x, a.x); a.y = fmaf(f, v[u].y, a.y);
                a.z = fmaf(f, v[u].z, a.z); a.w = fmaf(f, v[u].w, a.w);
            }
    }
    *(float4*)(&red[sg][d]) = a;
    if (d == 0) stat[sg] = make_float2(M, L);
    __syncthreads();
    if (threadIdx.x >= D) return;
    M = stat[0].x;
#pragma unroll
    for (int i = 1; i < SG; ++i) M = fmaxf(M, stat[i].x);
    const float ref = M == -INFINITY ? 0.f : M;
    float sum = 0.f;
    L = 0.f;
#pragma unroll
    for (int i = 0; i < SG; ++i) {
        const float f = expf(stat[i].x - ref);
        L = fmaf(f, stat[i].y, L);
        sum = fmaf(f, red[i][threadIdx.x], sum);
    }
    const bool some = mix_len[b] > 0;
    const size_t row = ((size_t)b * T_q + rho / group) * n_q_heads + g * group + rho % group;
    O[row * D + threadIdx.x] = some ? sum * (1.f / L) : 0.f;
    if (LSE && threadIdx.x == 0) LSE[row] = some ? lse_f32(M, L) : -INFINITY;
}

}  // namespace

vxl_status launch_prefill_f32(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Q, const void* K,
                              const void* V, void* O, float* LSE, hipStream_t s) {
    const int group = d->n_q_heads / d->n_kv_heads;
    const TokStrides ts = tok_strides(d, L->n_tokens);
    int n_cus = 0;
    const vxl_status st = device_cu_count(&n_cus);
    if (st != VXL_OK) return st;
    const int blocks = (std::min(L->longest, kF32Band) * group + kF32Rows - 1) / kF32Rows;       // of the longest band
    const bool long_first = (long long)L->n_tokens * d->n_q_heads > (long long)kF32Rows * n_cus;
    const dim3 grid = long_first ? folded_grid((long long)L->n_work[0] * blocks * d->n_kv_heads)
                                 : dim3(L->n_work[0], blocks, d->n_kv_heads);
#define VXL_LAUNCH(D, LONG_FIRST)                                                                               \
    hipLaunchKernelGGL((prefill_f32_kernel<D, LONG_FIRST>), grid, dim3(256), 0, s, (const float*)Q, (const float*)K, (const float*)V,  \
                       (float*)O, LSE, L->d_segs, L->d_work[0], L->d_tile_src, L->n_work[0], blocks, L->n_tokens,          \
                       d->n_kv_heads, group, scale, ts.qh, ts.qt, ts.kh, ts.kt)
    if (d->head_dim == 64) { if (long_first) VXL_LAUNCH(64, true); else VXL_LAUNCH(64, false); }
    else { if (long_first) VXL_LAUNCH(128, true); else VXL_LAUNCH(128, false); }
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

// Splits of the keys: as many workgroups of four waves as there are tiles for, 512 over all row blocks (two per compute
// unit; against 256: eight queries of 64 rows x 4 heads over 2,064 keys, D = 64, 45.8 -> 39.2 us, others equal).  Short
// sets stay with one workgroup per row block and no second launch; us with the gather, one workgroup -> splits,
// D = 64: 16 rows, 512 keys 15.5 -> 16.2, 768 keys 18.6 -> 16.4; 16 rows x 4 heads, 2,064 keys 39.4 -> 16.3.  D = 128:
// 256 keys 15.7 -> 16.3, 352 keys 20.1 -> 16.2, 16 rows x 4 heads, 2,064 keys 65.7 -> 18.4, 11,300 keys 297 -> 35.6.
// By the capacity, which is what the host knows: 40 keys in buffers for 5,000 pay for the second launch (6.1 -> 9.4, D =
// 128 6.6 -> 10.6, call by call) unless the caller gives no workspace.
DecodePlan decode_f32_plan(const vxl_attn_desc* d, int batch, int T, int l_cap) {
    DecodePlan p{};
    const long long rows = (long long)(d->n_q_heads / d->n_kv_heads) * T, units = (long long)batch * d->n_kv_heads;
    const long long blocks = (rows + kF32Rows - 1) / kF32Rows * units, tiles = ((long long)l_cap + 16 * kDecodeKB - 1) / (16 * kDecodeKB);
    const long long n_split = tiles <= (d->head_dim == 64 ? 18 : 8) ? 1 : std::min<long long>((tiles + 3) / 4, 512 / blocks);
    p.n_split = (int)std::max<long long>(1, n_split);
    p.split_len = l_cap;
    if (p.n_split > 1) {
        p.part_ml = align_up((size_t)(units * p.n_split * rows) * d->head_dim * sizeof(float), 256);
        p.total = p.part_ml + align_up((size_t)(units * p.n_split * rows) * sizeof(float2), 256);
    }
    return p;
}

// ws: scratch of decode_f32_plan(...).total bytes, or null (one split).
template <int D>
static vxl_status run_decode_f32(const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T, const void* K,
                                 const void* V, const void* Ksp, const void* Vsp, const int32_t* src_idx, int l_cap,
                                 int s_total, const TokStrides& ts, const int32_t* mix_len, void* O, float* LSE, void* ws,
                                 hipStream_t s) {
    const int group = d->n_q_heads / d->n_kv_heads;
    static PerDeviceOnce attr;
    const vxl_status st = attr.run([] {
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_f32_kernel<D, false, false>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, DecodeF32<D, false>::LDS_BYTES));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_f32_kernel<D, true, false>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, DecodeF32<D, false>::LDS_BYTES));
        return VXL_OK;
    });
    if (st != VXL_OK) return st;
    const DecodePlan p = decode_f32_plan(d, batch, T, l_cap);
    const int n_split = ws ? p.n_split : 1;
    float* part_o = (float*)ws;
    float2* part_ml = (float2*)((char*)ws + (ws ? p.part_ml : 0));
    const dim3 grid = folded_grid((long long)((group * T + kF32Rows - 1) / kF32Rows) * d->n_kv_heads * batch * n_split);
#define VXL_LAUNCH(MAPPED, SPLIT)                                                                                   \
    hipLaunchKernelGGL((decode_f32_kernel<D, MAPPED, SPLIT>), grid, dim3(DecodeF32<D, SPLIT>::THREADS),             \
                       (DecodeF32<D, SPLIT>::LDS_BYTES), s,                                                         \
                       (const float*)Qd, (const float*)K, (const float*)V, (const float*)Ksp, (const float*)Vsp,    \
                       src_idx, (float*)O, LSE, mix_len, T, d->n_q_heads, d->n_kv_heads, group, batch, l_cap, s_total, \
                       ts.kh, ts.kt, scale, n_split, part_o, part_ml)
    if (n_split > 1) { if (src_idx) VXL_LAUNCH(true, true); else VXL_LAUNCH(false, true); }
    else { if (src_idx) VXL_LAUNCH(true, false); else VXL_LAUNCH(false, false); }
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    if (n_split == 1) return VXL_OK;
    hipLaunchKernelGGL(decode_f32_merge_kernel<D>, dim3(d->n_kv_heads * group * T * batch), dim3(256), 0, s, part_o, part_ml,
                       (float*)O, LSE, mix_len, T, d->n_q_heads, d->n_kv_heads, group, n_split);
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

vxl_status launch_decode_f32(const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T, const void* Kmix,
                             const void* Vmix, int l_cap, const int32_t* mix_len, void* O, float* LSE, void* ws,
                             hipStream_t s) {
    const TokStrides none{};
    return d->head_dim == 64 ? run_decode_f32<64>(d, scale, Qd, batch, T, Kmix, Vmix, nullptr, nullptr, nullptr, l_cap,
                                                  0, none, mix_len, O, LSE, ws, s)
                             : run_decode_f32<128>(d, scale, Qd, batch, T, Kmix, Vmix, nullptr, nullptr, nullptr, l_cap,
                                                   0, none, mix_len, O, LSE, ws, s);
}

vxl_status launch_decode_f32_inplace(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Qd, int batch,
                                     int T, const void* K, const void* V, const void* Ksp, const void* Vsp,
                                     const int32_t* src_idx, int l_cap, const int32_t* mix_len, void* O, float* LSE,
                                     void* ws, hipStream_t s) {
    const TokStrides ts = tok_strides(d, L->n_tokens);
    return d->head_dim == 64 ? run_decode_f32<64>(d, scale, Qd, batch, T, K, V, Ksp, Vsp, src_idx, l_cap, L->s_total, ts,
                                                  mix_len, O, LSE, ws, s)
                             : run_decode_f32<128>(d, scale, Qd, batch, T, K, V, Ksp, Vsp, src_idx, l_cap, L->s_total,
                                                   ts, mix_len, O, LSE, ws, s);
}

}  // namespace vxl
