// Chunk-based pre-filling attention on the gfx950 matrix cores (bf16 inputs, fp32 accumulate).
//
// Pre-pass (once per call; small prompts do without): the K and V rows every later chunk may see -- the
// prefix rows followed by the kept rows of all chunks in chunk order -- are compacted into two contiguous
// buffers, so the history of chunk c is simply their first P + sparse_offsets[c] rows.
//
// Main kernel (prefill_dma_kernel): a persistent workgroup takes bands of query rows of one
// segment (the prefix or a chunk) and walks 64-key tiles  history[0, ctx_len)  then  own
// segment[0, diagonal]  with an online softmax; the arithmetic is in vxl_mfma.h.  256 rows and 8
// waves per workgroup (128 rows and 4 waves for small prompts), tiles streamed into an LDS ring by
// direct global-to-LDS loads.  A third instance of the same template (128 rows, 4 waves, a 2-stage
// ring, two workgroups per compute unit) is kept as an on-device cross-check.
#include <math.h>

#include <algorithm>
#include <atomic>

#include "vxl_internal.h"
#include "vxl_mfma.h"

namespace vxl {

namespace {

__device__ __forceinline__ uint4 zero4() { return make_uint4(0u, 0u, 0u, 0u); }

// ------------------------------------------------------------------------------------------
// Pre-pass: Kctx[g, r, :] = K[g, tile_src[r], :], same for V (zero rows where tile_src is -1).
// Its first workgroup also sets the work-queue counters of the persistent main kernel to `queue_start` (when
// `queue` is given), which saves that kernel's callers a launch of their own.
// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void compact_kv_kernel(const uint4* __restrict__ K, const uint4* __restrict__ V,
                                                         const int32_t* __restrict__ tile_src,
                                                         uint4* __restrict__ Kctx, uint4* __restrict__ Vctx,
                                                         int n_rows_pad, long long kv_head_u4, long long kv_tok_u4,
                                                         int* __restrict__ queue, int queue_start) {
    constexpr int LPR = D * 2 / 16, ROWS = 256 / LPR;
    if (queue && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 8) queue[threadIdx.x] = queue_start;
    const int r = blockIdx.x * ROWS + threadIdx.x / LPR, part = threadIdx.x % LPR, g = blockIdx.y;
    if (r >= n_rows_pad) return;
    const int src = tile_src[r];
    const size_t so = (size_t)g * kv_head_u4 + (size_t)max(src, 0) * kv_tok_u4 + part;   // (strides in 16-byte units)
    const size_t dk = ((size_t)g * n_rows_pad + r) * LPR + part;
    Kctx[dk] = src >= 0 ? K[so] : zero4();
    Vctx[dk] = src >= 0 ? V[so] : zero4();
}

// ------------------------------------------------------------------------------------------
// Main kernel: 8 waves = 256 query rows per workgroup (one workgroup per compute unit, two waves per
// SIMD), for small prompts 4 waves = 128 rows (the line is at launch_prefill_bf16).  K/V tiles are
// brought in by direct global->LDS loads into a ring of NS stages, two tiles ahead of the arithmetic:
// the staging stays out of the VALU/VGPR budget and the memory latency hides behind several tiles of
// arithmetic.
//
// The loads are issued from inline assembly: the compiler cannot see them, so it neither orders
// them against the LDS reads of other stages nor counts them in its own vmcnt bookkeeping; the
// kernel does both by hand (every wave issues the same number of loads per tile, and waits with
// vmcnt = loads still allowed in flight).  No compiler-visible vector memory operation may be
// outstanding while the ring runs: the query registers are forced complete before the first ring
// load, and the kernel must not spill (the build refuses a compile of it that uses scratch).
// ------------------------------------------------------------------------------------------
template <int D, int NS, int NW = 8>
struct PrefillDmaCfg {
    static constexpr int WAVES = NW;                          // 8 or 4: two or one per SIMD
    static constexpr int BM = 32 * WAVES;
    static constexpr int TILE = kKeyTile * D;                 // elements of one unpadded K (or V) tile
    static constexpr int STAGE = 2 * TILE;                    // K tile then V tile
    static constexpr int LDS_BYTES = NS * STAGE * 2 + 16;     // the ring and the slot of the work index
    static constexpr int PPR = D / 8;                         // 16-byte pieces per row
    static constexpr int RPI = 64 / PPR;                      // rows per load instruction (1 KiB)
    static constexpr int NI = kKeyTile / RPI;                 // instructions per tile per matrix
    static constexpr int IPW = NI / WAVES;                    // ... per wave
    static constexpr int GROUP = 2 * IPW;                     // loads per wave per tile (K and V)
};

// The kernel is persistent (except kDirect): the grid is as many workgroups as the chip holds at once (one per compute
// unit; two of 4 waves where their rings fit its LDS), and every workgroup keeps taking the next (band
// of query rows, part of its row-block x head grid) pair of its queue from a counter in global memory
// until the queue is empty.  The work list is sorted heaviest first, so this is greedy longest-first
// scheduling without gaps between workgroups.  With xpg > 0 there is one queue per KV head group,
// served by the xpg XCDs (blockIdx.x % 8, the order workgroups are dealt out in) whose L2 then
// holds that group's K and V; otherwise a single queue.  The counters must be zero at launch (kLate: the
// number of the queue's workgroups, whose first parts are their own numbers).
// How a workgroup comes by its parts (the lines are at launch_prefill_bf16):
//   kEarly   from the queue, the next part claimed as a part begins, which costs nothing: large prompts
//   kLate    from the queue, the next part claimed shortly before a part ends: with a few parts per workgroup it
//            goes to the one that is done first and not to the one that began first
//   kDirect  one part by its number in the launch; no queue and no pre-pass: history rows are read where they are,
//            prefix rows by their number and kept rows through the layout's table of source tokens, whose share of
//            a part lies in LDS behind the ring
enum { kEarly, kLate, kDirect };
// kDirect: the parts of an item and KV head that a launch has places for (direct_places), what the prefix's bands have more,
// and the KV heads that share a numbering (1, or all where they do not divide the XCDs).
struct PartPlaces { int places, extra, heads; };
template <int D, int NS, bool STRIDED, int NW = 8, int TAKE = kEarly>
__global__ __launch_bounds__(NW * 64, 2) void prefill_dma_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const uint16_t* __restrict__ Kctx, const uint16_t* __restrict__ Vctx, uint16_t* __restrict__ O,
    float* __restrict__ LSE, const Segment* __restrict__ segs, const WorkItem* __restrict__ work,
    int n_tokens, int n_q_heads, int group, int ctx_rows_pad, float scale, int n_items, int xpg,
    int* __restrict__ queue, long long q_head_arg, int q_tok_arg, long long kv_head_arg, int kv_tok_arg,
    const int32_t* __restrict__ hist_src, int n_prefix, PartPlaces pp) {      // (DIRECT; hist_src: source token of every history row)
    using C = PrefillDmaCfg<D, NS, NW>;
    constexpr bool DIRECT = TAKE == kDirect, LATE = TAKE == kLate;
    // Element strides of Q/O and K/V rows: the arguments, or (STRIDED false, the dense head-major
    // layout) constants, so that the dense instance carries no stride arithmetic or registers.
    const long long q_head = STRIDED ? q_head_arg : (long long)n_tokens * D;
    const long long kv_head = STRIDED ? kv_head_arg : (long long)n_tokens * D;
    const int q_tok = STRIDED ? q_tok_arg : D;
    const int kv_tok = STRIDED ? kv_tok_arg : D;
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    int* next_slot = (int*)(lds + NS * C::STAGE);
    int* kept = next_slot + 4;                                // DIRECT: source tokens of the history rows behind the prefix

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qid = xpg > 0 ? (int)(blockIdx.x & 7) / xpg : 0;            // this workgroup's queue
    const int listed = DIRECT ? n_items * pp.heads * pp.places : xpg > 0 ? n_items * group : n_items * n_q_heads;
    const int q_len_items = DIRECT ? listed + (n_prefix + C::BM - 1) / C::BM * pp.heads * pp.extra : listed;
    const float c2 = scale * kLog2e;
    const int r_in = lane / C::PPR, piece = lane % C::PPR;

    // Lane-constant parts of the refill addresses of a full tile: row and (swizzled) 16-byte piece
    // of this lane in each of the wave's load instructions -- for the compact history tiles
    // (rows D elements apart) and for the own tiles, read in place (rows kv_tok elements apart).
    uint32_t koff_ctx[C::IPW], voff_ctx[C::IPW], koff_own[C::IPW], voff_own[C::IPW];
#pragma unroll
    for (int i = 0; i < C::IPW; ++i) {
        const int row = (wave + i * C::WAVES) * C::RPI + r_in;
        const int kp = piece ^ ((row / (16 / C::PPR)) & (C::PPR - 1));
        constexpr int CPR = D * 2 / 64, RPL = D == 128 ? 1 : 2;
        const int vp = (((piece >> 2) ^ ((row / RPL) & (CPR - 1))) << 2) | (piece & 3);
        koff_ctx[i] = (uint32_t)row * (D * 2) + kp * 16;
        voff_ctx[i] = (uint32_t)row * (D * 2) + vp * 16;
        koff_own[i] = STRIDED ? (uint32_t)row * (uint32_t)(kv_tok * 2) + kp * 16 : koff_ctx[i];
        voff_own[i] = STRIDED ? (uint32_t)row * (uint32_t)(kv_tok * 2) + vp * 16 : voff_ctx[i];
    }

    int j;
    if constexpr (TAKE == kEarly) {
        if (tid == 0) next_slot[0] = atomicAdd(queue + qid, 1);
        __syncthreads();
        j = __builtin_amdgcn_readfirstlane(next_slot[0]);
    } else {
        j = xpg > 0 ? (int)(blockIdx.x >> 3) * xpg + (int)(blockIdx.x & 7) % xpg : (int)blockIdx.x;
    }
    // The descriptors of an item (two dependent scalar loads) are fetched while the item before it
    // runs, as soon as its index is known.
    auto item_of = [&](int jj) { return jj / (DIRECT ? pp.heads * pp.places : xpg > 0 ? group : n_q_heads); };
    WorkItem wi_next = {0, 0};
    Segment sg_next = {0, 0, 0, 0, 0};
    if (j < q_len_items) {
        if (DIRECT && j >= listed) wi_next = {0, (j - listed) / (pp.heads * pp.extra)};
        else wi_next = work[item_of(j)];
        sg_next = segs[wi_next.seg];
    }
  for (int par = 1; j < q_len_items; par ^= 1) {
    // A list entry is a band of C::BM query rows of a segment; with the `group` query heads that
    // share a KV head it makes a grid of (up to 8 row blocks of 32) x group cells, which is cut
    // row block major into `group` parts of 8 cells, one per wave.  A part spans few row blocks
    // (all heads of one or two of them), so all its waves stop at about the same own tile, and
    // the cells of a ragged last band fill as few parts as possible: cut head by head, every
    // part of such a band would run with most of its waves idle (variable chunk lengths: +11 %).
    // Parts left without cells walk one tile and write nothing.
    int g, part;                                              // KV head, part
    if constexpr (DIRECT) {
        const int item = item_of(j), places = j < listed ? pp.places : pp.extra;
        const int at = j < listed ? j - item * pp.heads * places : (j - listed) % (pp.heads * places);
        g = xpg > 0 ? qid : at / places;
        part = xpg > 0 ? at : at - g * places;
        // (in turn over the XCDs: a part's place decides its length)
        part = j < listed ? (part + item) % places : part + pp.places;
    } else {
        const int part_id = xpg > 0 ? qid * group + j % group : j % n_q_heads;
        g = part_id / group;
        part = part_id - g * group;
    }
    const WorkItem wi = wi_next;
    const Segment sg = sg_next;
    const int m0 = wi.m_tile * C::BM;
    const int band_blocks = min(C::WAVES, (sg.q_len - m0 + 31) / 32);
    const int cell = part * C::WAVES + wave;
    const int rb = cell / group;                              // this wave's row block and head
    const int h = g * group + (cell - rb * group);
    const bool idle = rb >= band_blocks;                      // (the grid of a ragged last band is smaller)
    const int wrow0 = m0 + rb * 32;
    if (DIRECT && part * C::WAVES >= band_blocks * group) return;
    const int n_ctx_t = (sg.ctx_len + kKeyTile - 1) / kKeyTile;
    const int rb_last = min(band_blocks - 1, (part * C::WAVES + C::WAVES - 1) / group);
    const int last_row = min(m0 + (rb_last + 1) * 32, sg.q_len) - 1;
    // own keys start `back` rows early; a part without cells still walks one tile (every wave idle)
    const int n_t = part * C::WAVES < band_blocks * group ? n_ctx_t + (last_row + sg.back) / kKeyTile + 1 : 1;

    const char* kctx_g = (const char*)(Kctx + (size_t)g * ctx_rows_pad * D);
    const char* vctx_g = (const char*)(Vctx + (size_t)g * ctx_rows_pad * D);
    const char* kall = (const char*)(K + (size_t)g * kv_head);        // (DIRECT) token 0
    const char* vall = (const char*)(V + (size_t)g * kv_head);
    const char* kown = (const char*)(K + (size_t)g * kv_head + (size_t)(sg.q_start - sg.back) * kv_tok);
    const char* vown = (const char*)(V + (size_t)g * kv_head + (size_t)(sg.q_start - sg.back) * kv_tok);

    // Tile t -> stage t % NS.  Every wave issues GROUP loads: instruction slots wave, wave + 8, ...
    auto issue = [&](int t) {
        const bool ctx = t < n_ctx_t;
        const int row0 = ctx ? t * kKeyTile : (t - n_ctx_t) * kKeyTile;
        const int rlim = ctx ? kKeyTile - 1 : min(kKeyTile - 1, sg.back + sg.q_len - 1 - row0);
        const uint32_t row_bytes = ctx && !DIRECT ? D * 2 : (uint32_t)kv_tok * 2;
        const char* kb = (ctx ? DIRECT ? kall : kctx_g : kown) + (size_t)row0 * row_bytes;
        const char* vb = (ctx ? DIRECT ? vall : vctx_g : vown) + (size_t)row0 * row_bytes;
        const uint32_t st = lds_base + (uint32_t)(t % NS) * (C::STAGE * 2);
        if (DIRECT && ctx && row0 + kKeyTile > n_prefix) {    // rows past the history's last repeat it (their scores are masked)
#pragma unroll
            for (int i = 0; i < C::IPW; ++i) {
                const int slot = wave + i * C::WAVES, row = slot * C::RPI + r_in;
                const int r = min(row0 + row, sg.ctx_len - 1);
                const int src = r < n_prefix ? r : kept[r - n_prefix];
                const uint32_t moved = (uint32_t)(src - row) * row_bytes;
                dma16(kall, koff_own[i] + moved, st + slot * 1024);
                dma16(vall, voff_own[i] + moved, st + C::TILE * 2 + slot * 1024);
            }
            return;
        }
        if (STRIDED && ctx && !DIRECT) {
#pragma unroll
            for (int i = 0; i < C::IPW; ++i) {
                const int slot = wave + i * C::WAVES;
                dma16(kb, koff_ctx[i], st + slot * 1024);
                dma16(vb, voff_ctx[i], st + C::TILE * 2 + slot * 1024);
            }
        } else if (rlim == kKeyTile - 1) {
#pragma unroll
            for (int i = 0; i < C::IPW; ++i) {
                const int slot = wave + i * C::WAVES;
                dma16(kb, koff_own[i], st + slot * 1024);
                dma16(vb, voff_own[i], st + C::TILE * 2 + slot * 1024);
            }
        } else {                                              // rows past the segment's last key repeat it
#pragma unroll
            for (int i = 0; i < C::IPW; ++i) {
                const int slot = wave + i * C::WAVES;
                const int row = slot * C::RPI + r_in;
                const uint32_t back_rows = (uint32_t)(row - min(row, rlim)) * row_bytes;
                dma16(kb, koff_own[i] - back_rows, st + slot * 1024);
                dma16(vb, voff_own[i] - back_rows, st + C::TILE * 2 + slot * 1024);
            }
        }
    };

    f32x16 o[1][D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[0][db] = zero16();
    float m_run = -INFINITY, l_run = 0.f;

    // The ring is used as two groups of TPB stages: while the tiles of one group are consumed the
    // other group is refilled, and the workgroup meets at ONE barrier per TPB tiles (fewer
    // meetings let the waves drift apart, which is what overlaps one wave's vector work with
    // another's matrix work).  Tile indices beyond the last are clamped to it, so that every wave
    // always issues the same number of loads; a clamped issue rewrites the last tile's own stage
    // with the same bytes, which is harmless.
    constexpr int TPB = NS / 2;                               // tiles per workgroup barrier: 2, or 1 with a 2-stage ring
    static_assert(NS == 2 * TPB && (TPB == 1 || TPB == 2), "two groups of TPB stages");
    // (DIRECT: a tile that needs the table is requested behind it)
    auto needs_table = [&](int t) { return DIRECT && t < n_ctx_t && (t + 1) * kKeyTile > n_prefix; };
#pragma unroll
    for (int t = 0; t < TPB; ++t)
        if (!needs_table(min(t, n_t - 1))) issue(min(t, n_t - 1));

    // The query rows are loaded after the ring has been started (both latencies then overlap) and
    // forced complete here: the compiler's wait for them covers the older ring loads as well, and
    // from here on no load it knows of is outstanding.
    bf16x8 qreg[1][D / 16];
    {
        // uniform base + 32-bit lane offset: the address stays out of the vector registers
        const char* qbase = (const char*)(Q + (size_t)h * q_head + (size_t)sg.q_start * q_tok);
        const uint32_t qoff = (uint32_t)min(wrow0 + l32, sg.q_len - 1) * (uint32_t)(q_tok * 2) + hi * 16;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            qreg[0][ks] = __builtin_bit_cast(bf16x8, *(const uint4*)(qbase + qoff + ks * 32));
        if constexpr (DIRECT)
            for (int i = tid; i < sg.ctx_len - n_prefix; i += C::WAVES * 64) kept[i] = hist_src[n_prefix + i];
        // the index of the item after this one is fetched in the same wait and read when this item is done
        if (TAKE == kEarly && tid == 0) next_slot[par] = atomicAdd(queue + qid, 1);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
            asm volatile("" :: "v"(__builtin_bit_cast(u32x4, qreg[0][ks])));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DIRECT) {
        if (sg.ctx_len > n_prefix) __syncthreads();           // (the table; without kept rows nothing of it is read)
#pragma unroll
        for (int t = 0; t < TPB; ++t)
            if (needs_table(min(t, n_t - 1))) issue(min(t, n_t - 1));
    }

    auto process = [&](int ti) {
        const bool is_ctx = ti < n_ctx_t;
        const int key0 = is_ctx ? ti * kKeyTile : (ti - n_ctx_t) * kKeyTile;
        const bool skip = idle || (!is_ctx && key0 > wrow0 + sg.back + 31);   // the tile lies above this wave's rows
        if (!skip) {
            const uint16_t* kt = lds + (ti % NS) * C::STAGE;
            const uint16_t* vt = kt + C::TILE;
            f32x16 s[1][2];
            qk_tile_ahead<D, 1>(kt, qreg, l32, hi, s);
            const bool need_mask = is_ctx ? (key0 + kKeyTile > sg.ctx_len) : (key0 + kKeyTile - 1 > wrow0 + sg.back);
            if (need_mask) {
                const int lim = is_ctx ? sg.ctx_len - key0 - 1 : wrow0 + sg.back + l32 - key0;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        s[0][kb][r] = acc_key(kb, r, hi) <= lim ? s[0][kb][r] : -INFINITY;
            }
            bf16x8 pb[1][2][2];
            softmax_tile<D / 32>(s[0], c2, m_run, l_run, o[0], pb[0]);
            pv_tile_ahead<D, 2>(vt, pb, lane, o);
        }
    };
    const int claim_t = max((n_t - 1) / TPB - 1, 0) * TPB;    // kLate: the meeting before the last one
    for (int t0 = 0; t0 < n_t; t0 += TPB) {
        // this wave's parts of tiles t0, t0+1 have landed -- and, at the item's first meeting, the
        // next item's index (an LDS store of wave 0, read by everybody right behind the barrier)
        wait_vmcnt0_lgkmcnt0();
        __builtin_amdgcn_s_barrier();                         // ... and everyone's; the other group is free
        int claimed = 0;
        if (LATE && t0 == claim_t && tid == 0) claimed = atomicAdd(queue + qid, 1);
        if (!DIRECT && t0 == (LATE ? claim_t + TPB : 0)) {    // the next item's index was written before this barrier
            const int jn = __builtin_amdgcn_readfirstlane(next_slot[par]);
            if (jn < q_len_items) {
                wi_next = work[item_of(jn)];
                sg_next = segs[wi_next.seg];
            }
        }
        if (t0 + TPB < n_t) issue(t0 + TPB);                  // (all waits are vmcnt(0): nothing is issued past the last tile,
        process(t0);                                          //  so the item does not end waiting for loads nobody reads)
        if (LATE && t0 == claim_t && tid == 0) next_slot[par] = claimed;
        if constexpr (TPB == 2) {
            if (t0 + TPB + 1 < n_t) issue(t0 + TPB + 1);      // the second refill between the two tiles
            if (t0 + 1 < n_t) process(t0 + 1);
        }
    }
    wait_vmcnt<0>();                                          // nothing of the ring is in flight when the item ends

    {
        const int q_off = wrow0 + l32;
        const float l_tot = l_run + __shfl_xor(l_run, 32);
        if (!idle) {
            const float inv = 1.f / l_tot;
            // uniform bases + 32-bit lane offsets, as for the query loads
            char* obase = (char*)(O + (size_t)h * q_head + (size_t)sg.q_start * q_tok);
            const uint32_t ooff = (uint32_t)q_off * (uint32_t)(q_tok * 2) + hi * 16;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int rq = 0; rq < 4; rq += 2) {
                    // A lane and its partner lane ^ 32 hold halves of the same 16-byte pieces of their row: of two pieces
                    // they swap one half each, so that either stores a whole one.
                    typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
                    u32x2 half[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        bf16x4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[0][db][(rq + p) * 4 + e] * inv);
                        half[p] = __builtin_bit_cast(u32x2, v);
                    }
                    const auto x = __builtin_amdgcn_permlane32_swap(half[0][0], half[1][0], false, false);
                    const auto y = __builtin_amdgcn_permlane32_swap(half[0][1], half[1][1], false, false);
                    if (q_off < sg.q_len) *(uint4*)(obase + ooff + (db * 32 + rq * 8) * 2) = make_uint4(x[0], y[0], x[1], y[1]);
                }
            if (LSE && hi == 0 && q_off < sg.q_len) (LSE + (size_t)h * n_tokens + sg.q_start)[q_off] = m_run * scale + logf(l_tot);
        }
    }
    if constexpr (DIRECT) return;
    __syncthreads();                    // every wave is done with this item's tiles; next_slot[par] is written
    j = __builtin_amdgcn_readfirstlane(next_slot[par]);
    if (LATE && n_t <= TPB && j < q_len_items) {                   // (an item of one meeting)
        wi_next = work[item_of(j)];
        sg_next = segs[wi_next.seg];
    }
  }
}

// Sets the queue counters of the persistent kernel (a kernel, not a memset: the call may be
// captured into a graph).
__global__ void reset_queue_kernel(int* queue, int queue_start) {
    if (threadIdx.x < 8) queue[threadIdx.x] = queue_start;
}

template <typename F>
vxl_status enable_big_lds(F kernel, int bytes) {
    VXL_HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return VXL_OK;
}

}  // namespace

static std::atomic<int> g_prefill_variant{0};
static std::atomic<hipEvent_t> g_ev_start{nullptr}, g_ev_stop{nullptr};
// Cross-check only (declared in vxl_debug.h): 0 = choose (8 waves, 256-row bands, one workgroup per
// compute unit; for small prompts 4 waves, 128-row bands); 1 = the same kernel as two independent
// 4-wave workgroups per compute unit (128-row bands, a 2-stage ring each, one meeting per tile); 2 = the
// 8-wave instance with the pre-pass and early claims whatever the size; 3 = with late claims; 4 = 4 waves, 128-row bands,
// with the pre-pass and the 4-stage ring.
extern "C" void vxl_debug_prefill_variant(int v) { g_prefill_variant = v >= 1 && v <= 4 ? v : 0; }
// Measurement hook (declared in vxl_debug.h): when both events are set, every vxl_chunk_prefill
// records them on its stream immediately before and after the main attention kernel (the pre-pass
// is outside the bracket).
extern "C" void vxl_debug_prefill_events(void* start, void* stop) {
    g_ev_start = (hipEvent_t)start;
    g_ev_stop = (hipEvent_t)stop;
}

// 32-bit byte offsets inside a segment's rows (longest segment plus its look-back)
static bool segments_fit_32_bits(const vxl_layout* L, const TokStrides& ts) {
    long long max_rows = 0;
    for (const Segment& sg : L->segs) max_rows = std::max<long long>(max_rows, (long long)sg.q_len + sg.back);
    return max_rows * std::max(ts.qt, ts.kt) * 2 < (1ll << 32) && ts.qt < (1ll << 30) && ts.kt < (1ll << 30);
}

template <int D, int NS, int NW = 8, int TAKE = kEarly>
static vxl_status run_prefill_dma(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Q,
                                  const void* K, const void* V, void* O, float* LSE, void* ws, hipStream_t s,
                                  bool spread = false) {
    using C = PrefillDmaCfg<D, NS, NW>;
    const TokStrides ts = tok_strides(d, L->n_tokens);
    if (!segments_fit_32_bits(L, ts)) return VXL_ERR_UNSUPPORTED;
    const PrefillWorkspace w = prefill_workspace(L, d);
    uint16_t* kctx = (uint16_t*)((char*)ws + w.kctx);
    uint16_t* vctx = (uint16_t*)((char*)ws + w.vctx);
    int* queue = (int*)((char*)ws + w.queue);
    const int n_rows_pad = L->n_ctx_tiles * kKeyTile;
    int n_cus = 0;                                            // per_cu persistent workgroups on each
    vxl_status st = device_cu_count(&n_cus);
    if (st != VXL_OK) return st;
    const int group = d->n_q_heads / d->n_kv_heads;
    const int xpg = 8 % d->n_kv_heads == 0 ? 8 / d->n_kv_heads : 0;
    constexpr int wl_i = NW == 8 ? 1 : 0;                     // the work list cut in bands of 32 * NW rows
    // workgroups per compute unit (`spread`: one, so that two of them do not take parts where another has none)
    const int per_cu = spread ? 1 : std::min(8 / NW, 163840 / C::LDS_BYTES);
    const long long n_pairs = (long long)L->n_work[wl_i] * d->n_q_heads;
    // no more workgroups than pairs (rounded up to whole rounds over the 8 XCDs when queues are per XCD group)
    const unsigned n_blocks = (unsigned)std::min<long long>((long long)per_cu * (n_cus / 8 * 8),
                                                            xpg ? (n_pairs + 7) / 8 * 8 : n_pairs);
    const int queue_start = TAKE != kLate ? 0 : xpg ? (int)(n_blocks / 8) * xpg : (int)n_blocks;      // the workgroups' first pairs
    if (L->n_ctx_tiles > 0) {
        constexpr int rows = 256 / (D * 2 / 16);
        hipLaunchKernelGGL((compact_kv_kernel<D>), dim3((n_rows_pad + rows - 1) / rows, d->n_kv_heads),
                           dim3(256), 0, s, (const uint4*)K, (const uint4*)V, L->d_tile_src, (uint4*)kctx,
                           (uint4*)vctx, n_rows_pad, ts.kh / 8, ts.kt / 8, queue, queue_start);
    } else {
        hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(64), 0, s, queue, queue_start);
    }
    VXL_HIP_TRY(hipGetLastError());
    static PerDeviceOnce attr;
    st = attr.run([] {
        const vxl_status a = enable_big_lds(prefill_dma_kernel<D, NS, false, NW, TAKE>, C::LDS_BYTES);
        return a != VXL_OK ? a : enable_big_lds(prefill_dma_kernel<D, NS, true, NW, TAKE>, C::LDS_BYTES);
    });
    if (st != VXL_OK) return st;
    hipEvent_t ev_start = g_ev_start, ev_stop = g_ev_stop;
    const bool timed = ev_start && ev_stop;
    if (timed) VXL_HIP_TRY(hipEventRecord(ev_start, s));
#define VXL_LAUNCH(STRIDED_)                                                                             \
    hipLaunchKernelGGL((prefill_dma_kernel<D, NS, STRIDED_, NW, TAKE>), dim3(n_blocks), dim3(NW * 64),          \
                       C::LDS_BYTES, s, (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, kctx,  \
                       vctx, (uint16_t*)O, LSE, L->d_segs, L->d_work[wl_i], L->n_tokens, d->n_q_heads,     \
                       group, n_rows_pad, scale, L->n_work[wl_i], xpg, queue, ts.qh, (int)ts.qt, ts.kh,    \
                       (int)ts.kt, nullptr, 0, PartPlaces{})
    if (dense_layout(d)) VXL_LAUNCH(false); else VXL_LAUNCH(true);
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    if (timed) VXL_HIP_TRY(hipEventRecord(ev_stop, s));
    return VXL_OK;
}

// Parts of `waves` cells per item and KV head that a launch of kDirect has places for: those of the longest band of a
// chunk, and behind all of them the others (`extra`) of the prefix's bands.  A workgroup that finds no cells ends at once,
// but the next ones have gone to other compute units by then: with places for a whole band's parts, a few units got all the
// parts of short chunks (eight waves, 250 chunks of 40 tokens, D = 64, four heads on two 50.7 -> 27.5 us, D = 128, four on
// one 105.1 -> 41.3).
static PartPlaces direct_places(const vxl_layout* L, int group, int waves, int heads) {
    auto parts = [&](int tokens) { return (std::min((tokens + 31) / 32, waves) * group + waves - 1) / waves; };
    const int of_chunks = L->longest_chunk > 0 ? parts(L->longest_chunk) : parts(L->n_prefix);
    return {of_chunks, std::max(0, parts(L->n_prefix) - of_chunks), heads};
}

// The instances without a pre-pass: `spread` keeps two workgroups of D = 64 off one compute unit by their LDS.
template <int D, int NW>
static vxl_status run_prefill_direct(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Q, const void* K,
                                     const void* V, void* O, float* LSE, hipStream_t s, bool spread) {
    using C = PrefillDmaCfg<D, 4, NW>;
    constexpr int kMaxLds = 163840;
    const TokStrides ts = tok_strides(d, L->n_tokens);
    if (!segments_fit_32_bits(L, ts)) return VXL_ERR_UNSUPPORTED;
    static PerDeviceOnce attr;
    const vxl_status st = attr.run([] {
        const vxl_status a = enable_big_lds(prefill_dma_kernel<D, 4, false, NW, kDirect>, kMaxLds);
        return a != VXL_OK ? a : enable_big_lds(prefill_dma_kernel<D, 4, true, NW, kDirect>, kMaxLds);
    });
    if (st != VXL_OK) return st;
    hipEvent_t ev_start = g_ev_start, ev_stop = g_ev_stop;
    const bool timed = ev_start && ev_stop;
    if (timed) VXL_HIP_TRY(hipEventRecord(ev_start, s));
    const int group = d->n_q_heads / d->n_kv_heads;
    const int xpg = 8 % d->n_kv_heads == 0 ? 8 / d->n_kv_heads : 0;
    constexpr int wl_i = NW == 8 ? 1 : 0;
    const PartPlaces pp = direct_places(L, group, NW, xpg ? 1 : d->n_kv_heads);
    const long long per_queue = ((long long)L->n_work[wl_i] * pp.places + (L->n_prefix + C::BM - 1) / C::BM * pp.extra) * pp.heads;
    const unsigned n_blocks = (unsigned)(xpg ? (per_queue + xpg - 1) / xpg * 8 : per_queue);
    const int lds = std::max(spread ? kMaxLds / 2 + 16 : 0, C::LDS_BYTES + L->s_total * 4);
#define VXL_LAUNCH(STRIDED_)                                                                             \
    hipLaunchKernelGGL((prefill_dma_kernel<D, 4, STRIDED_, NW, kDirect>), dim3(n_blocks), dim3(NW * 64), lds, s, \
                       (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, nullptr, nullptr,     \
                       (uint16_t*)O, LSE, L->d_segs, L->d_work[wl_i], L->n_tokens, d->n_q_heads, group, 0, \
                       scale, L->n_work[wl_i], xpg, nullptr, ts.qh, (int)ts.qt, ts.kh, (int)ts.kt,       \
                       L->d_tile_src, L->n_prefix, pp)
    if (dense_layout(d)) VXL_LAUNCH(false); else VXL_LAUNCH(true);
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    if (timed) VXL_HIP_TRY(hipEventRecord(ev_stop, s));
    return VXL_OK;
}

vxl_status device_cu_count(int* n_cus) {
    static std::mutex mu;
    static int count[kMaxDevices] = {};
    int dev = 0;
    VXL_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return VXL_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (count[dev] == 0) {
        int n = 0;
        VXL_HIP_TRY(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        count[dev] = n < 8 ? 8 : n;
    }
    *n_cus = count[dev];
    return VXL_OK;
}

// Parts with cells of all bands of `blocks` (4 or 8) 32-row blocks (see the cut in prefill_dma_kernel), from the
// layout's counts: with a walk over the segments a call at 4,096 chunks took the host 21.3 us, so 9.2.
static long long part_count(const vxl_layout* L, const vxl_attn_desc* d, int blocks) {
    const int group = d->n_q_heads / d->n_kv_heads;
    long long n = L->row_blocks8 * (8 / blocks) * group;
    for (int r = 1; r < 8; ++r)
        n += L->segs_mod8[r] * ((long long)(r / blocks) * group + ((long long)(r % blocks) * group + blocks - 1) / blocks);
    return n * d->n_kv_heads;
}

vxl_status launch_prefill_bf16(const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Q,
                               const void* K, const void* V, void* O, float* LSE, void* ws, hipStream_t s) {
    if (g_prefill_variant == 1)
        return d->head_dim == 128 ? run_prefill_dma<128, 2, 4>(L, d, scale, Q, K, V, O, LSE, ws, s)
                                  : run_prefill_dma<64, 2, 4>(L, d, scale, Q, K, V, O, LSE, ws, s);
    bool late = g_prefill_variant == 3;
    if (g_prefill_variant == 0 || g_prefill_variant == 4) {
        int n_cus = 0;
        const vxl_status st = device_cu_count(&n_cus);
        if (st != VXL_OK) return st;
        const long long parts4 = part_count(L, d, 4), parts8 = part_count(L, d, 8);
        const bool d64 = d->head_dim == 64, own_unit = parts4 <= n_cus;
        const bool half = 8 * parts4 <= 9 * parts8;            // most bands have four cells at most: eight waves are half idle
        // No pre-pass and no queue (kDirect) while the compute units have some thirty tiles each; the table of kept rows
        // has to fit beside the ring, and a token's row a 32-bit offset.  Beyond that the table costs more than the
        // pre-pass, and the queue deals better.  us, pre-pass and early claims -> direct, D = 128 unless said: 56 parts 16.9
        // -> 14.2; D = 64, 168 parts of four waves 15.0 -> 10.6; 280 parts, 12 tiles per unit 59.1 -> 46.2; 428 parts, 25
        // tiles 95.1 -> 77.3; but 492 parts, 51 tiles 128.3 against 116.4 with late claims; 598 parts, 36 tiles 125.8 and
        // 106.9; 1,820 parts, 154 tiles 357 and 343.
        const long long tiles = L->pair_count * d->n_q_heads / (16384ll * n_cus);
        const bool direct = g_prefill_variant == 0 && tiles < 30 &&
                            (long long)L->n_tokens * tok_strides(d, L->n_tokens).kt * 2 < (1ll << 32);
        const auto fits = [&](int lds) { return 4ll * L->s_total <= lds - (d64 ? 65552 : 131088); };   // (the ring, 16 bytes)
        const int hist_tiles = L->l_ctx / kKeyTile;            // of the last chunk
        // Bands of 128 rows, so that twice as many compute units have work, and one wave per SIMD, which walks its tiles at
        // twice the speed of two.  While every part has a compute unit of its own (D = 128, eight waves -> four: 228 parts
        // 21.9 -> 17.4, 216 parts 15.9 -> 12.7), unless chunks of four cells make as many parts either way (240 parts of
        // D = 64 11.6 -> 11.9); D = 128 with the pre-pass from 48 tiles of history on (60 tiles 77.4 -> 75.5, 95 tiles 118.3
        // -> 113.3, but 32 tiles 45.0 -> 45.8).  At D = 64, where two such workgroups fit a compute unit, up to eight parts
        // for each (14 heads on two, 150 chunks of 72 tokens, 1,800 parts 74.0 -> 66.2, of 40 tokens 38.5 -> 32.7; 4 on 4,
        // 250 of 72, 1,004 parts 77.2 -> 59.1, with the queue 80.2), but few parts of four cells over a longer history are
        // as well off with eight waves (404 parts, 28 tiles of history 29.2 -> 31.9; 11 tiles 20.2 -> 15.9).
        if (direct && own_unit && !half && fits(163840) && (d64 || hist_tiles <= 48))
            return d64 ? run_prefill_direct<64, 4>(L, d, scale, Q, K, V, O, LSE, s, true)
                       : run_prefill_direct<128, 4>(L, d, scale, Q, K, V, O, LSE, s, false);
        if (direct && d64 && !own_unit && parts4 <= 8ll * n_cus && fits(81920) && !(half && 4 * parts4 <= 7ll * n_cus && hist_tiles > 12))
            return run_prefill_direct<64, 4>(L, d, scale, Q, K, V, O, LSE, s, false);
        // Eight waves up to two parts per compute unit, at D = 128 four, of prompts with one head per KV head, whose queue
        // has no parts without cells, if they have few tiles (800 parts, 16 tiles 138.2 against 136.0 with the queue).
        // Beyond, and where the table does not fit, they lose to the queue or to four waves with the pre-pass (4 heads on
        // 4, 250 chunks of 40 tokens, half of them kept, 142.9 against 139.4 and 123.0).
        const bool alone = own_unit && !half;
        if (direct && !alone && parts8 <= (d64 || (d->n_q_heads == d->n_kv_heads && tiles >= 12) ? 2ll : 4ll) * n_cus && fits(163840))
            return d64 ? run_prefill_direct<64, 8>(L, d, scale, Q, K, V, O, LSE, s, false)
                       : run_prefill_direct<128, 8>(L, d, scale, Q, K, V, O, LSE, s, false);
        // Four waves with the pre-pass: while every part has a compute unit of its own (D = 128: 328 parts 23.0 -> 26.7),
        // and at D = 64, where two share a unit, with some six tiles per segment where the eight-wave form just needs a
        // second round (302 parts 107.1 -> 98.9) or many (802 parts 242 -> 204; but 402 parts 139.2 -> 147.6).
        const bool shared = d64 && !own_unit && parts4 <= 4ll * n_cus && L->seg_tiles > 6ll * L->n_seg &&
                            (4 * parts8 <= 5ll * n_cus || parts8 > 2ll * n_cus);
        if (g_prefill_variant == 4 || (own_unit && parts4 > parts8) || shared)
            return d64 ? run_prefill_dma<64, 4, 4>(L, d, scale, Q, K, V, O, LSE, ws, s, own_unit)
                       : run_prefill_dma<128, 4, 4>(L, d, scale, Q, K, V, O, LSE, ws, s);
        // The next part is claimed late up to four parts per compute unit, early above (1,820 parts 342 against 343, 4,104
        // parts 1,379 against 1,422); with one head per KV head up to two and a half (D = 64, 1,004 parts 315 -> 345, 684
        // parts 182.6 -> 186.0, but 604 parts 148.6 -> 137.5; D = 128, 964 parts 124.8 -> 126.9).
        late = 2 * parts8 <= (d->n_q_heads > d->n_kv_heads ? 8ll : 5ll) * n_cus;
    }
    if (late)
        return d->head_dim == 128 ? run_prefill_dma<128, 4, 8, kLate>(L, d, scale, Q, K, V, O, LSE, ws, s)
                                  : run_prefill_dma<64, 4, 8, kLate>(L, d, scale, Q, K, V, O, LSE, ws, s);
    return d->head_dim == 128 ? run_prefill_dma<128, 4>(L, d, scale, Q, K, V, O, LSE, ws, s)
                              : run_prefill_dma<64, 4>(L, d, scale, Q, K, V, O, LSE, ws, s);
}

}  // namespace vxl
