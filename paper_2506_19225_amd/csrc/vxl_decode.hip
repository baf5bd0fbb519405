// GQA decode attention over the mixed KV set (bf16, matrix cores): split-KV partials and the
// fixed-order log-sum-exp merge.
//
// The G*T query rows that share one KV head (G = query heads per KV head) are stacked along the
// query dimension: row rho = t*G + hg.  A workgroup owns one (query b, KV head g, row tile,
// key split) and streams its slice of Kmix/Vmix exactly once through LDS.
// Each workgroup writes a normalised partial output and the base-2 log-sum-exp of its scaled
// logits; the merge kernel combines the splits of a row with weights and a summation order
// that depend only on the split index, so the result does not depend on scheduling.
#include <algorithm>

#include "vxl_internal.h"
#include "vxl_mfma.h"

namespace vxl {

namespace {

// Row map of the in-place form (IND instances of the kernels below): the mixed KV set is not a
// buffer but a list of rows -- mixed row r of query b is token src_idx[b, r] of the dense K / V
// (KV head g at kv_head elements, rows kv_tok elements apart) or, if negative, row -1 - src_idx of
// the sparse buffers Ksp / Vsp [Hkv, S_total, D].
struct RowMap {
    const int32_t* src_idx;     // [B, l_cap]
    const uint16_t* Ksp;        // may be null when no entry is negative
    const uint16_t* Vsp;
    long long kv_head;          // elements
    long long kv_tok;           // elements
    int s_total;
};

__device__ __forceinline__ uint16_t f32_to_bf16(float v) {
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    b += 0x7fffu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// Four results of a row that has one split, whose merge is the value itself (`some`: the row's LSE is a number;
// like the merge, a row without keys or with an LSE that is none gives 0).
__device__ __forceinline__ void store_row4(uint16_t* p, float a, float b, float c, float d, bool some) {
    __attribute__((aligned(8))) uint16_t out[4] = {f32_to_bf16(a), f32_to_bf16(b), f32_to_bf16(c), f32_to_bf16(d)};
    *(uint2*)p = some ? *(const uint2*)out : make_uint2(0, 0);
}

// The keys of a split in the ring kernel: whole 64-key tiles, dealt out evenly by the length
// of the query's mixed set.  Cut by the capacity of its buffers, which variable chunk lengths leave partly empty,
// the last splits of a query had no keys and the others more than their share: eight questions of 224 rows over
// 25,500 of 35,410 rows (64 of 256 workgroups without keys), gather included, 285 -> 263 us.
// (The step kernel below keeps the cut by capacity: its first request does not wait for the length, and dealing
// its tiles out by workgroup or by wave in turn won 1 % on ragged sets and lost 1 to 4 % on full ones.)
struct KeyRange { int lo, hi; };
__device__ __forceinline__ KeyRange split_keys(int len, int split, int n_split) {
    const int tiles = (len + kKeyTile - 1) / kKeyTile, per = tiles / n_split, more = tiles % n_split;
    const int first = split * per + min(split, more);
    return {first * kKeyTile, min((first + per + (split < more ? 1 : 0)) * kKeyTile, len)};
}

// ------------------------------------------------------------------------------------------
// Kernel of the calls with many stacked query rows: 32 rows per wave, 4 waves (one per SIMD) or, beyond 128 rows, 8 (two)
// per workgroup (choose_ring draws the line), the split's 64-key tiles streamed into a ring of NS
// LDS stages by direct global->LDS loads, two tiles ahead of the arithmetic -- the structure of
// the streaming pre-filling kernel, without its causal part.
// Eight waves are bound by matrix and vector issue with the clock they draw (1.6 us per tile), which a long split
// repays.  Four walk a tile in 1.05 us, half the rows, so that a launch that fills the chip has half the splits: short
// splits are bound by start and end -- a call takes 9 us besides, and 0.5 us per MB of fp32 partial rows, written and
// merged.  With one wave per SIMD nothing hides its LDS reads, so their order is pinned as in the pre-filling kernel
// (1,456 tiles of 224 rows in 256 workgroups 45.7 -> 43.1 us; with eight waves 122.6 -> 124.5 on 418 MB).  The refills
// wait their turn between two tiles: both at the meeting delay the first one (238 -> 242 us with the gather), and one
// meeting per tile with three tiles ahead is no faster.  The loads are issued from inline
// assembly and counted by hand (every wave issues the same number per tile and waits with
// vmcnt = loads still allowed in flight), so the kernel must not spill, and the query registers
// are forced complete before the first ring load.
// Up to 128 rows, and up to 256 where a launch of eight waves is small, four waves took the place of a kernel that moved
// its tiles through registers into two LDS buffers, two workgroups per compute unit: faster in all of 110 random calls
// (D = 128: 49 rows, 3,982 keys 15.6 -> 13.3 us; 33 queries of 35 rows over 12,426 keys 417 -> 199).
// ------------------------------------------------------------------------------------------
template <int D, int NS, int NW>
struct DecodeRingCfg {
    static constexpr int WAVES = NW;
    static constexpr int RT = 32 * WAVES;                     // query rows per workgroup
    static constexpr int TILE = kKeyTile * D;                 // elements of one unpadded K (or V) tile
    static constexpr int STAGE = 2 * TILE;                    // K tile then V tile
    static constexpr int LDS_BYTES = NS * STAGE * 2;
    static constexpr int PPR = D / 8;                         // 16-byte pieces per row
    static constexpr int RPI = 64 / PPR;                      // rows per load instruction (1 KiB)
    static constexpr int NI = kKeyTile / RPI;                 // instructions per tile per matrix
    static constexpr int IPW = NI / WAVES;                    // ... per wave
    static constexpr int GROUP = 2 * IPW;                     // loads per wave per tile (K and V)
};

// IND (in-place form): the rows of a tile are reached through the row map.  A lane needs one map
// entry per load slot and tile; the entries of tiles t+2, t+3 are fetched (by loads issued from
// inline assembly, so that they ride in the hand-kept vmcnt count) when the loads of tiles t, t+1 are
// issued, and are complete behind the same vmcnt(0) that tiles t, t+1 wait for.
template <int D, int NS, int NW, bool IND = false, bool ONCE = false>
__global__ __launch_bounds__(64 * NW, 2) void decode_ring_kernel(
    const uint16_t* __restrict__ Qd, const uint16_t* __restrict__ Kmix, const uint16_t* __restrict__ Vmix,
    const int32_t* __restrict__ mix_len, float* __restrict__ part_o, float* __restrict__ part_lse, int T_q,
    int n_q_heads, int n_kv_heads, int group, int l_cap, float scale, RowMap rm, uint16_t* __restrict__ O, float* __restrict__ LSE) {
    using C = DecodeRingCfg<D, NS, NW>;
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = blockIdx.x, n_split = gridDim.x;
    const int g = blockIdx.y % n_kv_heads, rt = blockIdx.y / n_kv_heads;
    const int b = blockIdx.z;
    const int n_rows = group * T_q;
    const KeyRange keys = split_keys(__builtin_amdgcn_readfirstlane(min(max(mix_len[b], 0), l_cap)), split, n_split);
    const int k_lo = __builtin_amdgcn_readfirstlane(keys.lo), k_hi = __builtin_amdgcn_readfirstlane(keys.hi);
    const int wrow0 = rt * C::RT + wave * 32;
    const size_t part_base = (((size_t)b * n_kv_heads + g) * n_split + split) * (size_t)n_rows;

    if (k_lo >= k_hi) {                            // empty split: only its weight (zero) is recorded
        if (n_split > 1) {
            for (int r = rt * C::RT + tid; r < min(n_rows, (rt + 1) * C::RT); r += 64 * NW) part_lse[part_base + r] = -INFINITY;
        } else {
            for (int e = tid; e < min(n_rows - rt * C::RT, C::RT) * (D / 4); e += 64 * NW) {
                const int rho = rt * C::RT + e / (D / 4);
                const size_t row = ((size_t)b * T_q + rho / group) * n_q_heads + g * group + rho % group;
                store_row4(O + row * D + e % (D / 4) * 4, 0.f, 0.f, 0.f, 0.f, false);
                if (LSE && e % (D / 4) == 0) LSE[row] = -INFINITY;
            }
        }
        return;
    }
    const int n_t = (k_hi - k_lo + kKeyTile - 1) / kKeyTile;
    // (IND: Kmix / Vmix are the dense K / V of the layer)
    const char* kbase = IND ? (const char*)(Kmix + (size_t)g * rm.kv_head)
                            : (const char*)(Kmix + (((size_t)b * n_kv_heads + g) * (size_t)l_cap + k_lo) * D);
    const char* vbase = IND ? (const char*)(Vmix + (size_t)g * rm.kv_head)
                            : (const char*)(Vmix + (((size_t)b * n_kv_heads + g) * (size_t)l_cap + k_lo) * D);
    const long long ksp_delta = IND ? (const char*)(rm.Ksp + (size_t)g * rm.s_total * D) - kbase : 0;
    const long long vsp_delta = IND ? (const char*)(rm.Vsp + (size_t)g * rm.s_total * D) - vbase : 0;
    const long long kv_tok_bytes = IND ? rm.kv_tok * 2 : 0;
    const int32_t* src_s = IND ? rm.src_idx + (size_t)b * l_cap + k_lo : nullptr;      // map entries of this split
    const int r_in = lane / C::PPR, pp = lane % C::PPR;

    // IND: map entries of this lane's load slots for one tile
    struct TileMap { int e[C::IPW]; };
    auto load_map = [&](int t, TileMap& m) __attribute__((always_inline)) {
        const int row0 = t * kKeyTile;
        const int rlim = min(kKeyTile - 1, k_hi - k_lo - 1 - row0);
#pragma unroll
        for (int i = 0; i < C::IPW; ++i)
            m.e[i] = load_i32_hidden(src_s + row0 + min((wave + i * C::WAVES) * C::RPI + r_in, rlim));
    };
    // Tile t -> stage t % NS.  Every wave issues GROUP loads: instruction slots wave + i * WAVES, ...
    // Rows past the end of the split are clamped to its last row (scores masked, V finite).
    auto issue = [&](int t, const TileMap& m) __attribute__((always_inline)) {
        const int row0 = t * kKeyTile;
        const int rlim = min(kKeyTile - 1, k_hi - k_lo - 1 - row0);
        const char* kb = kbase + (size_t)row0 * (D * 2);
        const char* vb = vbase + (size_t)row0 * (D * 2);
        const uint32_t st = lds_base + (uint32_t)(t % NS) * (C::STAGE * 2);
#pragma unroll
        for (int i = 0; i < C::IPW; ++i) {
            const int slot = wave + i * C::WAVES;
            const int row = slot * C::RPI + r_in;
            const int kp = pp ^ ((row / (16 / C::PPR)) & (C::PPR - 1));
            constexpr int CPR = D * 2 / 64, RPL = D == 128 ? 1 : 2;
            const int vp = (((pp >> 2) ^ ((row / RPL) & (CPR - 1))) << 2) | (pp & 3);
            if constexpr (IND) {
                const long long ko = mapped_row_offset(m.e[i], kv_tok_bytes, D * 2, ksp_delta);
                const long long vo = mapped_row_offset(m.e[i], kv_tok_bytes, D * 2, vsp_delta);
                dma16_addr(kbase + ko + kp * 16, st + slot * 1024);
                dma16_addr(vbase + vo + vp * 16, st + C::TILE * 2 + slot * 1024);
            } else {
                const uint32_t roff = (uint32_t)min(row, rlim) * (D * 2);
                dma16_as<ONCE>(kb, roff + kp * 16, st + slot * 1024);
                dma16_as<ONCE>(vb, roff + vp * 16, st + C::TILE * 2 + slot * 1024);
            }
        }
    };
    // Two groups of TPB stages: one is consumed while the other is refilled, one workgroup barrier
    // per TPB tiles.
    constexpr int TPB = 2;
    static_assert(NS == 2 * TPB, "two groups of TPB stages");
    TileMap ma{}, mb{};                                       // entries of the next two tiles to be issued
    if constexpr (IND) {
        load_map(0, ma);
        load_map(min(1, n_t - 1), mb);
        wait_vmcnt<0>();
#pragma unroll
        for (int i = 0; i < C::IPW; ++i) { settle_i32(ma.e[i]); settle_i32(mb.e[i]); }
    }
    issue(0, ma);
    issue(min(1, n_t - 1), mb);
    if constexpr (IND) {                                      // entries of tiles 2, 3: complete behind the first meeting's wait
        load_map(min(2, n_t - 1), ma);
        load_map(min(3, n_t - 1), mb);
    }

    // Query rows: loaded after the ring has been started (the latencies overlap) and forced
    // complete here; from here on no load the compiler knows of is outstanding.
    bf16x8 qreg[1][D / 16];
    {
        const int rho = min(wrow0 + l32, n_rows - 1);
        const int t = rho / group, hg = rho % group;
        const uint4* src = (const uint4*)(Qd + (((size_t)b * T_q + t) * n_q_heads + g * group + hg) * D);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qreg[0][ks] = __builtin_bit_cast(bf16x8, src[ks * 2 + hi]);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
            asm volatile("" :: "v"(__builtin_bit_cast(u32x4, qreg[0][ks])));
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x16 o[1][D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[0][db] = zero16();
    float m_run = -INFINITY, l_run = 0.f;
    const float c2 = scale * kLog2e;
    const bool wave_active = wrow0 < n_rows;       // waves without rows only help with the loads

    auto process = [&](int ti) {
        if (!wave_active) return;
        const uint16_t* kt = lds + (ti % NS) * C::STAGE;
        const int key0 = k_lo + ti * kKeyTile;
        f32x16 s[1][2];
        if constexpr (NW == 4) qk_tile_ahead<D, 1>(kt, qreg, l32, hi, s);
        else qk_tile<D, 1>(kt, qreg, l32, hi, s);
        if (key0 + kKeyTile > k_hi) {
            const int lim = k_hi - key0 - 1;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[0][kb][r] = acc_key(kb, r, hi) <= lim ? s[0][kb][r] : -INFINITY;
        }
        bf16x8 pb[1][2][2];
        softmax_tile<D / 32>(s[0], c2, m_run, l_run, o[0], pb[0]);
        if constexpr (NW == 4) pv_tile_ahead<D, 2>(kt + C::TILE, pb, lane, o);
        else pv_tile<D, 1>(kt + C::TILE, pb, lane, o);
    };
    for (int t0 = 0; t0 < n_t; t0 += TPB) {
        wait_vmcnt<0>();                                      // this wave's parts of tiles t0, t0+1 have landed
        __builtin_amdgcn_s_barrier();                         // ... and everyone's; the other group is free
        if constexpr (IND) {
#pragma unroll
            for (int i = 0; i < C::IPW; ++i) { settle_i32(ma.e[i]); settle_i32(mb.e[i]); }
        }
        issue(min(t0 + TPB, n_t - 1), ma);
        if constexpr (IND) load_map(min(t0 + 2 * TPB, n_t - 1), ma);
        process(t0);
        issue(min(t0 + TPB + 1, n_t - 1), mb);
        if constexpr (IND) load_map(min(t0 + 2 * TPB + 1, n_t - 1), mb);
        if (t0 + 1 < n_t) process(t0 + 1);
    }
    wait_vmcnt<0>();                                          // drain the refills before the wave ends

    if (!wave_active) return;
    const int rho = wrow0 + l32;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (rho >= n_rows) return;
    const float inv = 1.f / l_tot, lse = m_run * c2 + __builtin_amdgcn_logf(l_tot);
    if (n_split == 1) {
        const size_t row = ((size_t)b * T_q + rho / group) * n_q_heads + g * group + rho % group;
        const bool some = fabsf(lse) < INFINITY;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                store_row4(O + row * D + db * 32 + rq * 8 + hi * 4, o[0][db][rq * 4] * inv, o[0][db][rq * 4 + 1] * inv,
                           o[0][db][rq * 4 + 2] * inv, o[0][db][rq * 4 + 3] * inv, some);
        if (LSE && hi == 0) LSE[row] = some ? lse * kLn2 : -INFINITY;
        return;
    }
    float* orow = part_o + (part_base + rho) * D;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            float4 v;
            v.x = o[0][db][rq * 4 + 0] * inv;
            v.y = o[0][db][rq * 4 + 1] * inv;
            v.z = o[0][db][rq * 4 + 2] * inv;
            v.w = o[0][db][rq * 4 + 3] * inv;
            *(float4*)(orow + db * 32 + rq * 8 + hi * 4) = v;
        }
    if (hi == 0) part_lse[part_base + rho] = lse;
}

// ------------------------------------------------------------------------------------------
// Kernel of the calls that are latency or streaming rather than matrix work: at most 32 stacked query
// rows (the generated token, T = 1..4 at G = 7), or a few row tiles of 32 over a short mixed set
// (decode_plan draws the line).  Every WAVE owns its own 32-key tiles (tile = NW*(split*tpw + i) + wave) and its
// own LDS tile pairs, filled by direct global->LDS loads; there is no workgroup barrier in the
// loop.  The waves' running (reference, sum, O) are merged through LDS in wave order and the
// workgroup writes one normalised partial + base-2 LSE per row.
// Two forms, both filling 128 KiB of LDS: NW = 4 waves with two tile pairs each -- the next tile
// is requested before the current one is worked on, so a wave waits for memory once, not once per
// tile (the default: 3-8 % faster on long streams, 5 % at a single tile per wave, where it spreads
// over twice as many compute units) -- and NW = 8 waves with one tile pair each (cross-check).
constexpr int kStepTile = 32;       // keys per wave tile
constexpr int kMaxStepTpw = 32;     // in-place form: tiles per wave whose row map fits the wave's LDS area

// ONE: the workgroup walks all keys of its rows, several tiles per wave, each against a reference of its own, which the
// split form has by giving every tile a wave (7 rows, 501 keys: error against float64 2.02e-3; with references kept over
// the tiles of a wave 2.25e-3, and 0.7 us less).
template <int D, int NW, int NBUF, bool IND = false, bool ROWS = false, int MF = 4, bool ONCE = false, bool ONE = false>
__global__ __launch_bounds__(64 * NW, 2) void decode_wave_kernel(
    const uint16_t* __restrict__ Qd, const uint16_t* __restrict__ Kmix, const uint16_t* __restrict__ Vmix,
    const int32_t* __restrict__ mix_len, float* __restrict__ part_o, float* __restrict__ part_lse, int T_q,
    int n_q_heads, int n_kv_heads, int group, int l_cap, int tiles_per_wave, int n_split, int n_units, int n_rtile, float scale,
    RowMap rm, uint16_t* __restrict__ O, float* __restrict__ LSE) {
    static_assert(!IND || NBUF == 2, "the in-place form exists for the double-buffered kernel only");
    constexpr int TK = kStepTile;
    constexpr int TILE_ELEMS = TK * D;                         // one unpadded tile
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    __shared__ float2 stats[NW][32];                           // per wave and row: reference logit, sum
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t* Kw = lds + wave * NBUF * 2 * TILE_ELEMS;         // this wave's K tile, then its V tile (NBUF times)
    uint16_t* Vw = Kw + TILE_ELEMS;
    // One row tile: grid (split, KV head, query).  Several (ROWS): a one-dimensional grid in which the row tiles of
    // a unit = (query, KV head, split) are neighbours on one XCD (workgroups go to the eight XCDs in turn),
    // whose L2 then serves all but the first of them: id = (unit / 8 * n_rtile + row tile) * 8 + unit % 8.
    int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z, row0 = 0;
    if (!ROWS) n_split = gridDim.x;
    if constexpr (ROWS) {
        const int seq = blockIdx.x / kXcds, unit = seq / n_rtile * kXcds + blockIdx.x % kXcds;
        row0 = seq % n_rtile * 32;
        if (unit >= n_units) return;
        split = unit % n_split;
        g = unit / n_split % n_kv_heads;
        b = unit / n_split / n_kv_heads;
    }
    const int all_rows = group * T_q, n_rows = ROWS ? min(32, all_rows - row0) : all_rows;   // rows of the call, of this workgroup
    const int len = min(max(mix_len[b], 0), l_cap);
    const int n_tiles = (len + TK - 1) / TK;
    const size_t part_base = (((size_t)b * n_kv_heads + g) * n_split + split) * (size_t)all_rows + row0;

    const float c2 = scale * kLog2e;
    // (IND: Kmix / Vmix are the dense K / V of the layer, read through the row map)
    const char* kbase = IND ? (const char*)(Kmix + (size_t)g * rm.kv_head)
                            : (const char*)(Kmix + ((size_t)b * n_kv_heads + g) * (size_t)l_cap * D);
    const char* vbase = IND ? (const char*)(Vmix + (size_t)g * rm.kv_head)
                            : (const char*)(Vmix + ((size_t)b * n_kv_heads + g) * (size_t)l_cap * D);
    const int tile0 = split * tiles_per_wave * NW + wave;      // this wave's tiles: tile0, tile0 + NW, ...
    // IND: the source rows of this wave's tiles go to LDS first (ordinary loads, complete before the
    // first hand-counted request), so that the requests depend on LDS reads only.
    __shared__ int32_t row_src[IND ? NW * kMaxStepTpw * TK : 1];
    int32_t* src_w = row_src + (IND ? wave * kMaxStepTpw * TK : 0);
    // byte distances from the dense to the sparse buffers (one base per tensor keeps the addresses in registers)
    const long long ksp_delta = IND ? (const char*)(rm.Ksp + (size_t)g * rm.s_total * D) - kbase : 0;
    const long long vsp_delta = IND ? (const char*)(rm.Vsp + (size_t)g * rm.s_total * D) - vbase : 0;
    const long long kv_tok_bytes = IND ? rm.kv_tok * 2 : 0;
    if constexpr (IND) {
        // (all entries up to the capacity, so that these loads do not wait for the length; entries at
        // and past the length may be anything and are never turned into addresses: request() clamps the
        // row index to the last valid one before it reads the map)
        const int32_t* src_b = rm.src_idx + (size_t)b * l_cap;
        for (int i = 0; i < tiles_per_wave; ++i) {
            const int tile = tile0 + i * NW;
            if (tile * TK >= l_cap) break;
            if (lane < TK) src_w[i * TK + lane] = src_b[min(tile * TK + lane, l_cap - 1)];
        }
        __builtin_amdgcn_s_waitcnt(0x0070);                    // vmcnt(0) lgkmcnt(0): the map is in LDS
        __builtin_amdgcn_wave_barrier();
    }

    // NBUF == 2: direct loads issued from inline assembly and counted by hand (a later request
    // must be allowed to stay in flight while an earlier tile is read).
    constexpr int PPR = D / 8, RPI = 64 / PPR, NL = TK / RPI;  // pieces per row; rows, 1 KiB lines per tile
    const uint32_t lds_w = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)Kw;
    // i_ = position of the tile among this wave's tiles (its row map is src_w + i_ * TK)
    // n_valid = rows that may be read: the mixed length, or (gathered form, first request only) the
    // capacity of the buffers, so that the first request does not wait for the load of the length.
    auto request = [&](int i_, int tile_, int buf, int n_valid) __attribute__((always_inline)) {
        const int key0_ = tile_ * TK;
        const int rlim_ = min(TK - 1, n_valid - 1 - key0_);
        const char* kb = kbase + (size_t)key0_ * (D * 2);
        const char* vb = vbase + (size_t)key0_ * (D * 2);
        const int r_in = lane / PPR, pp = lane % PPR;
        int src_row[NL];                                       // IND: source row of this lane's row in every load
        if constexpr (IND) {
            // rows x * RPI + r_in, clamped to the last valid one: a constant stride except at the clamp
            const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(src_w + i_ * TK);
            // A full tile whose 32 entries are consecutive rows of one source (a dense chunk: e0, e0 + 1,
            // ...; the sparse buffer: e0, e0 - 1, ...) is fetched like a tile of a gathered buffer, from
            // one scalar base with 32-bit lane offsets: the same number of loads, far fewer instructions.
            if (rlim_ == TK - 1) {
                int ent[1];
                lds_read_i32_hidden<1>(base + (lane & (TK - 1)) * 4, 0, ent);
                const int e0 = __builtin_amdgcn_readfirstlane(ent[0]);
                const int step = e0 >= 0 ? 1 : -1;
                if (kv_tok_bytes < (1ll << 26) &&                // (32 rows x stride must fit the 32-bit lane offset)
                    __builtin_amdgcn_ballot_w64(ent[0] != e0 + step * (lane & (TK - 1))) == 0) {
                    const char* kb1 = kbase + mapped_row_offset(e0, kv_tok_bytes, D * 2, ksp_delta);
                    const char* vb1 = vbase + mapped_row_offset(e0, kv_tok_bytes, D * 2, vsp_delta);
                    const uint32_t row_bytes = e0 >= 0 ? (uint32_t)kv_tok_bytes : (uint32_t)(D * 2);
#pragma unroll
                    for (int x = 0; x < NL; ++x) {
                        const int row = x * RPI + r_in;
                        const int kp = pp ^ ((row / (16 / PPR)) & (PPR - 1));
                        constexpr int CPR = D * 2 / 64, RPL = D == 128 ? 1 : 2;
                        const int vp = (((pp >> 2) ^ ((row / RPL) & (CPR - 1))) << 2) | (pp & 3);
                        const uint32_t kdst = lds_w + (uint32_t)buf * (4 * TILE_ELEMS) + x * 1024;
                        dma16(kb1, (uint32_t)row * row_bytes + kp * 16, kdst);
                        dma16(vb1, (uint32_t)row * row_bytes + vp * 16, kdst + 2 * TILE_ELEMS);
                    }
                    return;
                }
            }
            if (rlim_ == TK - 1) {
                lds_read_i32_hidden<NL>(base + r_in * 4, RPI * 4, src_row);
            } else {
#pragma unroll
                for (int x = 0; x < NL; ++x) {
                    int one[1];
                    lds_read_i32_hidden<1>(base + min(x * RPI + r_in, rlim_) * 4, 0, one);
                    src_row[x] = one[0];
                }
            }
        }
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const int row = x * RPI + r_in;
            const int kp = pp ^ ((row / (16 / PPR)) & (PPR - 1));
            constexpr int CPR = D * 2 / 64, RPL = D == 128 ? 1 : 2;
            const int vp = (((pp >> 2) ^ ((row / RPL) & (CPR - 1))) << 2) | (pp & 3);
            const uint32_t kdst = lds_w + (uint32_t)buf * (4 * TILE_ELEMS) + x * 1024;
            const uint32_t vdst = kdst + 2 * TILE_ELEMS;
            if constexpr (IND) {
                const long long ko = mapped_row_offset(src_row[x], kv_tok_bytes, D * 2, ksp_delta);
                const long long vo = mapped_row_offset(src_row[x], kv_tok_bytes, D * 2, vsp_delta);
                dma16_addr(kbase + ko + kp * 16, kdst);
                dma16_addr(vbase + vo + vp * 16, vdst);
            } else {
                const uint32_t roff = (uint32_t)min(row, rlim_) * (D * 2);
                dma16_as<ONCE>(kb, roff + kp * 16, kdst);
                dma16_as<ONCE>(vb, roff + vp * 16, vdst);
            }
        }
    };
    if constexpr (NBUF == 2) {
        // Gathered form: rows up to the capacity are readable memory whatever the length turns out
        // to be (rows past it are masked when the tile is worked on, and a wave without tiles drains
        // the request before the merge), so tile 0 is requested before the length has arrived.
        if constexpr (IND) { if (tile0 < n_tiles) request(0, tile0, 0, len); }
        else { if (tile0 * TK < l_cap) request(0, tile0, 0, l_cap); }
    }

    bf16x8 qreg[1][D / 16];
    {
        const int rho = row0 + min(l32, n_rows - 1);
        const int t = rho / group, hg = rho % group;
        const uint4* src = (const uint4*)(Qd + (((size_t)b * T_q + t) * n_q_heads + g * group + hg) * D);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qreg[0][ks] = __builtin_bit_cast(bf16x8, src[ks * 2 + hi]);
        if constexpr (NBUF == 2) {
            // forced complete here: the compiler's wait for them covers the older request of tile 0
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) {
                typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
                asm volatile("" :: "v"(__builtin_bit_cast(u32x4, qreg[0][ks])));
            }
        }
    }
    if constexpr (NBUF == 2 && !IND) {
        // The early request took rows past the mixed length as they are; their V values may be anything
        // (0 x NaN), so the one tile that straddles the length is fetched again with its rows clamped.
        // Loads of a wave return in order: the second copy lands on top of the first.
        if (tile0 < n_tiles && tile0 * TK + TK > len) {
            request(0, tile0, 0, len);
            wait_vmcnt<0>();
        }
    }
    f32x16 o[1][D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[0][db] = zero16();
    float m_run = -INFINITY, l_run = 0.f, m_top = -INFINITY;

    auto work = [&](const uint16_t* kt, const uint16_t* vt, int rlim, bool first) {
        f32x16 s[1][1];
        // (one wave per SIMD: nothing hides the LDS reads, so over several tiles they are pinned ahead of the instructions that
        // use them: 224 rows over 4,096 keys 14.2 -> 13.9 us, 112 over 10,000 15.1 -> 14.7; one row block, which waits for
        // memory, 0.99 to 1.01)
        if constexpr (ROWS) qk_tile_ahead<D, 3, 1>(kt, qreg, l32, hi, s);
        else qk_tile<D, 1, 1>(kt, qreg, l32, hi, s);
        if (rlim < TK - 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[0][0][r] = acc_key(0, r, hi) <= rlim ? s[0][0][r] : -INFINITY;
        }
        bf16x8 pb[1][1][2];
        if (ONE && !first) refer_to_tile<D / 32, 1>(s[0], c2, m_top, m_run, l_run, o[0]);
        softmax_tile<D / 32, 1>(s[0], c2, m_run, l_run, o[0], pb[0]);
        if constexpr (ROWS) pv_tile_ahead<D, 3, 1>(vt, pb, lane, o);
        else pv_tile<D, 1, 1>(vt, pb, lane, o);
    };
    if constexpr (NBUF == 1) {
        for (int i = 0; i < tiles_per_wave; ++i) {
            const int tile = tile0 + i * NW;
            if (tile >= n_tiles) break;
            const int key0 = tile * TK;
            const int rlim = min(TK - 1, len - 1 - key0);
            dma_tile_wave<D, TK>(kbase + (size_t)key0 * (D * 2), vbase + (size_t)key0 * (D * 2), Kw, Vw, lane, rlim);
            __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the tile is in LDS
            __builtin_amdgcn_wave_barrier();
            work(Kw, Vw, rlim, i == 0);
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        // tile i lives in pair i & 1; tile i + 1 is requested as soon as tile i - 1 has been worked on
        if (tiles_per_wave > 1 && tile0 + NW < n_tiles) request(1, tile0 + NW, 1, len);
        for (int i = 0; i < tiles_per_wave; ++i) {
            const int tile = tile0 + i * NW;
            if (tile >= n_tiles) break;
            if (i >= 1) {
                const bool more = i + 1 < tiles_per_wave && tile + NW < n_tiles;
                if (more) request(i + 1, tile + NW, (i + 1) & 1, len);
                if (more) wait_vmcnt<2 * NL>(); else wait_vmcnt<0>();      // tile i has landed
            }
            __builtin_amdgcn_wave_barrier();
            const uint16_t* kt = Kw + (i & 1) * 2 * TILE_ELEMS;
            work(kt, kt + TILE_ELEMS, min(TK - 1, len - 1 - tile * TK), i == 0);
            __builtin_amdgcn_wave_barrier();
        }
        wait_vmcnt<0>();                                       // (a wave without tiles: its early request of tile 0)
    }

    // ---- merge the waves (their tile buffers are free now): area [32 rows][D] floats per wave ----
    // A chain of LDS round trips at the end of every call, so it moves MF = 4 floats per lane and step: piece c4
    // of a row lies at c4 ^ row (mod the D / 4 pieces), which spreads the rows that a wave writes side by
    // side over all banks (unswizzled they all start at the same one).  One float (MF = 1) where the rows have
    // no more floats than the workgroup has threads: one step either way, and a quarter of the divisions (one
    // row, 4 KV heads of D = 64, 652 keys 7.0 -> 6.8 us; chosen inside the kernel the other calls pay 0.2).
    // Four floats against one: one layer of a generated token over 18,176 keys (with the merge
    // of the splits) 14.5 -> 13.7 us, a question of 224 rows on a 16k prompt, selection to decode, 33.5 -> 32.0.
    static_assert(32 * D * 4 <= 2 * TILE_ELEMS * 2, "merge area must fit a wave's tile pair");
    constexpr int PPR4 = D / 4;                                // 16-byte pieces per row
    float4* red = (float4*)Kw;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (l32 < n_rows) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                float4 v;
                v.x = o[0][db][rq * 4 + 0]; v.y = o[0][db][rq * 4 + 1];
                v.z = o[0][db][rq * 4 + 2]; v.w = o[0][db][rq * 4 + 3];
                red[l32 * PPR4 + ((db * 8 + rq * 2 + hi) ^ (l32 & (PPR4 - 1)))] = v;
            }
        if (hi == 0) stats[wave][l32] = make_float2(m_run, l_tot);
    }
    __syncthreads();
    constexpr int WSTRIDE = NBUF * 2 * TILE_ELEMS / 2;         // floats between the waves' areas
    const float* red0 = (const float*)lds;
    typedef __attribute__((ext_vector_type(MF))) float Vec;
    for (int e = tid; e < n_rows * (D / MF); e += 64 * NW) {
        const int row = e / (D / MF), dd = e % (D / MF) * MF;
        const int at = (row * PPR4 + ((dd >> 2) ^ (row & (PPR4 - 1)))) * 4 + (dd & 3);
        float2 st[NW];
        Vec v[NW];
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            st[w] = stats[w][row];
            v[w] = *(const Vec*)(red0 + w * WSTRIDE + at);
            M = fmaxf(M, st[w].x);
        }
        Vec acc = {};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const bool some = st[w].x != -INFINITY;
            const float f = some ? __builtin_amdgcn_exp2f((st[w].x - M) * c2) : 0.f;
            L = fmaf(f, st[w].y, L);
#pragma unroll
            for (int i = 0; i < MF; ++i) acc[i] = fmaf(f, some ? v[w][i] : 0.f, acc[i]);
        }
        const bool empty = M == -INFINITY;
#pragma unroll
        for (int i = 0; i < MF; ++i) acc[i] = empty ? 0.f : acc[i] / L;
        const float lse = empty ? -INFINITY : M * c2 + __builtin_amdgcn_logf(L);
        if (n_split == 1) {
            const int rho = row0 + row;
            const size_t out = ((size_t)b * T_q + rho / group) * n_q_heads + g * group + rho % group;
            const bool some = fabsf(lse) < INFINITY;
            if constexpr (MF == 4) store_row4(O + out * D + dd, acc[0], acc[1], acc[2], acc[3], some);
            else O[out * D + dd] = some ? f32_to_bf16(acc[0]) : (uint16_t)0;
            if (LSE && dd == 0) LSE[out] = some ? lse * kLn2 : -INFINITY;
            continue;
        }
        *(Vec*)(part_o + (part_base + row) * D + dd) = acc;
        if (dd == 0) part_lse[part_base + row] = lse;
    }
}

// The fixed-order merge of the key splits.  WPR waves per query row (4, one workgroup per row, or 1, four rows
// per workgroup): a thread takes four columns of every SG-th split, at most PRE of them requested together
// with their LSEs before the first weight exists, and folds them relative to the largest LSE it has seen; the
// SUB split groups of a wave are folded by lane exchange, the waves of a row through LDS, in an order that
// depends on the split index alone: a call gives the same bits every time.  Rows of splits with weight 0 are
// loaded but never used.
// Bound by latency, not volume: with the weights in LDS and three barriers in a chain, one workgroup per row, a
// call of 7 rows x 4 heads over 161 keys took 7.3 us, over 4,000 keys 8.7, of 448 rows x 8 over 512 keys 17.7;
// so 6.6, 8.3 and 13.4.
template <int D, int WPR, int PRE>
__global__ __launch_bounds__(256) void decode_merge_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_lse,
                                                           uint16_t* __restrict__ O, float* __restrict__ LSE,
                                                           int T_q, int n_q_heads, int n_kv_heads, int group,
                                                           int n_split) {
    constexpr int NV = D / 4;                       // lanes per row: a float4 each
    constexpr int SUB = 64 / NV, SG = WPR * SUB;    // split groups of a wave, of a row
    __shared__ __attribute__((aligned(16))) float red[WPR][D];
    __shared__ float2 stat[WPR];
    const int n_rows = group * T_q, lane = threadIdx.x & 63, dq = lane % NV;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rho = blockIdx.x * (4 / WPR) + wave / WPR, g = blockIdx.y, b = blockIdx.z;
    if (rho >= n_rows) return;                      // (whole waves; with WPR = 4 none)
    const size_t base = ((size_t)b * n_kv_heads + g) * n_split;
    const float* po = part_o + (base * n_rows + rho) * D + dq * 4;      // split s: s * n_rows rows further
    const float* pl = part_lse + base * n_rows + rho;
    const unsigned split_stride = (unsigned)n_rows * D;
    const size_t out_row = ((size_t)b * T_q + rho / group) * n_q_heads + g * group + rho % group;

    // (a part without weight counts 0 whatever it holds; a sum that is not a number stays one)
    auto part_weight = [](float m_part, float l_part, float m_all) __attribute__((always_inline)) {
        return l_part == 0.f ? 0.f : __builtin_amdgcn_exp2f(m_part - m_all);
    };
    auto scaled = [](float w, float x) __attribute__((always_inline)) { return w == 0.f ? 0.f : w * x; };
    float m = -INFINITY, l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = wave % WPR * SUB + lane / NV; s0 < n_split; s0 += PRE * SG) {
        float4 v[PRE];
        float e[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) e[i] = pl[(size_t)min(s0 + i * SG, n_split - 1) * n_rows];   // clamped: always a row of this (b, g)
#pragma unroll
        for (int i = 0; i < PRE; ++i) v[i] = *(const float4*)(po + (size_t)min(s0 + i * SG, n_split - 1) * split_stride);
        __builtin_amdgcn_sched_barrier(0);
        float m_new = m;
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            if (s0 + i * SG >= n_split) e[i] = -INFINITY;
            m_new = fmaxf(m_new, e[i]);
        }
        const float f = part_weight(m, l, m_new);
        l *= f;
        acc.x = scaled(f, acc.x); acc.y = scaled(f, acc.y); acc.z = scaled(f, acc.z); acc.w = scaled(f, acc.w);
        m = m_new;
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const float w = e[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(e[i] - m);
            l += w;
            if (w != 0.f) {
                acc.x = fmaf(w, v[i].x, acc.x);
                acc.y = fmaf(w, v[i].y, acc.y);
                acc.z = fmaf(w, v[i].z, acc.z);
                acc.w = fmaf(w, v[i].w, acc.w);
            }
        }
    }
#pragma unroll
    for (int o = NV; o < 64; o <<= 1) {
        const float m_o = __shfl_xor(m, o), l_o = __shfl_xor(l, o), M = fmaxf(m, m_o);
        const float4 a_o = make_float4(__shfl_xor(acc.x, o), __shfl_xor(acc.y, o), __shfl_xor(acc.z, o), __shfl_xor(acc.w, o));
        const float f = part_weight(m, l, M), f_o = part_weight(m_o, l_o, M);
        l = l * f + l_o * f_o;
        acc.x = scaled(f, acc.x) + scaled(f_o, a_o.x);
        acc.y = scaled(f, acc.y) + scaled(f_o, a_o.y);
        acc.z = scaled(f, acc.z) + scaled(f_o, a_o.z);
        acc.w = scaled(f, acc.w) + scaled(f_o, a_o.w);
        m = M;
    }
    // an empty mixed set (every split recorded weight 0): O = 0, LSE = -inf
    if constexpr (WPR > 1) {                        // a column per thread: one division in the chain
        if (lane < NV) *(float4*)(&red[wave][dq * 4]) = acc;
        if (lane == 0) stat[wave] = make_float2(m, l);
        __syncthreads();
        if (threadIdx.x >= D) return;
        float M = stat[0].x, a = 0.f;
#pragma unroll
        for (int w = 1; w < WPR; ++w) M = fmaxf(M, stat[w].x);
        l = 0.f;
#pragma unroll
        for (int w = 0; w < WPR; ++w) {
            const float f = part_weight(stat[w].x, stat[w].y, M);
            l = fmaf(f, stat[w].y, l);
            a += scaled(f, red[w][threadIdx.x]);
        }
        const bool empty = !(l > 0.f);
        O[out_row * D + threadIdx.x] = empty ? (uint16_t)0 : f32_to_bf16(a / l);
        if (LSE && threadIdx.x == 0) LSE[out_row] = empty ? -INFINITY : (M + __builtin_amdgcn_logf(l)) * kLn2;
    } else if (lane < NV) {
        const bool empty = !(l > 0.f);
        const float a[4] = {acc.x, acc.y, acc.z, acc.w};
        __attribute__((aligned(8))) uint16_t out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = empty ? (uint16_t)0 : f32_to_bf16(a[i] / l);
        *(uint2*)(O + out_row * D + dq * 4) = *(const uint2*)out;
        if (LSE && dq == 0) LSE[out_row] = empty ? -INFINITY : (m + __builtin_amdgcn_logf(l)) * kLn2;
    }
}

}  // namespace

// Buffers that one row tile reads once and the eight L2s (32 MB) do not hold, by their capacity, are streamed past the
// caches: 8 queries of 7 rows over 54 MB of mixed rows 28.0 -> 25.9 us, over 1.1 GB 227 -> 206, of 224 rows over 580 MB,
// gather included, 265 -> 255; but 8 MB, which the next call finds there, 8.0 -> 8.6, and 8 MB of rows in buffers for 80
// 11.3 -> 12.0.  (By the rows, decided in the kernel: those 11.8, but full sets 54.3 -> 55.3 and, a token of eight
// layers over 61,440 rows, 26.1 -> 26.9 a layer.)
static bool beyond_l2(const vxl_attn_desc* d, int batch, int l_cap) {
    return 4ll * batch * d->n_kv_heads * l_cap * d->head_dim > (32 << 20);
}

// The merge of a call: one wave per row while a thread's share of the splits is one batch of loads (8 splits: all
// 84 sizes measured 0 to 14 % faster so than with four), and where the rows alone fill the chip (448 rows x 8 heads,
// 16 splits 30.2 -> 28.4 us); otherwise four (28 rows of 16 and 31 splits: 8.4 -> 7.5 us and 9.4 -> 8.3).
template <int D>
static vxl_status launch_merge(int n_split, const float* part_o, const float* part_lse, void* O, float* LSE, int T,
                               const vxl_attn_desc* d, int batch, hipStream_t s) {
    if (n_split == 1) return VXL_OK;                          // (the kernel of the one split has written the results)
    const int group = d->n_q_heads / d->n_kv_heads, n_rows = group * T;
#define VXL_LAUNCH(WPR, PRE)                                                                                          \
    hipLaunchKernelGGL((decode_merge_kernel<D, WPR, PRE>), dim3((n_rows * WPR + 3) / 4, d->n_kv_heads, batch), dim3(256), \
                       0, s, part_o, part_lse, (uint16_t*)O, LSE, T, d->n_q_heads, d->n_kv_heads, group, n_split)
    if (n_split <= 8) VXL_LAUNCH(1, 4);
    else if ((long long)n_rows * d->n_kv_heads * batch >= 1024) VXL_LAUNCH(1, 8);
    else if (n_split <= 32) VXL_LAUNCH(4, 4);
    else VXL_LAUNCH(4, 8);
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return VXL_OK;
}

// How a call goes to the ring kernel of 8 or 4 waves (256 or 128 rows per workgroup; up to 128 rows always 4).
struct RingLaunch {
    int waves, n_split, n_rtile;
    bool spread;                // no two workgroups on a compute unit
    long long walk;             // tiles that the last workgroup has ended with
    float us;                   // estimate of kernel and merge
};
static RingLaunch ring_launch(const vxl_attn_desc* d, int batch, int rows, int l_cap, int most_splits, int n_cus, int waves,
                              bool in_place) {
    RingLaunch r{};
    const bool d64 = d->head_dim == 64;
    const int pairs = d->n_kv_heads * batch, tiles = (l_cap + kKeyTile - 1) / kKeyTile;
    r.waves = waves;
    r.n_rtile = (rows + 32 * waves - 1) / (32 * waves);
    const long long per_split = (long long)r.n_rtile * pairs;
    // One workgroup per compute unit: of the planned splits, which give every unit at least one, as many as run in
    // one round (gather included: 896 rows on six KV heads, 264 workgroups of 11 splits 118 us, 240 of 10 103; D =
    // 64, 700 rows on four, 264 workgroups 85, 252 62).  At D = 64 a unit holds two: kept apart by their LDS while every
    // workgroup has one of its own (301 rows, six heads, 252 of four waves over 23,178 keys 38.5 -> 28.6).
    r.n_split = (int)std::max(1ll, std::min<long long>(most_splits, n_cus / per_split));
    r.spread = d64 && r.n_split * per_split <= n_cus;
    const int slots = d64 && !r.spread ? 2 * n_cus : n_cus;
    const long long rounds = (r.n_split * per_split + slots - 1) / slots;
    // us of start, a tile (D = 64: of a workgroup alone on its unit, of one of two) and a MB of partial rows: least squares over
    // random calls of 129 to 1,400 rows.  Gathered, 139 (D = 128) and 120, in place 120 and 210; off by 6 to 8 % (rms) on the
    // half of the calls that was kept out of the fit.
    static constexpr float kUs[2][2][2][4] = {{{{8.9f, 1.62f, 1.62f, 0.51f}, {7.3f, 1.05f, 1.05f, 0.61f}},          // gathered
                                               {{7.1f, 1.04f, 1.73f, 0.72f}, {5.8f, 0.69f, 1.03f, 0.99f}}},
                                              {{{10.3f, 1.61f, 1.61f, 0.44f}, {8.4f, 1.10f, 1.10f, 0.62f}},         // in place
                                               {{7.9f, 1.08f, 2.24f, 0.70f}, {6.3f, 0.77f, 1.17f, 0.95f}}}};        // [D = 64][4 waves]
    const float* us = kUs[in_place][d64][waves == 4];
    r.walk = (tiles + r.n_split - 1) / r.n_split * rounds;
    const float mb = r.n_split > 1 ? 4e-6f * pairs * rows * r.n_split * d->head_dim : 0.f;
    r.us = us[0] + us[r.spread ? 1 : 2] * (float)r.walk + us[3] * mb;
    return r;
}

// Four waves where they are the shorter call by these estimates, in place by more than 4 %: over 159 gathered calls outside
// the fits the time is 0.92 of that of always eight (0.70 to 1.04), over 199 in place 0.92 (0.72 to 1.03; by 2 % three more were
// slower, to 1.04).  448 rows, 10,368 keys 29.4 -> 25.7 us; 588 rows x 8 queries, 674 keys, one split 26.2 -> 18.8; but 301 rows x 8,
// 23,830 keys 174.9 against 202 with four.  D = 64: not where a unit's two workgroups of four walk as many tiles each as its one
// of eight, the same waves that read the keys twice (in place, 1,316 rows x 8, 1,094 keys 27.4 with four, 25.1; 1,360 on eight
// heads x 3, 35,009 keys 673, 633; gathered, 1,233 on 16 heads x 3, 856 keys 23.4, 22.5).
static RingLaunch choose_ring(const vxl_attn_desc* d, int batch, int rows, int l_cap, int most_splits, int n_cus,
                              bool in_place) {
    const RingLaunch eight = ring_launch(d, batch, rows, l_cap, most_splits, n_cus, 8, in_place);
    const RingLaunch four = ring_launch(d, batch, rows, l_cap, most_splits, n_cus, 4, in_place);
    if (d->head_dim == 64 && !four.spread && eight.spread && four.walk >= eight.walk) return eight;
    return four.us < (in_place ? 0.96f : 0.98f) * eight.us && (long long)four.n_rtile * d->n_kv_heads <= 65535 ? four : eight;
}

// Test hook (vxl_debug.h): the waves of the ring kernel's workgroups on 256 compute units.
extern "C" int vxl_debug_decode_ring_waves(const vxl_attn_desc* d, int batch, int n_q_tokens, int l_cap, int in_place) {
    const DecodePlan p = decode_plan(d, batch, n_q_tokens, l_cap, !in_place);
    return choose_ring(d, batch, d->n_q_heads / d->n_kv_heads * n_q_tokens, l_cap, p.n_split, 256, in_place != 0)
        .waves;
}

template <int D, int NW>
static vxl_status launch_ring(const RingLaunch& rl, const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T,
                              const void* Kmix, const void* Vmix, int l_cap, const int32_t* mix_len, void* O, float* LSE,
                              float* part_o, float* part_lse, hipStream_t s, const RowMap* rm) {
    constexpr int kHalfLds = 81920;                           // of a compute unit
    constexpr int kRing = DecodeRingCfg<D, 4, NW>::LDS_BYTES, kApart = std::max(kRing, kHalfLds + 16);
    const int lds = rl.spread ? kApart : kRing;
    static PerDeviceOnce attr;
    const vxl_status ast = attr.run([] {
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_ring_kernel<D, 4, NW, false>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, kApart));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_ring_kernel<D, 4, NW, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, kApart));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_ring_kernel<D, 4, NW, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, kApart));
        return VXL_OK;
    });
    if (ast != VXL_OK) return ast;
    const dim3 grid(rl.n_split, rl.n_rtile * d->n_kv_heads, batch);
#define VXL_LAUNCH(...)                                                                                              \
    hipLaunchKernelGGL((decode_ring_kernel<D, 4, NW, __VA_ARGS__>), grid, dim3(64 * NW), lds, s, (const uint16_t*)Qd, \
                       (const uint16_t*)Kmix, (const uint16_t*)Vmix, mix_len, part_o, part_lse, T, d->n_q_heads,     \
                       d->n_kv_heads, d->n_q_heads / d->n_kv_heads, l_cap, scale, rm ? *rm : RowMap{}, (uint16_t*)O, LSE)
    if (rm) VXL_LAUNCH(true);
    else if (rl.n_rtile == 1 && beyond_l2(d, batch, l_cap)) VXL_LAUNCH(false, true);
    else VXL_LAUNCH(false);
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return launch_merge<D>(rl.n_split, part_o, part_lse, O, LSE, T, d, batch, s);
}

template <int D>
static vxl_status run_decode_ring(const DecodePlan& p, const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T,
                                  const void* Kmix, const void* Vmix, int l_cap, const int32_t* mix_len, void* O,
                                  float* LSE, void* ws, hipStream_t s, const RowMap* rm = nullptr) {
    float* part_o = (float*)((char*)ws + p.part_o);
    float* part_lse = (float*)((char*)ws + p.part_ml);
    int n_cus = 0;
    const vxl_status cst = device_cu_count(&n_cus);
    if (cst != VXL_OK) return cst;
    const int rows = d->n_q_heads / d->n_kv_heads * T;
    const RingLaunch rl = p.use_ring ? choose_ring(d, batch, rows, l_cap, p.n_split, n_cus, rm != nullptr)
                                     : ring_launch(d, batch, rows, l_cap, p.n_split, n_cus, 4, rm != nullptr);
    return rl.waves == 8
               ? launch_ring<D, 8>(rl, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, part_o, part_lse, s, rm)
               : launch_ring<D, 4>(rl, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, part_o, part_lse, s, rm);
}

template <int D>
static vxl_status run_decode_wave(const DecodePlan& p, const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T,
                                  const void* Kmix, const void* Vmix, int l_cap, const int32_t* mix_len, void* O,
                                  float* LSE, void* ws, hipStream_t s, const RowMap* rm = nullptr) {
    float* part_o = (float*)((char*)ws + p.part_o);
    float* part_lse = (float*)((char*)ws + p.part_ml);
    const int group = d->n_q_heads / d->n_kv_heads;
    const int n_rows = group * T;
    const int n_rtile = (n_rows + kRowBlock - 1) / kRowBlock;
    const int units = p.n_split * d->n_kv_heads * batch;
    const dim3 grid = n_rtile > 1 ? dim3((units + kXcds - 1) / kXcds * kXcds * n_rtile) : dim3(p.n_split, d->n_kv_heads, batch);
    constexpr int lds_bytes = 8 * 2 * kStepTile * D * 2;      // 8 tile pairs in either form
    static PerDeviceOnce attr;
    const vxl_status ast = attr.run([] {
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 8, 1>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, false, 4, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, false, 1, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, false, 1>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true, false, 1>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, false, 4, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, false, 1, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, false, true, 4, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true, false, 4, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true, false, 1, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        VXL_HIP_TRY(hipFuncSetAttribute((const void*)decode_wave_kernel<D, 4, 2, true, true, 4, false, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
        return VXL_OK;
    });
    if (ast != VXL_OK) return ast;
    const int tpw = p.split_len / ((p.step_waves == 8 ? 8 : 4) * kStepTile);
    // (the plan of the in-place form always has 4 waves; the row map of a wave's tiles must fit its LDS area)
    if (rm && tpw > kMaxStepTpw) return VXL_ERR_UNSUPPORTED;
#define VXL_LAUNCH(NW, ...)                                                                              \
    hipLaunchKernelGGL((decode_wave_kernel<D, NW, __VA_ARGS__>), grid, dim3(64 * NW), lds_bytes, s,       \
                       (const uint16_t*)Qd, (const uint16_t*)Kmix, (const uint16_t*)Vmix, mix_len, part_o, \
                       part_lse, T, d->n_q_heads, d->n_kv_heads, group, l_cap, tpw, p.n_split, units, n_rtile, \
                       scale, rm ? *rm : RowMap{}, (uint16_t*)O, LSE)
    const bool few = n_rows * D <= 64 * 4;                     // (see the merge of the waves)
    if (p.one) {
        if (rm) {
            if (n_rtile > 1) VXL_LAUNCH(4, 2, true, true, 4, false, true);
            else if (few) VXL_LAUNCH(4, 2, true, false, 1, false, true);
            else VXL_LAUNCH(4, 2, true, false, 4, false, true);
        }
        else if (n_rtile > 1) VXL_LAUNCH(4, 2, false, true, 4, false, true);
        else if (few) VXL_LAUNCH(4, 2, false, false, 1, false, true);
        else VXL_LAUNCH(4, 2, false, false, 4, false, true);
    }
    else if (rm) {
        if (n_rtile > 1) VXL_LAUNCH(4, 2, true, true);
        else if (few) VXL_LAUNCH(4, 2, true, false, 1);
        else VXL_LAUNCH(4, 2, true);
    }
    else if (p.step_waves == 8) VXL_LAUNCH(8, 1);
    else if (n_rtile > 1) VXL_LAUNCH(4, 2, false, true);
    else if (beyond_l2(d, batch, l_cap)) { if (few) VXL_LAUNCH(4, 2, false, false, 1, true); else VXL_LAUNCH(4, 2, false, false, 4, true); }
    else if (few) VXL_LAUNCH(4, 2, false, false, 1);
    else VXL_LAUNCH(4, 2);
#undef VXL_LAUNCH
    VXL_HIP_TRY(hipGetLastError());
    return launch_merge<D>(p.n_split, part_o, part_lse, O, LSE, T, d, batch, s);
}

// Scratch of the entry point that allocates nothing: one array per device, held until the process
// ends.  In host code the name below is only a stand-in for the symbol; the device address is
// asked for once per device (with that device current) and kept.
static __device__ __align__(256) unsigned char scratch[VXL_STATIC_SCRATCH_BYTES];

vxl_status decode_static_scratch(void** ptr) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    VXL_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return VXL_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        VXL_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return VXL_ERR_HIP;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return VXL_OK;
}

vxl_status launch_decode_bf16(const DecodePlan& p, const vxl_attn_desc* d, float scale, const void* Qd, int batch, int T,
                              const void* Kmix, const void* Vmix, int l_cap, const int32_t* mix_len, void* O,
                              float* LSE, void* ws, hipStream_t s) {
    if (p.step_waves != 0)
        return d->head_dim == 128
                   ? run_decode_wave<128>(p, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, ws, s)
                   : run_decode_wave<64>(p, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, ws, s);
    return d->head_dim == 128
               ? run_decode_ring<128>(p, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, ws, s)
               : run_decode_ring<64>(p, d, scale, Qd, batch, T, Kmix, Vmix, l_cap, mix_len, O, LSE, ws, s);
}

// In-place form: K / V are the dense tensors of the layer, rows reached through src_idx.
vxl_status launch_decode_bf16_inplace(const DecodePlan& p, const vxl_layout* L, const vxl_attn_desc* d, float scale, const void* Qd,
                                      int batch, int T, const void* K, const void* V, const void* Ksp,
                                      const void* Vsp, const int32_t* src_idx, int l_cap, const int32_t* mix_len,
                                      void* O, float* LSE, void* ws, hipStream_t s) {
    const TokStrides ts = tok_strides(d, L->n_tokens);
    const RowMap rm{src_idx, (const uint16_t*)Ksp, (const uint16_t*)Vsp, ts.kh, ts.kt, L->s_total};
    if (p.step_waves != 0)
        return d->head_dim == 128
                   ? run_decode_wave<128>(p, d, scale, Qd, batch, T, K, V, l_cap, mix_len, O, LSE, ws, s, &rm)
                   : run_decode_wave<64>(p, d, scale, Qd, batch, T, K, V, l_cap, mix_len, O, LSE, ws, s, &rm);
    return d->head_dim == 128
               ? run_decode_ring<128>(p, d, scale, Qd, batch, T, K, V, l_cap, mix_len, O, LSE, ws, s, &rm)
               : run_decode_ring<64>(p, d, scale, Qd, batch, T, K, V, l_cap, mix_len, O, LSE, ws, s, &rm);
}

}  // namespace vxl
