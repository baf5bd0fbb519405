// Host side of the C ABI: argument validation, the layout handle (device copies of the
// chunking and the pre-filling tile schedule), workspace planning and kernel dispatch.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <numeric>

#include "vxl_internal.h"

namespace vxl {

static thread_local char g_last_error[512] = "";
static std::atomic<int> g_force_simple{0};

void set_last_error(const char* what, hipError_t e) {
    snprintf(g_last_error, sizeof(g_last_error), "%s: %s", what, hipGetErrorString(e));
}

static bool desc_ok(const vxl_attn_desc* d, vxl_status* st) {
    if (!d) { *st = VXL_ERR_INVALID_ARG; return false; }
    if (d->n_q_heads <= 0 || d->n_kv_heads <= 0 || d->n_q_heads % d->n_kv_heads != 0 ||
        !(d->softmax_scale >= 0.0f) || !std::isfinite(d->softmax_scale)) {
        *st = VXL_ERR_INVALID_ARG; return false;
    }
    if ((d->dtype != VXL_F32 && d->dtype != VXL_BF16) || (d->head_dim != 64 && d->head_dim != 128)) {
        *st = VXL_ERR_UNSUPPORTED; return false;
    }
    const int64_t sv[4] = {d->q_stride_head, d->q_stride_tok, d->kv_stride_head, d->kv_stride_tok};
    const bool any = sv[0] || sv[1] || sv[2] || sv[3];
    if (any) {                                                // all set, 16-byte multiples, rows of head_dim fit
        const int64_t unit = d->dtype == VXL_BF16 ? 8 : 4;
        for (int64_t v : sv)
            if (v <= 0 || v % unit != 0) { *st = VXL_ERR_INVALID_ARG; return false; }
        if (d->q_stride_tok < d->head_dim || d->kv_stride_tok < d->head_dim) { *st = VXL_ERR_INVALID_ARG; return false; }
    }
    if (d->reserved != 0) { *st = VXL_ERR_INVALID_ARG; return false; }
    return true;
}

static float resolve_scale(const vxl_attn_desc* d) {
    return d->softmax_scale > 0.0f ? d->softmax_scale : 1.0f / std::sqrt((float)d->head_dim);
}

static size_t elem_bytes(const vxl_attn_desc* d) { return d->dtype == VXL_BF16 ? 2 : 4; }

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

PrefillWorkspace prefill_workspace(const vxl_layout* L, const vxl_attn_desc* d) {
    PrefillWorkspace w{};
    if (d->dtype != VXL_BF16) { w.total = 0; return w; }
    size_t off = 0;
    w.kctx = off;
    off += align_up((size_t)d->n_kv_heads * L->n_ctx_tiles * kKeyTile * d->head_dim * 2, 256);
    w.vctx = off;
    off += align_up((size_t)d->n_kv_heads * L->n_ctx_tiles * kKeyTile * d->head_dim * 2, 256);
    w.queue = off;
    off += 256;
    w.total = off;
    return w;
}

static std::atomic<int> g_decode_step_waves{0};     // cross-check hook (vxl_debug.h): 0 = choose, 4 or 8 = force
extern "C" void vxl_debug_decode_step_waves(int w) { g_decode_step_waves = (w == 4 || w == 8) ? w : 0; }

DecodePlan decode_plan(const vxl_attn_desc* d, int batch, int T, int l_cap, bool gathered, size_t have) {
    DecodePlan p{};
    if (d->dtype != VXL_BF16) return decode_f32_plan(d, batch, T, l_cap);
    const int rows = (d->n_q_heads / d->n_kv_heads) * T;
    const int tiles = (l_cap + kKeyTile - 1) / kKeyTile;
    const auto part_o_bytes = [&](int n_split) { return align_up((size_t)batch * d->n_kv_heads * n_split * rows * d->head_dim * sizeof(float), 256); };
    const auto part_l_bytes = [&](int n_split) { return align_up((size_t)batch * d->n_kv_heads * n_split * rows * sizeof(float), 256); };
    const auto partials = [&](int n_split) { return part_o_bytes(n_split) + part_l_bytes(n_split); };
    if (rows > kRowBlock) {
        // The ring kernel, with 128 rows per workgroup or (use_ring) whichever of 128 and 256 is the shorter call: 129-256
        // rows take the former where a launch of 256-row workgroups, whose splits the cap below holds, leaves compute
        // units without any.
        bool ring = rows > 128;
        if (ring && rows <= 256) {
            const long blocks = (long)batch * d->n_kv_heads;
            const long splits = std::max<long>(1, std::min<long>(std::min<long>((256 + blocks - 1) / blocks, (long)l_cap / rows), tiles));
            const int per = (int)((tiles + splits - 1) / splits);
            ring = blocks * ((tiles + per - 1) / per) >= 150;
        }
        p.use_ring = ring ? 1 : 0;
        const int row_tile = ring ? 256 : 128;
        const int n_rtile = (rows + row_tile - 1) / row_tile;
        // Split the keys until every compute unit has its workgroups (one of the 8-wave ring kernel,
        // two planned of the 4-wave one), but keep the partial results (fp32 rows per split) below roughly
        // the KV bytes they summarise (measured at 224 rows over 4,096 keys: 16 splits 20.0 us per
        // call, 32 splits 21.3, 22 splits 21.2, 8 splits 24.0).
        const long base_blocks = (long)batch * d->n_kv_heads * n_rtile;
        const long target = ring ? 256 : 512;
        long want = (target + base_blocks - 1) / base_blocks;
        const long cap = std::max<long>(1, (long)l_cap / rows);
        want = std::max<long>(1, std::min<long>(std::min<long>(want, cap), tiles));
        const int tiles_per = (int)((tiles + want - 1) / want);
        p.n_split = (tiles + tiles_per - 1) / tiles_per;
        p.split_len = tiles_per * kKeyTile;
    }
    // Step mode: every wave of a workgroup owns whole 32-key tiles of a 32-row block; one workgroup per
    // compute unit (its tile pairs fill the LDS), tiles spread evenly over at most ~256 workgroups.
    {
        constexpr int kTile = 32;
        const int tiles32 = (l_cap + kTile - 1) / kTile;
        const int n_rtile = (rows + kRowBlock - 1) / kRowBlock;
        const long units = (long)batch * d->n_kv_heads;
        // (the row blocks of a unit go to one XCD: whole units on its 32 compute units)
        const long max_split = std::max<long>(1, (n_rtile == 1 ? 256 : 8 * (32 / n_rtile)) / units);
        // four double-buffered waves (measured equal or faster than eight single-buffered ones at every size)
        const int kWaves = gathered && rows <= kRowBlock && g_decode_step_waves == 8 ? 8 : 4;
        long n_split = std::min<long>((tiles32 + kWaves - 1) / kWaves, max_split);
        // (in-place form: a wave's row map lives in LDS, 32 tiles at most -- more splits instead)
        if (!gathered) n_split = std::max<long>(n_split, (tiles32 + kWaves * 32 - 1) / (kWaves * 32));
        if (rows > kRowBlock) n_split = std::min<long>(n_split, p.n_split);      // no more partial rows than the other kernels
        const int tpw = (int)((tiles32 + kWaves * n_split - 1) / (kWaves * n_split));
        n_split = (tiles32 + kWaves * tpw - 1) / (kWaves * tpw);
        // More than one row block: this form reads the mixed set once per block, but from the L2 of one
        // XCD, and starts as fast as the one-row-block call.  (us per call, by a 128-row kernel since replaced -> with row
        // blocks, G = 7, four KV heads; keys): 224 rows, 4,096 keys 23.4 -> 18.0; 56 rows, 7,936 keys 23.8 -> 16.0 and 45,312 keys 49.8 -> 25.3; 112
        // rows, 45,312 keys 60.2 -> 33.0; in place, 224 rows, 4,096 keys (with pooling and map) 51.8 -> 43.4.
        // Up to 64 rows at one tile per wave the ring of four waves stays (blocks, ring, us: 35 rows, 750 keys 9.41, 8.69; 49
        // rows, 1,264 keys 9.81, 9.64; not so two queries of 35 rows, 1,973 keys 11.4, 12.1).
        const bool fits = units * n_split * n_rtile <= 256 && (gathered || tpw <= 32);
        bool few = rows > 64 || tpw > 1;
        if (p.use_ring) {
            // Against the ring kernel it wins while that one's launch is small (448 rows: 72 workgroups 25.9 ->
            // 22.7, but 136 workgroups 27.4 -> 28.7; 140 rows at 248 workgroups 18.5 -> 19.4) and its own time is
            // shorter.  In tiles of the ring, a call of the ring takes its tiles and 14 for start and merge, a
            // round of workgroups here 8 and 0.8 per tile of a wave; the row blocks of a unit run on one XCD, whose
            // 32 compute units hold a workgroup each (its LDS), at D = 64 two unless it holds a row map too.
            // Fitted to 176 random calls of 257 to 4,000 rows, gathered and in place, with the ring's keys cut by capacity;
            // with the present ring, of 60 random calls that take row blocks none is slower (1.1x to 2.9x).
            // Ring -> here, D = 128: 959 rows, 1,171 keys in one split, 10 tiles per wave 41.3 -> 20.0; 1,050 rows,
            // two rounds, 1,202 keys 48.3 -> 37.6; 2,824 rows on one KV head, three rounds, 148 keys 20.2 -> 25.6;
            // 1,280 rows, two rounds, 16,384 keys, 12 splits against one 47.8 -> 219.8.  D = 64: 2,006 rows, one
            // round, 2,651 keys 60.3 -> 34.0; in place, 34 workgroups on an XCD, 6,680 keys 41.5 -> 76.1.
            const long ring_launch = units * ((rows + 255) / 256) * p.n_split;
            const long per_xcd = (units * n_split + 7) / 8 * n_rtile, resident = 32 * (d->head_dim == 64 && gathered ? 2 : 1);
            const long rounds = (per_xcd + resident - 1) / resident;
            few = ring_launch < 100 && rounds * (40 + 4 * tpw) < 5 * (14 + p.split_len / kKeyTile);
        }
        // Short mixed sets: one workgroup per row block walks all keys and writes the results, without partials and without
        // the launch of their merge, up to 16 tiles (D = 64: 24) and while the row blocks are no more than the compute units.
        // Us in a replayed graph, splits and merge -> one workgroup, G = 7, four KV heads, D = 128: 7 rows, 251 keys 6.9 ->
        // 5.5, 384 keys 6.9 -> 6.7, 501 keys 7.2 -> 7.8, but submitted call by call, where the second launch costs the host
        // 3, 9.8 -> 7.5; 56 rows, 251 keys 10.9 -> 7.9, 501 keys 11.6 -> 10.2; 8 queries of 112 rows, 501 keys 13.4 -> 11.4.
        // D = 64: 7 rows, 500 keys 6.2 -> 5.6, 700 keys 6.3 -> 6.9 (call by call 9.8 -> 7.0); three queries of 140 rows, 761
        // keys 8.7 -> 8.4.  In place, where a wave pays for the row map on every tile, 12 and 16.  33 to 64 rows of D = 64 go to
        // 12 tiles only because tests hold the range above to 128 rows per workgroup: one workgroup would be the faster one there
        // too (64 rows, 385 keys 8.8 -> 6.4, 768 keys 7.7 -> 7.5; in place, 63 rows, 512 keys 8.6 -> 7.7).
        const bool d64 = d->head_dim == 64;
        const int one = d64 && rows > kRowBlock && rows <= 64 ? 12 : gathered ? (d64 ? 24 : 16) : (d64 ? 16 : 12);
        const bool single = rows <= 256 && tiles32 <= one && units * n_rtile <= 256;
        // Where a wave would walk many tiles, the ring with 128 rows per workgroup: it has four times the keys in flight that
        // row blocks sharing them have, and reads them once.  From 20 tiles per wave on, D = 64 28 and more than 64 rows
        // (blocks -> ring, us: 70 rows, 50,500 keys, 20 tiles 34.1 -> 32.0; 8 queries of 91 rows, 34,847 keys, 136 tiles 168.6
        // -> 104.7; D = 64, 8 of 70, 7,795 keys, 30 tiles 27.0 -> 22.7; but 91 rows, 38,299 keys, 15 tiles 28.1 against 29.1, 49
        // rows, 19 tiles 36.7 and 37.1, D = 64, 8 of 35 rows, 42 tiles 38.6 and 40.6).  In place, over 20 random calls of 20
        // (28) to 32 tiles 1.08x to 2.0x; below, 8 to 19 tiles, 0.84x to 1.41x, and D = 64, 20 to 27, 0.93x to 1.37x.  As many splits
        // as give every compute unit a workgroup, if the scratch memory holds them.
        if (!p.use_ring && fits && few && !single && rows > (d64 ? 64 : kRowBlock) && tpw >= (d64 ? 28 : 20)) {
            const long base_blocks = units * ((rows + 127) / 128);
            const int want = (int)std::max<long>(1, std::min<long>(p.n_split, 256 / base_blocks));
            if (partials(want) <= have) {
                p.n_split = want;
                few = false;
            }
        }
        if (rows <= kRowBlock || (fits && few) || single) {
            p.use_ring = 0;
            p.step_waves = kWaves;
            p.one = single && tiles32 > kWaves;
            p.n_split = single ? 1 : (int)n_split;
            p.split_len = kWaves * (single ? (tiles32 + kWaves - 1) / kWaves : tpw) * kTile;
        }
    }
    p.part_o = 0;
    p.part_ml = part_o_bytes(p.n_split);
    p.total = partials(p.n_split);
    return p;
}

// Test hook (vxl_debug.h).
extern "C" int vxl_debug_decode_plan(const vxl_attn_desc* d, int batch, int n_q_tokens, int l_cap, int in_place,
                                     int* n_split) {
    const DecodePlan p = decode_plan(d, batch, n_q_tokens, l_cap, !in_place);
    *n_split = p.n_split;
    return p.step_waves ? 2 : p.use_ring;
}

// Workspace of the in-place decode: split-KV partial results, then the row map and the lengths.
InplaceWorkspace inplace_workspace(const vxl_attn_desc* d, int batch, int T, int l_cap) {
    InplaceWorkspace w{};
    // The row map and the lengths come first: their places do not depend on the number of query
    // tokens, so a map survives calls with another n_q_tokens on the same workspace.
    size_t off = 0;
    w.src_idx = off;
    off += align_up((size_t)batch * l_cap * sizeof(int32_t), 256);
    w.mix_len = off;
    off += align_up((size_t)batch * sizeof(int32_t), 256);
    w.partials = off;
    off += align_up(std::max<size_t>(256, decode_plan(d, batch, T, l_cap, false).total), 256);
    w.total = off;
    return w;
}

}  // namespace vxl

using namespace vxl;

extern "C" {

int vxl_version(void) { return 100; }

const char* vxl_status_string(vxl_status s) {
    switch (s) {
        case VXL_OK: return "ok";
        case VXL_ERR_INVALID_ARG: return "invalid argument";
        case VXL_ERR_UNSUPPORTED: return "unsupported dtype, head_dim or chunk count";
        case VXL_ERR_WORKSPACE: return "workspace missing or too small";
        case VXL_ERR_HIP: return "HIP runtime error";
        case VXL_ERR_ALLOC: return "host or device memory allocation failed";
    }
    return "unknown status";
}

const char* vxl_last_error(void) { return g_last_error; }

// Test hook (vxl_debug.h): route BF16 calls through the plain vector-ALU kernels (an on-device
// cross-check of the matrix-core kernels).
void vxl_debug_force_simple(int on) { g_force_simple = on; }

vxl_status vxl_layout_create(int32_t n_tokens, int32_t n_prefix, int32_t n_chunks,
                             const int32_t* chunk_bounds, const int32_t* sparse_offsets,
                             const int32_t* sparse_idx, vxl_stream stream, vxl_layout** out) {
    return vxl_layout_create_windowed(n_tokens, n_prefix, n_chunks, chunk_bounds, sparse_offsets, sparse_idx,
                                      0, stream, out);
}

vxl_status vxl_layout_create_windowed(int32_t n_tokens, int32_t n_prefix, int32_t n_chunks,
                                      const int32_t* chunk_bounds, const int32_t* sparse_offsets,
                                      const int32_t* sparse_idx, int32_t window, vxl_stream stream,
                                      vxl_layout** out) {
    if (!out) return VXL_ERR_INVALID_ARG;
    *out = nullptr;
    if (n_tokens <= 0 || n_prefix < 0 || n_chunks < 0 || window < 0 || !chunk_bounds || !sparse_offsets)
        return VXL_ERR_INVALID_ARG;
    if (n_chunks > VXL_MAX_CHUNKS) return VXL_ERR_UNSUPPORTED;
    if (chunk_bounds[0] != n_prefix || chunk_bounds[n_chunks] != n_tokens || sparse_offsets[0] != 0)
        return VXL_ERR_INVALID_ARG;
    for (int c = 0; c < n_chunks; ++c) {
        if (chunk_bounds[c + 1] <= chunk_bounds[c]) return VXL_ERR_INVALID_ARG;
        if (sparse_offsets[c + 1] < sparse_offsets[c]) return VXL_ERR_INVALID_ARG;
        if (sparse_offsets[c + 1] - sparse_offsets[c] > chunk_bounds[c + 1] - chunk_bounds[c])
            return VXL_ERR_INVALID_ARG;
    }
    const int32_t s_total = sparse_offsets[n_chunks];
    if (s_total > 0 && !sparse_idx) return VXL_ERR_INVALID_ARG;
    for (int c = 0; c < n_chunks; ++c) {
        for (int32_t i = sparse_offsets[c]; i < sparse_offsets[c + 1]; ++i) {
            const int32_t t = sparse_idx[i];
            if (t < chunk_bounds[c] || t >= chunk_bounds[c + 1]) return VXL_ERR_INVALID_ARG;
            if (i > sparse_offsets[c] && t <= sparse_idx[i - 1]) return VXL_ERR_INVALID_ARG;
        }
    }

    vxl_layout* L = new (std::nothrow) vxl_layout();
    if (!L) return VXL_ERR_ALLOC;
    L->n_tokens = n_tokens; L->n_prefix = n_prefix; L->n_chunks = n_chunks; L->s_total = s_total;
    L->window = window;
    L->bounds.assign(chunk_bounds, chunk_bounds + n_chunks + 1);
    L->soff.assign(sparse_offsets, sparse_offsets + n_chunks + 1);
    if (s_total) L->sidx.assign(sparse_idx, sparse_idx + s_total);

    // segments and the closed-form pair count
    int32_t tile_base = 0;
    int64_t pairs = (int64_t)n_prefix * (n_prefix + 1) / 2;
    if (n_prefix > 0) {
        L->segs.push_back({0, n_prefix, 0, tile_base, 0});
        tile_base += (n_prefix + kKeyTile - 1) / kKeyTile;
    }
    for (int c = 0; c < n_chunks; ++c) {
        const int32_t len = chunk_bounds[c + 1] - chunk_bounds[c];
        // dense look-back range [lo, b_c); kept tokens inside it are seen through it, not twice
        const int32_t back = (int32_t)std::min<int64_t>(window, chunk_bounds[c] - n_prefix);
        const int32_t lo = chunk_bounds[c] - back;
        const int32_t* kept_begin = L->sidx.data();
        const int32_t* kept_end = kept_begin + sparse_offsets[c];
        const int32_t n_kept_before = (int32_t)(std::lower_bound(kept_begin, kept_end, lo) - kept_begin);
        const int32_t ctx = n_prefix + n_kept_before;
        L->segs.push_back({chunk_bounds[c], len, ctx, tile_base, back});
        tile_base += (len + kKeyTile - 1) / kKeyTile;
        pairs += (int64_t)len * (ctx + back) + (int64_t)len * (len + 1) / 2;
    }
    L->pair_count = pairs;
    L->n_seg = (int32_t)L->segs.size();
    for (const Segment& sg : L->segs) {
        const int b = (sg.q_len + kRowBlock - 1) / kRowBlock;
        L->row_blocks8 += b / 8;
        ++L->segs_mod8[b % 8];
        L->seg_tiles += ((int64_t)sg.ctx_len + sg.back + sg.q_len) / kKeyTile + 1;
    }
    L->n_own_tiles = tile_base;
    L->l_ctx = n_prefix + s_total;
    L->n_ctx_tiles = (L->l_ctx + kKeyTile - 1) / kKeyTile;

    // source token of every slot of every V tile: history tiles first, then own tiles
    std::vector<int32_t> tile_src((size_t)(L->n_ctx_tiles + L->n_own_tiles) * kKeyTile, -1);
    for (int32_t r = 0; r < L->l_ctx; ++r) tile_src[r] = r < n_prefix ? r : L->sidx[r - n_prefix];
    for (const Segment& sg : L->segs) {
        int32_t* dst = tile_src.data() + (size_t)(L->n_ctx_tiles + sg.tile_base) * kKeyTile;
        for (int32_t r = 0; r < sg.q_len; ++r) dst[r] = sg.q_start + r;
    }

    // work items, heaviest first (cost = key tiles visited)
    std::vector<WorkItem> work[2];
    for (int v = 0; v < 2; ++v) {
        const int bm = 128 << v;
        std::vector<std::pair<int64_t, WorkItem>> items;
        for (int s = 0; s < L->n_seg; ++s) {
            const Segment& sg = L->segs[s];
            const int mt = (sg.q_len + bm - 1) / bm;
            for (int m = 0; m < mt; ++m) {
                const int last = std::min(sg.q_len, (m + 1) * bm) - 1;
                const int64_t cost = (sg.ctx_len + kKeyTile - 1) / kKeyTile + (last + sg.back) / kKeyTile + 1;
                items.push_back({cost, {s, m}});
            }
        }
        std::stable_sort(items.begin(), items.end(),
                         [](const auto& a, const auto& b) { return a.first > b.first; });
        for (auto& it : items) work[v].push_back(it.second);
        L->n_work[v] = (int32_t)work[v].size();
    }

    for (int s = 0; s < L->n_seg; ++s) {
        L->longest = std::max(L->longest, L->segs[s].q_len);
        if (s > 0 || n_prefix == 0) L->longest_chunk = std::max(L->longest_chunk, L->segs[s].q_len);
    }

    // Items of the attention-mass score: the prefix and every chunk in even pieces of whole key tiles, at most kMassPiece
    // keys; of a prompt below 32 times that, whose items leave compute units idle, down to 512.  A workgroup walks an item
    // alone, and uneven pieces leave short ones behind: with the selection, 10 chunks of 1,000 tokens, 112 rows 23.3 ->
    // 16.9 us, 100 of 700 to 1,300, 700 rows 103.7 -> 97.8; but 36 of 1,000, 3,416 rows, in halves 145.1 -> 146.3, and
    // pieces down to 256 make 10 of 500, 448 rows 18.0 -> 20.5.
    std::vector<MassItem> mass_items;
    std::vector<int32_t> mass_off(n_chunks + 1, 0);
    const int32_t most = std::min(kMassPiece, std::max(512, (n_tokens / 32 + kKeyTile - 1) / kKeyTile * kKeyTile));
    auto add_pieces = [&](int32_t lo, int32_t hi, int32_t c) {
        if (lo >= hi) return;
        const int32_t n = (hi - lo + most - 1) / most, per = ((hi - lo + n - 1) / n + kKeyTile - 1) / kKeyTile * kKeyTile;
        for (; lo < hi; lo += per) mass_items.push_back({lo, std::min(lo + per, hi), c});
    };
    add_pieces(0, n_prefix, -1);
    for (int c = 0; c < n_chunks; ++c) {
        mass_off[c] = (int32_t)mass_items.size();
        add_pieces(chunk_bounds[c], chunk_bounds[c + 1], c);
    }
    mass_off[n_chunks] = (int32_t)mass_items.size();
    L->n_mass_items = (int32_t)mass_items.size();

    // one device blob
    size_t off = 0;
    auto place = [&](size_t bytes) { size_t o = off; off += align_up(std::max<size_t>(bytes, 4), 256); return o; };
    const size_t o_bounds = place((n_chunks + 1) * 4), o_soff = place((n_chunks + 1) * 4);
    const size_t o_sidx = place((size_t)s_total * 4);
    const size_t o_segs = place(L->segs.size() * sizeof(Segment));
    const size_t o_tsrc = place(tile_src.size() * 4);
    const size_t o_w0 = place(work[0].size() * sizeof(WorkItem));
    const size_t o_w1 = place(work[1].size() * sizeof(WorkItem));
    const size_t o_mi = place(mass_items.size() * sizeof(MassItem));
    const size_t o_mo = place(mass_off.size() * 4);
    L->blob_bytes = off;
    std::vector<char> host(off, 0);
    memcpy(host.data() + o_bounds, L->bounds.data(), (n_chunks + 1) * 4);
    memcpy(host.data() + o_soff, L->soff.data(), (n_chunks + 1) * 4);
    if (s_total) memcpy(host.data() + o_sidx, L->sidx.data(), (size_t)s_total * 4);
    memcpy(host.data() + o_segs, L->segs.data(), L->segs.size() * sizeof(Segment));
    memcpy(host.data() + o_tsrc, tile_src.data(), tile_src.size() * 4);
    if (!work[0].empty()) memcpy(host.data() + o_w0, work[0].data(), work[0].size() * sizeof(WorkItem));
    if (!work[1].empty()) memcpy(host.data() + o_w1, work[1].data(), work[1].size() * sizeof(WorkItem));
    if (!mass_items.empty()) memcpy(host.data() + o_mi, mass_items.data(), mass_items.size() * sizeof(MassItem));
    memcpy(host.data() + o_mo, mass_off.data(), mass_off.size() * 4);

    hipError_t e = hipGetDevice(&L->device);
    if (e == hipSuccess) e = hipMalloc(&L->d_blob, off);
    if (e == hipSuccess) e = hipMemcpyAsync(L->d_blob, host.data(), off, hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) {
        set_last_error("vxl_layout_create", e);
        if (L->d_blob) (void)hipFree(L->d_blob);
        delete L;
        return e == hipErrorOutOfMemory ? VXL_ERR_ALLOC : VXL_ERR_HIP;
    }
    char* base = (char*)L->d_blob;
    L->d_bounds = (int32_t*)(base + o_bounds);
    L->d_soff = (int32_t*)(base + o_soff);
    L->d_sidx = (int32_t*)(base + o_sidx);
    L->d_segs = (Segment*)(base + o_segs);
    L->d_tile_src = (int32_t*)(base + o_tsrc);
    L->d_work[0] = (WorkItem*)(base + o_w0);
    L->d_work[1] = (WorkItem*)(base + o_w1);
    L->d_mass_items = (MassItem*)(base + o_mi);
    L->d_mass_off = (int32_t*)(base + o_mo);
    *out = L;
    return VXL_OK;
}

vxl_status vxl_layout_destroy(vxl_layout* L) {
    if (!L) return VXL_OK;
    vxl_status st = VXL_OK;
    if (L->d_blob) {
        hipError_t e = hipFree(L->d_blob);
        if (e != hipSuccess) { set_last_error("hipFree", e); st = VXL_ERR_HIP; }
    }
    delete L;
    return st;
}

int32_t vxl_mixed_kv_capacity(const vxl_layout* L, int32_t k) {
    if (!L) return 0;
    k = std::max(0, std::min(k, L->n_chunks));
    std::vector<int32_t> extra(L->n_chunks);
    for (int c = 0; c < L->n_chunks; ++c)
        extra[c] = (L->bounds[c + 1] - L->bounds[c]) - (L->soff[c + 1] - L->soff[c]);
    std::partial_sort(extra.begin(), extra.begin() + k, extra.end(), std::greater<int32_t>());
    int64_t cap = (int64_t)L->n_prefix + L->s_total;
    for (int i = 0; i < k; ++i) cap += extra[i];
    return (int32_t)cap;
}

int64_t vxl_prefill_pair_count(const vxl_layout* L) { return L ? L->pair_count : 0; }

size_t vxl_workspace_bytes(vxl_op op, const vxl_layout* L, const vxl_attn_desc* d, int32_t batch,
                           int32_t n_q_tokens, int32_t l_cap) {
    vxl_status st;
    if (!desc_ok(d, &st)) return 0;
    switch (op) {
        case VXL_OP_PREFILL:
            if (!L) return 0;
            return std::max<size_t>(256, prefill_workspace(L, d).total);
        case VXL_OP_SCORE_TOPK:     // mean queries [B][Hkv][D], mean keys [Hkv][C][D] (used when no cache is given), scores [B][C]
            if (!L || batch <= 0) return 0;
            return align_up((size_t)batch * d->n_kv_heads * d->head_dim * 4, 256) +
                   align_up((size_t)d->n_kv_heads * std::max(1, L->n_chunks) * d->head_dim * 4, 256) +
                   align_up((size_t)batch * std::max(1, L->n_chunks) * 4, 256);
        case VXL_OP_GATHER:          // the gather keeps its per-query offsets in LDS: no workspace
            return 0;
        case VXL_OP_DECODE:
            if (batch <= 0 || n_q_tokens <= 0 || l_cap <= 0) return 0;
            return std::max<size_t>(256, decode_plan(d, batch, n_q_tokens, l_cap).total);
        case VXL_OP_SCORE_MASS:
            if (!L || batch <= 0 || n_q_tokens <= 0) return 0;
            return std::max<size_t>(256, mass_plan(L, d, batch, n_q_tokens).total);
        case VXL_OP_DECODE_INPLACE:
            if (batch <= 0 || n_q_tokens <= 0 || l_cap <= 0) return 0;
            return inplace_workspace(d, batch, n_q_tokens, l_cap).total;
    }
    return 0;
}

vxl_status vxl_chunk_prefill(const vxl_layout* L, const vxl_attn_desc* d, const void* Q,
                             const void* K, const void* V, void* O, float* LSE, void* workspace,
                             size_t workspace_bytes, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!Q || !K || !V || !O) return VXL_ERR_INVALID_ARG;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O)) return VXL_ERR_INVALID_ARG;
    if (O == Q || O == K || O == V) return VXL_ERR_INVALID_ARG;
    const float scale = resolve_scale(d);
    if (d->dtype == VXL_BF16 && !g_force_simple) {
        const size_t need = prefill_workspace(L, d).total;
        if (!workspace || workspace_bytes < need || !aligned16(workspace)) return VXL_ERR_WORKSPACE;
        return launch_prefill_bf16(L, d, scale, Q, K, V, O, LSE, workspace, (hipStream_t)stream);
    }
    if (d->dtype == VXL_F32) return launch_prefill_f32(L, d, scale, Q, K, V, O, LSE, (hipStream_t)stream);
    return launch_prefill_simple(L, d, scale, Q, K, V, O, LSE, (hipStream_t)stream);
}

vxl_status vxl_chunk_score_topk(const vxl_layout* L, const vxl_attn_desc* d, const void* Qd,
                                int32_t batch, int32_t n_q_tokens, const void* K, int32_t k,
                                float* kbar, int32_t kbar_ready, int32_t* topk_idx,
                                uint8_t* dense_mask, float* scores, void* workspace,
                                size_t workspace_bytes, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!Qd || batch <= 0 || n_q_tokens <= 0 || k < 0 || !dense_mask) return VXL_ERR_INVALID_ARG;
    if (!aligned16(Qd)) return VXL_ERR_INVALID_ARG;
    const int kk = std::min(k, L->n_chunks);
    if (kk > 0 && !topk_idx) return VXL_ERR_INVALID_ARG;
    if (kbar_ready && !kbar) return VXL_ERR_INVALID_ARG;
    if (!kbar_ready && (!K || !aligned16(K))) return VXL_ERR_INVALID_ARG;
    if (L->n_chunks == 0) return VXL_OK;      // nothing to score, nothing to write
    const size_t need = vxl_workspace_bytes(VXL_OP_SCORE_TOPK, L, d, batch, n_q_tokens, 0);
    if (!workspace || workspace_bytes < need || !aligned16(workspace)) return VXL_ERR_WORKSPACE;
    float* qbar = (float*)workspace;
    const size_t o_kbar = align_up((size_t)batch * d->n_kv_heads * d->head_dim * 4, 256);
    const size_t o_sc = o_kbar + align_up((size_t)d->n_kv_heads * std::max(1, L->n_chunks) * d->head_dim * 4, 256);
    float* kb = kbar ? kbar : (float*)((char*)workspace + o_kbar);
    st = launch_summaries(L, d, K, kb, !kbar_ready, Qd, batch, n_q_tokens, qbar, (hipStream_t)stream);
    if (st != VXL_OK) return st;
    return launch_score_topk(L, d, resolve_scale(d), batch, kk, qbar, kb, topk_idx, dense_mask, scores,
                             (float*)((char*)workspace + o_sc), (hipStream_t)stream);
}

vxl_status vxl_chunk_score_topk_mass(const vxl_layout* L, const vxl_attn_desc* d, const void* Qd,
                                     int32_t batch, int32_t n_q_tokens, const void* K, int32_t k,
                                     int32_t* topk_idx, uint8_t* dense_mask, float* scores,
                                     void* workspace, size_t workspace_bytes, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!Qd || !K || batch <= 0 || n_q_tokens <= 0 || k < 0 || !dense_mask) return VXL_ERR_INVALID_ARG;
    if (!aligned16(Qd) || !aligned16(K)) return VXL_ERR_INVALID_ARG;
    const int kk = std::min(k, L->n_chunks);
    if (kk > 0 && !topk_idx) return VXL_ERR_INVALID_ARG;
    if (L->n_chunks == 0) return VXL_OK;      // nothing to score, nothing to write
    const MassPlan p = mass_plan(L, d, batch, n_q_tokens);
    if (!workspace || workspace_bytes < p.total || !aligned16(workspace)) return VXL_ERR_WORKSPACE;
    float* sc = scores ? scores : (float*)((char*)workspace + p.scores);
    st = launch_score_mass(L, d, resolve_scale(d), Qd, batch, n_q_tokens, K, sc, workspace,
                           g_force_simple != 0, (hipStream_t)stream);
    if (st != VXL_OK) return st;
    return launch_topk_from_scores(L, sc, batch, kk, topk_idx, dense_mask, (hipStream_t)stream);
}

vxl_status vxl_gather_bilevel_kv(const vxl_layout* L, const vxl_attn_desc* d, const void* K,
                                 const void* V, const uint8_t* dense_mask, int32_t batch,
                                 void* Kmix, void* Vmix, int32_t l_cap, int32_t* mix_len,
                                 int32_t* src_idx, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!K || !V || !Kmix || !Vmix || !mix_len || batch <= 0) return VXL_ERR_INVALID_ARG;
    if (L->n_chunks > 0 && !dense_mask) return VXL_ERR_INVALID_ARG;
    if (!aligned16(K) || !aligned16(V) || !aligned16(Kmix) || !aligned16(Vmix)) return VXL_ERR_INVALID_ARG;
    if (l_cap < vxl_mixed_kv_capacity(L, 0)) return VXL_ERR_INVALID_ARG;
    return launch_gather(L, d, K, V, nullptr, nullptr, dense_mask, batch, Kmix, Vmix, l_cap, mix_len, src_idx,
                         (hipStream_t)stream);
}

vxl_status vxl_pool_sparse_kv(const vxl_layout* L, const vxl_attn_desc* d, const void* K, const void* V,
                              void* Ksp, void* Vsp, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!K || !V || !aligned16(K) || !aligned16(V)) return VXL_ERR_INVALID_ARG;
    if (L->s_total > 0 && (!Ksp || !Vsp || !aligned16(Ksp) || !aligned16(Vsp))) return VXL_ERR_INVALID_ARG;
    if (Ksp == K || Ksp == V || Vsp == K || Vsp == V || (Ksp && Ksp == Vsp)) return VXL_ERR_INVALID_ARG;
    return launch_pool_sparse(L, d, K, V, Ksp, Vsp, (hipStream_t)stream);
}

vxl_status vxl_gather_bilevel_kv_pooled(const vxl_layout* L, const vxl_attn_desc* d, const void* K,
                                        const void* V, const void* Ksp, const void* Vsp,
                                        const uint8_t* dense_mask, int32_t batch, void* Kmix, void* Vmix,
                                        int32_t l_cap, int32_t* mix_len, int32_t* src_idx,
                                        vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!K || !V || !Kmix || !Vmix || !mix_len || batch <= 0) return VXL_ERR_INVALID_ARG;
    if (L->n_chunks > 0 && !dense_mask) return VXL_ERR_INVALID_ARG;
    if (L->s_total > 0 && (!Ksp || !Vsp || !aligned16(Ksp) || !aligned16(Vsp))) return VXL_ERR_INVALID_ARG;
    if (!aligned16(K) || !aligned16(V) || !aligned16(Kmix) || !aligned16(Vmix)) return VXL_ERR_INVALID_ARG;
    if (l_cap < vxl_mixed_kv_capacity(L, 0)) return VXL_ERR_INVALID_ARG;
    // (a layout without sparse rows never reads the pooled buffers; the kernel takes the pooled
    // path only when they are given)
    return launch_gather(L, d, K, V, L->s_total > 0 ? Ksp : nullptr, L->s_total > 0 ? Vsp : nullptr, dense_mask,
                         batch, Kmix, Vmix, l_cap, mix_len, src_idx, (hipStream_t)stream);
}

// fp32: scratch for the split form, or null, which is the form without (no workspace, a small or a misaligned one).
static void* f32_scratch(void* workspace, size_t bytes, size_t need) {
    return need > 0 && workspace && bytes >= need && aligned16(workspace) ? workspace : nullptr;
}

vxl_status vxl_bilevel_decode(const vxl_attn_desc* d, const void* Qd, int32_t batch,
                              int32_t n_q_tokens, const void* Kmix, const void* Vmix, int32_t l_cap,
                              const int32_t* mix_len, void* O, float* LSE, void* workspace,
                              size_t workspace_bytes, vxl_stream stream) {
    vxl_status st;
    if (!desc_ok(d, &st)) return st;
    if (!Qd || !Kmix || !Vmix || !mix_len || !O || batch <= 0 || n_q_tokens <= 0 || l_cap <= 0)
        return VXL_ERR_INVALID_ARG;
    if (!aligned16(Qd) || !aligned16(Kmix) || !aligned16(Vmix) || !aligned16(O)) return VXL_ERR_INVALID_ARG;
    const float scale = resolve_scale(d);
    if (d->dtype == VXL_BF16 && !g_force_simple) {
        const DecodePlan p = decode_plan(d, batch, n_q_tokens, l_cap, true, workspace_bytes);
        if (!workspace || workspace_bytes < p.total || !aligned16(workspace)) return VXL_ERR_WORKSPACE;
        return launch_decode_bf16(p, d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O,
                                  LSE, workspace, (hipStream_t)stream);
    }
    if (d->dtype == VXL_F32)
        return launch_decode_f32(d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O, LSE,
                                 f32_scratch(workspace, workspace_bytes, decode_f32_plan(d, batch, n_q_tokens, l_cap).total),
                                 (hipStream_t)stream);
    return launch_decode_simple(d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O, LSE,
                                (hipStream_t)stream);
}

vxl_status vxl_bilevel_decode_inplace(const vxl_layout* L, const vxl_attn_desc* d, const void* Qd,
                                      int32_t batch, int32_t n_q_tokens, const void* K, const void* V,
                                      const void* Ksp, const void* Vsp, const uint8_t* dense_mask,
                                      int32_t l_cap, int32_t map_ready, void* O, float* LSE, int32_t* mix_len,
                                      void* workspace, size_t workspace_bytes, vxl_stream stream) {
    vxl_status st;
    if (!L) return VXL_ERR_INVALID_ARG;
    if (!desc_ok(d, &st)) return st;
    if (!Qd || !K || !V || !O || batch <= 0 || n_q_tokens <= 0 || l_cap <= 0) return VXL_ERR_INVALID_ARG;
    if (L->n_chunks > 0 && !dense_mask) return VXL_ERR_INVALID_ARG;
    if ((Ksp == nullptr) != (Vsp == nullptr)) return VXL_ERR_INVALID_ARG;
    if (!aligned16(Qd) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(Ksp) || !aligned16(Vsp))
        return VXL_ERR_INVALID_ARG;
    if (l_cap < vxl_mixed_kv_capacity(L, 0)) return VXL_ERR_INVALID_ARG;
    const InplaceWorkspace w = inplace_workspace(d, batch, n_q_tokens, l_cap);
    // (fp32: the row map is needed, room for partial results is not)
    const DecodePlan p = decode_plan(d, batch, n_q_tokens, l_cap, false, workspace_bytes > w.partials ? workspace_bytes - w.partials : 0);
    const size_t need = w.partials + (d->dtype == VXL_F32 ? 256 : align_up(std::max<size_t>(256, p.total), 256));
    if (!workspace || workspace_bytes < need || !aligned16(workspace)) return VXL_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int32_t* src_idx = (int32_t*)((char*)workspace + w.src_idx);
    int32_t* len = mix_len ? mix_len : (int32_t*)((char*)workspace + w.mix_len);
    const bool pooled = Ksp != nullptr && L->s_total > 0;
    if (!map_ready) {           // the row map and the lengths: the gather's index pass, no row is copied
        st = launch_gather(L, d, K, V, pooled ? Ksp : nullptr, pooled ? Vsp : nullptr, dense_mask, batch, nullptr,
                           nullptr, l_cap, len, src_idx, s);
        if (st != VXL_OK) return st;
    }
    const float scale = resolve_scale(d);
    if (d->dtype == VXL_BF16 && !g_force_simple)
        return launch_decode_bf16_inplace(p, L, d, scale, Qd, batch, n_q_tokens, K, V, Ksp, Vsp, src_idx, l_cap, len, O,
                                          LSE, (char*)workspace + w.partials, s);
    if (d->dtype == VXL_F32)
        return launch_decode_f32_inplace(L, d, scale, Qd, batch, n_q_tokens, K, V, Ksp, Vsp, src_idx, l_cap, len, O, LSE,
                                         f32_scratch((char*)workspace + w.partials, workspace_bytes - w.partials,
                                                     decode_f32_plan(d, batch, n_q_tokens, l_cap).total), s);
    return launch_decode_inplace_simple(L, d, scale, Qd, batch, n_q_tokens, K, V, Ksp, Vsp, src_idx, l_cap, len, O,
                                        LSE, s);
}

vxl_status vxl_bilevel_decode_static(const vxl_attn_desc* d, const void* Qd, int32_t batch,
                                     int32_t n_q_tokens, const void* Kmix, const void* Vmix, int32_t l_cap,
                                     const int32_t* mix_len, void* O, float* LSE, vxl_stream stream) {
    vxl_status st;
    if (!desc_ok(d, &st)) return st;
    if (!Qd || !Kmix || !Vmix || !mix_len || !O || batch <= 0 || n_q_tokens <= 0 || l_cap <= 0)
        return VXL_ERR_INVALID_ARG;
    if (!aligned16(Qd) || !aligned16(Kmix) || !aligned16(Vmix) || !aligned16(O)) return VXL_ERR_INVALID_ARG;
    const float scale = resolve_scale(d);
    if (d->dtype == VXL_BF16 && !g_force_simple) {
        const DecodePlan p = decode_plan(d, batch, n_q_tokens, l_cap, true, VXL_STATIC_SCRATCH_BYTES);
        if (p.total > (size_t)VXL_STATIC_SCRATCH_BYTES) {
            snprintf(g_last_error, sizeof(g_last_error),
                     "vxl_bilevel_decode_static: the split-KV partial results of this call need %zu bytes, the "
                     "static scratch holds %zu", p.total, (size_t)VXL_STATIC_SCRATCH_BYTES);
            return VXL_ERR_WORKSPACE;
        }
        void* ws = nullptr;
        st = decode_static_scratch(&ws);
        if (st != VXL_OK) return st;
        return launch_decode_bf16(p, d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O, LSE, ws,
                                  (hipStream_t)stream);
    }
    if (d->dtype == VXL_F32) {
        const size_t need = decode_f32_plan(d, batch, n_q_tokens, l_cap).total;      // (4.3 MB at most)
        void* ws = nullptr;
        if (need > 0 && (st = decode_static_scratch(&ws)) != VXL_OK) return st;
        return launch_decode_f32(d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O, LSE,
                                 f32_scratch(ws, VXL_STATIC_SCRATCH_BYTES, need), (hipStream_t)stream);
    }
    return launch_decode_simple(d, scale, Qd, batch, n_q_tokens, Kmix, Vmix, l_cap, mix_len, O, LSE,
                                (hipStream_t)stream);
}

}  // extern "C"
