// All four steps behind one entry point, with steps 1-3 in ONE kernel: a block featurizes a tile of
// flows straight into the shared-memory columns the forest walk reads (Section 3.1 of the paper: the fast
// model sees every flow, from its first k packets) and walks the forest on them; the feature row of a
// flow leaves the chip only if the gate (Section 3.2) hands the flow on to the slow model.
//
// Why: the feature step is bound by vector arithmetic and by its memory pattern, the walk by gathers;
// with several blocks per compute unit one block's feature phase runs under another's walk, and the
// feature matrix (256 bytes per flow written, then read again) is neither written nor read for the
// flows that stay with the fast model.
//
// The block has the walk's shape.  Where several lanes in different waves share a flow (see forest_core.h), the
// statistics are split between the waves too: a flow's 32 statistics of a window are four independent parts
// (ordered sums and order statistics, of sizes and of times), and a wave computes one part of one window for
// its flows.  A part needs one quantity in registers, so the kernel comes down to the 64 registers at which a
// compute unit holds 32 waves (with windows of up to 16 packets 13 to 17 of them are spilled in the feature phase).
// Large batches with few trees, which are the feature phase above all, go one lane per flow.
//
// Shared memory of a block: the tile [32 * windows][flows] floats; behind it, one after the other, the packets
// of the tile's flows as columns (several lanes per flow), the scratch columns of the sorting networks, and what the
// walk needs (vote counters, staged top records).
#include "featurize_core.h"
#include "forest_core.h"
#include "forest_wave.h"
#include "small_batch.h"

namespace sf {
int forest_setup(sf_ctx* ctx, const char* who, const sf_forest* f, uint32_t feat_ld, sfforest::FastArgs& a, uint32_t* result_words);
sfforest::TileShape forest_shape(sfforest::FastArgs& a, uint32_t result_words, uint32_t n_rows, uint32_t n_cu, uint32_t dmax, size_t* lds);
bool slow_gates(sf_ctx* ctx, const float* feat, uint32_t feat_ld, const sf_mlp* mlp, const sfsmall::GateRows& gate, const float* logits,
                const uint16_t* labels); // slow_infer.hip
int slow_infer_gated(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n, const sf_mlp* mlp, const sfsmall::GateRows& gate, const uint16_t* pred,
                     float* logits, uint16_t* labels);
}

namespace {

using namespace sfforest;

constexpr uint32_t kFusedWindows = 2, kFusedDepth = 16; // the most the fused kernel is built for

struct ClassifyArgs {
    uint32_t n_pkts;
    const uint32_t* off;
    const uint16_t* size;
    const float* iat;
    const uint8_t* dir;
    uint32_t n_windows;
    uint32_t depth[kFusedWindows];
    uint32_t wide_ok;  // the packet arrays start on 8-byte (size, time, direction) boundaries
    uint32_t wide16_ok; // sizes and times on 16-byte ones
    FastArgs fa;      // n_flows, model, outputs, gate; n_features = 32 * n_windows
};

// Staged packets of a tile: one column per flow, rows 0..KMAX-1 the sizes, KMAX..2 KMAX-1 the times, then the
// direction bits and the packet count.  Four words of padding per row: the lanes of a wave that write a row pair
// each for eight flows then fall on 64 different banks.
__host__ __device__ constexpr uint32_t stage_stride(uint32_t fpb) { return fpb + 4u; }
__host__ __device__ constexpr uint32_t stage_words(uint32_t kmax, uint32_t fpb) { return (2u * kmax + 2u) * stage_stride(fpb); }
// Groups of lanes that compute statistics side by side: whole waves, also where a tile has fewer than 64 flows
__host__ __device__ constexpr uint32_t feature_units(uint32_t fpb, uint32_t w) { return fpb >= 64u ? w : fpb * w / 64u; }
// every second unit sorts (see below) and has a scratch column of KMAX words per flow
__host__ __device__ constexpr uint32_t scratch_words(uint32_t kmax, uint32_t fpb, uint32_t w) { return feature_units(fpb, w) / 2u * kmax * fpb; }

// One part of one window's statistics for one flow per lane: kind 0 / 2: sums of sizes / times, kind 1 / 3: order
// statistics of sizes / times.  x: the quantity; col: scratch column; dst: the window's first row of the tile.
template <int N, int KMAX>
__device__ __forceinline__ void window_part(uint32_t kind, const float (&x)[KMAX], uint32_t dmask, int m, uint32_t* col, uint32_t fpb,
                                            float* dst)
{
    const uint32_t valid = (1u << m) - 1u, m1 = dmask & valid, m0 = ~dmask & valid; // (m <= 16)
    const int c1 = __popc(m1), c0 = m - c1;
    if ((kind & 1u) == 0u) {
        const float sum = sffeat::window_sums<true, N, KMAX>(x, valid, m0, m1, m, c0, c1, dst + (kind ? 5u : 0u) * fpb, fpb);
        if (kind == 0u) {
            dst[30u * fpb] = sum;
            dst[31u * fpb] = (float)m;
        }
    } else if (kind == 1u) {
        sffeat::window_order_sizes<true, N, KMAX>(x, valid, m1, m, c0, c1, col, fpb, dst + 2u * fpb, fpb);
    } else {
        // a time with its sign bit set anywhere in the wave: the order statistics take the general path
        uint32_t sign_bits = 0;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) sign_bits |= __float_as_uint(x[j]);
        const bool signed_times = __any((int)(sign_bits >> 31));
        sffeat::window_order_times<true, N, KMAX>(x, valid, m0, m1, m, c0, c1, signed_times, col, fpb, dst + 7u * fpb, fpb);
    }
}

// The features of a tile by parts: FPB flows, W >= 4 lanes per flow.
template <int FPB_, int W, int KMAX>
__device__ __forceinline__ void features_by_parts(const ClassifyArgs& c, float* xT, uint32_t* behind)
{
    constexpr uint32_t FPB = FPB_, BS = FPB * W, SS = stage_stride(FPB), UNITS = feature_units(FPB, W);
    constexpr uint32_t P = KMAX / 2; // lanes that fetch one flow's packets, two packets each
    static_assert((FPB * P) % 64u == 0 && (P == 4 || P == 8), "every flow's packets are fetched by lanes of one wave, whole waves take part");
    const FastArgs& a = c.fa;
    const uint32_t tid = threadIdx.x, flow0 = blockIdx.x * FPB;
    for (uint32_t q = tid; q < FPB * P; q += BS) {
        // consecutive lanes hold consecutive packets of a flow and the flows follow each other in memory, so the
        // loads of a wave are one contiguous piece (flows longer than the window leave gaps)
        const uint32_t f = q / P, p = q % P;
        // a slot past the last flow works on the last flow (its loads stay inside the arrays)
        const uint32_t flow = flow0 + f < a.n_flows ? flow0 + f : a.n_flows - 1u;
        uint32_t b = c.off[flow], e = c.off[flow + 1];
        b = b < c.n_pkts ? b : c.n_pkts; // clamp: malformed offsets must not leave the arrays
        e = e < c.n_pkts ? e : c.n_pkts;
        e = e < b ? b : e;
        const uint32_t n = e - b, dmax = c.depth[c.n_windows - 1u], avail = n < dmax ? n : dmax;
        float s[2] = {0.f, 0.f}, t[2] = {0.f, 0.f};
        uint32_t d = 0;
        const uint32_t o = b + 2u * p;
        if (2u * p + 1u < avail && (o & 1u) == 0 && c.wide_ok) {
            const uint32_t sz = *reinterpret_cast<const uint32_t*>(c.size + o);
            const float2 tm = *reinterpret_cast<const float2*>(c.iat + o);
            const uint32_t dd = *reinterpret_cast<const uint16_t*>(c.dir + o);
            s[0] = (float)(sz & 0xFFFFu);
            s[1] = (float)(sz >> 16);
            t[0] = tm.x;
            t[1] = tm.y;
            d = (dd & 1u) | ((dd >> 7) & 2u);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 2u; ++k) {
                if (2u * p + k < avail) {
                    s[k] = (float)c.size[o + k];
                    t[k] = c.iat[o + k];
                    d |= (uint32_t)(c.dir[o + k] & 1u) << k;
                }
            }
        }
        d <<= 2u * p;
#pragma unroll
        for (uint32_t k = 1; k < P; k *= 2) d |= (uint32_t)__shfl_xor((int)d, (int)k, 64);
        float* st = reinterpret_cast<float*>(behind) + f;
#pragma unroll
        for (uint32_t k = 0; k < 2u; ++k) {
            st[(2u * p + k) * SS] = s[k];
            st[(KMAX + 2u * p + k) * SS] = t[k];
        }
        if (p == 0u) {
            behind[2u * KMAX * SS + f] = d;
            behind[(2u * KMAX + 1u) * SS + f] = avail;
        }
    }
    __syncthreads();
    // unit u computes the parts u, u + UNITS, ... of the list (window 0 kinds 0..3, window 1 kinds 0..3)
    static_assert(UNITS == 4 || UNITS == 8, "a unit keeps its kind of part");
    uint32_t unit = FPB >= 64u ? tid / FPB : tid / 64u;
    unit = __builtin_amdgcn_readfirstlane(unit);
    const uint32_t slot = FPB >= 64u ? tid % FPB : tid % 64u;
    const bool has_flow = FPB >= 64u || slot < FPB;
    const uint32_t kind = unit & 3u;
    float x[KMAX];
    uint32_t dmask = 0;
    int avail = 0;
    const bool works = has_flow && (unit >> 2) < c.n_windows;
    if (works) {
        const float* st = reinterpret_cast<const float*>(behind) + slot + (kind >> 1) * KMAX * SS;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) x[j] = st[j * SS];
        dmask = behind[2u * KMAX * SS + slot];
        avail = (int)behind[(2u * KMAX + 1u) * SS + slot];
    }
    __syncthreads(); // the staged packets are in registers: their space is scratch now
    if (works) {
        uint32_t* col = behind + (unit >> 1) * (KMAX * FPB) + slot; // the lane's own column: no two lanes share a word
#pragma unroll 1
        for (uint32_t w = unit >> 2; w < c.n_windows; w += UNITS / 4u) {
            // nothing made from the packets for one part or window is kept for another (registers)
#pragma unroll
            for (int j = 0; j < KMAX; ++j) asm volatile("" : "+v"(x[j]));
            const int dw = (int)c.depth[w];
            const int m = avail < dw ? avail : dw;
            float* dst = xT + (size_t)(32u * w) * FPB + slot;
            // the smallest network that covers every lane's window (wave-uniform choice)
            if (KMAX > 8 && __any(m > 8))
                window_part<KMAX, KMAX>(kind, x, dmask, m, col, FPB, dst);
            else
                window_part<8, KMAX>(kind, x, dmask, m, col, FPB, dst);
        }
    }
}

// The features of a tile of 256 flows, one lane per flow: all statistics of a flow are one lane's serial chain, but its packets
// are fetched straight into registers and a comparison serves all of a window's statistics.
template <int KMAX>
__device__ __forceinline__ void features_by_lanes(const ClassifyArgs& c, float* xT, uint32_t* behind)
{
    constexpr uint32_t FPB = 256;
    const uint32_t tid = threadIdx.x, i = blockIdx.x * FPB + tid;
    // a lane past the last flow works on the last flow (its loads stay inside the arrays)
    const uint32_t flow = i < c.fa.n_flows ? i : c.fa.n_flows - 1u;
    uint32_t o = c.off[flow], e = c.off[flow + 1];
    o = o < c.n_pkts ? o : c.n_pkts; // clamp: malformed offsets must not leave the arrays
    e = e < c.n_pkts ? e : c.n_pkts;
    const uint32_t n = e > o ? e - o : 0u, dmax = c.depth[c.n_windows - 1u];
    const int avail = (int)(n < dmax ? n : dmax);
    float s[KMAX], t[KMAX];
    uint32_t dmask = 0;
    if (avail == KMAX && (o & 7u) == 0 && c.wide16_ok) {
        // whole window present and 16-byte aligned (array bases included): wide loads
        sffeat::RawPackets<KMAX> raw;
        sffeat::load_wide<KMAX>(c.size, c.iat, c.dir, o, raw);
        sffeat::decode_wide<KMAX>(raw, s, t, dmask);
    } else {
        sffeat::load_each<KMAX>(c.size, c.iat, c.dir, o, avail, s, t, dmask);
    }
    // a time with its sign bit set anywhere in the wave: the order statistics take the general path
    uint32_t sign_bits = 0;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) sign_bits |= __float_as_uint(t[j]);
    const bool signed_times = __any((int)(sign_bits >> 31));
    // windows from the last to the first: every one but the first takes the first window's columns (not written yet) as the
    // scratch of its sorting networks, the first the space behind the tile
    for (int w = (int)c.n_windows - 1; w >= 0; --w) {
        const int dw = (int)c.depth[w];
        const int m = avail < dw ? avail : dw;
        // every address below is the lane's own column: no two lanes (or waves) share a word
        uint32_t* col = (w > 0 ? reinterpret_cast<uint32_t*>(xT) : behind) + tid;
        float* dst = xT + (size_t)(32 * w) * FPB + tid;
        // the smallest network that covers every lane's window (wave-uniform choice)
        if (KMAX >= 16 && __any(m > 8))
            sffeat::window_stats<false, KMAX, KMAX>(s, t, dmask, m, signed_times, col, FPB, dst, FPB);
        else
            sffeat::window_stats<false, 8, KMAX>(s, t, dmask, m, signed_times, col, FPB, dst, FPB);
    }
}

// FPB flows per block, W lanes per flow (the walk's shape).
// One wave per 64 flows did all of this before (256 flows per block, one lane per flow).  The kernel, before -> after:
// 1,048,576 flows x 16 packets, windows of 8 and 16, 100 trees of depth 12, a quarter of the rows kept: 572 -> 541 us;
// windows of 5 and 10, depth 10, no rows: 468 -> 385 us; 97 ragged flows: 51 -> 11 us.  What bounds it: the walk's
// gathers (forest_core.h) and about 80 us of vector arithmetic for the statistics.  With a wave to a tree behind the same
// features (forest_wave.h; 128 flows, eight lanes a flow for the statistics): 500 -> 439 us and 367 -> 336.
template <int FPB_, int W, int ILP, int TAIL, int KMAX, bool KEEP_ROWS>
__device__ __forceinline__ void features_then_walk(const ClassifyArgs& c)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const FastArgs& a = c.fa;
    float* xT = reinterpret_cast<float*>(smem_raw); // [32 * windows][flows]
    uint32_t* behind = reinterpret_cast<uint32_t*>(xT + (size_t)a.n_features * FPB_);
    if constexpr (W == 1)
        features_by_lanes<KMAX>(c, xT, behind);
    else
        features_by_parts<FPB_, W, KMAX>(c, xT, behind);
    __syncthreads(); // the space behind the tile is free: the walk may stage its records there
    if constexpr (ILP == 0) { // a wave to a tree
        forest_walk_waves<FPB_ / 64, 4, false, KEEP_ROWS>(a, xT, blockIdx.x * FPB_, a.n_flows);
    } else {
        const uint32_t i = blockIdx.x * FPB_ + threadIdx.x % FPB_;
        forest_walk<FPB_, W, ILP, TAIL, false, false, false, KEEP_ROWS>(a, xT, i, i, i < a.n_flows);
    }
}
template <int FPB_, int W, int ILP, int TAIL, int KMAX, bool KEEP_ROWS>
__global__ __launch_bounds__(FPB_ * W, W == 1 ? 2 : FPB_ == 16 ? 4 : 8) void featurize_forest(ClassifyArgs c)
{
    features_then_walk<FPB_, W, ILP, TAIL, KMAX, KEEP_ROWS>(c);
}
// For batches whose blocks are all resident with more than 64 registers a lane (see launch_fused)
template <int FPB_, int W, int ILP, int TAIL, int KMAX, bool KEEP_ROWS>
__global__ __launch_bounds__(FPB_ * W, FPB_ * W == 1024 ? 4 : 6) void featurize_forest_few(ClassifyArgs c)
{
    features_then_walk<FPB_, W, ILP, TAIL, KMAX, KEEP_ROWS>(c);
}

template <int FPB, int W, int ILP, int TAIL, int KMAX, bool KEEP_ROWS>
int launch_fused(sf_ctx* ctx, const ClassifyArgs& c, size_t lds, int slot)
{
    const size_t parts = stage_words(KMAX, FPB) > scratch_words(KMAX, FPB, W) ? stage_words(KMAX, FPB) : scratch_words(KMAX, FPB, W);
    const size_t behind = W == 1 ? (size_t)(c.depth[0] > 8u ? 16 : 8) * FPB : parts; // (one lane per flow: the first window's network)
    const size_t lds_feat = ((size_t)c.fa.n_features * FPB + behind) * 4;
    if (lds_feat > lds) lds = lds_feat;
    const uint32_t grid = (c.fa.n_flows + FPB - 1u) / FPB;
    auto* kernel = featurize_forest<FPB, W, ILP, TAIL, KMAX, KEEP_ROWS>;
    // Windows up to 16 packets spill 13 to 17 of 64 registers in the feature phase, each a round trip when the blocks are few; 78 to 80 spill
    // none and hold six waves a SIMD (one block of sixteen waves a unit, which has no more).  Before, with 64 -> with them: 16,384 ragged flows,
    // windows 8 and 16, 100 trees of depth 10 16.5 -> 15.3 us, 40 trees 15.2 -> 13.8; 49,152, 100 trees of depth 2 17.1 -> 14.7; 60,000, 40 trees 21.5
    // -> 18.7; 32,768 with a wave to a tree 18.8 -> 17.9.  Past the line the occupancy counts: 65,536, 300 trees of depth 4 37.0 with 64, 39.1 with 80.
    if constexpr (KMAX == 16 && W > 1 && FPB > 16) {
        if (grid <= (uint32_t)ctx->n_cu * (FPB * W == 1024 ? 1u : 3u)) {
            kernel = featurize_forest_few<FPB, W, ILP, TAIL, KMAX, KEEP_ROWS>;
            slot = sf::kLdsClassifyFew + (KEEP_ROWS ? 3 : 0) + (ILP == 0 ? 0 : FPB == 128 ? 1 : 2);
        }
    }
    SF_ALLOW_LDS(ctx, slot, kernel);
    kernel<<<grid, FPB * W, lds, ctx->stream>>>(c);
    SF_LAUNCH_CHECK(ctx, "featurize_forest");
    return SF_OK;
}

template <int KMAX, bool KEEP_ROWS>
int launch_shape(sf_ctx* ctx, const ClassifyArgs& c, TileShape shape, size_t lds, int slot)
{
    switch (shape) {
    case kTile128Waves: return launch_fused<128, 8, 0, 0, KMAX, KEEP_ROWS>(ctx, c, lds, slot);
    case kTile128x4: return launch_fused<128, 4, 5, 2, KMAX, KEEP_ROWS>(ctx, c, lds, slot + 1);
    case kTile64x8: return launch_fused<64, 8, 3, 1, KMAX, KEEP_ROWS>(ctx, c, lds, slot + 2);
    case kTile16x32: return launch_fused<16, 32, 5, 2, KMAX, KEEP_ROWS>(ctx, c, lds, slot + 3);
    default: return launch_fused<256, 1, 10, 5, KMAX, KEEP_ROWS>(ctx, c, lds, slot + 4);
    }
}

// steps 1-3 for both entry points; keep_rows: feature rows of the flows the gate hands on are wanted
int run_features_and_forest(sf_ctx* ctx, const char* who, const sf_packets* pk, const sf_feat_cfg* cfg, const sf_forest* forest,
                            const uint16_t* host_vmin, uint32_t n_vmin, bool keep_rows, float* feat, uint32_t feat_ld,
                            uint16_t* pred, uint16_t* top_votes, uint16_t* labels, bool* labels_done)
{
    if (!pk || !cfg || !forest) return sf::fail(ctx, SF_EINVAL, "%s: packets, config or forest is NULL", who);
    if (!host_vmin || n_vmin < 1 || n_vmin > SF_MAX_CLASSES)
        return sf::fail(ctx, SF_EINVAL, "%s: host_vmin missing or n_vmin %u outside 1..%d", who, n_vmin, SF_MAX_CLASSES);
    if (cfg->n_windows < 1 || cfg->n_windows > SF_MAX_WINDOWS)
        return sf::fail(ctx, SF_EINVAL, "%s: n_windows %u outside 1..%d", who, cfg->n_windows, SF_MAX_WINDOWS);
    for (uint32_t w = 0; w < cfg->n_windows; ++w) {
        if (cfg->depth[w] < 1 || cfg->depth[w] > SF_MAX_DEPTH_PKTS)
            return sf::fail(ctx, SF_EINVAL, "%s: depth[%u] = %u outside 1..%d", who, w, cfg->depth[w], SF_MAX_DEPTH_PKTS);
        if (w && cfg->depth[w] <= cfg->depth[w - 1]) return sf::fail(ctx, SF_EINVAL, "%s: depths must be strictly increasing", who);
    }
    const uint32_t F = 32u * cfg->n_windows;
    if (keep_rows && feat_ld < F) return sf::fail(ctx, SF_EINVAL, "%s: feat_ld %u < %u", who, feat_ld, F);
    if (forest->n_features > F)
        return sf::fail(ctx, SF_EINVAL, "%s: the forest splits on %u features, the windows give %u", who, forest->n_features, F);
    if (pk->n_pkts >> 32) return sf::fail(ctx, SF_EINVAL, "%s: n_pkts exceeds 32-bit offsets", who);
    const uint32_t n = pk->n_flows;
    *labels_done = false;
    if (n == 0) return SF_OK;
    if (!pk->flow_off || !pred || !top_votes || (keep_rows && !feat))
        return sf::fail(ctx, SF_EINVAL, "%s: flow_off, feat, pred or top_votes is NULL", who);
    if (pk->n_pkts && (!pk->pkt_size || !pk->pkt_iat || !pk->pkt_dir)) return sf::fail(ctx, SF_EINVAL, "%s: packet arrays missing", who);

    // the forest with the tile's width (the walk's shared-memory layout follows the tile, not the model)
    sf_forest wide = *forest;
    wide.n_features = F;
    ClassifyArgs c = {};
    uint32_t result_words = 0;
    const uint32_t dmax = cfg->depth[cfg->n_windows - 1];
    int rc = sf::forest_setup(ctx, who, &wide, F, c.fa, &result_words);
    if (rc != SF_OK) return rc;
    // Which calls leave feature rows unwritten is part of the interface (serveflow.h), so it does not follow the block
    // shapes of the present kernel: windows of up to 16 packets, and 80 KB that hold the features and vote counters of 256
    // flows with as many staged pair-levels of records as the budget gives (none, one or more of every tree).
    const size_t first = ((size_t)F + result_words) * 1024 + (size_t)c.fa.n_trees * 16;
    uint32_t staged = 0;
    const bool under_gate_only =
        dmax <= kFusedDepth && plan_lds(c.fa, result_words, 256, first <= 80 * 1024 - 512 ? 80 * 1024 - 512 : 160 * 1024 - 1024, &staged) <= 80 * 1024;
    if (!under_gate_only && (!feat || feat_ld < F)) return sf::fail(ctx, SF_EINVAL, "%s: this shape needs the feature matrix", who);
    // What the fused kernel is built for: at most two windows, and a tile that leaves a unit two blocks of 128 flows.
    if (cfg->n_windows > kFusedWindows || dmax > kFusedDepth || F + result_words > 80u) {
        // other shapes: the same results from the separate kernels, with every feature row written
        rc = sf_featurize(ctx, pk, cfg, feat, feat_ld, nullptr);
        if (rc != SF_OK) return rc;
        return sf_fast_infer(ctx, feat, feat_ld, n, forest, nullptr, pred, top_votes, nullptr);
    }
    if (!under_gate_only) {
        // every row: a threshold above any vote count (the rule gives at most 10,176 trees here)
        static const uint16_t every = 0xFFFFu;
        host_vmin = &every;
        n_vmin = 1;
        keep_rows = true;
    }
    c.n_pkts = (uint32_t)pk->n_pkts;
    c.off = pk->flow_off;
    c.size = pk->pkt_size;
    c.iat = pk->pkt_iat;
    c.dir = pk->pkt_dir;
    c.n_windows = cfg->n_windows;
    for (uint32_t w = 0; w < kFusedWindows; ++w) c.depth[w] = w < cfg->n_windows ? cfg->depth[w] : 0;
    c.wide_ok = (((uintptr_t)c.size | (uintptr_t)c.iat | (uintptr_t)c.dir) & 7u) == 0;
    c.wide16_ok = c.wide_ok && (((uintptr_t)c.size | (uintptr_t)c.iat) & 15u) == 0;
    c.fa.n_flows = n;
    c.fa.n_rows = n;
    c.fa.pred = pred;
    c.fa.top = top_votes;
    c.fa.labels = labels; // the label array starts as the fast prediction (Section 4.4); the slow model overwrites its flows
    *labels_done = labels != nullptr;
    c.fa.feat_out = feat;
    c.fa.feat_out_ld = feat_ld;
    c.fa.feat_out16 = ((uintptr_t)feat & 15u) == 0 && (feat_ld & 3u) == 0;
    c.fa.n_vmin = n_vmin;
    for (uint32_t k = 0; k < SF_MAX_CLASSES; ++k) c.fa.vmin[k] = host_vmin[k < n_vmin ? k : n_vmin - 1];
    size_t lds = 0;
    const TileShape shape = sf::forest_shape(c.fa, result_words, n, (uint32_t)ctx->n_cu, dmax, &lds);
    const int slot = sf::kLdsClassify + (keep_rows ? 10 : 0) + (dmax > 8 ? 5 : 0);
    if (dmax <= 8) return keep_rows ? launch_shape<8, true>(ctx, c, shape, lds, slot) : launch_shape<8, false>(ctx, c, shape, lds, slot);
    return keep_rows ? launch_shape<16, true>(ctx, c, shape, lds, slot) : launch_shape<16, false>(ctx, c, shape, lds, slot);
}

} // namespace

namespace {
// labels = pred for every flow (the separate kernels do not write labels: one small copy)
__global__ __launch_bounds__(256) void labels_from_pred(const uint16_t* __restrict__ pred, uint16_t* __restrict__ labels, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) labels[i] = pred[i];
}
} // namespace

extern "C" int sf_featurize_fast_infer(sf_ctx* ctx, const sf_packets* pk, const sf_feat_cfg* cfg, const sf_forest* forest,
                                       const uint16_t* host_vmin, uint32_t n_vmin, float* feat, uint32_t feat_ld,
                                       uint16_t* pred, uint16_t* top_votes, uint16_t* labels)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_featurize_fast_infer: ctx is NULL");
    bool done = false;
    const int rc = run_features_and_forest(ctx, "sf_featurize_fast_infer", pk, cfg, forest, host_vmin, n_vmin, feat != nullptr, feat,
                                           feat_ld, pred, top_votes, labels, &done);
    if (rc != SF_OK || !labels || done || !pk || pk->n_flows == 0) return rc;
    uint32_t blocks = (pk->n_flows + 255u) / 256u;
    labels_from_pred<<<blocks > 4096u ? 4096u : blocks, 256, 0, ctx->stream>>>(pred, labels, pk->n_flows);
    SF_LAUNCH_CHECK(ctx, "labels_from_pred");
    return SF_OK;
}

extern "C" int sf_classify(sf_ctx* ctx, const sf_packets* pk, const sf_feat_cfg* cfg, const sf_forest* forest,
                           const uint16_t* host_vmin, uint32_t n_vmin, const sf_mlp* mlp, float* feat, uint32_t feat_ld,
                           uint16_t* pred, uint16_t* top_votes, uint32_t* esc_idx, uint32_t* esc_count, float* logits,
                           uint16_t* labels)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_classify: ctx is NULL");
    if (!cfg || !mlp || !pk) return sf::fail(ctx, SF_EINVAL, "sf_classify: packets, config or mlp is NULL");
    if (!esc_count) return sf::fail(ctx, SF_EINVAL, "sf_classify: esc_count is NULL");
    const bool raw = cfg->raw_pkts > 0;
    const uint32_t n = pk->n_flows;
    if (n && (!esc_idx || !labels)) return sf::fail(ctx, SF_EINVAL, "sf_classify: esc_idx or labels is NULL");
    bool labels_done = false;
    int rc = run_features_and_forest(ctx, "sf_classify", pk, cfg, forest, host_vmin, n_vmin, !raw, feat, feat_ld, pred, top_votes,
                                     labels, &labels_done);
    if (rc != SF_OK) return rc;
    sfsmall::GateRows gate = {top_votes, pred, n, n_vmin, esc_idx, esc_count, {}};
    if (!raw && sf::slow_gates(ctx, feat, feat_ld, mlp, gate, logits, labels)) {
        for (uint32_t c = 0; c < SF_MAX_CLASSES; ++c) gate.vmin[c] = host_vmin[c < n_vmin ? c : n_vmin - 1u];
        return sf::slow_infer_gated(ctx, feat, feat_ld, n, mlp, gate, labels_done ? nullptr : pred, logits, labels);
    }
    rc = sf_route(ctx, top_votes, pred, n, host_vmin, n_vmin, esc_idx, esc_count);
    if (rc != SF_OK || n == 0) return rc;
    return sf_slow_infer(ctx, raw ? nullptr : feat, raw ? 0u : feat_ld, raw ? pk : nullptr, raw ? cfg : nullptr, esc_idx, esc_count, n,
                         n, mlp, labels_done ? nullptr : pred, logits, labels);
}
