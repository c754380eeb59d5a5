// Steps 2-3: the fast model (a hard-voting ensemble of perfect binary trees) on every flow
// (Section 3.1 of the paper) and the integer form of the least-confidence score of
// Section 3.2 (top_votes = max_y votes[y]; LC = 1 - top_votes / n_trees).
//
// Also here: the same walk over the flows of a list (the middle tier of a three-tier cascade)
// and the boosted-tree form of the fast model (Section 4.1), whose leaves hold margins.
//
// Work split: a block holds a tile of flows, each flow's feature row as a shared-memory column
// [feature][flow], so the data-dependent fetch x[feat] of every lane of a wave lands in its own bank; the waves
// of the block split the trees between them.  The kernels here copy the rows of their tile into that layout; the
// walk itself comes in two forms: forest_wave.h (a wave to a tree: most calls with many trees and flows) and
// forest_core.h (the others, and the packed record format).
#include "forest_core.h"
#include "forest_wave.h"

namespace {

using namespace sfforest;

__global__ __launch_bounds__(256) void pack_forest(uint32_t n_trees, uint32_t depth, uint32_t n_features,
                                                   const uint16_t* __restrict__ nf, const float* __restrict__ nt,
                                                   PairRec* __restrict__ out)
{
    const uint32_t n_int = (1u << depth) - 1u;
    const uint32_t n_rec = recs_upto(pair_levels(depth));
    const uint64_t total = (uint64_t)n_trees * n_rec;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
         g += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t t = (uint32_t)(g / n_rec), r = (uint32_t)(g % n_rec);
        uint32_t j = 0;
        while (recs_upto(j + 1) <= r) ++j;                 // pair-level of record r
        const uint32_t pos = r - recs_upto(j);             // position within tree level 2j
        const uint32_t k0 = ((1u << (2u * j)) - 1u) + pos; // heap index of the record's top node
        const uint32_t ks[3] = {k0, 2u * k0 + 1u, 2u * k0 + 2u};
        float thr[3];
        uint32_t fe[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bool have = ks[q] < n_int;               // odd depth: the last records have no children
            uint32_t f = have ? nf[(size_t)t * n_int + ks[q]] : 0u;
            fe[q] = f < n_features ? f : n_features - 1u;  // clamp: a bad index must not leave the row
            thr[q] = have ? nt[(size_t)t * n_int + ks[q]] : 0.f;
        }
        PairRec p;
        p.thr0 = thr[0];
        p.thr1 = thr[1];
        p.thr2 = thr[2];
        p.feats = pack_feats(fe[0], fe[1], fe[2]);
        out[g] = p;
    }
}

template <int FPB_, int W, int ILP, int TAIL, bool WANT_LEAF, bool GBDT>
__global__ __launch_bounds__(FPB_ * W) void forest_votes(FastArgs a)
{
    constexpr uint32_t FPB = FPB_;         // flows per block
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const uint32_t F = a.n_features;
    float* xT = reinterpret_cast<float*>(smem_raw);                          // [F][FPB]
    const uint32_t tid = threadIdx.x;
    const uint32_t grp = tid / FPB;                        // which share of the trees this lane walks
    const uint32_t slot = tid % FPB;                       // flow slot in the block's tile
    const uint32_t i = blockIdx.x * FPB + slot;
    uint32_t n = a.n_flows;
    if (a.idx_count) {
        const uint32_t c = *a.idx_count;
        n = c < n ? c : n;
        if (blockIdx.x * FPB >= n) return; // the list ends before this block's tile (whole block leaves)
    }
    const bool live = i < n;
    uint32_t row = live ? i : n - 1; // idle lanes walk a valid row, write nothing
    if (a.idx) {
        row = a.idx[row];
        row = row < a.n_rows ? row : a.n_rows - 1u; // a bad list entry must not leave the matrix
    }
    {
        // the W lanes of a flow each copy their share of its row into the flow's column, several pieces requested before the
        // first is stored (one after the other, a large batch took 40 us for 32 features where memory needs 28)
        const float* x = a.feat + (size_t)row * a.ld;
        const uint32_t first = FPB >= 64u ? __builtin_amdgcn_readfirstlane(grp) : grp; // (whole waves: the loop is scalar)
        if ((a.ld & 3u) == 0 && (F & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0) {
            constexpr uint32_t AT_ONCE = W >= 8 ? 2 : 8 / W;
            auto put = [&](uint32_t q, const float4& v) {
                xT[(4 * q + 0) * FPB + slot] = v.x;
                xT[(4 * q + 1) * FPB + slot] = v.y;
                xT[(4 * q + 2) * FPB + slot] = v.z;
                xT[(4 * q + 3) * FPB + slot] = v.w;
            };
            uint32_t q = first;
            for (; q + (AT_ONCE - 1u) * W < F / 4u; q += AT_ONCE * W) {
                float4 v[AT_ONCE];
#pragma unroll
                for (uint32_t u = 0; u < AT_ONCE; ++u) v[u] = reinterpret_cast<const float4*>(x)[q + u * W];
#pragma unroll
                for (uint32_t u = 0; u < AT_ONCE; ++u) put(q + u * W, v[u]);
            }
            for (; q < F / 4u; q += W) put(q, reinterpret_cast<const float4*>(x)[q]);
        } else {
            for (uint32_t f = first; f < F; f += W) xT[f * FPB + slot] = x[f];
        }
    }
    forest_walk<FPB_, W, ILP, TAIL, (!GBDT && FPB >= 64u), WANT_LEAF, GBDT, false>(a, xT, i, row, live);
}

template <int FPB, int W, int ILP, int TAIL, bool GBDT>
int launch_votes(sf_ctx* ctx, const FastArgs& a, size_t lds, int slot)
{
    const uint32_t grid = (a.n_flows + FPB - 1) / FPB;
    if (a.leaf_idx) {
        SF_ALLOW_LDS(ctx, slot + 1, (forest_votes<FPB, W, ILP, TAIL, true, GBDT>));
        forest_votes<FPB, W, ILP, TAIL, true, GBDT><<<grid, FPB * W, lds, ctx->stream>>>(a);
    } else {
        SF_ALLOW_LDS(ctx, slot, (forest_votes<FPB, W, ILP, TAIL, false, GBDT>));
        forest_votes<FPB, W, ILP, TAIL, false, GBDT><<<grid, FPB * W, lds, ctx->stream>>>(a);
    }
    SF_LAUNCH_CHECK(ctx, "forest_votes");
    return SF_OK;
}

// The same in the form of forest_wave.h: 64 U flows a block, any number of waves
template <int U, int KW, bool GBDT>
__device__ __forceinline__ void tile_trees(const FastArgs& a, float* xT, uint32_t n) // xT: [F][FPB]
{
    constexpr uint32_t FPB = 64 * U;
    const uint32_t F = a.n_features, flow0 = blockIdx.x * FPB;
    if (flow0 >= n) return; // a list ends before this block's tile (whole block leaves)
    // A wave copies 16 columns of 64 rows at a time, a row to a lane: 64 bytes of a row are requested together.
    const uint32_t waves = blockDim.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool wide = (a.ld & 3u) == 0 && (F & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0;
    const uint32_t units = (F + 15u) / 16u * U;
    for (uint32_t k = wave; k < units; k += waves) {
        const uint32_t slot = lane + 64u * (k % U), f0 = k / U * 16u;
        uint32_t row = flow0 + slot;
        row = row < n ? row : n - 1u; // a slot past the end holds a valid row
        if (a.idx) {
            row = a.idx[row];
            row = row < a.n_rows ? row : a.n_rows - 1u; // a bad list entry must not leave the matrix
        }
        const float* x = a.feat + (size_t)row * a.ld + f0;
        float* dst = xT + (size_t)f0 * FPB + slot;
        if (wide) {
            float4 v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (f0 + 4u * u < F) v[u] = reinterpret_cast<const float4*>(x)[u];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (f0 + 4u * u < F) {
                    dst[(4u * u + 0u) * FPB] = v[u].x;
                    dst[(4u * u + 1u) * FPB] = v[u].y;
                    dst[(4u * u + 2u) * FPB] = v[u].z;
                    dst[(4u * u + 3u) * FPB] = v[u].w;
                }
        } else {
            for (uint32_t u = 0; u < 16u && f0 + u < F; ++u) dst[u * FPB] = x[u];
        }
    }
    forest_walk_waves<U, KW, GBDT, false>(a, xT, flow0, n);
}

// The tile follows the number of rows the host knows, a list's capacity.  A list that turns out short (up to 64 flows a unit with
// tiles of 128, 128 with tiles of 256) is walked 64 flows to a block, as many blocks as it needs: few tall tiles would leave units
// idle (capacity 1,048,576, 10,000 rows: 256 flows a block 1.42 to 1.78 times as long as blocks of 64, 128 flows 1.1 to 1.2 times).
template <int U, int KW, bool GBDT>
__global__ __launch_bounds__(1024, 8) void forest_trees(FastArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    float* xT = reinterpret_cast<float*>(smem_raw);
    uint32_t n = a.n_flows;
    if (a.idx_count) {
        const uint32_t c = *a.idx_count;
        n = c < n ? c : n;
        if (blockIdx.x * 64u >= n) return; // (most blocks of a short list: they leave before anything else is done)
        if (U > 1 && !GBDT && n <= a.short_list && (n + 63u) / 64u <= gridDim.x) {
            tile_trees<1, KW, GBDT>(a, xT, n);
            return;
        }
    }
    tile_trees<U, KW, GBDT>(a, xT, n);
}

template <int U, int KW, bool GBDT>
int launch_trees(sf_ctx* ctx, const FastArgs& a, uint32_t result_words, uint32_t waves, int slot)
{
    const size_t lds = wave_walk_lds(a.n_features, result_words, GBDT, 64u * U, waves, KW);
    SF_ALLOW_LDS(ctx, slot, (forest_trees<U, KW, GBDT>));
    forest_trees<U, KW, GBDT><<<(a.n_flows - 1u) / (64u * U) + 1u, 64u * waves, lds, ctx->stream>>>(a);
    SF_LAUNCH_CHECK(ctx, "forest_trees");
    return SF_OK;
}

// A block of forest_trees: 64 * u flows, window of kw pair-levels, waves
struct WaveShape {
    uint32_t u, kw, waves;
};

template <bool GBDT>
int launch_trees(sf_ctx* ctx, const FastArgs& a, uint32_t result_words, const WaveShape& s)
{
    const int slot = sf::kLdsTrees + (GBDT ? 5 : 0);
    if (s.u == 4u) return s.kw == 4u ? launch_trees<4, 4, GBDT>(ctx, a, result_words, s.waves, slot) : launch_trees<4, 3, GBDT>(ctx, a, result_words, s.waves, slot + 1);
    if (s.u == 2u) return s.kw == 4u ? launch_trees<2, 4, GBDT>(ctx, a, result_words, s.waves, slot + 2) : launch_trees<2, 3, GBDT>(ctx, a, result_words, s.waves, slot + 3);
    return launch_trees<1, 4, GBDT>(ctx, a, result_words, s.waves, slot + 4);
}

} // namespace

namespace sf {
size_t forest_pack_bytes(uint32_t n_trees, uint32_t depth)
{
    if (n_trees == 0 || depth == 0 || depth > SF_MAX_TREE_DEPTH) return 0;
    return align_up((size_t)n_trees * recs_upto(pair_levels(depth)) * sizeof(PairRec));
}
} // namespace sf

namespace {

// the model as the kernels see it: hard-voting forest (leaf_label) or boosted trees (leaf_value, base)
struct TreeModel {
    uint32_t n_trees, depth, n_classes, n_features;
    const uint16_t* node_feat;
    const float* node_thr;
    const uint8_t* leaf_label;
    const float* leaf_value;
    const float* base;
    const void* packed; // records made earlier by sf_forest_pack / sf_gbdt_pack, or NULL
};

struct Outputs {
    uint16_t* votes;
    uint16_t* pred;
    uint16_t* top_votes;
    uint16_t* leaf_idx;
    uint16_t* labels;
    float* margins;
    float* score;
    int score_kind;
};

int pack_into(sf_ctx* ctx, const TreeModel& m, PairRec* out)
{
    const uint64_t total = (uint64_t)m.n_trees * recs_upto(pair_levels(m.depth));
    uint64_t blocks = (total + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    pack_forest<<<(uint32_t)blocks, 256, 0, ctx->stream>>>(m.n_trees, m.depth, m.n_features, m.node_feat, m.node_thr, out);
    SF_LAUNCH_CHECK(ctx, "pack_forest");
    return SF_OK;
}

int check_model(sf_ctx* ctx, const char* who, const TreeModel& m)
{
    if (m.depth < 1 || m.depth > SF_MAX_TREE_DEPTH)
        return sf::fail(ctx, SF_EINVAL, "%s: depth %u outside 1..%d", who, m.depth, SF_MAX_TREE_DEPTH);
    if (m.n_trees < 1 || m.n_trees > 65535) return sf::fail(ctx, SF_EINVAL, "%s: n_trees %u outside 1..65535", who, m.n_trees);
    if (m.n_features < 1 || m.n_features > SF_MAX_FEATURES)
        return sf::fail(ctx, SF_EINVAL, "%s: n_features %u outside 1..%d", who, m.n_features, SF_MAX_FEATURES);
    if (!m.node_feat || !m.node_thr) return sf::fail(ctx, SF_EINVAL, "%s: model arrays missing", who);
    return SF_OK;
}

// The most trees for which the fused feature + forest kernel does a batch with one lane per flow (256 flows a block).  Splitting a
// flow's statistics between waves costs a third more instructions and pays where lanes are few or the walk is long; with few
// trees the kernel is its feature phase.  How well the blocks fill their rounds decides the rest (`full`, percent: two blocks a
// unit, with one window three).  One lane : best other shape, in us, ten classes: 1,048,576 flows of 16 packets, windows 8, 16:
// 5 trees 98 : 136, 47 trees of depth 4 216 : 245; window 16: 5 trees 64 : 94, 47 trees 130 : 155; ragged, window 8: 5 trees 50 : 66,
// 32 trees of depth 4 92 : 101, of depth 12 equal.  100,000 flows, windows 8, 16 (one round, 76 %): 5 trees 15 : 20.5, 47 trees 31 : 32.
// 140,000 (a second round with 7 % of its blocks): 8 trees equal, 47 trees 1.25 times as long.
uint32_t fused_one_lane_trees(uint32_t depth, uint32_t n_windows, uint32_t dmax, uint32_t n_rows, uint32_t n_cu)
{
    if (n_rows < 150u * n_cu) return 0u;
    const uint32_t blocks = (n_rows - 1u) / 256u + 1u, at_once = (n_windows == 1u ? 3u : 2u) * n_cu;
    const uint32_t rounds = (blocks + at_once - 1u) / at_once, full = (uint32_t)(100ull * blocks / ((uint64_t)rounds * at_once));
    if (dmax <= 8u) {
        if (n_windows == 2u) return full < 75u ? 0u : 6u;
        if (full < 45u) return 0u;
        return rounds <= 2u || depth > 8u ? 6u : depth <= 6u ? 80u : 24u;
    }
    if (n_windows == 2u) return full < 60u ? 6u : rounds == 1u ? 47u : full < 90u ? 24u : 64u;
    return full < 45u ? 6u : full < 60u ? 12u : full < 75u ? 32u : 64u;
}

// Which calls the form with a wave to a tree takes (forest_wave.h), and the block; false: the shapes of choose_shape.  Times are
// the walk's in us, this form : the best shape that choose_shape knows; 100 trees and ten classes unless another number is named.
//
// Voting form: sixteen waves a block, two blocks a unit (32 waves, all it holds).
//   Trees: from 48, a wave's trees are walked in rounds of sixteen and filling the tile has to be paid for (400,000 flows x 64
//     features, depth 12: 70 trees 107 : 127, 47 85 : 96, 20 55 : 52).  An odd depth gains most: the level left over is read from the window,
//     where the other form reads a record of the last pair-level from memory (64 trees of depth 5 50 : 61, of 7 67 : 72; depth 3, 200 trees
//     0.76 times as long).  Shallow trees of even depth gain less: from 96 at depth 6 and 8 (depth 8: 100 trees 84 : 96, 70 69 : 68), 192 up to
//     depth 4.  Depth 2 not up to 64 flows a unit (8,000 flows 9.7 : 9.4) nor, with more than 64 features and less than 400 trees, past 384
//     (400,000 x 128, 200 trees 92 : 83); depth 1 in large batches of up to 64 features (1,048,576 x 64, 200 trees 0.86 times as long, x 96
//     1.10, 100,000 x 32 1.10).  More than 112 features leave room for three pair-levels only: depth 7 to 10 from 64 trees past 384 flows
//     a unit (400,000 x 128, 48 trees of depth 7 79 : 75, of depth 9 97 : 94, 64 0.97 to 1.01 times as long).
//   In the fused kernel the tile is 128 flows always: nothing of depth 1, 2 and 4 (1,048,576 flows, windows 8 and 16, 200 trees of depth 4 1.06
//     times as long as 64 x 8, 5 and 8 1.17; 400,000, depth 1 1.16 and 1.28; but two windows, 300 trees of depth 4, 1,048,576 flows 0.95).  With
//     windows of up to 8 packets, whose features are done soon and leave the unit to the other form's walk, depth 3 from 300 trees, 5 from 192, 6 not
//     at all, 7, 9 and 10 from 64 past 256 flows a unit (400,000 flows, windows 5 and 8: 48 trees of depth 5 1.14 times as long, of depth 7 1.08, 64 of
//     depth 9 0.99; 192 of depth 3 1.03, of depth 6 1.09; 60,000, 48 trees of depth 7 0.90).
//   Flows: not where the blocks' last round has few of them, 128 to 192 flows a unit (0.97 times as fast in the mean of 550
//     models, at worst 0.81; 1.12 times below, 1.16 above) and 256 to 320 (1.05 in the mean, one in eight 0.91 to 0.97; 1.17 above); models that
//     gain little not from 384 to 432 either (100,003 flows: 200 trees of depth 4 1.05 times as long, of depth 2 1.02 to 1.08, 100 of depth 8 on 96
//     features 1.03, 64 of depth 9 on 128 1.05; fused, 192 trees of depth 6 1.09, windows 5 and 8, 192 of depth 8 1.10, 64 of depth 10 1.03).
//   Window: four pair-levels from depth 7 (400,000 x 64 features: depth 7 88 : 105, 10 105 : 119, 12 143 : 167, 13 277 : 357; three
//     pair-levels 101, 113, 153, 281), three where depth ends there or shared memory has no room for more (128 features: depth 6
//     86 : 101, 12 180 : 225; one block a unit with four 132, 215).
//   256 flows a block from 1,200 flows a unit, where two such blocks fit (32 features, depth 12: 1,048,576 flows 284 : 357, with 128
//     flows 314; 200,000 flows 80, with 128 72 : 82); 64 features have room for three pair-levels only (depth 6 67 : 79 and 8 84 : 96,
//     with 128 flows 77, 88; deeper 128 flows are better: 112 and 105 at depth 10).
//   64 flows a block up to 64 flows a unit, so that every unit has a block (8,000 flows 11.7 : 13.0; 20,000 flows 17 with 64, 15.8 with 128
//     : 18.4; 65,536 26 : 33).
//
// Boosted form, a wave to a class: 5 to 16 classes, in large batches with up to 64 features 3 and 4 too; the largest tile that
// leaves every unit a block and with which 18 waves or more are resident, four pair-levels before three (120 trees of depth 8,
// 400,000 flows x 64 features: 3 classes 145 : 197, 5 113 : 171, 8 103 : 156, 10 104 : 156, 16 97 : 163; 96 features: 4 classes 149 : 137, 5
// 147 : 202, 10 131 : 164; two classes 202 : 154; 10,000 flows, 3 and 4 classes 1.4 times as long; 8,000 flows, ten classes 13 : 20).  64 flows a block for trees up
// to depth 6 past 128 flows a unit only where four such blocks fit (128 features, 60 trees of depth 6, 400,000 flows: 8 classes with three blocks
// 94 : 89, 6 with four 0.91 times as long).
// dmax: packets of the deepest window (fused kernel), 0 for the stand-alone walk.
bool waves_take(uint32_t n_trees, uint32_t depth, uint32_t n_features, uint32_t dmax, uint32_t n_rows, uint32_t n_cu)
{
    const uint32_t per_cu = n_rows / n_cu; // (few flows: blocks of 16, see choose_shape)
    if (n_rows <= 24u * n_cu || (n_rows > 128u * n_cu && per_cu < 192u) || (n_rows > 256u * n_cu && per_cu < 320u)) return false;
    const bool short_windows = dmax != 0u && dmax <= 8u, even = depth == 6u || depth == 8u;
    if (n_rows > 384u * n_cu && per_cu < 432u) {
        if (dmax ? (even && n_trees > 128u && n_trees < 256u) || (short_windows && depth <= 10u && n_trees < (depth == 5u ? 256u : even ? 0u : 96u))
                 : (depth == 2u && n_trees < 400u) || (depth == 4u && n_trees < 300u) || (even && n_features >= 96u && n_trees < 128u) ||
                       (n_features > 112u && depth >= 7u && depth <= 10u && n_trees < 96u))
            return false;
    }
    if (dmax && (depth <= 2u || depth == 4u)) return depth == 4u && n_features > 32u && !short_windows && n_trees >= 256u && per_cu >= 3000u;
    switch (depth) {
    case 1: return n_trees >= 192u && n_features <= 64u && per_cu >= 1200u;
    case 2: return n_trees >= 192u && n_rows > 64u * n_cu && (n_features <= 64u || n_rows <= 384u * n_cu || n_trees >= 400u);
    case 3: return n_trees >= (short_windows ? 300u : 192u);
    case 4: return n_trees >= 192u;
    case 5: return n_trees >= (short_windows && n_rows > 256u * n_cu ? 192u : 48u);
    case 6: return n_trees >= 96u && !short_windows;
    case 8: return n_trees >= 96u;
    case 7:
    case 9:
    case 10: return n_trees >= ((short_windows && n_rows > 256u * n_cu) || (n_features > 112u && n_rows > 384u * n_cu) ? 64u : 48u);
    default: return n_trees >= 48u;
    }
}

bool choose_waves(const FastArgs& a, uint32_t result_words, bool gbdt, uint32_t n_rows, uint32_t n_cu, WaveShape* s)
{
    auto take = [&](uint32_t u, uint32_t kw, uint32_t waves, uint32_t least) { // least: waves a unit has to hold
        *s = {u, kw, waves};
        const uint32_t blocks = (uint32_t)(160u * 1024u / wave_walk_lds(a.n_features, result_words, gbdt, 64u * u, waves, kw));
        return (blocks * waves < 32u ? blocks : 32u / waves) * waves >= least;
    };
    const bool deep = a.depth > 6u;
    if (gbdt) {
        const uint32_t C = a.n_classes;
        if (n_rows <= 24u * n_cu || C > 16u || C < (a.n_features <= 64u && n_rows >= 384u * n_cu ? 3u : 5u)) return false;
        for (uint32_t u = n_rows >= 320u * n_cu ? 4u : n_rows >= 128u * n_cu ? 2u : 1u; u >= 2u; u /= 2u)
            if ((deep && take(u, 4, C, 18)) || take(u, 3, C, 18)) return true;
        return take(1, 4, C, !deep && n_rows >= 128u * n_cu && C > 4u ? 4u * C : 18u);
    }
    if (!waves_take(a.n_trees, a.depth, a.n_features, 0u, n_rows, n_cu)) return false;
    if (n_rows <= 64u * n_cu) return take(1, 4, 16, 32);
    if (n_rows >= 1200u * n_cu) {
        if (deep && take(4, 4, 16, 32)) return true;
        if (a.depth <= 8u && a.depth != 7u && take(4, 3, 16, 32)) return true;
    }
    return (deep && take(2, 4, 16, 32)) || take(2, 3, 16, 32);
}

// The shape of a block and its shared memory, by batch size and model.  All figures are the walk's time in
// microseconds for 64 features and 100 trees of depth 12 unless another model is named.
//   few flows: 16 flows x 32 lanes, nothing staged, so that even a small batch gives every compute unit a block and
//     a lane only a few trees one after the other.  4,000 flows: 11 us against 15 (64x8) and 54 (one lane per
//     flow); 10,000 flows: 17.6 against 16.1.  The line is 24 flows per compute unit (6,144).
//   otherwise 64 x 8, four blocks per compute unit where 40 KB hold the tile and a pair-level of records.  The stand-alone walk of what
//     the form with a wave to a tree does not take (48 to 95 trees of depth 6 or 8, to 191 up to depth 4, calls that want leaf numbers)
//     takes 128 x 8 from 3,000 flows per unit (with leaf numbers 2,000), where its 80 KB hold one pair-level more than the smaller tile
//     (1,048,576 flows, 80 trees of depth 8 on 96 features 231 : 246 for 64 x 8, on 64 193 : 199; 150 of depth 4 on 128 251 : 267; with leaf numbers
//     100 trees of depth 12 878 : 906; 600,000 flows, 100 trees of depth 10 with leaf numbers on 32 features 328 : 342, 64 of depth 6 on 96
//     features 1.05 times as long; 270,000 flows up to 1.1: blocks twice as large share out less evenly).  In the fused
//     kernel 128 flows in the form with a wave to a tree for the sizes that form takes (waves_take; the kernel in us before : after,
//     ten classes: 1,048,576 flows, windows 8 and 16, 100 trees of depth 12 500 : 439, no rows kept 479 : 395; windows 5 and 10, depth
//     10 367 : 336; 400,000 flows, 250 trees of depth 12 479 : 368, 100 of depth 8 133 : 126; 18,000 ragged flows 24 : 19, 65,000 43 : 34).
//   fewer than 48 trees: 128 x 4, five trees at once per lane; eight lanes would walk a handful each
//     (1,000,000 flows, 16 trees of depth 8: 62 against 76).
//   256 flows, one lane each, in large batches where lanes that share a flow have nothing to share or stand in each other's way:
//     a walk so short that reading the rows is all there is: 32 features, from 1,400 flows per unit (with up to four trees from
//     750), few and shallow trees (200,000 flows, four trees of depth 4 8.7 us against 9.6; 1,048,576 flows, one tree of depth 8 35 against 45, 12 of depth 4 44 against 51, 24 of depth 4 53 against 63; but 16 of
//     depth 6 1.13 times as long, and with 64 features equal);
//     trees of depth 13 and 14 with leaf numbers, whose records (87 KB a tree) the caches cannot hold for eight trees at a time, from 64 trees and
//     1,700 flows per unit (1,048,576 flows, 100 trees of depth 13 1330 against 1608, 64 of depth 14 821 against 912; 460,000 flows, 80 trees of depth 13
//     1.04 times as fast, 330,000 equal, 270,000 0.96).
// Boosted form: lanes split the classes, not the trees (see forest_walk), so a few large shares are better than
// many uneven ones: 256 x 2 (1,048,576 flows, 200 trees of depth 8: 585 against 599 for 64 x 4; with 32 features three blocks a
// unit, 1.1 to 1.2 times as fast as two with more staged), 64 x 4 up to 3 * 128 flows per unit (30,000 flows 39 against 83 with one
// lane per flow; two classes leave half of its lanes idle: with 40 trees or more 256 x 2 from 256 flows per unit, 95,000 flows
// x 60 trees of depth 8 1.3 times as fast), 16 x 16 for few flows.  One class and three leave lanes
// idle that 256 x 1 does not have (three classes, 1,048,576 flows x 32 features: 150 trees of depth 6 316 against 341, 60 of depth 1
// 82 against 120); five classes (calls with leaf numbers) only with 75 trees or more, 17 to 32 features and 3,000 flows per unit (1,048,576 flows x
// 32 features, 100 trees of depth 8 554 against 592, of depth 5 525 against 541; 50 of depth 8 282 against 277, on 16 features 265 against 254).
// dmax: packets of the deepest window (fused kernel), 0 for the stand-alone walk.
TileShape choose_shape(FastArgs& a, uint32_t result_words, bool gbdt, uint32_t n_rows, uint32_t n_cu, uint32_t dmax, size_t* lds)
{
    const uint32_t few = 24u * n_cu, many = 3u * 128u * n_cu;
    auto fit = [&](TileShape s, size_t first, uint32_t least) {
        // what `first` holds, or else a third or half of a unit's shared memory, with `least` pair-levels of records;
        // a forest too large for that goes without, in the smallest of these (or the whole) that holds the tile
        const size_t budgets[] = {first, 160 * 1024 / 3 - 256, 80 * 1024, 160 * 1024};
        for (int q = 0; q < 7; ++q) {
            const size_t b = budgets[q < 3 ? q : q - 3];
            *lds = plan_lds(a, result_words, kTileFlows[s], b, &a.top_pairs);
            if (*lds <= b && (q >= 3 || a.top_pairs >= least || a.depth / 2 < least)) return;
        }
    };
    if (n_rows <= few) {
        const TileShape s = gbdt ? kTile16x16g : kTile16x32;
        *lds = plan_lds(a, result_words, 16, 0, &a.top_pairs);
        return s;
    }
    if (gbdt) {
        const bool one_lane = a.n_classes == 1u || a.n_classes == 3u ||
                              (a.n_classes == 5u && a.n_features > 16u && a.n_features <= 32u && a.n_trees >= 75u && n_rows >= 3000u * n_cu);
        fit(one_lane ? kTile256x1g : kTile256x2g, 160 * 1024 / 3 - 256, 1);
        if (one_lane && n_rows >= many && *lds <= 80 * 1024) return kTile256x1g;
        if (n_rows >= (a.n_classes <= 2u && a.n_trees >= 40u ? 256u * n_cu : many) && *lds <= 80 * 1024) return kTile256x2g; // (one block per unit is slower than the smaller tile)
        fit(kTile64x4g, 40 * 1024, 1);
        return kTile64x4g;
    }
    bool one_lane;
    if (dmax)
        one_lane = a.n_trees <= fused_one_lane_trees(a.depth, a.n_features / 32u, dmax, n_rows, n_cu);
    else
        one_lane = (a.depth >= 13u && a.n_trees >= 64u && n_rows >= 1700u * n_cu) ||
                   (a.n_features <= 32u && (n_rows >= 1400u * n_cu
                                                ? (a.depth <= 5u ? a.n_trees < 48u : a.depth <= 7u ? a.n_trees <= 12u : a.depth <= 9u && a.n_trees <= 4u)
                                                : n_rows >= 750u * n_cu && a.depth <= 7u && a.n_trees <= 4u));
    if (one_lane) {
        fit(kTile256x1, 160 * 1024 / 3 - 256, 1);
        if (*lds <= 80 * 1024) return kTile256x1;
    }
    if (a.n_trees < 48u) {
        fit(kTile128x4, 40 * 1024, 1);
        return kTile128x4;
    }
    if (dmax && n_rows > 64u * n_cu && waves_take(a.n_trees, a.depth, a.n_features, dmax, n_rows, n_cu)) {
        *lds = wave_walk_lds(a.n_features, result_words, false, 128, 16, 4);
        return kTile128Waves;
    }
    fit(kTile64x8, 40 * 1024, 1);
    if (!dmax && n_rows >= (a.leaf_idx ? 2000u : 3000u) * n_cu) {
        uint32_t top = 0;
        const size_t wide = plan_lds(a, result_words, 128, 80 * 1024, &top);
        if (wide <= 80 * 1024 && top > a.top_pairs) {
            a.top_pairs = top;
            *lds = wide;
            return kTile128x8;
        }
    }
    return kTile64x8;
}

// The model part of the kernel arguments: checks, the packed records (made into the workspace when the model
// carries none) and the width of the vote counters.  *result_words: words of results a flow keeps in shared
// memory during the walk.  check_only: stop after the argument checks (a call on zero flows launches nothing).
int setup_trees(sf_ctx* ctx, const char* who, const TreeModel& m, bool gbdt, uint32_t feat_ld, FastArgs& a, uint32_t* result_words,
                bool check_only = false)
{
    if (m.depth < 1 || m.depth > SF_MAX_TREE_DEPTH)
        return sf::fail(ctx, SF_EINVAL, "%s: depth %u outside 1..%d", who, m.depth, SF_MAX_TREE_DEPTH);
    if (m.n_trees < 1 || m.n_trees > 65535) return sf::fail(ctx, SF_EINVAL, "%s: n_trees %u outside 1..65535", who, m.n_trees);
    if (m.n_classes < 1 || m.n_classes > SF_MAX_CLASSES)
        return sf::fail(ctx, SF_EINVAL, "%s: n_classes %u outside 1..%d", who, m.n_classes, SF_MAX_CLASSES);
    if (m.n_features < 1 || m.n_features > SF_MAX_FEATURES)
        return sf::fail(ctx, SF_EINVAL, "%s: n_features %u outside 1..%d", who, m.n_features, SF_MAX_FEATURES);
    if (m.n_features > feat_ld) return sf::fail(ctx, SF_EINVAL, "%s: n_features %u > feat_ld %u", who, m.n_features, feat_ld);
    if (!m.node_feat || !m.node_thr || (gbdt ? !m.leaf_value : !m.leaf_label))
        return sf::fail(ctx, SF_EINVAL, "%s: model arrays missing", who);
    if (check_only) return SF_OK;

    const PairRec* packed = (const PairRec*)m.packed;
    if (!packed) {
        sf::Carve ws(ctx);
        const size_t pack_bytes = sf::forest_pack_bytes(m.n_trees, m.depth);
        PairRec* mine = (PairRec*)ws.take(pack_bytes);
        if (!mine)
            return sf::fail(ctx, SF_ENOMEM, "%s: workspace has %zu bytes, packed trees need %zu", who, ctx->ws_bytes,
                            pack_bytes + sf::kFlagBytes);
        const int rc = pack_into(ctx, m, mine);
        if (rc != SF_OK) return rc;
        packed = mine;
    }
    a.leaf_value = m.leaf_value;
    a.base = m.base;
    a.n_trees = m.n_trees;
    a.depth = m.depth;
    a.n_classes = m.n_classes;
    a.n_features = m.n_features;
    a.recs = packed;
    a.leaf_label = m.leaf_label;
    a.vote_bits = a.n_trees <= 255 ? 8u : 16u;
    *result_words = gbdt ? a.n_classes : (a.n_classes * a.vote_bits + 31u) / 32u;
    return SF_OK;
}

// every entry point of this file: n_flows rows (all flows, or the capacity of the list idx)
int run_trees(sf_ctx* ctx, const char* who, const float* feat, uint32_t feat_ld, uint32_t n_flows, const uint32_t* idx,
              const uint32_t* idx_count, uint32_t n_rows, const TreeModel& m, bool gbdt, const Outputs& out)
{
    FastArgs a = {};
    uint32_t result_words = 0;
    size_t lds = 0;
    {
        const int rc = setup_trees(ctx, who, m, gbdt, feat_ld, a, &result_words, n_flows == 0);
        if (rc != SF_OK) return rc;
    }
    if (n_flows == 0) return SF_OK;
    if (!feat || !out.pred || (gbdt ? !out.score : !out.top_votes))
        return sf::fail(ctx, SF_EINVAL, "%s: feat, pred or %s is NULL", who, gbdt ? "score" : "top_votes");
    a.feat = feat;
    a.ld = feat_ld;
    a.n_flows = n_flows;
    a.idx = idx;
    a.idx_count = idx_count;
    a.n_rows = n_rows;
    a.labels = out.labels;
    a.margins = out.margins;
    a.score = out.score;
    a.score_kind = out.score_kind;
    a.votes = out.votes;
    a.pred = out.pred;
    a.top = out.top_votes;
    a.leaf_idx = out.leaf_idx;
    WaveShape wave;
    if (!a.leaf_idx && choose_waves(a, result_words, gbdt, n_flows, (uint32_t)ctx->n_cu, &wave)) {
        a.short_list = 32u * wave.u * (uint32_t)ctx->n_cu;
        return gbdt ? launch_trees<true>(ctx, a, result_words, wave) : launch_trees<false>(ctx, a, result_words, wave);
    }
    const TileShape shape = choose_shape(a, result_words, gbdt, n_flows, (uint32_t)ctx->n_cu, 0u, &lds);
    if (lds > 160 * 1024) return sf::fail(ctx, SF_EUNSUPPORTED, "%s: %zu bytes of shared memory needed", who, lds);
    const int slot = sf::kLdsForest + 2 * (int)shape;
    switch (shape) {
    case kTile128x4: return launch_votes<128, 4, 5, 4, false>(ctx, a, lds, slot);
    case kTile128x8: return launch_votes<128, 8, 3, 2, false>(ctx, a, lds, slot);
    case kTile64x8: return launch_votes<64, 8, 3, 2, false>(ctx, a, lds, slot);
    case kTile16x32: return launch_votes<16, 32, 5, 2, false>(ctx, a, lds, slot);
    case kTile256x1: return launch_votes<256, 1, 10, 5, false>(ctx, a, lds, slot);
    case kTile256x1g: return launch_votes<256, 1, 10, 5, true>(ctx, a, lds, slot);
    case kTile256x2g: return launch_votes<256, 2, 5, 2, true>(ctx, a, lds, slot);
    case kTile64x4g: return launch_votes<64, 4, 5, 2, true>(ctx, a, lds, slot);
    default: return launch_votes<16, 16, 5, 2, true>(ctx, a, lds, slot);
    }
}

int run_forest(sf_ctx* ctx, const char* who, const float* feat, uint32_t feat_ld, uint32_t n_flows, const uint32_t* idx,
               const uint32_t* idx_count, uint32_t n_rows, const sf_forest* f, uint16_t* votes, uint16_t* pred,
               uint16_t* top_votes, uint16_t* leaf_idx, uint16_t* labels)
{
    if (!f) return sf::fail(ctx, SF_EINVAL, "%s: forest is NULL", who);
    const TreeModel m = {f->n_trees, f->depth, f->n_classes, f->n_features, f->node_feat, f->node_thr, f->leaf_label,
                         nullptr, nullptr, f->packed};
    const Outputs out = {votes, pred, top_votes, leaf_idx, labels, nullptr, nullptr, 0};
    return run_trees(ctx, who, feat, feat_ld, n_flows, idx, idx_count, n_rows, m, false, out);
}

} // namespace

namespace sf {
// the hard-voting forest as kernel arguments, and the block shape of its walk (for the fused feature + forest entry point)
int forest_setup(sf_ctx* ctx, const char* who, const sf_forest* f, uint32_t feat_ld, sfforest::FastArgs& a, uint32_t* result_words)
{
    if (!f) return fail(ctx, SF_EINVAL, "%s: forest is NULL", who);
    const TreeModel m = {f->n_trees, f->depth, f->n_classes, f->n_features, f->node_feat, f->node_thr, f->leaf_label,
                         nullptr, nullptr, f->packed};
    return setup_trees(ctx, who, m, false, feat_ld, a, result_words);
}

sfforest::TileShape forest_shape(sfforest::FastArgs& a, uint32_t result_words, uint32_t n_rows, uint32_t n_cu, uint32_t dmax, size_t* lds)
{
    return choose_shape(a, result_words, false, n_rows, n_cu, dmax, lds);
}
} // namespace sf

extern "C" int sf_fast_infer(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n_flows,
                             const sf_forest* forest, uint16_t* votes, uint16_t* pred, uint16_t* top_votes,
                             uint16_t* leaf_idx)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_fast_infer: ctx is NULL");
    return run_forest(ctx, "sf_fast_infer", feat, feat_ld, n_flows, nullptr, nullptr, n_flows, forest, votes, pred,
                      top_votes, leaf_idx, nullptr);
}

extern "C" int sf_fast_infer_subset(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n_flows,
                                    const uint32_t* idx, const uint32_t* idx_count, uint32_t idx_cap,
                                    const sf_forest* forest, uint16_t* votes, uint16_t* pred, uint16_t* top_votes,
                                    uint16_t* labels)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_fast_infer_subset: ctx is NULL");
    if (idx_cap && n_flows == 0) return sf::fail(ctx, SF_EINVAL, "sf_fast_infer_subset: a list over zero flows");
    if (idx_cap && (!idx || !idx_count)) return sf::fail(ctx, SF_EINVAL, "sf_fast_infer_subset: idx or idx_count is NULL");
    return run_forest(ctx, "sf_fast_infer_subset", feat, feat_ld, idx_cap, idx, idx_count, n_flows, forest, votes, pred,
                      top_votes, nullptr, labels);
}

extern "C" int sf_gbdt_infer(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n_flows, const sf_gbdt* model,
                             int score_kind, float* margins, uint16_t* pred, float* score, uint16_t* leaf_idx)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_gbdt_infer: ctx is NULL");
    if (!model) return sf::fail(ctx, SF_EINVAL, "sf_gbdt_infer: model is NULL");
    if (score_kind != SF_SCORE_LC && score_kind != SF_SCORE_ENTROPY)
        return sf::fail(ctx, SF_EINVAL, "sf_gbdt_infer: score_kind %d is neither SF_SCORE_LC nor SF_SCORE_ENTROPY", score_kind);
    const TreeModel m = {model->n_trees, model->depth, model->n_classes, model->n_features, model->node_feat,
                         model->node_thr, nullptr, model->leaf_value, model->base, model->packed};
    const Outputs out = {nullptr, pred, nullptr, leaf_idx, nullptr, margins, score, score_kind};
    return run_trees(ctx, "sf_gbdt_infer", feat, feat_ld, n_flows, nullptr, nullptr, n_flows, m, true, out);
}

extern "C" size_t sf_forest_packed_bytes(uint32_t n_trees, uint32_t depth) { return sf::forest_pack_bytes(n_trees, depth); }

extern "C" int sf_forest_pack(sf_ctx* ctx, const sf_forest* f, void* packed)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_forest_pack: ctx is NULL");
    if (!f || !packed) return sf::fail(ctx, SF_EINVAL, "sf_forest_pack: forest or packed is NULL");
    if ((uintptr_t)packed & 15u) return sf::fail(ctx, SF_EINVAL, "sf_forest_pack: packed is not 16-byte aligned");
    const TreeModel m = {f->n_trees, f->depth, f->n_classes, f->n_features, f->node_feat, f->node_thr, f->leaf_label,
                         nullptr, nullptr, nullptr};
    const int rc = check_model(ctx, "sf_forest_pack", m);
    return rc != SF_OK ? rc : pack_into(ctx, m, (PairRec*)packed);
}

extern "C" int sf_gbdt_pack(sf_ctx* ctx, const sf_gbdt* g, void* packed)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_gbdt_pack: ctx is NULL");
    if (!g || !packed) return sf::fail(ctx, SF_EINVAL, "sf_gbdt_pack: model or packed is NULL");
    if ((uintptr_t)packed & 15u) return sf::fail(ctx, SF_EINVAL, "sf_gbdt_pack: packed is not 16-byte aligned");
    const TreeModel m = {g->n_trees, g->depth, g->n_classes, g->n_features, g->node_feat, g->node_thr, nullptr,
                         g->leaf_value, g->base, nullptr};
    const int rc = check_model(ctx, "sf_gbdt_pack", m);
    return rc != SF_OK ? rc : pack_into(ctx, m, (PairRec*)packed);
}
