// Device code of steps 2-3 shared by the stand-alone forest kernel and the fused feature + forest kernel:
// the walk of a hard-voting ensemble of perfect binary trees (the fast model that sees every flow,
// Section 3.1 of the paper; boosted form: Section 4.1) over a tile of flows whose feature rows already sit
// in shared memory as columns [feature][flow], and the score of Section 3.2 (top_votes = max_y votes[y],
// LC = 1 - top_votes / n_trees; entropy or LC of the softmax for boosted trees).
//
// What bounds the walk is gather throughput, of the caches' address path above all, so the forest is packed
// into 16-byte records that hold TWO levels: a node and both its children (three thresholds, three feature
// indices).  One 16-byte load then serves two visits.  Records form a quaternary heap per tree (record r has
// children 4r+1..4r+4); the records of the top levels of every tree are staged in shared memory, the deeper
// ones come through the cache; the leaf label is one byte load at the end.  A few trees are walked at once per
// lane to keep independent loads in flight.  Votes are integers in shared memory; nothing in the voting form
// rounds.
//
// The feature tile (F * 4 bytes per flow) is what fills shared memory, so it also limits how many flows a
// compute unit can hold.  Several waves therefore work on the same tile, each on its share of the trees: the
// unit then runs up to 32 waves instead of 8 and the address path stays 81 % busy (65 % before; 72 % in the fused kernel).  A wave's
// lanes all walk the SAME trees, for different flows: lanes that split the trees of one flow between them
// (as this code did before, for shapes with few resident waves) spread every record load over two to four
// times as many cache lines.  Measured, the walk alone, before -> after: 1,048,576 flows x 64 features, 100
// trees of depth 12: 0.588 -> 0.42 ms; depth 10: 0.375 -> 0.29 ms; 4,194,304 flows x 128 features, 500 trees of
// depth 10: 10.2 -> 6.2 ms; 65,536 flows, 200 trees of depth 10: 70 -> 46 us; 97 flows, 100 trees of depth 12:
// 53 -> 11 us.  Larger batches of many trees have a form of their own now, forest_wave.h.
#pragma once

#include <type_traits>

#include "common.h"

namespace sfforest {

constexpr uint32_t kFeatRot = 10; // the word of feature indices is rotated left by this (see forest_walk)

struct __align__(16) PairRec {
    float thr0, thr1, thr2; // node, its left child, its right child
    uint32_t feats;         // their feature indices as 8-bit fields (f0 | f1 << 8 | f2 << 16), rotated left by kFeatRot
};

__host__ __device__ inline uint32_t pack_feats(uint32_t f0, uint32_t f1, uint32_t f2)
{
    const uint32_t w = f0 | (f1 << 8) | (f2 << 16);
    return (w << kFeatRot) | (w >> (32u - kFeatRot));
}

__host__ __device__ inline uint32_t pair_levels(uint32_t depth) { return (depth + 1u) / 2u; }
__host__ __device__ inline uint32_t recs_upto(uint32_t j) { return ((1u << (2u * j)) - 1u) / 3u; } // (4^j-1)/3

struct FastArgs {
    const float* feat;
    uint32_t ld;
    uint32_t n_flows;          // rows to classify (the capacity of the list when idx is given)
    const uint32_t* idx;       // subset form: row j is flow idx[j]; NULL = row j is flow j
    const uint32_t* idx_count; // subset form: device-side length of idx
    uint32_t short_list;       // subset form: lists of up to this many rows are walked 64 flows to a block (forest_trees)
    uint32_t n_rows;           // subset form: rows of feat (list entries are clamped below it)
    uint16_t* labels;          // subset form, optional: labels[idx[j]] = pred of row j
    // boosted form: leaves hold margins instead of labels, tree t adds to class t % n_classes
    const float* leaf_value;   // [n_trees][2^depth]
    const float* base;         // [n_classes] initial margins, or NULL
    float* margins;            // optional [n][n_classes]
    float* score;              // [n]: LC or entropy of softmax(margins)
    int score_kind;
    uint32_t n_trees, depth, n_classes, n_features;
    uint32_t top_pairs; // pair-levels of every tree staged in shared memory
    uint32_t vote_bits; // width of one packed vote counter: 8 (n_trees <= 255) or 16
    const PairRec* recs;
    const uint8_t* leaf_label;
    uint16_t* votes;
    uint16_t* pred;
    uint16_t* top;
    uint16_t* leaf_idx;
    // fused form: the tile's rows are written to feat_out only for flows the gate hands on
    // (top_votes < vmin, or vmin[pred] with one threshold per class)
    float* feat_out;
    uint32_t feat_out_ld;
    uint32_t feat_out16; // feat_out is 16-byte aligned and its leading dimension a multiple of 4
    uint32_t n_vmin;
    uint16_t vmin[SF_MAX_CLASSES];
};

// How many pair-levels of every tree fit into shared memory beside the tile (kept within `budget` bytes) and the
// block's shared memory that makes.
inline size_t plan_lds(const FastArgs& a, uint32_t result_words, uint32_t fpb, size_t budget, uint32_t* top_pairs)
{
    const size_t fixed = ((size_t)a.n_features + result_words) * 4 * fpb;
    const uint32_t full_pairs = a.depth / 2;
    uint32_t t = 0;
    while (t < full_pairs && fixed + (size_t)a.n_trees * recs_upto(t + 1) * 16 <= budget) ++t;
    *top_pairs = t;
    return fixed + (size_t)a.n_trees * recs_upto(t) * 16;
}

// The shapes a block of the walk comes in (flows x lanes per flow), see choose_shape
enum TileShape { kTile128Waves, kTile128x4, kTile64x8, kTile16x32, kTile256x1, kTile256x2g, kTile64x4g, kTile16x16g, kTile256x1g, kTile128x8 };
constexpr uint32_t kTileFlows[] = {128, 128, 64, 16, 256, 256, 64, 16, 256, 128};

// A flow's result from its column of class margins: label, score of the softmax (in binary64) and what else was asked for
__device__ __forceinline__ void boosted_result(const FastArgs& a, const float* mcol, uint32_t stride, uint32_t i, uint32_t row)
{
    const uint32_t C = a.n_classes;
    uint32_t bc = 0;
    float bm = mcol[0];
    for (uint32_t c = 1; c < C; ++c) {
        const float m = mcol[c * stride];
        if (m > bm) { // strict: the lowest class wins a tie
            bm = m;
            bc = c;
        }
    }
    double z = 0.0;
    for (uint32_t c = 0; c < C; ++c) z += exp((double)mcol[c * stride] - (double)bm);
    double sc;
    if (a.score_kind == SF_SCORE_ENTROPY) {
        double h = 0.0;
        for (uint32_t c = 0; c < C; ++c) {
            const double p = exp((double)mcol[c * stride] - (double)bm) / z;
            if (p > 0.0) h -= p * log(p);
        }
        sc = h;
    } else {
        sc = 1.0 - 1.0 / z; // the largest probability is exp(0) / z
    }
    if (a.margins)
        for (uint32_t c = 0; c < C; ++c) a.margins[(size_t)i * C + c] = mcol[c * stride];
    a.pred[i] = (uint16_t)bc;
    a.score[i] = (float)sc;
    if (a.labels) a.labels[row] = (uint16_t)bc;
}

// A flow's result from its column of packed vote counters
__device__ __forceinline__ void vote_result(const FastArgs& a, const uint32_t* vcol, uint32_t stride, uint32_t i, uint32_t row,
                                            uint32_t& best, uint32_t& bestv)
{
    best = 0;
    bestv = 0;
    const uint32_t C = a.n_classes, per_shift = a.vote_bits == 8 ? 2u : 1u, vote_words = (C + (1u << per_shift) - 1u) >> per_shift;
    const uint32_t vmask = (1u << a.vote_bits) - 1u;
    for (uint32_t w = 0; w < vote_words; ++w) {
        const uint32_t word = vcol[w * stride];
        for (uint32_t k = 0; k < (1u << per_shift); ++k) {
            const uint32_t c = (w << per_shift) + k;
            if (c < C) {
                const uint32_t v = (word >> (k * a.vote_bits)) & vmask;
                if (a.votes) a.votes[(size_t)i * C + c] = (uint16_t)v;
                if (c == 0 || v > bestv) {
                    bestv = v;
                    best = c;
                }
            }
        }
    }
    a.pred[i] = (uint16_t)best;
    a.top[i] = (uint16_t)bestv;
    if (a.labels) a.labels[row] = (uint16_t)best;
}

// Shared memory of a block behind the feature tile xT ([n_features][FPB] floats, FPB flows per block):
// vote counters (or margins), then the staged top records.
// kIlp trees are walked at once per lane, kIlpTail in a last round when at most that many are left; EXACT: in that round just as
// many as are left (the walk alone in blocks of whole waves: 1,048,576 flows x 32 features, 4 trees of depth 13 on four lanes a
// flow 77 us against 62, 12 trees 155 against 120, 64 trees on eight lanes 1.06 times as long; not in small batches and in the
// fused kernel, where the longer kernel costs as much: 93 trees of depth 6 on 1,000 flows 5.1 us against 5.3).
// A block is FPB * W lanes; W lanes share one flow: group g = lane index / FPB.  With FPB a multiple of 64 a
// group is whole waves, so all lanes of a wave walk the same trees (their record gathers fall on the same few
// cache lines) and everything derived from the tree number is scalar.
// GBDT = false: leaves are class labels and the flow's result is the vote count per class; group g walks trees
// g, g + W, g + 2W, ...
// GBDT = true: leaves are binary32 margins; the flow's shared-memory column holds one binary32 sum per class,
// started at the initial margin and extended tree by tree in tree order (each addition rounded on its own, so
// the sums are reproducible bit for bit); group g owns the classes g, g + W, ... and walks their trees; the
// epilogue turns the sums into softmax probabilities in binary64 and into the score of Section 3.2.
// KEEP_ROWS: the fused form (see FastArgs::feat_out).
// i: the row of the outputs this lane's flow owns; row: its row in the feature matrix (subset form);
// live: false for lanes past the end (they walk a valid tile column and write nothing).
// The caller has filled xT (no barrier needed before the call: this function synchronises the block
// before the first read of the tile).
template <int FPB_, int W, int kIlp, int kIlpTail, bool EXACT, bool WANT_LEAF, bool GBDT, bool KEEP_ROWS>
__device__ __forceinline__ void forest_walk(const FastArgs& a, float* xT, uint32_t i, uint32_t row, bool live)
{
    constexpr uint32_t FPB = FPB_, BS = FPB * W; // flows and lanes per block
    constexpr uint32_t kColShift = FPB == 256 ? 10 : FPB == 128 ? 9 : FPB == 64 ? 8 : 6; // log2(bytes per feature column)
    static_assert((1u << kColShift) == 4u * FPB, "16, 64, 128 or 256 flows per block");
    const uint32_t F = a.n_features, C = a.n_classes, T = a.n_trees;
    const uint32_t top_recs = recs_upto(a.top_pairs);      // records per tree held in shared memory
    // vote counters, 32 / vote_bits classes per word, one column per FLOW: [vote_words][FPB]; the W lanes of
    // a flow add to it with shared-memory atomics (fields cannot carry into each other: a count is at most n_trees)
    const uint32_t per_shift = a.vote_bits == 8 ? 2u : 1u; // log2(counters per word)
    const uint32_t vote_words = GBDT ? C : (C + (1u << per_shift) - 1u) >> per_shift; // boosted: one float per class
    uint32_t* vT = reinterpret_cast<uint32_t*>(xT + (size_t)F * FPB);
    uint4* topT = reinterpret_cast<uint4*>(vT + (size_t)vote_words * FPB);   // [T][top_recs]
    const uint32_t tid = threadIdx.x;
    uint32_t grp = W == 1 ? 0u : tid / FPB;                // which share of the trees this lane walks
    if (FPB >= 64u) grp = __builtin_amdgcn_readfirstlane(grp);
    const uint32_t slot = tid % FPB;                       // flow slot in the block's tile
    if (GBDT) {
        for (uint32_t c = grp; c < C; c += W) vT[c * FPB + slot] = __float_as_uint(a.base ? a.base[c] : 0.f);
    } else {
        for (uint32_t c = grp; c < vote_words; c += W) vT[c * FPB + slot] = 0;
    }
    const uint32_t n_rec = recs_upto(pair_levels(a.depth));
    const uint4* recs = reinterpret_cast<const uint4*>(a.recs);
    for (uint32_t q = tid; q < T * top_recs; q += BS) {
        const uint32_t t = q / top_recs, r = q - t * top_recs;
        topT[q] = recs[(size_t)t * n_rec + r];
    }
    __syncthreads(); // the staged records and the feature columns are shared

    const uint32_t depth = a.depth;
    const uint32_t full_pairs = depth >> 1;
    const uint32_t lds_pairs = a.top_pairs < full_pairs ? a.top_pairs : full_pairs;
    const bool odd = depth & 1u;
    // The tile is read through absolute shared-memory addresses formed with bit operations: it heads the
    // block's shared memory, which in the kernels that use this walk is dynamic only, so the tile starts at
    // address 0 and "offset of the feature's row | offset of the flow's column" is the address.
    typedef __attribute__((address_space(3))) const float LdsFloat;
    const uint32_t tile_abs = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(xT);
    const uint32_t xl = tile_abs + slot * 4u; // address of the flow's column in the tile's first row
    uint32_t* vcol = vT + slot;
    const uint32_t rec_bytes = n_rec * 16u, top_bytes = top_recs * 16u;
    const uint32_t leaf_base = recs_upto(full_pairs); // record index of position 0 on tree level 2*full_pairs
    const uint32_t n_leaf = 1u << depth;

    // The three feature indices of a record sit in its last word as 8-bit fields, rotated so that the first
    // stands at bits 10..17: for a tile of 256 flows (a feature's row is 1024 bytes) masking the word gives
    // the byte offset of x[feature] in one operation, and a rotation by 8 or 16 bits brings a child's field
    // there.  Narrower tiles (two or four lanes per flow) rotate by one or two bits more.
    constexpr uint32_t kFieldMask = 0xFFu << kColShift;
    constexpr uint32_t kRot0 = kFeatRot - kColShift;
#define SF_FEAT_ROT(FW, SH) (*(LdsFloat*)(uintptr_t)((__builtin_amdgcn_alignbit((FW), (FW), (SH)) & kFieldMask) | xl))
#define SF_FEAT_0(FW) (kRot0 == 0u ? *(LdsFloat*)(uintptr_t)(((FW) & kFieldMask) | xl) : SF_FEAT_ROT(FW, kRot0))

    // Two visits from one record; o is the byte offset of the record inside its tree.  The child's feature is
    // fetched after the parent's test (two shared-memory reads per record, the second dependent on the first:
    // with this many waves resident fetching all three up front is no faster and costs registers).  The record
    // offset moves on as 4 * o + 16 * (1 + 2 * right0 + right1) = ((o + sh) << 2) - 16 + 16 * right1 with
    // sh = 8 or 16, the rotation that selects the child's feature field.
#define SF_PAIR_STEP(REC, O)                                                                              \
    do {                                                                                                  \
        const uint32_t fw = (REC).w;                                                                      \
        const float x0 = SF_FEAT_0(fw);                                                                   \
        const bool r0 = !(x0 <= __uint_as_float((REC).x));                                                \
        const uint32_t sh = r0 ? 16u : 8u;                                                                \
        const float tc = __uint_as_float(r0 ? (REC).z : (REC).y);                                         \
        const float xc = SF_FEAT_ROT(fw, sh + kRot0);                                                     \
        const bool rc = !(xc <= tc);                                                                      \
        (O) = (((O) + sh) << 2) + (rc ? 0u : 0xFFFFFFF0u);                                                \
    } while (0)

    // lane group g walks trees g, g+W, ... (boosted form: the trees of classes g, g+W, ...); every group runs
    // the same number of rounds so that the loop stays wave-uniform; a slot past the last tree repeats it and
    // does not vote
    const uint32_t my_classes = GBDT ? (C > grp ? (C - grp + W - 1u) / W : 0u) : 0u;
    uint32_t per_grp = GBDT && W > 1 ? (T + C - 1u) / C * ((C + W - 1u) / W) : (T + W - 1u) / W;
    if (FPB >= 64u && grp >= (GBDT ? C : T)) per_grp = 0; // (whole waves without a share)
    // one group: ILP trees from position q0 of the lane group's list
    auto walk_group = [&](auto ilp_tag, uint32_t q0) {
        constexpr int G = decltype(ilp_tag)::value;
        uint32_t o[G], tt[G], cls[G];
        bool tv[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            uint32_t t;
            if (GBDT && W > 1) {
                const uint32_t q = q0 + u, rnd = my_classes ? q / my_classes : 0u;
                cls[u] = grp + W * (q - rnd * my_classes);
                t = my_classes ? rnd * C + cls[u] : T;
            } else {
                t = (q0 + u) * W + grp;
            }
            o[u] = 0;
            tv[u] = q0 + u < per_grp && t < T;
            tt[u] = tv[u] ? t : T - 1u;
        }
        uint32_t j = 0;
        for (; j < lds_pairs; ++j) {
            uint4 rec[G];
#pragma unroll
            for (int u = 0; u < G; ++u)
                rec[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(topT) + tt[u] * top_bytes + o[u]);
#pragma unroll
            for (int u = 0; u < G; ++u) SF_PAIR_STEP(rec[u], o[u]);
        }
        const char* gb = reinterpret_cast<const char*>(a.recs);
        for (; j < full_pairs; ++j) {
            uint4 rec[G];
#pragma unroll
            for (int u = 0; u < G; ++u)
                rec[u] = *reinterpret_cast<const uint4*>(gb + (size_t)tt[u] * rec_bytes + o[u]);
#pragma unroll
            for (int u = 0; u < G; ++u) SF_PAIR_STEP(rec[u], o[u]);
        }
        uint32_t leaf[G];
        if (odd) {
            // one level left: only the record's top node counts
            uint4 rec[G];
#pragma unroll
            for (int u = 0; u < G; ++u)
                rec[u] = *reinterpret_cast<const uint4*>(gb + (size_t)tt[u] * rec_bytes + o[u]);
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const float x0 = SF_FEAT_0(rec[u].w);
                const bool r0 = !(x0 <= __uint_as_float(rec[u].x));
                leaf[u] = 2u * ((o[u] >> 4) - leaf_base) + (r0 ? 1u : 0u);
            }
        } else {
#pragma unroll
            for (int u = 0; u < G; ++u) leaf[u] = (o[u] >> 4) - leaf_base;
        }
        if (GBDT) {
            float val[G];
#pragma unroll
            for (int u = 0; u < G; ++u) val[u] = a.leaf_value[(size_t)tt[u] * n_leaf + leaf[u]];
#pragma unroll
            for (int u = 0; u < G; ++u) { // ascending u = ascending tree: the order of the sum
                if (tv[u]) {
                    float* m = reinterpret_cast<float*>(&vcol[(W > 1 ? cls[u] : tt[u] % C) * FPB]);
                    *m = *m + val[u];
                    if (WANT_LEAF && live) a.leaf_idx[(size_t)i * T + tt[u]] = (uint16_t)leaf[u];
                }
            }
            return;
        }
        uint32_t lab[G];
#pragma unroll
        for (int u = 0; u < G; ++u) lab[u] = a.leaf_label[(size_t)tt[u] * n_leaf + leaf[u]];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            if (tv[u]) {
                const uint32_t l = lab[u] < C ? lab[u] : C - 1u; // clamp: a bad label must not leave the tile
                // the flow's W lanes add to one column, from different waves: the add has to be atomic (one instruction)
                atomicAdd(&vcol[(l >> per_shift) * FPB], 1u << ((l & ((1u << per_shift) - 1u)) * a.vote_bits));
                if (WANT_LEAF && live) a.leaf_idx[(size_t)i * T + tt[u]] = (uint16_t)leaf[u];
            }
        }
    };
    {
        // A last round of up to kIlpTail trees runs as one of kIlpTail (a longer one as a full one with idle slots), with EXACT as
        // one of just as many trees: idle slots gather like the others.
        const uint32_t rem = per_grp % (uint32_t)kIlp;
        const bool short_tail = rem != 0 && rem <= (uint32_t)kIlpTail;
        const uint32_t full_end = short_tail ? per_grp - rem : per_grp;
        uint32_t q0 = 0;
        for (; q0 < full_end; q0 += kIlp) walk_group(std::integral_constant<int, kIlp>{}, q0);
        if (EXACT) {
            static_assert(!EXACT || (kIlpTail >= 1 && kIlpTail <= 5), "rounds of one to five trees");
            if (short_tail && rem == 1u) walk_group(std::integral_constant<int, 1>{}, q0);
            if (kIlpTail >= 2 && short_tail && rem == 2u) walk_group(std::integral_constant<int, 2>{}, q0);
            if (kIlpTail >= 3 && short_tail && rem == 3u) walk_group(std::integral_constant<int, 3>{}, q0);
            if (kIlpTail >= 4 && short_tail && rem == 4u) walk_group(std::integral_constant<int, 4>{}, q0);
            if (kIlpTail >= 5 && short_tail && rem == 5u) walk_group(std::integral_constant<int, 5>{}, q0);
        } else if (short_tail) {
            walk_group(std::integral_constant<int, kIlpTail>{}, q0);
        }
    }
#undef SF_PAIR_STEP
#undef SF_FEAT_0
#undef SF_FEAT_ROT
    if (W > 1) __syncthreads(); // all lanes of a flow have added their votes before its first lane reads them
    if (GBDT) {
        if (!live || grp != 0) return;
        boosted_result(a, reinterpret_cast<const float*>(vcol), FPB, i, row);
        return;
    }
    bool keep = false;
    if (live && grp == 0) {
        uint32_t best, bestv;
        vote_result(a, vT + slot, FPB, i, row, best, bestv);
        if (KEEP_ROWS) keep = bestv < a.vmin[a.n_vmin > 1u ? (best < a.n_vmin ? best : a.n_vmin - 1u) : 0u];
    }
    if (KEEP_ROWS) {
        // the features never left the chip: a row is written out only for a flow the gate hands on, each of the
        // flow's W lanes its share
        if (W > 1) {
            if (grp == 0) vT[slot] = keep ? 1u : 0u; // (the flow's first vote word: its only reader is done with it)
            __syncthreads();
            keep = vT[slot] != 0u;
        }
        if (keep) {
            float* dst = a.feat_out + (size_t)i * a.feat_out_ld;
            if (a.feat_out16) {
                for (uint32_t q = 4u * grp; q < F; q += 4u * W)
                    *reinterpret_cast<float4*>(dst + q) = make_float4(xT[(q + 0u) * FPB + slot], xT[(q + 1u) * FPB + slot],
                                                                    xT[(q + 2u) * FPB + slot], xT[(q + 3u) * FPB + slot]);
            } else {
                for (uint32_t q = grp; q < F; q += W) dst[q] = xT[q * FPB + slot];
            }
        }
    }
}

} // namespace sfforest
