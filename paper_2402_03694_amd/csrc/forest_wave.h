// The walk of forest_core.h in the form for large batches: a wave takes ONE tree at a time, for all flows of the
// block's tile (64 x U of them, U to a lane).
//
// Why: a record gather of a wave touches up to 64 cache lines, and with every lane of a wave on its own flow and the
// waves of a unit on dozens of different trees the lines a gather brings in are gone before another wave needs them:
// the walk waits for line fills.  Here a lane's U gathers of one level follow each other, through the same tree, and
// share their lines; what belongs to the tree and not to the flow is done once for all U:
//   - the tree's root record is read once (all lanes the same address) and its three feature rows are addressed once;
//   - the records of its first KW pair-levels pass through the wave's own window of shared memory, requested while the
//     tree before is walked (one coalesced load or two) and needing no barrier.  All trees get them there, however many
//     there are; the block-wide table of forest_walk holds fewer levels the more trees there are.
// The leaf's label (or margin) is added while the next tree's first levels are walked.
//
// The walk alone, before -> after: 1,048,576 flows x 64 features, 100 trees of depth 12 with splits drawn at random from the
// flows' values 435 -> 347 us, on the benchmark's workload 458 -> 400 to 416; x 32 features 363 -> 284; 4,194,304 x 128 features, 500 trees of depth
// 10 6.6 -> 4.9 ms; 65,536 flows, 200 trees of depth 10 48 -> 38 us; 20,011 flows x 96 features, 150 trees of depth 9 23 -> 19.5; boosted,
// 1,048,576 x 64, 200 trees of depth 8, ten classes 570 -> 413 us.  Which calls take it: waves_take and choose_waves (fast_infer.hip).
// What is left is shared memory (a feature read per visit) and vector arithmetic.  Tried and no better: scheduling barriers between
// the reads of a level's records, of its features and its tests; eight flows a lane; nine waves a block to make room for four pair-levels
// beside 256 flows of 64 features (337 us at 100 trees, but the trees rarely divide by nine).
#pragma once

#include "forest_core.h"

namespace sfforest {

// orders a wave's own shared-memory writes and reads (its instructions reach shared memory in program order)
__device__ __forceinline__ void window_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Shared memory of a block: tile (also the margins' place at the end), vote counters, the waves' windows.
inline size_t wave_walk_lds(uint32_t n_features, uint32_t result_words, bool gbdt, uint32_t flows, uint32_t waves, uint32_t window_levels)
{
    const size_t tile = gbdt ? (n_features > result_words ? n_features : result_words) : n_features + result_words;
    return tile * 4 * flows + (size_t)waves * recs_upto(window_levels) * 16;
}

// xT: [n_features][64 U] floats at the start of the block's shared memory, filled, a barrier behind it not needed.
// flow0: the block's first row; n: rows of the call.  A slot past the end holds a valid row's features and writes nothing.
// Voting form: any number of waves; wave w walks trees w, w + waves, ...; the trees left over after whole rounds are
// walked 64 flows at a time, so that all waves have a share of them.
// Boosted form: wave w owns class w (as many waves as classes): its margins stay in registers, extended tree by tree in
// tree order, each addition rounded on its own.
// KEEP_ROWS: the fused form (see FastArgs::feat_out); needs a number of waves that is a multiple of U.
template <int U, int KW, bool GBDT, bool KEEP_ROWS>
__device__ __forceinline__ void forest_walk_waves(const FastArgs& a, float* xT, uint32_t flow0, uint32_t n)
{
    constexpr uint32_t FPB = 64 * U;
    constexpr uint32_t kColShift = FPB == 256 ? 10 : FPB == 128 ? 9 : 8; // log2(bytes per feature column)
    static_assert((1u << kColShift) == 4u * FPB, "64, 128 or 256 flows per block");
    constexpr uint32_t kWin = (1u << (2 * KW)) / 3u; // records of KW pair-levels
    constexpr int KP = (int)((kWin + 63u) / 64u);    // loads that bring them
    const uint32_t F = a.n_features, C = a.n_classes, T = a.n_trees;
    const uint32_t per_shift = a.vote_bits == 8 ? 2u : 1u; // log2(counters per word)
    const uint32_t vote_words = (C + (1u << per_shift) - 1u) >> per_shift;
    const uint32_t waves = blockDim.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t* vT = reinterpret_cast<uint32_t*>(xT + (size_t)F * FPB); // voting form: [vote_words][FPB]
    uint4* windows = reinterpret_cast<uint4*>(xT + (size_t)(GBDT ? (F > C ? F : C) : F + vote_words) * FPB);
    uint4* win = windows + wave * kWin;
    if (!GBDT)
        for (uint32_t q = threadIdx.x; q < vote_words * FPB; q += waves * 64u) vT[q] = 0u;

    const uint32_t depth = a.depth, full_pairs = depth >> 1, levels = pair_levels(depth);
    const bool odd = depth & 1u;
    const uint32_t in_win = levels < (uint32_t)KW ? levels : (uint32_t)KW; // pair-levels in the window
    const uint32_t win_recs = recs_upto(in_win);
    const uint32_t win_pairs = in_win < full_pairs ? in_win : full_pairs;
    const uint32_t n_rec = recs_upto(levels), n_leaf = 1u << depth;
    const uint32_t leaf_base = recs_upto(full_pairs); // record index of position 0 on tree level 2 * full_pairs
    const uint4* recs = reinterpret_cast<const uint4*>(a.recs);

    // the tile heads the block's shared memory: "offset of the feature's row | offset of the flow's column" is the address,
    // and the flow's U columns are 256 bytes apart
    typedef __attribute__((address_space(3))) const float LdsFloat;
    const uint32_t tile_abs = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(xT);
    constexpr uint32_t kFieldMask = 0xFFu << kColShift;
    constexpr uint32_t kRot0 = kFeatRot - kColShift;
    auto row_of = [&](uint32_t fw, uint32_t sh, uint32_t xl) { // sh: 0, 8 or 16 + kRot0, the node's field
        return (__builtin_amdgcn_alignbit(fw, fw, sh) & kFieldMask) | xl;
    };
    auto x_at = [&](uint32_t addr, int u) { return ((LdsFloat*)(uintptr_t)addr)[64 * u]; };

    uint4 pre0, pre1; // the window of the tree that is walked next
    const uint32_t q0 = lane < win_recs ? lane : win_recs - 1u, q1 = lane + 64u < win_recs ? lane + 64u : win_recs - 1u;
    auto request = [&](uint32_t t) {
        const uint4* r = recs + (size_t)t * n_rec;
        pre0 = r[q0];
        if (KP > 1) pre1 = r[q1];
    };
    auto put = [&]() {
        window_sync(); // the tree before is done with the window
        win[q0] = pre0; // (lanes past the last record write that one once more)
        if (KP > 1) win[q1] = pre1;
        window_sync();
    };
    float acc[U];          // boosted form: the class's margins
    uint32_t pending[U];   // what the tree before gave: label, or margin as bits
    auto add_votes = [&](auto n_tag, uint32_t slot) {
        constexpr int N = decltype(n_tag)::value;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint32_t l = pending[u] < C ? pending[u] : C - 1u; // clamp: a bad label must not leave the tile
            // other waves add to the flow's column too: the add has to be atomic (one instruction)
            atomicAdd(&vT[(l >> per_shift) * FPB + slot + 64u * u], 1u << ((l & ((1u << per_shift) - 1u)) * a.vote_bits));
        }
    };
    auto add_margins = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = acc[u] + __uint_as_float(pending[u]);
    };
    // tree t for N flows a lane, the first of them at slot; between the window's levels and the rest, what the tree before left
    auto walk = [&](auto n_tag, uint32_t t, uint32_t slot, auto finish_before) {
        constexpr int N = decltype(n_tag)::value;
        const uint32_t xl = tile_abs + slot * 4u;
        const char* gb = reinterpret_cast<const char*>(recs + (size_t)t * n_rec);
        uint32_t o[N]; // byte offset of the flow's record inside its tree
        uint32_t j = 0;
        if (win_pairs) {
            const uint4 root = win[0];
            const uint32_t at0 = row_of(root.w, kRot0, xl), at1 = row_of(root.w, 8u + kRot0, xl), at2 = row_of(root.w, 16u + kRot0, xl);
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const bool r0 = !(x_at(at0, u) <= __uint_as_float(root.x));
                const bool rc = !(x_at(r0 ? at2 : at1, u) <= __uint_as_float(r0 ? root.z : root.y));
                o[u] = (r0 ? 48u : 16u) + (rc ? 16u : 0u);
            }
            j = 1;
        } else {
#pragma unroll
            for (int u = 0; u < N; ++u) o[u] = 0;
        }
        // two visits from one record each (see forest_walk)
        auto steps = [&](const uint4 (&rec)[N]) {
            float x0[N], xc[N];
            uint32_t sh[N];
#pragma unroll
            for (int u = 0; u < N; ++u) x0[u] = x_at(row_of(rec[u].w, kRot0, xl), u);
#pragma unroll
            for (int u = 0; u < N; ++u) {
                sh[u] = !(x0[u] <= __uint_as_float(rec[u].x)) ? 16u : 8u;
                xc[u] = x_at(row_of(rec[u].w, sh[u] + kRot0, xl), u);
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float tc = __uint_as_float(!(x0[u] <= __uint_as_float(rec[u].x)) ? rec[u].z : rec[u].y);
                o[u] = ((o[u] + sh[u]) << 2) + (!(xc[u] <= tc) ? 0u : 0xFFFFFFF0u);
            }
        };
        for (; j < win_pairs; ++j) {
            uint4 rec[N];
#pragma unroll
            for (int u = 0; u < N; ++u) rec[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(win) + o[u]);
            steps(rec);
        }
        finish_before();
        for (; j < full_pairs; ++j) {
            uint4 rec[N];
#pragma unroll
            for (int u = 0; u < N; ++u) rec[u] = *reinterpret_cast<const uint4*>(gb + o[u]);
            steps(rec);
        }
        uint32_t leaf[N];
        if (odd) { // one level left: only the record's top node counts
            uint4 rec[N];
            if (in_win > full_pairs) {
#pragma unroll
                for (int u = 0; u < N; ++u) rec[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(win) + o[u]);
            } else {
#pragma unroll
                for (int u = 0; u < N; ++u) rec[u] = *reinterpret_cast<const uint4*>(gb + o[u]);
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                leaf[u] = 2u * ((o[u] >> 4) - leaf_base) + (!(x_at(row_of(rec[u].w, kRot0, xl), u) <= __uint_as_float(rec[u].x)) ? 1u : 0u);
        } else {
#pragma unroll
            for (int u = 0; u < N; ++u) leaf[u] = (o[u] >> 4) - leaf_base;
        }
        if (GBDT) {
            const float* lv = a.leaf_value + (size_t)t * n_leaf;
#pragma unroll
            for (int u = 0; u < N; ++u) pending[u] = __float_as_uint(lv[leaf[u]]);
        } else {
            const uint8_t* ll = a.leaf_label + (size_t)t * n_leaf;
#pragma unroll
            for (int u = 0; u < N; ++u) pending[u] = ll[leaf[u]];
        }
    };
    constexpr std::integral_constant<int, U> all{};
    constexpr std::integral_constant<int, 1> one{};
    if (GBDT) {
        const uint32_t rounds = T > wave ? (T - wave - 1u) / C + 1u : 0u;
        if (rounds) request(wave);
        __syncthreads(); // the tile is filled
        const float b = a.base ? a.base[wave] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = b;
        for (uint32_t r = 0; r < rounds; ++r) {
            const uint32_t t = wave + r * C;
            put();
            request(r + 1u < rounds ? t + C : t);
            walk(all, t, lane, [&]() {
                if (r) add_margins();
            });
        }
        if (rounds) add_margins();
        __syncthreads(); // every wave is done with the tile: the margins take its place
#pragma unroll
        for (int u = 0; u < U; ++u) xT[wave * FPB + lane + 64u * u] = acc[u];
        __syncthreads();
        for (uint32_t s = threadIdx.x; s < FPB; s += waves * 64u) {
            const uint32_t i = flow0 + s;
            if (i < n) boosted_result(a, xT + s, FPB, i, i);
        }
        return;
    }
    {
        const uint32_t rounds = T / waves, left = T - rounds * waves, parts = left * U;
        const uint32_t first_left = rounds * waves;
        if (rounds || wave < parts) request(rounds ? wave : first_left + wave / U);
        __syncthreads(); // the tile is filled and the counters are cleared
        uint32_t before = 0; // 0: nothing pending, 1: a whole tree, 2: a part, of the flows at slot_before
        uint32_t slot_before = lane;
        auto finish = [&]() {
            if (before == 1u) add_votes(all, lane);
        };
        for (uint32_t r = 0; r < rounds; ++r) {
            const uint32_t t = wave + r * waves;
            put();
            request(r + 1u < rounds ? t + waves : wave < parts ? first_left + wave / U : t);
            walk(all, t, lane, finish);
            before = 1u;
        }
        finish();
        before = 0u;
        for (uint32_t k = wave; k < parts; k += waves) {
            put();
            const uint32_t k2 = k + waves;
            request(first_left + (k2 < parts ? k2 : k) / U);
            walk(one, first_left + k / U, lane + 64u * (k % U), [&]() {
                if (before) add_votes(one, slot_before);
            });
            before = 2u;
            slot_before = lane + 64u * (k % U);
        }
        if (before) add_votes(one, slot_before);
    }
    __syncthreads(); // all votes are in
    for (uint32_t s = threadIdx.x; s < FPB; s += waves * 64u) {
        const uint32_t i = flow0 + s;
        bool keep = false;
        if (i < n) {
            uint32_t row = i;
            if (a.idx) {
                row = a.idx[i];
                row = row < a.n_rows ? row : a.n_rows - 1u;
            }
            uint32_t best, bestv;
            vote_result(a, vT + s, FPB, i, row, best, bestv);
            if (KEEP_ROWS) keep = bestv < a.vmin[a.n_vmin > 1u ? (best < a.n_vmin ? best : a.n_vmin - 1u) : 0u];
        }
        if (KEEP_ROWS) vT[s] = keep ? 1u : 0u; // (the flow's first vote word: its only reader is done with it)
    }
    if (KEEP_ROWS) {
        // the features never left the chip: a row is written out only for a flow the gate hands on, by lanes of several waves
        __syncthreads();
        const uint32_t s = lane + 64u * (wave % U), share = wave / U, shares = waves / U;
        if (vT[s] != 0u) {
            float* dst = a.feat_out + (size_t)(flow0 + s) * a.feat_out_ld;
            if (a.feat_out16) {
                for (uint32_t q = 4u * share; q < F; q += 4u * shares)
                    *reinterpret_cast<float4*>(dst + q) =
                        make_float4(xT[(q + 0u) * FPB + s], xT[(q + 1u) * FPB + s], xT[(q + 2u) * FPB + s], xT[(q + 3u) * FPB + s]);
            } else {
                for (uint32_t q = share; q < F; q += shares) dst[q] = xT[q * FPB + s];
            }
        }
    }
}

} // namespace sfforest
