// The fused slow model on one row block of 32 rows, for lists that give a compute unit no more (up to 128 input values).  Nothing
// overlaps a block's tile there, so what counts is the chain from the row numbers to the label; what bounds it is the second
// layer's weights, half a megabyte through one unit's path to the cache.  So everything that does not depend on the rows is
// requested ahead of what does: the first layer's weights before the row numbers, the second layer's from the request for the rows
// on, through a ring of registers as deep as those allow, and the last layer's through the same ring.  Column blocks are dealt out to the waves in
// turn.  Each layer has its own place in shared memory, one barrier in between.  A row's logits are the same
// bits as in the tiles of run_tiles.  Whole call, half-height tile : this, us: 24 rows through 64-512-512-10 12.2 : 11.4, 8,000 15.5 : 13.3;
// 2,500 rows through 32-128-64-6 8.1 : 5.8; 5,000 through 96-300-200-7 10.8 : 9.0; 2,000 through 128-512-512-32 14.0 : 13.3.
#pragma once

#include "slow_tiles.h"

namespace sftiles {

constexpr int kFewRing = 8;        // k-steps of the weights in flight
constexpr uint32_t kFewInput = 128; // most input values
constexpr uint32_t kFewH = 32 * (kFewInput + 8) + 2 * 32 * LDH; // shared memory of the input and both hidden layers, in elements

// W waves; KS1: k-steps of the first layer (4 or 8); N1, N2: column blocks a wave of the first and second layer (1 or 2).  m.H holds kFewH elements.
template <int W, int KS1, int N1, int N2>
__device__ __forceinline__ void few_tile(const FusedArgs& a, const FusedSmem& m, uint32_t wave, uint32_t row0, uint32_t row_end)
{
    constexpr uint32_t kLdx = KS1 * 16 + 8;
    uint16_t *X = m.H, *H1 = X + 32 * kLdx, *H2 = H1 + 32 * LDH;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, at = weight_lane(lane);
    const uint32_t k2p = up(a.h1, kPadK), k3p = up(a.h2, kPadK), ks2 = k2p / 16u, ks3 = k3p / 16u;
    const uint32_t nb1 = up(a.h1, 32) / 32u, nb2 = up(a.h2, 32) / 32u;
    const bool whole = ((a.n_in | a.feat_ld) & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0;
    // (every wave makes the same number of requests, a block past the last one the last one's: the counter waits allow for all of
    // them only if they are not under branches)
    uint4 w1[KS1][N1], w2[kFewRing][N2];
    const uint4* p2[N2];
#pragma unroll
    for (int j = 0; j < N2; ++j) {
        const uint32_t nb = wave + W * j;
        p2[j] = a.w2s + (size_t)(nb < nb2 ? nb : nb2 - 1u) * ks2 * 64u + at;
    }
#pragma unroll
    for (int j = 0; j < N1; ++j) {
        const uint32_t nb = wave + W * j;
        const uint4* p1 = a.w1s + (size_t)(nb < nb1 ? nb : nb1 - 1u) * KS1 * 64u + at;
#pragma unroll
        for (int s = 0; s < KS1; ++s) w1[s][j] = p1[s * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr uint32_t kChunksRow = KS1 * 2; // pieces of eight input values in a row
    const uint32_t r = tid / kChunksRow, k = tid % kChunksRow * 8u;
    static_assert(32 * kChunksRow <= W * 64, "a piece a thread");
    const bool mine = tid < 32u * kChunksRow;
    const uint32_t row = row0 + (mine ? r : 0u);
    const bool there = mine && row < row_end;
    const uint32_t flow = clamp_row(a.esc_idx[row < row_end ? row : row0], a.n_rows);
    const uint32_t label_row = row0 + (lane & 31u), lr = label_row < row_end ? label_row : row0;
    const uint32_t dst = a.scatter ? a.scatter[lr] : clamp_row(a.esc_idx[lr], a.n_rows);
    // biases and input map, an entry a thread (a model without a map: any)
    static_assert(W * 64 == HMAX, "an entry a thread");
    const bool has_map = a.mu != nullptr;
    const uint32_t ki = tid < a.n_in ? tid : 0u;
    const float b1 = a.b1[tid < a.h1 ? tid : 0u], b2 = a.b2[tid < a.h2 ? tid : 0u], b3 = a.b3[tid < a.c ? tid : 0u];
    const float mu = (has_map ? a.mu : a.b1)[has_map ? ki : 0u], is = (has_map ? a.inv_sigma : a.b1)[has_map ? ki : 0u];
    float z[8];
    float4 x0, x1;
    const bool in0 = there && k < a.n_in, in1 = there && k + 4u < a.n_in;
    if (whole) {
        const float* p = a.feat + (size_t)flow * a.feat_ld;
        x0 = *reinterpret_cast<const float4*>(p + (in0 ? k : 0u));
        x1 = *reinterpret_cast<const float4*>(p + (in1 ? k + 4u : 0u));
    } else {
        load_chunk<false>(a, there ? flow : kNoFlow, k, z);
        x0 = make_float4(z[0], z[1], z[2], z[3]);
        x1 = make_float4(z[4], z[5], z[6], z[7]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kFewRing; ++s) {
        const uint32_t ks = (uint32_t)s < ks2 ? s : ks2 - 1u;
#pragma unroll
        for (int j = 0; j < N2; ++j) w2[s][j] = p2[j][ks * 64u];
    }
    __builtin_amdgcn_sched_barrier(0);
    m.s_b1[tid] = tid < a.h1 ? b1 : 0.f;
    m.s_b2[tid] = tid < a.h2 ? b2 : 0.f;
    if (tid < 32u) m.s_b3[tid] = tid < a.c ? b3 : 0.f;
    m.s_mu[tid] = has_map && tid < a.n_in ? mu : 0.f;
    m.s_is[tid] = has_map && tid < a.n_in ? is : 1.f;
    __syncthreads();
    z[0] = in0 ? x0.x : 0.f, z[1] = in0 ? x0.y : 0.f, z[2] = in0 ? x0.z : 0.f, z[3] = in0 ? x0.w : 0.f;
    z[4] = in1 ? x1.x : 0.f, z[5] = in1 ? x1.y : 0.f, z[6] = in1 ? x1.z : 0.f, z[7] = in1 ? x1.w : 0.f;
    if (mine) store_chunk(has_map, m.s_mu, m.s_is, a.clamp, X + r * kLdx + k, k, z);
    __syncthreads();

    f32x16 acc[2][1][1];
#pragma unroll
    for (int j = 0; j < N1; ++j) bias_acc<1, 1>(acc[j], m.s_b1, (wave + W * j) * 32u, lane);
    {
        const uint16_t* arow = X + (lane & 31u) * kLdx + 8u * (lane >> 5);
#pragma unroll
        for (int s = 0; s < KS1; ++s) {
            const bf16x8 fa = as_frag(*reinterpret_cast<const uint4*>(arow + s * 16));
#pragma unroll
            for (int j = 0; j < N1; ++j) acc[j][0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(w1[s][j]), fa, acc[j][0][0], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < N1; ++j) store_hidden<1, 1>(H1, acc[j], (wave + W * j) * 32u, k2p, nb1, lane);
    __syncthreads();
    {
#pragma unroll
        for (int j = 0; j < N2; ++j) bias_acc<1, 1>(acc[j], m.s_b2, (wave + W * j) * 32u, lane);
        const uint16_t* arow = H1 + (lane & 31u) * LDH + 8u * (lane >> 5);
        for (uint32_t k0 = 0; k0 < ks2; k0 += kFewRing) { // (ks2 is a multiple of 4)
            // refills: further down, then the last layer's first k-steps, N2 s + j in w2[s][j] (for the first wave; the others: anything)
            const bool more = k0 + kFewRing < ks2;
#pragma unroll
            for (int s0 = 0; s0 < kFewRing; s0 += 4) {
                if (k0 + s0 < ks2) {
                    uint4 fa[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) fa[q] = *reinterpret_cast<const uint4*>(arow + (k0 + s0 + q) * 16u);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int j = 0; j < N2; ++j)
                            acc[j][0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(w2[s0 + q][j]), as_frag(fa[q]), acc[j][0][0], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = s0; s < s0 + 4; ++s)
#pragma unroll
                    for (int j = 0; j < N2; ++j) {
                        const uint32_t ks = k0 + s + kFewRing, k3 = wave == 0 ? N2 * s + j : 0u;
                        const uint4* p = more ? p2[j] + (size_t)(ks < ks2 ? ks : ks2 - 1u) * 64u : a.w3s + (k3 < ks3 ? k3 : ks3 - 1u) * 64u + lane;
                        w2[s][j] = *p;
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int j = 0; j < N2; ++j) store_hidden<1, 1>(H2, acc[j], (wave + W * j) * 32u, k3p, nb2, lane);
    }
    __syncthreads();
    if (wave != 0) return;
    f32x16 c3;
#pragma unroll
    for (int v = 0; v < 16; ++v) c3[v] = m.s_b3[8u * (v >> 2) + 4u * (lane >> 5) + (v & 3)];
    const uint16_t* arow = H2 + (lane & 31u) * LDH + 8u * (lane >> 5);
    constexpr int kRing3 = kFewRing * N2;
    for (uint32_t k0 = 0; k0 < ks3; k0 += kRing3) { // (ks3 is a multiple of 4)
#pragma unroll
        for (int s0 = 0; s0 < kRing3; s0 += 4) {
            if (k0 + s0 < ks3) {
                uint4 fa[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) fa[q] = *reinterpret_cast<const uint4*>(arow + (k0 + s0 + q) * 16u);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(w2[(s0 + q) / N2][(s0 + q) % N2]), as_frag(fa[q]), c3, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = s0; q < s0 + 4; ++q) {
                const uint32_t ks = k0 + q + kRing3;
                w2[q / N2][q % N2] = a.w3s[(ks < ks3 ? ks : ks3 - 1u) * 64u + lane];
            }
        }
    }
    // the accumulator is transposed: lane l holds 16 classes of row l%32, lane l^32 the others
    const bool row_ok = label_row < row_end;
    uint32_t best = 4u * (lane >> 5);
    float bv = label_start(lane >> 5, c3[0]);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint32_t c = 8u * (v >> 2) + 4u * (lane >> 5) + (v & 3); // ascending in v
        const float y = c3[v];
        if (c < a.c) {
            if (a.logits && row_ok) a.logits[(size_t)label_row * a.c + c] = y;
            if (y > bv) {
                bv = y;
                best = c;
            }
        }
    }
    best = label_of(best, bv);
    if (lane < 32u && row_ok && dst < a.n_labels) a.labels[dst] = (uint16_t)best;
}

} // namespace sftiles
