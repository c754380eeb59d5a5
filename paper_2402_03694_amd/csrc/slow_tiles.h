// Tiles of the fused slow model: a block takes 32 to 128 rows through all three layers, its waves splitting the columns
// (512 of a hidden layer at most), the activations in shared memory.  Shared by the kernel that does nothing else
// (slow_fused.hip) and by the register form (slow_rows.hip), which ends a run of rows with such a tile.
#pragma once

#include <type_traits>

#include "mlp_common.h"
#include "slow_label.h"

namespace sftiles {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int FBM = 128;      // rows per tile
constexpr int HMAX = 512;     // widest hidden layer
constexpr int LDH = HMAX + 8; // activation row stride in elements
constexpr uint32_t kPadK = 64; // every K is padded to this (four k-steps of 16)

__host__ __device__ inline uint32_t up(uint32_t x, uint32_t m) { return (x + m - 1u) / m * m; }

struct FusedArgs {
    const uint32_t* esc_idx;  // row e reads feature row esc_idx[e] (clamped below n_rows) ...
    const uint32_t* scatter;  // ... and its label goes to labels[scatter[e]]; NULL = the same index
    const uint32_t* esc_count;
    uint32_t esc_cap;
    uint32_t n_rows, n_labels;
    const float* feat;
    uint32_t feat_ld;
    const float* mu;
    const float* inv_sigma;
    float clamp;
    uint32_t n_in, h1, h2, c;
    const uint4* w1s; // operand-ordered weights, see reorder_weights
    const uint4* w2s;
    const uint4* w3s;
    const float *b1, *b2, *b3;
    float* logits;
    uint16_t* labels;
    const uint16_t* pred; // labels of the flows that are not on the list, copied by the grid's first blocks; NULL = they stay
    uint32_t n_copy;      // blocks that copy
};

__device__ __forceinline__ bf16x8 as_frag(uint4 u)
{
    union {
        uint4 u;
        bf16x8 b;
    } c;
    c.u = u;
    return c.b;
}

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// two floats -> two bfloat16 (round to nearest even) in one word
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    union {
        bf16x2 b;
        uint32_t u;
    } c;
    c.b = __builtin_convertvector(v, bf16x2);
    return c.u;
}

// relu of two floats as bfloat16.  (One maximum with zero: fmaxf would pass its operand through another one first.  What lies
// past the largest finite number becomes the bfloat16 infinity all the same, NaN zero as in fmaxf.)
__device__ __forceinline__ uint32_t relu_pair(float lo, float hi)
{
    return pack_bf16(__builtin_amdgcn_fmed3f(lo, 0.f, 3.402823466e38f), __builtin_amdgcn_fmed3f(hi, 0.f, 3.402823466e38f));
}

constexpr int kMI = 4;     // 32-row blocks of the tallest tile (128 rows)
constexpr int kRing = 4;   // weight operands of this many k-steps are in flight (K is padded to 16 * kRing)

__device__ __forceinline__ uint32_t weight_lane(uint32_t lane) { return (lane & ~12u) | ((lane & 4u) << 1) | ((lane & 8u) >> 1); }

// A logit is one sum, from its bias on in order of K, in the tiles as in the passes of the register form: a row's logits do not depend
// on where in a list it stands, nor on the list's capacity or the input's alignment, which decide between the forms.
// W: waves of the block, NI: 32-column blocks per wave (W * NI up to 16), MI: 32-row blocks of the tile

// first kRing k-steps of a wave's weight operands (column blocks nb0 .. nb0+NI, clamped to the last real one)
template <int NI>
__device__ __forceinline__ void ring_fill(uint4 (&fb)[kRing][NI], const uint4* __restrict__ ws, uint32_t KS, uint32_t nb0,
                                          uint32_t nb_total, uint32_t lane)
{
    const uint32_t wl = weight_lane(lane);
#pragma unroll
    for (int s = 0; s < kRing; ++s) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const uint32_t nb = nb0 + j < nb_total ? nb0 + j : nb_total - 1u;
            fb[s][j] = ws[((size_t)nb * KS + s) * 64u + wl];
        }
        // ring order: the counter wait in front of an MFMA is placed for the worst order on any path
        // into the loop, and a fill issued out of order makes every k-step wait for the newest load
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The MFMA is issued with the WEIGHT operand first, so the 32x32 accumulator block holds the output transposed: element v
// of lane l belongs to activation row l%32 and to row 8*(v/4) + 4*(l/32) + v%4 of the weight operand.  A lane reads the weights of
// the lane whose number has bits 2 and 3 exchanged, which makes that column 16*(v/8) + 8*(l/32) + v%8: eight consecutive v are
// eight consecutive columns of one row, as the next layer's operand has them, and the epilogue writes 16 bytes at a time.
// acc[i][j] += W[cols of block nb0+j][K] * A[rows 32i..32i+32)[K]^T, KS a multiple of kRing.
// The weight operands sit in a ring of kRing register buffers; a buffer is refilled for k-step
// ks + kRing right after the MFMAs of k-step ks have been issued, so no load is waited for in the
// step that issues it and no register is copied.
// fb holds k-steps 0 .. kRing-1 of this layer on entry.  The last kRing refills of the loop fetch the
// first k-steps of the NEXT GEMM (operand array nws, nKS k-steps per column block, nnb_total column
// blocks), so that one starts without waiting for memory: its operands arrive during the epilogue
// in between.
template <int NI, int MI>
__device__ __forceinline__ void wave_gemm(const uint16_t* A, uint32_t lda, const uint4* __restrict__ ws, uint32_t KS,
                                          uint32_t nb0, uint32_t nb_total, uint32_t lane, f32x16 (&acc)[MI][NI],
                                          uint4 (&fb)[kRing][NI], const uint4* __restrict__ nws, uint32_t nKS,
                                          uint32_t nnb_total)
{
    if (nb0 >= nb_total) { // this wave has no columns in this layer
        ring_fill(fb, nws, nKS, nb0, nnb_total, lane);
        return;
    }
    const uint16_t* arow = A + (lane & 31u) * lda + 8u * (lane >> 5);
    const uint32_t at = weight_lane(lane);
    // a column block past the end repeats the last one; its results are never used
    const uint4 *wl[NI], *nwl[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const uint32_t nb = nb0 + j < nb_total ? nb0 + j : nb_total - 1u;
        wl[j] = ws + (size_t)nb * KS * 64u;
        const uint32_t nnb = nb0 + j < nnb_total ? nb0 + j : nnb_total - 1u;
        nwl[j] = nws + (size_t)nnb * nKS * 64u;
    }
    // the activation operands are double-buffered too: those of k-step ks+1 are read from shared
    // memory before the MFMAs of k-step ks are issued (H has 8 columns of padding, so the read
    // one step past the end stays inside the row)
    uint4 fa[2][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[0][i] = *reinterpret_cast<const uint4*>(arow + (size_t)i * 32u * lda);
    for (uint32_t k0 = 0; k0 < KS; k0 += kRing) {
        // where this round's refills come from: further down this layer, or the start of the next
        // GEMM (a select between wave-uniform pointers: no branch around the loads, which would
        // make the counter waits drain the ring)
        const bool more = k0 + kRing < KS;
        const uint4* src[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) src[j] = more ? wl[j] + (size_t)(k0 + kRing) * 64u : nwl[j];
#pragma unroll
        for (int s = 0; s < kRing; ++s) {
            const uint32_t kn = k0 + s + 1u < KS ? k0 + s + 1u : k0 + s;
#pragma unroll
            for (int i = 0; i < MI; ++i)
                fa[(s + 1) & 1][i] = *reinterpret_cast<const uint4*>(arow + (size_t)i * 32u * lda + kn * 16u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const bf16x8 b = as_frag(fb[s][j]);
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, as_frag(fa[s & 1][i]), acc[i][j], 0, 0, 0);
            }
            // refill for k-step k0 + s + kRing (or k-step s of the next GEMM)
#pragma unroll
            for (int j = 0; j < NI; ++j) fb[s][j] = src[j][s * 64u + at];
            // keep the refill here: left alone, the scheduler sinks it to just before its use
            // (to save registers) and every k-step then waits a full memory latency
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// H[row][col] = bfloat16(relu(acc)) for the wave's columns (the bias is already in acc).  Padding columns
// [n_valid, n_pad) inside the last real 32-column block come out as zeros by themselves (their weights and
// bias entries are zero); a column block past the last real one (nb_total) holds a repeat of that block's
// results in acc and is stored as zeros.
template <int NI, int MI>
__device__ __forceinline__ void store_hidden(uint16_t* H, const f32x16 (&acc)[MI][NI], uint32_t n0, uint32_t n_pad,
                                             uint32_t nb_total, uint32_t lane)
{
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const bool real = n0 / 32u + j < nb_total;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t col = n0 + j * 32u + 16u * e + 8u * (lane >> 5); // first of 8 consecutive columns
            if (col < n_pad) {
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const uint32_t row = i * 32u + (lane & 31u);
                    uint32_t y[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) y[q] = relu_pair(acc[i][j][8 * e + 2 * q], acc[i][j][8 * e + 2 * q + 1]);
                    *reinterpret_cast<uint4*>(H + row * LDH + col) = real ? make_uint4(y[0], y[1], y[2], y[3]) : make_uint4(0u, 0u, 0u, 0u);
                }
            }
        }
    }
}

// accumulators start at the bias of their column, so the epilogue has no add
template <int NI, int MI>
__device__ __forceinline__ void bias_acc(f32x16 (&acc)[MI][NI], const float* sbias, uint32_t n0, uint32_t lane)
{
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t col = n0 + j * 32u + 16u * (g >> 1) + 8u * (lane >> 5) + 4u * (g & 1);
            const float4 b = col < (uint32_t)HMAX ? *reinterpret_cast<const float4*>(sbias + col) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                acc[i][j][4 * g + 0] = b.x;
                acc[i][j][4 * g + 1] = b.y;
                acc[i][j][4 * g + 2] = b.z;
                acc[i][j][4 * g + 3] = b.w;
            }
        }
}

constexpr uint32_t kNoFlow = 0xFFFFFFFFu;
// a bad list entry must not leave the feature matrix
__device__ __forceinline__ uint32_t clamp_row(uint32_t f, uint32_t n_rows) { return f < n_rows ? f : n_rows - 1u; }
// 8-value input chunks a thread can hold in registers for the next tile
template <int W>
constexpr int kChunks = 16 / W;

// raw feature values [k, k+8) of one flow (zeros for a missing flow or past n_in)
// WHOLE: rows in whole 16-byte elements, and no branch: a thread's requests go out together, not one after the other's arrival
template <bool WHOLE>
__device__ __forceinline__ void load_chunk(const FusedArgs& a, uint32_t flow, uint32_t k, float (&z)[8])
{
    const bool there = flow != kNoFlow;
    const float* p = a.feat + (size_t)(there ? flow : 0u) * a.feat_ld;
    if (WHOLE) {
        const bool in0 = k < a.n_in, in1 = k + 4u < a.n_in;
        const float4 x0 = *reinterpret_cast<const float4*>(p + (in0 ? k : 0u)), x1 = *reinterpret_cast<const float4*>(p + (in1 ? k + 4u : 0u));
        const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) z[q] = there && (q < 4 ? in0 : in1) ? x[q] : 0.f;
        return;
    }
    p += k;
    if (there && k + 8u <= a.n_in && (a.feat_ld & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0) {
        const float4 x0 = reinterpret_cast<const float4*>(p)[0], x1 = reinterpret_cast<const float4*>(p)[1];
        z[0] = x0.x; z[1] = x0.y; z[2] = x0.z; z[3] = x0.w;
        z[4] = x1.x; z[5] = x1.y; z[6] = x1.z; z[7] = x1.w;
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) z[q] = there && k + q < a.n_in ? p[q] : 0.f;
    }
}

// standardise, clamp, round to bfloat16 and store one chunk of the input tile
// (s_mu / s_is: the input map in shared memory, zero / one past n_in; has_map false = identity)
__device__ __forceinline__ void store_chunk(bool has_map, const float* s_mu, const float* s_is, float clamp,
                                            uint16_t* dst, uint32_t k, float (&z)[8])
{
    if (has_map) {
        const float4 m0 = *reinterpret_cast<const float4*>(s_mu + k), m1 = *reinterpret_cast<const float4*>(s_mu + k + 4);
        const float4 i0 = *reinterpret_cast<const float4*>(s_is + k), i1 = *reinterpret_cast<const float4*>(s_is + k + 4);
        const float mu[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
        const float is[8] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float d = z[q] - mu[q];
            float t = d * is[q];
            t = t < -clamp ? -clamp : t;
            z[q] = t > clamp ? clamp : t;
        }
    }
    *reinterpret_cast<uint4*>(dst) =
        make_uint4(pack_bf16(z[0], z[1]), pack_bf16(z[2], z[3]), pack_bf16(z[4], z[5]), pack_bf16(z[6], z[7]));
}

// Tile schedule of run_tiles (one block, W waves, n_tiles consecutive tiles of MI row blocks):
//   top        the input tile is written from registers that were loaded during the previous
//              tile's last layer; the flow ids of the NEXT tile are requested
//   layer 1    MFMA, then the next tile's flow ids are parked in shared memory, epilogue -> H
//   layer 2    MFMA, epilogue -> H; the last layer's weight operands are requested
//   layer 3    the next tile's feature rows are requested (they arrive while layer 3 runs);
//              a wave takes a row block (waves beyond MI idle)
// Rows from row_end on belong to another block (or do not exist): they read as zeros and nothing of
// theirs is stored.
struct FusedSmem {
    uint16_t* H;      // [32 MI][LDH]; also the input tile
    uint32_t* s_flow; // [2][128]: this tile, next tile
    float *s_b1, *s_b2, *s_b3, *s_mu, *s_is;
};

template <int W, int NI, int MI>
__device__ __forceinline__ void run_tiles(const FusedArgs& a, const FusedSmem& m, uint32_t wave, uint32_t row_begin,
                                          uint32_t n_tiles, uint32_t row_end)
{
    constexpr uint32_t TM = MI * 32u; // rows per tile
    constexpr int kXr = kChunks<W>;
    constexpr int kW3 = HMAX / 16; // weight operands of the last layer
    static_assert(W >= MI && W * NI <= 16, "a wave for every row block, 512 columns at most");
    uint16_t* H = m.H;
    uint32_t* s_flow = m.s_flow;
    const uint32_t k1p = up(a.n_in, kPadK), k2p = up(a.h1, kPadK), k3p = up(a.h2, kPadK);
    const uint32_t ldx = k1p + 8; // input tile row stride
    const uint32_t n0 = wave * 32u * NI;
    const uint32_t nb1 = up(a.h1, 32) / 32u, nb2 = up(a.h2, 32) / 32u;
    const uint32_t chunks = k1p / 8u;
    const bool in_regs = TM * chunks <= (uint32_t)kXr * W * 64u; // the whole input tile fits the threads' registers
    const bool whole = ((a.n_in | a.feat_ld) & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0;
    const bool has_map = a.mu != nullptr;
    float xr[kXr][8];
    auto request_rows = [&](const uint32_t* flows, uint32_t tid) {
        auto each = [&](auto w) {
#pragma unroll
            for (int u = 0; u < kXr; ++u) {
                const uint32_t g = tid + u * W * 64u, r = g / chunks, k = (g - r * chunks) * 8u;
                load_chunk<decltype(w)::value>(a, r < TM ? flows[r] : kNoFlow, k, xr[u]);
            }
        };
        if (whole)
            each(std::true_type{});
        else
            each(std::false_type{});
    };
    // weight operands of layer 1's first k-steps; from here on every GEMM leaves the ring filled for the next one
    uint4 fb[kRing][NI];
    ring_fill(fb, a.w1s, k1p / 16u, wave * NI, nb1, threadIdx.x & 63u);
    __syncthreads(); // the previous run of tiles (if any) is done with the tile and the flow ids
    {
        // first tile: flow ids and feature rows are fetched here, with nothing to overlap them
        // (the lane index behind an opaque barrier, as in the loop: nothing computed from it here is shared
        // with, and kept alive across, another run of tiles)
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if (tid < TM) s_flow[tid] = row_begin + tid < row_end ? clamp_row(a.esc_idx[row_begin + tid], a.n_rows) : kNoFlow;
        __syncthreads();
        if (in_regs) request_rows(s_flow, tid);
    }
    uint32_t cur = 0;
    for (uint32_t ti = 0; ti < n_tiles; ++ti) {
        const uint32_t row0 = row_begin + ti * TM;
        const uint32_t next_row0 = row0 + TM;
        const bool has_next = ti + 1u < n_tiles;
        // Re-read the lane index behind an opaque barrier in every tile: otherwise every per-lane
        // address of the tile body is hoisted out of this loop and spilled around the MFMA loops.
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t lane = tid & 63u;
        const uint32_t* flow_cur = s_flow + cur * FBM;
        uint32_t* flow_next = s_flow + (cur ^ 1u) * FBM;
        // flow ids of the next tile: requested now, parked in shared memory after layer 1
        uint32_t nf = kNoFlow;
        if (has_next && tid < TM && next_row0 + tid < row_end) nf = clamp_row(a.esc_idx[next_row0 + tid], a.n_rows);
        // input tile of this tile (H is free: the previous tile's last layer ended with a barrier)
        if (in_regs) {
#pragma unroll
            for (int u = 0; u < kXr; ++u) {
                const uint32_t g = tid + u * W * 64u, r = g / chunks, k = (g - r * chunks) * 8u;
                if (r < TM) store_chunk(has_map, m.s_mu, m.s_is, a.clamp, H + r * ldx + k, k, xr[u]);
            }
        } else {
            for (uint32_t g = tid; g < TM * chunks; g += W * 64u) {
                const uint32_t r = g / chunks, k = (g - r * chunks) * 8u;
                float z[8];
                load_chunk<false>(a, flow_cur[r], k, z);
                store_chunk(has_map, m.s_mu, m.s_is, a.clamp, H + r * ldx + k, k, z);
            }
        }
        __syncthreads();

        f32x16 acc[MI][NI];
        // layer 1
        bias_acc<NI, MI>(acc, m.s_b1, n0, lane);
        wave_gemm<NI, MI>(H, ldx, a.w1s, k1p / 16u, wave * NI, nb1, lane, acc, fb, a.w2s, k2p / 16u, nb2);
        __syncthreads(); // every wave has read the input tile; H may be overwritten
        if (tid < TM) flow_next[tid] = nf;
        store_hidden<NI, MI>(H, acc, n0, k2p, nb1, lane);
        __syncthreads();
        // layer 2
        bias_acc<NI, MI>(acc, m.s_b2, n0, lane);
        // (the ring goes on to layer 1 of the next tile; after the last tile the fetch is not used)
        wave_gemm<NI, MI>(H, LDH, a.w2s, k2p / 16u, wave * NI, nb2, lane, acc, fb, a.w1s, k1p / 16u, nb1);
        __syncthreads();
        store_hidden<NI, MI>(H, acc, n0, k3p, nb2, lane);
        // layer 3: wave = row block.  The hidden accumulators are dead, so all its weight operands fit in registers; they are
        // requested before the barrier so that their latency overlaps it.  Behind the barrier the next tile's feature rows are requested,
        // consumed at the top of the next iteration.  The waves beyond MI have a branch of their own (with the two parts that are
        // theirs under branches instead, the operands cost registers in all of it).
        if (wave >= (uint32_t)MI) {
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            if (has_next && in_regs) request_rows(flow_next, tid);
            __syncthreads();
        } else {
            const uint32_t KS3 = k3p / 16u; // a multiple of 4
            uint4 wv[kW3];
#pragma unroll
            for (int g = 0; g < kW3 / 4; ++g) {
                const uint4* w = a.w3s + (4u * g < KS3 ? 4u * g : KS3 - 4u) * 64u + lane;
#pragma unroll
                for (int q = 0; q < 4; ++q) wv[4 * g + q] = w[q * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            if (has_next && in_regs) request_rows(flow_next, tid);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 c3;
#pragma unroll
            for (int v = 0; v < 16; ++v) c3[v] = m.s_b3[8u * (v >> 2) + 4u * (lane >> 5) + (v & 3)];
            const uint16_t* arow = H + (wave * 32u + (lane & 31u)) * LDH + 8u * (lane >> 5);
            // the activation operands of two k-steps are read while the two before are multiplied
            auto read2 = [&](uint4 (&f)[2], int s3) {
#pragma unroll
                for (int q = 0; q < 2; ++q) f[q] = *reinterpret_cast<const uint4*>(arow + (s3 + q) * 16);
            };
            uint4 fa[2][2];
            read2(fa[0], 0);
#pragma unroll
            for (int s3 = 0; s3 < kW3; s3 += 2) {
                if ((uint32_t)(s3 & ~3) >= KS3) continue;
                if (s3 + 2 < kW3) read2(fa[(s3 / 2 + 1) & 1], s3 + 2); // (past the layer's K: not used)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(wv[s3 + q]), as_frag(fa[(s3 / 2) & 1][q]), c3, 0, 0, 0);
            }
            __syncthreads(); // also: every wave is done reading H
            // the accumulator is transposed: lane l holds 16 classes of row l%32, lane l^32 the others
            const uint32_t r = wave * 32u + (lane & 31u);
            const bool row_ok = row0 + r < row_end;
            uint32_t best = 4u * (lane >> 5);
            float bv = label_start(lane >> 5, c3[0]);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t c = 8u * (v >> 2) + 4u * (lane >> 5) + (v & 3); // ascending in v
                const float y = c3[v];
                if (c < a.c) {
                    if (a.logits && row_ok) a.logits[(size_t)(row0 + r) * a.c + c] = y;
                    if (y > bv) {
                        bv = y;
                        best = c;
                    }
                }
            }
            best = label_of(best, bv);
            if (lane < 32u && row_ok) {
                const uint32_t dst = a.scatter ? a.scatter[row0 + r] : flow_cur[r];
                if (dst < a.n_labels) a.labels[dst] = (uint16_t)best;
            }
        }
        cur ^= 1u;
    }
}

} // namespace sftiles
