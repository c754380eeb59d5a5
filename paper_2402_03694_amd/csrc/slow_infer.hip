// Step 5: the slow model on the escalated flows only; its label replaces the fast one
// (Sections 3.1 and 4.4 of the paper).  The slow model is a 3-layer ReLU MLP.
//
// bfloat16 models run on the matrix cores: each layer is one tiled GEMM
// C[rows][N] = act(A[rows][K] * W[N][K]^T + b) built from 32x32x16 MFMA blocks with binary32
// accumulators.  Both operands are contiguous along K, which is exactly what an MFMA operand
// wants (each lane supplies 8 consecutive K values of one row or column).  The first layer
// builds its A tile on the fly from the escalated flows' feature rows (gather through the
// index list, standardise, clamp, round to bfloat16) or from packed header bits; the last
// layer adds the bias, finds the arg-max per row and scatters the label to the flow's slot.
// The row count comes from the device-side escalation count; blocks past it exit.
//
// binary32 models (small, used for the small workload) run on plain vector arithmetic.
#include <type_traits>

#include "mlp_common.h"
#include "slow_label.h"
#include "small_batch.h"

namespace sf {
// fused single-kernel form for narrow hidden layers (slow_fused.hip)
bool slow_fused_ok(const sf_mlp* mlp, bool raw_input);
size_t slow_fused_ws_bytes(const sf_mlp* mlp);
int slow_fused(sf_ctx* ctx, void* ws, bool ws_is_ordered, const float* feat, uint32_t feat_ld, uint32_t n_rows,
               const uint32_t* esc_idx, const uint32_t* scatter, const uint32_t* esc_count, uint32_t esc_cap,
               uint32_t n_labels, const sf_mlp* mlp, const uint16_t* pred, const sfsmall::GateRows* gate, float* logits, uint16_t* labels);
bool slow_fused_gates(sf_ctx* ctx, const sf_mlp* mlp, uint32_t n);
int copy_labels_async(sf_ctx* ctx, const uint16_t* pred, uint16_t* labels, uint32_t n);
int order_all(sf_ctx* ctx, const sf_mlp* mlp, void* out);
// one hidden layer of any width on operand-ordered weights (slow_wide.hip)
int wide_layer(sf_ctx* ctx, int amode, const sfmlp::LayerArgs& a, const void* w_ordered, uint32_t rows_cap);
uint32_t wide_blocks(const sf_ctx* ctx, uint32_t ldh, uint32_t rows_cap); // blocks of its launch
} // namespace sf

namespace {

using namespace sfmlp;

// The last layer of a wide model: logits = A * W3^T + b3 on bfloat16 activations (at most 64 classes), then the arg-max per row
// and the scatter of the label.  A logit is one chain of products in order of K, from zero on, and its bias at the end, whatever form
// makes it: mlp_wide_last (slow_wide.hip), which takes this layer along where it can, or one of the two here.
//   - Long lists: 256 rows a block (128 with more than 32 classes), a wave 32 of them, K walked by all waves together through shared memory in steps of two pieces
//     of 64, the next step requested ahead of the MFMAs.  What bounds it is HBM (200,000 rows of 2,048 values 216 us, 3.8 TB/s; straight
//     from the cache into registers, a row's operands are 32 lines to the address path, 270).
//   - Short ones: all waves of a block request the operands of 32 rows, a piece each and a round ahead, and put them into shared memory;
//     one wave multiplies.  What bounds it is the chain of latencies, and past a few blocks a unit that chain of MFMAs: 500 rows of 1,024 values
//     11.2 -> 6.1 us, 19,600 12.9 : 13.3.
//     Lists of up to three such blocks a unit go this way, two where the weights lie in rows (a block then gathers them line by
//     line), one with more than 32 classes; a block counts once for every 16 pieces (8 with more than 32 classes).  Short : long, whole call in
//     us: 12,546 rows through 32-256-1536-10 46.4 : 53.0, rows of weights 8,513 through 32-320-1536-4 44.4 : 48.7; 34,672 through 128-448-576-10,
//     4.2 blocks, 88.1 : 81.5, rows of weights 22,378 through 96-176-1042-16, 5.5, 79.2 : 69.4; 49 classes, 8,730 rows of 63 values, 42.2 : 38.2.
constexpr int LROWS = 32, LWAVES = 8, LPIECE = 64;
constexpr int LSTEP = 2 * LPIECE, LLDT = LSTEP + 8; // long lists: K of a step, row stride in shared memory
template <int NI> // 32-class blocks
struct LastShape {
    static constexpr int kTile = LWAVES * 32 / NI;  // long lists: rows of a block (33 to 64 classes: half the waves only load)
    static constexpr int kHeld = LWAVES / NI;       // short lists: pieces in shared memory at a time, a wave loads a piece's weights of 32 classes
    static constexpr int kRows = 4 / NI;            // ... and as many of the rows' four operands
    static constexpr size_t kShort = (size_t)kHeld * 4 * (1 + NI) * 1024, kLong = (size_t)(kTile + NI * 32) * LLDT * 2;
    static constexpr size_t kBias = kShort > kLong ? kShort : kLong; // the biases stand behind either
    static constexpr size_t kLds = kBias + NI * 32 * 4;
};

// The hidden layer before writes 128 rows a block, and blocks go to the eight dies in turn, each with a cache of its own.  A row is read
// on the die that wrote it: read on another, the next call's write of the same memory has that copy taken away first, and it is that
// launch which takes longer (13,544 rows through 64-576-6: 9.2 us, behind 32-row blocks in plain order 12.7).
constexpr uint32_t kDies = 8;
// first row of the 32 that block i of a short list takes; 32 blocks stand for eight row blocks of the layer before
__device__ __forceinline__ uint32_t short_rows(uint32_t i) { return (i / (kDies * 4u) * (kDies * 4u) + i % kDies * 4u + i / kDies % 4u) * LROWS; }
// first row of tile i of a long list: 128 rows from there on and, with tiles of 256, the 128 of the row block eight further on
template <int NI>
__device__ __forceinline__ uint32_t long_rows(uint32_t i) { return (NI == 1 ? i / kDies * (kDies * 2u) + i % kDies : i) * BM; }

// A tile of a long list (from r0 on, long_rows) by the whole block, K in steps of two pieces
template <int NI>
__device__ __forceinline__ void last_tile(const LayerArgs& a, uint32_t r0, uint32_t rows, unsigned char* smem, const float* s_bias, uint32_t tid, uint32_t lane, uint32_t wave)
{
    constexpr int LTILE = LastShape<NI>::kTile;
    static_assert(LTILE == (NI == 1 ? 2 : 1) * BM, "as long_rows has it");
    auto row_of = [=](uint32_t r) { return r0 + r + (r < (uint32_t)BM ? 0u : (kDies - 1u) * BM); }; // row r of the tile
    constexpr int kA = LTILE * LSTEP / 8 / (LWAVES * 64), kB = NI * 32 * LSTEP / 8 / (LWAVES * 64); // 16-byte pieces of a thread per step
    uint16_t *As = reinterpret_cast<uint16_t*>(smem), *Bs = As + LTILE * LLDT;
    const bool idle = NI > 1 && wave * 32u >= (uint32_t)LTILE; // (uniform)
    const uint32_t half = lane >> 5, r = (idle ? 0u : wave * 32u) + (lane & 31u); // this lane's row of the tile
    const uint32_t my_row = row_of(r), row = my_row < rows ? my_row : rows - 1u, dst = (a.scatter ? a.scatter : a.esc_idx)[a.row_begin + row];
    f32x16 y[NI]; // class 32 j + 8 * (v / 4) + 4 * half + v % 4
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) y[j][v] = 0.f;
    uint4 ra[kA], rb[kB];
    const uint32_t ck = tid % (LSTEP / 8) * 8u, cr = tid / (LSTEP / 8); // (rows of As: every 32nd from cr on)
    auto fetch = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < kA; ++u) { // (lda: whole pieces, zeros behind K; a row past the end: the last one again)
            const uint32_t q = row_of(cr + 32u * u);
            ra[u] = k0 + ck < a.lda ? *reinterpret_cast<const uint4*>(a.a_bf16 + (size_t)(q < rows ? q : rows - 1u) * a.lda + k0 + ck) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) rb[u] = weight_chunk(a.w, a.N, a.K, cr + 32u * u, k0 + ck);
    };
    fetch(0);
    for (uint32_t k0 = 0; k0 < a.K; k0 += LSTEP) {
        __syncthreads(); // the step before has been read
#pragma unroll
        for (int u = 0; u < kA; ++u) *reinterpret_cast<uint4*>(As + (cr + 32u * u) * LLDT + ck) = ra[u];
#pragma unroll
        for (int u = 0; u < kB; ++u) *reinterpret_cast<uint4*>(Bs + (cr + 32u * u) * LLDT + ck) = rb[u];
        __syncthreads();
        if (k0 + LSTEP < a.K) fetch(k0 + LSTEP);
        __builtin_amdgcn_sched_barrier(0); // keep the requests ahead of the MFMAs
        if (idle) continue;
#pragma unroll
        for (int s = 0; s < LSTEP / 16; ++s) {
            const uint32_t at = s * 16u + 8u * half;
#pragma unroll
            for (int j = 0; j < NI; ++j)
                y[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*reinterpret_cast<const uint4*>(Bs + (j * 32u + (lane & 31u)) * LLDT + at)),
                                                               as_bf16x8(*reinterpret_cast<const uint4*>(As + r * LLDT + at)), y[j], 0, 0, 0);
        }
    }
    if (!idle) last_rows<NI>(a, y, s_bias, a.N, half, my_row < rows, a.row_begin + my_row, dst);
    // (the next tile's first barrier stands before anything this one reads is written)
}

template <int NI>
__global__ __launch_bounds__(LWAVES * 64, 4) void mlp_last_layer(LayerArgs a, uint32_t short_tiles)
{
    typedef LastShape<NI> S;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint4 *s_a = reinterpret_cast<uint4*>(smem), *s_w = s_a + S::kHeld * 256; // [kHeld][4][64], [kHeld][4][NI][64]
    float* s_bias = reinterpret_cast<float*>(smem + S::kBias);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t total = *a.esc_count;
    total = total < a.esc_cap ? total : a.esc_cap;
    if (a.row_begin >= total) return;
    const uint32_t left = total - a.row_begin, rows = left < a.rows_cap ? left : a.rows_cap; // of this chunk
    if (a.units_before && wide_takes_last(rows, a.lda, a.units_before, a.k_before <= kWideSlab * kWideSlabs))
        return; // the layer before has taken this one along
    const uint32_t pieces = (a.K + LPIECE - 1u) / LPIECE, tiles = (rows + LROWS - 1u) / LROWS;
    if (tid < NI * 32u) s_bias[tid] = tid < a.N ? a.bias[tid] : 0.f; // (read several barriers on)
    constexpr uint32_t kOnce = NI == 1 ? 16 : 8; // pieces for which a block counts once
    if (tiles * ((pieces + kOnce - 1u) / kOnce) > short_tiles) {
        for (uint32_t i = blockIdx.x; long_rows<NI>(i) < rows; i += gridDim.x) last_tile<NI>(a, long_rows<NI>(i), rows, smem, s_bias, tid, lane, wave);
        return;
    }
    const uint32_t m = wave % S::kHeld, jw = wave / S::kHeld; // this wave's piece of a round and its classes
    u32x4 fa[S::kRows], fw[4];
    // this wave's share of the round from piece p0 on for the rows from r0 on (a row, piece or class past the last one: that one again)
    auto request = [&](uint32_t r0, uint32_t p0) __attribute__((always_inline)) {
        const uint32_t r = r0 + (lane & 31u), ks = (p0 + m < pieces ? p0 + m : pieces - 1u) * (LPIECE / 16u);
        const uint16_t* arow = a.a_bf16 + (size_t)(r < rows ? r : rows - 1u) * a.lda + 8u * (lane >> 5); // (lda: whole pieces, zeros behind K)
#pragma unroll
        for (int s = 0; s < S::kRows; ++s) fa[s] = *reinterpret_cast<const u32x4*>(arow + (ks + jw * S::kRows + s) * 16u);
        if (NI == 1 && a.wo_last) {
#pragma unroll
            for (int s = 0; s < 4; ++s) fw[s] = *reinterpret_cast<const u32x4*>(a.wo_last + (ks + s) * 64u + lane);
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint4 w = weight_chunk(a.w, a.N, a.K, jw * 32u + (lane & 31u), (ks + s) * 16u + 8u * (lane >> 5));
                fw[s] = u32x4{w.x, w.y, w.z, w.w};
            }
        }
    };
    const uint32_t blocks = (tiles + kDies * 4u - 1u) / (kDies * 4u) * (kDies * 4u); // (some of the last 32 have no rows)
    auto from = [&](uint32_t i) { // the next block from i on that has
        while (i < blocks && short_rows(i) >= rows) i += gridDim.x;
        return i;
    };
    uint32_t i = from(blockIdx.x);
    if (i >= blocks) return;
    request(short_rows(i), 0);
    for (uint32_t next; i < blocks; i = next) {
        const uint32_t r0 = short_rows(i), row = r0 + (lane & 31u);
        next = from(i + gridDim.x);
        uint32_t dst = 0;
        if (wave == 0) dst = (a.scatter ? a.scatter : a.esc_idx)[a.row_begin + (row < rows ? row : rows - 1u)];
        f32x16 y[NI]; // (of the first wave)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) y[j][v] = 0.f;
        for (uint32_t p0 = 0; p0 < pieces; p0 += S::kHeld) {
            // what was requested goes to shared memory, the next round is requested, the first wave multiplies
#pragma unroll
            for (int s = 0; s < S::kRows; ++s) *reinterpret_cast<u32x4*>(s_a + (m * 4u + jw * S::kRows + s) * 64u + lane) = fa[s];
#pragma unroll
            for (int s = 0; s < 4; ++s) *reinterpret_cast<u32x4*>(s_w + ((m * 4u + s) * NI + jw) * 64u + lane) = fw[s];
            __syncthreads();
            const bool more = p0 + S::kHeld < pieces;
            if (more || next < blocks) request(more ? r0 : short_rows(next), more ? p0 + S::kHeld : 0u);
            __builtin_amdgcn_sched_barrier(0);
            if (wave == 0) {
                constexpr int kRing = NI == 1 ? 4 : 2; // steps whose operands are on their way out of shared memory
                const uint32_t steps = (pieces - p0 < (uint32_t)S::kHeld ? pieces - p0 : S::kHeld) * 4u;
                u32x4 ca[kRing], cw[kRing][NI];
                auto read = [&](int s, uint32_t t) __attribute__((always_inline)) {
                    ca[s] = *reinterpret_cast<const u32x4*>(s_a + t * 64u + lane);
#pragma unroll
                    for (int j = 0; j < NI; ++j) cw[s][j] = *reinterpret_cast<const u32x4*>(s_w + (t * NI + j) * 64u + lane);
                };
#pragma unroll
                for (int s = 0; s < kRing; ++s) read(s, s);
                for (uint32_t t = 0; t < steps; t += kRing) {
                    const uint32_t after = t + kRing < steps ? t + kRing : t;
#pragma unroll
                    for (int s = 0; s < kRing; ++s) {
#pragma unroll
                        for (int j = 0; j < NI; ++j)
                            y[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cw[s][j]), __builtin_bit_cast(bf16x8, ca[s]), y[j], 0, 0, 0);
                        read(s, after + s);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            __syncthreads(); // the round has been read
        }
        if (wave == 0) last_rows<NI>(a, y, s_bias, a.N, lane >> 5, row < rows, a.row_begin + row, dst);
    }
}

// ---- binary32 model (plain vector arithmetic) ---------------------------------------------

struct F32Args {
    const uint32_t* esc_idx;
    const uint32_t* esc_count;
    uint32_t esc_cap, row_begin, rows_cap, n_rows;
    const float* feat;
    uint32_t feat_ld;
    const float* mu;
    const float* inv_sigma;
    float clamp;
    const uint32_t* off;
    const uint32_t* hdr;
    uint32_t hdr_words, raw_bits, raw_pkts, n_pkts;
    uint32_t n_in;
};

// input value k of the row that entry `flow` of the list names
__device__ __forceinline__ float f32_input_value(const F32Args& a, uint32_t flow, uint32_t k)
{
    flow = flow < a.n_rows ? flow : a.n_rows - 1u; // a bad list entry must not leave the input
    if (a.feat) {
        float v = a.feat[(size_t)flow * a.feat_ld + k];
        if (a.mu) {
            const float d = v - a.mu[k];
            v = d * a.inv_sigma[k];
            v = v < -a.clamp ? -a.clamp : v;
            v = v > a.clamp ? a.clamp : v;
        }
        return v;
    }
    uint32_t b0 = a.off[flow], e0 = a.off[flow + 1];
    b0 = b0 < a.n_pkts ? b0 : a.n_pkts;
    e0 = e0 < a.n_pkts ? e0 : a.n_pkts;
    const uint32_t np = e0 > b0 ? e0 - b0 : 0;
    const uint32_t j = k / a.raw_bits, b = k - j * a.raw_bits;
    if (j >= np) return 0.f;
    const uint32_t byte_i = b >> 3;
    const uint32_t word = a.hdr[(size_t)(b0 + j) * a.hdr_words + (byte_i >> 2)];
    return (float)(((word >> (8u * (byte_i & 3u))) >> (7u - (b & 7u))) & 1u);
}

// The whole model on 16 rows per block, or on 4 while that leaves a compute unit at most two blocks: the activations stay in
// shared memory, the weights go straight from the cache into registers.  A lane owns one row R = 16 (4) and up to four output
// columns of it: the R lanes of a group hold consecutive weights of a column, four to a lane, loaded as they lie, and the one a
// step needs is broadcast among them by the multiplication itself (a data-parallel operand), so that a term costs its multiply
// and its add and nothing else; a row's input serves all columns of the lane.  The sums run in order of the inputs, one multiply
// and one add per term, each rounded, as in f32_layer (the results are the same bits).  What bounds it is that arithmetic (two
// instructions a term, no packed ones) and, for few rows, latencies: the chain of loads in front, and the code itself, which a
// launch fetches anew, so there is one copy of each loop.  Weights and activations both through shared memory, whose reads cost
// as much as the arithmetic, with two barriers per 32 inputs : this, whole call in us: one row through 32-128-128-4 13.7 : 8.0,
// 2,000 15.3 : 10.4, 4,096 16.9 : 13.4; 200 rows through 64-256-256-10 38 : 17, 16,000 through 128-256-256-32 133 : 114 (77 % of
// the arithmetic's rate), 600 through 128-512-512-32 126 : 49.
constexpr uint32_t kF32Rows = 16, kF32FewRows = 4, kF32Waves = 8;
constexpr size_t kF32FusedLds = 160 * 1024 - 512;
constexpr double kF32FusedTerms = 1.5e10;

__host__ __device__ inline uint32_t up16(uint32_t x) { return (x + 15u) / 16u * 16u; }
// row strides of the two activation buffers: input and second hidden layer, first hidden layer and logits (whole groups of
// 16 inputs and a piece of four: 16 rows' pieces lie on distinct banks)
__host__ __device__ inline uint32_t f32_ld(uint32_t x, uint32_t y) { return up16(x > y ? x : y) + 4u; }
__host__ __device__ inline size_t f32_fused_lds(uint32_t n_in, uint32_t h1, uint32_t h2, uint32_t c)
{
    return ((size_t)kF32Rows * ((size_t)f32_ld(n_in, h2) + f32_ld(h1, c)) + 32) * 4; // (inputs are read up to 16 past a row)
}

// terms of the sums of one row, columns in whole waves
inline double f32_terms(uint32_t n_in, uint32_t h1, uint32_t h2, uint32_t c)
{
    const auto waves = [](uint32_t n) { return (double)((n + 63u) / 64u * 64u); };
    return n_in * waves(h1) + h1 * waves(h2) + h2 * waves(c);
}

struct F32Model {
    const float *w1, *b1, *w2, *b2, *w3, *b3;
    uint32_t h1, h2, c;
    const uint32_t* label_idx;
    float* logits;
    uint16_t* labels;
    uint32_t n_labels;
    const uint16_t* pred; // as in FusedArgs
    uint32_t n_copy;
};

// x of lane L of the R this lane belongs to
template <uint32_t R, uint32_t L>
__device__ __forceinline__ float of_lane(float x)
{
    constexpr int kCtrl = R == 16u ? 0x150 + (int)L /* row_newbcast */ : (int)(L * 0x55u) /* quad_perm */;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kCtrl, 0xF, 0xF, true));
}

// One layer as the lanes see it
struct F32Layer {
    const float *w, *bias;
    uint32_t K, N;
    bool wide; // rows of whole 16-byte pieces
};
// Columns of a lane: a wave takes 64 / R times as many at a time, so few that all waves have some.
template <uint32_t R>
__device__ __forceinline__ uint32_t f32_cols(uint32_t N)
{
    constexpr uint32_t kAll = 64u / R * kF32Waves;
    return R == 16u ? (N > 2u * kAll ? 4u : N > kAll ? 2u : 1u) : 1u;
}

// A lane's weights of 64 inputs: with 16 lanes to a group 4, with four lanes 16 in pieces of 16 inputs
template <uint32_t R>
constexpr int kF32Pieces = 16 / R;
template <uint32_t R>
struct F32Weights {
    float4 v[R == 16u ? 4 : 1][kF32Pieces<R>];
};

// [k, k + 64) of this lane's B columns from c0 on (past the last column: that one again; past K: zeros); none from N on
template <uint32_t R, int B>
__device__ __forceinline__ void f32_weights(const F32Layer& l, uint32_t c0, uint32_t k0, uint32_t lane, F32Weights<R>& r)
{
    if (c0 >= l.N) return;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const uint32_t col = c0 + 64u / R * b + lane / R;
        const float* p = l.w + (size_t)(col < l.N ? col : l.N - 1u) * l.K;
#pragma unroll
        for (int q = 0; q < kF32Pieces<R>; ++q) {
            const uint32_t k = k0 + 4u * R * q + 4u * (lane % R);
            float4& v = r.v[b][q];
            if (l.wide) {
                v = k < l.K ? *reinterpret_cast<const float4*>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                v.x = k < l.K ? p[k] : 0.f;
                v.y = k + 1u < l.K ? p[k + 1u] : 0.f;
                v.z = k + 2u < l.K ? p[k + 2u] : 0.f;
                v.w = k + 3u < l.K ? p[k + 3u] : 0.f;
            }
        }
    }
}
template <uint32_t R>
__device__ __forceinline__ void f32_first_weights(const F32Layer& l, uint32_t wave, uint32_t lane, F32Weights<R>& r)
{
    const uint32_t cols = f32_cols<R>(l.N), c0 = wave * (64u / R) * cols;
    if (R == 16u && cols == 4u)
        f32_weights<R, R == 16u ? 4 : 1>(l, c0, 0, lane, r);
    else if (R == 16u && cols == 2u)
        f32_weights<R, R == 16u ? 2 : 1>(l, c0, 0, lane, r);
    else
        f32_weights<R, 1>(l, c0, 0, lane, r);
}

// out[r][o] = act(sum_k in[r][k] * w[o][k] + b[o]) for this wave's columns; w holds the first weights on entry.  Terms are
// taken 16 at a time; those past K are zero times zero (a sum that starts at +0 is never -0, so they leave it as it is).
template <uint32_t R, int B>
__device__ __forceinline__ void f32_columns(const F32Layer& l, const float* in, uint32_t ld_in, float* out, uint32_t ld_out, bool relu, uint32_t wave,
                                            uint32_t lane, F32Weights<R>& w)
{
    constexpr uint32_t kCols = 64u / R, kStep = kCols * B * kF32Waves;
    const float* x = in + lane % R * ld_in;
    for (uint32_t c0 = wave * kCols * B; c0 < l.N; c0 += kStep) {
        float s[B], bias[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const uint32_t col = c0 + kCols * b + lane / R;
            bias[b] = l.bias[col < l.N ? col : l.N - 1u];
            s[b] = 0.f;
        }
        float4 xv[2][4]; // the inputs of 16 terms, the next ones read while one's are summed
        auto read = [&](float4 (&to)[4], uint32_t k) {
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) to[q] = *reinterpret_cast<const float4*>(x + k + 4u * q);
        };
        // four terms whose weights lane L of a column's group holds
        auto four = [&](auto L, const float4& xq, uint32_t piece) {
            float p[B];
            auto term = [&](float xk, auto part) {
#pragma unroll
                for (int b = 0; b < B; ++b) p[b] = of_lane<R, decltype(L)::value>(part(w.v[b][piece])) * xk;
#pragma unroll
                for (int b = 0; b < B; ++b) s[b] += p[b];
            };
            term(xq.x, [](const float4& v) { return v.x; });
            term(xq.y, [](const float4& v) { return v.y; });
            term(xq.z, [](const float4& v) { return v.z; });
            term(xq.w, [](const float4& v) { return v.w; });
        };
        auto sixteen = [&](auto g, uint32_t k) {
            constexpr uint32_t l0 = R == 16u ? 4u * decltype(g)::value : 0u, piece = R == 16u ? 0u : decltype(g)::value;
            const float4(&xq)[4] = xv[decltype(g)::value & 1u];
            read(xv[(decltype(g)::value + 1u) & 1u], k + 16u); // (past K: not used)
            __builtin_amdgcn_sched_barrier(0);
            four(std::integral_constant<uint32_t, l0>{}, xq[0], piece), four(std::integral_constant<uint32_t, l0 + 1u>{}, xq[1], piece);
            four(std::integral_constant<uint32_t, l0 + 2u>{}, xq[2], piece), four(std::integral_constant<uint32_t, l0 + 3u>{}, xq[3], piece);
        };
        read(xv[0], 0);
#pragma nounroll
        for (uint32_t k = 0; k < l.K; k += 64u) {
            // the next weights, of this pass or the first of the next one, are requested ahead of the arithmetic
            F32Weights<R> ahead;
            const bool more = k + 64u < l.K;
            f32_weights<R, B>(l, more ? c0 : c0 + kStep, more ? k + 64u : 0u, lane, ahead);
            sixteen(std::integral_constant<uint32_t, 0>{}, k);
            if (k + 16u < l.K) {
                sixteen(std::integral_constant<uint32_t, 1>{}, k + 16u);
                if (k + 32u < l.K) {
                    sixteen(std::integral_constant<uint32_t, 2>{}, k + 32u);
                    if (k + 48u < l.K) sixteen(std::integral_constant<uint32_t, 3>{}, k + 48u);
                }
            }
            w = ahead;
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const uint32_t col = c0 + kCols * b + lane / R;
            const float y = s[b] + bias[b];
            if (col < l.N) out[lane % R * ld_out + col] = (relu && y < 0.f) ? 0.f : y;
        }
    }
}

template <uint32_t R>
__device__ __forceinline__ void f32_rows(const F32Args& a, const F32Model& m, uint32_t block, uint32_t blocks, uint32_t total, float* sm)
{
    constexpr uint32_t kThreads = kF32Waves * 64;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lda = f32_ld(a.n_in, m.h2), ldb = f32_ld(m.h1, m.c);
    float *A = sm, *B = A + R * lda;
    auto layer_at = [&](uint32_t i) {
        F32Layer l;
        l.w = i == 0 ? m.w1 : i == 1u ? m.w2 : m.w3;
        l.bias = i == 0 ? m.b1 : i == 1u ? m.b2 : m.b3;
        l.K = i == 0 ? a.n_in : i == 1u ? m.h1 : m.h2;
        l.N = i == 0 ? m.h1 : i == 1u ? m.h2 : m.c;
        l.wide = (l.K & 3u) == 0 && (reinterpret_cast<uintptr_t>(l.w) & 15u) == 0;
        return l;
    };
    if (block * R >= total) return; // (nothing to request weights for: no rows of 16,850, 75-204-59-53, whole call 9.7 us with the requests, 5.3 without)
    // the first weights of a layer are requested ahead of what the layer waits for
    F32Weights<R> w;
    f32_first_weights<R>(layer_at(0), wave, lane, w);
    for (uint32_t row0 = block * R; row0 < total; row0 += blocks * R) {
        const uint32_t k_in = up16(a.n_in);
        for (uint32_t e = tid; e < R * k_in; e += kThreads) {
            const uint32_t r = e / k_in, k = e - r * k_in;
            A[r * lda + k] = k < a.n_in && row0 + r < total ? f32_input_value(a, a.esc_idx[row0 + r], k) : 0.f;
        }
        __syncthreads();
#pragma nounroll
        for (uint32_t i = 0; i < 3u; ++i) { // (a loop, so that the code is there once)
            const F32Layer l = layer_at(i);
            const float* in = i == 1u ? B : A;
            float* out = i == 1u ? A : B;
            const uint32_t ld_in = i == 1u ? ldb : lda, ld_out = i == 1u ? lda : ldb, cols = f32_cols<R>(l.N);
            if (R == 16u && cols == 4u)
                f32_columns<R, R == 16u ? 4 : 1>(l, in, ld_in, out, ld_out, i < 2u, wave, lane, w);
            else if (R == 16u && cols == 2u)
                f32_columns<R, R == 16u ? 2 : 1>(l, in, ld_in, out, ld_out, i < 2u, wave, lane, w);
            else
                f32_columns<R, 1>(l, in, ld_in, out, ld_out, i < 2u, wave, lane, w);
            f32_first_weights<R>(layer_at(i < 2u ? i + 1u : 0u), wave, lane, w);
            if (tid < R * 16u) { // zeros behind the outputs: the next layer's inputs past K
                const uint32_t c = up16(l.N) - 16u + (tid & 15u);
                if (c >= l.N) out[(tid >> 4) * ld_out + c] = 0.f;
            }
            __syncthreads();
        }
        if (m.logits)
            for (uint32_t e = tid; e < R * m.c; e += kThreads) {
                const uint32_t r = e / m.c;
                if (row0 + r < total) m.logits[(size_t)row0 * m.c + e] = B[r * ldb + (e - r * m.c)];
            }
        if (tid < R && row0 + tid < total) {
            const float* p = B + tid * ldb;
            uint32_t best = 0;
            float bv = p[0];
            for (uint32_t c = 1; c < m.c; ++c)
                if (p[c] > bv) {
                    bv = p[c];
                    best = c;
                }
            const uint32_t dst = m.label_idx[row0 + tid];
            if (dst < m.n_labels) m.labels[dst] = (uint16_t)best;
        }
    }
}

// few: the most rows that go four to a block.  The gate, if there is one, makes the list.
template <class Gate>
__global__ __launch_bounds__(kF32Waves * 64, 4) void f32_mlp(F32Args a, F32Model m, uint32_t few, Gate gate)
{
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const uint32_t block = blockIdx.x - m.n_copy, blocks = gridDim.x - m.n_copy;
    uint32_t total;
    if constexpr (std::is_same<Gate, sfsmall::GateRows>::value) {
        total = sfsmall::gate_rows<kF32Waves * 64>(gate, sm, [&](uint32_t n) {
            const uint32_t rows = n <= few ? kF32FewRows : kF32Rows;
            return [=](uint32_t p) { return p / rows % blocks == block; };
        });
        if (block == 0 && threadIdx.x == 0) *gate.esc_count = total;
        __syncthreads();
    } else {
        total = *a.esc_count;
        total = total < a.esc_cap ? total : a.esc_cap;
        if (blockIdx.x < m.n_copy) {
            sfsmall::copy_unlisted<kF32Waves * 64, false>(m.pred, m.labels, m.n_labels, a.esc_idx, total, blockIdx.x * sfsmall::kCopySlice,
                                                   reinterpret_cast<uint32_t*>(sm));
            return;
        }
    }
    if (total <= few)
        f32_rows<kF32FewRows>(a, m, block, blocks, total, sm);
    else
        f32_rows<kF32Rows>(a, m, block, blocks, total, sm);
}

__global__ __launch_bounds__(256) void f32_input(F32Args a, float* __restrict__ z)
{
    uint32_t total = *a.esc_count;
    total = total < a.esc_cap ? total : a.esc_cap;
    if (a.row_begin >= total) return;
    uint32_t rows = total - a.row_begin;
    rows = rows < a.rows_cap ? rows : a.rows_cap;
    const uint64_t n = (uint64_t)rows * a.n_in;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t r = (uint32_t)(g / a.n_in), k = (uint32_t)(g % a.n_in);
        z[g] = f32_input_value(a, a.esc_idx[a.row_begin + r], k);
    }
}

// out[r][o] = act(sum_k in[r][k] * w[o][k] + b[o]) in binary32, the sum taken in order of k (one multiply
// and one add per term, each rounded).  A block computes a 64 x 64 tile of outputs from K-slabs of 16 staged
// in shared memory; a thread owns a 4 x 4 patch (rows ty + 16 i, columns tx + 16 j).
constexpr int kF32Tile = 64, kF32Slab = 16;

__global__ __launch_bounds__(256) void f32_layer(const uint32_t* esc_count, uint32_t esc_cap, uint32_t row_begin,
                                                 uint32_t rows_cap, const float* __restrict__ in, uint32_t K,
                                                 const float* __restrict__ w, const float* __restrict__ bias,
                                                 uint32_t N, float* __restrict__ out, int relu)
{
    __shared__ float As[kF32Slab][kF32Tile + 1]; // [k][row]
    __shared__ float Ws[kF32Slab][kF32Tile + 1]; // [k][column]
    uint32_t total = *esc_count;
    total = total < esc_cap ? total : esc_cap;
    if (row_begin >= total) return;
    uint32_t rows = total - row_begin;
    rows = rows < rows_cap ? rows : rows_cap;
    const uint32_t r0 = blockIdx.x * kF32Tile, c0 = blockIdx.y * kF32Tile;
    if (r0 >= rows) return;
    const uint32_t tid = threadIdx.x, tx = tid & 15u, ty = tid >> 4;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
    for (uint32_t k0 = 0; k0 < K; k0 += kF32Slab) {
        // 64 x 16 values of each operand, four per thread: element e -> (row e / 16, k e % 16)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t e = tid + 256u * q, rr = e >> 4, kk = e & 15u;
            const bool kin = k0 + kk < K;
            As[kk][rr] = (kin && r0 + rr < rows) ? in[(size_t)(r0 + rr) * K + k0 + kk] : 0.f;
            Ws[kk][rr] = (kin && c0 + rr < N) ? w[(size_t)(c0 + rr) * K + k0 + kk] : 0.f;
        }
        __syncthreads();
        const uint32_t kn = K - k0 < (uint32_t)kF32Slab ? K - k0 : (uint32_t)kF32Slab;
        for (uint32_t kk = 0; kk < kn; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty + 16 * i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = Ws[kk][tx + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t r = r0 + ty + 16 * i;
        if (r >= rows) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t o = c0 + tx + 16 * j;
            if (o < N) {
                const float y = acc[i][j] + bias[o];
                out[(size_t)r * N + o] = (relu && y < 0.f) ? 0.f : y;
            }
        }
    }
}

__global__ __launch_bounds__(256) void f32_argmax(const uint32_t* label_idx, const uint32_t* esc_count, uint32_t esc_cap,
                                                  uint32_t row_begin, uint32_t rows_cap, const float* __restrict__ lg,
                                                  uint32_t C, float* __restrict__ logits, uint16_t* __restrict__ labels,
                                                  uint32_t n_labels)
{
    uint32_t total = *esc_count;
    total = total < esc_cap ? total : esc_cap;
    if (row_begin >= total) return;
    uint32_t rows = total - row_begin;
    rows = rows < rows_cap ? rows : rows_cap;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < rows; r += gridDim.x * blockDim.x) {
        const float* p = lg + (size_t)r * C;
        uint32_t best = 0;
        float bv = p[0];
        for (uint32_t c = 0; c < C; ++c) {
            const float v = p[c];
            if (logits) logits[(size_t)(row_begin + r) * C + c] = v;
            if (v > bv) {
                bv = v;
                best = c;
            }
        }
        const uint32_t dst = label_idx[row_begin + r];
        if (dst < n_labels) labels[dst] = (uint16_t)best;
    }
}

template <int NI>
int launch_last(sf_ctx* ctx, const LayerArgs& a, uint32_t rows_cap)
{
    SF_ALLOW_LDS(ctx, sf::kLdsLast + NI - 1, mlp_last_layer<NI>);
    const uint32_t tiles = (rows_cap + LROWS * 4u * kDies - 1u) / (LROWS * 4u * kDies) * (4u * kDies), most = 4u * (uint32_t)ctx->n_cu; // (rows that exist are dealt out in the kernel)
    mlp_last_layer<NI><<<tiles < most ? tiles : most, LWAVES * 64, LastShape<NI>::kLds, ctx->stream>>>(a, (NI > 1 ? 1u : a.wo_last ? 3u : 2u) * (uint32_t)ctx->n_cu);
    SF_LAUNCH_CHECK(ctx, "mlp_last_layer");
    return SF_OK;
}

// labels = pred for every flow; the slow labels are scattered over it afterwards
__global__ __launch_bounds__(256) void copy_labels(const uint16_t* __restrict__ pred, uint16_t* __restrict__ labels, uint32_t n)
{
    const uint32_t base = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (base + 8 <= n && ((reinterpret_cast<uintptr_t>(pred) | reinterpret_cast<uintptr_t>(labels)) & 15u) == 0) {
        *reinterpret_cast<uint4*>(labels + base) = *reinterpret_cast<const uint4*>(pred + base);
    } else {
        for (uint32_t k = base; k < n && k < base + 8; ++k) labels[k] = pred[k];
    }
}

uint32_t pad64(uint32_t x) { return (x + 63u) / 64u * 64u; }

} // namespace

namespace sf {
int copy_labels_async(sf_ctx* ctx, const uint16_t* pred, uint16_t* labels, uint32_t n)
{
    copy_labels<<<(n + 2047u) / 2048u, 256, 0, ctx->stream>>>(pred, labels, n);
    SF_LAUNCH_CHECK(ctx, "copy_labels");
    return SF_OK;
}
} // namespace sf

namespace {

int check_model(sf_ctx* ctx, const sf_mlp* mlp)
{
    if (!mlp) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: mlp is NULL");
    if (mlp->dtype != SF_F32 && mlp->dtype != SF_BF16) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: unknown dtype %d", mlp->dtype);
    if (!mlp->n_in || !mlp->n_h1 || !mlp->n_h2 || !mlp->n_classes)
        return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: a layer width is zero");
    if (mlp->n_classes > SF_MAX_CLASSES)
        return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: n_classes %u > %d", mlp->n_classes, SF_MAX_CLASSES);
    if (!mlp->w1 || !mlp->w2 || !mlp->w3 || !mlp->b1 || !mlp->b2 || !mlp->b3)
        return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: weights or biases missing");
    if ((mlp->mu == nullptr) != (mlp->inv_sigma == nullptr))
        return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: mu and inv_sigma come together");
    return SF_OK;
}

// the binary32 model in one launch; the rule is at run_slow()
bool f32_in_one(const sf_mlp* mlp, uint32_t esc_cap)
{
    return f32_fused_lds(mlp->n_in, mlp->n_h1, mlp->n_h2, mlp->n_classes) <= kF32FusedLds &&
           esc_cap * f32_terms(mlp->n_in, mlp->n_h1, mlp->n_h2, mlp->n_classes) <= kF32FusedTerms;
}

size_t row_bytes_of(const sf_mlp* mlp)
{
    return mlp->dtype == SF_BF16 ? ((size_t)pad64(mlp->n_h1) + pad64(mlp->n_h2)) * 2
                                 : ((size_t)mlp->n_in + mlp->n_h1 + mlp->n_h2 + mlp->n_classes) * 4;
}
uint64_t rows_in(const sf::Carve& ws, size_t row_bytes)
{
    const size_t avail = ws.left() > 4 * sf::kAlign ? ws.left() - 4 * sf::kAlign : 0;
    return avail / row_bytes / BM * BM;
}

// All entry points.  esc_idx: input rows (of feat, n_rows of them, or flows of raw_src); scatter: where the
// labels go (NULL = esc_idx); n_flows: entries of labels; gate: makes the list first (only where sf::slow_gates()).
int run_slow(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n_rows, const sf_packets* raw_src,
             const sf_feat_cfg* raw_cfg, const uint32_t* esc_idx, const uint32_t* scatter, const uint32_t* esc_count,
             uint32_t esc_cap, uint32_t n_flows, const sf_mlp* mlp, const uint16_t* pred, const sfsmall::GateRows* gate, float* logits,
             uint16_t* labels)
{
    if (const int rc = check_model(ctx, mlp); rc != SF_OK) return rc;
    if (n_flows == 0) return SF_OK;
    if (pred == labels) pred = nullptr;
    if (pred && !labels) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: labels is NULL");
    // labels = the fast prediction for every flow, also when nothing escalates (Section 4.4: the fast label stands unless the
    // slow model replaces it): by the slow model's (first) launch where it can, else by one before it
    const bool bf = mlp->dtype == SF_BF16, in_one = bf ? sf::slow_fused_ok(mlp, raw_src != nullptr) : f32_in_one(mlp, esc_cap) && n_flows <= sfsmall::kCopyRows;
    const bool reused = sfsmall::share(pred, (uint64_t)n_flows * 2u, logits, (uint64_t)esc_cap * mlp->n_classes * 4u);
    if (pred && ((!bf && !in_one) || reused || esc_cap == 0 || n_rows == 0)) {
        if (const int rc = sf::copy_labels_async(ctx, pred, labels, n_flows); rc != SF_OK) return rc;
        pred = nullptr;
    }
    if (esc_cap == 0 || n_rows == 0) return SF_OK;
    if ((feat == nullptr) == (raw_src == nullptr))
        return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: give exactly one of feat and raw_src");
    if (feat && mlp->n_in > feat_ld) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: n_in %u > feat_ld %u", mlp->n_in, feat_ld);
    if (raw_src) {
        if (!raw_cfg || !raw_src->pkt_hdr || !raw_src->flow_off || raw_src->hdr_words == 0)
            return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: raw input needs raw_cfg, flow_off and pkt_hdr");
        if (raw_cfg->raw_bits == 0 || raw_cfg->raw_bits > 32 * raw_src->hdr_words ||
            (uint64_t)raw_cfg->raw_pkts * raw_cfg->raw_bits != mlp->n_in)
            return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: raw_pkts*raw_bits must equal n_in and fit the header words");
        if (raw_src->n_flows != n_flows) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: raw_src->n_flows != n_flows");
        if (raw_src->n_pkts >> 32) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: n_pkts exceeds 32-bit offsets");
    }
    if (!esc_idx || !esc_count || !labels) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer: esc_idx, esc_count or labels is NULL");
    if (!scatter && esc_cap > n_flows) esc_cap = n_flows;

    sf::Carve ws(ctx);
    if (bf && in_one) {
        if (mlp->ordered)
            return sf::slow_fused(ctx, const_cast<void*>(mlp->ordered), true, feat, feat_ld, n_rows, esc_idx, scatter, esc_count,
                                  esc_cap, n_flows, mlp, pred, gate, logits, labels);
        const size_t need = sf::slow_fused_ws_bytes(mlp);
        void* w = ws.take(need);
        if (!w) return sf::fail(ctx, SF_ENOMEM, "sf_slow_infer: workspace too small for %zu bytes of re-ordered weights", need);
        return sf::slow_fused(ctx, w, false, feat, feat_ld, n_rows, esc_idx, scatter, esc_count, esc_cap, n_flows, mlp, pred, gate,
                              logits, labels);
    }
    const void *w1o = nullptr, *w2o = nullptr, *w3o = nullptr;
    if (bf && mlp->ordered) {
        w1o = mlp->ordered;
        w2o = (const char*)mlp->ordered + sf::reordered_bytes(mlp->n_h1, mlp->n_in);
        if (mlp->n_classes <= 32u) w3o = (const char*)w2o + sf::reordered_bytes(mlp->n_h2, mlp->n_h1);
    } else if (bf) {
        // operand-ordered copies of the two hidden layers' weights
        void* o1 = ws.take(sf::reordered_bytes(mlp->n_h1, mlp->n_in));
        void* o2 = ws.take(sf::reordered_bytes(mlp->n_h2, mlp->n_h1));
        if (!o1 || !o2) return sf::fail(ctx, SF_ENOMEM, "sf_slow_infer: workspace too small for the re-ordered weights");
        const sf::ReorderSpec specs[2] = {{mlp->w1, mlp->n_h1, mlp->n_in, o1}, {mlp->w2, mlp->n_h2, mlp->n_h1, o2}};
        const int rc = sf::reorder_weights_async(ctx, specs, 2);
        if (rc != SF_OK) return rc;
        w1o = o1;
        w2o = o2;
    }
    const uint32_t ld1 = bf ? pad64(mlp->n_h1) : mlp->n_h1, ld2 = bf ? pad64(mlp->n_h2) : mlp->n_h2;
    uint64_t rows_cap = rows_in(ws, row_bytes_of(mlp));
    if (rows_cap < sf::kSlowMinRows)
        return sf::fail(ctx, SF_ENOMEM, "sf_slow_infer: workspace holds %llu rows of hidden activations, need at least %u",
                        (unsigned long long)rows_cap, sf::kSlowMinRows);
    if (rows_cap > ((uint64_t)esc_cap + BM - 1) / BM * BM) rows_cap = ((uint64_t)esc_cap + BM - 1) / BM * BM;
    const uint32_t R = (uint32_t)rows_cap;

    if (bf) {
        uint16_t* h1 = (uint16_t*)ws.take((size_t)R * ld1 * 2);
        uint16_t* h2 = (uint16_t*)ws.take((size_t)R * ld2 * 2);
        if (!h1 || !h2) return sf::fail(ctx, SF_ENOMEM, "sf_slow_infer: workspace carve failed");
        for (uint32_t begin = 0; begin < esc_cap; begin += R) {
            LayerArgs a = {};
            a.esc_idx = esc_idx;
            a.scatter = scatter;
            a.esc_count = esc_count;
            a.esc_cap = esc_cap;
            a.row_begin = begin;
            a.n_rows = n_rows;
            a.n_labels = n_flows;
            a.labels = labels;
            a.pred = begin == 0 ? pred : nullptr;
            // layer 1
            a.feat = feat;
            a.feat_ld = feat_ld;
            a.mu = mlp->mu;
            a.inv_sigma = mlp->inv_sigma;
            a.clamp = mlp->clamp;
            if (raw_src) {
                a.off = raw_src->flow_off;
                a.hdr = raw_src->pkt_hdr;
                a.hdr_words = raw_src->hdr_words;
                a.raw_bits = raw_cfg->raw_bits;
                a.raw_pkts = raw_cfg->raw_pkts;
                a.n_pkts = (uint32_t)raw_src->n_pkts;
            }
            a.w = (const uint16_t*)mlp->w1;
            a.bias = mlp->b1;
            a.N = mlp->n_h1;
            a.K = mlp->n_in;
            a.h_out = h1;
            a.ldh = ld1;
            {
                const int rc = sf::wide_layer(ctx, raw_src ? A_RAW : A_FEAT, a, w1o, R);
                if (rc != SF_OK) return rc;
            }
            // layer 2
            a.pred = nullptr;
            a.a_bf16 = h1;
            a.lda = ld1;
            a.w = (const uint16_t*)mlp->w2;
            a.bias = mlp->b2;
            a.N = mlp->n_h2;
            a.K = mlp->n_h1;
            a.h_out = h2;
            a.ldh = ld2;
            a.wo_last = (const uint4*)w3o;
            a.b_last = mlp->b3;
            // Only with operand-ordered weights: each tile's two multiplying waves would gather the others line by line (70,077 rows through
            // 64-9-1032-10: its own launch 87 us, along with the second hidden layer 127).  And not where the first layer does most
            // of the work, eight times the second's: such a pass runs at the clock that the power allows, and the launch saved is paid back
            // at a lower one, by every kernel (a million flows of 10 x 480 header bits through 1024-512, whole passes of three processes each
            // 1,857-1,862 : 1,869-1,913, though the launches of the two layers are shorter; 100,000 rows of 20 x 480 1,694 : 1,707; a first layer
            // of 4.7 times the second's work, 210,000 rows of 5 x 480, 1,101 : 1,061; of twice, 647 : 606).
            a.n_last = w3o && mlp->n_in < 8u * mlp->n_h2 ? mlp->n_classes : 0u;
            a.logits = logits;
            {
                const int rc = sf::wide_layer(ctx, A_BF16, a, w2o, R);
                if (rc != SF_OK) return rc;
            }
            // layer 3
            a.units_before = a.n_last ? sf::wide_blocks(ctx, ld2, R) : 0u;
            a.k_before = mlp->n_h1;
            a.a_bf16 = h2;
            a.lda = ld2;
            a.w = (const uint16_t*)mlp->w3;
            a.bias = mlp->b3;
            a.N = mlp->n_classes;
            a.K = mlp->n_h2;
            a.h_out = nullptr;
            a.ldh = 0;
            a.rows_cap = R;
            {
                const int rc = a.N <= 32u ? launch_last<1>(ctx, a, R) : launch_last<2>(ctx, a, R);
                if (rc != SF_OK) return rc;
            }
        }
        return SF_OK;
    }

    F32Args f = {};
    f.esc_idx = esc_idx;
    f.esc_count = esc_count;
    f.esc_cap = esc_cap;
    f.n_rows = n_rows;
    f.feat = feat;
    f.feat_ld = feat_ld;
    f.mu = mlp->mu;
    f.inv_sigma = mlp->inv_sigma;
    f.clamp = mlp->clamp;
    if (raw_src) {
        f.off = raw_src->flow_off;
        f.hdr = raw_src->pkt_hdr;
        f.hdr_words = raw_src->hdr_words;
        f.raw_bits = raw_cfg->raw_bits;
        f.raw_pkts = raw_cfg->raw_pkts;
        f.n_pkts = (uint32_t)raw_src->n_pkts;
    }
    f.n_in = mlp->n_in;
    // The whole model in one launch where a block's activations fit (widths up to about 2,400 together) and as long as the terms of
    // all sums stay under the line: past it the tiles of f32_layer, which read a weight once for 64 rows, are a little faster.  Whole
    // call in us, layer by layer : one launch: 300 rows (of 30,000) through 100-1100-1100-50 632 : 282, 40,000 rows through
    // 128-256-256-32 409 : 279, 24,576 through 128-450-450-10 642 : 444, 100,000 through 64-128-128-4 259 : 202; around the line 30,000
    // through 20-600-600-10 (12.6e9 terms) 955 : 794, 500,000 through 64-128-128-4 (16e9) 913 : 995, 200,000 through 128-256-256-32
    // (23e9) 1,274 : 1,377, 32,768 through 128-650-650-10 (19e9) 1,224 : 1,307.
    // Four rows a block while that gives a compute unit at most two: 2,000 rows through 32-128-128-4 12.9 : 10.4, 1,500 through
    // 64-200-256-10 28.7 : 21.7; four of them against one of 16 rows, 4,096 rows, 18.6 : 13.4.  At most one where the second layer's weights
    // come in single values (no whole 16-byte pieces a row), whose requests two blocks pay twice: 1,183 rows through 32-683-364-47 two blocks of
    // four 153, one of 16 96; 1,902 through 154-551-315-27 153 : 88.  (Rows that exist: the kernel deals them out.)
    if (f32_in_one(mlp, esc_cap)) {
        F32Model m = {(const float*)mlp->w1, mlp->b1, (const float*)mlp->w2, mlp->b2, (const float*)mlp->w3, mlp->b3, mlp->n_h1, mlp->n_h2,
                      mlp->n_classes, scatter ? scatter : esc_idx, logits, labels, n_flows, pred, 0};
        if (pred) m.n_copy = (n_flows + sfsmall::kCopySlice - 1u) / sfsmall::kCopySlice;
        const size_t lds = f32_fused_lds(mlp->n_in, mlp->n_h1, mlp->n_h2, mlp->n_classes);
        const bool whole = (mlp->n_h1 & 3u) == 0 && ((uintptr_t)mlp->w2 & 15u) == 0;
        const uint32_t few = (whole ? 2u : 1u) * kF32FewRows * (uint32_t)ctx->n_cu;
        const uint32_t tiles = (esc_cap + kF32FewRows - 1u) / kF32FewRows;
        // Two blocks a unit are resident; with four, long lists even out (253,066 rows through 64-200-48-7 595 : 566), up to 65,536 rows the
        // other blocks are launches for nothing: 16,682 rows through 32-8-18-13 14.1 : 15.2, 18,369 through 32-56-8-37 18.6 : 20.8.
        const uint32_t most = (esc_cap > 65536u ? 4u : 2u) * (uint32_t)ctx->n_cu;
        const uint32_t grid = (tiles < most ? tiles : most) + m.n_copy;
        if (gate) {
            SF_ALLOW_LDS(ctx, sf::kLdsF32 + 1, f32_mlp<sfsmall::GateRows>);
            f32_mlp<<<grid, kF32Waves * 64, lds, ctx->stream>>>(f, m, few, *gate);
        } else {
            SF_ALLOW_LDS(ctx, sf::kLdsF32, f32_mlp<sfsmall::NoGate>);
            f32_mlp<<<grid, kF32Waves * 64, lds, ctx->stream>>>(f, m, few, sfsmall::NoGate{});
        }
        SF_LAUNCH_CHECK(ctx, "f32_mlp");
        return SF_OK;
    }
    float* z = (float*)ws.take((size_t)R * mlp->n_in * 4);
    float* h1 = (float*)ws.take((size_t)R * ld1 * 4);
    float* h2 = (float*)ws.take((size_t)R * ld2 * 4);
    float* lg = (float*)ws.take((size_t)R * mlp->n_classes * 4);
    if (!z || !h1 || !h2 || !lg) return sf::fail(ctx, SF_ENOMEM, "sf_slow_infer: workspace carve failed");
    for (uint32_t begin = 0; begin < esc_cap; begin += R) {
        f.row_begin = begin;
        f.rows_cap = R;
        auto blocks = [&](uint64_t n) { uint64_t b = (n + 255) / 256; return (uint32_t)(b > 16384 ? 16384 : (b ? b : 1)); };
        f32_input<<<blocks((uint64_t)R * mlp->n_in), 256, 0, ctx->stream>>>(f, z);
        SF_LAUNCH_CHECK(ctx, "f32_input");
        auto tiles = [&](uint32_t n_out) { return dim3((R + kF32Tile - 1) / kF32Tile, (n_out + kF32Tile - 1) / kF32Tile); };
        f32_layer<<<tiles(mlp->n_h1), 256, 0, ctx->stream>>>(esc_count, esc_cap, begin, R, z, mlp->n_in,
                                                                            (const float*)mlp->w1, mlp->b1, mlp->n_h1, h1, 1);
        SF_LAUNCH_CHECK(ctx, "f32_layer 1");
        f32_layer<<<tiles(mlp->n_h2), 256, 0, ctx->stream>>>(esc_count, esc_cap, begin, R, h1, mlp->n_h1,
                                                                            (const float*)mlp->w2, mlp->b2, mlp->n_h2, h2, 1);
        SF_LAUNCH_CHECK(ctx, "f32_layer 2");
        f32_layer<<<tiles(mlp->n_classes), 256, 0, ctx->stream>>>(
            esc_count, esc_cap, begin, R, h2, mlp->n_h2, (const float*)mlp->w3, mlp->b3, mlp->n_classes, lg, 0);
        SF_LAUNCH_CHECK(ctx, "f32_layer 3");
        f32_argmax<<<blocks(R), 256, 0, ctx->stream>>>(scatter ? scatter : esc_idx, esc_count, esc_cap, begin, R, lg,
                                                       mlp->n_classes, logits, labels, n_flows);
        SF_LAUNCH_CHECK(ctx, "f32_argmax");
    }
    return SF_OK;
}

} // namespace

namespace sf {

// Whether the slow model's launch can make the list too, on a feature matrix of n rows: small batches, a model that goes through one
// launch, and nothing that the gate or the slow model would refuse (their own calls then say what).  Every block reads what the gate
// looks at for all flows while others write labels and logits, so those are arrays of their own (labels may be pred if the gate does
// not look at it).  One launch less: the whole call on 97 flows with a 64-512-512-10 model 27.1 -> 25.9 us, on 4,096 with a binary32
// one 23.4 -> 21.4.
bool slow_gates(sf_ctx* ctx, const float* feat, uint32_t feat_ld, const sf_mlp* mlp, const sfsmall::GateRows& gate, const float* logits,
                const uint16_t* labels)
{
    const uint32_t n = gate.n;
    if (n == 0 || !feat || check_model(ctx, mlp) != SF_OK || mlp->n_in > feat_ld) return false;
    if (n > (mlp->dtype == SF_F32 ? sfsmall::kGateRowsF32 : sfsmall::kGateRows)) return false;
    const uint64_t flows = (uint64_t)n * 2u, rows = (uint64_t)n * mlp->n_classes * 4u;
    for (const uint16_t* read : {gate.top, gate.n_vmin > 1u ? gate.pred : gate.top})
        if (sfsmall::share(read, flows, labels, flows) || sfsmall::share(read, flows, logits, rows)) return false;
    if (Carve ws(ctx); !ws.take(route_scratch_bytes(n))) return false;
    Carve ws(ctx);
    if (mlp->dtype == SF_F32) return f32_in_one(mlp, n) && rows_in(ws, row_bytes_of(mlp)) >= kSlowMinRows;
    return slow_fused_gates(ctx, mlp, n) && (mlp->ordered || ws.take(slow_fused_ws_bytes(mlp)));
}

int slow_infer_gated(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n, const sf_mlp* mlp, const sfsmall::GateRows& gate, const uint16_t* pred,
                     float* logits, uint16_t* labels)
{
    if (pred && pred != labels) {
        if (const int rc = copy_labels_async(ctx, pred, labels, n); rc != SF_OK) return rc;
    }
    return run_slow(ctx, feat, feat_ld, n, nullptr, nullptr, gate.esc_idx, nullptr, gate.esc_count, n, n, mlp, nullptr, &gate, logits, labels);
}

} // namespace sf

extern "C" int sf_slow_infer(sf_ctx* ctx, const float* feat, uint32_t feat_ld, const sf_packets* raw_src,
                             const sf_feat_cfg* raw_cfg, const uint32_t* esc_idx, const uint32_t* esc_count,
                             uint32_t esc_cap, uint32_t n_flows, const sf_mlp* mlp, const uint16_t* pred, float* logits,
                             uint16_t* labels)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_slow_infer: ctx is NULL");
    return run_slow(ctx, feat, feat_ld, n_flows, raw_src, raw_cfg, esc_idx, nullptr, esc_count, esc_cap, n_flows, mlp, pred,
                    nullptr, logits, labels);
}

extern "C" int sf_slow_infer_pairs(sf_ctx* ctx, const float* feat, uint32_t feat_ld, uint32_t n_rows,
                                   const uint32_t* pair_row, const uint32_t* pair_flow, const uint32_t* n_pairs,
                                   uint32_t pair_cap, uint32_t n_flows, const sf_mlp* mlp, float* logits, uint16_t* labels)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_slow_infer_pairs: ctx is NULL");
    if (!feat) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer_pairs: feat is NULL");
    if (pair_cap && n_flows && n_rows && !pair_flow) return sf::fail(ctx, SF_EINVAL, "sf_slow_infer_pairs: pair_flow is NULL");
    return run_slow(ctx, feat, feat_ld, n_rows, nullptr, nullptr, pair_row, pair_flow, n_pairs, pair_cap, n_flows, mlp,
                    nullptr, nullptr, logits, labels);
}

extern "C" size_t sf_mlp_ordered_bytes(const sf_mlp* mlp)
{
    if (!mlp || mlp->dtype != SF_BF16 || !mlp->n_in || !mlp->n_h1 || !mlp->n_h2 || !mlp->n_classes) return 0;
    return sf::reordered_bytes(mlp->n_h1, mlp->n_in) + sf::reordered_bytes(mlp->n_h2, mlp->n_h1) +
           sf::reordered_bytes(32, mlp->n_h2);
}

extern "C" int sf_mlp_order(sf_ctx* ctx, const sf_mlp* mlp, void* ordered)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_mlp_order: ctx is NULL");
    if (!mlp || !ordered) return sf::fail(ctx, SF_EINVAL, "sf_mlp_order: mlp or ordered is NULL");
    if (mlp->dtype != SF_BF16) return sf::fail(ctx, SF_EINVAL, "sf_mlp_order: only bfloat16 models have an ordered copy");
    if (!mlp->n_in || !mlp->n_h1 || !mlp->n_h2 || !mlp->n_classes || mlp->n_classes > 32 || !mlp->w1 || !mlp->w2 || !mlp->w3)
        return sf::fail(ctx, SF_EINVAL, "sf_mlp_order: widths, class count (at most 32) or weights missing");
    if ((uintptr_t)ordered & 255u) return sf::fail(ctx, SF_EINVAL, "sf_mlp_order: ordered is not 256-byte aligned");
    return sf::order_all(ctx, mlp, ordered);
}
