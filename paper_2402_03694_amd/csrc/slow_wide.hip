// Step 5, one hidden layer of the slow model for any width (Sections 3.1 and 4.4 of the paper:
// the slow model runs on the escalated flows only): H_out = relu(A * W^T + b), bfloat16 in,
// binary32 MFMA accumulation, bfloat16 out.
//
// A block is eight waves and works on tiles of 128 rows x 512 output columns; wave w owns columns
// [64w, 64w+64) for all 128 rows (4x2 accumulators of v_mfma_f32_32x32x16_bf16, weight operand
// first, so a lane holds 4 consecutive columns of one row).  The A operand goes through shared memory in
// slabs of 64 K-values, made by the shared chunk loader (bfloat16 activations, gathered and standardised
// feature rows, or unpacked header bits).  The weight operand comes operand-ordered straight from the cache
// through a ring of register buffers, as in the fused kernel.
//
// What bounds it is the cache path (16 KB of weights and 4 KB of activations per k-step of 16, about 11 TB/s over
// the chip) and, before, the waits around it:
//   - three slab buffers: the slab after the next is stored while this one is multiplied, so the A operands of the
//     next k-step are read ahead across the slab's end too and the barrier there finds them in registers;
//   - activations are requested without a branch, so that the waits in the loop stay at "oldest request";
//   - one block per compute unit that goes from tile to tile: its weight ring, and with activations the slabs, run on
//     into the next tile.  (One block per tile paid launch, weight latency and write-out one after the other, and a
//     call whose list may hold every flow launched 4 to 20 times as many blocks as it had tiles.)
//   - a row block is walked through all its column blocks where that costs no compute unit a tile more than 1 in 16
//     (the activations of the blocks at work are then fetched from HBM once, not once per column block), or where K
//     fits the slab buffers (input rows are gathered once); else the tiles of a column block follow each other;
//   - a wave stages and writes its own 64 columns, 64 rows at a time: no barrier.
// 793 k rows, 2048 x 2048: 6.5 -> 5.6 ms (1.18 PFLOP/s), 128 -> 2048: 1.2 -> 0.97 ms; 209 k rows of 4,800 header bits
// -> 1024: 1.53 ms (1.34 PFLOP/s).  Whole passes: large workload 16.8 -> 15.2 ms, header bits 2.29 -> 2.09 ms, 65,536
// ragged flows through 1024-1024 0.167 -> 0.161 ms.
#include "mlp_common.h"

namespace sf {
int wide_layer(sf_ctx* ctx, int amode, const sfmlp::LayerArgs& a, const void* w_ordered, uint32_t rows_cap);
uint32_t wide_blocks(const sf_ctx* ctx, uint32_t ldh, uint32_t rows_cap);
}

namespace {

using namespace sfmlp;

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

constexpr int WBM = 128;          // rows per tile
constexpr int WBN = 512;          // columns per tile
constexpr int WWAVES = 8;
constexpr int WNI = 2, WMI = 4;   // 32-column / 32-row accumulator blocks per wave
constexpr int WSLAB = 64;         // K values per slab
constexpr int WLDS = WSLAB + 8;   // slab row stride (elements)
constexpr uint32_t WBUF = 3;      // slab buffers
constexpr int WRING = 4;          // = k-steps per slab
constexpr int WCOLS = WNI * 32;   // columns of a wave
constexpr int WLDO = WCOLS + 8;   // row stride of a wave's staged output (elements)
constexpr int WSTAGE = WBM / 2;   // rows of a wave's output staged at a time
constexpr size_t kSlabBytes = (size_t)WBUF * WBM * WLDS * 2;
constexpr size_t kStageBytes = (size_t)WSTAGE * WLDO * 2 + WCOLS * 4; // a wave's staged output rows and bias
constexpr size_t kWideLds = kSlabBytes + WWAVES * kStageBytes + WBM * 4; // slabs, waves' own space, flow ids
constexpr size_t kLastLds = (size_t)WBM * 32 * 4 + 32 * 4; // the last layer: a tile's sums between column blocks, biases
constexpr int LRING = 8;          // its weights in flight, k-steps
static_assert(WBN == 512 && WSLAB == kWideSlab && WBUF == kWideSlabs, "as the last layer's launch assumes");
constexpr int FCHUNK = 1024, FLD = FCHUNK + 8, FRING = 16; // few rows: K values in shared memory at a time, their row stride, k-steps of weights in flight
constexpr size_t kFewLds = (size_t)2 * kFewTileRows * FLD * 2;

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

// x, made anew: what is computed from it stays where it is written.  The write-out's addresses, the same for every tile,
// were otherwise computed once ahead of all loops, which left the main loop 10 to 50 registers short: 200,000 rows of 256
// features through 1024-1024 1,106 -> 889 us a call, 128 features through 520-128 296 -> 266 us.
__device__ __forceinline__ uint32_t again(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// orders a wave's own shared-memory writes and reads (its instructions reach shared memory in program order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// RESIDENT: every slab of a row block has a buffer of its own (K up to WBUF slabs).
// FORM: how header bits lie (A_RAW).
// LAST: the last layer goes along (a block holds all columns of a row, wide_takes_last): when the waves have staged 64 rows of their
// columns, two of them multiply 32 rows each with the last layer's weights, all columns in order of K, and the activations are neither
// written nor read back: 60,000 rows through 1024-1024-16 a whole call 169 -> 152 us, 200,000 through 1024-512-16 373 -> 330, the large
// workload's pass 14.1 -> 13.3 ms; which models and lists at run_slow and wide_takes_last.  A logit is one chain over K, and its bias at the end, as in mlp_last_layer: the same bits.
template <int AMODE, bool RESIDENT, int FORM, bool LAST>
__device__ __forceinline__ void wide_tiles(const LayerArgs& a, const uint4* __restrict__ ws, uint32_t n_cb, unsigned char* smem)
{
    uint16_t* slab = reinterpret_cast<uint16_t*>(smem);                                                  // [WBUF][128][WLDS]
    uint32_t* s_flow = reinterpret_cast<uint32_t*>(smem + kSlabBytes + WWAVES * kStageBytes);            // [128]
    uint32_t total = *a.esc_count;
    total = total < a.esc_cap ? total : a.esc_cap;
    if (a.row_begin >= total) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t* stage = reinterpret_cast<uint16_t*>(smem + kSlabBytes + wave * kStageBytes);               // this wave's [64][WLDO]
    float* s_bias = reinterpret_cast<float*>(smem + kSlabBytes + wave * kStageBytes + (size_t)WSTAGE * WLDO * 2); // this wave's [64]
    const uint32_t nb_total = (a.N + 31u) / 32u;
    const uint32_t KS = (a.K + WSLAB - 1) / WSLAB * WRING; // k-steps, padded to whole slabs
    const uint32_t n_slabs = KS / WRING;
    // What a block works on, item after item: a row block with all its column blocks (walk), or one tile, the tiles
    // of a column block following each other.
    const uint32_t rb_chunk = (a.rows_cap + WBM - 1u) / WBM, rb_exist = (total - a.row_begin + WBM - 1u) / WBM;
    const uint32_t rb_count = rb_exist < rb_chunk ? rb_exist : rb_chunk;
    const uint32_t rows = total - a.row_begin < a.rows_cap ? total - a.row_begin : a.rows_cap; // of this chunk
    const uint32_t units = gridDim.x;
    const bool walk = wide_walks(rb_count, n_cb, units, RESIDENT);
    float4* s_sums = reinterpret_cast<float4*>(smem + kWideLds); // [row block of 32][4][64]
    float* s_b3 = reinterpret_cast<float*>(smem + kWideLds + (size_t)WBM * 32 * 4);
    if (LAST && threadIdx.x < 32u) s_b3[threadIdx.x] = threadIdx.x < a.n_last ? a.b_last[threadIdx.x] : 0.f; // (read several barriers on)
    const uint32_t n_items = walk ? rb_count : rb_count * n_cb;
    const uint32_t cb_per_item = walk ? n_cb : 1u;

    // two 16-byte chunks of a slab per thread: rows r, 8 k-values each
    const uint32_t cr[2] = {tid / (WSLAB / 8), (tid + WWAVES * 64) / (WSLAB / 8)};
    const uint32_t ck = (tid % (WSLAB / 8)) * 8u;
    // raw-bit input: where the two rows' flows start and how many packets they have, once per row block (not per slab)
    uint32_t raw_b0[2] = {0u, 0u}, raw_n[2] = {0u, 0u};
    const float raw_per = AMODE == A_RAW ? 1.f / (float)a.raw_bits : 0.f;
    // where the thread's columns of a slab stand in a flow's header bits: slab sl of the first three
    struct Place {
        uint32_t j, b; // packet, bit
    };
    auto place_of = [&](uint32_t sl) {
        Place p = {0u, sl * WSLAB + ck};
        if (AMODE == A_RAW) raw_carry(a, raw_per, p.j, p.b);
        return p;
    };
    // Slab sl of row block rb as this thread's two chunks.  Header bits are only requested here, as words, and turned into
    // bfloat16 when the slab is stored: made here, the wave would wait for the words, and for every weight request
    // before them, ahead of the slab's MFMAs.  (100,000 rows of 8 x 31 bits through 1024-512: 242 us a call; with the bits
    // made here 432, of 10 x 477 bits 1,051 and 2,831.)
    auto fetch = [&](uint32_t rb, uint32_t sl, const Place& p, uint4 (&r)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (AMODE == A_RAW)
                r[u] = raw_words_at<FORM>(a, raw_b0[u], raw_n[u], p.j, p.b); // (past K: packets that raw_pkts leaves out)
            else if (AMODE == A_FEAT)
                r[u] = load_a_chunk<AMODE>(a, a.row_begin + rb * WBM + cr[u] < total, 0u, s_flow[cr[u]], sl * WSLAB + ck);
            else { // (lda is K rounded up to whole slabs and the padding holds zeros; a row past the end repeats the last one)
                const uint32_t left = rows - rb * WBM - 1u;
                const uint32_t at = (cr[u] < left ? cr[u] : left) * a.lda + ck;
                r[u] = *reinterpret_cast<const uint4*>(a.a_bf16 + (size_t)rb * WBM * a.lda + sl * WSLAB + at);
            }
        }
    };
    auto store = [&](uint32_t buf, const Place& p, const uint4 (&r)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            *reinterpret_cast<uint4*>(slab + buf * (WBM * WLDS) + cr[u] * WLDS + ck) =
                AMODE == A_RAW ? raw_bits_of<FORM>(a, r[u], p.b) : r[u];
    };
    // weight operands of a column block: a 32-column block past the end repeats the last one, its results are not
    // stored.  (A wave whose columns all lie past the end still runs the loop: a branch around the refills would
    // make the wait in front of the slab store, which is placed for the worst path, drain the whole ring once
    // per slab.)
    auto operands_of = [&](uint32_t cb, const uint4* (&w)[WNI]) {
#pragma unroll
        for (int j = 0; j < WNI; ++j) {
            const uint32_t nb = cb * (WBN / 32u) + wave * WNI + j;
            w[j] = ws + (size_t)(nb < nb_total ? nb : nb_total - 1u) * KS * 64u;
        }
    };
    auto bias_of = [&](uint32_t cb) {
        const uint32_t col = cb * WBN + wave * WCOLS + lane;
        return col < a.N ? a.bias[col] : 0.f;
    };
    const uint32_t arow_at = (lane & 31u) * WLDS + 8u * (lane >> 5); // this lane's place in an A operand
    const uint4* wl[WNI];
    uint4 fb[WRING][WNI]; // weight operands: a ring of WRING k-steps
    uint4 fa[2][WMI];     // A operands of this and of the next k-step
    uint32_t buf = 0;     // buffer of the current slab
    // stream: the A operand runs two slabs ahead of the MFMAs, on into the next item
    constexpr bool kSeamless = AMODE == A_BF16;
    bool filled = false; // the first slabs of the item are in place
    Place ahead = {0u, 0u}; // of the slab that is requested next

    for (uint32_t item = blockIdx.x; item < n_items; item += units) {
        const uint32_t rb = walk ? item : item % rb_count, cb_first = walk ? 0u : item / rb_count;
        const uint32_t next = item + units;
        const bool has_next = next < n_items;
        const uint32_t rb_next = walk ? next : next % rb_count, cb_next = walk ? 0u : next / rb_count;
        const uint32_t row0 = a.row_begin + rb * WBM; // first escalated row of the item
        if (!filled) {
            __syncthreads(); // the buffers and flow ids of the item before are free
            if (AMODE != A_BF16) {
                if (tid < WBM) {
                    uint32_t f = row0 + tid < total ? a.esc_idx[row0 + tid] : 0u;
                    s_flow[tid] = f < a.n_rows ? f : a.n_rows - 1u; // a bad list entry must not leave the input
                }
                __syncthreads();
            }
            if (AMODE == A_RAW) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    raw_b0[u] = raw_n[u] = 0u;
                    if (row0 + cr[u] < total) raw_flow_range(a, s_flow[cr[u]], raw_b0[u], raw_n[u]); // (no packets: the row reads as zeros)
                }
            }
            uint4 r0[2], r1[2];
            const Place p0 = place_of(0), p1 = place_of(1);
            ahead = place_of(2);
            fetch(rb, 0, p0, r0);
            if (n_slabs > 1u) fetch(rb, 1, p1, r1);
            if (item == blockIdx.x) { // (later items find the ring filled and their first bias in place)
                operands_of(cb_first, wl);
                s_bias[lane] = bias_of(cb_first);
#pragma unroll
                for (int s = 0; s < WRING; ++s) {
#pragma unroll
                    for (int j = 0; j < WNI; ++j) fb[s][j] = wl[j][s * 64 + lane];
                    __builtin_amdgcn_sched_barrier(0); // ring order: keeps the counter waits inside the loop at "oldest load"
                }
            }
            buf = 0;
            store(0, p0, r0);
            if (n_slabs > 1u) store(1, p1, r1);
            if (RESIDENT && n_slabs > 2u) {
                fetch(rb, 2, ahead, r0);
                store(2, ahead, r0);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < WMI; ++i) fa[0][i] = *reinterpret_cast<const uint4*>(slab + arow_at + i * 32 * WLDS);
        }
        filled = kSeamless && !RESIDENT && has_next;

        for (uint32_t c = 0; c < cb_per_item; ++c) {
            const uint32_t cb = cb_first + c, col0 = cb * WBN + wave * WCOLS; // this wave's first column
            const bool last_cb = c + 1u == cb_per_item;
            const uint32_t nb0 = col0 / 32u;
            // the ring goes on to the first k-steps of the next tile's column block (after the last tile: not used)
            const uint32_t cb_after = !last_cb ? cb + 1u : has_next ? cb_next : cb;
            const uint4* nwl[WNI];
            operands_of(cb_after, nwl);
            const float next_bias = bias_of(cb_after);
            // accumulators start at the bias of their column
            f32x16 acc[WMI][WNI];
#pragma unroll
            for (int j = 0; j < WNI; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 b = *reinterpret_cast<const float4*>(s_bias + j * 32u + 8u * g + 4u * (lane >> 5));
#pragma unroll
                    for (int i = 0; i < WMI; ++i) {
                        acc[i][j][4 * g + 0] = b.x;
                        acc[i][j][4 * g + 1] = b.y;
                        acc[i][j][4 * g + 2] = b.z;
                        acc[i][j][4 * g + 3] = b.w;
                    }
                }

            for (uint32_t sl = 0; sl < n_slabs; ++sl) {
                const bool more = sl + 1u < n_slabs;
                // the slab two steps on: of this row block (again from its start for the next column block), or of
                // the next item's.  Activations are requested without a branch, after the last item too (its own row
                // block again, not used): the counter waits in the loop are placed for the path with the fewest requests.
                uint4 ra[2];
                uint32_t sl2 = sl + 2u;
                bool want = true;
                if (!RESIDENT) {
                    uint32_t rb2 = rb;
                    if (sl2 >= n_slabs) {
                        sl2 -= n_slabs;
                        if (last_cb) {
                            rb2 = has_next ? rb_next : rb;
                            want = kSeamless;
                        }
                    }
                    if (sl2 == 0u) ahead = place_of(0);
                    if (want) fetch(rb2, sl2, ahead, ra);
                }
                const uint4* src[WNI]; // this slab's refills: the next slab of the column block, or the next tile's first
#pragma unroll
                for (int j = 0; j < WNI; ++j) src[j] = more ? wl[j] + (size_t)(sl + 1) * WRING * 64u : nwl[j];
                const uint32_t wrap = RESIDENT ? n_slabs : WBUF;
                const uint32_t nbuf = buf + 1u < wrap ? buf + 1u : 0u;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < WRING; ++s) {
                    // A operands of the next k-step, across the slab's end too (the next slab is in place already)
                    const uint16_t* an = slab + (s + 1 < WRING ? buf : nbuf) * (WBM * WLDS) + arow_at + (s + 1) % WRING * 16;
#pragma unroll
                    for (int i = 0; i < WMI; ++i) fa[(s + 1) & 1][i] = *reinterpret_cast<const uint4*>(an + i * 32 * WLDS);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < WNI; ++j) {
                        const bf16x8 b = as_bf16x8(fb[s][j]);
#pragma unroll
                        for (int i = 0; i < WMI; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, as_bf16x8(fa[s & 1][i]), acc[i][j], 0, 0, 0);
                    }
#pragma unroll
                    for (int j = 0; j < WNI; ++j) fb[s][j] = src[j][s * 64u + lane];
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (!RESIDENT) {
                    if (want) store(nbuf + 1u < WBUF ? nbuf + 1u : 0u, ahead, ra);
                    if (AMODE == A_RAW) { // (on to the next slab)
                        ahead.b += WSLAB;
                        raw_carry(a, raw_per, ahead.j, ahead.b);
                    }
                    __syncthreads(); // the slab after the next is in place; nobody reads this one any more
                }
                buf = nbuf;
            }
#pragma unroll
            for (int j = 0; j < WNI; ++j) wl[j] = nwl[j];

            // epilogue: relu, bfloat16; a wave stages 64 rows of its own columns and writes them as whole 128-byte
            // pieces (no other wave is involved, so there is no barrier).  A column block past the last real one holds
            // a repeat of that block's results: stored as zeros.  Columns in [N, ldh) are padding and hold zeros.
            s_bias[lane] = next_bias;
            const uint32_t ln = again(lane);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                // LAST: the wave that multiplies a row block of 32 requests the weights ahead of the rows (steps past the last one: that one again)
                const uint32_t steps = LAST ? ((a.ldh - cb * WBN < (uint32_t)WBN ? a.ldh - cb * WBN : (uint32_t)WBN) / 16u) : 0u;
                const bool mine = LAST && wave / 2u == (uint32_t)half;
                u32x4 lw[LAST ? LRING : 1];
                auto weights = [&](uint32_t t) __attribute__((always_inline)) {
                    return *reinterpret_cast<const u32x4*>(a.wo_last + (cb * (WBN / 16u) + (t < steps ? t : steps - 1u)) * 64u + ln);
                };
                if (mine) {
#pragma unroll
                    for (int t = 0; t < LRING; ++t) lw[LAST ? t : 0] = weights(t);
                }
                if (col0 < a.ldh) { // (ldh is a multiple of the wave's 64 columns)
#pragma unroll
                    for (int j = 0; j < WNI; ++j) {
                        const uint32_t real = nb0 + j < nb_total ? 0xFFFFFFFFu : 0u;
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const uint32_t cl = j * 32u + 8u * g + 4u * (ln >> 5); // column inside the wave's piece
#pragma unroll
                            for (int ih = 0; ih < WMI / 2; ++ih) {
                                const int i = half * (WMI / 2) + ih;
                                const uint32_t row = ih * 32u + (ln & 31u); // row inside the staged half
                                const float y0 = fmaxf(acc[i][j][4 * g + 0], 0.f), y1 = fmaxf(acc[i][j][4 * g + 1], 0.f);
                                const float y2 = fmaxf(acc[i][j][4 * g + 2], 0.f), y3 = fmaxf(acc[i][j][4 * g + 3], 0.f);
                                *reinterpret_cast<uint2*>(stage + row * WLDO + cl) =
                                    make_uint2(pack_bf16(y0, y1) & real, pack_bf16(y2, y3) & real);
                            }
                        }
                    }
                    if (!LAST) {
                        wave_sync();
#pragma unroll
                        for (int q = 0; q < WSTAGE / 8; ++q) {
                            const uint32_t rh = q * 8u + (ln >> 3), k = (ln & 7u) * 8u;
                            const uint32_t r = half * WSTAGE + rh;
                            const uint4 v = *reinterpret_cast<const uint4*>(stage + rh * WLDO + k);
                            if (row0 + r < total) *reinterpret_cast<uint4*>(a.h_out + (size_t)(rb * WBM + r) * a.ldh + col0 + k) = v;
                        }
                        wave_sync(); // the staged rows are out: the space may be written again
                    }
                }
                if (LAST) {
                    __syncthreads(); // all columns are staged
                    if (mine) {
                        const uint32_t blk = wave, in = (wave & 1u) * 32u + (ln & 31u); // row block of the tile, row inside the staged half
                        const unsigned char* arow = smem + kSlabBytes + ((size_t)in * WLDO + 8u * (ln >> 5)) * 2;
                        u32x4 ca[4];
                        auto rows_of = [&](uint32_t t) __attribute__((always_inline)) { // four steps: one wave's columns
                            const uint32_t w = t < steps ? t / 4u : steps / 4u - 1u;
#pragma unroll
                            for (int q = 0; q < 4; ++q) ca[q] = *reinterpret_cast<const u32x4*>(arow + w * kStageBytes + q * 32);
                        };
                        f32x16 sum[1];
                        if (cb == 0u) {
#pragma unroll
                            for (int v = 0; v < 16; ++v) sum[0][v] = 0.f;
                        } else {
#pragma unroll
                            for (int g = 0; g < 4; ++g) {
                                const float4 v = s_sums[(blk * 4u + g) * 64u + ln];
                                sum[0][4 * g] = v.x, sum[0][4 * g + 1] = v.y, sum[0][4 * g + 2] = v.z, sum[0][4 * g + 3] = v.w;
                            }
                        }
                        rows_of(0);
                        for (uint32_t t0 = 0; t0 < steps; t0 += LRING) {
#pragma unroll
                            for (int s = 0; s < LRING; s += 4) {
                                if (t0 + s < steps) { // (steps is a multiple of 4)
#pragma unroll
                                    for (int q = 0; q < 4; ++q)
                                        sum[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, lw[LAST ? s + q : 0]), __builtin_bit_cast(bf16x8, ca[q]), sum[0], 0, 0, 0);
                                    rows_of(t0 + s + 4);
                                }
                                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                for (int q = 0; q < 4; ++q) lw[LAST ? s + q : 0] = weights(t0 + s + q + LRING);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                        if (last_cb) {
                            const uint32_t row = row0 + blk * 32u + (ln & 31u);
                            const bool there = row < total;
                            last_rows<1>(a, sum, s_b3, a.n_last, ln >> 5, there, row, there ? (a.scatter ? a.scatter : a.esc_idx)[row] : 0u);
                        } else {
#pragma unroll
                            for (int g = 0; g < 4; ++g) s_sums[(blk * 4u + g) * 64u + ln] = make_float4(sum[0][4 * g], sum[0][4 * g + 1], sum[0][4 * g + 2], sum[0][4 * g + 3]);
                        }
                    }
                    __syncthreads(); // the staged rows have been read
                }
            }
            wave_sync();
        }
    }
}

// Few rows: a tile of 32 rows x 256 columns a block, a wave 32 columns.  What counts is the chain of latencies and the weights' way
// through one unit's path to the cache (half a megabyte for K = 1,024), so the weights are requested first, 16 k-steps ahead, and the
// rows' values come to shared memory 1,024 at a time, so that waves meet once in as many k-steps.  A sum starts at its bias and runs in
// order of K, as in the tiles: the same bits.  Tiles of 128 x 512 : these, whole call in us: one
// row through 64-1024-1024-10 42.0 : 18.5, 500 46.5 : 22.6, 2,000 46.6 : 27.4, 500 through 96-300-900-20 45.0 : 20.3.
template <int AMODE, int FORM>
__device__ __forceinline__ void wide_few(const LayerArgs& a, const uint4* __restrict__ ws, uint32_t rows, unsigned char* smem)
{
    uint16_t* A = reinterpret_cast<uint16_t*>(smem); // [2][32][FLD]
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t n_cb = (a.ldh + kFewTileCols - 1u) / kFewTileCols, cb = blockIdx.x % n_cb, row0 = blockIdx.x / n_cb * kFewTileRows;
    if (row0 >= rows) return;
    const uint32_t nb_total = (a.N + 31u) / 32u, nb = cb * (kFewTileCols / 32u) + wave, KS = (a.K + WSLAB - 1u) / WSLAB * (WSLAB / 16u);
    const uint4* w = ws + (size_t)(nb < nb_total ? nb : nb_total - 1u) * KS * 64u + lane;
    uint4 fb[FRING];
#pragma unroll
    for (int s = 0; s < FRING; ++s) fb[s] = w[((uint32_t)s < KS ? s : KS - 1u) * 64u];
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t r = tid >> 4, k8 = (tid & 15u) * 8u; // this thread's row and its first values of 128
    const uint32_t left = rows - row0 - 1u, mine = r < left ? r : left; // (a row past the end: the last one again, not stored)
    uint32_t flow = 0, raw_b0 = 0, raw_n = 0;
    if (AMODE != A_BF16) {
        flow = a.esc_idx[a.row_begin + row0 + mine];
        flow = flow < a.n_rows ? flow : a.n_rows - 1u; // a bad list entry must not leave the input
        if (AMODE == A_RAW) raw_flow_range(a, flow, raw_b0, raw_n);
    }
    constexpr int kMine = FCHUNK / 128; // 16-byte pieces of a thread
    uint32_t __attribute__((ext_vector_type(4))) ra[kMine]; // (as uint4 the compiler keeps the array in memory)
    auto fetch = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < kMine; ++u) {
            uint4 v;
            const uint32_t k = k0 + u * 128u + k8;
            if (AMODE == A_RAW) {
                const uint32_t j = k / a.raw_bits, b = k - j * a.raw_bits;
                const uint4 words = raw_words_at<FORM>(a, raw_b0, raw_n, j, b); // (past K: packets that raw_pkts leaves out)
                v = raw_bits_of<FORM>(a, words, b);
            } else if (AMODE == A_FEAT) {
                v = load_a_chunk<AMODE>(a, true, 0u, flow, k);
            } else { // (lda is K rounded up to whole slabs and the padding holds zeros)
                const uint32_t at = k < a.lda ? k : 0u;
                v = *reinterpret_cast<const uint4*>(a.a_bf16 + (size_t)(row0 + mine) * a.lda + at);
            }
            ra[u] = {v.x, v.y, v.z, v.w};
        }
    };
    auto store = [&](uint32_t buf) {
#pragma unroll
        for (int u = 0; u < kMine; ++u) *reinterpret_cast<uint4*>(A + ((size_t)buf * kFewTileRows + r) * FLD + u * 128 + k8) = make_uint4(ra[u].x, ra[u].y, ra[u].z, ra[u].w);
    };
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint32_t col = nb * 32u + 8u * (v >> 2) + 4u * (lane >> 5) + (v & 3);
        const float b = a.bias[col < a.N ? col : a.N - 1u];
        acc[v] = col < a.N ? b : 0.f; // (padding holds zeros: an infinite value there would not vanish behind a zero weight)
    }
    fetch(0);
    store(0);
    __syncthreads();
    uint32_t buf = 0;
    for (uint32_t c0 = 0; c0 < KS; c0 += FCHUNK / 16) {
        const bool more = c0 + FCHUNK / 16 < KS;
        if (more) fetch((c0 + FCHUNK / 16) * 16u);
        const uint32_t end = more ? c0 + FCHUNK / 16 : KS;
        const uint16_t* arow = A + ((size_t)buf * kFewTileRows + (lane & 31u)) * FLD + 8u * (lane >> 5);
        for (uint32_t k0 = c0; k0 < end; k0 += FRING) { // (KS is a multiple of 4)
#pragma unroll
            for (int s0 = 0; s0 < FRING; s0 += 4) {
                if (k0 + s0 < end) {
                    uint4 fa[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) fa[q] = *reinterpret_cast<const uint4*>(arow + (k0 - c0 + s0 + q) * 16u);
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fb[s0 + q]), as_bf16x8(fa[q]), acc, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = s0; s < s0 + 4; ++s) {
                    const uint32_t ks = k0 + s + FRING;
                    fb[s] = w[(ks < KS ? ks : KS - 1u) * 64u];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (more) {
            store(buf ^ 1u);
            __syncthreads(); // the next values are in place; the buffer before is written again a chunk further on
            buf ^= 1u;
        }
    }
    // relu, bfloat16; a column block past the last real one holds zeros, as the padding does
    const uint32_t real = nb < nb_total ? 0xFFFFFFFFu : 0u;
    if (nb * 32u < a.ldh && (lane & 31u) <= left) {
        uint16_t* out = a.h_out + (size_t)(row0 + (lane & 31u)) * a.ldh + nb * 32u + 4u * (lane >> 5);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<uint2*>(out + 8 * g) = make_uint2(pack_bf16(fmaxf(acc[4 * g], 0.f), fmaxf(acc[4 * g + 1], 0.f)) & real,
                                                                pack_bf16(fmaxf(acc[4 * g + 2], 0.f), fmaxf(acc[4 * g + 3], 0.f)) & real);
    }
}

// this block's share of labels = pred, 16 bytes a thread at a time where both are aligned
__device__ __forceinline__ void copy_labels_slice(const uint16_t* __restrict__ pred, uint16_t* __restrict__ labels, uint32_t n)
{
    const uint32_t step = gridDim.x * WWAVES * 64u, at = blockIdx.x * WWAVES * 64u + threadIdx.x;
    const uint32_t whole = ((reinterpret_cast<uintptr_t>(pred) | reinterpret_cast<uintptr_t>(labels)) & 15u) == 0 ? n / 8u : 0u;
    for (uint32_t i = at; i < whole; i += step) reinterpret_cast<uint4*>(labels)[i] = reinterpret_cast<const uint4*>(pred)[i];
    for (uint32_t i = whole * 8u + at; i < n; i += step) labels[i] = pred[i];
}

// The form for the rows that there are.  (A copy of the code for each: with and without the last layer through one, the write-out
// of the activations cost 2,400 clocks a tile more.)
template <int AMODE, bool RESIDENT, int FORM, bool LAST>
__device__ __forceinline__ void wide_any(const LayerArgs& a, const uint4* __restrict__ ws, uint32_t n_cb, unsigned char* smem)
{
    uint32_t total = *a.esc_count;
    total = total < a.esc_cap ? total : a.esc_cap;
    // the fast labels, which the last layer's launch writes over (as a launch of their own: 4.6 us for 65,536 flows, here under 2)
    if (AMODE != A_BF16 && a.pred) copy_labels_slice(a.pred, a.labels, a.n_labels);
    if (a.row_begin >= total) return;
    const uint32_t left = total - a.row_begin, rows = left < a.rows_cap ? left : a.rows_cap;
    if (wide_few_tiles(rows, a.ldh) <= gridDim.x)
        wide_few<AMODE, FORM>(a, ws, rows, smem);
    else if (LAST && wide_takes_last(rows, a.ldh, gridDim.x, RESIDENT))
        wide_tiles<AMODE, RESIDENT, FORM, LAST>(a, ws, n_cb, smem);
    else
        wide_tiles<AMODE, RESIDENT, FORM, false>(a, ws, n_cb, smem);
}

template <int AMODE, bool RESIDENT, int FORM>
__global__ __launch_bounds__(WWAVES * 64) void mlp_wide_layer(LayerArgs a, const uint4* __restrict__ ws, uint32_t n_cb)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    wide_any<AMODE, RESIDENT, FORM, false>(a, ws, n_cb, smem);
}

template <bool RESIDENT>
__global__ __launch_bounds__(WWAVES * 64) void mlp_wide_last(LayerArgs a, const uint4* __restrict__ ws, uint32_t n_cb)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    wide_any<A_BF16, RESIDENT, 0, true>(a, ws, n_cb, smem);
}

template <int AMODE, bool RESIDENT, int FORM, bool LAST>
int launch_wide(sf_ctx* ctx, int slot, LayerArgs a, const void* w_ordered, uint32_t rows_cap)
{
    auto* kernel = mlp_wide_layer<AMODE, RESIDENT, FORM>;
    if constexpr (LAST) kernel = mlp_wide_last<RESIDENT>;
    SF_ALLOW_LDS(ctx, slot, kernel);
    a.rows_cap = rows_cap;
    const uint32_t n_cb = (a.ldh + WBN - 1) / WBN;
    kernel<<<sf::wide_blocks(ctx, a.ldh, rows_cap), WWAVES * 64, (kWideLds > kFewLds ? kWideLds : kFewLds) + (LAST ? kLastLds : 0), ctx->stream>>>(a, (const uint4*)w_ordered, n_cb);
    SF_LAUNCH_CHECK(ctx, "mlp_wide_layer");
    return SF_OK;
}

template <int AMODE, int FORM, bool LAST = false>
int launch_wide(sf_ctx* ctx, int slot, const LayerArgs& a, const void* w_ordered, uint32_t rows_cap)
{
    if ((a.K + WSLAB - 1) / WSLAB <= WBUF) return launch_wide<AMODE, true, FORM, LAST>(ctx, slot, a, w_ordered, rows_cap);
    return launch_wide<AMODE, false, FORM, LAST>(ctx, slot + 1, a, w_ordered, rows_cap);
}

} // namespace

namespace sf {

uint32_t wide_blocks(const sf_ctx* ctx, uint32_t ldh, uint32_t rows_cap)
{
    const uint64_t tiles = wide_few_tiles(rows_cap, ldh);
    return tiles < (uint64_t)ctx->n_cu ? (uint32_t)tiles : (uint32_t)ctx->n_cu; // one block per compute unit
}

int wide_layer(sf_ctx* ctx, int amode, const sfmlp::LayerArgs& a, const void* w_ordered, uint32_t rows_cap)
{
    if (amode == A_BF16 && a.n_last) return launch_wide<A_BF16, 0, true>(ctx, sf::kLdsWideLast, a, w_ordered, rows_cap);
    if (amode == A_BF16) return launch_wide<A_BF16, 0>(ctx, sf::kLdsWide, a, w_ordered, rows_cap);
    if (amode == A_FEAT) return launch_wide<A_FEAT, 0>(ctx, sf::kLdsWide + 2, a, w_ordered, rows_cap);
    if ((a.raw_bits & 7u) == 0) return launch_wide<A_RAW, RAW_BYTES>(ctx, sf::kLdsWide + 4, a, w_ordered, rows_cap);
    if (a.raw_bits > 8u) return launch_wide<A_RAW, RAW_LONG>(ctx, sf::kLdsWide + 6, a, w_ordered, rows_cap);
    return launch_wide<A_RAW, RAW_SHORT>(ctx, sf::kLdsWide + 8, a, w_ordered, rows_cap);
}

} // namespace sf
