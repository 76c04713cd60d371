// The GEMMs of the sparse and the dense MLP where there are too few of the larger tiles to fill the chip: tiles of 64 x 64.
// Internal to mlp.hip.
//
// A workgroup of four waves (32 x 32 of the tile each) walks the contraction in steps of 64.  A step's operands are two tiles
// of 8 KB in a ring of four stages in LDS, and the step after the one that is multiplied is already in registers, so a stage is
// free again as soon as its operands have been read: two workgroups per CU have 128 KB in flight.  (One with eight stages
// takes the same time where it is alone and up to 1.7 times as long where tiles wait for a CU.)
//
// Bound: the CU's path from L2 (about 60 bytes a cycle: 273 cycles for the 16 KB of a step, of which the products take 128)
// once the ring hides the latency.  Measured, in us against the chunk's tiles: first GEMM 9 chunks of 192 x 395 of 7488 x 4864
// 44 -> 19, 4 x 249 of 5248 x 1408 22 -> 8.9; second 9.3 -> 5.0 (the latter), dense 509 x 4800 x 640 51 -> 19; but 17 chunks x 1229
// of 12 288 x 3072 36 and 44, 38 and 56: where the larger tiles fill the chip they fetch a third of the bytes.
#pragma once
#include "common.h"

namespace chipmunk {

constexpr int kSmallTile = 64;
constexpr int kSmallStages = 4;
constexpr int kSmallStage = 2 * kSmallTile * 128;        // bytes: two operand tiles of 64 x 64
constexpr int kSmallRow1 = kSmallTile * 2 + 16;          // row strides (bytes) of the results on their way out: first GEMM,
constexpr int kSmallRow2 = kSmallTile * 4 + 16;          // bf16, and second, fp32

// Waits until at most `steps` steps' transfers (four per wave and step) are outstanding, as far as the ring holds any.
__device__ __forceinline__ void wait_small_steps(int steps) {
    static_assert(kSmallStages == 4, "the cases below");
    if (steps >= 3) wait_vmem_at_most<12>();
    else if (steps == 2) wait_vmem_at_most<8>();
    else if (steps == 1) wait_vmem_at_most<4>();
    else wait_vmem_at_most<0>();
}

// acc[a][c] += P_a Q_c over all steps.  request(t): the wave's four transfers of step t into stage t % 4; read(set, t): the
// wave's operands of step t from there.
template <typename Request, typename Read>
__device__ __forceinline__ void small_contraction(int steps, f32x4 (&acc)[2][2], Request&& request, Read&& read) {
    typedef bf16x8 Operands[2][2][2];                    // [P, Q][block][slice of 32]
    Operands even, odd;
    constexpr int NS = kSmallStages;
    for (int t = 0; t < min(NS, steps); t++) request(t);
    wait_small_steps(min(NS, steps) - 1);
    lds_accesses_then_barrier();
    read(even, 0);
    auto step = [&](auto ends_c, int t, Operands& now, Operands& next) {
        constexpr bool ends = decltype(ends_c)::value;   // the ring runs empty
        if (ends) wait_small_steps(min(NS - 2, steps - 2 - t));   // step t + 1 has landed
        else wait_vmem_at_most<(NS - 2) * 4>();
        lds_accesses_then_barrier();                     // for every wave; and every wave holds its operands of step t
        if (!ends || t + 1 < steps) read(next, t + 1);
        __builtin_amdgcn_sched_barrier(0);               // the reads lead: they land behind this step's products
        if (!ends || t + NS < steps) request(t + NS);
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int c = 0; c < 2; c++)
                    acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now[0][a][ks], now[1][c][ks], acc[a][c], 0, 0, 0);
    };
    int t = 0;
    for (; t + NS + 1 < steps; t += 2) {
        step(std::false_type{}, t, even, odd);
        step(std::false_type{}, t + 1, odd, even);
    }
    for (; t < steps; t += 2) {
        step(std::true_type{}, t, even, odd);
        if (t + 1 < steps) step(std::true_type{}, t + 1, odd, even);
    }
    lds_accesses_then_barrier();                         // every wave is done with the stages
}

// The tiles in runs, one per XCD (xcd_run_tile).  Sparse: a chunk's tiles back to back, those of one piece of its list (the same
// gathered rows) next to each other; dense: in bands of eight row tiles.
template <bool SPARSE>
__device__ __forceinline__ bool small_tile_of_block(int col_tiles, int units, int parts, int* unit, int* part, int* col_tile) {
    if (!SPARSE) {
        *part = 0;
        return xcd_tile_of_block_grouped((int)blockIdx.x >> 3, col_tiles, units, unit, col_tile);
    }
    int tile;
    if (!xcd_run_tile((int)blockIdx.x & 7, (int)blockIdx.x >> 3, units * col_tiles * parts, &tile)) return false;
    const int rest = tile / parts;
    *part = tile - rest * parts;
    *unit = rest / col_tiles;
    *col_tile = rest - *unit * col_tiles;
    return true;
}

// First GEMM: a[n][f] = act(<x[n], w1[f]> + b1[f]) for 64 tokens and 64 neurons; sparse: of a chunk's list, with the delta
// epilogue.  The products add in the order of the larger tiles, so the results are theirs bit for bit.
template <int MODE>
__global__ __launch_bounds__(256, 2) void mlp_small_gemm1_kernel(Gemm1Params p) {
    constexpr bool SPARSE = MODE == kSparseDelta;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    __shared__ int32_t s_neuron[kSmallTile];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = w & 1, g = lane >> 4, l16 = lane & 15;

    int unit, part, col_tile;
    if (!small_tile_of_block<SPARSE>(p.col_tiles, p.units, p.parts, &unit, &part, &col_tile)) return;
    const int b = unit / p.NB, row0 = (unit - b * p.NB) * p.parts * kSmallTile + part * kSmallTile;
    const int col0 = col_tile * kSmallTile;
    const int count = SPARSE ? min(p.counts[unit], p.k_stride) : p.F;   // clamped like the indices below
    if (row0 >= p.N || col0 >= count) return;
    if (tid < kSmallTile) {   // columns at or beyond count compute a duplicate that is never stored
        const int at = min(col0 + tid, count - 1);
        s_neuron[tid] = SPARSE ? min(max(p.idx[(int64_t)unit * p.k_stride + at], 0), p.F - 1) : at;
    }
    __syncthreads();

    const i32x4 xbuf = raw_buffer_words(p.x + (int64_t)b * p.N * p.D, (uint32_t)p.N * p.D * 2u);
    const i32x4 wbuf = raw_buffer_words(p.w1, (uint32_t)p.F * p.D * 2u);
    uint32_t xoff[2], woff[2];                           // 8 rows of 128 bytes a transfer; 16-byte chunks XOR-swizzled by the row
#pragma unroll
    for (int n = 0; n < 2; n++) {
        const int row = (n * 4 + w) * 8 + (lane >> 3);
        const uint32_t chunk = (uint32_t)((lane & 7) ^ ((row >> 1) & 7)) * 16u;
        xoff[n] = (uint32_t)min(row0 + row, p.N - 1) * (uint32_t)(p.D * 2) + chunk;
        woff[n] = (uint32_t)s_neuron[row] * (uint32_t)(p.D * 2) + chunk;
    }
    // the thread's two cells (eight tokens of a neuron) and its bias: requested here, used behind the contraction
    const uint16_t* bias_src = p.b1 ? p.b1 : p.w1;       // a valid address when there is none
    uint16_t bias_raw[2];
#pragma unroll
    for (int c = 0; c < 2; c++) bias_raw[c] = bias_src[s_neuron[wn * 32 + c * 16 + l16]];
    const int ch = tid & 7, tok0 = row0 + ch * 8;
    uint16_t* cell[2];                                   // tokens clamped to the row's start where the chunk ends early: not used
    u32x4 old8[2];
#pragma unroll
    for (int n = 0; n < 2; n++) {
        cell[n] = p.a_cache + ((int64_t)b * p.F + s_neuron[n * 32 + (tid >> 3)]) * p.a_ld + (tok0 < p.N ? tok0 : 0);
        if (SPARSE) old8[n] = *reinterpret_cast<const u32x4*>(cell[n]);
    }

    const uint32_t lds0 = lds_address(smem);
    auto request = [&](int t) {
        const uint32_t stage = lds0 + (uint32_t)((t & (kSmallStages - 1)) * kSmallStage), from = (uint32_t)t * 128u;
#pragma unroll
        for (int n = 0; n < 2; n++) {
            load_buffer_to_lds_16B(xbuf, xoff[n], from, stage + (n * 4 + w) * 1024);
            load_buffer_to_lds_16B(wbuf, woff[n], from, stage + kSmallStage / 2 + (n * 4 + w) * 1024);
        }
    };
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
    const uint32_t in_row = (uint32_t)((g ^ ((l16 >> 1) & 7)) * 16);
    uint32_t xat[2], wat[2];                             // by slice; opaque, so that what is added stays in the reads' offset field
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
        xat[ks] = smem_at + (uint32_t)((wm * 32 + l16) * 128) + (in_row ^ (64u * ks));
        wat[ks] = smem_at + (uint32_t)(kSmallStage / 2 + (wn * 32 + l16) * 128) + (in_row ^ (64u * ks));
        asm volatile("" : "+v"(xat[ks]), "+v"(wat[ks]));
    }
    auto read = [&](bf16x8 (&op)[2][2][2], int t) {
        const uint32_t stage = (uint32_t)((t & (kSmallStages - 1)) * kSmallStage);
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < 2; a++) {
                op[0][a][ks] = lds_read_b128(xat[ks] + stage + a * 2048);
                op[1][a][ks] = lds_read_b128(wat[ks] + stage + a * 2048);
            }
    };
    f32x4 acc[2][2] = {};
    small_contraction(p.D / kBK, acc, request, read);

    // activations through LDS as [neuron][token]; then per cell: delta^T, the new activations
    auto to_lds = [&](auto form) {
        constexpr int ACT = decltype(form)::value;
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const float bias = p.b1 ? bf16_bits_to_float(bias_raw[c]) : 0.f;
#pragma unroll
            for (int a = 0; a < 2; a++) {
                const f32x4 v = acc[a][c];
                *reinterpret_cast<u32x2*>(smem + (wn * 32 + c * 16 + l16) * kSmallRow1 + (wm * 32 + a * 16 + 4 * g) * 2) =
                    u32x2{pack_bf16x2(gelu<ACT>(v[0] + bias), gelu<ACT>(v[1] + bias)),
                          pack_bf16x2(gelu<ACT>(v[2] + bias), gelu<ACT>(v[3] + bias))};
            }
        }
    };
    if (p.act == CHIPMUNK_ACT_GELU_ERF) to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_ERF>{});
    else to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_TANH>{});
    lds_accesses_then_barrier();
    u32x4 a8[2];
#pragma unroll
    for (int n = 0; n < 2; n++) a8[n] = *reinterpret_cast<const u32x4*>(smem + (n * 32 + (tid >> 3)) * kSmallRow1 + ch * 16);
    const int64_t c_tokens = (int64_t)p.parts * kSmallTile;
#pragma unroll
    for (int n = 0; n < 2; n++) {
        const int s = col0 + n * 32 + (tid >> 3);
        // tokens past N and padding rows of the contraction must read as zero in the second GEMM
        const int nvalid = s < count ? min(8, p.N - tok0) : 0;
        const int64_t at = ((int64_t)unit * p.k_pad + s) * c_tokens + part * kSmallTile + ch * 8;
        if (SPARSE) {
            u32x4 d8;
#pragma unroll
            for (int e2 = 0; e2 < 4; e2++) {
                float dlo = bf16_bits_to_float(a8[n][e2] & 0xffffu) - bf16_bits_to_float(old8[n][e2] & 0xffffu);
                float dhi = bf16_bits_to_float(a8[n][e2] >> 16) - bf16_bits_to_float(old8[n][e2] >> 16);
                if (2 * e2 >= nvalid) dlo = 0.f;
                if (2 * e2 + 1 >= nvalid) dhi = 0.f;
                d8[e2] = pack_bf16x2(dlo, dhi);
            }
            *reinterpret_cast<u32x4*>(p.delta_t + at) = d8;   // s < k_pad: the list's last tile of 64 lies below it
        }
        if (SPARSE && p.act_t) {   // deferred write-back: one coalesced store, whole cell
            if (nvalid > 0) *reinterpret_cast<u32x4*>(p.act_t + at) = a8[n];
        } else if (nvalid == 8) {
            *reinterpret_cast<u32x4*>(cell[n]) = a8[n];
        } else {                   // the cells past N in the last chunk stay as they are
            for (int e = 0; e < nvalid; e++) cell[n][e] = (uint16_t)(a8[n][e >> 1] >> (16 * (e & 1)));
        }
    }
}

// Second GEMM: o[n][d] (+)= sum_s a[s][n] w2[f(s)][d] (+ b2[d]) for 64 tokens and 64 output columns.  Both operands have the
// contraction index slowest and come out of LDS through the transposing read.  SPARSE: dynamic LDS ends with the list as
// byte offsets of the w2 rows, padded to whole steps (a slot at or beyond count repeats the last row; its deltas are zero).
template <bool SPARSE>
__global__ __launch_bounds__(256, 2) void mlp_small_gemm2_kernel(Gemm2Params p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wt = w >> 1, wc = w & 1, g = lane >> 4, l16 = lane & 15;
    if (SPARSE && p.act_t && (int)blockIdx.x >= p.tile_blocks) {
        // (the chunk's size a constant in each call: the loop divides by it)
        if (p.parts == 3) write_back_activations(p, (int)blockIdx.x - p.tile_blocks, 192);
        else write_back_activations(p, (int)blockIdx.x - p.tile_blocks, 128);
        return;
    }
    int unit, part, col_tile;
    if (!small_tile_of_block<SPARSE>(p.col_tiles, p.units, p.parts, &unit, &part, &col_tile)) return;
    const int b = unit / p.NB, c_tokens = p.parts * kSmallTile;
    const int row0 = (unit - b * p.NB) * c_tokens + part * kSmallTile;
    const int d0 = col_tile * kSmallTile;
    const int count = SPARSE ? min(p.counts[unit], p.k_stride) : p.F;
    if (row0 >= p.N || count <= 0) return;               // nothing selected: the cache stays as it is
    const int steps = (count + kBK - 1) / kBK;
    uint32_t* s_row = reinterpret_cast<uint32_t*>(smem + kSmallStages * kSmallStage);
    if (SPARSE) {
        const int32_t* list = p.idx + (int64_t)unit * p.k_stride;
        for (int s = tid; s < steps * kBK; s += 256)
            s_row[s] = (uint32_t)min(max(list[min(s, count - 1)], 0), p.F - 1) * (uint32_t)(p.D * 2);
    }
    // what is added to (the cached output, or the bias): requested here, used behind the contraction
    const int ch = tid & 7;
    u32x4 old8[2];
#pragma unroll
    for (int n = 0; n < 2; n++) {
        const int tok = min(row0 + n * 32 + (tid >> 3), p.N - 1);
        // (the dense form without a bias reads the output buffer and does not use it)
        const uint16_t* src = !SPARSE && p.bias ? p.bias + d0 + ch * 8 : p.o + ((int64_t)b * p.N + tok) * p.D + d0 + ch * 8;
        if (SPARSE) {
            old8[n] = *reinterpret_cast<const u32x4*>(src);
        } else {                                         // b2 is aligned to four elements only
            const u32x2 lo = *reinterpret_cast<const u32x2*>(src), hi = *reinterpret_cast<const u32x2*>(src + 4);
            old8[n] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    }
    if (SPARSE) __syncthreads();

    const int64_t a_row = SPARSE ? c_tokens : p.a_ld;    // elements between consecutive contraction rows
    const i32x4 abuf = SPARSE ? raw_buffer_words(p.a_t + (int64_t)unit * p.k_pad * c_tokens, (uint32_t)p.k_pad * c_tokens * 2u)
                              : raw_buffer_words(p.a_t + (int64_t)b * p.F * p.a_ld, (uint32_t)p.F * (uint32_t)p.a_ld * 2u);
    const i32x4 wbuf = raw_buffer_words(p.w2, (uint32_t)p.F * p.D * 2u);
    const uint32_t astep = (uint32_t)(kBK * a_row * 2), wstep = SPARSE ? 0u : (uint32_t)(kBK * p.D * 2);
    uint32_t aoff[2], woff[2];
    int srow[2];
#pragma unroll
    for (int n = 0; n < 2; n++) {
        const int row = (n * 4 + w) * 8 + (lane >> 3), col = ((lane & 7) ^ (row & 6)) * 8;
        // dense: tokens beyond N repeat the last ones that exist and are not stored
        aoff[n] = (uint32_t)(row * a_row * 2) + (uint32_t)(SPARSE ? part * kSmallTile + col : min(row0 + col, (p.N - 1) & ~7)) * 2u;
        woff[n] = (SPARSE ? 0u : (uint32_t)row * (uint32_t)(p.D * 2)) + (uint32_t)(d0 + col) * 2u;
        srow[n] = row;
    }
    const uint32_t lds0 = lds_address(smem);
    uint32_t row_at[2] = {};                             // SPARSE: the w2 rows of the next step to be requested
    if (SPARSE) row_at[0] = s_row[srow[0]], row_at[1] = s_row[srow[1]];
    auto request = [&](int t) {
        const uint32_t stage = lds0 + (uint32_t)((t & (kSmallStages - 1)) * kSmallStage);
#pragma unroll
        for (int n = 0; n < 2; n++) {
            load_buffer_to_lds_16B(abuf, aoff[n], (uint32_t)t * astep, stage + (n * 4 + w) * 1024);
            load_buffer_to_lds_16B(wbuf, woff[n] + row_at[n], (uint32_t)t * wstep, stage + kSmallStage / 2 + (n * 4 + w) * 1024);
        }
        if (SPARSE) {
            const int next = min(t + 1, steps - 1) * kBK;
#pragma unroll
            for (int n = 0; n < 2; n++) row_at[n] = s_row[next + srow[n]];
        }
    };
    // P: w2 columns, Q: tokens.  Within 16 lanes, lane i addresses row i / 4 of four and 4 consecutive columns.
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
    const int trow = 4 * g + (l16 >> 2);
    uint32_t wat[2], aat[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int sub = (l16 & 3) >> 1, swz = trow & 6;   // eight rows' 32-byte pieces in 256 different bytes
        wat[i] = smem_at + (uint32_t)(kSmallStage / 2 + trow * 128 + (((wc * 4 + i * 2 + sub) ^ swz) * 16) + 8 * (l16 & 1));
        aat[i] = smem_at + (uint32_t)(trow * 128 + (((wt * 4 + i * 2 + sub) ^ swz) * 16) + 8 * (l16 & 1));
        asm volatile("" : "+v"(wat[i]), "+v"(aat[i]));
    }
    auto read = [&](bf16x8 (&op)[2][2][2], int t) {
        const uint32_t stage = (uint32_t)((t & (kSmallStages - 1)) * kSmallStage);
        auto block = [&](uint32_t at) -> bf16x8 {
            typedef __attribute__((ext_vector_type(8))) short short8v;
            return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lds_read_tr16_at(at), lds_read_tr16_at(at + 16 * 128),
                                                                              0, 1, 2, 3, 4, 5, 6, 7));
        };
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int i = 0; i < 2; i++) {
                op[0][i][ks] = block(wat[i] + stage + ks * 32 * 128);
                op[1][i][ks] = block(aat[i] + stage + ks * 32 * 128);
            }
    };
    f32x4 acc[2][2] = {};
    small_contraction(steps, acc, request, read);

    // fp32 through LDS as [token][column], added to once and stored in runs of 128 bytes
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int c = 0; c < 2; c++)
            *reinterpret_cast<f32x4*>(smem + (wt * 32 + c * 16 + l16) * kSmallRow2 + (wc * 32 + a * 16 + 4 * g) * 4) = acc[a][c];
    lds_accesses_then_barrier();
    const bool add_nothing = !SPARSE && !p.bias;
#pragma unroll
    for (int n = 0; n < 2; n++) {
        const int tl = n * 32 + (tid >> 3);
        f32x4 sum[2];
#pragma unroll
        for (int h = 0; h < 2; h++) sum[h] = *reinterpret_cast<const f32x4*>(smem + tl * kSmallRow2 + ch * 32 + h * 16);
        u32x4 res;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t o2 = add_nothing ? 0u : old8[n][e];
            res[e] = pack_bf16x2(bf16_bits_to_float(o2 & 0xffffu) + sum[e >> 1][2 * (e & 1)],
                                 bf16_bits_to_float(o2 >> 16) + sum[e >> 1][2 * (e & 1) + 1]);
        }
        if (row0 + tl < p.N) *reinterpret_cast<u32x4*>(p.o + ((int64_t)b * p.N + row0 + tl) * p.D + d0 + ch * 8) = res;
    }
}

}  // namespace chipmunk
