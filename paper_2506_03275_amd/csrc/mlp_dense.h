// The two GEMMs of the dense MLP (Alg. 5) at sizes that fill the chip, the scores GEMM (Alg. 7), and the first GEMM of the
// column-sparse form where its tiles make fewer rounds.  Internal to mlp.hip, which chooses between these and the tiles of
// 192 or 128 x 128 that the column-sparse form uses.
//
// One workgroup of eight waves owns a 256 x 256 tile of the result and walks the contraction in steps of 64.  A step's
// operands are four half tiles of 16 KB in LDS (P0, P1: 128 rows each of the operand that lies along the result's
// contiguous axis, Q0, Q1: of the other), two steps deep; each wave multiplies 128 x 64 of the tile as four quadrants
// P_i x Q_j of 64 x 32 (16 MFMAs 16x16x32 each).
//
// Bound: the matrix cores, as long as nothing but their instructions is waited for.  With one workgroup per CU and two
// waves per SIMD the waves take turns: while waves 0-3 run 32 products, waves 4-7 read the operands of theirs from LDS
// and request tile transfers, and the other way round (waves 4-7 run one barrier behind).  A half tile is requested
// again as soon as both groups have read it, so that 64 to 96 KB per CU are in flight and a transfer has at least a step
// (about 1.3 us) to land:
//     slot    reads                        requests                       then multiplies
//     0       P0 and Q1 (step t)           Q0 (step t + 2), P1 (t + 1)    P0 x Q0, P0 x Q1
//     1       P1 (t) and Q0 (step t + 1)   P0 and Q1 (t + 2)              P1 x Q1, P1 x Q0
// A slot ends with its LDS reads complete and with the wave's share of what the next slot reads landed: always all but
// the transfers of the last two slots (8, or fewer where P is narrower).
//
// Measured at 18 000 tokens, D 5120, F 13 824 (5.1 TFLOP): both GEMMs 4.79 ms with 192 x 128 tiles, 3.74 ms with these
// (1.36 PFLOP/s; the second GEMM's 1420 tiles are 5.5 rounds of the CUs); 4608 x 3072 x 12 288: 721 and 547 us.  The matrix
// pipes are busy 75 % of the cycles (83 % in the second GEMM) at 1.7 to 1.8 GHz: the chip is at its power limit, so cycles
// saved by themselves come back as a lower clock (with four slots of 16 products per step instead of two of 32 it took
// 2 % more cycles and the same time).  Without the transfers (the same two steps over and over) the first GEMM takes
// 1.48 ms instead of 1.89, without the epilogue 1.66.  Persistent workgroups that request the next tile's first steps
// in the last steps of the one before, with the results turned round in 16 x 64 pieces beside the operands, measured 1 to
// 5 % slower than one workgroup per tile.
//
// The scores GEMM of the token-merged pre-activation (602 chunks x 12 288 neurons x 2 x 3072): 110 us and 13 us for the sum of
// two pieces with tiles of 128 x 128 over [hi | lo] against [w1 | w1], 75 us in one piece with these (1.22 PFLOP/s); 24
// chunks: 28 and 21 us.
#pragma once
#include "common.h"

namespace chipmunk {

enum DenseGemm { kFirst = 0, kSecond = 1, kScores = 2, kDelta = 3 };

struct DenseGemmParams {
    const uint16_t* x;       // [B, N, D]; scores: the chunk means in split precision, [N][hi 0..D-1 | lo 0..D-1]
    const uint16_t* w1;      // [F, D]
    const uint16_t* w2;      // [F, D]
    const uint16_t* bias;    // first GEMM: b1 [F]; second: b2 [D]; or null
    uint16_t* a_cache;       // [B, F, a_ld]: result of the first GEMM, operand of the second
    uint16_t* out;           // [B, N, D]
    int64_t a_ld;
    float* scores;           // scores: [pieces][N][F]
    int N, D, F, act;
    // column-sparse delta form of the first GEMM (kDelta): see Gemm1Params
    const int32_t* idx;
    const int32_t* counts;
    uint16_t* delta_t;
    uint16_t* act_t;
    int NB, k_stride, k_pad, units;
    int tiles_p, tiles_q;    // tiles along the result's contiguous axis and along the other
    int pieces;              // the contraction is cut into so many runs of whole steps (second grid dimension; scores only)
};

constexpr int kDenseTile = 256;
constexpr int kDenseHalf = 128 * 64 * 2;                 // bytes of a half tile
constexpr int kDenseStage = 4 * kDenseHalf;              // P0, P1, Q0, Q1 (P may be narrower: the rest lies idle)
constexpr int kDenseRow = (kDenseTile + 8) * 2;          // row stride (bytes) of the result tile on its way out
constexpr int kDenseLds = kDenseTile * kDenseRow > 2 * kDenseStage ? kDenseTile * kDenseRow : 2 * kDenseStage;

// Asynchronous 16-byte load to LDS like load_buffer_to_lds_16B, with a wave-uniform part of the offset.
__device__ __forceinline__ void load_buffer_to_lds_16B(i32x4 buffer, uint32_t byte_offset, uint32_t uniform_offset,
                                                       uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_wave_base), "v"(byte_offset), "s"(buffer), "s"(uniform_offset)
                 : "memory");
}

// C += A B (16x16x32) with C in accumulation registers.  With the builtin the compiler keeps the 128 accumulators among
// the other registers, moves them from product to product and spills (364 bytes); held apart, they leave 128 registers to
// the operands and addresses, of which the loops need about 110 (the second GEMM's epilogue keeps 20 bytes in scratch
// memory, the other forms nothing).  The compiler does not know the products' latency: whatever else reads C waits first
// (finish_products: 32 cycles, the products' results take at most 19), and no accumulator may be moved inside a loop,
// which a test checks in the compiled kernels.
__device__ __forceinline__ void mfma_in_place(f32x4& c, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void finish_products() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// kFirst:  a_cache[f][n] = act(<x[n], w1[f]> + b1[f]): P = tokens, Q = neurons, both operands with the contraction index
//          fastest.
// kSecond: out[n][d] = sum_f a_cache[f][n] w2[f][d] + b2[d]: P = output columns, Q = tokens, both with the contraction
//          index slowest (transposing LDS reads).
// kScores: scores[n][f] = <hi[n] + lo[n], w1[f]>, n a chunk: P = BM neurons, Q0 = the high parts of 128 chunk means, Q1 = their
//          low parts, so a step fetches w1 once for two products.  High and low parts have accumulators of their own:
//          added to the high parts' sum, every low product costs it a rounding (602 x 3072 x 12 288, the GEMM alone: 4.9e-7
//          off, apart 3.4e-7; same time).  With BM = 128 the high parts are added in two sums, one per slice of a step,
//          half as long.
// kDelta:  kFirst for the BM tokens of a chunk and 256 of its selected neurons, with the epilogue of the column-sparse form.
template <int MODE, int BM = kDenseTile>
__global__ __launch_bounds__(512, 2) void mlp_dense_gemm_kernel(DenseGemmParams p) {
    constexpr bool SECOND = MODE == kSecond, SCORES = MODE == kScores, DELTA = MODE == kDelta;
    constexpr bool TWO_SUMS = SCORES && BM == 128;           // the high parts' products in two sums, one per slice of a step
    constexpr int PB = BM / 64;                              // 16-row blocks of P per wave and half
    constexpr int HP = BM * 64;                              // bytes of a half tile of P
    constexpr int PT = HP / 1024;                            // its transfers: 16, 12 or 8 for the eight waves
    __shared__ int32_t s_neuron[DELTA ? kDenseTile : 1];
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = w >> 2, wq = w & 3;
    const int g = lane >> 4, l16 = lane & 15;

    int p0, q0, b, piece = 0, unit = 0, count = 0;
    if constexpr (DELTA) {
        // all column tiles of a chunk on one XCD
        int col_tile;
        if (!xcd_tile_of_block(p.tiles_q, p.units, &unit, &col_tile)) return;
        b = unit / p.NB;
        p0 = (unit % p.NB) * BM;
        q0 = col_tile * kDenseTile;
        count = min(p.counts[unit], p.k_stride);
        if (q0 >= ((count + kBK - 1) / kBK) * kBK) return;   // nothing to compute or to zero
        // neuron of each column (columns at or beyond count compute a duplicate that is never stored)
        if (tid < kDenseTile) {
            const int at = min(q0 + tid, max(count - 1, 0));
            s_neuron[tid] = min(max(p.idx[(int64_t)unit * p.k_stride + at], 0), p.F - 1);
        }
        __syncthreads();
    } else {
        // Each XCD takes one run of the tiles, ordered so that the 32 tiles its CUs work on at a time are a block of 8 x 4:
        // 12 strips of operands in that XCD's L2 instead of 33.
        const int tiles = p.tiles_p * p.tiles_q;
        const int per_xcd = (tiles + 7) >> 3;
        const int slot = (int)blockIdx.x >> 3;
        const int tile = ((int)blockIdx.x & 7) * per_xcd + slot;
        if (slot >= per_xcd || tile >= tiles) return;
        const int band = tile / (8 * p.tiles_q), in_band = tile - band * 8 * p.tiles_q;
        const int band_p = min(8, p.tiles_p - 8 * band);
        const int tq = in_band / band_p, tp = 8 * band + (in_band - tq * band_p);
        p0 = tp * BM;
        q0 = tq * (SCORES ? 128 : kDenseTile);
        b = SCORES ? 0 : blockIdx.y;
        piece = SCORES ? blockIdx.y : 0;
    }

    // operand sources: per-lane byte offsets of the wave's two transfers per half tile, clamped into the tensors
    // (rows beyond the end repeat the last one and are not stored)
    const uint16_t* xb = p.x + (int64_t)b * p.N * p.D;
    uint16_t* ab = p.a_cache + (int64_t)b * p.F * p.a_ld;
    const i32x4 wbuf = raw_buffer_words(SECOND ? p.w2 : p.w1, (uint32_t)p.F * p.D * 2u);
    const i32x4 xbuf = raw_buffer_words(xb, (uint32_t)p.N * p.D * (SCORES ? 4u : 2u));
    const i32x4 pbuf = MODE == kFirst || DELTA ? xbuf : wbuf;
    const i32x4 qbuf = MODE == kFirst || DELTA ? wbuf : SCORES ? xbuf : raw_buffer_words(ab, (uint32_t)p.F * (uint32_t)p.a_ld * 2u);
    const uint32_t pstep = SECOND ? 64u * p.D * 2u : 128u, qstep = SECOND ? 64u * (uint32_t)p.a_ld * 2u : 128u;
    uint32_t poff[2][2], qoff[2][2];   // [half][transfer]
#pragma unroll
    for (int hf = 0; hf < 2; hf++)
#pragma unroll
        for (int n = 0; n < 2; n++) {
            if (!SECOND) {             // 8 rows of 128 bytes; 16-byte chunks XOR-swizzled by the row
                const int prow = (n * 8 + w) * 8 + (lane >> 3), row = (w * 2 + n) * 8 + (lane >> 3);
                const uint32_t chunk = (uint32_t)((lane & 7) ^ ((row >> 1) & 7)) * 16u;
                const int last_p = SCORES ? p.F - 1 : p.N - 1;
                poff[hf][n] = (uint32_t)min(p0 + hf * (BM / 2) + prow, last_p) * (uint32_t)(p.D * 2) +
                              (uint32_t)((lane & 7) ^ ((prow >> 1) & 7)) * 16u;
                qoff[hf][n] = DELTA ? (uint32_t)s_neuron[hf * 128 + row] * (uint32_t)(p.D * 2) + chunk : SCORES ? (uint32_t)min(q0 + row, p.N - 1) * (uint32_t)(p.D * 4) + (uint32_t)(hf * p.D * 2) + chunk
                                     : (uint32_t)min(q0 + hf * 128 + row, p.F - 1) * (uint32_t)(p.D * 2) + chunk;
            } else {                   // 4 contraction rows of 256 bytes
                const int row = (w * 2 + n) * 4 + (lane >> 4);
                const int col = ((lane & 15) ^ swizzle_rows16(row)) * 8;
                poff[hf][n] = (uint32_t)row * (uint32_t)(p.D * 2) + (uint32_t)(min(p0 + hf * 128, p.D - 128) + col) * 2u;
                qoff[hf][n] = (uint32_t)row * (uint32_t)(p.a_ld * 2) + (uint32_t)min(q0 + hf * 128 + col, (p.N - 1) & ~7) * 2u;
            }
        }
    const int all_steps = (SECOND ? p.F : p.D) / 64;
    const int step0 = SCORES ? (int)((int64_t)all_steps * piece / p.pieces) : 0;
    const int steps = (SCORES ? (int)((int64_t)all_steps * (piece + 1) / p.pieces) : all_steps) - step0;   // at least one
    const uint32_t lds0 = lds_address(smem);
    // half tile `hf` of P or Q of step t (past the end the last step again, into a place nobody reads)
    auto request = [&](bool is_q, int hf, int t) {
        const uint32_t stage = lds0 + (uint32_t)((t & 1) * kDenseStage);
        const uint32_t from = (uint32_t)(step0 + min(t, steps - 1)) * (is_q ? qstep : pstep);
#pragma unroll
        for (int n = 0; n < 2; n++) {
            if (is_q) {
                load_buffer_to_lds_16B(qbuf, qoff[hf][n], from, stage + 2 * HP + hf * kDenseHalf + (w * 2 + n) * 1024);
            } else {   // the wave's second transfer of P exists for 16, 12 (waves 0-3) or 8 (none) transfers per half
                const int at = SECOND ? w * 2 + n : n * 8 + w;
                if (n == 0 || PT == 16 || (PT == 12 && w < 4)) load_buffer_to_lds_16B(pbuf, poff[hf][n], from, stage + hf * HP + at * 1024);
            }
        }
    };

    // LDS read addresses in the first stage; the second lies at the XOR of kDenseStage
    static_assert((kDenseStage & (kDenseStage - 1)) == 0, "stages are told apart by one address bit");
    constexpr int NPA = SECOND ? 4 : 2, NQA = 2;
    uint32_t pat[NPA], qat[NQA];
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
    if (!SECOND) {
        const uint32_t in_row = (uint32_t)((g ^ ((l16 >> 1) & 7)) * 16);
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            pat[ks] = (uint32_t)((wp * (BM / 4) + l16) * 128) + (in_row ^ (64u * ks));
            qat[ks] = (uint32_t)(2 * HP + (wq * 32 + l16) * 128) + (in_row ^ (64u * ks));
        }
    } else {
        const int row = 4 * g + (l16 >> 2);
        const int s = swizzle_rows16(row), c = (l16 & 3) >> 1;
#pragma unroll
        for (int i = 0; i < 4; i++) pat[i] = (uint32_t)(row * 256 + ((wp * 8 + i * 2 + c) ^ s) * 16 + 8 * (l16 & 1));
#pragma unroll
        for (int i = 0; i < 2; i++)
            qat[i] = (uint32_t)(2 * HP + row * 256 + ((wq * 4 + i * 2 + c) ^ s) * 16 + 8 * (l16 & 1));
    }
    // the LDS base is aligned to the two stages' size, or added below the bit that tells them apart
#pragma unroll
    for (int i = 0; i < NPA; i++) pat[i] += smem_at;
#pragma unroll
    for (int i = 0; i < NQA; i++) qat[i] += smem_at;

    // One operand block of 16 rows x 32 contraction entries: block `i` of half `hf`, slice ks.  The order of the
    // contraction entries inside a slice is the same for P and Q, which is all that matters.
    auto read_block = [&](const auto& at, int i, int hf_bytes, int ks) -> bf16x8 {
        if constexpr (!SECOND) {
            return lds_read_b128(at[ks] + (uint32_t)(hf_bytes + i * 2048));
        } else {
            const uint32_t a = at[i] + (uint32_t)(hf_bytes + ks * 32 * 256);
            typedef __attribute__((ext_vector_type(8))) short short8v;
            return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lds_read_tr16_at(a), lds_read_tr16_at(a + 16 * 256),
                                                                              0, 1, 2, 3, 4, 5, 6, 7));
        }
    };

    f32x4 acc[2][TWO_SUMS ? 3 : 2][PB][2];   // [half of P][half of Q; third: Q0's second slice]
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < (TWO_SUMS ? 3 : 2); j++)
#pragma unroll
            for (int a = 0; a < PB; a++)
#pragma unroll
                for (int c = 0; c < 2; c++) acc[i][j][a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 P[PB][2], Q0[2][2], Q1[2][2], Q0next[2][2];   // [block][slice]
    auto read_p = [&](int hf) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < PB; a++) P[a][ks] = read_block(pat, a, hf * HP, ks);
    };
    auto read_q = [&](bf16x8 (&Q)[2][2], int hf) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int c = 0; c < 2; c++) Q[c][ks] = read_block(qat, c, hf * kDenseHalf, ks);
    };
    auto other_stage = [&](auto& at) {
        for (uint32_t& a : at) a ^= kDenseStage;
    };
    auto turn = [&]() {   // the end of a slot
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto ready = [&]() {  // the slot's LDS reads are complete, the next slot's operands have landed
        __builtin_amdgcn_sched_barrier(0);
        // the transfers of the last two slots: four of Q and two of P's halves
        if (PT == 16 || (PT == 12 && wp == 0)) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
        turn();
    };
    auto multiply = [&](f32x4 (&C)[PB][2], f32x4 (&C1)[PB][2], const bf16x8 (&Q)[2][2]) {   // C1: of the second slice
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < PB; a++)
#pragma unroll
                for (int c = 0; c < 2; c++) mfma_in_place(ks == 0 ? C[a][c] : C1[a][c], P[a][ks], Q[c][ks]);
    };

    request(true, 0, 0);
    request(false, 0, 0);
    request(true, 1, 0);
    request(true, 0, 1);
    request(false, 1, 0);
    request(false, 0, 1);
    request(true, 1, 1);
    ready();                                     // Q0, P0 and Q1 of the first step
    read_q(Q0, 0);
    lds_accesses_then_barrier();                 // read by every wave before the first step requests Q0 again
    if (wp == 1) turn();                         // waves 4-7 run one slot behind from here
    auto contract = [&](auto both_c) {
    constexpr bool both = decltype(both_c)::value;
#pragma unroll 1
    for (int t = 0; t < steps; t++) {
        read_p(0);
        read_q(Q1, 1);
        request(true, 0, t + 2);
        request(false, 1, t + 1);
        ready();
        __builtin_amdgcn_s_setprio(1);
        multiply(acc[0][0], acc[0][TWO_SUMS ? 2 : 0], Q0);
        if constexpr (both) multiply(acc[0][1], acc[0][1], Q1);
        __builtin_amdgcn_s_setprio(0);
        turn();
        read_p(1);
        other_stage(pat);
        other_stage(qat);
        read_q(Q0next, 0);
        request(false, 0, t + 2);
        request(true, 1, t + 2);
        ready();
        __builtin_amdgcn_s_setprio(1);
        if constexpr (both) multiply(acc[1][1], acc[1][1], Q1);
        multiply(acc[1][0], acc[1][TWO_SUMS ? 2 : 0], Q0);
        __builtin_amdgcn_s_setprio(0);
        if (t + 1 == steps) finish_products();   // in the loop: behind it the compiler may move accumulators at once
        turn();
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int c = 0; c < 2; c++) Q0[c][ks] = Q0next[c][ks];
    }
    };
    // A chunk's last tile may need its first 128 columns only.  Two loops, not a branch in one: around a branch the compiler
    // moves accumulators between registers in every step.
    if (!DELTA || q0 + 128 < count) contract(std::true_type{});
    else if constexpr (DELTA) contract(std::false_type{});
    if constexpr (SCORES) {
        // four consecutive neurons of one chunk per lane and block: 64-byte runs, joined in L2
        if (wp == 0) turn();
        wait_all_memory();                       // the transfers past the end must have landed before the wave may end
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const int n = q0 + wq * 32 + c * 16 + l16;
            float* row = p.scores + ((int64_t)piece * p.N + n) * p.F + p0 + wp * (BM / 4) + 4 * g;
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int a = 0; a < PB; a++) {
                    f32x4 sum = acc[i][0][a][c];
                    if (TWO_SUMS) sum += acc[i][TWO_SUMS ? 2 : 0][a][c];
                    sum += acc[i][1][a][c];
                    if (n < p.N && p0 + i * (BM / 2) + wp * (BM / 4) + a * 16 < p.F) *reinterpret_cast<f32x4*>(row + i * (BM / 2) + a * 16) = sum;
                }
        }
        return;
    } else if constexpr (DELTA) {
        // ---- epilogue of the column-sparse form: activations through LDS as [neuron][token]; then per cell (a neuron's eight
        // tokens) the cached activations are read (requested up front), the new ones and delta^T written ----
        constexpr int CPR = BM / 8, ITEMS = kDenseTile * CPR / 512, ROW = BM * 2 + 16;
        static_assert(kDenseTile * CPR % 512 == 0, "the tile's cells must divide over the threads");
        const bool has_bias = p.bias != nullptr;
        const uint16_t* bias_src = has_bias ? p.bias : p.w1;   // a valid address when there is none
        uint16_t b1[2][2];
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int c = 0; c < 2; c++) b1[j][c] = bias_src[s_neuron[j * 128 + wq * 32 + c * 16 + l16]];
        // address of a cached cell; tokens clamped to the row's start where the chunk ends early: read, not used
        auto cell = [&](int nl, int ch) -> uint16_t* {
            const int tok0 = p0 + ch * 8;
            return ab + (int64_t)s_neuron[nl] * p.a_ld + (tok0 < p.N ? tok0 : 0);
        };
        u32x4 old8[ITEMS];
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid + n * 512, nl = item / CPR;
            old8[n] = *reinterpret_cast<const u32x4*>(cell(nl, item - nl * CPR));
        }
        if (wp == 0) turn();
        wait_all_memory();                           // the transfers past the end have landed before LDS is reused
        turn();
        auto to_lds = [&](auto form) {
            constexpr int ACT = decltype(form)::value;
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    const float bq = has_bias ? bf16_bits_to_float(b1[j][c]) : 0.f;
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int a = 0; a < PB; a++) {
                            const f32x4 v = acc[i][j][a][c];
                            *reinterpret_cast<u32x2*>(smem + (j * 128 + wq * 32 + c * 16 + l16) * ROW +
                                                      (i * (BM / 2) + wp * (BM / 4) + a * 16 + 4 * g) * 2) =
                                u32x2{pack_bf16x2(gelu<ACT>(v[0] + bq), gelu<ACT>(v[1] + bq)),
                                      pack_bf16x2(gelu<ACT>(v[2] + bq), gelu<ACT>(v[3] + bq))};
                        }
                }
        };
        if (p.act == CHIPMUNK_ACT_GELU_ERF) to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_ERF>{});
        else to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_TANH>{});
        lds_accesses_then_barrier();
        // The thread's cells are worked out again from here on: held across the activations, beside the accumulators and what
        // the cells held, the addresses of all loads and stores went to scratch memory (72 bytes at BM = 192; without them
        // the whole delta of 394 chunks x 968 of 13 824 x 5120 1891 -> 1873 us, of 47 x 1229 of 12 288 x 3072 188 -> 184).
        int tid_again = tid;
        asm volatile("" : "+v"(tid_again));
        u32x4 a8[ITEMS];
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid_again + n * 512, nl = item / CPR;
            a8[n] = *reinterpret_cast<const u32x4*>(smem + nl * ROW + (item - nl * CPR) * 16);
        }
        const int64_t at0 = (int64_t)unit * p.k_pad * BM;
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid_again + n * 512, nl = item / CPR, ch = item - nl * CPR, s = q0 + nl;
            // tokens past N and padding rows of the contraction must read as zero in the second GEMM
            const int nvalid = s < count ? min(8, p.N - (p0 + ch * 8)) : 0;
            u32x4 d8;
#pragma unroll
            for (int e2 = 0; e2 < 4; e2++) {
                float dlo = bf16_bits_to_float(a8[n][e2] & 0xffffu) - bf16_bits_to_float(old8[n][e2] & 0xffffu);
                float dhi = bf16_bits_to_float(a8[n][e2] >> 16) - bf16_bits_to_float(old8[n][e2] >> 16);
                if (2 * e2 >= nvalid) dlo = 0.f;
                if (2 * e2 + 1 >= nvalid) dhi = 0.f;
                d8[e2] = pack_bf16x2(dlo, dhi);
            }
            if (s < p.k_pad) *reinterpret_cast<u32x4*>(p.delta_t + at0 + (int64_t)s * BM + ch * 8) = d8;
        }
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid_again + n * 512, nl = item / CPR, ch = item - nl * CPR, s = q0 + nl;
            const int nvalid = s < count ? min(8, p.N - (p0 + ch * 8)) : 0;
            if (p.act_t) {   // deferred write-back: one coalesced store, whole cell
                if (nvalid > 0) *reinterpret_cast<u32x4*>(p.act_t + at0 + (int64_t)s * BM + ch * 8) = a8[n];
            } else if (nvalid == 8) {
                *reinterpret_cast<u32x4*>(cell(nl, ch)) = a8[n];
            } else {         // the cells past N in the last chunk stay as they are
                for (int e = 0; e < nvalid; e++) cell(nl, ch)[e] = (uint16_t)(a8[n][e >> 1] >> (16 * (e & 1)));
            }
        }
    } else {
    // ---- epilogue: bias (and activation), bf16, through LDS as [q][p], out in runs of 512 bytes ----
    // the bias is requested in front of the last waits
    const bool has_bias = p.bias != nullptr;
    const uint16_t* bias_src = has_bias ? p.bias : SECOND ? p.w2 : p.w1;   // a valid address when there is none
    u32x2 b4[2][4];                              // SECOND: the bias of the lane's four columns per block
    uint16_t b1[2][2];                           // else: of its neuron
    if constexpr (SECOND) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int a = 0; a < PB; a++)
                b4[i][a] = *reinterpret_cast<const u32x2*>(bias_src + min(p0 + i * 128 + wp * 64 + a * 16 + 4 * g, p.D - 4));
    } else {
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int c = 0; c < 2; c++) b1[j][c] = bias_src[min(q0 + j * 128 + wq * 32 + c * 16 + l16, p.F - 1)];
    }
    if (wp == 0) turn();
    wait_all_memory();                           // the transfers past the end have landed before LDS is reused
    turn();
    auto to_lds = [&](auto form) {
        constexpr int ACT = decltype(form)::value;
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int c = 0; c < 2; c++)
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int a = 0; a < PB; a++) {
                        const f32x4 v = acc[i][j][a][c];
                        u32x2 packed;
                        if constexpr (!SECOND) {
                            const float bq = has_bias ? bf16_bits_to_float(b1[j][c]) : 0.f;
                            packed = u32x2{pack_bf16x2(gelu<ACT>(v[0] + bq), gelu<ACT>(v[1] + bq)),
                                           pack_bf16x2(gelu<ACT>(v[2] + bq), gelu<ACT>(v[3] + bq))};
                        } else {
                            const u32x2 bp = has_bias ? b4[i][a] : u32x2{0u, 0u};
                            packed = u32x2{pack_bf16x2(v[0] + bf16_bits_to_float(bp[0] & 0xffffu), v[1] + bf16_bits_to_float(bp[0] >> 16)),
                                           pack_bf16x2(v[2] + bf16_bits_to_float(bp[1] & 0xffffu), v[3] + bf16_bits_to_float(bp[1] >> 16))};
                        }
                        *reinterpret_cast<u32x2*>(smem + (j * 128 + wq * 32 + c * 16 + l16) * kDenseRow +
                                                  (i * 128 + wp * 64 + a * 16 + 4 * g) * 2) = packed;
                    }
    };
    if (!SECOND && p.act == CHIPMUNK_ACT_GELU_ERF) to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_ERF>{});
    else to_lds(std::integral_constant<int, CHIPMUNK_ACT_GELU_TANH>{});
    lds_accesses_then_barrier();
    const int limit_p = SECOND ? p.D : p.N, limit_q = SECOND ? p.N : p.F;
    const int64_t ld = SECOND ? p.D : p.a_ld;
    const int pc = p0 + (tid & 31) * 8, qr = q0 + (tid >> 5);
    uint16_t* dst = (SECOND ? p.out + (int64_t)b * p.N * p.D : ab) + (int64_t)qr * ld + pc;
    u32x4 row[16];
#pragma unroll
    for (int n = 0; n < 16; n++) row[n] = *reinterpret_cast<const u32x4*>(smem + (n * 16 + (tid >> 5)) * kDenseRow + (tid & 31) * 16);
    if (pc + 8 <= limit_p) {
#pragma unroll
        for (int n = 0; n < 16; n++)
            if (qr + n * 16 < limit_q) *reinterpret_cast<u32x4*>(dst + n * 16 * ld) = row[n];
    } else {   // the cells past N stay as they are
        for (int n = 0; n < 16; n++)
            for (int e = 0; e < limit_p - pc; e++)
                if (qr + n * 16 < limit_q) dst[n * 16 * ld + e] = *reinterpret_cast<const uint16_t*>(smem + (n * 16 + (tid >> 5)) * kDenseRow + (tid & 31) * 16 + e * 2);
    }
    }
}

}  // namespace chipmunk
