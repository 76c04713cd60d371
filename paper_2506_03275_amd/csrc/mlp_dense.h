// The two GEMMs of the dense MLP (Alg. 5) at sizes that fill the chip, and the scores GEMM (Alg. 7).  Internal to mlp.hip,
// which chooses between these and the tiles of 192 or 128 x 128 that the column-sparse form uses.
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
// the youngest 8 transfers.
//
// Measured at 18 000 tokens, D 5120, F 13 824 (5.1 TFLOP): both GEMMs 4.79 ms with 192 x 128 tiles, 3.93 ms with these
// (1.30 PFLOP/s; first 1.34, second 1.20, whose 1420 tiles are 5.5 rounds of the CUs); 4608 x 3072 x 12 288: 734 and
// 569 us.  The matrix pipes are busy 76 % of the cycles at 1.7 to 1.8 GHz: the chip is at its power limit, so cycles
// saved by themselves come back as a lower clock (with four slots of 16 products per step instead of two of 32 it took
// 2 % more cycles and the same time).  Without the transfers (the same two steps over and over) the first GEMM takes
// 1.48 ms instead of 1.89, without the epilogue 1.66.  Persistent workgroups that request the next tile's first steps
// in the last steps of the one before, with the results turned round in 16 x 64 pieces beside the operands, measured 1 to
// 5 % slower than one workgroup per tile.
//
// The scores GEMM of the token-merged pre-activation (602 chunks x 12 288 neurons x 2 x 3072): 110 us and 13 us for the sum of
// two pieces with tiles of 128 x 128 over [hi | lo] against [w1 | w1], 75 us in one piece with these (1.22 PFLOP/s); 24
// chunks: 28 and 19 us.
#pragma once
#include "common.h"

namespace chipmunk {

enum DenseGemm { kFirst = 0, kSecond = 1, kScores = 2 };

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
    int tiles_p, tiles_q;    // tiles along the result's contiguous axis and along the other
    int pieces;              // the contraction is cut into so many runs of whole steps (second grid dimension; scores only)
};

constexpr int kDenseTile = 256;
constexpr int kDenseHalf = 128 * 64 * 2;                 // bytes of a half tile
constexpr int kDenseStage = 4 * kDenseHalf;              // P0, P1, Q0, Q1
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
// the operands and addresses, of which the kernel needs about 100.  The compiler does not know the products' latency:
// whatever else reads C waits first (finish_products).
__device__ __forceinline__ void mfma_in_place(f32x4& c, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void finish_products() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// kFirst:  a_cache[f][n] = act(<x[n], w1[f]> + b1[f]): P = tokens, Q = neurons, both operands with the contraction index
//          fastest.
// kSecond: out[n][d] = sum_f a_cache[f][n] w2[f][d] + b2[d]: P = output columns, Q = tokens, both with the contraction
//          index slowest (transposing LDS reads).
// kScores: scores[n][f] = <hi[n] + lo[n], w1[f]>, n a chunk: P = neurons, Q0 = the high parts of 128 chunk means, Q1 = their
//          low parts; both go into the same accumulators, so a step fetches w1 once for two products.  256 x 128 tiles.
template <int MODE>
__global__ __launch_bounds__(512, 2) void mlp_dense_gemm_kernel(DenseGemmParams p) {
    constexpr bool SECOND = MODE == kSecond, SCORES = MODE == kScores;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = w >> 2, wq = w & 3;
    const int g = lane >> 4, l16 = lane & 15;

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
    const int p0 = tp * kDenseTile, q0 = tq * (SCORES ? 128 : kDenseTile);
    const int b = SCORES ? 0 : blockIdx.y, piece = SCORES ? blockIdx.y : 0;

    // operand sources: per-lane byte offsets of the wave's two transfers per half tile, clamped into the tensors
    // (rows beyond the end repeat the last one and are not stored)
    const uint16_t* xb = p.x + (int64_t)b * p.N * p.D;
    uint16_t* ab = p.a_cache + (int64_t)b * p.F * p.a_ld;
    const i32x4 wbuf = raw_buffer_words(SECOND ? p.w2 : p.w1, (uint32_t)p.F * p.D * 2u);
    const i32x4 xbuf = raw_buffer_words(xb, (uint32_t)p.N * p.D * (SCORES ? 4u : 2u));
    const i32x4 pbuf = MODE == kFirst ? xbuf : wbuf;
    const i32x4 qbuf = MODE == kFirst ? wbuf : SCORES ? xbuf : raw_buffer_words(ab, (uint32_t)p.F * (uint32_t)p.a_ld * 2u);
    const uint32_t pstep = SECOND ? 64u * p.D * 2u : 128u, qstep = SECOND ? 64u * (uint32_t)p.a_ld * 2u : 128u;
    uint32_t poff[2][2], qoff[2][2];   // [half][transfer]
#pragma unroll
    for (int hf = 0; hf < 2; hf++)
#pragma unroll
        for (int n = 0; n < 2; n++) {
            if (!SECOND) {             // 8 rows of 128 bytes; 16-byte chunks XOR-swizzled by the row
                const int row = (w * 2 + n) * 8 + (lane >> 3);
                const uint32_t chunk = (uint32_t)((lane & 7) ^ ((row >> 1) & 7)) * 16u;
                const int last_p = SCORES ? p.F - 1 : p.N - 1;
                poff[hf][n] = (uint32_t)min(p0 + hf * 128 + row, last_p) * (uint32_t)(p.D * 2) + chunk;
                qoff[hf][n] = SCORES ? (uint32_t)min(q0 + row, p.N - 1) * (uint32_t)(p.D * 4) + (uint32_t)(hf * p.D * 2) + chunk
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
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + (uint32_t)w * 2048u);
    // half tile `hf` of P or Q of step t (past the end the last step again, into a place nobody reads)
    auto request = [&](bool is_q, int hf, int t) {
        const uint32_t dst = lds0 + (uint32_t)((t & 1) * kDenseStage + (is_q ? 2 : 0) * kDenseHalf + hf * kDenseHalf);
        const uint32_t from = (uint32_t)(step0 + min(t, steps - 1)) * (is_q ? qstep : pstep);
#pragma unroll
        for (int n = 0; n < 2; n++)
            load_buffer_to_lds_16B(is_q ? qbuf : pbuf, is_q ? qoff[hf][n] : poff[hf][n], from, dst + n * 1024);
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
            pat[ks] = (uint32_t)((wp * 64 + l16) * 128) + (in_row ^ (64u * ks));
            qat[ks] = (uint32_t)(2 * kDenseHalf + (wq * 32 + l16) * 128) + (in_row ^ (64u * ks));
        }
    } else {
        const int row = 4 * g + (l16 >> 2);
        const int s = swizzle_rows16(row), c = (l16 & 3) >> 1;
#pragma unroll
        for (int i = 0; i < 4; i++) pat[i] = (uint32_t)(row * 256 + ((wp * 8 + i * 2 + c) ^ s) * 16 + 8 * (l16 & 1));
#pragma unroll
        for (int i = 0; i < 2; i++)
            qat[i] = (uint32_t)(2 * kDenseHalf + row * 256 + ((wq * 4 + i * 2 + c) ^ s) * 16 + 8 * (l16 & 1));
    }
    // the LDS base is aligned to the two stages' size, or added below the bit that tells them apart
#pragma unroll
    for (int i = 0; i < NPA; i++) pat[i] += smem_at;
#pragma unroll
    for (int i = 0; i < NQA; i++) qat[i] += smem_at;

    // One operand block of 16 rows x 32 contraction entries: block `i` of half `hf`, slice ks.  The order of the
    // contraction entries inside a slice is the same for P and Q, which is all that matters.
    auto read_block = [&](const auto& at, int i, int hf, int ks) -> bf16x8 {
        if constexpr (!SECOND) {
            return lds_read_b128(at[ks] + (uint32_t)(hf * kDenseHalf + i * 2048));
        } else {
            const uint32_t a = at[i] + (uint32_t)(hf * kDenseHalf + ks * 32 * 256);
            typedef __attribute__((ext_vector_type(8))) short short8v;
            return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lds_read_tr16_at(a), lds_read_tr16_at(a + 16 * 256),
                                                                              0, 1, 2, 3, 4, 5, 6, 7));
        }
    };

    constexpr int NJ = SCORES ? 1 : 2;
    f32x4 acc[2][NJ][4][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < NJ; j++)
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 2; c++) acc[i][j][a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 P[4][2], Q0[2][2], Q1[2][2], Q0next[2][2];   // [block][slice]
    auto read_p = [&](int hf) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < 4; a++) P[a][ks] = read_block(pat, a, hf, ks);
    };
    auto read_q = [&](bf16x8 (&Q)[2][2], int hf) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int c = 0; c < 2; c++) Q[c][ks] = read_block(qat, c, hf, ks);
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
        asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        turn();
    };
    auto multiply = [&](f32x4 (&C)[4][2], const bf16x8 (&Q)[2][2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 2; c++) mfma_in_place(C[a][c], P[a][ks], Q[c][ks]);
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
#pragma unroll 1
    for (int t = 0; t < steps; t++) {
        read_p(0);
        read_q(Q1, 1);
        request(true, 0, t + 2);
        request(false, 1, t + 1);
        ready();
        __builtin_amdgcn_s_setprio(1);
        multiply(acc[0][0], Q0);
        multiply(acc[0][NJ - 1], Q1);
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
        multiply(acc[1][NJ - 1], Q1);
        multiply(acc[1][0], Q0);
        __builtin_amdgcn_s_setprio(0);
        turn();
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int c = 0; c < 2; c++) Q0[c][ks] = Q0next[c][ks];
    }
    if constexpr (SCORES) {
        // four consecutive neurons of one chunk per lane and block: 64-byte runs, joined in L2
        finish_products();
        if (wp == 0) turn();
        wait_all_memory();                       // the transfers past the end must have landed before the wave may end
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const int n = q0 + wq * 32 + c * 16 + l16;
            float* row = p.scores + ((int64_t)piece * p.N + n) * p.F + p0 + wp * 64 + 4 * g;
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int a = 0; a < 4; a++)
                    if (n < p.N && p0 + i * 128 + wp * 64 + a * 16 < p.F) *reinterpret_cast<f32x4*>(row + i * 128 + a * 16) = acc[i][0][a][c];
        }
        return;
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
            for (int a = 0; a < 4; a++)
                b4[i][a] = *reinterpret_cast<const u32x2*>(bias_src + min(p0 + i * 128 + wp * 64 + a * 16 + 4 * g, p.D - 4));
    } else {
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int c = 0; c < 2; c++) b1[j][c] = bias_src[min(q0 + j * 128 + wq * 32 + c * 16 + l16, p.F - 1)];
    }
    finish_products();
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
                    for (int a = 0; a < 4; a++) {
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
