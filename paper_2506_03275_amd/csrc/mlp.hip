// Column-sparse delta MLP (Sec. 3.3.2 "Sparse Delta Steps", App. B.3.1, Alg. 6),
// the dense MLP of a dense step (Alg. 5) and the token-merged pre-activation
// (Alg. 7) for gfx950.
//
// GEMM1  pre[tok, s] = <x[tok], w1[idx[s]]>: one workgroup owns (token chunk,
//        128 selected neurons).  The x tile and the gathered w1 rows stream
//        through LDS (asynchronous 16-byte loads, three tile buffers: two
//        contraction steps in flight while one is consumed, K tile 64)
//        into bf16 MFMA 32x32x16.  Epilogue: bias, activation, rounding to
//        bf16, a transpose through LDS to the neuron-major layout of a_cache,
//        then per 8 consecutive tokens of one neuron: read the cached
//        activation, write the new one, write delta^T to the workspace.  Each
//        (chunk, neuron) cell has one writer: no atomics.
// GEMM2  o_cache[tok, :] += sum_s delta[tok, s] * w2[idx[s], :]: one workgroup
//        owns (token chunk, 128 output columns) and walks the selected rows in
//        steps of 32.  Both operands are stored with the contraction index as
//        the slow axis (delta^T rows, w2 rows), so both come out of LDS through
//        the transposing 64-bit read.  Epilogue: fp32 tile through LDS, add to
//        the cached output in fp32, round once, store in 256-byte runs.
// The dense MLP of a small problem is the same two kernels with "every neuron
// selected": GEMM1 writes a_cache only and GEMM2 reads its A operand from a_cache
// and adds b2.  Large ones and the scores GEMM have tiles of their own
// (mlp_dense.h), and so have the GEMMs with too few tiles to fill the chip
// (mlp_small.h).
#include "common.h"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace chipmunk {

constexpr int64_t kAllL2 = 32 << 20, kLastLevelCache = 256 << 20;   // bytes
constexpr int kBN = 128;  // neurons (GEMM1) or output columns (GEMM2) per workgroup
constexpr int kBK = 64;   // contraction tile

enum Gemm1Mode { kSparseDelta = 0, kDenseAct = 1 };

// Workgroups are dispatched to the eight XCDs round-robin by linear id, and each XCD has its own L2.  Tile of the workgroup in
// slot `slot` of XCD `xcd` when each XCD takes one run of `tiles` tiles, the runs equally long to one tile; false for the ids that
// pad the grid.
__device__ __forceinline__ bool xcd_run_tile(int xcd, int slot, int tiles, int* tile) {
    const int each = tiles >> 3, more = tiles & 7;
    *tile = xcd * each + min(xcd, more) + slot;
    return slot < each + (xcd < more ? 1 : 0);
}
static int xcd_grid_size(int col_tiles, int units) { return (col_tiles * units + 7) / 8 * 8; }

// The column-sparse forms: the tiles of one token chunk share that chunk's x rows (GEMM1) or delta^T rows (GEMM2) and nothing
// else, so they run on one XCD, chunk u on XCD u % 8, its column tiles back to back.  The last units % 8 chunks are cut into
// eight runs of tiles instead: as whole chunks they left XCDs idle.  Whole deltas in us, 12 chunks x 1515 of 4096 x 3072: 134 -> 97,
// 18 x 2216 of 9088 x 3200: 160 -> 133, 9 x 4914 of 10 112 x 3840: 242 -> 199; 394 x 968 of 13 824 x 5120: 1884 and 1884 (every
// chunk in such a run: 1887 against 1870, 434 chunks of 2432 x 4992 624 against 614).
__device__ __forceinline__ bool xcd_tile_of_slot(int slot, int col_tiles, int units, int* unit, int* col_tile) {
    const int xcd = (int)blockIdx.x & 7;
    const int whole = units >> 3, local = slot / col_tiles;   // chunks per XCD taken whole
    if (local < whole) {
        *unit = local * 8 + xcd;
        *col_tile = slot - local * col_tiles;
        return true;
    }
    int tile;
    if (!xcd_run_tile(xcd, slot - whole * col_tiles, (units & 7) * col_tiles, &tile)) return false;
    const int of_rest = tile / col_tiles;
    *unit = whole * 8 + of_rest;
    *col_tile = tile - of_rest * col_tiles;
    return true;
}

__device__ __forceinline__ bool xcd_tile_of_block(int col_tiles, int units, int* unit, int* col_tile) {
    return xcd_tile_of_slot((int)blockIdx.x >> 3, col_tiles, units, unit, col_tile);
}

// The dense forms (every neuron selected) share the weight tiles between chunks as well, and a weight tile is as large as a
// chunk's rows: the tiles stand in bands of eight chunks, column tile by column tile, so that what runs side by side on an
// XCD (64 workgroups at most) reads eight row tiles and eight weight tiles, each eight times.  (Eight chunks and eight column
// tiles at a time with both padded to eight, whole MLP in us: 19 chunks of 192 x 1536 x 11 264 330 -> 272, 17 x 3584 x 1728 113 -> 88.)
__device__ __forceinline__ bool xcd_tile_of_block_grouped(int slot, int col_tiles, int units, int* unit, int* col_tile) {
    int tile;
    if (!xcd_run_tile((int)blockIdx.x & 7, slot, col_tiles * units, &tile)) return false;
    const int band = tile / (8 * col_tiles), in_band = tile - band * 8 * col_tiles;
    const int height = min(8, units - 8 * band);
    *col_tile = in_band / height;
    *unit = 8 * band + in_band - *col_tile * height;
    return true;
}

// ACT is a template argument so that a tile's activations are straight-line code: with the form chosen by a
// run-time branch inside, every element became a basic block of its own and its dozen dependent instructions
// ran one after the other.
template <int ACT>
__device__ __forceinline__ float gelu(float x) {
    if (ACT == CHIPMUNK_ACT_GELU_ERF) return 0.5f * x * (1.f + erff(x * 0.70710678118654752f));
    // tanh form: 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3);  -2 u log2(e) = x (A + B x^2)
    const float t = x * __builtin_fmaf(x * x, -0.10294324f, -2.3022082f);
    return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(t));  // v_rcp_f32: 1 ulp, the result is rounded to bf16
}

}  // namespace chipmunk
#include "mlp_dense.h"
namespace chipmunk {

struct Gemm1Params {
    const uint16_t* x;       // [B, N, D]
    const uint16_t* w1;      // [F, D]
    const uint16_t* b1;      // [F] or null
    const int32_t* idx;      // [units, k_stride] or null (dense)
    const int32_t* counts;   // [units] or null
    uint16_t* a_cache;       // [B, F, a_ld]
    uint16_t* delta_t;       // workspace [units, k_pad, BM]
    uint16_t* act_t;         // null, or workspace [units, k_pad, BM]: the new activations go here (same layout as
                             // delta_t) instead of into a_cache; the second GEMM's launch writes them back
    int64_t a_ld;
    int N, NB, D, F;
    int k_stride, k_pad, act;
    int col_tiles, units;    // launch geometry (see xcd_tile_of_block)
    int parts;               // tiles of 64 x 64 only: row tiles per unit
};

// Three tile buffers: two contraction steps are in flight while one is consumed (120 KB, one workgroup per CU): measured
// against two buffers and two workgroups per CU, which keep the same number of bytes in flight, the MLP delta takes 11 %
// less time and the dense MLP 9 % less.
template <int BM, int MODE>
__global__ __launch_bounds__(320, 1) void mlp_gemm1_kernel(Gemm1Params p) {
    // A fifth wave issues every tile transfer of the workgroup; the four product waves issue none.  A wave issues in
    // order, so a transfer that waits for room in the memory pipeline holds up the products behind it.
    // The loader wave takes part in every barrier of the kernel and in nothing else.
    constexpr int NS = 3;
    constexpr int VW = 4;                          // waves whose share of the transfers the loader wave carries
    constexpr int MT = BM / 64;                    // 32-row MFMA tiles per wave (wave tile = BM/2 x 64)
    constexpr int XT = BM * 128;                   // bytes of the x tile  [BM][64] bf16
    constexpr int WT = kBN * 128;                  // bytes of the w1 tile [128][64] bf16
    constexpr int STAGE = XT + WT;
    constexpr int NIX = BM / 32;                   // 16-byte loads per lane for the x tile
    constexpr int NIW = kBN / 32;
    constexpr int TS = BM * 2 + 16;                // row stride of the transposed epilogue tile
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    __shared__ int32_t s_neuron[kBN];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool loader = w == 4;                    // wave-uniform
    const int wm = w >> 1, wn = w & 1;
    const int l32 = lane & 31, h = lane >> 5;

    int unit, col_tile;                            // unit = (batch, token chunk)
    if (MODE == kDenseAct ? !xcd_tile_of_block_grouped((int)blockIdx.x >> 3, p.col_tiles, p.units, &unit, &col_tile)
                          : !xcd_tile_of_block(p.col_tiles, p.units, &unit, &col_tile))
        return;
    const int b = unit / p.NB, chunk = unit % p.NB;
    const int row0 = chunk * BM;
    const int col0 = col_tile * kBN;
    const int count = p.counts ? min(p.counts[unit], p.k_stride) : p.F;   // clamped like the indices below: a bad
                                                                          // entry must not leave the tensors
    if (col0 >= count && MODE != kSparseDelta) return;
    if (MODE == kSparseDelta && col0 >= ((count + kBK - 1) / kBK) * kBK) return;  // nothing to compute or to zero

    // neuron of each of the 128 columns of this tile (clamped: columns at or beyond count
    // compute a duplicate that is never stored)
    if (tid < kBN) {
        int s = col0 + tid;
        int last = max(count - 1, 0);
        int f = p.idx ? min(max(p.idx[(int64_t)unit * p.k_stride + min(s, last)], 0), p.F - 1) : min(s, last);
        s_neuron[tid] = f;
    }
    __syncthreads();

    // per-lane source offsets (bytes) of the asynchronous tile loads; the K offset is uniform
    uint32_t xoff[NIX * VW], woff[NIW * VW];
#pragma unroll
    for (int i = 0; i < NIX; i++)
#pragma unroll
        for (int v = 0; v < VW; v++) {
            int row = (i * 4 + v) * 8 + (lane >> 3);
            int chunk16 = (lane & 7) ^ ((row >> 1) & 7);
            int tok = min(row0 + row, p.N - 1);
            xoff[i * VW + v] = (uint32_t)tok * (uint32_t)(p.D * 2) + chunk16 * 16;
        }
#pragma unroll
    for (int i = 0; i < NIW; i++)
#pragma unroll
        for (int v = 0; v < VW; v++) {
            int row = (i * 4 + v) * 8 + (lane >> 3);
            int chunk16 = (lane & 7) ^ ((row >> 1) & 7);
            woff[i * VW + v] = (uint32_t)s_neuron[row] * (uint32_t)(p.D * 2) + chunk16 * 16;
        }
    const uint16_t* xb = p.x + (int64_t)b * p.N * p.D;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    // One of the transfers that bring contraction step kt into buffer `stage`.
    auto issue_piece = [&](int kt, int stage, int j) {   // j < (NIX + NIW) * VW; piece (i, v) = (j / VW, j % VW)
        const int i = j / VW, v = j % VW;
        if (i < NIX) {
            load_global_to_lds_16B(xb + kt * kBK, xoff[j], lds0 + stage * STAGE + i * 4096 + v * 1024);
        } else {
            load_global_to_lds_16B(p.w1 + kt * kBK, woff[j - NIX * VW], lds0 + stage * STAGE + XT + (i - NIX) * 4096 + v * 1024);
        }
    };

    f32x16 acc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int nt = 0; nt < 2; nt++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[mt][nt][r] = 0.f;

    // LDS read offsets: row l32 of a 32-row tile, 16-byte chunk (2*ks + h) ^ swizzle(row)
    const int sw = (l32 >> 1) & 7;
    const int aoff = (wm * (BM / 2) + l32) * 128 + ((h ^ sw) * 16);
    const int boff = XT + (wn * 64 + l32) * 128 + ((h ^ sw) * 16);

    const int ktiles = p.D / kBK;
    constexpr int NP = NIX + NIW;
    if (loader) {
#pragma unroll
        for (int st = 0; st < NS - 1; st++)
#pragma unroll
            for (int j = 0; j < NP * VW; j++) issue_piece(min(st, ktiles - 1), st, j);
    }
    int stage = 0;
    static_assert((NS - 2) * NP * VW < 64, "the transfer counter has six bits");
    if (loader) {
        for (int kt = 0; kt < ktiles; kt++) {
            wait_vmem_at_most<(NS - 2) * NP * VW>();
            __syncthreads();
            // past the end the last step is fetched again into a buffer nobody reads
            const int kt_next = min(kt + NS - 1, ktiles - 1);
            const int fill = (stage + NS - 1) % NS;
#pragma unroll
            for (int j = 0; j < NP * VW; j++) issue_piece(kt_next, fill, j);
            stage = stage + 1 == NS ? 0 : stage + 1;
        }
        wait_all_memory();                 // the transfers must have landed before the epilogue reuses the buffers
        lds_accesses_then_barrier();       // the two barriers of the epilogue
        lds_accesses_then_barrier();
        return;
    }
    for (int kt = 0; kt < ktiles; kt++) {
        __syncthreads();   // the loader wave has waited for this step's transfers
        const uint8_t* sb = smem + stage * STAGE;
        // The operands of contraction sub-step ks + 1 are requested ahead of the products of sub-step ks (two
        // register sets): with one wave per SIMD nothing else covers the LDS latency between a read and its product.
        bf16x8 aop[2][MT], bop[2][2];
        auto read_operands = [&](int ks, int set) {
#pragma unroll
            for (int nt = 0; nt < 2; nt++)
                bop[set][nt] = *reinterpret_cast<const bf16x8*>(sb + nt * 32 * 128 + (boff ^ (32 * ks)));
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
                aop[set][mt] = *reinterpret_cast<const bf16x8*>(sb + mt * 32 * 128 + (aoff ^ (32 * ks)));
        };
        read_operands(0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, MT + 2, 0);
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            if (ks + 1 < 4) {
                read_operands(ks + 1, (ks + 1) & 1);
                __builtin_amdgcn_sched_group_barrier(0x100, MT + 2, 0);   // the reads lead the block
            }
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
#pragma unroll
                for (int nt = 0; nt < 2; nt++)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop[ks & 1][mt], bop[ks & 1][nt], acc[mt][nt], 0, 0, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            }
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // ---- epilogue: bias, activation, bf16, transpose to [neuron][token] through LDS ----
    constexpr int CPR = BM / 8;                  // 16-byte chunks (8 tokens) per neuron row
    constexpr int ITEMS = kBN * CPR / 256;       // (neuron, 8 tokens) cells per thread
    static_assert(kBN * CPR % 256 == 0, "the tile's cells must divide over the threads");
    // The cached activations of this thread's cells are requested here, ahead of the activation arithmetic and
    // the transposition, so that their latency is paid once and in the shadow of that work.  One 16-byte load per
    // cell whatever the case (cells past the end of the row or of the list read a valid address and are not
    // used): a_ld is a multiple of 8 and at least N, so a cell that starts below N ends inside its row.
    // bias of the lane's two neuron columns: requested first (the activation arithmetic waits for these only) and
    // without a branch (w1 stands in as a valid address when there is no bias)
    const uint16_t* bias_src = p.b1 ? p.b1 : p.w1;
    uint16_t bias_raw[2];
#pragma unroll
    for (int nt = 0; nt < 2; nt++) bias_raw[nt] = bias_src[s_neuron[wn * 64 + nt * 32 + l32]];
    u32x4 old8[ITEMS];
    uint16_t* cell[ITEMS];   // the thread's cells in a_cache (token clamped to the row's start where the chunk ends early)
#pragma unroll
    for (int n = 0; n < ITEMS; n++) {
        const int item = tid + n * 256;
        const int nl = item / CPR, ch = item - nl * CPR;
        const int tok0 = row0 + ch * 8;
        cell[n] = p.a_cache + ((int64_t)b * p.F + s_neuron[nl]) * p.a_ld + (tok0 < p.N ? tok0 : 0);
        if (MODE == kSparseDelta) old8[n] = *reinterpret_cast<const u32x4*>(cell[n]);
    }
    lds_accesses_then_barrier();  // every wave is done with the stage buffers
    float bias[2];
#pragma unroll
    for (int nt = 0; nt < 2; nt++) bias[nt] = p.b1 ? bf16_bits_to_float(bias_raw[nt]) : 0.f;
    auto activate_tile = [&](auto form) {
        constexpr int ACT = decltype(form)::value;
#pragma unroll
        for (int nt = 0; nt < 2; nt++) {
            int nl = wn * 64 + nt * 32 + l32;
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int rg = 0; rg < 4; rg++) {
                    int tl = wm * (BM / 2) + mt * 32 + rg * 8 + h * 4;
                    float a0 = gelu<ACT>(acc[mt][nt][rg * 4 + 0] + bias[nt]);
                    float a1 = gelu<ACT>(acc[mt][nt][rg * 4 + 1] + bias[nt]);
                    float a2 = gelu<ACT>(acc[mt][nt][rg * 4 + 2] + bias[nt]);
                    float a3 = gelu<ACT>(acc[mt][nt][rg * 4 + 3] + bias[nt]);
                    u32x2 v = {pack_bf16x2(a0, a1), pack_bf16x2(a2, a3)};
                    *reinterpret_cast<u32x2*>(smem + nl * TS + tl * 2) = v;
                }
        }
    };
    if (p.act == CHIPMUNK_ACT_GELU_ERF) activate_tile(std::integral_constant<int, CHIPMUNK_ACT_GELU_ERF>{});
    else activate_tile(std::integral_constant<int, CHIPMUNK_ACT_GELU_TANH>{});
    lds_accesses_then_barrier();
    // The cells are handled in three sweeps (read the transposed tile, form the deltas, store) of straight-line
    // code: in one loop with a branch per cell every cell waited for its own LDS reads, and the compiler, which
    // counts a wait as if no store had been issued on the way, made it wait for the stores of the cells before.
    u32x4 a8[ITEMS];
#pragma unroll
    for (int n = 0; n < ITEMS; n++) {
        const int item = tid + n * 256;
        const int nl = item / CPR, ch = item - nl * CPR;
        a8[n] = *reinterpret_cast<const u32x4*>(smem + nl * TS + ch * 16);
    }
    if (MODE == kSparseDelta) {
        // the cached activations, requested before the activation arithmetic, are taken as arrived in one wait
#pragma unroll
        for (int n = 0; n < ITEMS; n++) asm volatile("" ::"v"(old8[n]), "v"(a8[n]));
        uint16_t* dunit = p.delta_t + (int64_t)unit * p.k_pad * BM;
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid + n * 256;
            const int nl = item / CPR, ch = item - nl * CPR;
            const int s = col0 + nl;
            // tokens past N and padding rows of the contraction must read as zero in GEMM2
            const int nvalid = s < count ? min(8, p.N - (row0 + ch * 8)) : 0;
            u32x4 d8;
#pragma unroll
            for (int e2 = 0; e2 < 4; e2++) {
                float dlo = bf16_bits_to_float(a8[n][e2] & 0xffffu) - bf16_bits_to_float(old8[n][e2] & 0xffffu);
                float dhi = bf16_bits_to_float(a8[n][e2] >> 16) - bf16_bits_to_float(old8[n][e2] >> 16);
                if (2 * e2 >= nvalid) dlo = 0.f;
                if (2 * e2 + 1 >= nvalid) dhi = 0.f;
                d8[e2] = pack_bf16x2(dlo, dhi);
            }
            if (s < p.k_pad) *reinterpret_cast<u32x4*>(dunit + (s * BM + ch * 8)) = d8;
        }
    }
#pragma unroll
    for (int n = 0; n < ITEMS; n++) {
        const int item = tid + n * 256;
        const int nl = item / CPR, ch = item - nl * CPR;
        const int s = col0 + nl;
        const int nvalid = s < count ? min(8, p.N - (row0 + ch * 8)) : 0;
        if (MODE == kSparseDelta && p.act_t) {   // deferred write-back: one coalesced store, whole cell
            if (nvalid > 0) *reinterpret_cast<u32x4*>(p.act_t + ((int64_t)unit * p.k_pad + s) * BM + ch * 8) = a8[n];
        } else if (nvalid == 8) {
            *reinterpret_cast<u32x4*>(cell[n]) = a8[n];
        } else {  // the cells past N in the last chunk stay as they are
            for (int e = 0; e < nvalid; e++) cell[n][e] = (uint16_t)(a8[n][e >> 1] >> (16 * (e & 1)));
        }
    }
}

struct Gemm2Params {
    const uint16_t* a_t;     // sparse: delta^T workspace [units, k_pad, BM]; dense: a_cache [B, F, a_ld]
    const uint16_t* w2;      // [F, D]
    const uint16_t* bias;    // dense: b2 [D] or null
    const int32_t* idx;      // [units, k_stride] or null
    const int32_t* counts;   // [units] or null
    uint16_t* o;             // sparse: o_cache in/out; dense: out
    int64_t a_ld;
    int N, NB, D, F, k_stride, k_pad;
    int col_tiles, units;    // launch geometry (see xcd_tile_of_block)
    // Deferred cache write-back (App. B.3.3): workgroups with id >= tile_blocks, one per unit, copy the new
    // activations that the first GEMM left in act_t into a_cache while the tile workgroups of this launch compute.
    const uint16_t* act_t;   // null: no write-back workgroups
    uint16_t* a_cache;
    int tile_blocks;
    int whole;               // tiles per XCD that a workgroup takes whole; the others are taken 64 rows at a time
    int parts;               // tiles of 64 x 64 only: row tiles per unit
};

// The deferred write-back of chunk u's new activations, by a workgroup of 256 threads.  These workgroups have the highest ids,
// so they start when the tile workgroups' last round leaves compute units free, and their memory traffic runs beside that
// round's products.  Bound: the round trips of a thread, beyond the XCD's L2 where another XCD ran the chunk's first GEMM, so a
// thread requests four cells before it stores the first.  Whole calls in us, one cell at a time and four: 16 chunks of 128 x 2000
// of 4096 x 1024 93.1, 58.5 (72.6 while a chunk stayed on its XCD); 24 of 192 x 1229 of 12 288 x 3072 123.5, 97.2; 94 x 967 of
// 13 824 x 5120 494, 470.
__device__ __forceinline__ void write_back_activations(const Gemm2Params& p, int u, int c) {
    constexpr int AHEAD = 4;
    const int ub = u / p.NB, urow0 = (u % p.NB) * c;
    const int cells = c / 8, n = max(min(p.counts[u], p.k_stride), 0) * cells;
    for (int first = threadIdx.x; first < n; first += 256 * AHEAD) {
        int f[AHEAD];
        u32x4 a8[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; i++) {
            const int item = min(first + i * 256, n - 1), s = item / cells, ch = item - s * cells;
            f[i] = p.idx[(int64_t)u * p.k_stride + s];
            a8[i] = *reinterpret_cast<const u32x4*>(p.act_t + ((int64_t)u * p.k_pad + s) * c + ch * 8);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; i++) {
            const int item = first + i * 256, tok0 = urow0 + item % cells * 8;
            const int nvalid = item < n ? min(8, p.N - tok0) : 0;
            uint16_t* arow = p.a_cache + ((int64_t)ub * p.F + min(max(f[i], 0), p.F - 1)) * p.a_ld + tok0;
            if (nvalid == 8) {
                *reinterpret_cast<u32x4*>(arow) = a8[i];
            } else {  // the cells past N in the last chunk stay as they are
                for (int e = 0; e < nvalid; e++) arow[e] = (uint16_t)(a8[i][e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

// 16-byte chunk position of an A^T or w2 tile row: four rows of 64 bytes (what 32 lanes of a transposing read ask for) lie in 256
// different bytes.  Rows of 128 or 384 bytes alternate between the halves by themselves.
template <int ROWB>
__device__ __forceinline__ int swizzle_at(int row) {
    if (ROWB % 256 != 0) return (row & 2) << 1;
    return ((row & 3) << 2) | ((row >> 2) & 3);
}

// 4-byte form of load_buffer_to_lds_16B: lane l deposits its dword at lds_wave_base + 4 l
__device__ __forceinline__ void load_buffer_to_lds_4B(i32x4 buffer, uint32_t byte_offset, uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds_wave_base), "v"(byte_offset), "s"(buffer)
                 : "memory");
}

// the same buffer `bytes` further on
__device__ __forceinline__ i32x4 buffer_moved_on(i32x4 buffer, uint32_t bytes) {
    const uint64_t base = ((uint64_t)(uint32_t)buffer[1] << 32 | (uint32_t)buffer[0]) + bytes;
    buffer[0] = (int)(uint32_t)base;
    buffer[1] = (int)(uint32_t)(base >> 32);
    return buffer;
}

constexpr int kGemm2K = 32;   // contraction tile of the second GEMM
template <int ROWS>
struct Gemm2Shape {           // of a workgroup that owns ROWS token rows
    static constexpr int kStages = ROWS == 192 ? 3 : 4;
    static constexpr int kListSlots = 8;                            // kStages + 2 are in use at a time
    static constexpr int kStage = kGemm2K * (ROWS * 2 + kBN * 2);   // A^T tile [32][ROWS], w2 tile [32][128]
    static constexpr int kList = kListSlots * 4 * 256;              // 64 list entries per wave and slot
    static constexpr int kEpilogue = (ROWS / 2) * (kBN * 4 + 32);   // half the fp32 result
    static constexpr int kLds = (kStages * kStage > kEpilogue ? kStages * kStage : kEpilogue) + kList;
};

// The work of one workgroup: ROWS rows (the chunk's, or its 64 rows `part`) and 128 output columns.
// The contraction runs in steps of 32 through a ring of kStages stages; the step after the one that is multiplied is already in
// registers, so a stage is free again as soon as its operands have been read.  The list comes the same way: every wave keeps
// a ring of its own of slices of 64 entries in LDS, kStages steps ahead of the gather that uses them, so no load into
// registers stands between the transfers and nothing waits for more than the step it needs.  With two buffers of 64 rows, one
// drained at the head of every step, a CU had 40 KB in flight on average and took 10 TB/s into LDS.  Whole deltas in us, two
// buffers and this ring: 394 chunks x 968 of 13 824 x 5120 1860 -> 1785, 24 x 1229 of 12 288 x 3072 101 -> 96.5, c = 128: 1350 x
// 442 of 6144 x 2944 1440 -> 1324; dense, 11 chunks of 128 x 2176 x 5760: 120 -> 104.
// LONG: a chunk's rows of A^T may be more than 32 bits of bytes.
template <int BM, int ROWS, bool DENSE, bool STREAM, bool LONG>
__device__ __forceinline__ void gemm2_rows(const Gemm2Params& p, int unit, int part, int col_tile) {
    typedef Gemm2Shape<ROWS> Shape;
    constexpr int NS = Shape::kStages, SLOTS = Shape::kListSlots, STAGE = Shape::kStage;
    constexpr int MT = ROWS / 64;                  // 32-row MFMA tiles per wave (wave tile = ROWS/2 x 64)
    constexpr int RBA = ROWS * 2;                  // bytes per row of the A^T tile
    constexpr int CPA = ROWS / 8;                  // 16-byte chunks per A^T row
    constexpr int AT = kGemm2K * RBA;              // A^T tile bytes
    constexpr int NIA = kGemm2K * CPA / 256;       // loads per lane, A^T tile
    constexpr int NIW = kGemm2K * 16 / 256;        // loads per lane, w2 tile
    constexpr int G = NIA + NIW + (DENSE ? 0 : 1); // transfers of a wave and step, with the slice of the list
    constexpr int CS = kBN * 4 + 32;               // row stride (bytes) of the fp32 epilogue tile
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = w & 1;
    const int l16 = lane & 15, mb = (lane >> 4) & 1, h = lane >> 5;
    const int b = unit / p.NB, chunk = unit % p.NB;
    const int row0 = chunk * BM + part * ROWS;
    const int d0 = col_tile * kBN;
    const int count = DENSE ? p.F : min(p.counts[unit], p.k_stride);
    if (row0 >= p.N || count <= 0) return;         // nothing selected: the cache stays as it is
    const int steps = (count + kGemm2K - 1) / kGemm2K;

    // A^T source: row (selected slot or neuron) -> tokens of this chunk
    const int64_t a_row = DENSE ? p.a_ld : BM;     // elements between consecutive contraction rows
    i32x4 abuf = DENSE ? raw_buffer_words(p.a_t + (int64_t)b * p.F * p.a_ld, (uint32_t)p.F * (uint32_t)p.a_ld * 2u)
                       : raw_buffer_words(p.a_t + (int64_t)unit * p.k_pad * BM, LONG ? 0xffffffffu : (uint32_t)p.k_pad * BM * 2u);
    const i32x4 wbuf = raw_buffer_words(p.w2, (uint32_t)p.F * p.D * 2u);
    const i32x4 ibuf = DENSE ? wbuf : raw_buffer_words(p.idx + (int64_t)unit * p.k_stride, (uint32_t)p.k_stride * 4u);
    constexpr int kMove = 1 << 17;                 // LONG: the steps' offsets count from `moved`, which follows in steps this far apart
    int moved = 0;
    const uint32_t astep = (uint32_t)(kGemm2K * a_row * 2), wstep = DENSE ? (uint32_t)(kGemm2K * p.D * 2) : 0u;
    uint32_t aoff[NIA], woff[NIW];
#pragma unroll
    for (int i = 0; i < NIA; i++) {
        const int q = (i * 4 + w) * 64 + lane;     // linear 16-byte chunk of the tile
        const int row = q / CPA, pos = q - row * CPA;
        int c16 = pos ^ swizzle_at<RBA>(row);
        // dense: tokens beyond N read any valid data, their rows are not stored
        const int tok = DENSE ? (row0 + c16 * 8 < p.N ? row0 + c16 * 8 : row0) : part * ROWS + c16 * 8;
        aoff[i] = (uint32_t)(row * a_row * 2) + (uint32_t)tok * 2u;
    }
    int wrow[NIW];
#pragma unroll
    for (int i = 0; i < NIW; i++) {
        wrow[i] = (i * 4 + w) * 4 + (lane >> 4);
        woff[i] = (uint32_t)((lane & 15) ^ swizzle_at<256>(wrow[i])) * 16u + (uint32_t)d0 * 2u + (DENSE ? (uint32_t)wrow[i] * (uint32_t)(p.D * 2) : 0u);
    }
    const uint32_t lds0 = lds_address(smem);
    const uint32_t list0 = lds0 + (uint32_t)(Shape::kLds - Shape::kList) + (uint32_t)w * (SLOTS * 256u);
    // slice s: list entries 32 s ..; entries past the end repeat the last one (their deltas are zero)
    auto request_slice = [&](int s) {
        if (!DENSE) load_buffer_to_lds_4B(ibuf, (uint32_t)min(s * kGemm2K + lane, count - 1) * 4u, list0 + (uint32_t)((s & (SLOTS - 1)) * 256));
    };
    uint32_t row_at[NIW] = {};                     // byte offsets of the w2 rows of the step that is requested next
    auto read_slice = [&](int s) {
        if (!DENSE) {
            const uint32_t at = list0 + (uint32_t)((s & (SLOTS - 1)) * 256);
#pragma unroll
            for (int i = 0; i < NIW; i++)
                row_at[i] = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>((uintptr_t)(at + (uint32_t)wrow[i] * 4u));
        }
    };
    // one of the NIA + NIW transfers of step t into stage t % NS
    auto request_piece = [&](int t, uint32_t stage, int j) {
        if (j < NIA) {
            load_buffer_to_lds_16B(abuf, aoff[j], (uint32_t)(t - moved) * astep, stage + (uint32_t)((j * 4 + w) * 1024));
        } else {
            const int i = j - NIA;
            const uint32_t row = DENSE ? 0u : (uint32_t)min(max((int)row_at[i], 0), p.F - 1) * (uint32_t)(p.D * 2);
            load_buffer_to_lds_16B(wbuf, woff[i] + row, (uint32_t)t * wstep, stage + (uint32_t)(AT + (i * 4 + w) * 1024));
        }
    };

    f32x16 acc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int nt = 0; nt < 2; nt++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[mt][nt][r] = 0.f;

    // Transposing reads.  For a k-step of 16 contraction rows, half h of the wave takes rows 8h..8h+7 as two groups of 4;
    // inside a block of 16 lanes, lane i addresses row (i/4) of the group and 4 consecutive columns 4*(i%4).
    typedef __attribute__((ext_vector_type(8))) short short8v;
    uint32_t rat[MT][2], rwt[2][2];                // [block][group of 4 rows]: read addresses in stage 0, + 16 rows per k-step
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
#pragma unroll
    for (int rd = 0; rd < 2; rd++) {
        const int row = 8 * h + (l16 >> 2) + 4 * rd, tcol = 4 * (l16 & 3);
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const int col = wm * (ROWS / 2) + mt * 32 + mb * 16 + tcol;
            rat[mt][rd] = smem_at + (uint32_t)(row * RBA + ((col >> 3) ^ swizzle_at<RBA>(row)) * 16 + (col & 7) * 2);
        }
#pragma unroll
        for (int nt = 0; nt < 2; nt++) {
            const int col = wn * 64 + nt * 32 + mb * 16 + tcol;
            rwt[nt][rd] = smem_at + (uint32_t)(AT + row * 256 + ((col >> 3) ^ swizzle_at<256>(row)) * 16 + (col & 7) * 2);
        }
        // opaque, so that the k-step stays in the reads' offset field
#pragma unroll
        for (int mt = 0; mt < MT; mt++) asm volatile("" : "+v"(rat[mt][rd]));
#pragma unroll
        for (int nt = 0; nt < 2; nt++) asm volatile("" : "+v"(rwt[nt][rd]));
    }
    struct Operands { bf16x8 a[2][MT], w[2][2]; };   // [k-step]
    auto read = [&](Operands& op, uint32_t stage) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
#pragma unroll
            for (int nt = 0; nt < 2; nt++)
                op.w[ks][nt] = __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(
                    lds_read_tr16_at(rwt[nt][0] + stage + ks * 16 * 256), lds_read_tr16_at(rwt[nt][1] + stage + ks * 16 * 256), 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
                op.a[ks][mt] = __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(
                    lds_read_tr16_at(rat[mt][0] + stage + ks * 16 * RBA), lds_read_tr16_at(rat[mt][1] + stage + ks * 16 * RBA), 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };

    if (!DENSE) {
#pragma unroll
        for (int s = 0; s < NS + 2; s++) request_slice(s);
        wait_all_memory();
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int t = 0; t < NS; t++) {
        if (t < steps) {
            read_slice(t);
#pragma unroll
            for (int j = 0; j < NIA + NIW; j++) request_piece(t, lds0 + t * STAGE, j);
            if (t >= 2) request_slice(t + NS);
        }
    }
    read_slice(NS);
    if (steps >= NS) wait_vmem_at_most<(NS - 1) * G - (DENSE ? 0 : 1)>();
    else wait_vmem_at_most<0>();
    lds_accesses_then_barrier();
    Operands even, odd;
    read(even, 0);
    // (stage numbers wrap at NS, which is no power of two: they travel with the steps)
    uint32_t here = 0;                             // byte offset of the stage of step t
    auto after = [&](uint32_t stage) { return stage + STAGE == NS * STAGE ? 0u : stage + STAGE; };
    auto step = [&](auto ends_c, int t, Operands& now, Operands& next) {
        constexpr bool ends = decltype(ends_c)::value;   // no more steps to request
        if (!ends || steps - 2 - t >= NS - 2) wait_vmem_at_most<(NS - 2) * G>();   // step t + 1 has landed
        else if (NS == 4 && steps - 2 - t == 1) wait_vmem_at_most<G>();
        else wait_vmem_at_most<0>();
        lds_accesses_then_barrier();               // for every wave; and every wave holds its operands of step t
        const uint32_t there = after(here);
        if (!ends || t + 1 < steps) read(next, there);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
#pragma unroll
                for (int nt = 0; nt < 2; nt++)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(now.a[ks][mt], now.w[ks][nt], acc[mt][nt], 0, 0, 0);
                if (!ends) {
                    constexpr int each = (NIA + NIW + 2 * MT - 1) / (2 * MT);
#pragma unroll
                    for (int e = 0; e < each; e++)
                        if ((ks * MT + mt) * each + e < NIA + NIW) request_piece(t + NS, lds0 + here, (ks * MT + mt) * each + e);
                }
            }
        if (!ends) {
            request_slice(t + 2 * NS);
            read_slice(t + NS + 1);
        }
        here = there;
    };
    int t = 0;
    for (;;) {
        const int end = LONG ? min(steps, moved + kMove + NS + 1) : steps;
        for (; t + NS + 1 < end; t += 2) {
            step(std::false_type{}, t, even, odd);
            step(std::false_type{}, t + 1, odd, even);
        }
        if (!LONG || end == steps) break;          // (a move at every step: 75 600 x 5120 x 7 % 1740 -> 1752 us; like this 1735)
        abuf = buffer_moved_on(abuf, kMove * astep);
        moved = t;
    }
    if (t + NS < steps) {
        step(std::false_type{}, t, even, odd);
        t++;
        even = odd;
    }
    for (; t < steps; t += 2) {
        step(std::true_type{}, t, even, odd);
        if (t + 1 < steps) step(std::true_type{}, t + 1, odd, even);
    }

    // ---- epilogue: fp32 tile through LDS, one half of the token rows at a time ----
    // What is added to (the cached output, or the bias of the dense form) is requested for both halves before the
    // tile goes through LDS: the reads are in flight behind the barriers instead of one round trip per item.
    const int l32 = lane & 31;
    constexpr int ITEMS = (ROWS / 2) * 32 / 256;     // 16-byte groups of four output columns per thread and half
    static_assert((ROWS / 2) * 32 % 256 == 0, "the half tile must divide over the threads");
    u32x2 old[2][ITEMS];
#pragma unroll
    for (int half = 0; half < 2; half++)
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid + n * 256;
            const int tl = item >> 5, ch = item & 31;
            const int tok = row0 + half * (ROWS / 2) + tl;
            // one load per item whatever the case (a token past the end reads the last token's row, the dense form
            // without a bias reads the output buffer; neither value is used): branches here would make every
            // load wait for the one before
            const uint16_t* src = (DENSE && p.bias)
                                      ? p.bias + d0 + ch * 4
                                      : p.o + ((int64_t)b * p.N + min(tok, p.N - 1)) * p.D + d0 + ch * 4;
            const u32x2* at = reinterpret_cast<const u32x2*>(src);
            old[half][n] = STREAM ? __builtin_nontemporal_load(at) : *at;
        }
    const bool add_nothing = DENSE && !p.bias;
#pragma unroll
    for (int half = 0; half < 2; half++) {
        lds_accesses_then_barrier();
        if (wm == half) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int nt = 0; nt < 2; nt++)
#pragma unroll
                    for (int r = 0; r < 16; r++) {
                        int tl = mt * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
                        int dl = wn * 64 + nt * 32 + l32;
                        *reinterpret_cast<float*>(smem + tl * CS + dl * 4) = acc[mt][nt][r];
                    }
        }
        lds_accesses_then_barrier();
        if (half == 0) {
            // Every value requested above is taken as arrived before the first store, in one wait.  The stores sit
            // in branches, so the waits the compiler counts per item assume that none was issued: left to the
            // loop, the second half's items would wait for the first half's stores.
#pragma unroll
            for (int hh = 0; hh < 2; hh++)
#pragma unroll
                for (int n = 0; n < ITEMS; n++) asm volatile("" ::"v"(old[hh][n]));
        }
        // two sweeps of straight-line code (read the staged tile, then merge and store): in one loop with the
        // store's branch inside, every item waited for its own LDS read
        f32x4 a4[ITEMS];
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid + n * 256;
            a4[n] = *reinterpret_cast<const f32x4*>(smem + (item >> 5) * CS + (item & 31) * 16);
        }
#pragma unroll
        for (int n = 0; n < ITEMS; n++) {
            const int item = tid + n * 256;
            const int tl = item >> 5, ch = item & 31;
            const int tok = row0 + half * (ROWS / 2) + tl;
            uint16_t* orow = p.o + ((int64_t)b * p.N + tok) * p.D + d0 + ch * 4;
            const u32x2 o2 = add_nothing ? u32x2{0, 0} : old[half][n];
            float o0 = bf16_bits_to_float(o2[0] & 0xffffu) + a4[n][0];
            float o1 = bf16_bits_to_float(o2[0] >> 16) + a4[n][1];
            float o2f = bf16_bits_to_float(o2[1] & 0xffffu) + a4[n][2];
            float o3 = bf16_bits_to_float(o2[1] >> 16) + a4[n][3];
            u32x2 res = {pack_bf16x2(o0, o1), pack_bf16x2(o2f, o3)};
            if (tok < p.N) {
                if (STREAM) __builtin_nontemporal_store(res, reinterpret_cast<u32x2*>(orow));
                else *reinterpret_cast<u32x2*>(orow) = res;
            }
        }
    }
}


// PARTS: the tiles of an XCD beyond `whole` are taken 64 rows at a time.  (An instance of its own: with the second body in the
// same kernel launches that never reach it were 0.5 to 1 % slower.)
// STREAM: the cached output is read and written past the caches' usual order of replacement, which leaves them to the weights:
// where it is over twice the XCDs' L2s.  Whole deltas in us without and with: 75 600 x 5120 (774 MB) 1777, 1728; 28 438 x 4096
// (233 MB) 216, 196; 19 327 x 2304 (89 MB) 92.6, 85.3; 2 x 7394 x 1792 (53 MB) 41.7, 42.9; 7669 x 1536 (24 MB) 37.6, 39.0.  An
// output of up to half the last-level cache could be read from there by the next kernel: delta and the addition that reads it, four
// blocks in turn, 42 sizes of 65 to 126 MB: 0.977 to 1.013 of the time without, 0.995 in the mean (the delta alone 0.996 to 1.135,
// 1.029); 18 of 126 to 250 MB: 0.998 to 1.029.
template <int BM, bool DENSE, bool PARTS, bool STREAM>
__global__ __launch_bounds__(256, 2) void mlp_gemm2_kernel(Gemm2Params p) {
    if (!DENSE && p.act_t && (int)blockIdx.x >= p.tile_blocks) {
        write_back_activations(p, (int)blockIdx.x - p.tile_blocks, BM);
        return;
    }
    int unit, col_tile;
    const int slot = (int)blockIdx.x >> 3;
    constexpr int parts = BM / 64;
    const int beyond = PARTS ? slot - p.whole : -1, tile_slot = beyond < 0 ? slot : p.whole + beyond / parts;
    if (DENSE ? !xcd_tile_of_block_grouped(tile_slot, p.col_tiles, p.units, &unit, &col_tile)
              : !xcd_tile_of_slot(tile_slot, p.col_tiles, p.units, &unit, &col_tile))
        return;
    if constexpr (PARTS) {
        if (beyond >= 0) {
            gemm2_rows<BM, 64, DENSE, STREAM, false>(p, unit, beyond % parts, col_tile);
            return;
        }
    }
    gemm2_rows<BM, BM, DENSE, STREAM, !DENSE && !PARTS>(p, unit, 0, col_tile);
}

}  // namespace chipmunk
#include "mlp_small.h"
namespace chipmunk {

// Chunk means of x in split precision: mean = hi + lo with hi = bf16(mean), lo = bf16(mean - hi); out row = [hi(0..D-1) |
// lo(0..D-1)].  A workgroup owns (chunk, 512 columns): each of its eight waves sums an eighth of the chunk's rows for 64
// groups of 8 columns, the partial sums meet in LDS.
// Bound: HBM (x read once).  A wave requests six rows (16 bytes per lane each) before it adds the first: with one row at
// a time and four waves a small problem took as many round trips as a wave had rows: 24 chunks of 192 x 3072 15.5 -> 6.9
// us, 8 of 128 x 256 7.2 -> 4.4 us, 602 of 192 x 3072 139 -> 127 us (5.6 TB/s).
// STREAM: loads past the caches' usual order of replacement, for an x that does not fit the last-level cache.  Means and
// scores together, us without and with: 709 MB 220.6, 201.6; 414 MB 127, 109; 298 MB 108, 99; 162 MB (just read) 43.8,
// 47.3.
// LANES: lanes per row, 64 or, where a workgroup per 512 columns leaves the chip idle, 16 (128 columns, four rows a load:
// a chunk of 192 is requested at once).
constexpr int kMeanWaves = 8, kMeanAhead = 6;
template <bool STREAM, int LANES>
__global__ __launch_bounds__(64 * kMeanWaves) void chunk_mean_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ xm,
                                                                     int N, int NB, int D, int c) {
    constexpr int ROWS = 64 / LANES;                 // rows per load
    __shared__ float s_part[kMeanWaves - 1][8][LANES];
    const int col_blocks = (D / 8 + LANES - 1) / LANES;   // grid.x = units * col_blocks
    const int unit = blockIdx.x / col_blocks;
    const int b = unit / NB, chunk = unit % NB;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int col8 = (blockIdx.x % col_blocks) * LANES + lane % LANES;
    const bool live = col8 * 8 < D;
    const int r0 = chunk * c, r1 = min(N, r0 + c);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (live) {
        const uint16_t* xc = x + (int64_t)b * N * D + col8 * 8;
        for (int r = r0 + w * ROWS + lane / LANES; r < r1; r += kMeanWaves * ROWS * kMeanAhead) {
            u32x4 v[kMeanAhead];
#pragma unroll
            for (int i = 0; i < kMeanAhead; i++) {
                const u32x4* at = reinterpret_cast<const u32x4*>(xc + (int64_t)min(r + i * kMeanWaves * ROWS, r1 - 1) * D);
                v[i] = STREAM ? __builtin_nontemporal_load(at) : *at;
            }
#pragma unroll
            for (int i = 0; i < kMeanAhead; i++) {
                const bool exists = r + i * kMeanWaves * ROWS < r1;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t pair = exists ? v[i][e] : 0u;
                    s[2 * e] += bf16_bits_to_float(pair & 0xffffu);
                    s[2 * e + 1] += bf16_bits_to_float(pair >> 16);
                }
            }
        }
    }
    if (ROWS == 4) {
#pragma unroll
        for (int e = 0; e < 8; e++) s[e] = rows4_sum(s[e]);
    }
    if (w > 0 && lane < LANES) {
#pragma unroll
        for (int e = 0; e < 8; e++) s_part[w - 1][e][lane] = s[e];
    }
    __syncthreads();
    if (w > 0 || lane >= LANES || !live) return;
#pragma unroll
    for (int i = 0; i < kMeanWaves - 1; i++)
#pragma unroll
        for (int e = 0; e < 8; e++) s[e] += s_part[i][e][lane];
    const float inv = 1.f / (float)(r1 - r0);
    u32x4 hi4, lo4;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        float m0 = s[2 * e] * inv, m1 = s[2 * e + 1] * inv;
        uint32_t hp = pack_bf16x2(m0, m1);
        hi4[e] = hp;
        lo4[e] = pack_bf16x2(m0 - bf16_bits_to_float(hp & 0xffffu), m1 - bf16_bits_to_float(hp >> 16));
    }
    uint16_t* orow = xm + (int64_t)unit * 2 * D;
    *reinterpret_cast<u32x4*>(orow + col8 * 8) = hi4;
    *reinterpret_cast<u32x4*>(orow + D + col8 * 8) = lo4;
}

// Scores of few chunks: T[n][f] = <hi[n] + lo[n], w1[f]> for up to 16 UB chunks and 16 NBK neurons per workgroup.
// Bound: w1 from memory, read once, as long as the means, which every workgroup reads whole from L2, are few
// (few_scores).  The eight waves of a workgroup cut the contraction among them, 64 entries (a cache line of a row) at a
// time in turn, and load both operands from memory in the products' own layout; the partial sums meet in LDS in a fixed
// order, so no partial result goes through memory and nothing is left for another launch.
constexpr int kFewWaves = 8;
template <int UB, int NBK>
__global__ __launch_bounds__(64 * kFewWaves) void mlp_few_scores_kernel(const uint16_t* __restrict__ xm, const uint16_t* __restrict__ w1,
                                                                       float* __restrict__ T, int units, int D, int F) {
    constexpr int AHEAD = UB * NBK <= 2 && NBK == 1 ? 2 : 1;   // more was not faster: the waves cover each other
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    f32x4 (*s_part)[NBK * UB][64] = reinterpret_cast<f32x4 (*)[NBK * UB][64]>(smem);
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int f0 = (int)blockIdx.x * 16 * NBK;
    const __amdgpu_buffer_rsrc_t wbuf = raw_buffer(w1, (uint32_t)F * D * 2u), mbuf = raw_buffer(xm, (uint32_t)units * D * 4u);
    uint32_t wat[NBK], mat[UB];   // byte offsets of the lane's rows; chunks beyond the last repeat it and are not stored
#pragma unroll
    for (int nb = 0; nb < NBK; nb++) wat[nb] = (uint32_t)(f0 + nb * 16 + l16) * (uint32_t)(D * 2) + g * 16;
#pragma unroll
    for (int ub = 0; ub < UB; ub++) mat[ub] = (uint32_t)min(ub * 16 + l16, units - 1) * (uint32_t)(D * 4) + g * 16;
    struct Entries { bf16x8 w[NBK][2], m[UB][2][2]; };   // [slice of 32]; means: [high, low][slice]
    auto load = [&](Entries& e, int at) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            const int from = at * 128 + ks * 64;
#pragma unroll
            for (int nb = 0; nb < NBK; nb++) e.w[nb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wbuf, wat[nb], from, 0));
#pragma unroll
            for (int ub = 0; ub < UB; ub++)
#pragma unroll
                for (int hl = 0; hl < 2; hl++)
                    e.m[ub][hl][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(mbuf, mat[ub], from + hl * D * 2, 0));
        }
    };
    f32x4 acc[NBK][UB][2] = {};   // high and low parts apart: added to the high parts' sum, every low product costs it a rounding
    const int all = D / 64;
    Entries ring[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; i++) load(ring[i], min(w + i * kFewWaves, all - 1));
    for (int at = w; at < all; at += AHEAD * kFewWaves) {
#pragma unroll
        for (int i = 0; i < AHEAD; i++) {
            if (at + i * kFewWaves < all) {
#pragma unroll
                for (int ks = 0; ks < 2; ks++)
#pragma unroll
                    for (int nb = 0; nb < NBK; nb++)
#pragma unroll
                        for (int ub = 0; ub < UB; ub++)
#pragma unroll
                            for (int hl = 0; hl < 2; hl++)
                                acc[nb][ub][hl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ring[i].w[nb][ks], ring[i].m[ub][hl][ks], acc[nb][ub][hl], 0, 0, 0);
            }
            if (at + (i + AHEAD) * kFewWaves < all) load(ring[i], at + (i + AHEAD) * kFewWaves);
        }
    }
#pragma unroll
    for (int nb = 0; nb < NBK; nb++)
#pragma unroll
        for (int ub = 0; ub < UB; ub++) s_part[w][nb * UB + ub][lane] = acc[nb][ub][0] + acc[nb][ub][1];
    __syncthreads();
    for (int i = threadIdx.x; i < NBK * UB * 64; i += 64 * kFewWaves) {
        const int block = i >> 6, l = i & 63, n = block % UB * 16 + (l & 15);
        f32x4 sum = s_part[0][block][l];
#pragma unroll
        for (int ww = 1; ww < kFewWaves; ww++) sum += s_part[ww][block][l];
        if (n < units) *reinterpret_cast<f32x4*>(T + (int64_t)n * F + f0 + block / UB * 16 + (l >> 4) * 4) = sum;
    }
}

// out[i] = sum over the pieces of a split contraction, in piece order (deterministic)
__global__ __launch_bounds__(256) void sum_pieces_kernel(const float* __restrict__ part, float* __restrict__ out,
                                                         int64_t n4, int pieces) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int pc = 0; pc < pieces; pc += 4) {   // four pieces requested before the first is added
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = reinterpret_cast<const f32x4*>(part)[min(pc + j, pieces - 1) * n4 + i];
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (pc + j < pieces) acc += v[j];
    }
    reinterpret_cast<f32x4*>(out)[i] = acc;
}

template <int BM, int MODE>
static int32_t launch_gemm1(Gemm1Params p, int col_tiles, int units, hipStream_t s) {
    p.col_tiles = col_tiles;
    p.units = units;
    constexpr int lds = 3 * (BM * 128 + kBN * 128);
    // set at every launch: the attribute is kept per device (a flag remembered here would not be)
    if (hipFuncSetAttribute((const void*)mlp_gemm1_kernel<BM, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, lds) !=
        hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    hipLaunchKernelGGL((mlp_gemm1_kernel<BM, MODE>), dim3((unsigned)xcd_grid_size(col_tiles, units)), dim3(320), lds, s, p);
    return launch_status();
}

// whether the delta's cached output passes the caches by (STREAM)
static bool stream_output(int64_t units, int c, int D) { return units * c * D * 2 > 2 * kAllL2; }

// whole: tiles per XCD that a workgroup takes whole
template <int BM, bool DENSE>
static int32_t launch_gemm2(Gemm2Params p, int col_tiles, int units, int64_t whole, hipStream_t s) {
    p.col_tiles = col_tiles;
    p.units = units;
    const int slots = xcd_grid_size(col_tiles, units) / 8;
    p.whole = (int)std::min<int64_t>(whole, slots);
    p.tile_blocks = 8 * (p.whole + (slots - p.whole) * (BM / 64));
    const int grid = p.tile_blocks + (p.act_t ? units : 0);
    auto launch = [&](auto kernel, int lds) {
        if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return (int32_t)CHIPMUNK_ERR_LAUNCH;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), lds, s, p);
        return launch_status();
    };
    constexpr int lds = Gemm2Shape<BM>::kLds, lds64 = Gemm2Shape<64>::kLds;
    constexpr int lds_parts = lds > lds64 ? lds : lds64;
    if (!DENSE && stream_output(units, BM, p.D))
        return p.whole == slots ? launch(mlp_gemm2_kernel<BM, DENSE, false, !DENSE>, lds)
                                : launch(mlp_gemm2_kernel<BM, DENSE, true, !DENSE>, lds_parts);
    return p.whole == slots ? launch(mlp_gemm2_kernel<BM, DENSE, false, false>, lds)
                            : launch(mlp_gemm2_kernel<BM, DENSE, true, false>, lds_parts);
}

// Tiles of 64 x 64.  `units`: sparse: chunks of `parts` row tiles; dense: row tiles of all batches (parts = 1).
template <int MODE>
static int32_t launch_small_gemm1(Gemm1Params p, int units, hipStream_t s) {
    p.col_tiles = (p.k_stride + kSmallTile - 1) / kSmallTile;
    p.units = units;
    constexpr int lds = kSmallStages * kSmallStage;
    if (hipFuncSetAttribute((const void*)mlp_small_gemm1_kernel<MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    hipLaunchKernelGGL((mlp_small_gemm1_kernel<MODE>), dim3((unsigned)xcd_grid_size(p.col_tiles * p.parts, units)), dim3(256), lds, s, p);
    return launch_status();
}
template <bool SPARSE>
static int32_t launch_small_gemm2(Gemm2Params p, int units, hipStream_t s) {
    p.col_tiles = p.D / kSmallTile;
    p.units = units;
    const int lds = kSmallStages * kSmallStage + (SPARSE ? p.k_pad * 4 : 0);
    if (hipFuncSetAttribute((const void*)mlp_small_gemm2_kernel<SPARSE>, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    p.tile_blocks = xcd_grid_size(p.col_tiles * p.parts, units);
    hipLaunchKernelGGL((mlp_small_gemm2_kernel<SPARSE>), dim3((unsigned)(p.tile_blocks + (p.act_t ? units : 0))), dim3(256), lds, s, p);
    return launch_status();
}

// ---- which tiles a GEMM takes ----
// Every form is priced as rounds of the busiest XCD's workgroups over its 32 CUs (tiles of a chunk's rows or of 256 x 256: one
// workgroup per CU in the first GEMM and for 256 x 256, else two) plus a last round that is partly filled, and the cheapest is
// taken.  In us: `call` + (`step` n + `end`) x (whole rounds + last), n contraction steps (64 in the first GEMM, 32 in the
// second), last = `few` + `few_more` 2 x for a share x <= 1/2 of the slots and `many` + `many_more` (2 x - 1) beyond.  Fitted to
// the kernels' times at 450 sizes of the delta and 330 of the dense MLP from 500 tokens up to 2.5 TFLOP, one launch after the
// other; the large tiles' prices were then lowered by 5 (delta, c = 128) and 8 % (dense) and those of 64 x 64 in the dense form by
// 5, which whole calls in a row ask for, where the clock is lower: over 100 and 80 calls the chosen first GEMM costs 0.8 and
// 1.0 % of a call against the best one, the second 0.4 and 0.2 %.
struct Price { double step, end, call, few, few_more, many, many_more; };
static double price(const Price& p, int64_t tiles_per_xcd, int slots, int steps) {
    const int64_t last = tiles_per_xcd % slots;
    const double x = (double)last / slots;
    const double share = last == 0 ? 0. : x <= 0.5 ? p.few + p.few_more * 2. * x : p.many + p.many_more * (2. * x - 1.);
    return p.call + (p.step * steps + p.end) * ((double)(tiles_per_xcd / slots) + share);
}
static int64_t per_xcd(int64_t tiles) { return (tiles + 7) / 8; }
// A launch has fewer than 2^32 threads: 256 for each of the tiles of 64 x 64, up to six of which stand for one of the chunk's.
static bool small_launches(int64_t tiles_per_xcd) { return tiles_per_xcd * 8 * 256 < 1LL << 32; }

enum FirstForm { kFirstChunk = 0, kFirstLarge = 1, kFirstSmall = 2 };   // 128 neurons of a chunk; 256 (dense: and 256 tokens); 64 x 64
// Kernel times (chunk, large, small), us: delta, c = 192, 9 chunks x 395 of 7488 x 4864: 44, 83, 19; 47 x 1229 of 12 288 x 3072: 96, 82,
// -; 394 x 968 of 13 824 x 5120: 945, 815, -; c = 128, 14 x 1156 of 6080 x 3840: 37, 55, 30; dense 700 x 1536 x 8192: 26, 45, 34; 893 x
// 1664 x 1024 17, 41, 7; 4608 x 3072 x 12 288: 352, 274, -.
// Tiles of 64 x 64 are left out where they take more than two rounds, but for contractions of at most 14 steps (of 100 calls two fewer
// are 4 per cent slower than with the best tiles), and for lists of more than half the neurons, which were not measured.
// *us: the price of the form that is taken.
static FirstForm first_form(bool sparse, int B, int N, int D, int F, int c, int k_stride, double* us = nullptr) {
    static const Price chunk_delta[2] = {{0.74, 10.87, 6, 0.52, 0.19, 0.71, 0.19}, {0.648, 5, 6, 0.46, 0.2, 0.66, 0.2}};   // c = 192, 128
    static const Price large_delta[2] = {{1.222, 21.22, 6, 0.67, 0.17, 0.84, 0.17}, {1.015, 9.69, 5.7, 0.55, 0.17, 0.72, 0.17}};
    static const Price small_delta = {0.411, 2.64, 4.53, 0.35, 0.12, 0.77, 0.17};
    static const Price chunk_dense[2] = {{0.654, 6.67, 6, 0.58, 0.16, 0.74, 0.16}, {0.473, 5.31, 3.15, 0.48, 0.25, 0.72, 0.25}};
    static const Price large_dense = {1.305, 14.63, 5.52, 0.64, 0.19, 0.83, 0.19};
    static const Price small_dense = {0.347, 1.58, 4.66, 0.32, 0.17, 0.81, 0.14};
    const int at = c == 192 ? 0 : 1, steps = D / kBK, parts = c / kSmallTile;
    const int64_t chunks = (int64_t)B * ((N + c - 1) / c);
    const int width = sparse ? k_stride : F;
    auto cols = [&](int tile) { return (int64_t)((width + tile - 1) / tile); };
    const int64_t small_tiles = per_xcd((sparse ? chunks * parts : (int64_t)B * ((N + kSmallTile - 1) / kSmallTile)) * cols(kSmallTile));
    const int64_t large_tiles = sparse ? per_xcd(chunks * cols(kDenseTile))
                                       : B * per_xcd((int64_t)((N + kDenseTile - 1) / kDenseTile) * cols(kDenseTile));
    const double chunk = price((sparse ? chunk_delta : chunk_dense)[at], per_xcd(chunks * cols(kBN)), 32, steps);
    const double large = price(sparse ? large_delta[at] : large_dense, large_tiles, 32, steps);
    const double small = price(sparse ? small_delta : small_dense, small_tiles, 64, steps);
    const bool large_fits = sparse || B <= 65535;   // the dense form takes the batch from the second grid dimension
    const bool small_fits = small_launches(small_tiles) && (small_tiles <= 128 || steps <= 14) && (!sparse || k_stride <= F / 2);
    const FirstForm form = small_fits && small < chunk && (!large_fits || small < large) ? kFirstSmall
                           : large_fits && large < chunk                               ? kFirstLarge
                                                                                       : kFirstChunk;
    if (us) *us = form == kFirstSmall ? small : form == kFirstLarge ? large : chunk;
    return form;
}

// Second GEMM.  kSecondChunk: a workgroup per chunk and 128 columns; those beyond `whole` tiles per XCD take 64 rows each where they
// fill that XCD's 32 CUs at most once: of the last round of two per CU (24 chunks x 1229 of 12 288 x 3072, 72 tiles per XCD: 54.6 ->
// 47.2 us; 80 to 97 per cent of the time over 23 sizes with one to three whole rounds), of the only round those beyond one per CU, or all
// of them where that fills the chip better.  In an only round the CUs with two whole tiles are the last to end, more so since the
// ring leaves little idle beside a single one: dense, c = 128, 33 tiles, 2449 x 1664 x 10 304 with two buffers a workgroup 127.6 us, with
// the ring 139.6.  Whole calls, 33 to 48 tiles (c = 192: 42), all whole and like this: 0.85 to 1.01 over 1133 sizes, 0.93 in the mean (one at
// 1.08); 49 to 63 tiles, if they were taken so, 1.06 to 1.25.
enum SecondForm { kSecondChunk = 0, kSecondLarge = 1, kSecondSmall = 2 };
struct SecondPlan {
    SecondForm form;
    int64_t whole;   // tiles per XCD
    double us;       // its price
};
constexpr int kSmallList = 4096;   // entries of a list that fit LDS beside the ring of tiles of 64 x 64, two workgroups per CU
// Kernel times (whole, parts, small, large), us: delta, c = 192, 4 chunks x 249 of 5248 x 1408: 9.3, 5.6, 5.0, -; 9 x 395 of 7488 x 4864: 18,
// 19, 25, -; dense 509 x 4800 x 640: 52, 28, 20, 77; 536 x 2688 x 7808: 98, 57, 71, 148; 2990 x 2816 x 10 048: 216, 315, 390, 208.
static SecondPlan second_plan(bool sparse, int B, int N, int D, int F, int c, int k_stride) {
    static const Price whole_delta[2] = {{0.639, 9.19, 2.06, 0.54, 0.15, 0.89, 0.19}, {0.487, 7.22, 1.58, 0.52, 0.17, 0.84, 0.29}};   // c = 192, 128
    static const Price parts_delta[2] = {{0.321, 4.17, 1.41, 0.57, 0.18, 0.93, 0.12}, {0.328, 4.26, 1.52, 0.52, 0.19, 0.92, 0.11}};
    static const Price small_delta = {0.195, 2.78, 0.93, 0.57, 0.25, 1, 0.21};
    static const Price whole_dense[2] = {{0.697, 5.2, 3.82, 0.45, 0.16, 0.84, 0.2}, {0.546, 0.57, 5.74, 0.41, 0.15, 0.74, 0.2}};
    static const Price parts_dense[2] = {{0.359, 2.5, 2.16, 0.43, 0.12, 0.77, 0.24}, {0.359, 2.5, 1.47, 0.41, 0.17, 0.84, 0.2}};
    static const Price small_dense = {0.237, 2.5, 0, 0.42, 0.19, 0.94, 0.09};
    static const Price large_dense = {0.69, 6.9, 2.75, 0.65, 0.17, 0.81, 0.17};
    const int at = c == 192 ? 0 : 1, parts = c / 64;
    const int steps = sparse ? (k_stride + kGemm2K - 1) / kGemm2K : F / kGemm2K;
    const int64_t chunks = (int64_t)B * ((N + c - 1) / c), tiles = per_xcd(chunks * (D / kBN));
    const Price& whole = (sparse ? whole_delta : whole_dense)[at];
    const Price& part = (sparse ? parts_delta : parts_dense)[at];
    SecondPlan plan = {kSecondChunk, tiles, 0.};
    if (sparse && ((int64_t)k_stride + kBN - 1) / kBN * kBN * c * 2 >= 1LL << 32) return plan;   // whole chunks only: more bytes than the parts' offsets hold
    const int64_t beyond = tiles > 64 ? tiles % 64 : tiles - 32;
    double best;
    if (beyond > 0 && beyond * parts <= 32) {
        plan.whole = tiles - beyond;
        // (a part beside a whole tile costs about a third of what it takes alone)
        best = price(whole, plan.whole, 64, steps) + (tiles > 64 ? 1. : 0.35) * (price(part, beyond * parts, 64, steps) - part.call);
    } else {
        best = price(whole, tiles, 64, steps);
    }
    auto consider = [&](SecondPlan other, double us) {
        if (us < best) best = us, plan = other;
    };
    consider({kSecondChunk, 0, 0.}, price(part, tiles * parts, 64, steps));
    if (sparse) {
        const int64_t small_tiles = per_xcd(chunks * parts * (D / kSmallTile));
        if (small_launches(small_tiles) && (k_stride + kBN - 1) / kBN * kBN <= kSmallList)
            consider({kSecondSmall, 0, 0.}, price(small_delta, small_tiles, 64, steps));
    } else {
        const int64_t small_tiles = per_xcd((int64_t)B * ((N + kSmallTile - 1) / kSmallTile) * (D / kSmallTile));
        if (small_launches(small_tiles)) consider({kSecondSmall, 0, 0.}, price(small_dense, small_tiles, 64, steps));
        if (B <= 65535)
            consider({kSecondLarge, 0, 0.}, price(large_dense, B * per_xcd((int64_t)((N + kDenseTile - 1) / kDenseTile) * ((D + kDenseTile - 1) / kDenseTile)), 32, steps));
    }
    plan.us = best;
    return plan;
}

// The rows of a chunk's tile in the two GEMMs of a dense MLP, whose tiles need not follow the chunks: those of the other
// chunk size where the prices above say 6 % less, for the widths that models have (hidden wider than the model's).  In
// the second GEMM up to 4.5e10 products: beyond, the prices of its tiles of 192 and 128 rows are not that exact (1.01 of
// the time over 59 sizes).  In the first without a limit: 4.5e10 to 1.6e11 products 0.94 (1759 sizes, one lost more than
// 1 %).  Against the first GEMM's tiles of 64 x 64 13 % less: their price errs by more (7 to 13 % less by price: 0.98 of
// the time, of 825 sizes 221 lost more than 1 %, up to 16).
// Parts of 64 tokens whose rows in the cache are whole lines (a_ld a multiple of 64: 128 bytes) keep their rows: the price is that
// of rows that meet two lines, and they are up to a fifth quicker (830 tokens x 2688 x 5440, a_ld 832, second GEMM 45.1 us in
// parts, 52.3 on whole tiles of 128, priced 55.8 and 52.3; the change gave 0.97 of the time over 497 sizes, 119 of which lost
// more than 1 %, up to 9).
// Whole calls, of the time on the chunk's rows, 11 000 sizes of 5e8 to 3e11 products: 0.91 in the mean, both GEMMs on 128 rows
// instead of 192 0.84, the first 0.91, the second 0.93; on 192 instead of 128 the first 0.92, the second 0.94, both 0.84.
// One in 150 loses more than 2 %, 8 % at most: second GEMMs that go from parts of 64 rows to whole tiles of 128, with four to
// nine chunks whose last one has few rows.
constexpr double kOtherRows = 0.94, kOtherRowsThanSmall = 0.87;
struct DenseRows { int first, second; };
static DenseRows dense_rows(int B, int N, int D, int F, int c, int64_t a_ld) {
    const int other = 192 + 128 - c;
    DenseRows rows = {c, c};
    if (F <= D || D < 512) return rows;
    double us, other_us;
    const double less = first_form(false, B, N, D, F, c, 0, &us) == kFirstSmall ? kOtherRowsThanSmall : kOtherRows;
    if (first_form(false, B, N, D, F, other, 0, &other_us) == kFirstChunk && other_us < less * us) rows.first = other;
    if ((double)B * N * D * F < 4.5e10) {
        const SecondPlan plan = second_plan(false, B, N, D, F, c, 0), other_plan = second_plan(false, B, N, D, F, other, 0);
        const bool parts_of_lines = plan.form == kSecondChunk && plan.whole == 0 && a_ld % 64 == 0;
        if (!parts_of_lines && other_plan.form == kSecondChunk && other_plan.us < kOtherRows * plan.us) rows.second = other;
    }
    return rows;
}

template <int MODE, int BM = kDenseTile>
static int32_t launch_dense_gemm(DenseGemmParams p, int second_dim, hipStream_t s) {
    const int width = MODE == kFirst ? p.N : MODE == kSecond ? p.D : p.F, height = MODE == kFirst ? p.F : p.N;
    const int tile_q = MODE == kScores ? 128 : kDenseTile;
    p.tiles_p = (width + BM - 1) / BM;
    p.tiles_q = (height + tile_q - 1) / tile_q;
    // set at every launch: the attribute is kept per device (a flag remembered here would not be)
    if (hipFuncSetAttribute((const void*)mlp_dense_gemm_kernel<MODE, BM>, hipFuncAttributeMaxDynamicSharedMemorySize, kDenseLds) !=
        hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    const int per_xcd = (p.tiles_p * p.tiles_q + 7) / 8;
    hipLaunchKernelGGL((mlp_dense_gemm_kernel<MODE, BM>), dim3((unsigned)(per_xcd * 8), (unsigned)second_dim), dim3(512), kDenseLds, s, p);
    return launch_status();
}

template <int BM>
static int32_t launch_delta_gemm(DenseGemmParams p, hipStream_t s) {
    p.tiles_p = 1;
    p.tiles_q = (p.k_stride + kDenseTile - 1) / kDenseTile;
    constexpr int lds = 2 * kDenseStage;
    static_assert(kDenseTile * (BM * 2 + 16) <= lds, "the activations' tile fits the stages");
    if (hipFuncSetAttribute((const void*)mlp_dense_gemm_kernel<kDelta, BM>, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    hipLaunchKernelGGL((mlp_dense_gemm_kernel<kDelta, BM>), dim3((unsigned)xcd_grid_size(p.tiles_q, p.units)), dim3(512), lds, s, p);
    return launch_status();
}

static int round_up(int v, int m) { return (v + m - 1) / m * m; }

static int32_t check_mlp_shapes(int B, int N, int D, int F, int c) {
    if (B < 1 || N < 1 || D < 1 || F < 1) return CHIPMUNK_ERR_SHAPE;
    if (c != 128 && c != 192) return CHIPMUNK_ERR_UNSUPPORTED;
    if (D % 128 != 0 || F % 64 != 0) return CHIPMUNK_ERR_UNSUPPORTED;
    if ((int64_t)N * D * 2 >= (1LL << 32) || (int64_t)F * D * 2 >= (1LL << 32)) return CHIPMUNK_ERR_SHAPE;
    if ((int64_t)B * ((N + c - 1) / c) * ((F + kBN - 1) / kBN + D / kBN) > 0x3fffffffLL) return CHIPMUNK_ERR_SHAPE;
    return CHIPMUNK_OK;
}

}  // namespace chipmunk

using namespace chipmunk;

extern "C" size_t chipmunk_mlp_workspace_bytes(int B, int N, int D, int F, int c, int k_stride) {
    if (check_mlp_shapes(B, N, D, F, c) != CHIPMUNK_OK || k_stride < 0 || k_stride > F) return 0;
    int64_t units = (int64_t)B * ((N + c - 1) / c);
    return (size_t)(units * round_up(k_stride > 0 ? k_stride : 1, kBN) * c * 2);
}

// Pieces of the contraction that the workspace has room for: what workgroups of 128 neurons x 128 chunks over [hi | lo] would
// take to fill the GPU.  The plan below never takes more.
static int tile_mean_pieces(int units, int F) {
    int blocks = ((units + 127) / 128) * ((F + kBN - 1) / kBN);
    int pieces = 1;
    while (pieces < 16 && blocks * pieces < 768) pieces *= 2;
    return pieces;
}

// How the scores GEMM runs: into how many pieces its contraction is cut, and whether on the tiles of 128 neurons that add
// the high parts in two sums (mlp_dense.h) or on those of 256 that add them in one.
//   - Up to six contraction steps: one piece, two sums; a sum of pieces is a launch of its own, and 128 neurons fill more
//     CUs.  Whole calls in us on tiles of 256 in one piece, in pieces, and like this, D = 256: 8 chunks x 1024 neurons 12.3,
//     12.3, 10.6; 94 x 4096 14.6, 17.2, 11.6; 300 x 12 288 20.8, 32.9, 22.2; D = 384: 14.2, 12.3, 11.6; 16.5, 19.2, 12.6; 24.2,
//     36.5, 25.6; D = 128: 10.4, 11.6, 9.4; 13.1, 15.9, 10.6; 17.1, 30.3, 17.8.
//   - Otherwise as many pieces as let the tiles have a CU each.  Every XCD takes an eighth of the tiles, rounded up, so 32 CUs
//     over that: with 256 over the tiles, 20 tiles in 12 pieces were 36 workgroups on one XCD and a second round (12 chunks x
//     2688 x 4928: 24.5 us, in 10 pieces 19.3; 50 tiles: 28.3, 21.2).  Tiles of 128 where there are pieces and they fill
//     as many CUs: they leave half as many partial results (the same two sizes 16.8 and 20.1; 4 tiles of 256 34.4, 30.4; 60
//     34.3, 29.9).  48 tiles of 256, five pieces: 28.4 us; 240, one piece: 198.6.
//   - If the sums are then longer than is exact enough, half as many pieces as that takes, in two sums each (in one sum each,
//     twice the pieces: 156 tiles of D = 2688 172 us, like this 160; 70 tiles of D = 2048 99, 89).
// Exact enough: no larger an error than the sum of tile_mean_pieces() pieces over [hi | lo], half of them high parts.  Eight
// products are added with one rounding, whose error goes with the sum so far; in units of the variance that one
// rounding of the result has, a sum of n = D / 8 such additions cut into h chains leaves n / (2 h), adding the chains up h / 2,
// and each rounding at the size of the result 1.  (GEMM alone against 64 bits at 602 x 3072 x 12 288: 3.4e-7, by this count 3.4e-7.)
struct ScoresPlan {
    int pieces;
    bool two_sums;
};
static ScoresPlan scores_plan(int units, int D, int F) {
    const int steps = D / kBK;
    if (steps <= 6) return {1, true};
    auto fill = [&](int width) {   // pieces of tiles this wide
        const int tiles = ((F + width - 1) / width) * ((units + 127) / 128);
        return std::min(std::max(1, std::min(32 / ((tiles + 7) / 8), 16)), steps);
    };
    const int one = fill(kDenseTile), two = fill(128);
    const int chains = std::min(std::max(1, tile_mean_pieces(units, F) / 2), steps);
    const double additions = D / 8, allowed = additions / (2 * chains) + 1.5 * chains;
    const bool one_is_exact = additions / (2 * one) + 0.5 * (one + 1) <= allowed;
    const bool two_is_exact = additions / (4 * two) + 0.5 * (two + 3) <= allowed;
    if (one > 1 && 2 * two >= one && two_is_exact) return {two, true};
    if (one_is_exact) return {one, false};
    return {two_is_exact ? two : std::max(1, chains / 2), true};
}

// Chunk means by workgroups of 128 columns where those of 512 leave most of the CUs without one.  Whole calls in us, 512
// and 128 columns: 8 chunks of 192 x 3072 (F = 4096) 13.3, 12.0; 24 x 1024 (12 288) 14.3, 13.1; beyond the limit 60 x
// 2048 (4096) 25.9, 26.2; 108 x 512 (3136) 17.4, 18.3.
static bool narrow_means(int units, int D) { return (D + 511) / 512 * units <= 96; }

// Few chunks: a workgroup per 16, 32 or 64 neurons, up to 16 384 neurons the fewest that give every CU at most one, with
// all chunks.  Every workgroup reads all means (4 D bytes a chunk), which is what sets the limits of units * D; just
// above 8192 neurons the workgroups are fewest and read most.  Whole calls in us, with the tiles of mlp_dense.h (and the
// sum of their pieces) and with these: 3 chunks x 512 x 2048 neurons 12.0, 8.8; 8 x 1024 x 4096 13.3, 8.7; 8 x 3072 x
// 12 288 28.0, 20.8; 16 x 3072 x 8192 24.2, 18.3; 24 x 1024 x 12 288 19.8, 13.1; 24 x 3072 x 12 288 32.3, 28.8; 40 x 1408
// x 4096 16.0, 14.4.
// The limits by 1863 sizes, W1 not in the caches, of the time with the tiles (few chunks to many):
//     F = 64: 24 000 0.81 to 1.01, 30 000 up to 1.03 (D = 3712);   512: 41 000 0.84 to 0.99, 46 000 up to 1.02;
//     1536: 41 000 0.81 to 0.96; below 2048 neurons with D above 4608 1.0 to 1.4 (a long contraction in a few
//     workgroups);
//     4160: 57 000 0.94 to 1.00 (D above F up to 1.03), 66 000 1.01 to 1.14;   8256: 41 000 0.76 to 0.98, 50 000 up to 1.05;
//     11 328 to 16 384: 74 000 0.75 to 0.97, 90 000 up to 1.02.
// Beyond 16 384 neurons some CUs have more than one workgroup, each with all means: up to 16 chunks 0.71 to 0.97, 24 up
// to 1.15, 48 up to 1.47 (131 072 neurons).
static int few_neuron_blocks(int F) { return F <= 16 * 256 ? 1 : F <= 32 * 256 ? 2 : 4; }
static bool few_scores(int units, int D, int F) {
    if (units > (F <= 64 * 256 ? 48 : 16) || (F < 2048 && D > 4608)) return false;
    const int64_t limit = F < 256 ? 24576 : F < 2048 ? 40960 : F <= 32 * 256 ? 57344 : F <= 44 * 256 ? 40960 : 73728;
    return (int64_t)units * D <= limit;
}

// Workspace of the token-merged pre-activation with the contraction cut in `pieces`: the chunk means in split
// precision [units, 2 D] bf16 (rounded up to 256 bytes), then, with more than one piece, the pieces' partial
// results [pieces, units, F] fp32.  0 when the shapes are out of range.
static size_t tile_mean_bytes(int B, int N, int D, int F, int c, int pieces) {
    if (check_mlp_shapes(B, N, D, F, c) != CHIPMUNK_OK) return 0;
    const int64_t units = (int64_t)B * ((N + c - 1) / c);
    if (units > 0x7fffff || units * 2 * D * 2 >= (1LL << 32)) return 0;
    const size_t means = ((size_t)units * 2 * D * 2 + 255) / 256 * 256;
    return means + (pieces > 1 ? (size_t)pieces * units * F * sizeof(float) : 0);
}

extern "C" size_t chipmunk_mlp_tile_mean_workspace_bytes(int B, int N, int D, int F, int c) {
    if (check_mlp_shapes(B, N, D, F, c) != CHIPMUNK_OK) return 0;
    const int64_t units = (int64_t)B * ((N + c - 1) / c);
    if (units > 0x7fffff) return 0;
    return tile_mean_bytes(B, N, D, F, c, tile_mean_pieces((int)units, F));
}

// The column-sparse delta MLP; `deferred`: the activation-cache write-back runs in the second GEMM's launch
// (workspace: delta^T, then the new activations in the same layout).
static int32_t run_mlp_sparse_delta(const uint16_t* x, const uint16_t* w1, const uint16_t* b1, const uint16_t* w2,
                                    const int32_t* idx, const int32_t* counts, uint16_t* a_cache, int64_t a_ld,
                                    uint16_t* o_cache, int B, int N, int D, int F, int c, int k_stride, int act,
                                    void* ws, size_t ws_bytes, void* stream, bool deferred) {
    if (!x || !w1 || !w2 || !idx || !counts || !a_cache || !o_cache) return CHIPMUNK_ERR_NULL;
    int32_t st = check_mlp_shapes(B, N, D, F, c);
    if (st != CHIPMUNK_OK) return st;
    if (k_stride < 0 || k_stride > F || a_ld < N) return CHIPMUNK_ERR_SHAPE;
    if (act != CHIPMUNK_ACT_GELU_ERF && act != CHIPMUNK_ACT_GELU_TANH) return CHIPMUNK_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(w1) || !aligned16(w2) || !aligned16(a_cache) || !aligned16(o_cache) ||
        !aligned16(idx) || !aligned16(counts) || !aligned16(ws) || (reinterpret_cast<uintptr_t>(b1) & 1u) ||
        (a_ld % 8) != 0)
        return CHIPMUNK_ERR_ALIGN;
    if (k_stride == 0) return CHIPMUNK_OK;
    const size_t delta_bytes = chipmunk_mlp_workspace_bytes(B, N, D, F, c, k_stride);
    const size_t need = deferred ? 2 * delta_bytes : delta_bytes;
    if (!ws || ws_bytes < need) return CHIPMUNK_ERR_WORKSPACE;
    const int NB = (N + c - 1) / c, units = B * NB;
    const int k_pad = round_up(k_stride, kBN);
    hipStream_t s = (hipStream_t)stream;
    uint16_t* act_t = deferred ? (uint16_t*)((char*)ws + delta_bytes) : nullptr;

    Gemm1Params g1;
    g1.x = x; g1.w1 = w1; g1.b1 = b1; g1.idx = idx; g1.counts = counts; g1.a_cache = a_cache;
    g1.delta_t = (uint16_t*)ws; g1.act_t = act_t; g1.a_ld = a_ld;
    g1.N = N; g1.NB = NB; g1.D = D; g1.F = F;
    g1.k_stride = k_stride; g1.k_pad = k_pad; g1.act = act;
    g1.parts = c / kSmallTile;
    const FirstForm first = first_form(true, B, N, D, F, c, k_stride);
    if (first == kFirstSmall) {
        st = launch_small_gemm1<kSparseDelta>(g1, units, s);
    } else if (first == kFirstLarge) {
        DenseGemmParams g;
        g.x = x; g.w1 = w1; g.w2 = nullptr; g.bias = b1; g.a_cache = a_cache; g.out = nullptr; g.scores = nullptr; g.a_ld = a_ld;
        g.N = N; g.D = D; g.F = F; g.act = act; g.pieces = 1;
        g.idx = idx; g.counts = counts; g.delta_t = (uint16_t*)ws; g.act_t = act_t;
        g.NB = NB; g.k_stride = k_stride; g.k_pad = k_pad; g.units = units;
        st = c == 192 ? launch_delta_gemm<192>(g, s) : launch_delta_gemm<128>(g, s);
    } else {
        st = c == 192 ? launch_gemm1<192, kSparseDelta>(g1, k_pad / kBN, units, s)
                      : launch_gemm1<128, kSparseDelta>(g1, k_pad / kBN, units, s);
    }
    if (st != CHIPMUNK_OK) return st;

    Gemm2Params g2;
    g2.a_t = (const uint16_t*)ws; g2.w2 = w2; g2.bias = nullptr; g2.idx = idx; g2.counts = counts; g2.o = o_cache;
    g2.a_ld = a_ld; g2.N = N; g2.NB = NB; g2.D = D; g2.F = F; g2.k_stride = k_stride; g2.k_pad = k_pad;
    g2.act_t = act_t; g2.a_cache = a_cache; g2.parts = c / kSmallTile;
    const SecondPlan second = second_plan(true, B, N, D, F, c, k_stride);
    if (second.form == kSecondSmall) return launch_small_gemm2<true>(g2, units, s);
    return c == 192 ? launch_gemm2<192, false>(g2, D / kBN, units, second.whole, s) : launch_gemm2<128, false>(g2, D / kBN, units, second.whole, s);
}

extern "C" int32_t chipmunk_mlp_sparse_delta(const uint16_t* x, const uint16_t* w1, const uint16_t* b1,
                                             const uint16_t* w2, const int32_t* idx, const int32_t* counts,
                                             uint16_t* a_cache, int64_t a_ld, uint16_t* o_cache, int B, int N,
                                             int D, int F, int c, int k_stride, int act, void* ws,
                                             size_t ws_bytes, void* stream) {
    return run_mlp_sparse_delta(x, w1, b1, w2, idx, counts, a_cache, a_ld, o_cache, B, N, D, F, c, k_stride, act, ws,
                                ws_bytes, stream, false);
}

extern "C" size_t chipmunk_mlp_overlapped_workspace_bytes(int B, int N, int D, int F, int c, int k_stride) {
    return 2 * chipmunk_mlp_workspace_bytes(B, N, D, F, c, k_stride);
}

extern "C" int32_t chipmunk_mlp_sparse_delta_overlapped(const uint16_t* x, const uint16_t* w1, const uint16_t* b1,
                                                        const uint16_t* w2, const int32_t* idx,
                                                        const int32_t* counts, uint16_t* a_cache, int64_t a_ld,
                                                        uint16_t* o_cache, int B, int N, int D, int F, int c,
                                                        int k_stride, int act, void* ws, size_t ws_bytes,
                                                        void* stream) {
    return run_mlp_sparse_delta(x, w1, b1, w2, idx, counts, a_cache, a_ld, o_cache, B, N, D, F, c, k_stride, act, ws,
                                ws_bytes, stream, true);
}

extern "C" int32_t chipmunk_mlp_dense(const uint16_t* x, const uint16_t* w1, const uint16_t* b1,
                                      const uint16_t* w2, const uint16_t* b2, uint16_t* out, uint16_t* a_cache,
                                      int64_t a_ld, int B, int N, int D, int F, int c, int act, void* stream) {
    if (!x || !w1 || !w2 || !out || !a_cache) return CHIPMUNK_ERR_NULL;
    int32_t st = check_mlp_shapes(B, N, D, F, c);
    if (st != CHIPMUNK_OK) return st;
    if (a_ld < N) return CHIPMUNK_ERR_SHAPE;
    if ((int64_t)F * a_ld * 2 >= (1LL << 32)) return CHIPMUNK_ERR_SHAPE;
    if (act != CHIPMUNK_ACT_GELU_ERF && act != CHIPMUNK_ACT_GELU_TANH) return CHIPMUNK_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(w1) || !aligned16(w2) || !aligned16(a_cache) || !aligned16(out) ||
        (reinterpret_cast<uintptr_t>(b1) & 1u) || (reinterpret_cast<uintptr_t>(b2) & 7u) || (a_ld % 8) != 0)
        return CHIPMUNK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    DenseGemmParams g;
    g.x = x; g.w1 = w1; g.w2 = w2; g.a_cache = a_cache; g.out = out; g.a_ld = a_ld;
    g.scores = nullptr; g.N = N; g.D = D; g.F = F; g.act = act; g.pieces = 1;

    const DenseRows rows = dense_rows(B, N, D, F, c, a_ld);
    const FirstForm first = first_form(false, B, N, D, F, rows.first, 0);
    const SecondPlan second = second_plan(false, B, N, D, F, rows.second, 0);
    const int row_tiles = (N + kSmallTile - 1) / kSmallTile;   // of 64 x 64
    if (first == kFirstLarge) {
        g.bias = b1;
        st = launch_dense_gemm<kFirst>(g, B, s);
    } else {
        Gemm1Params g1;
        g1.x = x; g1.w1 = w1; g1.b1 = b1; g1.idx = nullptr; g1.counts = nullptr; g1.a_cache = a_cache;
        g1.delta_t = nullptr; g1.act_t = nullptr; g1.a_ld = a_ld;
        g1.N = N; g1.NB = (N + rows.first - 1) / rows.first; g1.D = D; g1.F = F;
        g1.k_stride = F; g1.k_pad = F; g1.act = act; g1.parts = 1;
        if (first == kFirstSmall) {
            g1.NB = row_tiles;
            st = launch_small_gemm1<kDenseAct>(g1, B * row_tiles, s);
        } else {
            st = rows.first == 192 ? launch_gemm1<192, kDenseAct>(g1, (F + kBN - 1) / kBN, B * g1.NB, s)
                                   : launch_gemm1<128, kDenseAct>(g1, (F + kBN - 1) / kBN, B * g1.NB, s);
        }
    }
    if (st != CHIPMUNK_OK) return st;
    if (second.form == kSecondLarge) {
        g.bias = b2;
        return launch_dense_gemm<kSecond>(g, B, s);
    }
    Gemm2Params g2;
    g2.a_t = a_cache; g2.w2 = w2; g2.bias = b2; g2.idx = nullptr; g2.counts = nullptr; g2.o = out;
    g2.a_ld = a_ld; g2.N = N; g2.NB = (N + rows.second - 1) / rows.second; g2.D = D; g2.F = F; g2.k_stride = F; g2.k_pad = F;
    g2.act_t = nullptr; g2.a_cache = nullptr; g2.parts = 1;
    if (second.form == kSecondSmall) {
        g2.NB = row_tiles;
        return launch_small_gemm2<false>(g2, B * row_tiles, s);
    }
    return rows.second == 192 ? launch_gemm2<192, true>(g2, D / kBN, B * g2.NB, second.whole, s)
                              : launch_gemm2<128, true>(g2, D / kBN, B * g2.NB, second.whole, s);
}

// chunk means -> scores GEMM (-> sum of the pieces); ws holds tile_mean_bytes(..., pieces) bytes
static int32_t run_tile_mean(const uint16_t* x, const uint16_t* w1, float* T, int B, int N, int D, int F, int c,
                             void* ws, int pieces, hipStream_t s) {
    const int NB = (N + c - 1) / c, units = B * NB;
    const bool stream_x = (int64_t)B * N * D * 2 > kLastLevelCache;
    const bool narrow = !stream_x && narrow_means(units, D);
    hipLaunchKernelGGL((stream_x ? chunk_mean_kernel<true, 64> : narrow ? chunk_mean_kernel<false, 16> : chunk_mean_kernel<false, 64>),
                       dim3((unsigned)((narrow ? D / 128 : (D / 8 + 63) / 64) * units)), dim3(64 * kMeanWaves), 0, s, x, (uint16_t*)ws, N, NB, D, c);
    if (launch_status() != CHIPMUNK_OK) return CHIPMUNK_ERR_LAUNCH;
    // scores[unit, f] = <hi(unit) + lo(unit), w1_f>
    if (few_scores(units, D, F)) {
        const int blocks = few_neuron_blocks(F);
        auto launch = [&](auto kernel) {
            const int lds = kFewWaves * blocks * ((units + 15) / 16) * 1024;
            if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return (int32_t)CHIPMUNK_ERR_LAUNCH;
            hipLaunchKernelGGL(kernel, dim3((unsigned)(F / (16 * blocks))), dim3(64 * kFewWaves), lds, s, (const uint16_t*)ws, w1, T, units, D, F);
            return launch_status();
        };
        if (units <= 16) return launch(blocks == 1 ? mlp_few_scores_kernel<1, 1> : blocks == 2 ? mlp_few_scores_kernel<1, 2> : mlp_few_scores_kernel<1, 4>);
        if (units <= 32) return launch(blocks == 1 ? mlp_few_scores_kernel<2, 1> : blocks == 2 ? mlp_few_scores_kernel<2, 2> : mlp_few_scores_kernel<2, 4>);
        return launch(blocks == 1 ? mlp_few_scores_kernel<3, 1> : blocks == 2 ? mlp_few_scores_kernel<3, 2> : mlp_few_scores_kernel<3, 4>);
    }
    const ScoresPlan plan = scores_plan(units, D, F);
    pieces = std::min(pieces, plan.pieces);
    size_t means = ((size_t)units * 2 * D * 2 + 255) / 256 * 256;
    float* partial = pieces > 1 ? (float*)((char*)ws + means) : T;
    DenseGemmParams g;
    g.x = (const uint16_t*)ws; g.w1 = w1; g.w2 = nullptr; g.bias = nullptr; g.a_cache = nullptr; g.out = nullptr; g.a_ld = 0;
    g.scores = partial; g.N = units; g.D = D; g.F = F; g.act = 0; g.pieces = pieces;
    int32_t st = plan.two_sums ? launch_dense_gemm<kScores, 128>(g, pieces, s) : launch_dense_gemm<kScores>(g, pieces, s);
    if (st != CHIPMUNK_OK || pieces == 1) return st;
    int64_t n4 = (int64_t)units * F / 4;
    hipLaunchKernelGGL(sum_pieces_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, partial, T, n4, pieces);
    return launch_status();
}

extern "C" int32_t chipmunk_mlp_tile_mean_preact(const uint16_t* x, const uint16_t* w1, float* T, int B, int N,
                                                 int D, int F, int c, void* ws, size_t ws_bytes, void* stream) {
    if (!x || !w1 || !T) return CHIPMUNK_ERR_NULL;
    int32_t st = check_mlp_shapes(B, N, D, F, c);
    if (st != CHIPMUNK_OK) return st;
    if (!aligned16(x) || !aligned16(w1) || !aligned16(T) || !aligned16(ws)) return CHIPMUNK_ERR_ALIGN;
    const int64_t units = (int64_t)B * ((N + c - 1) / c);
    if (units > 0x7fffff || units * 2 * D * 2 >= (1LL << 32)) return CHIPMUNK_ERR_SHAPE;
    const int pieces = tile_mean_pieces((int)units, F);
    size_t need = tile_mean_bytes(B, N, D, F, c, pieces);
    if (!ws || need == 0 || ws_bytes < need) return CHIPMUNK_ERR_WORKSPACE;
    return run_tile_mean(x, w1, T, B, N, D, F, c, ws, pieces, (hipStream_t)stream);
}

// ---- the token-merged pre-activation for callers that cannot allocate ---------------------------------------
// Same kernels as chipmunk_mlp_tile_mean_preact; the workspace is a fixed array in device memory that belongs to
// the library.  Each GPU the library runs on holds its own copy at its own address: the address is looked up once
// per device (with that device current) and kept; host code passes that address, never the array's name, to the
// kernels.
namespace chipmunk {

constexpr size_t kStaticScratchBytes = 32u << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

static std::mutex scratch_mutex;
static void* scratch_address[kMaxDevices];   // per device, 0 until looked up

static int32_t scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CHIPMUNK_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_address[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return CHIPMUNK_ERR_LAUNCH;
        scratch_address[dev] = ptr;
    }
    *out = scratch_address[dev];
    return CHIPMUNK_OK;
}

}  // namespace chipmunk

extern "C" size_t chipmunk_mlp_tile_mean_preact_static_capacity(void) { return kStaticScratchBytes; }

extern "C" int32_t chipmunk_mlp_tile_mean_preact_static(const uint16_t* x, const uint16_t* w1, float* T, int B, int N,
                                                        int D, int F, int c, void* stream) {
    if (!x || !w1 || !T) return CHIPMUNK_ERR_NULL;
    int32_t st = check_mlp_shapes(B, N, D, F, c);
    if (st != CHIPMUNK_OK) return st;
    if (!aligned16(x) || !aligned16(w1) || !aligned16(T)) return CHIPMUNK_ERR_ALIGN;
    const int64_t units = (int64_t)B * ((N + c - 1) / c);
    if (units > 0x7fffff || units * 2 * D * 2 >= (1LL << 32)) return CHIPMUNK_ERR_SHAPE;
    // as many pieces of the contraction as the general entry point uses, or as many as fit the array beside the chunk
    // means; with one piece the scores go straight to T
    int pieces = scores_plan((int)units, D, F).pieces;
    while (pieces > 1 && tile_mean_bytes(B, N, D, F, c, pieces) > kStaticScratchBytes) pieces--;
    const size_t need = tile_mean_bytes(B, N, D, F, c, pieces);
    if (need == 0 || need > kStaticScratchBytes) return CHIPMUNK_ERR_WORKSPACE;   // the chunk means alone do not fit
    void* ws = nullptr;
    st = scratch_of_current_device(&ws);
    if (st != CHIPMUNK_OK) return st;
    // every byte of the array that the kernels read in this call is written by this call first (the chunk means
    // by chunk_mean_kernel, every piece's partial scores by the scores GEMM): nothing has to start at zero
    return run_tile_mean(x, w1, T, B, N, D, F, c, ws, pieces, (hipStream_t)stream);
}

// What the rules above choose for these sizes: whether the two dense GEMMs take the tiles of 256 x 256, whether the delta
// takes 256 neurons per workgroup, and the scores GEMM's pieces and sums (0 and 0: the kernel for few chunks).  Not part
// of the library's interface: for the tests, which have to reach each form and otherwise would not see that a rule has
// moved.
extern "C" void chipmunk_internal_mlp_form(int B, int N, int D, int F, int c, int k_stride, int a_ld, int32_t* out) {
    const int units = B * ((N + c - 1) / c);
    const ScoresPlan plan = few_scores(units, D, F) ? ScoresPlan{0, false} : scores_plan(units, D, F);
    const DenseRows rows = dense_rows(B, N, D, F, c, a_ld);
    out[0] = first_form(false, B, N, D, F, rows.first, 0) == kFirstLarge;
    out[1] = second_plan(false, B, N, D, F, rows.second, 0).form == kSecondLarge;
    out[2] = first_form(true, B, N, D, F, c, k_stride) == kFirstLarge;
    out[3] = plan.pieces;
    out[4] = plan.pieces == 0 ? 0 : plan.two_sums ? 2 : 1;
}

// The same for every form of the GEMMs: the dense MLP's first (FirstForm) and second (SecondForm, and the tiles per XCD taken
// whole), then the delta's.
extern "C" void chipmunk_internal_mlp_tiles(int B, int N, int D, int F, int c, int k_stride, int a_ld, int64_t* out) {
    for (int sparse = 0; sparse < 2; sparse++) {
        const DenseRows rows = sparse ? DenseRows{c, c} : dense_rows(B, N, D, F, c, a_ld);
        const SecondPlan plan = second_plan(sparse, B, N, D, F, rows.second, k_stride);
        out[3 * sparse] = first_form(sparse, B, N, D, F, rows.first, k_stride);
        out[3 * sparse + 1] = plan.form;
        out[3 * sparse + 2] = plan.whole;
    }
}

// the rows of a chunk's tile in the dense MLP's GEMMs
extern "C" void chipmunk_internal_mlp_dense_rows(int B, int N, int D, int F, int c, int a_ld, int32_t* out) {
    const DenseRows rows = dense_rows(B, N, D, F, c, a_ld);
    out[0] = rows.first;
    out[1] = rows.second;
}

// whether a delta with these sizes has its cached output pass the caches by
extern "C" int32_t chipmunk_internal_mlp_streams(int B, int N, int D, int c) { return stream_output((int64_t)B * ((N + c - 1) / c), c, D); }

// how the scores of these sizes are made: 16-neuron blocks of a workgroup where the chunks are few, else 0; whether the
// means come in workgroups of 128 columns
extern "C" void chipmunk_internal_scores_form(int B, int N, int D, int F, int c, int32_t* out) {
    const int units = B * ((N + c - 1) / c);
    out[0] = few_scores(units, D, F) ? few_neuron_blocks(F) : 0;
    out[1] = (int64_t)B * N * D * 2 <= kLastLevelCache && narrow_means(units, D);
}
