// Column-sparse delta attention for gfx950 (Sec. 3.3.1 "Sparse Delta Steps",
// Alg. 3), and dense attention as the special case "every column selected".
//
// One workgroup (4 waves) owns one chunk of c query rows of one (batch, head).
// It walks the chunk's selected key columns in tiles of 32: the K and V rows
// named by the index list are gathered from global memory straight into LDS
// (16-byte asynchronous loads, one K or V row = E*2 contiguous bytes), two
// tiles per workgroup barrier and double buffered: the two tiles of the next
// step are in flight while the two of this step are consumed by bf16 MFMA
// 16x16x32 with an fp32 online softmax.  Two workgroups share a compute unit
// (two waves per SIMD): a wave hides nothing behind its own MFMAs, the other
// wave's vector and LDS instructions are what runs in their shadow.
//
// Register-level layout.  Scores are produced transposed, S^T = K Q^T, so a
// lane holds, for ONE query (lane % 16), the scores of 4 key rows per 16-row
// block (rows 4*(lane/16)+0..3).  Two such blocks are exactly the 8 contraction
// entries the lane must supply as the B operand of O^T += V^T P^T, so the
// probabilities go from the softmax into the second MFMA without leaving
// registers.  V^T tiles come from LDS through the transposing 64-bit read.
// Each wave owns NQB blocks of 16 queries (c = 64*NQB).
#include "common.h"

#include <type_traits>

namespace chipmunk {

struct AttnParams {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const uint16_t* base;
    uint16_t* out;
    const int32_t* idx;
    const int32_t* counts;
    float* row_m;   // optional [B,H,N]: the reference the row's exponentials were taken against, in units of the
                    // scaled scores (natural logarithm); within 2^8 of the row maximum, not necessarily equal to it
    float* row_l;   // optional [B,H,N]: sum_j exp(score_j - row_m)
    int N, NB, c, k_stride;
    int whole;      // the first so many chunks have a workgroup each, the others are walked in parts (attn_part_form)
    int by_xcd;     // see attn_run_of_xcd
    float sl2;      // softmax_scale * log2(e)
    float o_scale;
    // fused column sums with given normalisers (Alg. 4): dense launches of the FUSED kernel only
    const float* prev_m;   // [B,H,N], natural-log units like row_m
    const float* prev_l;   // [B,H,N]
    float* colsum;         // [B,H,NB,ld_colsum]
    int64_t ld_colsum;
    int first = 0;         // every column: the launch's first chunk
};

constexpr int kTileRows = 32;         // key rows per LDS tile = one step of the online softmax
constexpr int kTilesPerStep = 2;      // tiles consumed between two workgroup barriers
constexpr int kStages = 2 * kTilesPerStep;  // tile buffers (K tile + V tile each): one step in use, one in flight
constexpr int kColsumTileRows = 64;   // the column-sum kernel keeps 64-row tiles, double buffered
constexpr float kRescaleSlack = 8.f;  // running max may lag the true max by 2^8 before a rescale

// XOR swizzle of the 16-byte chunk position inside a row of the LDS tile
template <int E>
__device__ __forceinline__ int swizzle(int row) {
    return E == 128 ? swizzle_rows16(row) : (row >> 1) & 7;
}

template <int E, int NQB>
struct AttnState {
    f32x4 O[E / 16][NQB];
    f32x4 L[NQB];     // softmax denominator, accumulated by the MFMA against a row of ones
    bf16x8 Q[E / 32][NQB];
    f32x4 negm[NQB];  // -m in all four registers (m: the running reference max, in units of the raw scores <q,k>; it
                      // is replaced by the first tile's row maximum): the C operand that starts every score accumulation
};

// The work on one tile of 32 selected key rows is split in three pieces so that
// the kernel can software-pipeline them: scores of tile t+1 (MFMA) are issued
// next to the exponentials of tile t (VALU), and the max bookkeeping of tile t+1
// (VALU) next to the P.V products of tile t (MFMA).

// S^T = K Q^T - m for one tile: raw scores relative to the reference max (the MFMA adds -m for free where a
// separate subtraction would cost one vector instruction per score).  kaddr[es]: the lane's read address for
// contraction slice es in tile buffer 0; tile_off: byte offset of the tile buffer (compile-time at the call).
// between(j), j = 0 .. E/16 - 1, is called after the j-th group of NQB products: the kernel issues one of the next
// step's tile transfers there, so that the transfers are spread over the products instead of queueing up in one
// burst during which the wave issues nothing else.
// K operands are requested KPF groups ahead of the products that consume them.  One group ahead is enough: the
// other wave of the SIMD covers what latency is left, and deeper prefetch only costs registers (measured equal
// for the column-sparse launch, 2 % slower for the dense one)
template <int E, int NQB, int KPF, typename Between>
__device__ __forceinline__ void attn_scores(f32x4 (&S)[2][NQB], const AttnState<E, NQB>& st, const uint32_t (&kaddr)[E / 32],
                                            int tile_off, Between&& between) {
    constexpr int ROWB = E * 2;
    constexpr int NG = E / 16;   // groups of NQB products: group j = contraction slice j / 2, key rows 16 (j % 2) ..
    bf16x8 kop[NG];
#pragma unroll
    for (int j = 0; j < KPF; j++) kop[j] = lds_read_b128(kaddr[j / 2] + tile_off + (j % 2) * 16 * ROWB);
    __builtin_amdgcn_sched_group_barrier(0x100, KPF, 0);  // the LDS reads lead the block
#pragma unroll
    for (int j = 0; j < NG; j++) {
        const int es = j / 2, u = j % 2;
        if (j + KPF < NG) {
            const int jn = j + KPF;
            kop[jn] = lds_read_b128(kaddr[jn / 2] + tile_off + (jn % 2) * 16 * ROWB);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int qb = 0; qb < NQB; qb++)
            S[u][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[j], st.Q[es][qb], es == 0 ? st.negm[qb] : S[u][qb], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NQB, 0);
        between(j);
    }
}

// Inside a step (kTilesPerStep tiles) the rows of the LDS tiles are a fixed permutation of the step's list
// positions: every lane of the gather fetches kTilesPerStep * NI consecutive positions (one vector load of column
// numbers) and deals them out over the tiles.  Row q of tile s holds list position  step_base + list_pos(s, q).
// The softmax does not care about the order; only the mask of the unit's last tiles and the column sums do.
template <int E>
__device__ __forceinline__ int list_pos_in_step(int s, int q) {
    constexpr int NI = E / 64;                       // gather loads per wave, tile and matrix
    constexpr int LANEROWS = kTileRows / NI;         // rows of a tile that one such load of every wave covers
    return (q % LANEROWS) * (kTilesPerStep * NI) + s * NI + q / LANEROWS;
}

// The last tiles of a unit: rows whose list position is at or beyond `count` score -inf.  IN_ORDER: the rows of the step's
// tiles are its positions in order (the last step of a column list).
template <int E, int NQB, bool IN_ORDER = false>
__device__ __forceinline__ void attn_mask_tail(f32x4 (&S)[2][NQB], int step_base, int s, int count, int g) {
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int row = u * 16 + 4 * g + r;
            bool dead = step_base + (IN_ORDER ? s * kTileRows + row : list_pos_in_step<E>(s, row)) >= count;
#pragma unroll
            for (int qb = 0; qb < NQB; qb++)
                if (dead) S[u][qb][r] = -INFINITY;
        }
}

// Raise the reference max where this tile's relative scores exceed the slack
// (2^8 in probability, given here in raw score units); O, the denominator and the
// tile's relative scores are rescaled (rare after the first tiles).  The common
// case costs a lane only the max over its own 8 scores per query block: the reduction over the four lanes that share a query runs when some
// lane of the wave has seen an excess.  The first tile of a unit sets the
// reference to the tile's row maximum, whatever its sign.
template <int E, int NQB>
__device__ __forceinline__ void attn_update_max(AttnState<E, NQB>& st, f32x4 (&S)[2][NQB], bool first, float sl2,
                                                float slack) {
    float mx[NQB];
    bool need = first;
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
        float a = fmaxf(fmaxf(S[0][qb][0], S[0][qb][1]), S[0][qb][2]);
        float b = fmaxf(fmaxf(a, S[0][qb][3]), S[1][qb][0]);
        float c = fmaxf(fmaxf(b, S[1][qb][1]), S[1][qb][2]);
        mx[qb] = fmaxf(c, S[1][qb][3]);
        need |= mx[qb] > slack;
    }
    if (__builtin_amdgcn_ballot_w64(need) != 0) {
#pragma unroll
        for (int qb = 0; qb < NQB; qb++) {
            float d = rows4_max(mx[qb]);             // the tile's row maximum relative to the reference
            float up = first ? d : fmaxf(d, 0.f);    // the reference only rises, except when it is first set
            float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-up * sl2);   // O and L are still zero on the first tile
            const float nm = st.negm[qb][0] - up;
            st.negm[qb] = f32x4{nm, nm, nm, nm};
            st.L[qb] *= alpha;
#pragma unroll
            for (int eb = 0; eb < E / 16; eb++) st.O[eb][qb] *= alpha;
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int r = 0; r < 4; r++) S[u][qb][r] -= up;
        }
    }
}

// P = exp2(S*sl2) in bf16, the denominator, and O^T += V^T P^T.
// The transposing V reads do not depend on the probabilities: the first kVPrefetch
// operands are requested before the exponentials, the rest kVPrefetch steps ahead
// of the MFMAs that consume them, so LDS latency stays off the MFMA chain.
constexpr int kVPrefetch = 2;        // (1 in the kernel with the column sums)

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {  // x of the lane that the DPP control CTRL names
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}

// acc[4 u + r] is the lane's value for tile key row 16 u + 4 g + r.  Sums each of the eight over the 16 lanes of
// the row (the wave's 16 queries of a block) and writes them to part[32] in tile key order.  Halving exchange:
// at each step a lane keeps half of its values and hands the other half to a partner that keeps those, so 8 adds
// stand in for 32.  Partners: lane ^ 15, ^ 7, ^ 3, ^ 1; the value a lane ends with is 4 bit3 + 2 bit2 + bit1.
// In the first two steps the lanes that keep the other half are whole banks of four, so a second add with a bank mask takes
// the place of the two selects: 16 instructions instead of 22 (40 heads x 18 000 with column sums 5673 -> 5602 us, the same
// sums).  A DPP operand must not have been written by the two instructions before: the order below keeps them apart, and the nop
// what the compiler puts in front, because it does not look inside.
__device__ __forceinline__ void row16_sums_to_lds(float (&x)[8], float* part, int g, int l16) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %4, %4 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %5, %5 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %6, %6 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %7, %7 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "+&v"(x[0]), "+&v"(x[1]), "+&v"(x[2]), "+&v"(x[3])   // written before the others are read
        : "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
    const bool b1 = l16 & 2;
    float z = (b1 ? x[1] : x[0]) + dpp_f32<0x1b>(b1 ? x[0] : x[1]);   // quad_perm 3,2,1,0
    z += dpp_f32<0xb1>(z);                                             // quad_perm 1,0,3,2
    if (!(l16 & 1)) part[(l16 & 8 ? 16 : 0) + 4 * g + ((l16 >> 1) & 3)] = z;
}

// COLSUM (Alg. 4): also the tile's column sums with given normalisers.  The weight of (key, query) there is
// exp2(score * sl2 - prev_m2) / prev_l = p * wq, with p the probability formed here against the running
// reference st.m and wq = exp2(st.m * sl2 + off) per query, off = -prev_m2 - log2(prev_l) (-inf: no such query).
template <int E, int NQB, bool COLSUM = false, int VPF = kVPrefetch>
__device__ __forceinline__ void attn_weights_and_pv(AttnState<E, NQB>& st, const f32x4 (&S)[2][NQB],
                                                    const uint32_t (&vaddr)[E / 16], int tile_off, float sl2, bf16x8 ones,
                                                    const float* off = nullptr, float* part = nullptr, int g = 0,
                                                    int l16 = 0) {
    constexpr int ROWB = E * 2;
    constexpr int NEB = E / 16;
    typedef __attribute__((ext_vector_type(8))) short short8v;
    short4v vlo[NEB], vhi[NEB];
#pragma unroll
    for (int eb = 0; eb < VPF; eb++) {
        vlo[eb] = lds_read_tr16_at(vaddr[eb] + tile_off);
        vhi[eb] = lds_read_tr16_at(vaddr[eb] + tile_off + 16 * ROWB);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * VPF, 0);  // the LDS reads lead the block
    bf16x8 pop[NQB];
    float acc[8];
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
        float pv[8];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                pv[u * 4 + r] = __builtin_amdgcn_exp2f(S[u][qb][r] * sl2);
        if (COLSUM) {
            // the cap keeps wq finite, so that a zero probability times it stays zero
            const float wq = __builtin_amdgcn_exp2f(fminf(__builtin_fmaf(-st.negm[qb][0], sl2, off[qb]), 126.f));
#pragma unroll
            for (int j = 0; j < 8; j++) acc[j] = qb == 0 ? pv[j] * wq : __builtin_fmaf(pv[j], wq, acc[j]);
        }
        u32x4 packed;
#pragma unroll
        for (int t = 0; t < 4; t++) packed[t] = pack_bf16x2(pv[2 * t], pv[2 * t + 1]);
        pop[qb] = __builtin_bit_cast(bf16x8, packed);
    }
    if (COLSUM) row16_sums_to_lds(acc, part, g, l16);
    // denominator from the same bf16 probabilities that weight V
#pragma unroll
    for (int qb = 0; qb < NQB; qb++)
        st.L[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pop[qb], st.L[qb], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, NQB, 0);
#pragma unroll
    for (int eb = 0; eb < NEB; eb++) {
        if (eb + VPF < NEB) {
            vlo[eb + VPF] = lds_read_tr16_at(vaddr[eb + VPF] + tile_off);
            vhi[eb + VPF] = lds_read_tr16_at(vaddr[eb + VPF] + tile_off + 16 * ROWB);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        short8v both = __builtin_shufflevector(vlo[eb], vhi[eb], 0, 1, 2, 3, 4, 5, 6, 7);
        bf16x8 vop = __builtin_bit_cast(bf16x8, both);
#pragma unroll
        for (int qb = 0; qb < NQB; qb++)
            st.O[eb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, pop[qb], st.O[eb][qb], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NQB, 0);
    }
}

constexpr int kBlockColumns = CHIPMUNK_ATTN_BLOCK_COLUMNS;   // key columns per entry of a block list
static_assert(kBlockColumns % (kTilesPerStep * kTileRows) == 0, "a step never straddles two blocks");

// Workgroups go to the eight XCDs in turn (id modulo 8).  Position of workgroup `id` of `all` when each XCD takes one run of
// the positions, so that a head's K and V are read through one or two L2s instead of all eight; without it neighbouring
// chunks of a head run side by side on all XCDs.
__device__ __forceinline__ uint32_t attn_run_of_xcd(uint32_t id, uint32_t all) {
    const uint32_t xcd = id & 7, each = all >> 3, more = all & 7;
    return xcd * each + min(xcd, more) + (id >> 3);
}
// Eight heads in work at a time are worth it while their K and V stay in the last-level cache (256 MB).  Column lists, 7 to
// 10 % kept: 24 x 2304: 26.6 -> 22.1 us; 24 x 4608 (single round): 34.1 -> 33.0; 40 x 9000: 209 -> 202; 24 x 18 000: 301 -> 295;
// 24 x 30 000 (8 heads: 123 MB): 734 -> 726; 24 x 60 000 (246 MB): 2677 -> 2736; 24 x 115 456: 9597 -> 10 253 us.
static int attn_by_xcd(int N, int E) { return (int64_t)N * E <= (1 << 22); }

// What the kernel walks.  kColumnList: the unit's list of columns.  kEveryColumn: no list, every column (dense).
// kFusedDense: every column, and the column sums of Alg. 4 are formed from the same score tiles.  kBlockList: the
// unit's list names blocks of kBlockColumns consecutive columns (the [c, 128] block sparsity of Table 2); the list
// positions are the blocks' columns in order, so the rows of a step are one contiguous run of K and V.
enum AttnMode { kColumnList = 0, kFusedDense = 1, kBlockList = 2, kEveryColumn = 3 };

// The work of one workgroup: NWAVES waves, each owning NQB blocks of 16 queries; 16 * NQB * NWAVES rows, chunk `unit` or
// part `part` of it.
// KEYS = 2: the workgroup has half as many rows, and two waves share them: one takes the first tile of every step, the
// other the second, each with a reference, denominator and accumulator of its own, and the two meet through LDS at the
// end.  What bounds a workgroup of 64 rows is its chain of tiles and the LDS reads of its waves, each of which reads all
// of K and V: with 64 rows shared by pairs the waves read half as much, with 32 the chain is half as long (times at
// attn_part_form).
template <int E, int NQB, int NWAVES, int MODE, int KEYS = 1>
__device__ __forceinline__ void attn_rows(const AttnParams& p, int64_t unit, int part) {
    constexpr bool FUSED = MODE == kFusedDense;
    constexpr bool BLOCKS = MODE == kBlockList;
    static_assert(KEYS == 1 || (KEYS == kTilesPerStep && !FUSED && !BLOCKS), "a wave takes all tiles of a step or one");
    // Every column in order: the columns are the list positions.  A mode of its own and not a null list inside
    // kColumnList: there the branch on the pointer put a wait for all memory behind each step's tile requests (the
    // compiler guards the registers that the other branch loads the column numbers into).
    constexpr bool NOLIST = FUSED || MODE == kEveryColumn;
    constexpr int ROWB = E * 2;           // bytes per K/V row
    constexpr int CH = ROWB / 16;         // 16-byte chunks per row
    constexpr int RPI = 64 / CH;          // rows covered by one wave-wide 16-byte load
    constexpr int NI = kTileRows / (RPI * NWAVES);  // such loads per wave per tile and matrix
    constexpr int NT = 64 * NWAVES;
    constexpr int TILE = kTileRows * ROWB;
    constexpr int STAGE = 2 * TILE;       // K tile then V tile

    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];  // the tile buffers and, with three query blocks, base rows
    // FUSED: per-wave column sums of the two tiles of a step, double buffered over steps
    __shared__ float s_part[FUSED ? 2 * NWAVES * kTilesPerStep * kTileRows : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int g = lane >> 4;
    const int l16 = lane & 15;

    constexpr int ROWS = 16 * NQB * NWAVES / KEYS;   // query rows of a workgroup
    const int wr = w / KEYS, kg = KEYS == 1 ? 0 : wu % KEYS;   // the wave's rows, and its tile of a step
    const int64_t bh = unit / p.NB;
    const int chunk = (int)(unit % p.NB);
    const int row0 = chunk * p.c + part * ROWS;
    const int rows_valid = min(ROWS, p.N - row0);
    if (rows_valid <= 0) return;              // the last chunk may end before this part of it
    // Contents of counts and idx are the caller's precondition; they are clamped all the same so that a bad
    // entry reads a wrong row instead of leaving the tensors.
    // (block lists: counts and k_stride are in blocks; `count` is in list positions = columns all the same)
    const int entries = __builtin_amdgcn_readfirstlane(p.counts ? min(p.counts[unit], p.k_stride) : p.N);
    int count = BLOCKS ? entries * kBlockColumns : entries;
    // The length is hidden from the compiler's value tracking: knowing that a block list's length is a multiple
    // of two steps, it fuses the two copies of the step below into one scheduling region and then needs far
    // more registers than there are (hundreds of bytes of spills in the main loop).
    asm volatile("" : "+s"(count));

    const int64_t head_off = bh * (int64_t)p.N * E;
    const uint16_t* qh = p.q + head_off;
    const uint16_t* kh = p.k + head_off;
    const uint16_t* vh = p.v + head_off;
    const uint16_t* baseh = p.base ? p.base + head_off : nullptr;
    uint16_t* outh = p.out + head_off;

    if (count <= 0) {  // nothing selected: the output is the cache, bit for bit
        for (int t = tid; t < rows_valid * CH; t += NT) {
            int64_t off = (int64_t)(row0 + t / CH) * E + (t % CH) * 8;
            u32x4 val = baseh ? *reinterpret_cast<const u32x4*>(baseh + off) : u32x4{0, 0, 0, 0};
            *reinterpret_cast<u32x4*>(outh + off) = val;
        }
        return;
    }

    AttnState<E, NQB> st;
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
        st.negm[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        st.L[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int eb = 0; eb < E / 16; eb++) st.O[eb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        int qrow = (wr * NQB + qb) * 16 + l16;
#pragma unroll
        for (int es = 0; es < E / 32; es++) {
            u32x4 val = u32x4{0, 0, 0, 0};
            if (qrow < rows_valid)
                val = *reinterpret_cast<const u32x4*>(qh + (int64_t)(row0 + qrow) * E + 32 * es + 8 * g);
            st.Q[es][qb] = __builtin_bit_cast(bf16x8, val);
        }
    }
    const bool wave_active = wu / KEYS * NQB * 16 < rows_valid;   // wave-uniform, and known to be
    const float slack = kRescaleSlack / p.sl2;
    // FUSED: -prev_m (log2 units) - log2(prev_l) of the lane's queries; -inf drops a query row that does not exist
    float off[NQB];
    if (FUSED) {
#pragma unroll
        for (int qb = 0; qb < NQB; qb++) {
            int qrow = (w * NQB + qb) * 16 + l16;
            off[qb] = -INFINITY;
            if (qrow < rows_valid) {
                const int64_t at = bh * p.N + row0 + qrow;
                off[qb] = -p.prev_m[at] * 1.4426950408889634f - __builtin_amdgcn_logf(p.prev_l[at]);
            }
        }
    }
    const int active_waves = min(NWAVES, (rows_valid + NQB * 16 - 1) / (NQB * 16));
    float* colsum_row = FUSED ? p.colsum + unit * p.ld_colsum : nullptr;
    auto flush_column_sums = [&](int tile0) {  // sums of tiles tile0, tile0+1: the waves' partial sums -> global
        if (FUSED && tid < kTilesPerStep * kTileRows) {
            const float* part = s_part + ((tile0 / kTilesPerStep) & 1) * (NWAVES * kTilesPerStep * kTileRows);
            float v = 0.f;
            for (int ww = 0; ww < active_waves; ww++) v += part[ww * (kTilesPerStep * kTileRows) + tid];
            const int j = tile0 * kTileRows + list_pos_in_step<E>(tid / kTileRows, tid % kTileRows);
            if (j < p.N) colsum_row[j] = v;
        }
    };
    const u32x4 ones_bits = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

    // per-lane LDS read addresses (bytes, the LDS base included) inside a 16-row group of tile buffer 0: one per
    // contraction slice, because the slice number enters through the XOR swizzle, not additively
    const int koff = l16 * ROWB + ((g ^ swizzle<E>(l16)) * 16);
    const int vrow = 4 * g + (l16 >> 2);
    const int voff = vrow * ROWB + (((((l16 & 3) >> 1)) ^ swizzle<E>(vrow)) * 16) + 8 * (l16 & 1);
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
    uint32_t kaddr[E / 32], vaddr[E / 16];
#pragma unroll
    for (int es = 0; es < E / 32; es++) kaddr[es] = smem_at + (uint32_t)((koff ^ (64 * es)) + kg * STAGE);
#pragma unroll
    for (int eb = 0; eb < E / 16; eb++) vaddr[eb] = smem_at + (uint32_t)((voff ^ (32 * eb)) + kg * STAGE);
    // The LDS base is a link-time constant; left visible, the compiler would keep the offsets without it and add
    // it again at every read.  Behind this barrier each address is just a register.
#pragma unroll
    for (int es = 0; es < E / 32; es++) asm volatile("" : "+v"(kaddr[es]));
#pragma unroll
    for (int eb = 0; eb < E / 16; eb++) asm volatile("" : "+v"(vaddr[eb]));

    // Gather bookkeeping.  Load i of this wave fills rows (i*NWAVES+w)*RPI .. +RPI-1 of
    // the tile; the lane owns row (i*NWAVES+w)*RPI + lane/CH, LDS chunk position lane%CH,
    // and therefore fetches the logical chunk  position ^ swizzle(row).
    const int sel = lane / CH;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + (uint32_t)w * 1024u);
    // whole steps: the rows of a step's tiles interleave the step's list positions (list_pos_in_step), so the last
    // step runs all its tiles, masked
    const int ntiles = (count + kTilesPerStep * kTileRows - 1) / (kTilesPerStep * kTileRows) * kTilesPerStep;
    uint32_t chunk_off[NI];  // byte offset of the lane's chunk inside the row it fetches
#pragma unroll
    for (int i = 0; i < NI; i++) chunk_off[i] = (uint32_t)(((lane % CH) ^ swizzle<E>((i * NWAVES + w) * RPI + sel)) * 16);

    // K, V and the unit's index list are read through buffer resources: the hardware checks every
    // offset against the tensor's size (an out-of-range access returns zero), so neither the column
    // numbers nor the positions in the list are clamped with vector instructions.  A slot of the list
    // at or beyond `count` reads as column 0: a valid row, whose scores the last tile masks.
    const i32x4 kbuf = raw_buffer_words(kh, (uint32_t)p.N * ROWB);
    const i32x4 vbuf = raw_buffer_words(vh, (uint32_t)p.N * ROWB);
    const i32x4 bbuf = raw_buffer_words(baseh ? baseh + (int64_t)row0 * E : nullptr, baseh ? (uint32_t)rows_valid * ROWB : 0u);
    const int32_t* idxg = !NOLIST && p.idx ? p.idx + unit * (int64_t)p.k_stride : nullptr;
    // two views of the unit's list: its whole row (positions below k_stride: the vector loads of the steps that lie
    // inside the list) and the part below count (a position at or beyond count reads as 0: the list's last step)
    const __amdgpu_buffer_rsrc_t ibuf_row = raw_buffer(idxg, idxg ? (uint32_t)p.k_stride * 4u : 0u);
    const __amdgpu_buffer_rsrc_t ibuf = raw_buffer(idxg, idxg ? (uint32_t)entries * 4u : 0u);

    // Every lane fetches the column numbers of the tile rows it fills, one step ahead of the gather that uses
    // them: the load is issued behind that step's tile transfers and has landed, like those, when the next step
    // starts with its wait for all memory.  A lane's kTilesPerStep * NI rows of a step hold consecutive list
    // positions (list_pos_in_step), so one vector load brings them all.  The list's last step is the only one
    // that can reach beyond count: its columns are fetched once, up front, entry by entry through the view that
    // ends at count (colt), and the step before it (or the prologue) gathers from those.
    constexpr int RPL = kTilesPerStep * NI;       // rows (= column numbers) per lane and step
    static_assert(RPL == 4 || RPL == 2, "the column numbers of a step come as one 16- or 8-byte load per lane");
    int colv[RPL], colt[RPL];
    int next_pos = (w * RPI + sel) * RPL;         // the lane's first list position in the next step to load
    if constexpr (MODE == kColumnList) {
        // (in order, not interleaved: a last step of at most one tile's positions then needs only its first tile)
        const int last_pos = (ntiles - kTilesPerStep) * kTileRows + w * RPI + sel;
#pragma unroll
        for (int s = 0; s < kTilesPerStep; s++)
#pragma unroll
            for (int i = 0; i < NI; i++)
                colt[s * NI + i] = __builtin_amdgcn_raw_buffer_load_b32(ibuf, (last_pos + s * kTileRows + i * NWAVES * RPI) * 4, 0, 0);
    }
    int blockv = 0;                               // BLOCKS: the block that holds the next step to gather (the same in every lane)
    int block_now = 0, block_next = 0;            // BLOCKS: first column of the block of the step in work / of the next step
    auto load_cols = [&]() {
        if constexpr (NOLIST) return;  // gather_offsets forms the columns from the positions
        if constexpr (BLOCKS) {        // one list entry serves kBlockColumns positions; past the list's end it reads as block 0
            blockv = __builtin_amdgcn_raw_buffer_load_b32(ibuf, (next_pos / kBlockColumns) * 4, 0, 0);
            next_pos += kTilesPerStep * kTileRows;
            return;
        }
        if constexpr (RPL == 4) {
            const u32x4 c4 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ibuf_row, next_pos * 4, 0, 0));
#pragma unroll
            for (int j = 0; j < RPL; j++) colv[j] = (int)c4[j];
        } else {
            const u32x2 c2 = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(ibuf_row, next_pos * 4, 0, 0));
#pragma unroll
            for (int j = 0; j < RPL; j++) colv[j] = (int)c2[j];
        }
        next_pos += kTilesPerStep * kTileRows;
    };
    // One of the E/16 transfers that fill buffer half `half` with the tiles whose columns are in colv: piece j is
    // the K (j even) or V (j odd) part of load i = (j/2) % NI of tile s = j / (2 NI).
    uint32_t goff[kTilesPerStep][NI];   // byte offset of the lane's chunk inside the head's K (and V) matrix
    // from the column numbers that have landed: once per step, ahead of the products; `last`: the step to gather
    // is the list's last one
    int gather_pos = (w * RPI + sel) * RPL;       // FUSED: the lane's first list position in the next step to gather
    auto gather_offsets = [&](bool last) {
#pragma unroll
        for (int s = 0; s < kTilesPerStep; s++)
#pragma unroll
            for (int i = 0; i < NI; i++) {
                int col;
                if constexpr (NOLIST) col = min(gather_pos + s * NI + i, p.N - 1);   // column = position
                else if constexpr (BLOCKS) col = min(blockv * kBlockColumns + (gather_pos % kBlockColumns) + s * NI + i, p.N - 1);
                else col = last ? colt[s * NI + i] : colv[s * NI + i];
                goff[s][i] = (uint32_t)col * ROWB + chunk_off[i];
                // formed here, not again in front of every transfer (the kernel with the column sums has no
                // registers for that and lets the compiler form them where it likes)
                if constexpr (!FUSED) asm volatile("" : "+v"(goff[s][i]));
            }
        gather_pos += kTilesPerStep * kTileRows;
        if constexpr (BLOCKS) {
            block_now = block_next;
            block_next = __builtin_amdgcn_readfirstlane(blockv) * kBlockColumns;
        }
    };
    auto gather_piece = [&](auto half_c, int j) {
        constexpr int half = decltype(half_c)::value;
        const int s = j / (2 * NI), i = (j / 2) % NI;
        const uint32_t dst = lds0 + (uint32_t)((half * kTilesPerStep + s) * STAGE + i * NWAVES * 1024);
        if (j & 1) load_buffer_to_lds_16B(vbuf, goff[s][i], dst + TILE);
        else load_buffer_to_lds_16B(kbuf, goff[s][i], dst);
    };
    static_assert(kTilesPerStep * NI * 2 == E / 16, "one transfer per group of score products");

    // KEYS = 2: a wave merges and stores half the columns of its rows.  The base rows' part of those waits in registers,
    // as it is stored: the lane's eight columns of two blocks (requested here or in the last step: the same time).
    u32x4 half_base[KEYS == 1 ? 1 : NQB][KEYS == 1 ? 1 : E / 64];
    if constexpr (KEYS == 2) {
#pragma unroll
        for (int qb = 0; qb < NQB; qb++)
#pragma unroll
            for (int pair = 0; pair < E / 64; pair++) {
                const int qrow = min((wr * NQB + qb) * 16 + l16, rows_valid - 1);
                half_base[qb][pair] = baseh ? *reinterpret_cast<const u32x4*>(baseh + (int64_t)(row0 + qrow) * E + (kg * (E / 32) + 2 * pair + (g & 1)) * 16 + (g >> 1) * 8)
                                            : u32x4{0, 0, 0, 0};
            }
    }

    // The query loads must not be left pending into the loop: a wait for them inside
    // the loop would also wait for every tile transfer in flight.  The columns of the
    // first step are requested beside them: one round trip for both.
    load_cols();
    wait_all_memory();

    // first step in flight; columns of the second step requested
    gather_offsets(ntiles <= kTilesPerStep);
#pragma unroll
    for (int j = 0; j < E / 16; j++) gather_piece(std::integral_constant<int, 0>{}, j);
    load_cols();

    // The base rows that the results are merged with are brought to LDS in the last step, in the place of a next step's
    // tiles: each wave its own rows, a query block's 16 rows at a time, two blocks of every wave in the free buffer half
    // and a third behind the buffers.  Fetched after the last step instead, they cost a round trip of their own in which
    // nothing else runs (and in a short launch all workgroups ask for theirs at once).  16-byte chunks are XOR-swizzled
    // by the row.
    constexpr int BLOCKB = 16 * ROWB;     // bytes of a query block's base rows
    constexpr int BASE_PIECES = BLOCKB / 1024;
    const int base_row = (w * NQB * 16 + sel) * ROWB;
    auto base_place = [&](int half_in_use, int qb) -> uint32_t {   // within the buffers, without the LDS base
        return qb < 2 ? (uint32_t)((half_in_use ^ 1) * kTilesPerStep * STAGE + (w * 2 + qb) * BLOCKB)
                      : (uint32_t)(kStages * STAGE + (w * (NQB - 2) + qb - 2) * BLOCKB);
    };
    auto base_swizzle = [](int row) { return (E == 128 ? row : row >> 1) & (CH - 1); };   // of the row inside the block

    // One step: the kTilesPerStep tiles in buffer half `half`.  The half is a compile-time constant (the loop
    // below alternates two copies of the step), so every LDS offset of the step is an immediate of its read.
    // The next step's tiles are requested between the score products of this step's first tile, and the columns
    // of the step after that behind them.  The list's last step has a copy of its own (LAST): it requests the base rows
    // instead, masks the positions beyond the list, and leaves out a tile that has none; its half, `last_half`, has
    // been added to the addresses.  Without a list the last step runs in the loop, and its requests reach past the end into
    // the buffer that nobody reads: few callers merge there, the kernel with the column sums has no registers left for a
    // third copy (244 bytes of spills, 8.0 ms instead of 5.9 at 40 heads x 18 000), and the plain one is faster as well
    // (24 x 115 456: 125.6 -> 124.0 ms, 40 x 18 000: 5.23 -> 5.17).
    auto step = [&](auto half_c, auto last_c, int t, int last_half) {
        constexpr int half = decltype(half_c)::value;
        constexpr bool LAST = decltype(last_c)::value;
        wait_all_memory();
        __syncthreads();  // this step's tiles have landed for every wave; the other half is free to refill
        if constexpr (!LAST) gather_offsets(t + 2 * kTilesPerStep >= ntiles);
        if constexpr (LAST && BLOCKS) block_now = block_next;
        if (FUSED && t > 0) flush_column_sums(t - kTilesPerStep);
        if constexpr (KEYS == 2) {
            f32x4 S[2][NQB];
            // Both waves take their first reference from the unit's first tile, which the second one multiplies for that
            // alone: as long as nothing raises it, a weight's rounding to bf16 is the same whichever wave forms it and
            // however the rows are walked.
            if (half == 0 && t == 0 && kg == 1) {
                uint32_t first_tile[E / 32];
#pragma unroll
                for (int es = 0; es < E / 32; es++) first_tile[es] = kaddr[es] - STAGE;
                attn_scores<E, NQB, 1>(S, st, first_tile, 0, [](int) {});
                if constexpr (LAST) attn_mask_tail<E, NQB, true>(S, 0, 0, count, g);
                else if (NOLIST && kTilesPerStep >= ntiles) attn_mask_tail<E, NQB>(S, 0, 0, count, g);
                attn_update_max<E, NQB>(st, S, true, p.sl2, slack);
            }
            if constexpr (LAST) {
                if ((t + kg) * kTileRows >= count) return;
                attn_scores<E, NQB, 1>(S, st, kaddr, half * kTilesPerStep * STAGE, [](int) {});
                attn_mask_tail<E, NQB, true>(S, t * kTileRows, kg, count, g);
            } else {
                attn_scores<E, NQB, 1>(S, st, kaddr, half * kTilesPerStep * STAGE,
                                       [&](int j) { gather_piece(std::integral_constant<int, half ^ 1>{}, j); });
                load_cols();
                if (NOLIST && t + kTilesPerStep >= ntiles) attn_mask_tail<E, NQB>(S, t * kTileRows, kg, count, g);
            }
            attn_update_max<E, NQB>(st, S, t == 0 && kg == 0, p.sl2, slack);
            attn_weights_and_pv<E, NQB, false, kVPrefetch>(st, S, vaddr, half * kTilesPerStep * STAGE + TILE, p.sl2, ones);
            return;
        }
#pragma unroll
        for (int s = 0; s < kTilesPerStep; s++) {
            const int tile_off = (half * kTilesPerStep + s) * STAGE;   // a constant once the loop over s is unrolled
            if (LAST && MODE == kColumnList && s > 0 && (t + s) * kTileRows >= count) break;
            f32x4 S[2][NQB];
            if (s == 0 && !LAST) {
                attn_scores<E, NQB, 1>(S, st, kaddr, tile_off,
                                    [&](int j) { gather_piece(std::integral_constant<int, half ^ 1>{}, j); });
                load_cols();
            } else if (s == 0) {
                attn_scores<E, NQB, 1>(S, st, kaddr, tile_off, [&](int j) {
                    if (!baseh) return;
                    for (int n = j; n < NQB * BASE_PIECES; n += E / 16) {
                        const int qb = n / BASE_PIECES, i = n % BASE_PIECES, row = i * RPI + sel;
                        load_buffer_to_lds_16B(bbuf, (uint32_t)(base_row + (qb * 16 + i * RPI) * ROWB + (((lane % CH) ^ base_swizzle(row)) * 16)),
                                               lds_address(smem) + __builtin_amdgcn_readfirstlane(base_place(last_half, qb)) + i * 1024);
                    }
                });
            } else {
                attn_scores<E, NQB, 1>(S, st, kaddr, tile_off, [](int) {});
            }
            if constexpr (BLOCKS) {   // only the sequence's last block can reach beyond N; it may stand anywhere in the list
                const int col0 = block_now + (t * kTileRows) % kBlockColumns;
                if (col0 + kTilesPerStep * kTileRows > p.N) attn_mask_tail<E, NQB>(S, col0, s, p.N, g);
            } else if constexpr (LAST) {
                attn_mask_tail<E, NQB, MODE == kColumnList>(S, t * kTileRows, s, count, g);
            } else if constexpr (NOLIST) {
                if (t + kTilesPerStep >= ntiles) attn_mask_tail<E, NQB>(S, t * kTileRows, s, count, g);
            }
            attn_update_max<E, NQB>(st, S, t + s == 0, p.sl2, slack);
            attn_weights_and_pv<E, NQB, FUSED, FUSED ? 1 : kVPrefetch>(st, S, vaddr, tile_off + TILE, p.sl2, ones, off,
                                               s_part + ((half * NWAVES + w) * kTilesPerStep + s) * kTileRows, g, l16);
        }
    };
    const int last_tile = ntiles - kTilesPerStep;   // first tile of the last step
    const int loop_end = NOLIST ? ntiles : last_tile;
#pragma unroll 1
    for (int t = 0; t < loop_end; t += 2 * kTilesPerStep) {
        step(std::integral_constant<int, 0>{}, std::false_type{}, t, 0);
        if (t + kTilesPerStep >= loop_end) break;
        step(std::integral_constant<int, 1>{}, std::false_type{}, t + kTilesPerStep, 0);
    }
    const int last_half = (last_tile / kTilesPerStep) & 1;
    if constexpr (!NOLIST) {
        const uint32_t shift = (uint32_t)(last_half * kTilesPerStep * STAGE);
#pragma unroll
        for (int es = 0; es < E / 32; es++) kaddr[es] += shift;
#pragma unroll
        for (int eb = 0; eb < E / 16; eb++) vaddr[eb] += shift;
        step(std::integral_constant<int, 0>{}, std::true_type{}, last_tile, last_half);
    }
    wait_all_memory();  // the base rows (NOLIST: the transfers behind the last step) have landed
    // The transfers' asm names no memory and the wait is no barrier to the compiler: without this it might read the base rows
    // from LDS ahead of the wait (other tiles are read behind a workgroup barrier; a wave's base rows are its own).
    asm volatile("" ::: "memory");
    if (FUSED) {
        __syncthreads();  // the last step's partial sums are complete
        flush_column_sums(last_tile);
    }

    if constexpr (KEYS == 2) {
        // Each wave hands the half of its columns that the other one stores, and its reference and denominator, over in
        // LDS.
        constexpr int HALF = E / 32;          // blocks of 16 columns
        constexpr int AREA = NQB * HALF * 1024, STATS = NWAVES * AREA;
        static_assert(STATS + NWAVES * NQB * 512 <= kStages * STAGE, "the halves fit the tile buffers");
        lds_accesses_then_barrier();          // every wave is done with the tiles
#pragma unroll
        for (int qb = 0; qb < NQB; qb++) {
#pragma unroll
            for (int i = 0; i < HALF; i++)
                *reinterpret_cast<f32x4*>(smem + w * AREA + (qb * HALF + i) * 1024 + lane * 16) = kg ? st.O[i][qb] : st.O[HALF + i][qb];
            *reinterpret_cast<f32x2*>(smem + STATS + (w * NQB + qb) * 512 + lane * 8) = f32x2{st.negm[qb][0], st.L[qb][0]};
        }
        lds_accesses_then_barrier();
        if (!wave_active) return;
#pragma unroll
        for (int qb = 0; qb < NQB; qb++) {
            const f32x2 theirs = *reinterpret_cast<const f32x2*>(smem + STATS + ((w ^ 1) * NQB + qb) * 512 + lane * 8);
            const float m = fmaxf(-st.negm[qb][0], -theirs[0]);
            const float mine = __builtin_amdgcn_exp2f((-st.negm[qb][0] - m) * p.sl2), their = __builtin_amdgcn_exp2f((-theirs[0] - m) * p.sl2);
            const float ltot = st.L[qb][0] * mine + theirs[1] * their;
            const float f = p.o_scale / ltot, f_mine = f * mine, f_their = f * their;
            const int qrow = (wr * NQB + qb) * 16 + l16;
            u32x4 r[HALF / 2];
#pragma unroll
            for (int pair = 0; pair < HALF / 2; pair++) {
                // lanes 16 apart hold each other's halves of two blocks, which the swap brings to the accumulators'
                // places
                const u32x4 base = half_base[qb][pair];
                const auto b02 = __builtin_amdgcn_permlane16_swap(base[0], base[2], false, false);
                const auto b13 = __builtin_amdgcn_permlane16_swap(base[1], base[3], false, false);
                u32x2 sum[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const int eb = 2 * pair + i;
                    const f32x4 o = *reinterpret_cast<const f32x4*>(smem + (w ^ 1) * AREA + (qb * HALF + eb) * 1024 + lane * 16);
                    const f32x4 own = kg ? st.O[HALF + eb][qb] : st.O[eb][qb];
                    const u32x2 b = {b02[i], b13[i]};
                    sum[i] = u32x2{pack_bf16x2(bf16_bits_to_float(b[0] & 0xffffu) + (f_mine * own[0] + f_their * o[0]),
                                               bf16_bits_to_float(b[0] >> 16) + (f_mine * own[1] + f_their * o[1])),
                                   pack_bf16x2(bf16_bits_to_float(b[1] & 0xffffu) + (f_mine * own[2] + f_their * o[2]),
                                               bf16_bits_to_float(b[1] >> 16) + (f_mine * own[3] + f_their * o[3]))};
                }
                const auto lo = __builtin_amdgcn_permlane16_swap(sum[0][0], sum[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(sum[0][1], sum[1][1], false, false);
                r[pair] = u32x4{lo[0], hi[0], lo[1], hi[1]};
            }
            if (qrow >= rows_valid) continue;
            if (p.row_m && g == 0 && kg == 0) {
                p.row_m[bh * p.N + row0 + qrow] = m * (p.sl2 * 0.6931471805599453f);
                p.row_l[bh * p.N + row0 + qrow] = ltot;
            }
#pragma unroll
            for (int pair = 0; pair < HALF / 2; pair++)
                *reinterpret_cast<u32x4*>(outh + (int64_t)(row0 + qrow) * E + (kg * HALF + 2 * pair + (g & 1)) * 16 + (g >> 1) * 8) = r[pair];
        }
        return;
    }
    if (!wave_active) return;
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
        float ltot = st.L[qb][0];
        float f = p.o_scale / ltot;
        int qrow = (w * NQB + qb) * 16 + l16;
        const int64_t row_off = (int64_t)(row0 + min(qrow, rows_valid - 1)) * E + 4 * g;
        u32x2 bases[NOLIST ? E / 16 : 1];
        if (MODE == kEveryColumn && baseh) {   // all requested before the first store
#pragma unroll
            for (int eb = 0; eb < E / 16; eb++) bases[eb] = *reinterpret_cast<const u32x2*>(baseh + row_off + eb * 16);
        }
        if (qrow < rows_valid) {
            if (p.row_m && g == 0) {
                p.row_m[bh * p.N + row0 + qrow] = -st.negm[qb][0] * (p.sl2 * 0.6931471805599453f);
                p.row_l[bh * p.N + row0 + qrow] = ltot;
            }
            // A lane holds four columns of each block of 16; lanes 16 apart exchange halves of two blocks, so that each stores
            // eight columns in one piece and a row leaves in runs of 64 bytes.  (In runs of 32: 24 heads x 4608, 7 % of the
            // columns 34.8 us, like this 32.4; 16 x 2 heads x 3982, 3 %: 25.9, 23.5; 24 x 115 456 0.2 %.)
#pragma unroll
            for (int pair = 0; pair < E / 32; pair++) {
                u32x2 r[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const int eb = 2 * pair + i;
                    u32x2 b = u32x2{0, 0};
                    if (MODE == kEveryColumn && baseh) b = bases[eb];
                    if (!NOLIST && baseh)
                        b = *reinterpret_cast<const u32x2*>(smem + base_place(last_half, qb) + l16 * ROWB +
                                                            (((2 * eb + (g >> 1)) ^ base_swizzle(l16)) * 16) + (g & 1) * 8);
                    float o0 = bf16_bits_to_float(b[0] & 0xffffu) + f * st.O[eb][qb][0];
                    float o1 = bf16_bits_to_float(b[0] >> 16) + f * st.O[eb][qb][1];
                    float o2 = bf16_bits_to_float(b[1] & 0xffffu) + f * st.O[eb][qb][2];
                    float o3 = bf16_bits_to_float(b[1] >> 16) + f * st.O[eb][qb][3];
                    r[i] = u32x2{pack_bf16x2(o0, o1), pack_bf16x2(o2, o3)};
                }
                const auto lo = __builtin_amdgcn_permlane16_swap(r[0][0], r[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(r[0][1], r[1][1], false, false);
                *reinterpret_cast<u32x4*>(outh + row_off - 4 * g + (2 * pair + (g & 1)) * 16 + (g >> 1) * 8) = u32x4{lo[0], hi[0], lo[1], hi[1]};
            }
        }
    }
}

// How the chunks that have no workgroup of their own are walked (attn_part_form).
enum AttnPart { kRows64 = 0, kRows64Shared = 1, kRows32Shared = 2 };

// A workgroup per chunk, or, with a column list or every column, for the first p.whole chunks only: each of the others is
// walked by a workgroup per 64 or 32 rows.  Those are the launch's last, partly filled round, or all of a small launch.
template <int E, int NQB, int NWAVES, int MODE = kColumnList, int PART = kRows64>
__global__ __launch_bounds__(64 * NWAVES, NWAVES == 4 ? 2 : 1) void attn_sparse_delta_kernel(AttnParams p) {
    uint32_t id = blockIdx.x, all = gridDim.x;
    if constexpr (MODE == kColumnList || MODE == kEveryColumn) {
        const uint32_t whole = (uint32_t)p.whole;   // a multiple of eight, or all of them
        const uint32_t first = MODE == kEveryColumn ? (uint32_t)p.first : 0;   // a refresh's last round
        if (id >= whole) {
            id -= whole;
            all -= whole;
            if (p.by_xcd) id = attn_run_of_xcd(id, all);
            constexpr int PARTS = PART == kRows32Shared ? 2 * NQB : NQB;   // per chunk
            attn_rows<E, PART == kRows64Shared ? 2 : 1, NWAVES, MODE, PART == kRows64 ? 1 : 2>(p, first + whole + id / PARTS, (int)(id % PARTS));
            return;
        }
        all = whole;
    }
    if (p.by_xcd) id = attn_run_of_xcd(id, all);
    if constexpr (MODE == kEveryColumn) id += (uint32_t)p.first;
    attn_rows<E, NQB, NWAVES, MODE>(p, id, 0);
}

// Column sums of the attention probabilities (Sec. 3.3.1, the tensor D; Alg. 4):
//   D[b,h,i,j] = sum over the rows q of chunk i of exp(scale*s_qj - m_q) / l_q
// with (m_q, l_q) either from the dense attention pass of the same step (exact sums) or
// carried over from an earlier step (the stale-normaliser approximation of App. B.2).  Scores are produced as
// S = Q K^T (queries on the rows of the MFMA result), so that the sum over the
// chunk's queries is a sum over a lane's registers, the wave's four 16-lane
// rows and the workgroup's four waves.
struct ColsumParams {
    const uint16_t* q;
    const uint16_t* k;
    const float* row_m;
    const float* row_l;
    float* colsum;
    int64_t ld;
    int N, NB, c;
    float sl2;
    int pieces;   // a chunk's keys are cut into so many runs of whole tiles, one workgroup each
    int first = 0;   // the launch's first chunk
};

// What bounds it: the vector instructions of the scores.  A score costs an FMA, an exponential (two issue slots) and an
// FMA (the weight's 1 / l) beside a quarter of an MFMA's issue slot; four waves per SIMD cover each other's phases.
// The 64 sums of a tile are folded over the four lane groups by three swaps and three adds instead of four times two of
// each, transfers go through a buffer resource (a key beyond N reads as zero and is not stored) with offsets that only
// step on, and the two buffer halves are two copies of the step, so every LDS offset is an immediate.  24 heads x 18 000
// tokens: 1.90 ms in one run over the keys with two waves per SIMD, 1.78 ms now (1.12 PFLOP/s of scores); 24 x 4608: 165
// and 126 us.  1 / l is a factor: as part of the exponential's addend (-m - log l, half the registers, 1.75 ms) it is
// rounded at twice the argument's magnitude, and the sums are three times as far off (7e-8 against 2.2e-7 and more).
// Four other orders of the same work (all scores of a tile first, two blocks at a time, exponentials pinned between the
// products with three and four waves per SIMD) measured equal or slower.
template <int E, int NQB>
__global__ __launch_bounds__(256, 4) void attn_colsum_kernel(ColsumParams p) {
    constexpr int ROWB = E * 2;
    constexpr int CH = ROWB / 16;
    constexpr int RPI = 64 / CH;
    constexpr int NI = kColsumTileRows / (RPI * 4);
    constexpr int TILE = kColsumTileRows * ROWB;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * TILE];
    __shared__ float s_part[2][4][kColsumTileRows];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int g = lane >> 4, l16 = lane & 15;
    const int64_t unit = p.first + blockIdx.x / p.pieces;
    const int piece = (int)(blockIdx.x % p.pieces);
    const int64_t bh = unit / p.NB;
    const int chunk = (int)(unit % p.NB);
    const int row0 = chunk * p.c;
    const int rows_valid = min(p.c, p.N - row0);
    const uint16_t* qh = p.q + bh * (int64_t)p.N * E;
    const uint16_t* kh = p.k + bh * (int64_t)p.N * E;
    float* drow = p.colsum + unit * p.ld;

    bf16x8 Q[E / 32][NQB];
    float m2v[NQB][4], il[NQB][4];
#pragma unroll
    for (int qb = 0; qb < NQB; qb++) {
        int qrow = (w * NQB + qb) * 16 + l16;
#pragma unroll
        for (int es = 0; es < E / 32; es++) {
            u32x4 val = u32x4{0, 0, 0, 0};
            if (qrow < rows_valid)
                val = *reinterpret_cast<const u32x4*>(qh + (int64_t)(row0 + qrow) * E + 32 * es + 8 * g);
            Q[es][qb] = __builtin_bit_cast(bf16x8, val);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {  // the MFMA result holds query 4g+r of the block in register r
            int qr = (w * NQB + qb) * 16 + 4 * g + r;
            bool ok = qr < rows_valid;
            m2v[qb][r] = ok ? p.row_m[bh * p.N + row0 + qr] * 1.4426950408889634f : 0.f;
            il[qb][r] = ok ? 1.f / p.row_l[bh * p.N + row0 + qr] : 0.f;
        }
    }
    const int koff = l16 * ROWB + ((g ^ swizzle<E>(l16)) * 16);
    const int grow0 = w * RPI + lane / CH;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + (uint32_t)w * 1024u);
    // this piece's tiles [tile0, ntiles) of the chunk's keys (no more pieces than tiles: none is empty)
    const int all_tiles = (p.N + kColsumTileRows - 1) / kColsumTileRows;
    const int tile0 = (int)((int64_t)all_tiles * piece / p.pieces);
    const int ntiles = (int)((int64_t)all_tiles * (piece + 1) / p.pieces);
    // The head's K matrix through a buffer resource: a key at or beyond N reads as zero; its sum is not stored.
    const i32x4 kbuf = raw_buffer_words(kh, (uint32_t)p.N * ROWB);
    uint32_t goff[NI];
#pragma unroll
    for (int i = 0; i < NI; i++) {
        const int row = grow0 + 4 * RPI * i;
        goff[i] = (uint32_t)(tile0 * kColsumTileRows + row) * ROWB + (uint32_t)(((lane % CH) ^ swizzle<E>(row)) * 16);
    }
    const uint32_t smem_at = (uint32_t)(uintptr_t)CHIPMUNK_LDS_PTR(smem);
    uint32_t kaddr[E / 32];
#pragma unroll
    for (int es = 0; es < E / 32; es++) {
        kaddr[es] = smem_at + (uint32_t)(koff ^ (64 * es));
        asm volatile("" : "+v"(kaddr[es]));   // just a register: see the attention kernel
    }

    auto gather = [&](int stage) {
#pragma unroll
        for (int i = 0; i < NI; i++) {
            load_buffer_to_lds_16B(kbuf, goff[i], lds0 + (uint32_t)(stage * TILE + i * 4096));
            goff[i] += kColsumTileRows * ROWB;
        }
    };
    auto flush = [&](int t) {  // sums of tile t: four waves' partials -> global
        if (tid < kColsumTileRows) {
            int j = t * kColsumTileRows + tid;
            const int s = (t - tile0) & 1;
            float v = s_part[s][0][tid] + s_part[s][1][tid] + s_part[s][2][tid] + s_part[s][3][tid];
            if (j < p.N) drow[j] = v;
        }
    };
    // scores of 16 keys (columns of the result) against the wave's queries (rows)
    auto scores = [&](f32x4 (&S)[NQB], int off_b) {
        bf16x8 kop[E / 32];
#pragma unroll
        for (int es = 0; es < E / 32; es++) kop[es] = lds_read_b128(kaddr[es] + off_b);
#pragma unroll
        for (int es = 0; es < E / 32; es++)
#pragma unroll
            for (int qb = 0; qb < NQB; qb++)
                S[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Q[es][qb], kop[es], es == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : S[qb], 0, 0, 0);
    };
    // the sum over the lane's queries of one key's weights
    auto weights = [&](const f32x4 (&S)[NQB]) {
        float part = 0.f;
#pragma unroll
        for (int qb = 0; qb < NQB; qb++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(S[qb][r], p.sl2, -m2v[qb][r]));
                part = qb + r == 0 ? e * il[qb][r] : __builtin_fmaf(e, il[qb][r], part);
            }
        return part;
    };

    auto step = [&](auto stage_c, int t) {
        constexpr int stage = decltype(stage_c)::value;
        wait_all_memory();
        __syncthreads();
        gather(stage ^ 1);   // past the last tile too: into a buffer nobody reads
        if (t > tile0) flush(t - 1);
        float part[kColsumTileRows / 16];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            f32x4 S[NQB];
            scores(S, stage * TILE + u * 16 * ROWB);
            part[u] = weights(S);
        }

        // sums over the four lane groups: each swap brings two keys' halves together, so that a group ends with the
        // total of one of the four key blocks (group g: block 2 (g % 2) + g / 2)
        auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(part[0]), __float_as_uint(part[1]), false, false);
        auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(part[2]), __float_as_uint(part[3]), false, false);
        const float x01 = __uint_as_float(a[0]) + __uint_as_float(a[1]), x23 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
        auto d = __builtin_amdgcn_permlane16_swap(__float_as_uint(x01), __float_as_uint(x23), false, false);
        s_part[stage][w][(((g & 1) << 1) | (g >> 1)) * 16 + l16] = __uint_as_float(d[0]) + __uint_as_float(d[1]);
    };
    gather(0);
#pragma unroll 1
    for (int t = tile0; t < ntiles; t += 2) {
        step(std::integral_constant<int, 0>{}, t);
        if (t + 1 >= ntiles) break;
        step(std::integral_constant<int, 1>{}, t + 1);
    }
    wait_all_memory();   // the transfers behind the last tile must have landed before the wave may end
    __syncthreads();
    flush(ntiles - 1);
}

template <int E, int NQB, int NWAVES, int MODE = kColumnList, int PART = kRows64>
static int32_t launch_attn_variant(const AttnParams& p, int64_t units, hipStream_t s) {
    // the tile buffers, and behind them, where there is a list, each wave's third block of base rows
    constexpr int lds = kStages * 2 * kTileRows * E * 2 + ((MODE == kColumnList || MODE == kBlockList) && NQB > 2 ? NWAVES * (NQB - 2) * 16 * E * 2 : 0);
    // set at every launch: the attribute is kept per device, and a flag remembered here would be neither
    // per device nor safe between host threads
    if (hipFuncSetAttribute((const void*)attn_sparse_delta_kernel<E, NQB, NWAVES, MODE, PART>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return CHIPMUNK_ERR_LAUNCH;
    hipLaunchKernelGGL((attn_sparse_delta_kernel<E, NQB, NWAVES, MODE, PART>), dim3((unsigned)units), dim3(64 * NWAVES), lds, s, p);
    return launch_status();
}

// Query rows per workgroup (64 * blocks).  A workgroup of fewer rows takes less time per tile, though more per row: the
// K and V tiles are fetched and read from LDS all the same.  So three blocks per wave (192 rows) are right for whole
// rounds of the 512 workgroup slots (two per CU), and 64 rows for a last round that would leave slots empty.
// Measured time of a 32-key tile in us, with two workgroups on the CU and with one (dense launches of 2 to 40 heads, 1024
// to 18 000 tokens; for E = 64 more than two fit, the figures stand for the same throughput with two):
//     E = 128:  1 block 0.60 / 0.37   2 blocks 0.94 / 0.55   3 blocks 1.27 / 0.80
//     E =  64:  1 block 0.31 / 0.24   2 blocks 0.50 / 0.38   3 blocks 0.74 / 0.52
// and a launch takes (whole rounds) x (the first) + (a last round of more than half the slots: the first; of at most
// half: the second), which orders the measured launches correctly: 24 heads x 4608 x 128: 268, 252 and 305 us with
// three, two and one block throughout; 12 x 2304: 57, 43, 45; 2 x 1024: 29.9, 21.7, 15.7; 24 x 3456 (432 workgroups of 192
// rows): 136, 152, 185; 40 x 18 000: 5259, 5833, 7405.
// With the last round alone in parts: 24 x 4608 x 128 220 us (512 whole chunks and 64 in three parts each), as a column list
// of 323 40.2 -> 34.9 us; 24 x 4608 x 64 145 -> 136 us.
static double attn_rounds_cost(int E, int blocks, int64_t workgroups) {
    static const double paired[2][3] = {{0.31, 0.50, 0.74}, {0.60, 0.94, 1.27}};
    static const double alone[2][3] = {{0.24, 0.38, 0.52}, {0.37, 0.55, 0.80}};
    const int e = E == 128, last = (int)(workgroups % 512);
    return (double)(workgroups / 512) * paired[e][blocks - 1] +
           (last == 0 ? 0. : last <= 256 ? alone[e][blocks - 1] : paired[e][blocks - 1]);
}

// How many of `units` chunks of `blocks` * 64 rows have a workgroup each: all, or those of the whole rounds.  *cost: what
// the launch then takes.  Parts have to come out 4 % cheaper: they read their list and its K and V rows two or three times,
// which the prices of tiles leave out (column lists, parts / whole priced and measured: 8 heads x 57 180, 3 %: 0.99, 1.07;
// 3 x 82 722, 18 %, ragged: 0.98, 1.08; 31 x 14 649, 36 %: 0.99, 1.02; in 220 sizes those priced below 0.96 lost by 2 % at
// most).  Parts are priced as a workgroup per 64 rows; those that pairs of waves walk take 0.7 to 0.97 of that
// (attn_part_form), which only leaves some launches near the line whole.
static int64_t attn_whole_chunks(int E, int blocks, int64_t units, double* cost) {
    const int64_t last = units % 512, rounds = units - last;
    const double whole = attn_rounds_cost(E, blocks, units);
    const double parts = attn_rounds_cost(E, blocks, rounds) + attn_rounds_cost(E, 1, last * blocks);
    const bool in_parts = parts < 0.96 * whole;
    *cost = in_parts ? parts : whole;
    return in_parts ? rounds : units;
}

// How `parts` parts of 64 rows are walked, by the keys each has to walk.  kRows32Shared halves the chain of tiles and has
// twice the workgroups: as long as those find an empty CU (E = 64: two to a CU cost each little).  kRows64Shared takes
// three quarters of the time per step, and a merge of more rows: where the workgroups of 32 rows would meet on the CUs,
// and for long walks. Launches in us of 64 rows, 64 shared and 32 shared, column lists, E = 128:
//     parts  72: 128 keys 5.5, 6.7, 5.1   256 7.0, 8.0, 6.1   512 9.8, 10.1, 8.0   1024 15.7, 14.7, 11.7
//                2048 27.3, 23.8, 19.2
//           180: 256 7.2, 8.0, 8.1   512 9.9, 10.3, 10.9   768 12.7, 12.4, 13.1   1024 15.7, 14.9, 15.9
//                2048 27.5, 23.9, 25.2
//           360: 512 13.5, 15.4, 17.5   1024 21.6, 22.5, 27.4   2048 37.2, 35.8, 45.7
// E = 64:   108: 128 keys 4.5, 5.0, 4.2   512 7.2, 7.3, 6.0
//           180: 384 6.5, 6.8, 6.8   768 9.2, 9.1, 9.0   2048 18.7, 17.0, 16.4
//           360: 1024 13.9, 14.8, 16.4   2048 23.9, 23.8, 27.1
// Every column: E = 128, 192 parts, 512 keys 9.7, 9.3, 9.5; E = 64: 256 5.3, 5.4, 5.0.
// Behind 512 whole chunks, E = 128: 120 parts, 256 keys 29.6, 30.0, 29.3   2048 110.8, 107.2, 104.6
//           192: 512 39.8, 40.8, 42.3   1024 61.1, 60.2, 65.5; E = 64 (192 rows): 192: 1024 40.9, 41.3, 44.7
//                2048 67.9, 66.7, 73.4; every column, E = 64: 189, 960 keys 37.6, 36.0, 39.5.
// Whole chunks of 128 rows at E = 64 have four workgroups to a CU, which the shared walk's registers in the same kernel
// make three (133 and 138 instead of 128 and 122).  That costs a list's whole rounds more than it saves behind them: 512
// chunks and 272 to 400 parts of 2048 to 6000 keys 1.04 to 1.10 of the time, 176 to 248 parts 0.98 to 1.01, behind 1024
// 0.99 to 1.02.  (Held to 128 registers, 6 of them in scratch memory: 0.99 to 1.03.)  Every column comes to 128 rows only
// behind 1024 chunks: 768 to 1700 keys 0.97 to 1.02, from 2304 0.98 to 0.99.
static AttnPart attn_part_form(int E, int rows, int64_t whole, int64_t parts, int keys, bool list) {
    if (parts <= 128) return keys > 3 * kTileRows ? kRows32Shared : kRows64;
    if (whole > 0 && list && E == 64 && rows == 128) return kRows64;
    if (whole > 0) return keys >= (!list ? 768 : E == 128 ? 1024 : 2048) ? kRows64Shared : kRows64;
    if (parts <= 256) {
        if (E == 64) return keys >= (list ? 768 : 256) ? kRows32Shared : kRows64;
        return keys >= (list ? 768 : 512) ? kRows64Shared : kRows64;
    }
    return keys >= 2048 && (!list || E == 128) ? kRows64Shared : kRows64;
}

template <int MODE, int PART>
static int32_t launch_attn_parts_as(const AttnParams& p, int E, int64_t units, hipStream_t s) {
    const int blocks = p.c / 64;
    const int64_t groups = p.whole + (units - p.whole) * blocks * (PART == kRows32Shared ? 2 : 1);
    if (E == 128 && blocks == 3) return launch_attn_variant<128, 3, 4, MODE, PART>(p, groups, s);
    if (E == 128) return launch_attn_variant<128, 2, 4, MODE, PART>(p, groups, s);
    if (blocks == 3) return launch_attn_variant<64, 3, 4, MODE, PART>(p, groups, s);
    constexpr int part = MODE == kColumnList && PART == kRows64Shared ? kRows64 : PART;   // (never asked for: see attn_part_form)
    return launch_attn_variant<64, 2, 4, MODE, part>(p, groups, s);
}

template <int MODE>
static int32_t launch_attn_parts(AttnParams p, int E, int64_t units, hipStream_t s) {
    const int blocks = p.c / 64;
    double cost;
    p.whole = (int)attn_whole_chunks(E, blocks, units, &cost);
    const AttnPart form = attn_part_form(E, p.c, p.whole, (units - p.whole) * blocks, MODE == kColumnList ? p.k_stride : p.N, MODE == kColumnList);
    if (form == kRows32Shared) return launch_attn_parts_as<MODE, kRows32Shared>(p, E, units, s);
    if (form == kRows64Shared) return launch_attn_parts_as<MODE, kRows64Shared>(p, E, units, s);
    return launch_attn_parts_as<MODE, kRows64>(p, E, units, s);
}

// Without a list the rows need not follow the chunks: 128 or 192 at a time, whichever is cheaper.
static int attn_dense_rows(int64_t bh, int N, int E) {
    double cost[2];
    for (int i = 0; i < 2; i++) {
        const int rows = i == 0 ? 192 : 128;
        attn_whole_chunks(E, rows / 64, bh * ((N + rows - 1) / rows), &cost[i]);
    }
    return cost[1] < cost[0] ? 128 : 192;
}

static int32_t launch_attn(const AttnParams& p, int E, int64_t units, hipStream_t s) {
    if (p.idx) return launch_attn_parts<kColumnList>(p, E, units, s);
    const int64_t bh = units / p.NB;
    AttnParams d = p;
    d.c = attn_dense_rows(bh, p.N, E);
    d.NB = (p.N + d.c - 1) / d.c;
    return launch_attn_parts<kEveryColumn>(d, E, bh * d.NB, s);
}

static int32_t launch_attn_fused(const AttnParams& p, int E, int64_t units, hipStream_t s) {
    if (E == 128 && p.c == 192) return launch_attn_variant<128, 3, 4, kFusedDense>(p, units, s);
    if (E == 128 && p.c == 128) return launch_attn_variant<128, 2, 4, kFusedDense>(p, units, s);
    if (E == 64 && p.c == 192) return launch_attn_variant<64, 3, 4, kFusedDense>(p, units, s);
    return launch_attn_variant<64, 2, 4, kFusedDense>(p, units, s);
}

static int32_t launch_attn_blocks(const AttnParams& p, int E, int64_t units, hipStream_t s) {
    if (E == 128 && p.c == 192) return launch_attn_variant<128, 3, 4, kBlockList>(p, units, s);
    if (E == 128 && p.c == 128) return launch_attn_variant<128, 2, 4, kBlockList>(p, units, s);
    if (E == 64 && p.c == 192) return launch_attn_variant<64, 3, 4, kBlockList>(p, units, s);
    return launch_attn_variant<64, 2, 4, kBlockList>(p, units, s);
}

// Into how many pieces the column-sum pass cuts a chunk's keys.  Four workgroups fit a CU, and a CU with three of them takes
// longer than one with two: with few chunks the keys are cut until there are at least eight workgroups per CU, each with at
// least four tiles (each piece's sums are its own, so nothing is merged).  24 heads x 24 chunks x 4608 keys, dense attention
// and sums together: 422 us in one piece, 402 in two, 394 in four (the rule), 399 in eight.
static int colsum_pieces(int64_t units, int N) {
    const int tiles = (N + kColsumTileRows - 1) / kColsumTileRows;
    int pieces = 1;
    while (units * pieces < 8 * 256 && 2 * pieces * 4 <= tiles) pieces *= 2;
    return pieces;
}

static int32_t launch_colsum(ColsumParams cp, int E, int64_t units, hipStream_t s) {
    cp.pieces = colsum_pieces(units, cp.N);
    dim3 grid((unsigned)(units * cp.pieces)), block(256);
    if (E == 128 && cp.c == 192) hipLaunchKernelGGL((attn_colsum_kernel<128, 3>), grid, block, 0, s, cp);
    else if (E == 128 && cp.c == 128) hipLaunchKernelGGL((attn_colsum_kernel<128, 2>), grid, block, 0, s, cp);
    else if (E == 64 && cp.c == 192) hipLaunchKernelGGL((attn_colsum_kernel<64, 3>), grid, block, 0, s, cp);
    else hipLaunchKernelGGL((attn_colsum_kernel<64, 2>), grid, block, 0, s, cp);
    return launch_status();
}

// Shape rules common to the attention entry points.  Offsets of K/V rows inside one head are 32-bit byte offsets.
static int32_t check_attn_shapes(int B, int H, int N, int E, int c, float softmax_scale) {
    if (B < 1 || H < 1 || N < 1) return CHIPMUNK_ERR_SHAPE;
    if (!is_positive_finite_scalar(softmax_scale)) return CHIPMUNK_ERR_SHAPE;
    if (E != 64 && E != 128) return CHIPMUNK_ERR_UNSUPPORTED;
    if (c != 128 && c != 192) return CHIPMUNK_ERR_UNSUPPORTED;
    if ((int64_t)N * E * 2 >= (1LL << 32)) return CHIPMUNK_ERR_SHAPE;
    if ((int64_t)B * H * ((N + c - 1) / c) > 0x7fffffffLL) return CHIPMUNK_ERR_SHAPE;
    return CHIPMUNK_OK;
}

}  // namespace chipmunk

using namespace chipmunk;

extern "C" int32_t chipmunk_attn_sparse_delta(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                              const int32_t* idx, const int32_t* counts,
                                              const uint16_t* base, uint16_t* out, int B, int H, int N,
                                              int E, int c, int k_stride, float softmax_scale,
                                              float o_scale, void* stream) {
    if (!q || !k || !v || !out) return CHIPMUNK_ERR_NULL;
    if ((idx == nullptr) != (counts == nullptr)) return CHIPMUNK_ERR_NULL;
    if (idx && !base) return CHIPMUNK_ERR_NULL;
    if (k_stride < 0 || !is_finite_scalar(o_scale)) return CHIPMUNK_ERR_SHAPE;
    if (int32_t st = check_attn_shapes(B, H, N, E, c, softmax_scale)) return st;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(base) ||
        !aligned16(idx) || !aligned16(counts))
        return CHIPMUNK_ERR_ALIGN;
    int NB = (N + c - 1) / c;
    int64_t units = (int64_t)B * H * NB;
    AttnParams p;
    p.q = q; p.k = k; p.v = v; p.base = base; p.out = out; p.idx = idx; p.counts = counts;
    p.row_m = nullptr; p.row_l = nullptr;
    p.prev_m = nullptr; p.prev_l = nullptr; p.colsum = nullptr; p.ld_colsum = 0;
    p.N = N; p.NB = NB; p.c = c; p.whole = 0; p.by_xcd = attn_by_xcd(N, E); p.k_stride = k_stride;
    p.sl2 = softmax_scale * 1.4426950408889634f;
    p.o_scale = o_scale;
    return launch_attn(p, E, units, (hipStream_t)stream);
}

extern "C" int32_t chipmunk_attn_block_sparse_delta(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                                    const int32_t* blocks, const int32_t* block_counts,
                                                    const uint16_t* base, uint16_t* out, int B, int H, int N,
                                                    int E, int c, int kb_stride, float softmax_scale,
                                                    float o_scale, void* stream) {
    if (!q || !k || !v || !out || !blocks || !block_counts || !base) return CHIPMUNK_ERR_NULL;
    if (kb_stride < 0 || !is_finite_scalar(o_scale)) return CHIPMUNK_ERR_SHAPE;
    if (int32_t st = check_attn_shapes(B, H, N, E, c, softmax_scale)) return st;
    if ((int64_t)kb_stride * kBlockColumns > 0x7fffffffLL) return CHIPMUNK_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(base) ||
        (reinterpret_cast<uintptr_t>(blocks) & 3u) || (reinterpret_cast<uintptr_t>(block_counts) & 3u))
        return CHIPMUNK_ERR_ALIGN;
    int NB = (N + c - 1) / c;
    int64_t units = (int64_t)B * H * NB;
    AttnParams p;
    p.q = q; p.k = k; p.v = v; p.base = base; p.out = out; p.idx = blocks; p.counts = block_counts;
    p.row_m = nullptr; p.row_l = nullptr;
    p.prev_m = nullptr; p.prev_l = nullptr; p.colsum = nullptr; p.ld_colsum = 0;
    p.N = N; p.NB = NB; p.c = c; p.whole = 0; p.by_xcd = attn_by_xcd(N, E); p.k_stride = kb_stride;
    p.sl2 = softmax_scale * 1.4426950408889634f;
    p.o_scale = o_scale;
    return launch_attn_blocks(p, E, units, (hipStream_t)stream);
}

extern "C" size_t chipmunk_attn_dense_workspace_bytes(int B, int H, int N) {
    if (B < 1 || H < 1 || N < 1) return 0;
    return (size_t)B * H * N * 2 * sizeof(float);
}

extern "C" int32_t chipmunk_attn_dense(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out,
                                       float* colsum, int64_t ld_colsum, int B, int H, int N, int E, int c,
                                       float softmax_scale, void* ws, size_t ws_bytes, void* stream) {
    if (!q || !k || !v || !out) return CHIPMUNK_ERR_NULL;
    if (int32_t st = check_attn_shapes(B, H, N, E, c, softmax_scale)) return st;
    if (colsum && ld_colsum < N) return CHIPMUNK_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(colsum) || !aligned16(ws) ||
        (colsum && (ld_colsum % 4) != 0))
        return CHIPMUNK_ERR_ALIGN;
    if (colsum && (!ws || ws_bytes < chipmunk_attn_dense_workspace_bytes(B, H, N))) return CHIPMUNK_ERR_WORKSPACE;
    int NB = (N + c - 1) / c;
    int64_t units = (int64_t)B * H * NB;
    hipStream_t s = (hipStream_t)stream;
    AttnParams p;
    p.q = q; p.k = k; p.v = v; p.base = nullptr; p.out = out; p.idx = nullptr; p.counts = nullptr;
    p.row_m = colsum ? (float*)ws : nullptr;
    p.row_l = colsum ? (float*)ws + (int64_t)B * H * N : nullptr;
    p.prev_m = nullptr; p.prev_l = nullptr; p.colsum = nullptr; p.ld_colsum = 0;
    p.N = N; p.NB = NB; p.c = c; p.whole = 0; p.by_xcd = attn_by_xcd(N, E); p.k_stride = 0;
    p.sl2 = softmax_scale * 1.4426950408889634f;
    p.o_scale = 1.f;
    int32_t st = launch_attn(p, E, units, s);
    if (st != CHIPMUNK_OK || !colsum) return st;
    ColsumParams cp;
    cp.q = q; cp.k = k; cp.row_m = p.row_m; cp.row_l = p.row_l; cp.colsum = colsum; cp.ld = ld_colsum;
    cp.N = N; cp.NB = NB; cp.c = c; cp.sl2 = p.sl2;
    return launch_colsum(cp, E, units, s);
}

extern "C" int32_t chipmunk_attn_colsum_stale(const uint16_t* q, const uint16_t* k, const float* prev_m,
                                              const float* prev_l, float* colsum, int64_t ld_colsum, int B, int H,
                                              int N, int E, int c, float softmax_scale, void* stream) {
    if (!q || !k || !prev_m || !prev_l || !colsum) return CHIPMUNK_ERR_NULL;
    if (int32_t st = check_attn_shapes(B, H, N, E, c, softmax_scale)) return st;
    if (ld_colsum < N) return CHIPMUNK_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(colsum) || (ld_colsum % 4) != 0 ||
        (reinterpret_cast<uintptr_t>(prev_m) & 3u) || (reinterpret_cast<uintptr_t>(prev_l) & 3u))
        return CHIPMUNK_ERR_ALIGN;
    int NB = (N + c - 1) / c;
    int64_t units = (int64_t)B * H * NB;
    ColsumParams cp;
    cp.q = q; cp.k = k; cp.row_m = prev_m; cp.row_l = prev_l; cp.colsum = colsum; cp.ld = ld_colsum;
    cp.N = N; cp.NB = NB; cp.c = c; cp.sl2 = softmax_scale * 1.4426950408889634f;
    return launch_colsum(cp, E, units, (hipStream_t)stream);
}

// A refresh in one kernel has a workgroup per chunk and no other split; apart, the sums come in pieces of the keys and the
// attention in workgroups of 64 rows.  One kernel and apart, us: 48 chunks 4 heads x 2201 x 128 68.5, 47.9; 30, 6 x 826 x 64
// 25.5, 22.6; 78, 13 x 1008 x 64 29.5, 25.2; 96, 16 x 1091 x 128 41.2, 41.8; 110, 22 x 928 x 128 36.3, 38.1, but 10 x 2026 x 128
// 64.7, 63.1; 117, 9 x 2390 x 64 58.0, 50.7 (81 to 121 chunks of 1587 keys and more: 1.03 to 1.34 times, ten sizes).  Short keys
// cost the second launch: 16 chunks, 8 x 199 x 64 15.3, 17.9; 48, 16 x 456 x 64 19.1, 18.7; 78, 26 x 438 x 128 23.1, 24.5.
// The sums' error against 64 bits, one kernel and apart: 2e-7 to 4e-7, 5e-8 to 7e-8 (RMS).
static bool refresh_apart(int64_t units, int N) { return (units <= 80 && N >= 640) || (units <= 120 && N >= 1536); }

// How many of a refresh's chunks the one kernel takes, the first ones; the sums and the attention of the others are made
// apart. More than 120 chunks: apart while the attention's workgroups of 64 rows all have a slot, which long keys make
// worth the second reading; a workgroup of the one kernel is quick with 128 rows at E = 128, so there only while each has
// a CU.  One kernel and apart, E = 64: 128 chunks of 192 rows, 5000 to 6500 keys 0.74 of the time, 160, 2300 to 3000
// 0.89, 170 0.96, 180 1.21; 200 of 128 rows 0.98, 6500 and more 0.84; E = 128: 125 of 128 rows 0.79, 135 1.09; 150 of 192
// rows, 2300 to 3000 keys 1.01, from 4500 0.96, from 6500 0.91; 175 1.2.
// Beyond a round of all slots (three workgroups to a CU at E = 64 with 128 rows, else two): a last round of few chunks
// takes the one kernel more than half as long as a full one.  Apart, last rounds of up to 50, to 75 and to 100 chunks,
// behind one round, E = 128, 192 rows: 2300 to 3500 keys 0.91, 0.92, 0.99 of the time, from 6000 0.86, 0.88, 0.94 (544
// chunks, 17 heads x 6008: 396 and 342 us), up to 1536 keys 0.96, -, 1.07; 128 rows: 1536 to 2300 keys 0.95, 0.97, 1.01,
// from 6000 0.88, 0.91, 0.91; behind two rounds 0.94, 0.95, 0.99 and (128 rows) 0.96, 0.97, 0.99; behind three (up to 60
// chunks) 0.96 to 0.98 and (128 rows) 0.98 to 1.01 below 4000 keys, 0.975 to 0.99 from there; behind four and more the
// workgroups no longer end together: 0.98 to 1.04.  E = 64, 128 rows behind 768: 2300 to 3500 keys 0.98, 1.00, 1.02, from
// 3500 0.95, 0.97, 0.99; behind 1536 0.99 to 1.02.  Last rounds that begin at half of the slots: 0.95 to 1.3.
static int64_t refresh_fused_chunks(int64_t units, int N, int E, int c) {
    if (refresh_apart(units, N)) return 0;
    const int64_t parts = units * (c / 64);
    if (E == 64 ? parts <= 512 && N >= 2300 : c == 192 ? parts <= 512 && N >= 5000 : parts <= 256 && N >= 2300) return 0;
    const bool three = E == 64 && c == 128;
    const int64_t slots = three ? 768 : 512, last = units % slots, rounds = units / slots;
    const int keys = three ? 3500 : c == 128 && rounds == 3 ? 4000 : 2300;
    return rounds >= 1 && rounds <= (three ? 1 : 3) && last <= 80 && N >= keys ? units - last : units;
}

extern "C" int32_t chipmunk_attn_dense_colsum_stale(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                                    uint16_t* out, const float* prev_m, const float* prev_l,
                                                    float* colsum, int64_t ld_colsum, float* new_m, float* new_l,
                                                    int B, int H, int N, int E, int c, float softmax_scale,
                                                    void* stream) {
    if (!q || !k || !v || !out || !prev_m || !prev_l || !colsum) return CHIPMUNK_ERR_NULL;
    if ((new_m == nullptr) != (new_l == nullptr)) return CHIPMUNK_ERR_NULL;
    if (int32_t st = check_attn_shapes(B, H, N, E, c, softmax_scale)) return st;
    if (ld_colsum < N) return CHIPMUNK_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(colsum) || (ld_colsum % 4) != 0)
        return CHIPMUNK_ERR_ALIGN;
    for (const float* f : {prev_m, prev_l, (const float*)new_m, (const float*)new_l})
        if (reinterpret_cast<uintptr_t>(f) & 3u) return CHIPMUNK_ERR_ALIGN;
    int NB = (N + c - 1) / c;
    int64_t units = (int64_t)B * H * NB;
    AttnParams p;
    p.q = q; p.k = k; p.v = v; p.base = nullptr; p.out = out; p.idx = nullptr; p.counts = nullptr;
    p.row_m = new_m; p.row_l = new_l;
    p.prev_m = prev_m; p.prev_l = prev_l; p.colsum = colsum; p.ld_colsum = ld_colsum;
    p.N = N; p.NB = NB; p.c = c; p.whole = 0; p.by_xcd = attn_by_xcd(N, E); p.k_stride = 0;
    p.sl2 = softmax_scale * 1.4426950408889634f;
    p.o_scale = 1.f;
    const hipStream_t s = (hipStream_t)stream;
    const int64_t fused = refresh_fused_chunks(units, N, E, c);
    if (fused > 0) {
        const int32_t st = launch_attn_fused(p, E, fused, s);
        if (st != CHIPMUNK_OK || fused == units) return st;
    }
    // apart, the sums first: the attention may write its statistics over the ones that the sums take
    ColsumParams cp;
    cp.q = q; cp.k = k; cp.row_m = prev_m; cp.row_l = prev_l; cp.colsum = colsum; cp.ld = ld_colsum;
    cp.N = N; cp.NB = NB; cp.c = c; cp.sl2 = p.sl2;
    cp.first = p.first = (int)fused;
    const int32_t st = launch_colsum(cp, E, units - fused, s);
    if (st != CHIPMUNK_OK) return st;
    return fused == 0 ? launch_attn(p, E, units, s) : launch_attn_parts<kEveryColumn>(p, E, units - fused, s);
}

// Whether a refresh is made apart by the number and length of its chunks alone; how many chunks the one kernel takes, by
// all rules.  For the tests, like the next.
extern "C" int32_t chipmunk_internal_attn_refresh_apart(int B, int H, int N, int c) { return refresh_apart((int64_t)B * H * ((N + c - 1) / c), N); }

extern "C" int32_t chipmunk_internal_attn_refresh_fused(int B, int H, int N, int E, int c) {
    return (int32_t)refresh_fused_chunks((int64_t)B * H * ((N + c - 1) / c), N, E, c);
}

// How the chunks that have no workgroup of their own are walked (AttnPart); -1: there are none.
extern "C" int32_t chipmunk_internal_attn_part_form(int B, int H, int N, int E, int c, int k_stride, int list) {
    const int64_t bh = (int64_t)B * H;
    const int rows = list ? c : attn_dense_rows(bh, N, E);
    const int64_t units = bh * ((N + rows - 1) / rows);
    double cost;
    const int64_t whole = attn_whole_chunks(E, rows / 64, units, &cost);
    return whole == units ? -1 : attn_part_form(E, rows, whole, (units - whole) * (rows / 64), list ? k_stride : N, list);
}

// What the rules above choose for these sizes: the rows of a workgroup that takes a whole chunk, the chunks that have one, the
// chunks walked in parts (attn_part_form), and the pieces of the column-sum pass.  Not part of the library's interface:
// for the tests, which have to reach each form and otherwise would not see that a rule has moved.
extern "C" void chipmunk_internal_attn_form(int B, int H, int N, int E, int c, int list, int32_t* out) {
    const int64_t bh = (int64_t)B * H;
    const int rows = list ? c : attn_dense_rows(bh, N, E);
    const int64_t units = bh * ((N + rows - 1) / rows);
    double cost;
    const int64_t whole = attn_whole_chunks(E, rows / 64, units, &cost);
    out[0] = rows;
    out[1] = (int32_t)whole;
    out[2] = (int32_t)(units - whole);
    out[3] = colsum_pieces(bh * ((N + c - 1) / c), N);
}
