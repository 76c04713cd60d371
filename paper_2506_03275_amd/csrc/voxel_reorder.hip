// Voxel token reorder and its inverse (Alg. 1; Sec. 3.2.1) for gfx950.
//
// The permutation has a closed form, so no index table is read: every wave
// computes the source (or destination) row of its token from the grid geometry
// and moves the row with 128-bit (or 32-bit) accesses, five of them in flight.  The copy touches each
// byte once on the way in and once on the way out: it is bound by HBM.
#include "common.h"

#include <algorithm>

namespace chipmunk {

// n / d for 0 <= n < 2^31 as (mulhi(n, m) + n) >> s with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1 (Granlund and
// Montgomery, "Division by invariant integers using multiplication"): three instructions where the compiler's division by a
// run-time number takes about twenty, ten times over before a wave can ask for its row.
struct Divisor {
    uint32_t d, m, s;
    explicit Divisor(int64_t value) : d((uint32_t)(value > 1 ? value : 1)), s(0) {
        while (s < 31 && (1u << s) < d) s++;
        m = (uint32_t)(((((uint64_t)1 << s) - d) << 32) / d) + 1u;
    }
    __device__ __forceinline__ int div(int n) const { return (int)((__umulhi((uint32_t)n, m) + (uint32_t)n) >> s); }
    __device__ __forceinline__ int div_mod(int n, int* rest) const {
        const int q = div(n);
        *rest = n - q * (int)d;
        return q;
    }
};

struct VoxelGeom {
    int n_prefix, H, W;
    int vt, vh, vw;
    int Tf, Hf, Wf;   // extent covered by full voxels in each dimension
    int n_full;       // tokens inside full voxels
    int grid;         // T*H*W
    int N;
    // divisors that a grid without full voxels, or without a remainder, does not reach stand at 1
    Divisor volume, voxels_w, voxels_h, by_vh, by_vw, edge_w, frame_rest, by_w, by_hw, by_n;
};

// position before the reorder of the token that sits at position i after it
__device__ __forceinline__ int voxel_old_position(const VoxelGeom& g, int i) {
    if (i < g.n_prefix) return i;
    int j = i - g.n_prefix;
    if (j >= g.grid) return i;  // suffix
    int t, h, w;
    if (j < g.n_full) {
        int r, wc, hc, dh, dw;
        const int tc = g.voxels_h.div_mod(g.voxels_w.div_mod(g.volume.div_mod(j, &r), &wc), &hc);
        const int dt = g.by_vh.div_mod(g.by_vw.div_mod(r, &dw), &dh);
        t = tc * g.vt + dt;
        h = hc * g.vh + dh;
        w = wc * g.vw + dw;
    } else {
        // remainder, in raster order: inside a frame t < Tf the rows h < Hf give their
        // columns w >= Wf, then the rows h >= Hf are whole; frames t >= Tf are whole.
        int rho = j - g.n_full;
        int edge = g.Hf * (g.W - g.Wf);
        int per_frame = edge + (g.H - g.Hf) * g.W;
        int in_frames = g.Tf * per_frame;
        int r;
        if (rho < in_frames) {
            t = g.frame_rest.div_mod(rho, &r);
            if (r < edge) {
                h = g.edge_w.div_mod(r, &w);
                w += g.Wf;
            } else {
                h = g.Hf + g.by_w.div_mod(r - edge, &w);
            }
        } else {
            t = g.Tf + g.by_hw.div_mod(rho - in_frames, &r);
            h = g.by_w.div_mod(r, &w);
        }
    }
    return g.n_prefix + (t * g.H + h) * g.W + w;
}

__global__ __launch_bounds__(256) void voxel_perm_kernel(VoxelGeom g, int32_t* perm, int32_t* inv_perm) {
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= g.N) return;
    int old = voxel_old_position(g, i);
    if (perm) perm[i] = old;
    if (inv_perm) inv_perm[old] = i;
}

// One wave per row; the waves of the first batch also write the permutation, which would be a launch of its own.  VEC is
// u32x4 (16-byte words) or uint32_t.  STREAM: loads and stores past the caches' usual order of replacement (the rules are at the
// launch).  us before (one word per lane at a time, the permutation by a kernel of its own, plain divisions) and now: 7 MB 9.8, 7.4;
// 25 MB 12.1, 9.6; 69 MB 30.3, 27.7; 290 MB 108, 94.6; 774 MB 293, 259.5 (6.0 TB/s).  U: rows of 10 240 bytes, 812 MB, with 3, 4, 5, 6
// and 8 words of a lane in flight 285, 282, 274, 272, 269; of 6144 bytes 270, 270, 264, 262, 261; small copies alike.
template <typename VEC, bool STREAM>
__global__ __launch_bounds__(256) void voxel_copy_kernel(VoxelGeom g, const VEC* __restrict__ src, VEC* __restrict__ dst, int64_t total_rows,
                                                         int words_per_row, int inverse, int32_t* __restrict__ perm,
                                                         int32_t* __restrict__ inv_perm) {
    constexpr int U = 5;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t wave = (int64_t)blockIdx.x * 4 + w, nwaves = (int64_t)gridDim.x * 4;
    for (int64_t row = wave; row < total_rows; row += nwaves) {
        const int b = total_rows <= 0x7fffffff ? g.by_n.div((int)row) : (int)(row / g.N);
        const int i = (int)(row - (int64_t)b * g.N);
        const int old = voxel_old_position(g, i);
        if (b == 0 && lane == 0) {
            if (perm) perm[i] = old;
            if (inv_perm) inv_perm[old] = i;
        }
        const int64_t from = (int64_t)b * g.N + (inverse ? i : old);
        const int64_t to = (int64_t)b * g.N + (inverse ? old : i);
        const VEC* s = src + from * words_per_row;
        VEC* d = dst + to * words_per_row;
        for (int x = lane; x < words_per_row; x += 64 * U) {   // U words per lane requested before the first is stored
            VEC v[U];
#pragma unroll
            for (int u = 0; u < U; u++)
                if (x + 64 * u < words_per_row) v[u] = STREAM ? __builtin_nontemporal_load(s + x + 64 * u) : s[x + 64 * u];
#pragma unroll
            for (int u = 0; u < U; u++)
                if (x + 64 * u < words_per_row) {
                    if (STREAM) __builtin_nontemporal_store(v[u], d + x + 64 * u);
                    else d[x + 64 * u] = v[u];
                }
        }
    }
}

}  // namespace chipmunk

using namespace chipmunk;

extern "C" int32_t chipmunk_voxel_reorder(const void* src, void* dst, int32_t* perm, int32_t* inv_perm,
                                          int batch, int n_prefix, int T, int H, int W, int n_suffix,
                                          int vt, int vh, int vw, int row_bytes, int inverse, void* stream) {
    if ((src == nullptr) != (dst == nullptr)) return CHIPMUNK_ERR_NULL;
    if (!src && !perm && !inv_perm) return CHIPMUNK_ERR_NULL;
    if (n_prefix < 0 || n_suffix < 0 || T < 1 || H < 1 || W < 1 || vt < 1 || vh < 1 || vw < 1)
        return CHIPMUNK_ERR_SHAPE;
    int64_t N64 = (int64_t)n_prefix + (int64_t)T * H * W + n_suffix;
    if (N64 > 0x7fffffffLL) return CHIPMUNK_ERR_SHAPE;
    if (src && (batch < 1 || row_bytes < 1)) return CHIPMUNK_ERR_SHAPE;
    if (src && (row_bytes % 4) != 0) return CHIPMUNK_ERR_ALIGN;
    if ((reinterpret_cast<uintptr_t>(perm) & 3u) || (reinterpret_cast<uintptr_t>(inv_perm) & 3u) ||
        (reinterpret_cast<uintptr_t>(src) & 3u) || (reinterpret_cast<uintptr_t>(dst) & 3u))
        return CHIPMUNK_ERR_ALIGN;
    if (src) {  // the two buffers must not overlap
        const char* s0 = (const char*)src;
        const char* d0 = (const char*)dst;
        int64_t bytes = (int64_t)batch * N64 * row_bytes;
        if (s0 < d0 + bytes && d0 < s0 + bytes) return CHIPMUNK_ERR_SHAPE;
    }
    const int Tf = (T / vt) * vt, Hf = (H / vh) * vh, Wf = (W / vw) * vw;
    const int64_t rest = (int64_t)Hf * (W - Wf) + (int64_t)(H - Hf) * W;   // of a frame t < Tf
    const bool full = Tf > 0 && Hf > 0 && Wf > 0;
    const VoxelGeom g = {n_prefix, H, W, vt, vh, vw, Tf, Hf, Wf, Tf * Hf * Wf, T * H * W, (int)N64,
                         Divisor(full ? (int64_t)vt * vh * vw : 1), Divisor(Wf / vw), Divisor(Hf / vh), Divisor(full ? vh : 1),
                         Divisor(full ? vw : 1), Divisor(W - Wf), Divisor(rest), Divisor(W), Divisor((int64_t)H * W), Divisor(N64)};
    hipStream_t s = (hipStream_t)stream;
    if (!src) {
        hipLaunchKernelGGL(voxel_perm_kernel, dim3((g.N + 255) / 256), dim3(256), 0, s, g, perm, inv_perm);
        return launch_status();
    }
    const int64_t total_rows = (int64_t)batch * g.N;
    const bool wide = row_bytes % 16 == 0 && aligned16(src) && aligned16(dst);
    const int words = row_bytes / (wide ? 16 : 4);
    // A launch has fewer than 2^32 threads; rows beyond are strided over the waves.  Of rows that are less than one word per lane a
    // wave takes several: its start costs more than such a row.  us with a wave per row and like this: 24 heads x 128 columns of 16
    // bits 12 MiB 15.3, 15.4, 40 MiB 38.8, 30.7, 150 MiB 161, 120, 600 MiB 644, 453; 64 columns 100 MiB 200, 137; 384 columns 600 MiB 254,
    // 240; 448 columns 600 MiB 229, 236.
    const int64_t blocks = std::min<int64_t>((total_rows + 3) / 4, words < 64 ? 1 << 14 : 1 << 22);
    // Past the caches: a source and a destination that do not fit the last-level cache (256 MB) together.  Call alone, with a
    // reader of the destination, and from the writer of the source to that reader, us without and with: 100 MiB 31.9, 35.5; 65.3,
    // 69.2; 106.5, 101.2; 128 MiB 40.5, 44.5; 83.7, 87.9; 142, 132; 140 MiB 47.3, 48.9; 101, 94.9; 153, 144; 180 MiB 70.1, 61.7; 133, 121;
    // 194, 190; 600 MiB 221, 192; 422, 399; 625, 592.  Not shorter rows and not words of 4 bytes, whose stores leave in pieces: 600 MiB of
    // 256 columns 368, 395; 564, 601; 769, 784; of 2510 columns (4-byte words) 250, 261; 451, 471; 653, 662.
    const bool stream_through = wide && words >= 64 && total_rows * row_bytes > (int64_t)128 << 20;
    auto launch = [&](auto kernel, auto from, auto to) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, g, from, to, total_rows, words, inverse, perm, inv_perm);
    };
    if (stream_through) launch(voxel_copy_kernel<u32x4, true>, (const u32x4*)src, (u32x4*)dst);
    else if (wide) launch(voxel_copy_kernel<u32x4, false>, (const u32x4*)src, (u32x4*)dst);
    else launch(voxel_copy_kernel<uint32_t, false>, (const uint32_t*)src, (uint32_t*)dst);
    return launch_status();
}
