// Runs a kernel's source on the CPU: every thread of a workgroup is a fibre, and each operation between the lanes of a wave, or
// between the waves of a workgroup, is a point that all of them reach before one goes on.  For kernels whose lanes reach these
// operations together.  Of the cross-lane operations only those that the kernels under test use are here.
#pragma once
#include <math.h>
#include <stdint.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <vector>

#include "chipmunk.h"

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct float4 { float x, y, z, w; };
struct int4 { int x, y, z, w; };
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
typedef void* hipStream_t;
enum { hipSuccess = 0, hipFuncAttributeMaxDynamicSharedMemorySize = 0 };
inline int hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }

namespace lanes {

struct Meeting { unsigned arrived = 0, round = 0; };
struct Fibre {
    ucontext_t context;
    std::vector<char> stack;
    bool done = false;
};
inline std::vector<Fibre> fibres;
inline ucontext_t scheduler;
inline unsigned current, threads;
inline Meeting barrier;
inline std::vector<Meeting> waves;
inline std::vector<uint64_t> published[2];
inline dim3 block;
inline std::function<void()> body;

inline void meet(Meeting& m, unsigned of) {
    const unsigned round = m.round;
    if (++m.arrived == of) {
        m.arrived = 0;
        m.round++;
    }
    while (m.round == round) swapcontext(&fibres[current].context, &scheduler);
}
// what every lane of the wave gave, by lane (two sets in turn: a lane may be at the next operation before another has read)
inline const uint64_t* exchange(uint64_t mine) {
    const unsigned me = current;
    Meeting& wave = waves[me / 64];
    std::vector<uint64_t>& set = published[wave.round & 1];
    set[me] = mine;
    meet(wave, 64);
    return &set[me / 64 * 64];
}
inline void trampoline() {
    body();
    fibres[current].done = true;
    swapcontext(&fibres[current].context, &scheduler);
}
template <typename Kernel, typename... Args>
void launch(Kernel kernel, dim3 grid, dim3 group, Args... args) {
    threads = group.x;
    fibres.assign(threads, Fibre());
    for (Fibre& f : fibres) f.stack.resize(1 << 16);
    for (int i = 0; i < 2; i++) published[i].assign(threads, 0);
    body = [=] { kernel(args...); };
    for (block.x = 0; block.x < grid.x; block.x++) {
        waves.assign(threads / 64, Meeting());
        barrier = Meeting();
        for (Fibre& f : fibres) {
            f.done = false;
            getcontext(&f.context);
            f.context.uc_stack.ss_sp = f.stack.data();
            f.context.uc_stack.ss_size = f.stack.size();
            makecontext(&f.context, trampoline, 0);
        }
        for (bool more = true; more;) {
            more = false;
            for (current = 0; current < threads; current++) {
                if (!fibres[current].done) swapcontext(&scheduler, &fibres[current].context);
                more |= !fibres[current].done;
            }
        }
    }
}
// an array that counts the accesses beyond its end
inline int overruns;
template <typename T, unsigned N>
struct Checked {
    T values[N + 1];
    T& operator[](unsigned i) {
        overruns += i >= N;
        return values[std::min(i, N)];
    }
};
struct Thread { struct { operator unsigned() const { return current; } } x; };
struct Block { struct { operator unsigned() const { return block.x; } } x; };

inline int dpp(int old, int mine, int control) {   // row_shr:1 to row_shr:15
    const uint64_t* all = exchange((uint32_t)mine);
    const int lane = current & 63, from = control & 15;
    return (lane & 15) >= from ? (int)(uint32_t)all[lane - from] : old;
}
inline uint64_t ballot(bool mine) {
    const uint64_t* all = exchange(mine);
    uint64_t bits = 0;
    for (int i = 0; i < 64; i++) bits |= all[i] << i;
    return bits;
}
inline int lane_of(int mine, int lane) { return (int)(uint32_t)exchange((uint32_t)mine)[lane]; }
inline uint32_t below(uint32_t who, uint32_t base, int first) {
    const int n = std::clamp((int)(current & 63) - first, 0, 32);
    return base + (uint32_t)__builtin_popcountll(who & ((1ull << n) - 1));
}
template <typename T> T add(T* at, T v) { T old = *at; *at = old + v; return old; }
template <typename T> T set_bits(T* at, T v) { T old = *at; *at = old | v; return old; }
template <typename T> T keep_bits(T* at, T v) { T old = *at; *at = old & v; return old; }

}  // namespace lanes

static lanes::Thread threadIdx;
static lanes::Block blockIdx;

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __syncthreads() lanes::meet(lanes::barrier, lanes::threads)
#define __float_as_uint(x) __builtin_bit_cast(uint32_t, (float)(x))
#define __uint_as_float(x) __builtin_bit_cast(float, (uint32_t)(x))
#define __builtin_amdgcn_update_dpp(old, v, control, rows, banks, bound) lanes::dpp(old, v, control)
#define __shfl_xor(v, mask) lanes::lane_of(v, (int)(lanes::current & 63) ^ (mask))
#define __clz(v) ((v) ? __builtin_clz(v) : 32)
#define __popc(v) __builtin_popcount(v)
#define __ffs(v) __builtin_ffs(v)
#define __builtin_amdgcn_readlane(v, lane) lanes::lane_of(v, lane)
#define __builtin_amdgcn_readfirstlane(v) lanes::lane_of(v, 0)
#define __builtin_amdgcn_ballot_w64(v) lanes::ballot(v)
#define __builtin_amdgcn_mbcnt_lo(who, base) lanes::below(who, base, 0)
#define __builtin_amdgcn_mbcnt_hi(who, base) lanes::below(who, base, 32)
#define __builtin_amdgcn_fmed3f(a, b, c) fmaxf(fminf(a, b), fminf(fmaxf(a, b), c))
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() lanes::exchange(0)
#define atomicAdd lanes::add<uint32_t>
#define atomicOr lanes::set_bits<uint32_t>
#define atomicAnd lanes::keep_bits<uint32_t>
#define hipLaunchKernelGGL(kernel, grid, group, lds, stream, ...) lanes::launch(kernel, grid, group, __VA_ARGS__)

using std::max;
using std::min;

namespace chipmunk {
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
inline int32_t launch_status() { return 0; }
inline uint32_t smem[40960];
}  // namespace chipmunk

extern "C" int host_lanes_overruns() {   // since the last call of it
    const int n = lanes::overruns;
    lanes::overruns = 0;
    return n;
}
extern "C" int host_lanes_barriers() { return (int)lanes::barrier.round; }   // that the last workgroup passed
