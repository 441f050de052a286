// Many steps per launch on a 1D lattice with zero-gradient ends.  Internal
// header (not part of the C ABI), on top of plbm_sweep.h.
//
// A model M gives the storage and arithmetic type T, the number of
// populations Q1, the index I0 of the still one (or -1), the parameters P
// (with nx) and shift / collide of one node.
//
// A workgroup holds one node per thread and takes `steps` steps on it; the
// populations between the steps are exchanged through LDS (two buffers, one
// barrier a step).  Its nodes are the tile's plus reach * (steps - 1) on each
// side, computed again by the neighbours; a tile that holds the whole lattice
// has no such halo and takes up to TUBE_STEPS steps.  The ghost nodes beyond an
// end hold the end node's own post-collision populations, so past the first
// step (whose ghosts are in memory) their pull is a clamped index.
//
// What bounds it: single steps of short lattices take 4.1 us each, 2 us of
// them the kernel, whatever the length; here a step is one trip through LDS
// and one collision.  1000 nodes in FP64, 500 steps: 14 launches of 35 or 36 steps
// on 22 workgroups of 256 threads, 46 of whose nodes are their own; 11.6 us each,
// 0.32 a step (write, barrier, read, collision: vector instructions in 0.38 of the
// issue slots), 1984 -> 161 us a call.  200000 nodes in FP32, 100 steps: 4 launches
// of 25, vector instructions in 0.83 of the slots, 387 -> 59.
#pragma once
#include "plbm_sweep.h"

namespace {

constexpr int TUBE_T = 1024;          // most nodes (threads) of a workgroup
// Most steps of a launch: 0.5 to 3 ms, so that a call of any length is made of
// short kernels, at 4 us for each of them.
constexpr int TUBE_STEPS = 4096;
static_assert(TUBE_STEPS % 2 == 0, "launches in place take an even number of steps");

struct TubePlan {
    int launches;                     // each takes n / launches steps, the first n % launches one more
    int tile;                         // nodes a workgroup writes
    int threads;
    bool whole;                       // one workgroup holds the lattice: TUBE_STEPS steps a launch, in place
};

template <class M>
constexpr size_t tube_lds_bytes(int threads)
{
    return (size_t)2 * (M::Q1 - (M::I0 >= 0 ? 1 : 0)) * threads * sizeof(typename M::T);
}

// The cheapest of a few plans by what was measured on MI355X (D1Q5, us): 4 a
// launch, and per step 0.12 + 0.0005 times the threads a compute unit runs in
// FP64, 0.18 + 0.0003 times in FP32 (64 nodes in one workgroup 0.23 and 0.21,
// 1000 nodes 0.62 and 0.49; on 256 threads and 20 steps a launch 0.40 and
// 0.41).  Whole multiples of 256 threads load the four SIMDs alike: 320
// threads took 0.49 where 256 took 0.40.
template <class M>
inline TubePlan tube_plan(int nx, int n, int reach)
{
    const bool wide = sizeof(typename M::T) == 8;
    const double base = wide ? 0.12 : 0.18, per = wide ? 0.0005 : 0.0003;
    auto cost = [&](const TubePlan &t, int resident) {
        return 4.0 * t.launches + n * (base + per * t.threads * resident);
    };
    TubePlan best = {(n - 1) / TUBE_STEPS + 1, nx, (nx + 63) / 64 * 64, true};
    double least = nx <= TUBE_T ? cost(best, 1) : HUGE_VAL;
    for (int threads = 256; threads <= TUBE_T; threads += 256)
        for (int steps : {1, 8, 12, 16, 20, 24, 32, 40, 48, 64}) {
            TubePlan t = {(n - 1) / steps + 1, 0, threads, false};
            // as many launches, modulo two, as there are steps: the state
            // ends in the buffer where single steps leave it
            if ((t.launches ^ n) & 1) ++t.launches;
            if (t.launches > n) continue;
            t.tile = threads - 2 * reach * ((n - 1) / t.launches);
            if (t.tile < 32) continue;
            const int tiles = (nx - 1) / t.tile + 1;
            const double c = cost(t, (tiles - 1) / SWEEP_CUS + 1);
            if (c < least) {
                least = c;
                best = t;
            }
        }
    return best;
}

template <class M>
__device__ __forceinline__ void tube(const typename M::T *src, typename M::T *dst, const typename M::P &p, int x0,
                                     int x1, int reach, int steps, typename M::T *lds)
{
    using T = typename M::T;
    constexpr int Q1 = M::Q1, COLS = Q1 - (M::I0 >= 0 ? 1 : 0);
    const long long ps = (long long)p.nx + 2 * PLBM_GHOST;
    const int halo = reach * (steps - 1);
    const int lo = max(0, x0 - halo), hi = min(p.nx, x1 + halo);
    const int nodes = hi - lo, stride = blockDim.x;
    const int l = min((int)threadIdx.x, nodes - 1);     // threads past the nodes repeat the last
    T f[Q1];
    int at[Q1];
#pragma unroll
    for (int k = 0; k < Q1; ++k) {
        const int v = M::shift(p, k);
        f[k] = src[k * ps + lo + l + PLBM_GHOST - v];
        at[k] = (M::I0 >= 0 && k > M::I0 ? k - 1 : k) * stride + min(max(l - v, 0), nodes - 1);
    }
    M::collide(f, p);
    T *buf = lds, *other = lds + COLS * stride;
#pragma unroll 1
    for (int s = 1; s < steps; ++s) {
#pragma unroll
        for (int k = 0; k < Q1; ++k)
            if (k != M::I0) buf[(M::I0 >= 0 && k > M::I0 ? k - 1 : k) * stride + l] = f[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < Q1; ++k)
            if (k != M::I0) f[k] = buf[at[k]];
        M::collide(f, p);
        T *const t = buf;
        buf = other;
        other = t;
    }
    const int x = lo + (int)threadIdx.x;
    if (x < x0 || x >= x1) return;
#pragma unroll
    for (int k = 0; k < Q1; ++k) {
        dst[k * ps + x + PLBM_GHOST] = f[k];
        if (x == 0)
            for (int g = 0; g < PLBM_GHOST; ++g) dst[k * ps + g] = f[k];
        if (x == p.nx - 1)
            for (int g = 0; g < PLBM_GHOST; ++g) dst[k * ps + p.nx + PLBM_GHOST + g] = f[k];
    }
}

template <class M>
__global__ __launch_bounds__(TUBE_T) void k_tube(const typename M::T *src, typename M::T *dst, typename M::P p,
                                                 int tile, int reach, int steps)
{
    extern __shared__ __align__(16) unsigned char tube_lds[];
    const int x0 = blockIdx.x * tile;
    tube<M>(src, dst, p, x0, min(x0 + tile, p.nx), reach, steps, reinterpret_cast<typename M::T *>(tube_lds));
}

// Takes n steps and returns n, the result in fa when n is even and in fb when it
// is odd; or none where a launch would take one step and is all it costs, which
// the single step's kernel does faster (D1Q3 FP32 up to 200000 nodes 3.5 us a call,
// 4.1 here; 60 million nodes 298, 266 here).
template <class M>
int run_tube(const typename M::P &p, void *fa, void *fb, int n, int reach, hipStream_t st)
{
    using T = typename M::T;
    if (n < 1) return 0;
    const TubePlan t = tube_plan<M>(p.nx, n, reach);
    if (t.launches == n && (double)p.nx * M::Q1 * sizeof(T) < 1e7) return 0;
    for (int k = 0; k < t.launches; ++k) {
        int steps = n / t.launches + (k < n % t.launches ? 1 : 0);
        T *src = static_cast<T *>((k & 1) ? fb : fa);
        T *dst = static_cast<T *>((k & 1) ? fa : fb);
        if (t.whole) {                // the last takes what is left, an odd number into fb
            const bool last = k == t.launches - 1;
            steps = last ? n - k * TUBE_STEPS : TUBE_STEPS;
            src = static_cast<T *>(fa);
            dst = static_cast<T *>(last && (n & 1) ? fb : fa);
        }
        hipLaunchKernelGGL(k_tube<M>, dim3((p.nx - 1) / t.tile + 1), dim3(t.threads),
                           tube_lds_bytes<M>(t.threads), st, src, dst, p, t.tile, reach, steps);
    }
    return n;
}

} // namespace
