// Several fused steps per launch on a small periodic 2D lattice.  Internal
// header (not part of the C ABI); the models are plbm_sweep.h's.
//
// A workgroup writes the BX x BY output nodes of D steps and holds, one node
// per thread, the region around them that the first step is needed on:
// R (D - 1) nodes more on each side, R = max |v|.  Each step pulls from the
// region the step before left in LDS and is needed on R nodes less a side.
// Values between the steps are held in the storage type, as in plbm_sweep.h,
// so D fused steps give bitwise what D single steps give.
//
// What bounds it: a launch costs about 4 us on a small lattice whatever it
// does, and a sweep goes through its rows one after another; here all nodes
// go at once, at the price of computing the region's margin several times.
// Three steps of D2Q25 FP32 256^2 on 16 x 16 nodes (one workgroup a CU, twice the
// nodes computed that are written) take 9 us: vector instructions in 0.60 of the
// issue slots, the waves waiting 0.42 of their cycles for loads, LDS and barriers.
// Measured (us a step, single -> tiles; 8 x 8 nodes and three steps up to one
// tile per CU, then 16 x 16): D2Q25 64^2 FP64 4.9 -> 2.5, FP32 4.7 -> 2.2, FP16
// 4.5 -> 2.3; 256^2 FP64 6.5 -> 4.1, FP32 4.1 -> 2.8, FP16 5.0 -> 3.2.
#pragma once
#include "plbm_sweep.h"

namespace {

// The region of a tile of M::T populations, one node per thread.
template <class M, int BX, int BY, int D>
struct TileShape {
    static constexpr int R = Lines<M>::R, RX = BX + 2 * R * (D - 1), RY = BY + 2 * R * (D - 1);
    static constexpr int NODES = RX * RY, THREADS = (NODES + 63) / 64 * 64;
    static constexpr size_t LDS = (size_t)M::Q1 * M::Q1 * NODES * sizeof(typename M::T);
    static_assert(THREADS <= 1024 && LDS <= SWEEP_LDS, "the region of a tile fits one workgroup");
};

// Tile b of the lattice, tiles_x to a row of them.
template <class M, int BX, int BY, int D>
__device__ __forceinline__ void tile_steps(const typename M::T *__restrict__ src, typename M::T *__restrict__ dst,
                                           const typename M::P &p, int b, int tiles_x,
                                           typename M::T *__restrict__ lds)
{
    using C = typename M::C;
    using S = TileShape<M, BX, BY, D>;
    constexpr int Q1 = M::Q1, NP = Q1 * Q1;
    const int nx = p.nx, ny = p.ny;
    const int ty = b / tiles_x, tx = b - ty * tiles_x;
    // threads past the region repeat its last node and write nothing
    const int node = min((int)threadIdx.x, S::NODES - 1);
    const int ry = node / S::RX, rx = node - ry * S::RX;
    const int x = wrap_mod(tx * BX - S::R * (D - 1) + rx, nx), y = wrap_mod(ty * BY - S::R * (D - 1) + ry, ny);
    const uint32_t key = M::KEYED ? M::key((uint32_t)y * (uint32_t)nx + (uint32_t)x) : 0u;
    C f[NP];
#pragma unroll
    for (int j = 0; j < Q1; ++j) {
        int ys = y - M::V[j];
        ys += (ys < 0) ? ny : 0;
        ys -= (ys >= ny) ? ny : 0;
#pragma unroll
        for (int i = 0; i < Q1; ++i) {
            int xs = x - M::V[i];
            xs += (xs < 0) ? nx : 0;
            xs -= (xs >= nx) ? nx : 0;
            f[i + Q1 * j] = M::dec(src[(ys * NP + i + Q1 * j) * nx + xs], i + Q1 * j, p);
        }
    }
    M::collide(f, p);
#pragma unroll
    for (int s = 1; s < D; ++s) {
        if (s > 1) lds_barrier();
#pragma unroll
        for (int k = 0; k < NP; ++k) lds[k * S::NODES + node] = M::enc(f[k], k, p, key);
        lds_barrier();
        if (rx >= s * S::R && rx < S::RX - s * S::R && ry >= s * S::R && ry < S::RY - s * S::R) {
#pragma unroll
            for (int j = 0; j < Q1; ++j)
#pragma unroll
                for (int i = 0; i < Q1; ++i)
                    f[i + Q1 * j] = M::dec(lds[(i + Q1 * j) * S::NODES + node - M::V[j] * S::RX - M::V[i]],
                                           i + Q1 * j, p);
            M::collide(f, p);
        }
    }
    const int ox = rx - S::R * (D - 1), oy = ry - S::R * (D - 1);
    if ((int)threadIdx.x >= S::NODES || ox < 0 || ox >= BX || oy < 0 || oy >= BY || tx * BX + ox >= nx ||
        ty * BY + oy >= ny)
        return;
#pragma unroll
    for (int k = 0; k < NP; ++k) store_stream<false>(M::enc(f[k], k, p, key), &dst[(y * NP + k) * nx + x]);
}

template <class M, int BX, int BY, int D>
__global__ __launch_bounds__((TileShape<M, BX, BY, D>::THREADS)) void
k_tile(const typename M::T *__restrict__ src, typename M::T *__restrict__ dst, typename M::P p, int tiles_x)
{
    extern __shared__ __align__(16) unsigned char tile_lds[];
    tile_steps<M, BX, BY, D>(src, dst, p, xcd_tile(blockIdx.x, gridDim.x), tiles_x,
                             reinterpret_cast<typename M::T *>(tile_lds));
}

// Launches of fused steps fa -> fb -> fa ..; the state ends in the buffer where
// single steps leave it (see fused_launches).
template <class M>
class TileRun {
public:
    TileRun(const typename M::P &p, void *fa, void *fb, hipStream_t st) : p_(p), buf_{fa, fb}, st_(st) {}
    int launches() const { return launches_; }

    // whether one tile per compute unit holds the lattice
    template <int BX, int BY>
    bool one_round() const
    {
        return (long long)((p_.nx + BX - 1) / BX) * ((p_.ny + BY - 1) / BY) <= SWEEP_CUS;
    }
    // whether they are faster than single steps (see LaunchTime)
    template <int BX, int BY, int D>
    bool pay(const LaunchTime &t) const
    {
        const double tiles = (double)((p_.nx + BX - 1) / BX) * ((p_.ny + BY - 1) / BY);
        return t.us(std::ceil(tiles / SWEEP_CUS), (double)p_.nx * p_.ny) < D * single_us<M>(p_.nx, p_.ny);
    }
    // as many of n steps as launches of D take; n becomes what is left
    template <int BX, int BY, int D>
    void take(int &n)
    {
        const int count = fused_launches<D>(n);
        for (int k = 0; k < count; ++k) launch<BX, BY, D>();
        n -= count * D;
    }

private:
    template <int BX, int BY, int D>
    void launch()
    {
        using S = TileShape<M, BX, BY, D>;
        using T = typename M::T;
        const int tiles_x = (p_.nx + BX - 1) / BX, tiles_y = (p_.ny + BY - 1) / BY;
        hipLaunchKernelGGL((k_tile<M, BX, BY, D>), dim3(tiles_x * tiles_y), dim3(S::THREADS), S::LDS, st_,
                           (const T *)buf_[launches_ & 1], (T *)buf_[~launches_ & 1], p_, tiles_x);
        ++launches_;
    }
    const typename M::P &p_;
    void *buf_[2];
    hipStream_t st_;
    int launches_ = 0;
};

// Most nodes of a lattice taken by tiles: their indices are 32 bits wide.
constexpr long long TILE_NODES = 1 << 20;

} // namespace
