// libplbm device code for gfx950: the fused collide-and-stream step of the
// parametric lattice Boltzmann method (arXiv:1402.5487, Eq. srt with the
// equilibrium of Eq. eqdist / Eq. rdr), initialisation, moments and the FP64
// invariant reductions, plus the C-ABI launchers that validate and enqueue
// them.
//
// Design (memory-bound streaming kernel, measured on MI355X):
//  * Pull scheme with A/B buffers: each node gathers population k from
//    src_k(x - v_k) and writes its post-collision value to dst_k(x), so every
//    population is read once and written once per step with wave-contiguous
//    addresses, and the step is race-free by construction.
//  * Row-interleaved layout (y * q + k) * nx + x: the 25 rows one output row
//    reads come from seven contiguous blocks and its 25 writes form one
//    contiguous block, far fewer concurrent DRAM streams than 25 separate
//    planes (measured +10-15% bandwidth).
//  * One workgroup per tile of 256 nodes of one row (four wave64 side by
//    side).  Tiles are numbered so that each of the eight XCDs gets a
//    contiguous run: neighbouring tiles, whose shifted windows share cache
//    lines at their edges, meet in the same L2.  Resident workgroups per CU
//    are capped (see PLBM_LDS_CAP_*).
//  * Addressing: per output row the wave computes five scalar row bases (one
//    per y velocity, periodic wrap applied to the uniform row index) and each
//    lane keeps five 32-bit offsets (one per x velocity), so each of the 50
//    accesses is a scalar base plus a vector offset.  Only the waves whose
//    windows cross the periodic seam in x take a per-node wrapped path.
//  * Calls of several steps take two or three per launch, larger lattices on
//    strips (plbm_sweep.h), smaller ones on tiles (plbm_tile.h): the populations
//    between the steps stay in LDS and registers and are read and written once.
//  * Arithmetic per node: column/row sums give rho, j and sum f|v|^2; the
//    Maxwell moments follow mu_(n+1) = u mu_n + n theta mu_(n-1); the 1D rule
//    r = C mu uses the reduced table of a symmetric velocity set; f_eq =
//    rho r^x_i r^y_j, with the relaxation folded into a_i = omega rho r^x_i
//    so each population costs one multiply and one FMA.  FP64 storage
//    computes in FP64; the other forms compute in FP32.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include <mutex>

#include "plbm_device.h"
#include "plbm_internal.h"
#include "plbm_sweep.h"
#include "plbm_tile.h"
#include "plbm_tube.h"

// Scratch of the calls that ask for sums, one array for plbm_step_noalloc and one
// for the others: the per-workgroup FP64 partial sums of the launch (at most
// NOALLOC_BLOCKS workgroups, four doubles each) and the four reduced sums behind
// them; one call at a time holds an array (see sums_begin).  Each GPU the library
// runs on holds its own copies until the process ends.  Every workgroup of a
// sums launch writes its own four partials before the reduction reads them, so
// nothing in it has to start at zero.  Host code must not use this name as a device address: it
// takes the address hipGetSymbolAddress returns for the current device.
constexpr int NOALLOC_BLOCKS = 8192;
constexpr int SCRATCH_ELEMS = (NOALLOC_BLOCKS + 1) * 4;
static __device__ __align__(256) double scratch[2 * SCRATCH_ELEMS];

namespace {

// The step launch: either one block per tile, or (persistent) a grid of a
// few blocks per CU that walk the tiles in order, block b taking tile
// it * gridDim.x + (b's slot); a slot maps the eight XCDs to eight contiguous
// runs of tiles, so the blocks sharing an L2 work on neighbouring tiles and
// all blocks sweep memory together.  Every block ends when its next tile
// index passes ntiles.
template <class S, int NV, bool SUMS, bool NTS>
__global__ __launch_bounds__(TX, PLBM_MIN_WAVES) void k_step2d(const typename S::T *__restrict__ src,
                                                               typename S::T *__restrict__ dst,
                                                               KParams p,
                                                               double *__restrict__ partials)
{
    LaneSums<4> sums;
    const int slot = xcd_tile(blockIdx.x, gridDim.x);
#pragma unroll 1
    for (int tile = slot; tile < p.ntiles; tile += gridDim.x) {
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        step_tile<S, NV, SUMS, NTS>(src, dst, p, tile, acc);
        if constexpr (SUMS) sums.add(acc);
    }
    if constexpr (SUMS) sums.store(partials + (size_t)blockIdx.x * 4);
}

// The same step, also writing the pre-collision fields of the state it reads
// (the moments its collision uses, in its arithmetic).
template <class S, int NV, bool NTS>
__global__ __launch_bounds__(TX, PLBM_MIN_WAVES) void k_step2d_fields(const typename S::T *__restrict__ src,
                                                                      typename S::T *__restrict__ dst,
                                                                      KParams p, FieldsOut fo)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int slot = xcd_tile(blockIdx.x, gridDim.x);
#pragma unroll 1
    for (int tile = slot; tile < p.ntiles; tile += gridDim.x)
        step_tile<S, NV, false, NTS, true>(src, dst, p, tile, acc, fo);
}

// Two or three steps in one launch (plbm_sweep.h).
template <class S, int D, bool NTS, bool FIELDS>
__global__ __launch_bounds__(sweep_threads<Thermal25<S>>(), (sweep_per_cu<Thermal25<S>, D>())) void
k_step2d_sweep(const typename S::T *__restrict__ src, typename S::T *__restrict__ dst, KParams p, SweepGrid g,
              FieldsOut fo)
{
    extern __shared__ __align__(16) unsigned char sweep_lds[];
    sweep<Thermal25<S>, D, NTS, FIELDS>(src, dst, p, g, xcd_tile(blockIdx.x, gridDim.x),
                                        reinterpret_cast<typename S::T *>(sweep_lds), fo);
}

// ---------------------------------------------------------------------------
// 2D initialisation: the buffer whose pull is f_eq.  Node x computes its own
// equilibrium and scatters population k to x - v_k, so that pulling it back
// from x - v_k returns f_eq_k(x).  The equilibrium is evaluated in FP64 and
// rounded once into the storage type.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void equilibrium2d(double rho, double ux, double uy, double th,
                                              const KParams &p, double (&feq)[NQ])
{
    double rx[Q], ry[Q];
    rule1d<Fp64Math>(ux, th, p, rx);
    rule1d<Fp64Math>(uy, th, p, ry);
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int i = 0; i < Q; ++i) feq[i + Q * j] = rho * rx[i] * ry[j];
}

template <class S>
__global__ __launch_bounds__(TX) void k_init2d(const double *__restrict__ rho,
                                               const double *__restrict__ ux,
                                               const double *__restrict__ uy,
                                               const double *__restrict__ th,
                                               typename S::T *__restrict__ dst, KParams p)
{
    const int segs = (p.nx + TX - 1) / TX;
    const long long total = (long long)segs * p.ny;
#pragma unroll 1
    for (long long t = blockIdx.x; t < total; t += gridDim.x) {
        const int y = (int)(t / segs);
        const int x = (int)(t - (long long)y * segs) * TX + threadIdx.x;
        if (x >= p.nx) continue;
        const long long n = (long long)y * p.nx + x;    // fields are (ny, nx) row-major
        double feq[NQ];
        equilibrium2d(rho[n], ux[n], uy[n], th[n], p, feq);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            int yd = y - p.sx[j];
            yd += (yd < 0) ? p.ny : 0;
            yd -= (yd >= p.ny) ? p.ny : 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                int xd = x - p.sx[i];
                xd += (xd < 0) ? p.nx : 0;
                xd -= (xd >= p.nx) ? p.nx : 0;
                const int k = i + Q * j;
                dst[k * p.pstride + (long long)yd * p.rstride + xd] =
                    S::enc((typename S::C)feq[k], k, p, S::key((uint32_t)n));
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 2D moments of the pulled (pre-collision) state, in FP64.
// ---------------------------------------------------------------------------
template <class S>
__global__ __launch_bounds__(TX) void k_moments2d(const typename S::T *__restrict__ src, KParams p,
                                                  double *__restrict__ rho, double *__restrict__ ux,
                                                  double *__restrict__ uy, double *__restrict__ th,
                                                  double *__restrict__ partials)
{
    LaneSums<4> sums;
    const int segs = (p.nx + TX - 1) / TX;
    const long long total = (long long)segs * p.ny;
#pragma unroll 1
    for (long long t = blockIdx.x; t < total; t += gridDim.x) {
        const int y = (int)(t / segs);
        const int x = (int)(t - (long long)y * segs) * TX + threadIdx.x;
        if (x >= p.nx) continue;
        double f[NQ];
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            int ys = y - p.sx[j];
            ys += (ys < 0) ? p.ny : 0;
            ys -= (ys >= p.ny) ? p.ny : 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                int xs = x - p.sx[i];
                xs += (xs < 0) ? p.nx : 0;
                xs -= (xs >= p.nx) ? p.nx : 0;
                const int k = i + Q * j;
                f[k] = (double)S::dec(src[k * p.pstride + (long long)ys * p.rstride + xs], k, p);
            }
        }
        double r, jx, jy, e;
        sums2d<Fp64Math>(f, p, r, jx, jy, e);
        const double inv = 1.0 / r;
        const double u = jx * inv, w = jy * inv;
        const long long n = (long long)y * p.nx + x;
        if (rho) rho[n] = r;
        if (ux) ux[n] = u;
        if (uy) uy[n] = w;
        if (th) th[n] = 0.5 * (e * inv - u * u - w * w);
        const double all[4] = {r, jx, jy, e};
        sums.add(all);
    }
    if (partials) sums.store(partials + (size_t)blockIdx.x * 4);
}

// ---------------------------------------------------------------------------
// 1D (D1Q5) kernels on the ghost-padded layout: node x at x + 3.
// ---------------------------------------------------------------------------
template <class S>
__device__ __forceinline__ void collide1d(typename S::C (&f)[Q], const KParams &p)
{
    using C = typename S::C;
    const SymRule<C> &R = S::R(p);
    const C rho = (f[0] + (f[1] + f[2])) + (f[3] + f[4]);
    const C j = fma(R.a, f[1] - f[2], R.b * (f[3] - f[4]));
    const C e = fma(R.a2, f[1] + f[2], R.b2 * (f[3] + f[4]));
    const C inv = C(1) / rho;
    const C u = j * inv;
    const C theta = e * inv - u * u;
    C r[Q];
    rule1d<S>(u, theta, p, r);
    const C w = R.omega;
    const C keep = C(1) - w, wr = w * rho;
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = fma(keep, f[i], wr * r[i]);
}

// One step, optionally with the FP64 sums of what it stores (several: plbm_tube.h).
template <class S, bool SUMS>
__global__ __launch_bounds__(TX) void k_step1d(const typename S::T *__restrict__ src,
                                               typename S::T *__restrict__ dst, KParams p,
                                               double *__restrict__ partials)
{
    using C = typename S::C;
    const int x = blockIdx.x * TX + threadIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (x < p.nx) {
        C f[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k)
            f[k] = S::dec(src[k * p.pstride + x + PLBM_GHOST - p.sx[k]], k, p);
        collide1d<S>(f, p);
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const auto h = S::enc(f[k], k, p, (uint32_t)x);
            dst[k * p.pstride + x + PLBM_GHOST] = h;
            // zero-gradient ends: ghosts take the edge node's post-collision value
            if (x == 0)
                for (int g = 0; g < PLBM_GHOST; ++g) dst[k * p.pstride + g] = h;
            if (x == p.nx - 1)
                for (int g = 0; g < PLBM_GHOST; ++g) dst[k * p.pstride + p.nx + PLBM_GHOST + g] = h;
        }
        if constexpr (SUMS) {
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                const double g = (double)S::dec(S::enc(f[k], k, p, (uint32_t)x), k, p);
                const double vk = (double)p.sx[k];
                acc[0] += g; acc[1] += g * vk; acc[3] += g * vk * vk;
            }
        }
    }
    if constexpr (SUMS) block_sums_store<4>(acc, partials + (size_t)blockIdx.x * 4);
}

// Many steps per launch (plbm_tube.h).
template <class S>
struct Thermal5 {
    using T = typename S::T;
    using P = KParams;
    static constexpr int Q1 = Q, I0 = 0;
    static __device__ __forceinline__ int shift(const P &p, int k) { return p.sx[k]; }
    static __device__ __forceinline__ void collide(T (&f)[Q], const P &p) { collide1d<S>(f, p); }
};

template <class S>
__global__ __launch_bounds__(TX) void k_init1d(const double *__restrict__ rho,
                                               const double *__restrict__ ux,
                                               const double *__restrict__ th,
                                               typename S::T *__restrict__ dst, KParams p)
{
    // padded index q holds node y = q - 3; population k there must be
    // f_eq_k(y + v_k) so that the pull at y + v_k returns it.
    const int q = blockIdx.x * TX + threadIdx.x;
    if (q >= p.nx + 2 * PLBM_GHOST) return;
    const int y = q - PLBM_GHOST;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        int s = y + p.sx[k];
        s = s < 0 ? 0 : (s >= p.nx ? p.nx - 1 : s);   // never pulled; kept finite
        double r[Q];
        rule1d<Fp64Math>(ux[s], th[s], p, r);
        dst[k * p.pstride + q] = S::enc((typename S::C)(rho[s] * r[k]), k, p, (uint32_t)q);
    }
}

template <class S>
__global__ __launch_bounds__(TX) void k_moments1d(const typename S::T *__restrict__ src, KParams p,
                                                  double *__restrict__ rho, double *__restrict__ ux,
                                                  double *__restrict__ th,
                                                  double *__restrict__ partials)
{
    const int x = blockIdx.x * TX + threadIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (x < p.nx) {
        double r = 0.0, j = 0.0, e = 0.0;
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const double f = (double)S::dec(src[k * p.pstride + x + PLBM_GHOST - p.sx[k]], k, p);
            const double vk = (double)p.sx[k];
            r += f;
            j += f * vk;
            e += f * vk * vk;
        }
        const double u = j / r;
        if (rho) rho[x] = r;
        if (ux) ux[x] = u;
        if (th) th[x] = e / r - u * u;
        acc[0] = r; acc[1] = j; acc[3] = e;
    }
    if (partials) block_sums_store<4>(acc, partials + (size_t)blockIdx.x * 4);
}

// ---------------------------------------------------------------------------
// Deviation scales: per-plane max |f_eq_k - rho0 w_k| over the nodes.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(TX) void k_devmax2d(const double *__restrict__ rho,
                                                 const double *__restrict__ ux,
                                                 const double *__restrict__ uy,
                                                 const double *__restrict__ th, KParams p,
                                                 const double *__restrict__ base,
                                                 double *__restrict__ partials)
{
    __shared__ double red[NQ][TX / 64];
    double m[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) m[k] = 0.0;
    const int segs = (p.nx + TX - 1) / TX;
    const long long total = (long long)segs * p.ny;
#pragma unroll 1
    for (long long t = blockIdx.x; t < total; t += gridDim.x) {
        const int y = (int)(t / segs);
        const int x = (int)(t - (long long)y * segs) * TX + threadIdx.x;
        if (x >= p.nx) continue;
        const long long n = (long long)y * p.nx + x;
        double feq[NQ];
        equilibrium2d(rho[n], ux[n], uy[n], th[n], p, feq);
#pragma unroll
        for (int k = 0; k < NQ; ++k) m[k] = fmax(m[k], fabs(feq[k] - base[k]));
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        double v = m[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
        if (lane == 0) red[k][wv] = v;
    }
    __syncthreads();
    if (threadIdx.x < NQ) {
        double v = 0.0;
        for (int w = 0; w < TX / 64; ++w) v = fmax(v, red[threadIdx.x][w]);
        partials[(size_t)blockIdx.x * NQ + threadIdx.x] = v;
    }
}

// ---------------------------------------------------------------------------
// Host helpers
// ---------------------------------------------------------------------------
inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

thread_local char g_last_error[160] = "";

int hip_ok(hipError_t e)
{
    if (e == hipSuccess) return PLBM_OK;
    std::snprintf(g_last_error, sizeof(g_last_error), "%s (%d)", hipGetErrorString(e), (int)e);
    return PLBM_EHIP;
}

// The runtime's last-error slot is per thread and sticky: clear whatever an
// earlier, unrelated call left there before launching, then read it back.
inline void clear_launch_error() { (void)hipGetLastError(); }
inline int launch_status() { return hip_ok(hipGetLastError()); }

// Each device's scratch arrays: who holds one, and its device address, looked up
// once (with that device current) and kept.  plbm_step_noalloc's own comes first:
// a call that may not allocate waits for others of its kind only, never for the
// end of a plbm_step on another stream.
constexpr int MAX_DEVICES = 64;
struct Scratch {
    std::mutex mu;
    double *dev = nullptr;
};
Scratch g_scratch[2][MAX_DEVICES];

// The address of the current device's scratch of a kind, whose lock the caller
// holds.
int scratch_address(Scratch &s, int kind)
{
    if (s.dev) return PLBM_OK;
    void *ptr = nullptr;
    const int rc = hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (rc != PLBM_OK) return rc;
    if (!ptr) return PLBM_EHIP;
    s.dev = static_cast<double *>(ptr) + kind * SCRATCH_ELEMS;
    return PLBM_OK;
}

// Takes plbm_step_noalloc's scratch of the current device, waiting for whoever
// holds it.
int scratch_wait(plbm::SumsArea &a)
{
    int dev = -1;
    int rc = hip_ok(hipGetDevice(&dev));
    if (rc != PLBM_OK) return rc;
    if (dev < 0 || dev >= MAX_DEVICES) return PLBM_EUNSUPPORTED;
    Scratch &s = g_scratch[0][dev];
    s.mu.lock();
    rc = scratch_address(s, 0);
    if (rc != PLBM_OK) {
        s.mu.unlock();
        return rc;
    }
    a.part = s.dev;
    a.held = &s.mu;
    return PLBM_OK;
}

// Workgroups of a 2D launch over `tiles` tiles or row segments; max_blocks
// caps the grid (the kernels walk the remaining tiles in a grid-stride loop).
inline int grid_capped(long long tiles, int max_blocks)
{
    return std::min(grid_for(tiles), max_blocks);
}

template <class S, bool SUMS>
int launch_step(const KParams &p, const plbm_desc *d, const void *src, void *dst, double *partials,
                hipStream_t st, int &nblocks, int max_blocks = MAX_GRID)
{
    using T = typename S::T;
    clear_launch_error();
    if (d->dim == 2) {
        nblocks = grid_capped(p.ntiles, max_blocks);
        const size_t lds = sizeof(T) == 2 ? (d->rounding == PLBM_ROUND_STOCHASTIC ? PLBM_LDS_CAP_16SR
                                                                                 : PLBM_LDS_CAP_16)
                                          : PLBM_LDS_CAP_WIDE;
        const bool nts = single_step_nt(p.nx, p.ny, NQ, sizeof(T));
        auto *kernel = p.nv == 2 ? (nts ? k_step2d<S, 2, SUMS, true> : k_step2d<S, 2, SUMS, false>)
                                 : (nts ? k_step2d<S, 1, SUMS, true> : k_step2d<S, 1, SUMS, false>);
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(TX), lds, st, (const T *)src, (T *)dst, p, partials);
    } else if constexpr (sizeof(T) >= 4) {
        nblocks = (p.nx + TX - 1) / TX;
        hipLaunchKernelGGL((k_step1d<S, SUMS>), dim3(nblocks), dim3(TX), 0, st, (const T *)src, (T *)dst, p, partials);
    }
    return launch_status();
}

// D fused steps src -> dst.
template <class S, int D, bool FIELDS>
int launch_sweep(const KParams &p, const void *src, void *dst, hipStream_t st, FieldsOut fo = FieldsOut{})
{
    using T = typename S::T;
    using M = Thermal25<S>;
    const SweepGrid g = sweep_grid<M, D>(p.nx, p.ny);
    clear_launch_error();
    auto *kernel = rows_on_lines(p.nx, sizeof(T)) ? k_step2d_sweep<S, D, true, FIELDS>
                                                  : k_step2d_sweep<S, D, false, FIELDS>;
    hipLaunchKernelGGL(kernel, dim3(g.wgs), dim3(sweep_threads<M>()), (sweep_lds_bytes<M, D>()), st,
                       (const T *)src, (T *)dst, p, g, fo);
    return launch_status();
}

template <class S>
int run_steps(const KParams &p, const plbm_desc *d, void *fa, void *fb, int nsteps, const plbm::StepCall &call,
              hipStream_t st);

// Of n steps in launches of three, those that pairs take instead, an even number
// of pairs (see fused_launches): a step or two left over cost more (FP32 4096^2:
// three 675 us, a pair 624, one 600).
inline int pairs_beside_threes(int n)
{
    const int pairs = n % 3 == 0 ? 0 : n % 3 == 1 ? 2 : 4;
    return std::min(pairs, fused_launches<2>(n));
}

// Launches of D, fa -> fb -> ..
template <class S, int D>
int run_sweeps(const KParams &p, void *fa, void *fb, int launches, hipStream_t st)
{
    int rc = PLBM_OK;
    for (int k = 0; k < launches && rc == PLBM_OK; ++k)
        rc = launch_sweep<S, D, false>(p, (k & 1) ? fb : fa, (k & 1) ? fa : fb, st);
    return rc;
}

// The first D of n steps, with the fields of the state they read; an even depth
// takes a second launch for the state to be where so many single steps leave it.
template <class S, int D>
int run_sweeps_fields(const KParams &p, const plbm_desc *d, void *fa, void *fb, int n, FieldsOut fo,
                      const plbm::StepCall &call, hipStream_t st)
{
    int rc = launch_sweep<S, D, true>(p, fa, fb, st, fo);
    if (D % 2 == 0) {
        if (rc == PLBM_OK) rc = launch_sweep<S, D, false>(p, fb, fa, st);
        n -= D;
    } else {
        std::swap(fa, fb);
    }
    n -= D;
    return rc == PLBM_OK && n > 0 ? run_steps<S>(p, d, fa, fb, n, call, st) : rc;
}

// Which lattices take tiles of fused steps (plbm_tile.h) and which shape: the
// smallest of 8 x 8, 16 x 16 and 20 x 20 nodes (16-bit, FP32) that gives each CU at
// most one tile, three steps each; past those two steps on a larger tile,
// whose margin is less of it, up to the size from which strips are faster.
// Measured (us a step, single / pairs / tiles): FP64 384^2 15.5 / 11.2 / 8.2,
// 768^2 44 / 30 / 26, 1024^2 73 / 47 / 60; FP32 384^2 7.2 / 7.3 / 5.1, 768^2 23.8 /
// 15.5 / 13.9, 1024^2 37.7 / 25.6 / 24.4; FP16 384^2 5.5 / - / 4.2, 768^2 14.2 / - /
// 12.1, 1024^2 21.9 / 24 / 22.0.
template <class S>
bool use_tiles(const KParams &p)
{
    return paper_set(p) && (long long)p.nx * p.ny <= (sizeof(typename S::T) == 4 ? TILE_NODES : 700000);
}

template <class S>
void tile_steps(const KParams &p, void *fa, void *fb, int &n, hipStream_t st)
{
    using M = Thermal25<S>;
    constexpr size_t elem = sizeof(typename S::T);
    TileRun<M> run(p, fa, fb, st);
    if (run.template one_round<8, 8>()) return run.template take<8, 8, 3>(n);
    if (run.template one_round<16, 16>()) return run.template take<16, 16, 3>(n);
    if constexpr (elem < 8)
        if (run.template one_round<20, 20>()) return run.template take<20, 20, 3>(n);
    constexpr int BX = elem == 4 ? 16 : 24, BY = elem == 2 ? 24 : 16;
    if (run.template pay<BX, BY, 2>(M::TILE2)) run.template take<BX, BY, 2>(n);
    if (run.template pay<16, 16, 3>(M::TILE3)) run.template take<16, 16, 3>(n);
}

// How many steps a strip of a larger lattice takes (plbm_sweep.h); 1: single
// steps.  Measured (us a step, single / two / three): FP64 4096^2 1050 / 622 / -, FP32
// 519 / 324 / 225, FP32 1501 x 1100 65 / 43 / 33.  The 16-bit forms are bound by
// vector work, of which short chunks add up to as much again: FP16 1024^2 21.9 /
// 24, 1501 x 1100 40.4 / 29.5, 4096^2 278 / 212.  Rows that leave half the lanes
// of their strips idle (a quarter: 16-bit) stay with single steps.
// FP32 takes three if the strips use 3/4 of their lanes (257 x 4100 - / 26 / 32) and
// its workgroups, one a CU, come to fewer rows: a row of three steps takes 2.06
// us, a row of each of two workgroups of pairs 3.1 (70000 x 16, two rounds of 313:
// 46 / 26 / 36).  And either has to be faster than single steps (see LaunchTime).
template <class S>
int sweep_depth(const KParams &p, const plbm_desc *d)
{
    constexpr bool narrow = sizeof(typename S::T) == 2;
    using M = Thermal25<S>;
    if (d->dim != 2 || !sweep_fits<M>(p.nx) || !paper_set(p)) return 1;
    if (narrow && (long long)p.nx * p.ny < 1500000) return 1;
    const SweepGrid g = sweep_grid<M, 2>(p.nx, p.ny);
    const long long used = (long long)p.nx * g.per, lanes = (long long)g.strips * sweep_threads<M>();
    if (narrow ? 4 * used < 3 * lanes : 2 * used < lanes) return 1;
    if constexpr (sizeof(typename S::T) == 4) {
        const SweepGrid g3 = sweep_grid<M, 3>(p.nx, p.ny);
        const long long lanes3 = (long long)g3.strips * sweep_threads<M>();
        if (4 * (long long)p.nx * g3.per >= 3 * lanes3 &&
            2.06 / 3 * sweep_rounds<M, 3>(g3) <= 3.1 / 2 * sweep_rounds<M, 2>(g) &&
            strips_pay<M, 3>(g3, M::TRIPLE, p.nx, p.ny))
            return 3;
    }
    return narrow || strips_pay<M, 2>(g, M::PAIR, p.nx, p.ny) ? 2 : 1;
}

template <class S>
int run_steps(const KParams &p, const plbm_desc *d, void *fa, void *fb, int nsteps, const plbm::StepCall &call,
              hipStream_t st)
{
    double *const sums = call.sums;
    const int fusable = call.fusable(nsteps);
    int nb = 0;
    int s0 = 0;
    if (d->dim == 2 && use_tiles<S>(p)) {
        int left = fusable;
        clear_launch_error();
        tile_steps<S>(p, fa, fb, left, st);
        const int rc = launch_status();
        if (rc != PLBM_OK) return rc;
        s0 = fusable - left;
    }
    if (const int depth = s0 == 0 ? sweep_depth<S>(p, d) : 1; depth > 1) {
        const int n = fusable;
        const int pairs = depth == 3 ? pairs_beside_threes(n) : fused_launches<2>(n);
        if constexpr (sizeof(typename S::T) == 4) {
            if (depth == 3) {
                const int threes = (n - 2 * pairs) / 3;
                const int rc = run_sweeps<S, 3>(p, fa, fb, threes, st);
                if (rc != PLBM_OK) return rc;
                s0 = 3 * threes;
            }
        }
        const int rc = run_sweeps<S, 2>(p, (s0 & 1) ? fb : fa, (s0 & 1) ? fa : fb, pairs, st);
        if (rc != PLBM_OK) return rc;
        s0 += 2 * pairs;
    }
    if constexpr (sizeof(typename S::T) >= 4) {
        if (d->dim == 1) {
            clear_launch_error();
            s0 = run_tube<Thermal5<S>>(p, fa, fb, fusable, std::max(std::abs(p.sx[1]), std::abs(p.sx[3])), st);
            const int rc = launch_status();
            if (rc != PLBM_OK) return rc;
        }
    }
    for (int s = s0; s < nsteps; ++s) {
        const void *src = (s & 1) ? fb : fa;
        void *dst = (s & 1) ? fa : fb;
        const bool last = (s == nsteps - 1);
        if (last && sums) {
            int blocks = d->dim == 2 ? grid_for(p.ntiles) : (p.nx + TX - 1) / TX;
            plbm::SumsArea area;
            if (call.noalloc) blocks = std::min(blocks, NOALLOC_BLOCKS);
            int rc = call.noalloc ? scratch_wait(area) : plbm::sums_begin(area, 4, blocks, d->dim == 2, st);
            if (rc != PLBM_OK) return rc;
            rc = launch_step<S, true>(p, d, src, dst, area.part, st, nb, blocks);
            return plbm::sums_end(area, 4, blocks, rc, sums, st);
        }
        int rc = launch_step<S, false>(p, d, src, dst, nullptr, st, nb);
        if (rc != PLBM_OK) return rc;
    }
    return PLBM_OK;
}

// 2D steps of which the first also writes the fields of the state it reads: a
// fused launch where those are taken, else a step of its own.
template <class S>
int run_steps_fields(const KParams &p, const plbm_desc *d, void *fa, void *fb, int nsteps, FieldsOut fo,
                     const plbm::StepCall &call, hipStream_t st)
{
    using T = typename S::T;
    const int fusable = call.fusable(nsteps);
    const int depth = use_tiles<S>(p) ? 1 : sweep_depth<S>(p, d);
    if constexpr (sizeof(T) == 4)
        if (depth == 3 && fusable - 2 * pairs_beside_threes(fusable) >= 3)
            return run_sweeps_fields<S, 3>(p, d, fa, fb, nsteps, fo, call, st);
    if (depth > 1 && fused_launches<2>(fusable) > 0)
        return run_sweeps_fields<S, 2>(p, d, fa, fb, nsteps, fo, call, st);
    clear_launch_error();
    const size_t lds = sizeof(T) == 2 ? (d->rounding == PLBM_ROUND_STOCHASTIC ? PLBM_LDS_CAP_16SR : PLBM_LDS_CAP_16)
                                      : PLBM_LDS_CAP_WIDE;
    const bool nts = single_step_nt(p.nx, p.ny, NQ, sizeof(T));
    auto *kernel = p.nv == 2 ? (nts ? k_step2d_fields<S, 2, true> : k_step2d_fields<S, 2, false>)
                             : (nts ? k_step2d_fields<S, 1, true> : k_step2d_fields<S, 1, false>);
    hipLaunchKernelGGL(kernel, dim3(grid_for(p.ntiles)), dim3(TX), lds, st, (const T *)fa, (T *)fb, p, fo);
    const int rc = launch_status();
    return rc == PLBM_OK && nsteps > 1 ? run_steps<S>(p, d, fb, fa, nsteps - 1, call, st) : rc;
}

template <class S>
int launch_init(const KParams &p, const plbm_desc *d, const double *rho, const double *ux,
                const double *uy, const double *th, void *f, hipStream_t st)
{
    using T = typename S::T;
    clear_launch_error();
    if (d->dim == 2) {
        hipLaunchKernelGGL(k_init2d<S>, dim3(grid_for((long long)((p.nx + TX - 1) / TX) * p.ny)),
                           dim3(TX), 0, st, rho, ux, uy, th, (T *)f, p);
    } else {
        hipLaunchKernelGGL(k_init1d<S>, dim3((p.nx + 2 * PLBM_GHOST + TX - 1) / TX), dim3(TX), 0,
                           st, rho, ux, th, (T *)f, p);
    }
    return launch_status();
}

template <class S>
int launch_moments(const KParams &p, const plbm_desc *d, const void *f, double *rho, double *ux,
                   double *uy, double *th, double *partials, hipStream_t st, int &nblocks,
                   int max_blocks)
{
    using T = typename S::T;
    clear_launch_error();
    if (d->dim == 2) {
        nblocks = grid_capped((long long)((p.nx + TX - 1) / TX) * p.ny, max_blocks);
        hipLaunchKernelGGL(k_moments2d<S>, dim3(nblocks), dim3(TX), 0, st, (const T *)f, p, rho,
                           ux, uy, th, partials);
    } else {
        nblocks = (p.nx + TX - 1) / TX;
        hipLaunchKernelGGL(k_moments1d<S>, dim3(nblocks), dim3(TX), 0, st, (const T *)f, p, rho, ux,
                           th, partials);
    }
    return launch_status();
}

#define PLBM_DISPATCH(d, FN, ...)                                                        \
    switch ((d)->storage + 8 * (d)->rounding) {                                          \
    case PLBM_F64: return FN<StF64>(__VA_ARGS__);                                        \
    case PLBM_F32: return FN<StF32>(__VA_ARGS__);                                        \
    case PLBM_F16DEV: return FN<StF16>(__VA_ARGS__);                                     \
    case PLBM_BF16DEV: return FN<StBF16>(__VA_ARGS__);                                   \
    case PLBM_F16DEV + 8 * PLBM_ROUND_STOCHASTIC: return FN<StF16SR>(__VA_ARGS__);       \
    case PLBM_BF16DEV + 8 * PLBM_ROUND_STOCHASTIC: return FN<StBF16SR>(__VA_ARGS__);     \
    default: return PLBM_EINVAL;                                                         \
    }

int init_dispatch(const KParams &p, const plbm_desc *d, const double *rho, const double *ux,
                  const double *uy, const double *th, void *f, hipStream_t st)
{
    PLBM_DISPATCH(d, launch_init, p, d, rho, ux, uy, th, f, st);
}

int step_dispatch(const KParams &p, const plbm_desc *d, void *fa, void *fb, int n, const plbm::StepCall &call,
                  hipStream_t st)
{
    PLBM_DISPATCH(d, run_steps, p, d, fa, fb, n, call, st);
}

int step_fields_dispatch(const KParams &p, const plbm_desc *d, void *fa, void *fb, int n, FieldsOut fo,
                         const plbm::StepCall &call, hipStream_t st)
{
    PLBM_DISPATCH(d, run_steps_fields, p, d, fa, fb, n, fo, call, st);
}

int moments_dispatch(const KParams &p, const plbm_desc *d, const void *f, double *rho, double *ux,
                     double *uy, double *th, double *part, hipStream_t st, int &nb,
                     int max_blocks = MAX_GRID)
{
    PLBM_DISPATCH(d, launch_moments, p, d, f, rho, ux, uy, th, part, st, nb, max_blocks);
}

// Plain streaming copy, 16 bytes per thread: the calibration kernel for
// achievable HBM bandwidth and for the byte counters of a profiler.
typedef float CopyVec __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_stream_copy(const CopyVec *__restrict__ a,
                                                     CopyVec *__restrict__ b, size_t n)
{
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(a[i], b + i);
}

} // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
namespace plbm {
void note_hip_error(const char *what, int code)
{
    std::snprintf(g_last_error, sizeof(g_last_error), "%s (%d)", what, code);
}

int sums_begin(SumsArea &a, int nv, int &blocks, bool walks, void *stream)
{
    hipStream_t st = as_stream(stream);
    const int most = SCRATCH_ELEMS / nv - 1;
    if (walks) blocks = std::min(blocks, most);
    int dev = -1, of = -1;
    if (blocks <= most && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < MAX_DEVICES &&
        (!st || (hipStreamGetDevice(st, &of) == hipSuccess && of == dev)) && g_scratch[1][dev].mu.try_lock()) {
        Scratch &s = g_scratch[1][dev];
        if (scratch_address(s, 1) == PLBM_OK) {
            a.part = s.dev;
            a.held = &s.mu;
            return PLBM_OK;
        }
        s.mu.unlock();
    }
    return hip_ok(hipMallocAsync((void **)&a.part, ((size_t)blocks + 1) * nv * sizeof(double), st));
}

int sums_end(SumsArea &a, int nv, int blocks, int rc, double *host, void *stream)
{
    hipStream_t st = as_stream(stream);
    double *out = a.part + (size_t)blocks * nv;
    if (rc == PLBM_OK) {
        clear_launch_error();
        if (nv == 4)
            hipLaunchKernelGGL(k_reduce_partials<4>, dim3(1), dim3(RED_THREADS), 0, st, a.part, blocks, out);
        else
            hipLaunchKernelGGL(k_reduce_partials<5>, dim3(1), dim3(RED_THREADS), 0, st, a.part, blocks, out);
        rc = launch_status();
    }
    if (rc == PLBM_OK) rc = hip_ok(hipMemcpyAsync(host, out, nv * sizeof(double), hipMemcpyDeviceToHost, st));
    const int done = hip_ok(hipStreamSynchronize(st));
    if (rc == PLBM_OK) rc = done;
    if (a.held) a.held->unlock();
    else (void)hipFreeAsync(a.part, st);
    a = SumsArea{};
    if (rc != PLBM_OK) return rc;
    for (int m = 0; m < nv; ++m)
        if (!std::isfinite(host[m])) return PLBM_ENONFINITE;
    return PLBM_OK;
}
} // namespace plbm

extern "C" int plbm_init(const plbm_desc *d, const double *rho, const double *ux,
                         const double *uy, const double *theta, void *f, void *stream)
{
    if (d && d->dim == 3) return PLBM_EINVAL;
    if (plbm::gen_handles(d)) return plbm::gen_init(d, rho, ux, uy, theta, f, stream);
    if (d && d->q1d == 3) return plbm::q3_init(d, rho, ux, uy, f, stream);
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!rho || !ux || !theta || !f || (d->dim == 2 && !uy)) return PLBM_EINVAL;
    return init_dispatch(p, d, rho, ux, uy, theta, f, as_stream(stream));
}

namespace {
int step_entry(const plbm_desc *d, void *f_a, void *f_b, int nsteps, const plbm::StepCall &call, void *stream)
{
    // a step of its own leaves the state before where it read it
    if (d && d->dim == 3) return plbm::q125_step(d, f_a, f_b, nsteps, call.sums, stream);
    if (plbm::gen_handles(d)) return plbm::gen_step(d, f_a, f_b, nsteps, call, stream);
    if (d && d->q1d == 3) return plbm::q3_step(d, f_a, f_b, nsteps, call, stream);
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!f_a || !f_b || f_a == f_b || nsteps < 0) return PLBM_EINVAL;
    if (nsteps == 0) {
        if (call.sums) return plbm_moments(d, f_a, nullptr, nullptr, nullptr, nullptr, call.sums, stream);
        return PLBM_OK;
    }
    return step_dispatch(p, d, f_a, f_b, nsteps, call, as_stream(stream));
}

int step_fields_entry(const plbm_desc *d, void *f_a, void *f_b, int nsteps, FieldsOut fo,
                      const plbm::StepCall &call, void *stream)
{
    if (!d) return PLBM_EINVAL;
    if (d->dim != 2 || plbm::gen_handles(d) || d->q1d != Q) return PLBM_EUNSUPPORTED;
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!f_a || !f_b || f_a == f_b || nsteps < 1) return PLBM_EINVAL;
    return step_fields_dispatch(p, d, f_a, f_b, nsteps, fo, call, as_stream(stream));
}
} // namespace

extern "C" int plbm_step(const plbm_desc *d, void *f_a, void *f_b, int nsteps, double *sums,
                         void *stream)
{
    plbm::StepCall call;
    call.sums = sums;
    call.keep = true;
    return step_entry(d, f_a, f_b, nsteps, call, stream);
}

extern "C" int plbm_advance(const plbm_desc *d, void *f_a, void *f_b, int nsteps, double *sums, void *stream)
{
    plbm::StepCall call;
    call.sums = sums;
    return step_entry(d, f_a, f_b, nsteps, call, stream);
}

extern "C" int plbm_step_fields(const plbm_desc *d, void *f_a, void *f_b, int nsteps, double *rho, double *ux,
                                double *uy, double *theta, void *stream)
{
    plbm::StepCall call;
    call.keep = true;
    return step_fields_entry(d, f_a, f_b, nsteps, FieldsOut{{rho, ux, uy, theta}}, call, stream);
}

extern "C" int plbm_advance_fields(const plbm_desc *d, void *f_a, void *f_b, int nsteps, double *rho, double *ux,
                                   double *uy, double *theta, void *stream)
{
    return step_fields_entry(d, f_a, f_b, nsteps, FieldsOut{{rho, ux, uy, theta}}, plbm::StepCall{}, stream);
}

extern "C" int plbm_step_noalloc(const plbm_desc *d, void *f_a, void *f_b, int nsteps,
                                 double *sums, void *stream)
{
    if (d && d->dim == 3) return PLBM_EUNSUPPORTED;
    if (plbm::gen_handles(d) || (d && d->q1d != Q)) return PLBM_EUNSUPPORTED;
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!f_a || !f_b || f_a == f_b || nsteps < 0) return PLBM_EINVAL;
    // the 1D kernels run one workgroup per 256 nodes: at most NOALLOC_BLOCKS
    // of them fit the scratch when sums are asked for
    if (sums && d->dim == 1 && (p.nx + TX - 1) / TX > NOALLOC_BLOCKS) return PLBM_EINVAL;
    hipStream_t st = as_stream(stream);
    plbm::StepCall call;
    call.sums = sums;
    call.keep = true;
    call.noalloc = true;
    if (nsteps > 0) return step_dispatch(p, d, f_a, f_b, nsteps, call, st);
    if (!sums) return PLBM_OK;
    plbm::SumsArea area;
    rc = scratch_wait(area);
    if (rc != PLBM_OK) return rc;
    int nb = 0;
    rc = moments_dispatch(p, d, f_a, nullptr, nullptr, nullptr, nullptr, area.part, st, nb, NOALLOC_BLOCKS);
    return plbm::sums_end(area, 4, nb, rc, sums, st);
}

extern "C" int plbm_moments(const plbm_desc *d, const void *f, double *rho, double *ux,
                            double *uy, double *theta, double *sums, void *stream)
{
    if (d && d->dim == 3) return PLBM_EINVAL;
    if (plbm::gen_handles(d)) return plbm::gen_moments(d, f, rho, ux, uy, theta, sums, stream);
    if (d && d->q1d == 3)
        return plbm::q3_moments(d, f, rho, ux, uy, theta, sums, stream);
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!f) return PLBM_EINVAL;
    hipStream_t st = as_stream(stream);
    int nb = 0;
    if (!sums) return moments_dispatch(p, d, f, rho, ux, uy, theta, nullptr, st, nb);
    int blocks = d->dim == 2 ? grid_for((long long)((p.nx + TX - 1) / TX) * p.ny) : (p.nx + TX - 1) / TX;
    plbm::SumsArea area;
    rc = plbm::sums_begin(area, 4, blocks, d->dim == 2, st);
    if (rc != PLBM_OK) return rc;
    rc = moments_dispatch(p, d, f, rho, ux, uy, theta, area.part, st, nb, blocks);
    return plbm::sums_end(area, 4, blocks, rc, sums, st);
}

extern "C" int plbm_dev_scales(plbm_desc *d, const double *rho, const double *ux,
                               const double *uy, const double *theta, void *stream)
{
    if (!d || d->dim != 2 || d->storage < PLBM_F16DEV) return PLBM_EINVAL;
    // validation with provisional unit scales
    for (int k = 0; k < NQ; ++k) d->scale[k] = 1.0f;
    KParams p;
    int rc = make_params(d, p);
    if (rc != PLBM_OK) return rc;
    if (!rho || !ux || !uy || !theta) return PLBM_EINVAL;
    hipStream_t st = as_stream(stream);
    double w[3], base[NQ];
    rest_weights(p.r64, d->theta0, w);
    for (int k = 0; k < NQ; ++k) base[k] = d->rho0 * w[vclass(k % Q)] * w[vclass(k / Q)];
    const dim3 g(grid_for((long long)((p.nx + TX - 1) / TX) * p.ny));
    const size_t nb = g.x;
    double *buf = nullptr;
    const size_t bytes = (NQ + nb * NQ) * sizeof(double);
    rc = hip_ok(hipMallocAsync((void **)&buf, bytes, st));
    if (rc != PLBM_OK) return rc;
    rc = hip_ok(hipMemcpyAsync(buf, base, NQ * sizeof(double), hipMemcpyHostToDevice, st));
    if (rc == PLBM_OK) {
        clear_launch_error();
        hipLaunchKernelGGL(k_devmax2d, g, dim3(TX), 0, st, rho, ux, uy, theta, p, buf, buf + NQ);
        rc = launch_status();
    }
    double *host = rc == PLBM_OK ? new double[nb * NQ] : nullptr;
    if (rc == PLBM_OK)
        rc = hip_ok(hipMemcpyAsync(host, buf + NQ, nb * NQ * sizeof(double), hipMemcpyDeviceToHost, st));
    if (rc == PLBM_OK) rc = hip_ok(hipStreamSynchronize(st));
    (void)hipFreeAsync(buf, st);
    if (rc == PLBM_OK) {
        double cmax[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (int k = 0; k < NQ; ++k)
            for (size_t b = 0; b < nb; ++b) {
                const double m = host[b * NQ + k];
                if (!std::isfinite(m)) rc = PLBM_ENONFINITE;
                else cmax[pclass(k)] = std::fmax(cmax[pclass(k)], m);
            }
        // Floor: the FP32 collision leaves absolute rounding noise of a few
        // 2^-24 rho0 in any population, which must stay a small deviation
        // (|h| of order 10) rather than overflow it; an initial state at
        // rest (deviations of FP64 rounding, ~1e-17) would otherwise get
        // scales near 1e-20.
        const int e_floor = (int)std::floor(std::log2(d->rho0)) - 26;
        if (rc == PLBM_OK)
            for (int k = 0; k < NQ; ++k) {
                // smallest e with max deviation <= 2^e * 2^10 over the class
                const double m = cmax[pclass(k)];
                int e = m > 0.0 ? (int)std::ceil(std::log2(m)) - 10 : e_floor;
                if (m > 0.0 && std::ldexp(1.0, e + 10) < m) e += 1;
                d->scale[k] = (float)std::ldexp(1.0, std::max(e, e_floor));
            }
    }
    delete[] host;
    return rc;
}

extern "C" int plbm_stream_copy(const void *src, void *dst, size_t bytes, void *stream)
{
    if (!src || !dst || bytes == 0 || (bytes % 16) != 0) return PLBM_EINVAL;
    if (((uintptr_t)src | (uintptr_t)dst) % 16 != 0) return PLBM_EINVAL;
    const size_t n = bytes / 16;
    const size_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffffu) return PLBM_EINVAL;
    clear_launch_error();
    hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)blocks), dim3(256), 0, as_stream(stream),
                       (const CopyVec *)src, (CopyVec *)dst, n);
    return launch_status();
}

extern "C" const char *plbm_last_hip_error(void) { return g_last_error; }
