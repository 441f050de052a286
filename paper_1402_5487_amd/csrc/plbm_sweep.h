// Several fused steps per launch on a periodic 2D lattice: a strip of columns
// is swept in y and the populations between the steps never leave the CU.
// Internal header (not part of the C ABI), on top of plbm_device.h.
//
// A model M gives the storage type T, the arithmetic type C, the velocities
// V[Q1] of one axis (compile time), the parameters P (with nx and ny), and
// dec / enc / key / collide of one node.  R = max |v|, q = Q1^2.
//
// A workgroup owns the output nodes [xs, xs + w) x
// [ya, yb) of D steps; a thread holds one of at most SPAN columns.  In iteration `it` stage s
// (the step s of the D) takes row ya - R (D - 1) + it - s R: R rows behind
// stage s - 1, whose population (i, j) of row r it reads at row r + v_j, i.e.
// v_j + R iterations after it was made.  So the line of velocity j holds
// v_j + R + 1 rows, (R + 1) Q1 rows in all for a symmetric set.  The shifted x
// velocities keep theirs in LDS (a neighbouring lane reads them), v_i = 0 in
// registers (the same lane does).  Values between the steps are held in the
// storage type, encoded and decoded as through memory, so the fused steps
// give bitwise what D launches of the single step give.
//
// What bounds it: D single steps read and write every population D times at
// the HBM rate; here once, plus the halo (R (D - 1) columns and rows on each
// side are computed twice by neighbours).  Vector instructions then fill, of the
// issue slots of busy compute units: D2Q25 4096^2 FP64 pairs 0.19 and FP32 threes
// 0.45, which move 5.9 and 5.6 TB/s (a copy: 6.3) and are bound by that; FP16 pairs
// 0.82 at 4.8 TB/s, BF16 with stochastic rounding 1501 x 1100 1.0, D2Q9 FP32 2048^2
// fives 0.89 at 4.6, which are bound by the vector work.
#pragma once
#include <type_traits>

#include "plbm_device.h"

namespace {

constexpr int SWEEP_CUS = 256;            // compute units of an MI355X
constexpr size_t SWEEP_LDS = 160 * 1024;  // LDS of one of them

// What a launch takes on an MI355X, in microseconds: `base`, `unit` for what its
// workgroups do one after another (rounds of tiles, rows of strips), and
// `mnode` for a million nodes read and written.  A launch of several steps is
// taken where it is faster than the single steps it stands for: on lattices of
// a few rows a tile or a strip computes several times its own nodes.  Fitted to
// lattices of 3 to 48 rows and 3000 to 300000 nodes a row, to 10 % (16-bit strips,
// taken on large lattices only, have no such rule).  What the rule changed, us a
// step before and after: D2Q25 FP16 100000 x 3 32.7 and 8.9, FP64 37.2 and 20.9; D2Q9
// FP32 300000 x 3 27.2 and 7.6; D2Q49 FP32 10000 x 3 9.1 and 5.8.
struct LaunchTime {
    double base, unit, mnode;
    double us(double units, double nodes) const { return base + unit * units + 1e-6 * mnode * nodes; }
};
// A single step, whose workgroups take as long on shorter rows as on 64 nodes (50
// to 90).
template <class M>
inline double single_us(int nx, int ny)
{
    return M::SINGLE.us(0, (double)std::max(nx, 64) * ny);
}

// The delay lines of a velocity set.
template <class M>
struct Lines {
    static constexpr int reach()
    {
        int r = 0;
        for (int i = 0; i < M::Q1; ++i) r = M::V[i] > r ? M::V[i] : (-M::V[i] > r ? -M::V[i] : r);
        return r;
    }
    static constexpr int R = reach();
    static constexpr int len(int j) { return M::V[j] + R + 1; }
    static constexpr int base(int j)           // first LDS row of line j
    {
        int b = 0;
        for (int k = 0; k < j; ++k) b += len(k);
        return b;
    }
    static constexpr int rbase(int j)          // first register of line j
    {
        int b = 0;
        for (int k = 0; k < j; ++k) b += len(k) - 1;
        return b;
    }
    static constexpr int still()               // the x velocity 0, or -1
    {
        for (int i = 0; i < M::Q1; ++i)
            if (M::V[i] == 0) return i;
        return -1;
    }
    static constexpr int I0 = still();
    static constexpr int ROWS = base(M::Q1);
    static constexpr int REGS = I0 < 0 ? 1 : rbase(M::Q1);
    static constexpr int COLS = M::Q1 - (I0 >= 0 ? 1 : 0);    // x velocities kept in LDS
    static constexpr int column(int i) { return I0 >= 0 && i > I0 ? i - 1 : i; }
};

// Threads of a workgroup: whole waves over M::SPAN columns.
template <class M>
constexpr int sweep_threads() { return (M::SPAN + 63) / 64 * 64; }
template <class M, int D>
constexpr size_t sweep_lds_bytes()
{
    return (size_t)(D - 1) * Lines<M>::ROWS * Lines<M>::COLS * M::SPAN * sizeof(typename M::T);
}
// Workgroups a CU holds, M::WGS at most (one wave of each on every SIMD).
template <class M, int D>
constexpr int sweep_per_cu()
{
    return (int)(SWEEP_LDS / sweep_lds_bytes<M, D>()) < M::WGS ? (int)(SWEEP_LDS / sweep_lds_bytes<M, D>()) : M::WGS;
}

// Of n steps, the launches of D that leave the state in the buffer where
// single steps leave it: any number for odd D, an even one for even D.
template <int D>
inline int fused_launches(int n) { return D & 1 ? n / D : n / D & ~1; }

// Strips of w columns and chunks of h rows.  Workgroup b of a lattice takes
// strip b % strips of `per` chunks side by side, from chunk b / strips * per on
// (T / per threads each).  span: the columns held, the strip's and its halo; a
// strip that is the whole row closes on itself and has none.
struct SweepGrid {
    int strips, chunks, w, h, span, per, wgs;
    __host__ void rows(int ny, int height)
    {
        h = height;
        chunks = (ny + h - 1) / h;
        wgs = strips * ((chunks + per - 1) / per);
    }
    // chunks of one height, `height` at most
    __host__ void even_rows(int ny, int height)
    {
        const int n = (ny + height - 1) / height;
        rows(ny, (ny + n - 1) / n);
    }
};

// Which of the g.per chunks side by side a thread works on.  The kernel asks
// once per wave, so sweep_grid puts no more of them side by side than the
// workgroup has waves.
__host__ __device__ inline int sweep_side(const SweepGrid &g, int thread, int threads)
{
    return thread * g.per / threads;
}

// The partition of an nx x ny lattice.  Strips begin on cache lines, whole or
// half (M::line<D>() bytes): stores that end inside a line left the D2Q25 pair at
// 4096^2 at 489 us a step in FP32 against 373.  Chunks: as many rounds of
// resident workgroups as leave them about M::rounds_h<D>() rows.  Long chunks
// spread the accesses over so much memory that the D2Q25 FP32 pair at 4096^2
// took 373 us a step with 157 rows, 318 with 64 and 313 with 16; a last round
// of a few workgroups costs as much as a full one (D2Q9 FP32 2048^2, 1.1
// rounds: 22.6 us a step, one: 17).
template <class M, int D>
constexpr int sweep_align() { return M::template line<D>() / (int)sizeof(typename M::T); }
template <class M, int D>
constexpr int sweep_wmax()
{
    return (M::SPAN - 2 * Lines<M>::R * (D - 1)) / sweep_align<M, D>() * sweep_align<M, D>();
}
// Rows that the rounds of resident workgroups compute one after another.
template <class M, int D>
inline long long sweep_rounds(const SweepGrid &g)
{
    constexpr int slots = SWEEP_CUS * sweep_per_cu<M, D>();
    return (long long)((g.wgs + slots - 1) / slots) * (g.h + 2 * Lines<M>::R * (D - 1));
}
template <class M, int D>
inline SweepGrid sweep_grid(int nx, int ny)
{
    constexpr int align = sweep_align<M, D>(), wmax = sweep_wmax<M, D>();
    constexpr int slots = SWEEP_CUS * sweep_per_cu<M, D>();
    SweepGrid g;
    g.per = 1;
    if (nx <= M::SPAN) {
        // chunks side by side, each of whole waves: two waves (D2Q49 in FP64) take
        // two at most
        constexpr int waves = sweep_threads<M>() / 64;
        static_assert(waves == 1 || waves == 2 || waves == 4, "the chunks side by side share the waves evenly");
        g.strips = 1;
        g.w = g.span = nx;
        for (int per = waves; per > 1 && g.per == 1; per /= 2)
            if (nx <= sweep_threads<M>() / per && nx * per <= M::SPAN) g.per = per;
    } else {
        g.strips = (nx + wmax - 1) / wmax;
        g.w = ((nx + g.strips - 1) / g.strips + align - 1) / align * align;
        g.strips = (nx + g.w - 1) / g.w;
        g.span = g.w + 2 * Lines<M>::R * (D - 1);
    }
    // rounds of resident workgroups, each filled alike
    auto chunk_rows = [&](int rounds) {
        const int chunks = std::max(1, rounds * slots * g.per / g.strips);
        return (ny + chunks - 1) / chunks;
    };
    g.rows(ny, chunk_rows(std::max(1, chunk_rows(1) / M::template rounds_h<D>())));
    // More strips than resident workgroups, each the whole height: up to four
    // chunks where those fill the rounds better (D2Q49 FP64 30000 x 48, 289 strips for
    // 256 workgroups: 230 us a step whole, 219 in single steps, 184 in three chunks).
    // Two workgroups a CU share its rounds unevenly: FP32 pairs of 150000 x 16 55 whole, 59
    // in two chunks.
    if (sweep_per_cu<M, D>() == 1 && g.chunks == 1 && g.strips > slots)
        for (int chunks = 2; chunks <= 4; ++chunks) {
            SweepGrid t = g;
            t.rows(ny, (ny + chunks - 1) / chunks);
            if (sweep_rounds<M, D>(t) < sweep_rounds<M, D>(g)) g = t;
        }
    return g;
}

// Barrier for LDS traffic only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ int wrap_mod(int a, int n)
{
    a %= n;
    return a < 0 ? a + n : a;
}

// Stores of one row block through a buffer descriptor: a lane whose byte
// offset lies past the block writes nothing, so the stores need no branch and
// the wait for the next row's loads can count them (a branch around them
// makes the compiler wait for every store in flight).  A block holds less
// than 2^31 bytes (see sweep_fits).
constexpr unsigned SWEEP_DROP = 0x80000000u;
template <bool NTS>
struct RowStore {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ RowStore(void *base, unsigned bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000)) {}
    static constexpr int AUX = NTS ? 2 : 0;                      // non-temporal
    __device__ __forceinline__ void put(double v, unsigned vo, unsigned so) const
    {
        typedef unsigned U2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, vo, so, AUX);
    }
    __device__ __forceinline__ void put(float v, unsigned vo, unsigned so) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, vo, so, AUX);
    }
    __device__ __forceinline__ void put(uint16_t v, unsigned vo, unsigned so) const
    {
        __builtin_amdgcn_raw_buffer_store_b16(v, r, vo, so, AUX);
    }
};

template <class M>
inline bool sweep_fits(int nx)
{
    return (long long)M::Q1 * M::Q1 * nx * (long long)sizeof(typename M::T) < (1ll << 31);
}

// D steps of the strip.  NTS: see store_stream.  FIELDS (models with collide(f, p, mom)): the first
// step also writes the fields of the owned nodes.
template <class M, int D, bool NTS, bool FIELDS = false>
__device__ __forceinline__ void sweep(const typename M::T *__restrict__ src, typename M::T *__restrict__ dst,
                                      const typename M::P &p, const SweepGrid &g, int b,
                                      typename M::T *__restrict__ lds, const FieldsOut &fo = FieldsOut{})
{
    using T = typename M::T;
    using C = typename M::C;
    using L = Lines<M>;
    constexpr int Q1 = M::Q1, NP = Q1 * Q1, I0 = L::I0;
    constexpr int halo = L::R * (D - 1);
    const int nx = p.nx, ny = p.ny;
    const int c = b / g.strips, xs = (b - c * g.strips) * g.w;
    // this thread's chunk, uniform over its wave, and its place in the strip;
    // a chunk past the last writes nothing
    const int side = __builtin_amdgcn_readfirstlane(sweep_side(g, (int)threadIdx.x, sweep_threads<M>()));
    const int t = (int)threadIdx.x - side * (sweep_threads<M>() / g.per);
    const int ya = (c * g.per + side) * g.h, yb = min(ya + g.h, ny);
    const long long rowelems = (long long)NP * nx;
    const unsigned colbytes = (unsigned)nx * (unsigned)sizeof(T);
    // threads 0 .. w - 1 hold the strip's own columns, the next ones the halo
    // on its right and as many more that on its left; threads past them repeat
    // the last (no new bytes)
    const int w = g.w, span = g.span, edge = (span - w) / 2;
    const int tc = min(t, span - 1), col0 = side * span;
    const int x = wrap_mod(xs + (tc < w + edge ? tc : tc - span), nx);
    const bool own = t < w && xs + t < nx;
    const unsigned vo = own ? (unsigned)x * (unsigned)sizeof(T) : SWEEP_DROP;
    // where column x - v_i stands in memory and among the strip's (the strip
    // closes on itself: what wraps is read by columns that nothing needs)
    unsigned lo[Q1];
    int col[Q1];
#pragma unroll
    for (int i = 0; i < Q1; ++i) {
        int c = x - M::V[i];
        c += (c < 0) ? nx : 0;
        c -= (c >= nx) ? nx : 0;
        lo[i] = (unsigned)c * (unsigned)sizeof(T) + (unsigned)i * colbytes;
        c = tc - M::V[i];
        c += (c < 0) ? span : 0;
        c -= (c >= span) ? span : 0;
        col[i] = L::column(i) * M::SPAN + col0 + c;
        asm volatile("" : "+v"(lo[i]), "+v"(col[i]));
    }
    T raw[NP], h[NP], reg[D - 1][L::REGS];
#pragma unroll
    for (int s = 0; s < D - 1; ++s)
#pragma unroll
        for (int m = 0; m < L::REGS; ++m) reg[s][m] = T(0);
    auto load_row = [&](int yr) {
#pragma unroll
        for (int j = 0; j < Q1; ++j) {
            int ys = yr - M::V[j];
            ys += (ys < 0) ? ny : 0;
            ys -= (ys >= ny) ? ny : 0;
            const T *base = src + (ys * rowelems + (long long)(Q1 * j) * nx);
#pragma unroll
            for (int i = 0; i < Q1; ++i) {
                const T *q = &base[lo[i] / sizeof(T)];
                // the still column reads the wave's own nodes only
                raw[i + Q1 * j] = i == I0 ? __builtin_nontemporal_load(q) : *q;
            }
        }
    };
    const int iters = g.h + 2 * halo;      // the same for all chunks: they share the barriers
    int slot[Q1];                       // of each line: the row being written, then the oldest
#pragma unroll
    for (int j = 0; j < Q1; ++j) slot[j] = 0;
    auto row_of = [&](int it, int s) {  // the lattice row of stage s
        return wrap_mod(ya - halo + it - s * L::R, ny);
    };
    auto key_of = [&](int it, int s) {
        return M::KEYED ? M::key((uint32_t)row_of(it, s) * (uint32_t)nx + (uint32_t)x) : 0u;
    };
    auto put_lines = [&](int s) {
        T *ring = lds + s * (L::ROWS * L::COLS * M::SPAN) + col0 + tc;
#pragma unroll
        for (int j = 0; j < Q1; ++j)
#pragma unroll
            for (int i = 0; i < Q1; ++i)
                if (i != I0) ring[((L::base(j) + slot[j]) * L::COLS + L::column(i)) * M::SPAN] = h[i + Q1 * j];
    };
    // stage s of iteration `it`: f <- the rows stage s - 1 left, relaxed
    auto stage = [&](int s, C(&f)[NP]) {
        const T *ring = lds + (s - 1) * (L::ROWS * L::COLS * M::SPAN);
#pragma unroll
        for (int j = 0; j < Q1; ++j) {
            int old = slot[j] + 1 == L::len(j) ? 0 : slot[j] + 1;
            const T *row = ring + (L::base(j) + old) * (L::COLS * M::SPAN);
#pragma unroll
            for (int i = 0; i < Q1; ++i) {
                T v;
                if (i != I0) v = row[col[i]];
                else if (L::len(j) == 1) v = h[i + Q1 * j];
                else v = reg[s - 1][L::rbase(j) + (L::len(j) > 1 ? L::len(j) - 2 : 0)];
                f[i + Q1 * j] = M::dec(v, i + Q1 * j, p);
            }
        }
        // the registers' lines move on by one row, newest first
        if constexpr (I0 >= 0) {
#pragma unroll
            for (int j = 0; j < Q1; ++j)
#pragma unroll
                for (int m = L::len(j) - 2; m >= 0; --m)
                    reg[s - 1][L::rbase(j) + m] = m == 0 ? h[I0 + Q1 * j] : reg[s - 1][L::rbase(j) + m - 1];
        }
        M::collide(f, p);
    };
    auto next_slot = [&]() {
#pragma unroll
        for (int j = 0; j < Q1; ++j) slot[j] = slot[j] + 1 == L::len(j) ? 0 : slot[j] + 1;
    };
    // stages 0 .. D - 2 of an iteration, and the next row's loads behind the
    // first of them
    auto front = [&](int it, int yr, int ynext) {
        C f[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) f[k] = M::dec(raw[k], k, p);
        if constexpr (FIELDS) {
            C mom[4];
            M::collide(f, p, mom);
            if (own && it >= halo && it < yb - ya + halo) {
                const long long n = (long long)yr * nx + x;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (fo.p[q]) fo.p[q][n] = (double)mom[q];
            }
        } else {
            M::collide(f, p);
        }
        const uint32_t k0 = key_of(it, 0);
#pragma unroll
        for (int k = 0; k < NP; ++k) h[k] = M::enc(f[k], k, p, k0);
        put_lines(0);
        load_row(ynext);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 1; s < D - 1; ++s) {
            lds_barrier();
            stage(s, f);
            const uint32_t ks = key_of(it, s);
#pragma unroll
            for (int k = 0; k < NP; ++k) h[k] = M::enc(f[k], k, p, ks);
            put_lines(s);
        }
        lds_barrier();
    };
    int yr = row_of(0, 0);              // ya may lie past ny in a chunk that does not exist
    load_row(yr);
#pragma unroll 1
    for (int it = 0; it < 2 * halo; ++it) {
        const int yn = yr + 1 == ny ? 0 : yr + 1;
        front(it, yr, yn);
        C f[NP];
        stage(D - 1, f);                // moves the last stage's registers on
        if constexpr (D == 2) lds_barrier();
        next_slot();
        yr = yn;
    }
    // as many (dropped) stores behind the loads as the loop leaves there, so
    // that its wait for the loads may let that many stores pass
    {
        const RowStore<NTS> out(dst, colbytes * NP);
#pragma unroll
        for (int k = 0; k < NP; ++k) out.put(raw[k], SWEEP_DROP, (unsigned)k * colbytes);
    }
#pragma unroll 1
    for (int it = 2 * halo; it < iters; ++it) {
        // the last time: a row read before, not used
        const int yn = it + 1 == iters ? yr : (yr + 1 == ny ? 0 : yr + 1);
        front(it, yr, yn);
        C f[NP];
        stage(D - 1, f);
        const int yo = ya + it - 2 * halo;
        const uint32_t ko = M::KEYED ? M::key((uint32_t)yo * (uint32_t)nx + (uint32_t)x) : 0u;
        // a row past the chunk's: a block of no bytes, which drops every store
        const bool in = yo < yb;
        const RowStore<NTS> out(dst + (in ? yo : 0) * rowelems, in ? colbytes * NP : 0);
#pragma unroll
        for (int k = 0; k < NP; ++k) out.put(M::enc(f[k], k, p, ko), vo, (unsigned)k * colbytes);
        if constexpr (D == 2) lds_barrier();
        next_slot();
        yr = yn;
    }
}

// Whether the strips of D steps are faster than single steps (see LaunchTime).
template <class M, int D>
inline bool strips_pay(const SweepGrid &g, const LaunchTime &t, int nx, int ny)
{
    // few rounds end together, many one after another
    const double rounds = (double)g.wgs / (SWEEP_CUS * sweep_per_cu<M, D>());
    const double rows = (rounds > 4 ? rounds : std::ceil(rounds)) * (g.h + 2 * Lines<M>::R * (D - 1));
    return t.us(rows, (double)nx * ny) < D * single_us<M>(nx, ny);
}

// The thermal model of plbm_device.h with the set {0, +-1, +-3} in the paper's
// order (paper_set: whether p's is that one).  It takes two steps a strip; FP32
// also three, whose 160 KB of LDS leave one workgroup a CU.  FP64 has no room for
// a third step; the 16-bit forms have and gain 6 % (FP16 4096^2 200 us a step against
// 212), less than the single steps left over cost calls of 4 or 8 steps.
template <class S>
struct Thermal25 {
    using T = typename S::T;
    using C = typename S::C;
    using P = KParams;
    static constexpr int Q1 = Q;
    static constexpr int V[Q] = {0, 1, -1, 3, -3};
    static constexpr bool KEYED = S::keyed;
    static constexpr int SPAN = 256, WGS = 4;
    // see LaunchTime: tiles of two steps (FP64 24 x 16 nodes, FP32 16 x 16, 16-bit
    // 24 x 24) and of three (16 x 16), strips of two and of three
    static constexpr int FORM = sizeof(T) == 8 ? 0 : sizeof(T) == 4 ? 1 : KEYED ? 3 : 2;
    static constexpr LaunchTime SINGLES[4] = {{3.5, 0, 72.7}, {3.1, 0, 36.2}, {3.1, 0, 19.7}, {3.8, 0, 20.1}};
    static constexpr LaunchTime TILES2[4] = {{2.4, 4.0, 57.5}, {5.0, 1.0, 22.6}, {4.0, 3.3, 7.7}, {4.2, 3.7, 8.2}};
    static constexpr LaunchTime TILES3[4] = {{2.5, 6.2, 63}, {3.9, 3.4, 20.6}, {3.8, 4.7, 17.8}, {3.2, 5.3, 18}};
    static constexpr LaunchTime SINGLE = SINGLES[FORM], TILE2 = TILES2[FORM], TILE3 = TILES3[FORM];
    static constexpr LaunchTime PAIR = sizeof(T) == 8 ? LaunchTime{2.5, 2.1, 42.9} : LaunchTime{2.8, 1.4, 26.4};
    static constexpr LaunchTime TRIPLE = {4.7, 1.5, 10.4};
    // Half lines where 128 B would cost a quarter of the lanes (16-bit) or a
    // twelfth (FP32 threes: 2500^2 106 us a step with 224 columns, 102 with 240;
    // 2048 x 4096 139, 126), and one workgroup of each CU writes.
    template <int D>
    static constexpr int line() { return sizeof(T) == 2 || (sizeof(T) == 4 && D == 3) ? 64 : 128; }
    // Tall chunks, as each computes 3 rows per step but the first twice at
    // either end (FP32 4096^2 in threes, us a step: 335 with 16 rows, 254 with
    // 53, 225 with one round of 316; FP64 2048^2 175 with 16, 160 with 93).  Two
    // FP32 workgroups fit a CU in pairs, and lose more to the spread of
    // their accesses (see sweep_grid).
    template <int D>
    static constexpr int rounds_h() { return sizeof(T) == 2 ? 32 : sizeof(T) == 4 && D == 2 ? 16 : 160; }
    static __device__ __forceinline__ C dec(T h, int k, const P &p) { return S::dec(h, k, p); }
    static __device__ __forceinline__ T enc(C f, int k, const P &p, uint32_t key)
    {
        const T h = S::enc(f, k, p, key);
        if constexpr (std::is_same_v<S, StF16>) {
            // one value at a time: the compiler turns pairs into an FP32 FMA
            // and a packed conversion, which rounds twice where the single
            // step's v_fma_mixlo_f16 rounds once
            _Float16 one = __builtin_bit_cast(_Float16, h);
            asm("" : "+v"(one));
            return __builtin_bit_cast(T, one);
        } else {
            return h;
        }
    }
    static __device__ __forceinline__ uint32_t key(uint32_t node) { return S::key(node); }
    static __device__ __forceinline__ void collide(C (&f)[NQ], const P &p) { collide2d<S>(f, p); }
    static __device__ __forceinline__ void collide(C (&f)[NQ], const P &p, C (&mom)[4]) { collide2d<S>(f, p, mom); }
};
inline bool paper_set(const KParams &p)
{
    for (int i = 0; i < Q; ++i)
        if (p.sx[i] != Thermal25<StF32>::V[i]) return false;
    return true;
}

} // namespace
