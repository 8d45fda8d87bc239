// device.hpp -- device-side building blocks shared by the PISO kernels:
// grid geometry, periodic neighbour indexing, the fourth-order face
// interpolation, and deterministic grid-wide reductions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace pisoc {

constexpr int kBlock = 256;       // threads per block of every field kernel
constexpr int kMaxRed = 8;        // values per grid reduction
constexpr int kMaxCorr = 4;
constexpr int kMaxClasses = 8;
constexpr int kIterInf = 0x7fffffff;

// Constants of one grid size and gas, passed by value to the kernels.  A
// launch covers `batch` members of the same size stacked along z (member m owns
// the blocks with blockIdx.z in [m nz, (m+1) nz) and the cells [m N, (m+1) N) of
// every field; vector components are NT = batch N apart).
struct Phys {
    int n;
    int cz;             // cells per thread along z
    int nz;             // blocks per member along z
    int batch;          // members in the launch
    size_t N, NT;       // cells per member, cells of all members
    double h, inv_h, inv_h2, V, inv_V, A;
    double gamma, C, mu;
    double g[3];        // gravity (settling drift; with two-way coupling also buoyancy)
    // Fourier closure (FP64 single grids): p = rho R T with the energy
    // equation; tn: T^n, ts: T* of the current step (set before each step)
    int fourier;
    double R, cv, kappa;
    const double* tn;
    const double* ts;
    // BDF2 (FP64 single grids, gathered kernels): the state at t^{n-1}
    // (density deviation, velocity, and one class's bulk density, set per
    // class); the coefficients are DevState::bdf
    int bdf2;
    const double* rm1;
    const double* um1;
    const double* rjm1;
};

// Variable-step BDF2 coefficients, d/dt y ~ (c0 y^{n+1} - c1 y^n + c2 y^{n-1}) / dt
// with w = dt / dt_prev (w = 0, backward Euler, when there is no previous step).
__host__ __device__ inline void bdf2_coef(double dt, double dt_prev, double (&c)[3]) {
    const double w = isfinite(dt_prev) ? dt / dt_prev : 0.0;
    c[0] = (1.0 + 2.0 * w) / (1.0 + w);
    c[1] = 1.0 + w;
    c[2] = w * w / (1.0 + w);
}

// The compressibility factor of the corrector: psi = rho / (gamma_psi p) with
// gamma_psi = gamma for the barotropic closure (d rho / d p of C rho^gamma)
// and 1 for the ideal gas at the predicted temperature (1 / (R T)).
__host__ __device__ inline double gamma_psi(const Phys& ph) { return ph.fourier ? 1.0 : ph.gamma; }

// State of one pressure solve, kept on the device so that CG never returns to
// the host between iterations.
struct PcgState {
    double bb;        // reference ||b||^2 of the current solve
    double rr;        // ||r||^2 of the last checked iterate
    double tol2;      // tol^2 of the current (inner) solve
    double tol_final; // p_tol^2: the requested relative residual, squared
    double alphah[2]; // alpha_{k-1}, written by CG iteration k in slot k & 1
    double cheb[2];   // c0, c1 of the Chebyshev polynomial preconditioner
    int32_t it_stop;  // iteration index at which the solve stopped (kIterInf: running)
    int32_t maxit;
    int32_t iters;
    int32_t converged;
    int32_t skip;     // 1: the refinement already meets the tolerance; later rounds do nothing
};

// State of the momentum predictor's BiCGStab (mom_tol > 0), on the device.
struct BicgState {
    double rho, rho_old, alpha, omega;  // (rh, r_k), (rh, r_{k-1}), alpha_k, omega_k
    double bb, rr;                      // ||b||^2 and ||r||^2 of the last checked iterate
    int32_t it_stop;                    // iteration count at the stop (kIterInf: running)
    int32_t iters, converged, pad;
};

// Per-member device state, read back by the host after a batch of work.
struct DevState {
    double dt, dt_prev, sigma, t;
    PcgState pcg;
    int32_t flags;
    int32_t pad0;
    double mass_gas;   // sum rho V of the last step
    double usq;        // sum |u|^2 of the last step
    double rho_min;
    double mass_p[kMaxClasses];
    double red[kMaxRed];
    // constants of the member: rho and p are stored as deviations from
    // (rho_ref, p_ref); particle response times
    double rho_ref, p_ref;
    double tau[kMaxClasses];
    double aff[2];     // per-member affine coefficients of a statistics pass
    // record of the current step, per corrector
    int32_t it_corr[kMaxCorr];     // CG iterations, all rounds
    int32_t rounds_corr[kMaxCorr]; // FP64 refinement rounds
    int32_t it_first[kMaxCorr];    // iterations of the first (fresh) solve
    int32_t it_later[kMaxCorr];    // most iterations of one later refinement round
    double rel_corr[kMaxCorr];     // final ||r|| / ||b||
    // accumulated over the steps since the host last cleared them
    int32_t flags_acc;
    int32_t steps_acc;
    int32_t it_first_max[kMaxCorr];
    int32_t it_later_max[kMaxCorr];
    // two-way coupling: mean mixture density <rho + sum_j rho_j> (a constant of
    // the run: gas and dust masses are conserved exactly)
    double rhom_mean;
    // the dust's Courant number of the step (max over the classes)
    double courant_dust;
    // BDF2 coefficients of the step (c0, c1, c2), written by the predictor
    double bdf[3];
    BicgState bicg;
};

// A cell and the periodic offsets to the cells up to two steps away along
// each axis (every stencil here reaches at most two cells): computed once per
// cell, so that each neighbour address is one add.
struct CellIdx {
    size_t p;               // this cell (member base included)
    int off[3][5];          // off[d][s + 2]: index offset of the cell s steps along d
    __device__ inline CellIdx(int n, int i, int j, int k, size_t base) {
        p = base + (size_t)i + (size_t)n * ((size_t)j + (size_t)n * (size_t)k);
        const int nn = n * n;
#pragma unroll
        for (int s = -2; s <= 2; ++s) {
            off[0][s + 2] = wrap_delta(i, s, n);
            off[1][s + 2] = wrap_delta(j, s, n) * n;
            off[2][s + 2] = wrap_delta(k, s, n) * nn;
        }
    }
    static __device__ inline int wrap_delta(int i, int s, int n) {
        int a = i + s;
        a = a < 0 ? a + n : (a >= n ? a - n : a);
        return a - i;
    }
    // cell reached by s steps along axis d (|s| <= 2)
    __device__ inline size_t sh(int d, int s) const {
        return p + (size_t)(ptrdiff_t)off[d][s + 2];
    }
    __device__ inline size_t self() const { return p; }
};

// Fourth-order central interpolation onto face P + (s + 1/2) e_d:
// weights (-1, 9, 9, -1)/16 on cells P+s-1 .. P+s+2 along d.
template <typename T>
__device__ inline T i4(const T* __restrict__ q, const CellIdx& c, int d, int s) {
    T a = q[c.sh(d, s - 1)], b = q[c.sh(d, s)], e = q[c.sh(d, s + 1)], f = q[c.sh(d, s + 2)];
    return (T(9) * (b + e) - (a + f)) * T(0.0625);
}

// I4 of T-stored values evaluated in the arithmetic of R (FP64 evaluation of
// FP32-stored fields).
template <typename R, typename T>
__device__ inline R i4r(const T* __restrict__ q, const CellIdx& c, int d, int s) {
    R a = (R)q[c.sh(d, s - 1)], b = (R)q[c.sh(d, s)], e = (R)q[c.sh(d, s + 1)],
      f = (R)q[c.sh(d, s + 2)];
    return (R(9) * (b + e) - (a + f)) * R(0.0625);
}

// Scheduling fence placed after a cell's gathered loads: the compiler may not
// move the arithmetic that uses them above it, nor the loads below it, so all
// of the cell's loads are in flight before the first wait.
__device__ inline void loads_issued() { __builtin_amdgcn_sched_barrier(0); }

// A field on the cross-shaped stencil of reach 2, gathered into registers so
// that all of its loads are in flight together: v[0] is the cell, v[1 + 4d + t]
// the cells -2, -1, +1, +2 (t = 0..3) steps along axis d.
template <typename T>
__device__ inline void gather13(const T* __restrict__ q, const CellIdx& c, T (&v)[13]) {
    v[0] = q[c.self()];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        v[1 + 4 * d] = q[c.sh(d, -2)];
        v[2 + 4 * d] = q[c.sh(d, -1)];
        v[3 + 4 * d] = q[c.sh(d, 1)];
        v[4 + 4 * d] = q[c.sh(d, 2)];
    }
}

// The gathered value s steps along d (|s| <= 2).
template <typename T>
__device__ inline T g13(const T (&v)[13], int d, int s) {
    return s == 0 ? v[0] : v[1 + 4 * d + (s < 0 ? s + 2 : s + 1)];
}

// I4 onto face P + (s + 1/2) e_d from gathered values (same operations as i4).
template <typename T>
__device__ inline T i4g(const T (&v)[13], int d, int s) {
    const T a = g13(v, d, s - 1), b = g13(v, d, s), e = g13(v, d, s + 1), f = g13(v, d, s + 2);
    return (T(9) * (b + e) - (a + f)) * T(0.0625);
}

// I4 of gathered values evaluated in the arithmetic of R (same operations as i4r).
template <typename R, typename T>
__device__ inline R i4gr(const T (&v)[13], int d, int s) {
    const R a = (R)g13(v, d, s - 1), b = (R)g13(v, d, s), e = (R)g13(v, d, s + 1),
            f = (R)g13(v, d, s + 2);
    return (R(9) * (b + e) - (a + f)) * R(0.0625);
}

// Gauss-I4 cell derivative along d from gathered values (same operations as dgauss).
template <typename T>
__device__ inline T dgauss13(const T (&v)[13], int d, T inv_h) {
    return (i4g(v, d, 0) - i4g(v, d, -1)) * inv_h;
}

// The cross of reach 1: v[0] the cell, v[1 + 2d] and v[2 + 2d] the cells -1
// and +1 along axis d.
template <typename T>
__device__ inline void gather7(const T* __restrict__ q, const CellIdx& c, T (&v)[7]) {
    v[0] = q[c.self()];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        v[1 + 2 * d] = q[c.sh(d, -1)];
        v[2 + 2 * d] = q[c.sh(d, 1)];
    }
}

// The five cells -2..2 along axis d: v[s + 2].
template <typename T>
__device__ inline void gather_line(const T* __restrict__ q, const CellIdx& c, int d, T (&v)[5]) {
#pragma unroll
    for (int s = -2; s <= 2; ++s) v[s + 2] = q[c.sh(d, s)];
}

// I4 onto face s + 1/2 along the gathered line (same operations as i4r).
template <typename R, typename T>
__device__ inline R i4l(const T (&v)[5], int s) {
    const R a = (R)v[s + 1], b = (R)v[s + 2], e = (R)v[s + 3], f = (R)v[s + 4];
    return (R(9) * (b + e) - (a + f)) * R(0.0625);
}

// Gauss-theorem cell derivative along d from I4 face values.
template <typename T>
__device__ inline T dgauss(const T* __restrict__ q, const CellIdx& c, int d, T inv_h) {
    return (i4(q, c, d, 0) - i4(q, c, d, -1)) * inv_h;
}

__device__ inline int flat_tid() { return threadIdx.x + blockDim.x * threadIdx.y; }
__device__ inline unsigned num_blocks() { return gridDim.x * gridDim.y * gridDim.z; }

constexpr unsigned kXcds = 8;   // accelerator complex dies, each with its own L2

// Logical number of this block.  The blocks of a launch are dealt to the XCDs
// round-robin in order of their hardware number; renumbering them so that each
// XCD receives one contiguous range of logical numbers keeps neighbouring tiles,
// and the halo cells they share, in the same XCD's L2.  Tiles, members and
// reduction partials are all indexed by the logical number.  REST: also where 8
// does not divide the blocks (a pressure solve of 160^3 takes 8 % less so, but one of
// 448^3 or 576^3 on the 64-wide CG tiles 5 % more).
template <bool REST = true>
__device__ inline unsigned flat_bid() {
    const unsigned f = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned B = num_blocks(), q = B / kXcds, r = B % kXcds, x = f % kXcds;
    if (!REST && r) return f;
    return x * q + (x < r ? x : r) + f / kXcds;   // the first r XCDs hold one block more
}

// Logical 3D block coordinates (x fastest) of this block.
struct BlockXYZ {
    int x, y, z;
};
template <bool REST = true>
__device__ inline BlockXYZ block_xyz() {
    const unsigned L = flat_bid<REST>();
    return {(int)(L % gridDim.x), (int)((L / gridDim.x) % gridDim.y),
            (int)(L / (gridDim.x * gridDim.y))};
}

// Store that streams past the caches: the written line does not displace
// lines still to be read (a z-march's halo rows and planes) from L2.
template <typename T>
__device__ inline void stream_st(T* p, T v) { __builtin_nontemporal_store(v, p); }

// Load of a value no other tile reads (a z-march's own point values), with
// the same streaming hint.
template <typename T>
__device__ inline T stream_ld(const T* p) { return __builtin_nontemporal_load(p); }

// Barrier that orders only LDS accesses across the block: it waits for this
// wave's LDS operations, not for its global loads in flight, so loads issued
// for a later plane of a z-march stay in flight across it (a plain
// __syncthreads() also waits for every outstanding global access).
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <bool MAX>
__device__ inline double combine(double a, double b) {
    if constexpr (MAX) return a > b ? a : b;
    else return a + b;
}

// v as seen through a DPP lane movement; lanes without a source get `idle`.
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double v, double idle) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v), o = __builtin_bit_cast(uint64_t, idle);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)u, CTRL,
                                                              ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32),
                                                              (int)(uint32_t)(u >> 32), CTRL, ROWS,
                                                              0xf, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int NV, unsigned MAXMASK, int CTRL, int ROWS>
__device__ inline void dpp_step(double (&v)[NV]) {
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        if ((MAXMASK >> c) & 1u) v[c] = combine<true>(v[c], dpp_move<CTRL, ROWS>(v[c], -__builtin_inf()));
        else v[c] = combine<false>(v[c], dpp_move<CTRL, ROWS>(v[c], 0.0));
    }
}

// The wave's total of each of NV values, valid in lane 63 (component c a
// maximum when bit c of MAXMASK is set, else a sum; the order of operations is
// fixed).  Shifts within each row of 16 lanes, then row 0 into 1 and 2 into 3,
// then rows 0-1 into 2-3, all by DPP register moves: through LDS permutes the
// 84 of a CG launch's seven sums took every wave of the block through the one
// LDS unit.
template <int NV, unsigned MAXMASK>
__device__ inline void wave_reduce_all(double (&v)[NV]) {
    dpp_step<NV, MAXMASK, 0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
    dpp_step<NV, MAXMASK, 0x112, 0xf>(v);
    dpp_step<NV, MAXMASK, 0x114, 0xf>(v);
    dpp_step<NV, MAXMASK, 0x118, 0xf>(v);
    dpp_step<NV, MAXMASK, 0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
    dpp_step<NV, MAXMASK, 0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
}

// Block reduction of NV values over the block's first `waves` waves of 64 (at
// most kMaxWaves; the others' values are not looked at).  Thread c < NV returns
// the total of component c.  The order of operations is fixed, so the result
// is bitwise reproducible.  The waves' totals are combined by one thread per
// component with all of its LDS reads in flight together: one thread reading
// them all in turn was a chain of NV x waves LDS latencies at both ends of
// every CG launch.  With the totals above, a CG iteration takes 15.7 instead
// of 20.1 us at 32^3 and 34.6 instead of 43.8 us at 128^3 (FP64).  LDS_ONLY: the barrier orders only LDS accesses
// (lds_barrier), so global loads and stores in flight stay in flight.
constexpr int kMaxWaves = 16;
template <int NV, unsigned MAXMASK, bool LDS_ONLY = false>
__device__ inline double block_reduce(double (&v)[NV], double* lds, int waves) {
    const int tid = flat_tid();
    const int lane = tid & 63, wave = tid >> 6;
    if (wave < waves) {   // the same for the whole wave
        wave_reduce_all<NV, MAXMASK>(v);
        if (lane == 63)
#pragma unroll
            for (int c = 0; c < NV; ++c) lds[wave * NV + c] = v[c];
    }
    if (LDS_ONLY) lds_barrier();
    else __syncthreads();
    double acc = 0.0;
    if (tid < NV) {
        const bool mx = (MAXMASK >> tid) & 1u;
        double t[kMaxWaves];
#pragma unroll
        for (int w = 0; w < kMaxWaves; ++w) t[w] = lds[(w < waves ? w : 0) * NV + tid];
        acc = t[0];
#pragma unroll
        for (int w = 1; w < kMaxWaves; ++w) {
            const double u = mx ? combine<true>(acc, t[w]) : acc + t[w];
            acc = w < waves ? u : acc;
        }
    }
    return acc;
}
__device__ inline int block_waves() { return (int)(blockDim.x * blockDim.y + 63) >> 6; }

// Per-block partials of a grid-wide reduction: the block's totals go to
// part[c * num_blocks + block].  No fence is needed: the partials are consumed
// by a later kernel on the same stream.
template <int NV, unsigned MAXMASK, bool LDS_ONLY = false, bool REST = true>
__device__ inline void block_partials(double (&v)[NV], double* part) {
    __shared__ double lds[kMaxWaves * NV];
    const double t = block_reduce<NV, MAXMASK, LDS_ONLY>(v, lds, block_waves());
    const int c = flat_tid();
    if (c < NV) part[(size_t)c * num_blocks() + flat_bid<REST>()] = t;
}

// The same per chunk of a march (a batch's block totals each chunk that a single
// grid's block marches over): a wave leaves its totals of a chunk in LDS, and the
// waves are added after the march, in block_reduce's order, so that a chunk costs
// neither a barrier nor a chain of LDS reads.  us of an FP64 step with a block's total
// per chunk, so: 64 members of 16^3 1396 and 1226, 24 of 32^3 1363 and 1240.
__host__ __device__ constexpr size_t lds_after(size_t bytes) { return (bytes + 7) / 8 * 8; }
constexpr size_t chunk_sums_lds(int chunks, int threads, int columns) {
    return sizeof(double) * (size_t)chunks * (threads / 64) * columns;
}
template <int NV, unsigned MAXMASK>
struct ChunkSums {
    double* lds;    // chunk_sums_lds of them
    int held = 0;   // chunks added
    __device__ explicit ChunkSums(void* at) : lds(reinterpret_cast<double*>(at)) {}
    __device__ void add(double (&v)[NV]) {
        wave_reduce_all<NV, MAXMASK>(v);
        const int tid = flat_tid();
        if ((tid & 63) == 63)
#pragma unroll
            for (int c = 0; c < NV; ++c) lds[(held * block_waves() + (tid >> 6)) * NV + c] = v[c];
        ++held;
    }
    // chunk h to slot + h step of each column, the columns `column` apart
    __device__ void store(double* part, size_t column, size_t slot, size_t step) const {
        const int waves = block_waves();
        lds_barrier();
        for (int i = flat_tid(); i < held * NV; i += (int)blockDim.x) {
            const int h = i / NV, c = i - h * NV;
            const double* w0 = lds + h * waves * NV + c;
            double t = w0[0];
            for (int w = 1; w < waves; ++w) {
                const double x = w0[w * NV];
                t = (MAXMASK >> c) & 1u ? combine<true>(t, x) : t + x;
            }
            part[c * column + slot + h * step] = t;
        }
    }
};

// Partials of an earlier kernel on their way to this thread: its first one of
// each of NV columns (nbt apart, count nb from `first` on).  Loading them ahead
// of the totals (reduce_loaded) lets other loads be issued in between.
template <int NV>
struct PartLoad {
    const double* part;
    size_t nbt, first;
    unsigned nb;
    double x[NV];
};
template <int NV>
__device__ inline PartLoad<NV> load_partials(const double* __restrict__ part, size_t nbt,
                                             size_t first, unsigned nb) {
    PartLoad<NV> l;
    l.part = part;
    l.nbt = nbt;
    l.first = first;
    l.nb = nb;
    const unsigned tid = flat_tid(), b = tid < nb ? tid : nb - 1;
#pragma unroll
    for (int c = 0; c < NV; ++c) l.x[c] = part[(size_t)c * nbt + first + b];
    return l;
}

// The totals of the columns of l, in every thread.
template <int NV, unsigned MAXMASK, bool LDS_ONLY = false>
__device__ inline void reduce_loaded(const PartLoad<NV>& l, double (&out)[NV]) {
    __shared__ double lds[kMaxWaves * NV];
    __shared__ double tot[NV];
    const unsigned tid = flat_tid(), nthr = blockDim.x * blockDim.y;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const bool mx = (MAXMASK >> c) & 1u;
        out[c] = tid < l.nb ? l.x[c] : (mx ? -__builtin_inf() : 0.0);
    }
    for (unsigned b = tid + nthr; b < l.nb; b += nthr)
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const double x = l.part[(size_t)c * l.nbt + l.first + b];
            out[c] = ((MAXMASK >> c) & 1u) ? combine<true>(out[c], x) : out[c] + x;
        }
    const int held = (int)((l.nb + 63) >> 6), waves = block_waves();   // waves that hold partials
    const double t = block_reduce<NV, MAXMASK, LDS_ONLY>(out, lds, held < waves ? held : waves);
    if (tid < NV) tot[tid] = t;
    if (LDS_ONLY) lds_barrier();
    else __syncthreads();
#pragma unroll
    for (int c = 0; c < NV; ++c) out[c] = tot[c];
}

// Totals of count partials per column starting at `first`, columns nbt apart.
template <int NV, unsigned MAXMASK, bool LDS_ONLY = false>
__device__ inline void reduce_partials_strided(const double* __restrict__ part, size_t nbt,
                                               size_t first, unsigned nb, double (&out)[NV]) {
    reduce_loaded<NV, MAXMASK, LDS_ONLY>(load_partials<NV>(part, nbt, first, nb), out);
}

// Totals of one member's partials: an earlier kernel with nbt blocks in all
// wrote column c of block b at part[c nbt + b]; member m owns the blocks
// [m nbt/batch, (m+1) nbt/batch).
template <int NV>
__device__ inline PartLoad<NV> load_member(const double* __restrict__ part, unsigned nbt, int batch,
                                           int m) {
    const unsigned per = nbt / (unsigned)batch;
    return load_partials<NV>(part, nbt, (size_t)m * per, per);
}
template <int NV, unsigned MAXMASK, bool LDS_ONLY = false>
__device__ inline void reduce_member(const double* __restrict__ part, unsigned nbt, int batch,
                                     int m, double (&out)[NV]) {
    reduce_loaded<NV, MAXMASK, LDS_ONLY>(load_member<NV>(part, nbt, batch, m), out);
}

// Totals of partials written by an earlier kernel with `nb` blocks.  Every
// block of the calling kernel computes the same totals in the same order
// (bitwise identical, deterministic); all threads receive them.
template <int NV, unsigned MAXMASK>
__device__ inline void reduce_partials(const double* __restrict__ part, unsigned nb,
                                       double (&out)[NV]) {
    reduce_partials_strided<NV, MAXMASK>(part, nb, 0, nb, out);
}

// Round to nearest even FP32 -> BF16 (bit pattern); NaN stays NaN.
__host__ __device__ inline uint16_t f2bf(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Pressure deviation p(rho) - p_ref for rho = rho_ref + r (p_ref = C rho_ref^gamma),
// written with log1p/expm1 so that it stays accurate for small r in FP32.
__device__ inline double pdev(double r, double rho_ref, double p_ref, double gamma) {
    return p_ref * expm1(gamma * log1p(r / rho_ref));
}
__device__ inline float pdev(float r, double rho_ref, double p_ref, double gamma) {
    return (float)p_ref * expm1f((float)gamma * log1pf(r / (float)rho_ref));
}

}  // namespace pisoc
