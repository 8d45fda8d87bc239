// launch.hpp -- host-side launch wrappers of the PISO kernels (one set per
// storage type T), used by the step orchestration in pisoc.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "device.hpp"

namespace pisoc {

struct Launch {
    dim3 grid, block;
    unsigned nblocks;   // all members
    int cz;             // cells per thread along z
    int nz;             // blocks per member along z
    int v = 0;          // CG kernel: cells per lane along x of the full-row form (0: tiles)
    int h = 0;          // and wavefronts per x-row
    int rows = 0;       // and x-rows per block of its flat form (0: another form)
    int sub = 0;        // planes per partial sum of a block (cz, or a divisor of it)
    unsigned nparts = 0;   // partial sums per column, all members
    bool gathered = false;   // a fused pass on the gathered launch (k_gather)
    bool nt = false;    // and its once-read fields streamed past the caches (make_spmv_launch)
};

constexpr int kTargetBlocks = 2048;
constexpr int kTX = 64, kTY = 8;     // x-y tile of the z-marching kernels
constexpr int kTiledBlocks = 1024;

// Blocks of 64x4 (n >= 64) or 32x8 threads over x-y; each thread walks cz
// consecutive cells along z, with cz chosen for about kTargetBlocks blocks.
Launch make_launch(int n, int batch = 1);

// The same kernels with blocks of bx x (kBlock / bx) threads and cz cells per
// thread along z (bx a power of two in 16..256, 1 <= cz <= n).
Launch make_launch_shaped(int n, int batch, int bx, int cz);

// Launch of the z-marching field kernels: on 64 x 8 tiles for n a multiple of 64
// from 128 on, marching over at least 8 planes; else from 40 on on flattened rows
// (rows x-rows per block), whole ones up to 128 (flat_field_rows) and segments of
// them (seg_width) beyond; below 40 nblocks is 0.  Blocks march
// over exactly min(cz_tile, n) planes when cz_tile > 0 (a tuned choice; the
// default's own cz changes nothing).
// The tiles against flattened rows or segments, us of a step's field kernels, tiles
// first: FP32 128^3 573, 621; 192^3 1633, 1850; 256^3 3830, 5200; 320^3 7370, 8580; FP64
// 192^3 2690, 2820; 256^3 6090, 6960; 320^3 12230, 12580; at 128^3 alone, and in FP64
// alone, the rows are the faster (854, 788).
// Flattened rows: as many as fit 512 threads (256 registers a thread in FP64), at
// least 4, so that the y halo is no larger than the block's own rows: n <= 128.
// Below n = 40 the gathered kernels are as fast (the launch's latency is all).
// z is cut for one block per CU: a single grid of 70^3 takes 3-plane marches.  A
// batch's blocks march over several of the single grid's chunks (16 members of 64^3
// in 3-plane marches took 18 % longer, reading two halo planes for each of their
// own), as cut_by_rounds has it, and add their sums up per chunk, so that a member's
// (mass, ||b||^2) are those of a run of its own.  ms of a step cut for one block per
// CU over all members, so: FP32 12 members of 64^3 2.10 and 1.92, 24 3.91 and 3.50; FP64
// 24 of 64^3 6.52 and 6.21, 8 of 100^3 8.10 and 7.27.
constexpr int kFlatFieldRows = 4, kFlatFieldThreads = 512, kFlatFieldBlocks = 256;
constexpr int kFlatFieldMinN = 40, kFlatFieldMaxN = kFlatFieldThreads / kFlatFieldRows;
constexpr int flat_field_rows(int n) {
    return n >= kFlatFieldMinN && n <= kFlatFieldMaxN ? kFlatFieldThreads / n : 0;
}
// Segments: the fewest per row of at most kSegMost columns, in whole 64-byte lines
// of doubles, so 64 to 96 columns and 5 to 7 rows per 512 threads (whole rows of
// 160 would leave 3 rows a y halo larger than themselves).  Up to kCutMinN z is cut
// for kSegBlocks blocks and marches of at least 8 planes, whatever the batch: half as
// many blocks took 9 % longer for an FP64 step of 200^3 (6 % less at 136^3), twice
// as many 1-2 % longer from 136^3 to 200^3, four times 3-7 %.
// Beyond, a plane alone takes hundreds of blocks, and a count just past a multiple of
// the CUs leaves most of them idle in the last round: cut_by_rounds, of 9 cuts into 1
// to 11 chunks swept at 17 sizes and precisions from 264 to 500 within 3 % of the
// fastest each time.  Field kernels of a step, ms, gathered, 512 blocks, now: FP32
// 288^3 7.6, 6.9, 5.9; 336^3 13.6, 16.2, 11.4; 352^3 14.4, 18.0, 12.9; 400^3 24.2, 20.7,
// 16.2; FP64 336^3 25.5, 23.7, 16.1; 400^3 45.1, 30.7, 23.9.
constexpr int kSegBlocks = 512, kCutMinN = 256, kCutHalo = 4;
constexpr int kSegMost = 96, kSegWidth = 64, kSegRows = 5;
__host__ __device__ constexpr int seg_width(int n, int gx) { return ((n + gx - 1) / gx + 7) / 8 * 8; }
Launch make_tiled_launch(int n, int batch = 1, int cz_tile = 0);

// Launch of the CG kernel for fields of elem_bytes per value.
// * n = 128 and 256: the full-row form, blocks of kRowWaves wavefronts, about
//   kRowBlocks blocks per member (v cells per lane, h wavefronts per row): at
//   256 one wavefront per x-row and 4 cells per lane in FP32, two per x-row and
//   2 cells per lane in FP64 (4 doubles per lane spill registers); at 128 one
//   wavefront per x-row and 2 cells per lane.
// * Multiples of 64 from 320 on: tiles of 64 x (8 spmv_rows) cells, 64 x 8
//   threads each owning spmv_rows rows (v = 0; two rows in FP64 halve the
//   tile's y halo; in FP32 two measured no faster).  At 320 the flat form took
//   643 against 549 us in FP64 (272 against 255 in FP32): three rows per block
//   leave it a y halo as large as the tile; at 192 and below it is the faster.
// * Other multiples of kSmallTX beyond small_tiles_above: tiles of kSmallTX x
//   kSmallTX cells, one thread per column (block.x = kSmallTX), kSmallChunks chunks
//   of z.  There two full rows are all that the flat form's LDS holds (FP64) or none
//   (FP32, and FP64 from 385 on, where the gathered form would be left).  us per
//   iteration in FP64, flat or gathered, tiles: 336^3 776, 745; 352^3 914, 871; 368^3
//   1019, 1017; 400^3 2367, 1266; 480^3 3886, 2255; 624^3 8999, 4832; in FP32 528^3
//   2779, 2099; 624^3 3960, 3392, but 352^3 398, 622.  Of 1 to 12 chunks 4 is within
//   4 % of the fastest at 19 sizes.
// * Every other n with flat_rows(n) >= 2 (FP64 up to 384, FP32 up to 512): the flat
//   form, rows x-rows per block.
// nblocks is 0 when none is available.  Tiles march over at least 8 planes, or
// like the flat form's single grids over exactly min(cz_tile, n) when cz_tile > 0
// (a tuned choice; the full-row form ignores it).
// nt (full-row form): the fields a CG iteration reads once (r, q, p_old of the
// main rows) are loaded non-temporally, so that w and diag, which every
// iteration of a solve reads again, stay in the memory-side cache (kMallBytes)
// between launches.  Taken when the iteration's nine fields do not fit in that
// cache but w and diag fit in 60 % of it: at 256^3 in FP32 the CG then takes
// 5 % less time; in FP64 (w and diag 268 MB) it took 8 % more.
constexpr double kMallBytes = 256.0 * 1024 * 1024;
constexpr int spmv_rows(int elem_bytes) { return elem_bytes == 8 ? 2 : 1; }
constexpr int kFlatBeforeTiles = 256;
constexpr int kSmallTX = 16, kSmallChunks = 4;
constexpr int small_tiles_above(int elem_bytes) { return elem_bytes == 8 ? 320 : 512; }
// Rows per block of the flat form: as many as fit 512 threads up to n = 64, 768
// up to 100, 1024 beyond (larger blocks read less halo; smaller ones spread the
// same planes over more CUs and shorter marches), but up to n = 40 in
// about 8 blocks per plane, of at least 8 rows, where whole planes would leave CUs
// idle and a few rows make a batch of many blocks.  ms of a step with 8 blocks of 2 to
// 4 rows, with 8 rows: 64 members of 16^3 1.40 and 0.95 (1.25 on 16 x 16 tiles), 24 of
// 32^3 1.36 and 1.23 (1.35); us per iteration of one grid of 16^3 9.1 and 8.5, of 32^3
// 9.5 and 9.5.  z is then cut for one
// block per CU (kFlatBlocks), so that no block waits for another to end and the
// launch's head totals few partials: of the shapes swept from 16 to 256 in both
// precisions the rule's is within 10 % of the fastest, and half or twice as many
// blocks take 5-40 % longer.  From n = 257 on by cut_by_rounds, of 11 cuts swept at 18
// sizes within 5 % of the fastest (FP64 330^3 757 us per iteration, 360^3 1196 with
// two blocks per CU and 975 now; FP32 400^3 632 and 552).
// A batch has blocks enough without short marches, and with the single grid's
// most of a block's time is its head and halo planes: its blocks march over
// several chunks (the partial sums stay per chunk, so a member's are those of a run
// of its own), for at most kFlatBatchBlocks in all, and up to 512 threads for no
// more waves than are resident at once (kFlatBatchWaves: 16 per CU, four per SIMD).
// Captured FP32 steps, ms, with at most 1024 blocks, so: 12 members of 48^3 1.57 and
// 1.44 (16 x 16 tiles 1.43), 10 of 52^3 1.53 and 1.41, 8 of 56^3 1.49 and 1.36, 6 of 64^3
// 1.33 both; 24 of 32^3 0.94, with half as many blocks 1.04.  Wider blocks, one per
// CU, gain from 256 blocks at some sizes (5 of 80^3 2.23 and 2.01) and lose at others
// (6 of 120^3 9.13 and 10.67 in FP64).
// The block's LDS (two plane sets of R + 4 rows of w and R + 2 of p) stays
// within kFlatLds beside the reduction's.
constexpr int kFlatBlocks = 256, kFlatBatchBlocks = 1024, kFlatBatchWaves = 4096;
constexpr size_t kFlatLds = 60 * 1024, kFlatLdsAll = 62 * 1024;   // without, with a batch's chunk sums
constexpr size_t flat_cg_lds(int n, int rows, int elem_bytes) {
    return (size_t)2 * (2 * rows + 6) * n * elem_bytes;
}
constexpr int flat_rows(int n, int elem_bytes) {
    int r = (n <= 64 ? 512 : n <= 100 ? 768 : 1024) / n;
    if (n <= 40) r = n <= 32 ? 8 : (n + 7) / 8;
    while (r >= 2 && flat_cg_lds(n, r, elem_bytes) > kFlatLds) --r;
    return r;
}
constexpr int kRowWaves = 8, kRowBlocks = 256;
// Wavefronts per x-row of the full-row CG form for n and elem_bytes (0: none).
constexpr int row_waves(int n, int elem_bytes) {
    return n == 128 ? 1 : n != 256 ? 0 : elem_bytes == 4 ? 1 : 2;
}
Launch make_spmv_launch(int n, int batch, int elem_bytes, int cz_tile = 0);

// dst[0..count) = v (FP64).
void fill_value(hipStream_t s, double* dst, size_t count, double v);

// psi/dt = diag - (1/h^2) sum_f I4(w)_f of a captured pressure system (n^3 FP64).
void psidt_of(hipStream_t s, int n, const double* diag, const double* w, double* out);

// Partial-sum columns written by one CG iteration.
constexpr int kCgCols = 7;
// The momentum predictor's BiCGStab: partial slots from PS_CG for (rh.r, r.r,
// b.b), (rh.v) and (t.s, t.t).
constexpr int kBicgRes = 0, kBicgV = 3, kBicgTs = 4;
// Chebyshev-preconditioned CG: one set of columns per iteration (r.z, r.r,
// p.q), sets alternating by k & 1 from PS_CG, the interval's end after them.
constexpr int kChebRes = 0, kChebDir = 2, kChebSet = 3;

// Partial-sum slots in the workspace (columns of num_blocks doubles each).
enum PartSlot {
    PS_U = 0,      // 3 columns: r.z, r.r, b.b (CG system set-up)
    PS_CG = 3,     // 2 x kCgCols columns: CG iteration k in set k & 1
    PS_MASS = PS_CG + 2 * kCgCols,   // 3 columns: sum r, sum |u|^2, max(-rho)
    PS_CFL = PS_MASS + 3,            // 1 column: Courant maxima (k_cfl); must follow PS_MASS
    PS_STAT = PS_CFL + 1,            // 4 columns: statistics
    // 2 kMaxClasses columns: class c's dust finish writes, from PS_DUST + 2c
    // on, columns of nb partials each: sum rho_j, then max(-rho_j)
    PS_DUST = PS_STAT + 4,
    // 2 kMaxClasses columns: class c's first sweep writes, from PS_DDIAG + 2c
    // on, columns of nb partials each: max(-diagonal) of its implicit
    // equation, then its maximal Courant rate sum_f |G_f| / (2 rho V)
    PS_DDIAG = PS_DUST + 2 * kMaxClasses,
    PS_COLUMNS = PS_DDIAG + 2 * kMaxClasses
};

// Operands of CG iteration k.  Reads r_{k-1}, p_{k-1}, q_{k-1} (rin, pold,
// qold; only rin = r_0 at k = 0), diag and w, and at even k >= 2 p_{k-2}
// (pold2) and x; writes r_k (k >= 1), p_k, q_k and, at even k and at the
// stop, x.  part_in: the partials of iteration k-1 (kCgCols columns),
// at k = 0 those of the set-up kernel (r.z, r.r, b.b), written by nb_in
// blocks; part_out: this iteration's.  fresh: the set-up's b.b is the
// reference ||b||^2 of the solve; xzero: the solve started from x = 0 without
// x being written.
template <typename T>
struct CgArgs {
    const T* rin;
    T* rout;
    const T *diag, *w, *pold, *pold2;
    T* pnew;
    const T* qold;
    T *q, *x;
    const double* part_in;
    unsigned nb_in;
    double* part_out;
    int fresh, maxit, xzero;
};

template <typename T>
struct Ops {
    static void cast_in(hipStream_t s, const double* src, T* dst, size_t count, double shift);
    static void cast_out(hipStream_t s, const T* src, double* dst, size_t count, double shift);
    // one member's pressure p_ref + p_dev(r) (r points at the member's cells)
    // p = C rho^gamma, or rho R T with temp non-null (Fourier closure)
    static void pressure_out(hipStream_t s, const Phys& ph, double rho_ref, double p_ref,
                             const T* r, double* dst, const double* temp = nullptr);
    static void init_phi(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                         const T* r, const T* u, T* phi);
    static void cfl(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                    const T* r, const T* phi, double* part);
    // TL: the tiled z-march when available; nb_cfl: the number of Courant
    // partials in part_cfl (from cfl, or from the previous step's last
    // corrector pass)
    static void predict(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                        DevState* st, const double* part_cfl, unsigned nb_cfl, double dt_fixed,
                        double cfl, double growth, double dt_max, const T* rn, const T* un,
                        const T* phi, T* rs, T* aP, T* divu, T* pn);
    // Field kernels taking TL run as k_tiled z-marches when TL.nblocks > 0;
    // those that write partials return how many (blocks of the launch used).
    static void mom_source(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                           const DevState* st, const T* rn, const T* un, const T* divu, T* src);
    // TL: tiled launch (used when TL.nblocks > 0)
    static void mom_sweep(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                          const DevState* st, const T* uin, T* uout, const T* phi, const T* aP,
                          const T* src, const T* pn);
    static void hbya(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                     const DevState* st, const T* uin, T* hb, const T* phi, const T* aP,
                     const T* src, const T* rk, T* w, T* p0);
    // CG starts from x = 0 without x being written (see pcg_spmv's xzero).
    // TL: the tiled z-march when available.  Returns the number of partials
    // written to part_u (blocks of the launch used).
    static unsigned corr_rhs(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                             DevState* st, const T* rn, const T* rk, const T* w, const T* hb,
                             const T* p0, T* phiH, T* r, T* diag, double* part_u, double* snap_b,
                             double* snap_diag, double* snap_p0, double* b64);
    // from_zero: x64 is zero and not read (first round of a solve from zero);
    // xf: the new x64n rounded to T (not aliasing d); store_x = false (with
    // from_zero): x64n = d exactly, neither x64n nor xf is written
    static unsigned refine(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                           DevState* st, const double* x64, const T* d, double* x64n, T* xf,
                           const double* b64, const T* w, const T* diag, T* r32,
                           double* part_u, bool from_zero, bool store_x);
    // CG iteration k (one kernel); TL: the CG launch of make_spmv_launch
    // (used when TL.nblocks > 0)
    static void pcg_iter(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                         DevState* st, int k, const CgArgs<T>& a);
    static void helm_apply(const Launch& L, hipStream_t s, const Phys& ph, const T* psidt,
                           const T* w, const T* x, T* y);
    // the momentum predictor solved to a tolerance: BiCGStab set-up (x = u^n
    // in place) and iteration i >= 1 (three launches)
    static void bicg_init(const Launch& L, hipStream_t s, const Phys& ph, DevState* st, const T* x,
                          const T* F, const T* aP, const T* src, const T* pn, T* r, T* rh,
                          double* part);
    static void bicg_iter(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                          DevState* st, int i, double tol2, int maxit, T* x, T* r, const T* rh,
                          T* const w[6], const T* F, const T* aP, double* part_res, double* part_v,
                          double* part_ts);
    // Fourier closure: the energy predictor's coefficients and one Jacobi sweep
    static void energy_setup(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                             const T* rn, const T* rs, const T* phi, const T* divu, const T* pn,
                             double* aT, double* sT);
    static void energy_sweep(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                             const DevState* st, const double* tin, double* tout, const T* phi,
                             const double* aT, const double* sT);
    // CG preconditioned by a Chebyshev polynomial (stand-alone solve): the
    // interval's lower end, then per iteration the residual/preconditioner and
    // the direction/operator launches
    static void cheb_theta(const Launch& L, hipStream_t s, const Phys& ph, const T* psidt,
                           const T* diag, double* part);
    static void cheb_res(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                         DevState* st, int k, const T* rin, T* rout, const T* q, const T* p,
                         const T* diag, const T* w, T* x, T* z, const double* part_theta,
                         unsigned nb_theta, const double* part_prev, double* part_out);
    static void cheb_dir(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                         DevState* st, int k, const T* z, const T* pin, T* pout, T* q,
                         const T* diag, const T* w, const double* part_u, unsigned nb_u,
                         const double* part_prev, double* part_cur, int maxit);
    static void helm_start(const Launch& L, hipStream_t s, const Phys& ph, DevState* st,
                           const T* psidt, const T* w, const T* b, const T* x, T* r, T* diag,
                           double* part_u);
    static void corr_flux(const Launch& L, hipStream_t s, const Phys& ph, const T* p0, const T* x,
                          const T* w, const T* phiH, T* phik, T* pt, double* snap_x);
    // corr_flux and corr_update in one pass (TL: the tiled or the gathered launch), p not
    // stored; the last corrector writes, from part_mass on, columns of nb
    // partials each: the three of the mass budget, then the Courant maxima of
    // the new state (4 nb <= 4 max_blocks: within PS_MASS and PS_CFL).
    // Returns nb.
    static unsigned corr_finish_fused(const Launch& TL, hipStream_t s, const Phys& ph,
                                      const DevState* st, bool last, const T* p0, const T* x,
                                      const T* w, const T* phiH, T* phik, double* snap_x,
                                      const T* rn, const T* hb, const T* aP, T* rk, T* u,
                                      double* part_mass);
    static unsigned corr_update(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                                bool last, const T* rn, const T* phik, const T* hb, const T* pt,
                                const T* aP, T* rk, T* u, double* part_mass);
    static void dudt(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                     const DevState* st, const T* un, const T* u1, T* acc);
    static void dust_flux(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                          const DevState* st, int cls, const T* phi, const T* r1, const T* acc,
                          T* G, const T* rhoj, const T* rn, T* Y);
    // part_diag non-null (the class's first sweep): partials max(-diagonal)
    // of the implicit equation and max of the dust's Courant rate (two
    // columns of the launch's block count); returns the launch's block count
    static unsigned dust_sweep(const Launch& L, const Launch& TL, hipStream_t s, const Phys& ph,
                               const DevState* st, const T* Yin, T* Yout, const T* G,
                               const T* rhoj, const T* r1, double* part_diag);
    static void dust_faceflux(const Launch& L, hipStream_t s, const Phys& ph, const T* Y, T* G);
    // partials: two columns of L.nblocks from part on, sum rho_j and max(-rho_j);
    // fdo (two-way coupling, else null): the class's own-face fluxes go into the
    // next step's dust flux F_d (written by the first class, added by the others)
    static void dust_finish(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                            const T* rhoj, const T* F, T* rhoj1, double* part, T* fdo,
                            bool first);
    // two-way coupling: initial dust mass fluxes fd = I4(sum_j rho_j) I4(u) A
    static void init_fd(const Launch& L, hipStream_t s, const Phys& ph, int ncls,
                        const T* rhoj, const T* u, T* fd);
    // two-way coupling: a_P and the source of the mixture, and its mass flux fm
    static void mixture(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                        int ncls, const T* rn, const T* un, const T* rhoj, const T* phi,
                        const T* fd, T* fm, T* aP, T* src);
    // dust_faceflux and dust_finish in one tiled pass (TL.nblocks > 0), F not
    // stored; returns the number of partials written per column (two columns,
    // as dust_finish)
    static unsigned dust_finish_fused(const Launch& TL, hipStream_t s, const Phys& ph,
                                      const DevState* st, const T* Y, const T* G,
                                      const T* rhoj, T* rhoj1, double* part, T* fdo,
                                      bool first);
    static void stats_gas(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                          const T* r, const T* u, double* part);
    // st non-null: per-member (a, b) = st[m].aff
    static void sum_affine_sq(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                              const T* x, double a, double b, double* part);
    // learned guess
    static void net_stats(const Launch& L, hipStream_t s, const Phys& ph, const T* b,
                          const T* diag, const T* p0, double* part);
    static void net_input(const Launch& L, hipStream_t s, const Phys& ph, DevState* st,
                          const double* part, const T* b, const T* diag, const T* p0,
                          uint16_t* x4, float* x2, const T* psol, float* tgt);
    // g = s1 y (y: the network's output) or, with gd set, g = gd
    static void guess_start(const Launch& L, hipStream_t s, const Phys& ph, const DevState* st,
                            const float* y, const T* gd, const T* w, const T* diag, const T* b,
                            const double* b64, T* g, T* mg, double* part);
    static void guess_apply(const Launch& L, hipStream_t s, const Phys& ph, DevState* st,
                            const double* part_g, const T* g, const T* mg, const T* diag, T* r,
                            T* x, double* x64, const double* b64, T* bsave, double* part_u);
    // per member, where the guess does not lower ||r|| (totals in st[m].red[1..2])
    static void guess_revert(const Launch& L, hipStream_t s, const Phys& ph, DevState* st, T* r,
                             T* x, double* x64, const double* b64, const T* bsave,
                             const T* diag, double* part_u);
};

// Per member: totals of nv partial columns (written by a launch of nbt blocks
// over `batch` members) into st[m].red[off ..].
void finalize_sums(hipStream_t s, const double* part, unsigned nbt, int batch, int nv,
                   DevState* st, int off);
// Total of nb partials (one column) into dst[0].
void sum_partials(hipStream_t s, const double* part, unsigned nb, double* dst);
// Per member: end-of-step mass budget and flags.
// nb_mass: partials of the last corrector update; nb_dust: of the dust finish
// (class c's two columns from part_dust + 2 c cls_stride); nb_diag: of the
// first dust sweep (class c's two columns from part_diag + 2 c cls_stride)
void step_finish(hipStream_t s, const Phys& ph, DevState* st, const double* part_mass,
                 unsigned nb_mass, const double* part_dust, int ncls, unsigned nb_dust,
                 const double* part_diag, unsigned nb_diag, size_t cls_stride);
// Per member: t += dt, dt_prev = dt (the step is accepted); fold the step
// record into the accumulators.
void commit(hipStream_t s, DevState* st, int batch);
// Per member: clear the accumulators.
void clear_acc(hipStream_t s, DevState* st, int batch);
// Per member: the end of a refinement round, from its column ||r64||^2 of nbt
// partials (see k_refine_end).
void refine_end(hipStream_t s, const double* part, unsigned nbt, int batch, DevState* st, int corr,
                int round, double tau_min);
// Per member: CG tolerance (squared) for the next solve.
void set_tol(hipStream_t s, DevState* st, int batch, double tol2);
// Per member: affine coefficients for sum_affine_sq (see k_set_affine).
void set_affine(hipStream_t s, DevState* st, int batch, int mode, double N);
// Per member: corrector corr's solves in the step record, and the next fresh
// solve's tolerance (see k_record_solve).
void record_solve(hipStream_t s, DevState* st, int batch, int corr, int round, bool refined,
                  double tol2);
// Per member: clear the step flags; the first solve's tolerance.
void clear_flags(hipStream_t s, DevState* st, int batch, double tol2);

}  // namespace pisoc
