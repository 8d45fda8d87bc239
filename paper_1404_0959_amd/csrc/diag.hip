// diag.hip -- diagnostics of the velocity field on gfx950: the energy
// spectrum and the Taylor micro-scale (through a radix-4 Stockham FFT whose
// lines cross LDS between stages), and the second invariant Q of the velocity
// gradient.  These are the paper's validation quantities of the flow (Results
// section: energy spectrum, Taylor micro-scale; third figure: Q iso-surfaces).
//
// Filtered statistics: the separable top-hat of width 2h (weights 1/4, 1/2,
// 1/4 per axis), the sub-grid stress, its energy and the energy flux to the
// sub-grid scales (the a-priori tests the paper plans for its DNS data base).
//
// Spectrum: u_hat(k) = DFT(u)(k) / n^3 over integer wavevectors with
// components in [-n/2, n/2); shell s gathers the k with s - 1/2 <= |k| <
// s + 1/2, E(s) = sum over the shell of |u_hat|^2 / 2, so sum_s E(s) =
// <|u|^2>/2.  Taylor micro-scale lambda = sqrt(5 sum E / D) with D = sum_k
// |k|^2 |u_hat(k)|^2 / 2.  Every sum runs in a fixed order (bitwise
// reproducible).
//
// Also here: the plain streaming kernel that measures the practical HBM
// ceiling of a given mix of reads and writes (no stencil, no reduction).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdint>
#include <new>
#include <utility>

#include "../../include/pisoc.h"
#include "device.hpp"

namespace pisoc {
namespace {

using cplx = double2;

// ---- FFT ----
// Radix-4 Stockham transforms (one radix-2 stage first when log2 n is odd) of
// lines of n complex values, a block holding L lines in LDS, one radix-4
// butterfly per thread and stage.  A stage with sub-transforms of size Ns takes
// x[j + r n/4], r = 0..3, times exp(-2 pi i k r / (4 Ns)), k = j mod Ns, and leaves
// its four outputs at 4 (j - k) + k + r Ns.  The first stage's inputs come
// straight from global memory and the last one's outputs leave from registers,
// so a line crosses LDS once per stage boundary.
//
// The input is real: the x pass transforms two rows as one complex line and
// keeps the H = n/2 + 1 non-negative kx of each (f(-k) = conj f(k)); y and z
// passes run on that half, the z pass bins |f|^2 without writing it back.  The
// three components share every launch.  Bound: memory, 8 + 8 (x), 16 (y) and 8
// bytes per cell and component (z) against 120 with full complex fields and
// separate binning passes.  256^3, all components: 0.15 ms each for x and y (5.4
// TB/s), 0.21 for z and the shells, in place of 3.2 together.
constexpr int kFftItems = 512;       // butterflies per block and stage
constexpr int kSpecBlocks = 768;     // blocks (partials) of the binning pass
constexpr int kMaxBins2 = 2;         // shells per thread: at most 888 (n = 1024) over 512

bool pow2(int n) { return n >= 8 && n <= 1024 && (n & (n - 1)) == 0; }
int ilog2(int n) {
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

// Shell of an integer |k|^2: s with s - 1/2 <= sqrt(k2) < s + 1/2, in integers
// ((s + 1/2)^2 <= k2 <=> k2 >= s^2 + s + 1 for integer k2).
inline int shell_of(int64_t k2) {
    int64_t s = (int64_t)sqrt((double)k2);
    while (s * s > k2) --s;
    while ((s + 1) * (s + 1) <= k2) ++s;
    return (int)(s + (k2 >= s * s + s + 1 ? 1 : 0));
}

// Pitch of a half row of n/2 + 1 values: whole 128-byte lines, so that the y and z
// passes' tiles of 8 kx are lines.
__host__ __device__ inline int half_pitch(int n) { return (n / 2 + 8) / 8 * 8; }
// and of a plane: one line more than its rows, so that a z line's values do not
// all lie a multiple of 32 KiB apart.
__host__ __device__ inline size_t plane_pitch(int n) { return (size_t)n * half_pitch(n) + 8; }

__device__ inline cplx cmul(cplx a, cplx b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }

// tw[m] = exp(-2 pi i m / n)
__global__ void k_fft_table(cplx* tw, int n) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double sn, cs;
    sincospi(-2.0 * (double)m / (double)n, &sn, &cs);
    tw[m] = {cs, sn};
}

// The stages between the thread's inputs a (elements j + r n/4 of its line) and
// its last butterfly's outputs, which stay in a: element base + r n/4 of the
// line.  S(e) is the LDS slot of element e of the thread's line; act: the
// thread has a line (every thread takes the barriers).
template <class SLOT>
__device__ inline int fft_stages(cplx (&a)[4], int n, int logn, int j, bool act, cplx* lds,
                                 const cplx* W, SLOT&& S) {
    const int q = n >> 2;
    int Ns = 1;
    auto exchange = [&](const int (&to)[4]) {
        if (act)
#pragma unroll
            for (int r = 0; r < 4; ++r) lds[S(to[r])] = a[r];
        __syncthreads();
        if (act)
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = lds[S(j + r * q)];
        __syncthreads();
    };
    if (logn & 1) {
        const cplx s0 = {a[0].x + a[2].x, a[0].y + a[2].y}, d0 = {a[0].x - a[2].x, a[0].y - a[2].y};
        const cplx s1 = {a[1].x + a[3].x, a[1].y + a[3].y}, d1 = {a[1].x - a[3].x, a[1].y - a[3].y};
        a[0] = s0;
        a[1] = d0;
        a[2] = s1;
        a[3] = d1;
        exchange({2 * j, 2 * j + 1, 2 * (j + q), 2 * (j + q) + 1});
        Ns = 2;
    }
    for (;;) {
        const int k = j & (Ns - 1);
        if (Ns > 1) {
            const int st = k * (q / Ns);   // exp(-2 pi i k r / (4 Ns)) = W[r k n / (4 Ns)]
#pragma unroll
            for (int r = 1; r < 4; ++r) a[r] = cmul(a[r], W[r * st]);
        }
        const cplx b0 = {a[0].x + a[2].x, a[0].y + a[2].y}, b1 = {a[0].x - a[2].x, a[0].y - a[2].y};
        const cplx b2 = {a[1].x + a[3].x, a[1].y + a[3].y};
        const cplx b3 = {a[1].y - a[3].y, a[3].x - a[1].x};   // -i (a1 - a3)
        a[0] = {b0.x + b2.x, b0.y + b2.y};
        a[1] = {b1.x + b3.x, b1.y + b3.y};
        a[2] = {b0.x - b2.x, b0.y - b2.y};
        a[3] = {b1.x - b3.x, b1.y - b3.y};
        const int base = 4 * (j - k) + k;
        if (4 * Ns == n) return base;
        exchange({base, base + Ns, base + 2 * Ns, base + 3 * Ns});
        Ns *= 4;
    }
}

// x pass: row pairs 2 p, 2 p + 1 of component blockIdx.y as one complex line;
// with Z the line's transform the rows' are (Z(k) + conj Z(-k)) / 2 and
// (Z(k) - conj Z(-k)) / (2 i).
__global__ void __launch_bounds__(kFftItems) k_fft_x(const double* __restrict__ u, cplx* __restrict__ f,
                                                     const cplx* __restrict__ tw, int n, int logn, int L) {
    extern __shared__ cplx lds_fft[];
    cplx* const W = lds_fft + (size_t)L * n;
    const int tid = threadIdx.x, q = n >> 2, H = n / 2 + 1, Hp = half_pitch(n);
    const size_t nn = (size_t)n * n, N = nn * n;
    for (int m = tid; m < n; m += blockDim.x) W[m] = tw[m];
    __syncthreads();
    const int l = tid / q, j = tid & (q - 1);
    const bool act = l < L;
    const double* r0 = u + blockIdx.y * N + (size_t)(blockIdx.x * L + (act ? l : 0)) * 2 * n;
    cplx a[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = {r0[j + r * q], r0[n + j + r * q]};
    auto S = [&](int e) { return l * n + e; };
    const int base = fft_stages(a, n, logn, j, act, lds_fft, W, S);
    if (act)
#pragma unroll
        for (int r = 0; r < 4; ++r) lds_fft[S(base + r * q)] = a[r];
    __syncthreads();
    const int row0 = blockIdx.x * L * 2;   // first row within the component
    for (int t = tid; t < L * 2 * H; t += blockDim.x) {
        const int row = t / H, k = t - row * H;
        const cplx* Z = lds_fft + (row >> 1) * n;
        const cplx zp = Z[k], zm = Z[(n - k) & (n - 1)];
        const int z = (row0 + row) / n, y = (row0 + row) - z * n;   // n a power of two
        f[(blockIdx.y * n + z) * plane_pitch(n) + (size_t)y * Hp + k] = row & 1 ? cplx{0.5 * (zp.y + zm.y), 0.5 * (zm.x - zp.x)}
                         : cplx{0.5 * (zp.x + zm.x), 0.5 * (zp.y - zm.y)};
    }
}

// y pass in place: L lines at consecutive kx (the last tile of a row may hold
// fewer) of one plane of one component.
__global__ void __launch_bounds__(kFftItems) k_fft_y(cplx* __restrict__ f, const cplx* __restrict__ tw,
                                                     int n, int logn, int L) {
    extern __shared__ cplx lds_fft[];
    cplx* const W = lds_fft + (size_t)L * n;
    const int tid = threadIdx.x, q = n >> 2, H = n / 2 + 1, Hp = half_pitch(n);
    for (int m = tid; m < n; m += blockDim.x) W[m] = tw[m];
    __syncthreads();
    const int l = tid % L, j = tid / L, kx = blockIdx.x * L + l;
    const bool act = j < q && kx < H;
    cplx* line = f + blockIdx.y * plane_pitch(n) + (act ? kx : 0);   // blockIdx.y: plane of a component
    cplx a[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = line[(size_t)(act ? j + r * q : 0) * Hp];
    const int base = fft_stages(a, n, logn, j, act, lds_fft, W, [&](int e) { return e * L + l; });
    if (act)
#pragma unroll
        for (int r = 0; r < 4; ++r) line[(size_t)(base + r * q) * Hp] = a[r];
}

// floor(sqrt(v)) for 0 <= v <= 887 888 (the last shell's end at n = 1024): the
// hardware root is within 1 ulp (6e-5 below 1024), and the roots of r^2 - 1 and r^2 lie
// 1 / (2 r) >= 5.6e-4 apart.
__device__ inline int isqrt(int v) { return (int)(__builtin_amdgcn_sqrtf((float)v) + 1.5e-4f); }

// z pass and binning: tiles of L lines at consecutive kx and one ky, dealt to the
// blocks in turn.  The lines' energies e = |f|^2 / (2 n^6), twice for the kx whose
// conjugate half is not stored, go to LDS, line by line; then the threads sum the
// shells: on a line, shell s holds the |kz| with s^2 - s + 1 <= k^2 <= s^2 + s, a
// run of them.  G = threads / shells groups share the lines (one thread per
// shell left half the block idle), their sums are added at the end; each runs
// over tiles, lines and |kz| in a fixed order.  part[block][0 / 1][s]: E(s), and
// the shell's sum of |k|^2 e.
__global__ void __launch_bounds__(kFftItems) k_fft_z_bins(const cplx* __restrict__ f,
                                                          const cplx* __restrict__ tw, int n, int logn,
                                                          int L, int bins, double inv_n6,
                                                          double* __restrict__ part) {
    extern __shared__ cplx lds_fft[];
    cplx* const W = lds_fft + (size_t)L * n;
    double* const en = reinterpret_cast<double*>(lds_fft);
    const int tid = threadIdx.x, nthr = blockDim.x, q = n >> 2, H = n / 2 + 1, Hp = half_pitch(n);
    for (int m = tid; m < n; m += nthr) W[m] = tw[m];
    const int l = tid % L, j = tid / L;
    const int tx = (H + L - 1) / L, tiles = 3 * n * tx;
    const int G = nthr / bins > 1 ? nthr / bins : 1;
    const int grp = G > 1 ? tid / bins : 0, s0 = G > 1 ? tid - grp * bins : tid;
    double E[kMaxBins2] = {}, D[kMaxBins2] = {};
    // a tile's inputs, loaded while the last tile's shells are summed
    const size_t pp = plane_pitch(n);
    cplx a[4];
    auto load = [&](int t) {
        const int kx = (t % tx) * L + l, ky = (t / tx) % n, c = t / (tx * n);
        const bool act = j < q && kx < H;
        const cplx* line = f + (size_t)c * n * pp + (size_t)ky * Hp + (act ? kx : 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = line[(size_t)(act ? j + r * q : 0) * pp];
    };
    if ((int)blockIdx.x < tiles) load(blockIdx.x);
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int x0 = (t % tx) * L, ky = (t / tx) % n, kx = x0 + l;
        const bool act = j < q && kx < H;
        __syncthreads();   // the last tile's energies are summed (and W is there)
        const int base = fft_stages(a, n, logn, j, act, lds_fft, W, [&](int e) { return e * L + l; });
        const double w = (kx == 0 || kx == n / 2 ? 0.5 : 1.0) * inv_n6;
        if (act)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                en[l * (n + 1) + base + r * q] = w * (a[r].x * a[r].x + a[r].y * a[r].y);
        if (t + (int)gridDim.x < tiles) load(t + gridDim.x);
        lds_barrier();
        const int kys = ky < n / 2 ? ky : n - ky, lines = H - x0 < L ? H - x0 : L;
#pragma unroll
        for (int i = 0; i < kMaxBins2; ++i) {
            const int s = s0 + i * nthr;
            if (s >= bins || grp >= G) break;
            const int top = s * s + s, bot = s == 0 ? 0 : s * s - s + 1;
            for (int y = grp; y < lines; y += G) {
                const int kxy = (x0 + y) * (x0 + y) + kys * kys;
                if (top < kxy) break;   // kxy grows with y
                const int hi = isqrt(top - kxy), lo = bot <= kxy ? 0 : isqrt(bot - kxy - 1) + 1;
                const int end = hi < n / 2 ? hi : n / 2;
                const double* e0 = en + y * (n + 1);
                for (int m = lo; m <= end; ++m) {
                    // kz = m and -m, one and the same at 0 and n / 2
                    const double e = (m == 0 || m == n / 2 ? 0.5 : 1.0) * (e0[m] + e0[(n - m) & (n - 1)]);
                    E[i] += e;
                    D[i] += (double)(kxy + m * m) * e;
                }
            }
        }
    }
    // the groups' sums, in group order
    __syncthreads();
    if (G > 1 && grp < G) {
        en[(grp * bins + s0) * 2] = E[0];
        en[(grp * bins + s0) * 2 + 1] = D[0];
    }
    __syncthreads();
    if (grp != 0) return;
    for (int g = 1; g < G; ++g) {
        E[0] += en[(g * bins + s0) * 2];
        D[0] += en[(g * bins + s0) * 2 + 1];
    }
    double* out = part + (size_t)blockIdx.x * 2 * bins;
#pragma unroll
    for (int i = 0; i < kMaxBins2; ++i) {
        const int s = s0 + i * nthr;
        if (s >= bins) break;
        out[s] = E[i];
        out[bins + s] = D[i];
    }
}

// Totals over the blocks, in 16 slices added in order.
__global__ void __launch_bounds__(1024) k_spectrum_total(const double* __restrict__ part, int nb,
                                                         int count, double* __restrict__ out) {
    __shared__ double lds[16][64];
    const int ex = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + ex;
    const int per = (nb + 15) / 16, b0 = sl * per, b1 = b0 + per < nb ? b0 + per : nb;
    double s = 0.0;
    if (e < count)
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += part[(size_t)b * count + e];
    lds[sl][ex] = s;
    __syncthreads();
    if (sl != 0 || e >= count) return;
    s = lds[0][ex];
#pragma unroll
    for (int r = 1; r < 16; ++r) s += lds[r][ex];
    out[e] = s;
}

// ---- stencil diagnostics ----
// z-marches over 64 x 8 columns of cells, any n: a block stages each plane of its
// column with a halo of H cells in LDS (positions wrapped, so that a column past
// the grid's edge holds the periodic images and its threads only skip their
// outputs), the next plane's loads in flight meanwhile; what the z direction
// needs waits in register queues.  Before, every cell gathered its stencils
// through the caches: 39 loads for Q, 81 for the filter, whose nine filtered
// fields then went through memory.  256^3: Q 0.17 ms instead of 0.52 (3.1 TB/s of
// its four words), the filtered statistics 0.48 instead of 1.55.  Bound: staging,
// barrier and arithmetic in turn, with two to three blocks per CU to overlap them.
// A small grid is the launch and one march: us per call with 4 planes, so: Q 54 and
// 50, statistics 64 and 56 from 8^3 to 32^3 (48^3 53 and 52, 65 and 62).
constexpr int kMX = 64, kMY = 8, kMThreads = kMX * kMY, kMBlocks = 1024, kMCus = 256;
constexpr int kSY = 4;   // rows of the kernels that keep a ring of planes
struct March {
    dim3 grid;
    int cz;
    unsigned blocks;
};
March make_march(int n, int rows = kMY) {
    March m;
    const int gx = (n + kMX - 1) / kMX, gy = (n + rows - 1) / rows;
    int nz = kMBlocks * (kMY / rows) / (gx * gy);
    nz = nz < 1 ? 1 : nz;
    // shorter marches than 4 planes only while the blocks are no more than the CUs
    int least = 1;
    while (least < 4 && gx * gy * ((n + least - 1) / least) > kMCus) ++least;
    m.cz = std::max((n + nz - 1) / nz, std::min(n, least));
    nz = (n + m.cz - 1) / m.cz;
    m.grid = dim3(gx, gy, nz);
    m.blocks = (unsigned)gx * gy * nz;
    return m;
}

// One plane of NF fields with a halo of H cells around 64 x RY: staged values in
// flight and where they go.
template <int NF, int H, int RY = kMY>
struct Stage {
    static constexpr int kW = kMX + 2 * H, kR = RY + 2 * H, kCells = kW * kR, kThreads = kMX * RY;
    static constexpr int kPer = (kCells + kThreads - 1) / kThreads;
    size_t src[kPer];
    double v[NF][kPer];
    __device__ void init(int n, int i0, int j0, int tid) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int c = tid + q * kThreads, y = c / kW, x = c - y * kW;
            const int gx = (i0 - H + x + n) % n, gy = (j0 - H + y + n) % n;   // n >= 8 > H
            src[q] = c < kCells ? (size_t)gx + (size_t)n * gy : 0;
        }
    }
    __device__ void load(const double* f, size_t N, size_t plane) {
#pragma unroll
        for (int m = 0; m < NF; ++m)
#pragma unroll
            for (int q = 0; q < kPer; ++q) v[m][q] = f[m * N + plane + src[q]];
    }
    __device__ void store(double* lds, int tid) const {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int c = tid + q * kThreads;
            if (c < kCells)
#pragma unroll
                for (int m = 0; m < NF; ++m) lds[m * kCells + c] = v[m][q];
        }
    }
};

// Gauss-I4 derivative (I4(q)_{P+1/2} - I4(q)_{P-1/2}) / h from the cells -2..2.
__device__ inline double dgauss5(double a, double b, double c, double d, double e, double inv_h) {
    return ((9.0 * (c + d) - (b + e)) * 0.0625 - (9.0 * (b + c) - (a + d)) * 0.0625) * inv_h;
}

// The gradient of three fields on the plane two behind the last one staged: its
// x and y neighbours from the plane's ring slot p (the three fields C apart, rows
// W apart), its z neighbours from the queue c.
__device__ inline void march_grad(const double* p, int W, int C, const double (&c)[3][5], double inv_h,
                                  double (&G)[3][3]) {
#pragma unroll
    for (int m = 0; m < 3; ++m, p += C) {
        G[m][0] = dgauss5(p[-2], p[-1], c[m][2], p[1], p[2], inv_h);
        G[m][1] = dgauss5(p[-2 * W], p[-W], c[m][2], p[W], p[2 * W], inv_h);
        G[m][2] = dgauss5(c[m][0], c[m][1], c[m][2], c[m][3], c[m][4], inv_h);
    }
}

// Q = -(1/2) sum_ij (d_j u_i)(d_i u_j) per cell with the Gauss-I4 cell
// derivative d_j q = (I4(q)_{P+1/2 e_j} - I4(q)_{P-1/2 e_j}) / h; partial sums
// of Q and of (d_i u_i)^2 (the discrete identity sum Q = -(1/2) sum (div u)^2
// holds for these antisymmetric, commuting difference operators).
__global__ void __launch_bounds__(kMX * kSY) k_qcrit(int n, int cz, double inv_h,
                                                     const double* __restrict__ u,
                                                     double* __restrict__ q, double* part) {
    typedef Stage<3, 2, kSY> St;
    constexpr int W = St::kW, C = St::kCells;
    __shared__ double lds[3 * 3 * C];   // a ring of three planes
    const BlockXYZ bp = block_xyz();
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + kMX * ty;
    const int i0 = bp.x * kMX, j0 = bp.y * kSY, k0 = bp.z * cz, k1 = k0 + cz < n ? k0 + cz : n;
    const size_t nn = (size_t)n * n, N = nn * n;
    const bool act = i0 + tx < n && j0 + ty < n;
    const size_t col = act ? (size_t)(i0 + tx) + (size_t)n * (j0 + ty) : 0;
    const int at = (ty + 2) * W + tx + 2;
    St st;
    st.init(n, i0, j0, tid);
    double c[3][5] = {}, v[2] = {0.0, 0.0};
    auto plane = [&](int k) { return nn * (size_t)((k + n) % n); };
    st.load(u, N, plane(k0 - 2));
    int slot = 0;
    for (int k = k0 - 2; k < k1 + 2; ++k, slot = slot == 2 ? 0 : slot + 1) {
        double* const pk = lds + slot * 3 * C;
        st.store(pk, tid);
        st.load(u, N, plane(k + 1 < k1 + 2 ? k + 1 : k));
        lds_barrier();
#pragma unroll
        for (int m = 0; m < 3; ++m) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c[m][t] = c[m][t + 1];
            c[m][4] = pk[m * C + at];
        }
        if (k >= k0 + 2 && act) {
            double G[3][3];   // of plane k - 2, whose ring slot is the next one
            march_grad(lds + (slot == 2 ? 0 : slot + 1) * 3 * C + at, W, C, c, inv_h, G);
            double Q = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) Q -= 0.5 * G[a][b] * G[b][a];
            const double div = G[0][0] + G[1][1] + G[2][2];
            stream_st(q + (col + nn * (size_t)(k - 2)), Q);
            v[0] += Q;
            v[1] += div * div;
        }
        lds_barrier();
    }
    block_partials<2, 0u>(v, part);
}

__global__ void __launch_bounds__(kBlock) k_qcrit_total(const double* part, unsigned nb,
                                                        double* out) {
    double t[2];
    reduce_partials<2, 0u>(part, nb, t);
    if (flat_tid() == 0) {
        out[0] = t[0];
        out[1] = t[1];
    }
}

// The separable top-hat of width 2h (weights 1/4, 1/2, 1/4 along each axis) over
// the staged plane's x and y, around the cell at `at`.
template <class F>
__device__ inline double tophat_xy(int W, F&& f) {
    double r[3];
#pragma unroll
    for (int y = -1; y <= 1; ++y)
        r[y + 1] = 0.25 * (f(y * W - 1) + f(y * W + 1)) + 0.5 * f(y * W);
    return 0.25 * (r[0] + r[2]) + 0.5 * r[1];
}

// Filtered (a-priori sub-grid) statistics, first pass: u_bar.
__global__ void __launch_bounds__(kMThreads) k_sgs_filter(int n, int cz, const double* __restrict__ u,
                                                          double* __restrict__ ub) {
    typedef Stage<3, 1> St;
    __shared__ double lds[3 * St::kCells];
    const BlockXYZ bp = block_xyz();
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + kMX * ty;
    const int i0 = bp.x * kMX, j0 = bp.y * kMY, k0 = bp.z * cz, k1 = k0 + cz < n ? k0 + cz : n;
    const size_t nn = (size_t)n * n, N = nn * n;
    const bool act = i0 + tx < n && j0 + ty < n;
    const size_t col = act ? (size_t)(i0 + tx) + (size_t)n * (j0 + ty) : 0;
    const int at = (ty + 1) * St::kW + tx + 1;
    St st;
    st.init(n, i0, j0, tid);
    double f[3][3];
    auto plane = [&](int k) { return nn * (size_t)((k + n) % n); };
    st.load(u, N, plane(k0 - 1));
    for (int k = k0 - 1; k < k1 + 1; ++k) {
        st.store(lds, tid);
        st.load(u, N, plane(k + 1 < k1 + 1 ? k + 1 : k));
        lds_barrier();
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const double* p = lds + m * St::kCells + at;
            f[m][0] = f[m][1];
            f[m][1] = f[m][2];
            f[m][2] = tophat_xy(St::kW, [&](int o) { return p[o]; });
        }
        lds_barrier();
        if (k < k0 + 1 || !act) continue;
#pragma unroll
        for (int m = 0; m < 3; ++m)
            ub[m * N + col + nn * (size_t)(k - 1)] = 0.25 * (f[m][0] + f[m][2]) + 0.5 * f[m][1];
    }
}

// Second pass, per cell: bar(u_i u_j) filtered on the fly,
// tau_ij = bar(u_i u_j) - u_bar_i u_bar_j, k_sgs = tau_ii / 2,
// S_bar_ij = (d_j u_bar_i + d_i u_bar_j) / 2 (Gauss-I4), Pi = -tau_ij S_bar_ij;
// partial sums of |u_bar|^2 / 2, k_sgs, Pi and of the cells with Pi < 0.
// Columns of 64 x 4 cells, a ring of three u_bar planes in LDS and running sums of
// the products' z filter keep the registers at 164: with the derivatives of
// three planes and the products of three in registers (250 of them) one block of
// 64 x 8 had a CU to itself, 395 us at 256^3 against 309.
__global__ void __launch_bounds__(kMX * kSY) k_sgs_stats(int n, int cz, double inv_h,
                                                         const double* __restrict__ u,
                                                         const double* __restrict__ ub, double* part) {
    typedef Stage<3, 1, kSY> Su;
    typedef Stage<3, 2, kSY> Sb;
    constexpr int W = Sb::kW, C = Sb::kCells;
    __shared__ double lds[3 * Su::kCells + 3 * 3 * C];
    double* const ldsb = lds + 3 * Su::kCells;
    const BlockXYZ bp = block_xyz();
    const int tx = threadIdx.x, ty = threadIdx.y, tid = tx + kMX * ty;
    const int i0 = bp.x * kMX, j0 = bp.y * kSY, k0 = bp.z * cz, k1 = k0 + cz < n ? k0 + cz : n;
    const size_t nn = (size_t)n * n, N = nn * n;
    const bool act = i0 + tx < n && j0 + ty < n;
    const int au = (ty + 1) * Su::kW + tx + 1, ab = (ty + 2) * W + tx + 2;
    Su su;
    Sb sb;
    su.init(n, i0, j0, tid);
    sb.init(n, i0, j0, tid);
    // bar(u u) in the order xx, xy, xz, yy, yz, zz: with P(k) the plane's x-y
    // filtered product, f[0] = P(k - 1) / 4 + P(k) / 2 and f[1] = P(k) / 4 of the
    // last plane k staged
    constexpr int kA[6] = {0, 0, 0, 1, 1, 2}, kB[6] = {0, 1, 2, 1, 2, 2};
    double f[6][2] = {}, c[3][5] = {};
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    auto plane = [&](int k) { return nn * (size_t)((k + n) % n); };
    // step k stages u_bar's plane k and u's plane k - 1; the output plane is k - 2
    su.load(u, N, plane(k0 - 3));
    sb.load(ub, N, plane(k0 - 2));
    int slot = 0;
    for (int k = k0 - 2; k < k1 + 2; ++k, slot = slot == 2 ? 0 : slot + 1) {
        double* const pb = ldsb + slot * 3 * C;
        su.store(lds, tid);
        sb.store(pb, tid);
        const int kn = k + 1 < k1 + 2 ? k + 1 : k;
        su.load(u, N, plane(kn - 1));
        sb.load(ub, N, plane(kn));
        lds_barrier();
        double bar[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) bar[e] = f[e][0];
#pragma unroll
        for (int y = -1; y <= 1; ++y) {
            double a[3][3];
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int x = 0; x < 3; ++x) a[m][x] = lds[m * Su::kCells + au + y * Su::kW + x - 1];
            const double wy = y == 0 ? 0.5 : 0.25;
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const double r = wy * (0.25 * (a[kA[e]][0] * a[kB[e]][0] + a[kA[e]][2] * a[kB[e]][2]) +
                                       0.5 * (a[kA[e]][1] * a[kB[e]][1]));
                if (y == -1) f[e][0] = r;   // the plane's P, in turn
                else f[e][0] += r;
            }
        }
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            const double P = f[e][0];
            bar[e] += 0.25 * P;
            f[e][0] = f[e][1] + 0.5 * P;
            f[e][1] = 0.25 * P;
        }
#pragma unroll
        for (int m = 0; m < 3; ++m) {
#pragma unroll
            for (int t = 0; t < 4; ++t) c[m][t] = c[m][t + 1];
            c[m][4] = pb[m * C + ab];
        }
        if (k >= k0 + 2 && act) {
            // the output plane's x and y derivatives: its ring slot is the next one
            double G[3][3];
            march_grad(ldsb + (slot == 2 ? 0 : slot + 1) * 3 * C + ab, W, C, c, inv_h, G);
            double ks = 0.0, pi = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const int a = kA[e], b = kB[e];
                const double tau = bar[e] - c[a][2] * c[b][2];
                if (a == b) ks += 0.5 * tau;
                pi -= (a == b ? 1.0 : 2.0) * tau * 0.5 * (G[a][b] + G[b][a]);
            }
            v[0] += 0.5 * (c[0][2] * c[0][2] + c[1][2] * c[1][2] + c[2][2] * c[2][2]);
            v[1] += ks;
            v[2] += pi;
            v[3] += pi < 0.0 ? 1.0 : 0.0;
        }
        lds_barrier();
    }
    block_partials<4, 0u>(v, part);
}

__global__ void __launch_bounds__(kBlock) k_sgs_total(const double* part, unsigned nb,
                                                      double* out) {
    double t[4];
    reduce_partials<4, 0u>(part, nb, t);
    if (flat_tid() == 0)
        for (int c = 0; c < 4; ++c) out[c] = t[c];
}

constexpr unsigned kMaxMarch = 4096;   // blocks of a march: n = 1024 has 16 x 256 columns of 4 rows

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Workspace: the spectrum's half-complex fields or u_bar (never both at once),
// twiddles, binning partials and totals, the stencil kernels' partials.
struct DiagLayout {
    size_t field, tw, part, total_out, qpart, bytes;
};
DiagLayout diag_layout(int n) {
    DiagLayout d{};
    const size_t nn = (size_t)n * n;
    const int bins = shell_of(3LL * (n / 2) * (n / 2)) + 1;
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off = align256(off + b);
        return o;
    };
    d.field = take(std::max(sizeof(cplx) * 3 * n * plane_pitch(n), sizeof(double) * 3 * nn * n));
    d.tw = take(sizeof(cplx) * n);
    d.part = take(sizeof(double) * 2 * (size_t)kSpecBlocks * bins);
    d.total_out = take(sizeof(double) * 2 * bins);
    d.qpart = take(sizeof(double) * (4 * kMaxMarch + 16));
    d.bytes = off;
    return d;
}

// Streaming probe: out_w[i] = (w + 1) * (in_0[i] + ... + in_{R-1}[i]) over
// 16-byte vectors, a flat grid walking the arrays with a grid stride,
// non-temporal loads and stores (as the step's kernels stream their fields).
constexpr int kStreamThreads = 256, kStreamBlocks = 16384;
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int kStreamMaxReads = 12, kStreamMaxWrites = 8;
struct StreamPtrs {
    const f4v* in[kStreamMaxReads];
    f4v* out[kStreamMaxWrites];
};

template <int R, int W>
__global__ void __launch_bounds__(kStreamThreads) k_stream(StreamPtrs p, size_t n4) {
    const size_t stride = (size_t)gridDim.x * kStreamThreads;
    for (size_t i = (size_t)blockIdx.x * kStreamThreads + threadIdx.x; i < n4; i += stride) {
        f4v a = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < R; ++r) a += __builtin_nontemporal_load(p.in[r] + i);
#pragma unroll
        for (int w = 0; w < W; ++w) __builtin_nontemporal_store(a * (float)(w + 1), p.out[w] + i);
    }
}

template <int R, int W>
void launch_stream_rw(dim3 g, hipStream_t s, const StreamPtrs& p, size_t n4) {
    hipLaunchKernelGGL((k_stream<R, W>), g, dim3(kStreamThreads), 0, s, p, n4);
}

// launchers of k_stream<R, W>, R = 1..kStreamMaxReads, W = 1..kStreamMaxWrites
using StreamLaunch = void (*)(dim3, hipStream_t, const StreamPtrs&, size_t);
template <int R, int... Ws>
constexpr std::array<StreamLaunch, sizeof...(Ws)> stream_row(std::integer_sequence<int, Ws...>) {
    return {{&launch_stream_rw<R, Ws + 1>...}};
}
template <int... Rs>
constexpr std::array<std::array<StreamLaunch, kStreamMaxWrites>, sizeof...(Rs)> stream_table(
    std::integer_sequence<int, Rs...>) {
    return {{stream_row<Rs + 1>(std::make_integer_sequence<int, kStreamMaxWrites>{})...}};
}
constexpr auto kStreamLaunch = stream_table(std::make_integer_sequence<int, kStreamMaxReads>{});

}  // namespace
}  // namespace pisoc

using namespace pisoc;

extern "C" {

int32_t pisoc_diag_spectrum_bins(int32_t n) {
    if (!pow2(n)) return 0;
    return shell_of(3LL * (n / 2) * (n / 2)) + 1;
}

size_t pisoc_diag_workspace_bytes(int32_t n) {
    if (n < PISOC_MIN_N || n > PISOC_MAX_N) return 0;
    return diag_layout(n).bytes;
}

pisoc_status pisoc_diag_spectrum(int32_t n, const double* d_u, double* h_E, int32_t nbins,
                                 double* h_taylor, double* h_dsum, void* d_ws, size_t ws_bytes,
                                 void* hip_stream) {
    if (!pow2(n) || !d_u || !h_E || nbins != pisoc_diag_spectrum_bins(n)) return PISOC_ERR_INVALID;
    const DiagLayout Ly = diag_layout(n);
    if (!d_ws || ws_bytes < Ly.bytes || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    char* ws = reinterpret_cast<char*>(d_ws);
    cplx* f = reinterpret_cast<cplx*>(ws + Ly.field);
    cplx* tw = reinterpret_cast<cplx*>(ws + Ly.tw);
    double* part = reinterpret_cast<double*>(ws + Ly.part);
    double* tot = reinterpret_cast<double*>(ws + Ly.total_out);
    const size_t N = (size_t)n * n * n;
    const int logn = ilog2(n), q = n / 4, H = n / 2 + 1;
    const double inv_n6 = 1.0 / ((double)N * (double)N);
    // lines per block: of the x pass (row pairs, a power of two), of the others
    // (consecutive kx, the H of them in tiles of nearly equal width)
    const int Lx = std::min(kFftItems / q, n * n / 2);
    const int Lmax = kFftItems / q;
    int tx = (H + Lmax - 1) / Lmax, L = (H + tx - 1) / tx;
    if (Lmax >= 8) {   // whole 128-byte lines
        L = (L + 7) / 8 * 8;
        tx = (H + L - 1) / L;
    }
    const dim3 bx((Lx * q + 63) / 64 * 64), b((L * q + 63) / 64 * 64);
    const size_t ldsx = sizeof(cplx) * ((size_t)Lx * n + n), lds = sizeof(cplx) * ((size_t)L * n + n);
    const int nb = std::min(kSpecBlocks, 3 * n * tx);
    hipLaunchKernelGGL(k_fft_table, dim3((n + 255) / 256), dim3(256), 0, s, tw, n);
    hipLaunchKernelGGL(k_fft_x, dim3(n * n / 2 / Lx, 3), bx, ldsx, s, d_u, f, tw, n, logn, Lx);
    hipLaunchKernelGGL(k_fft_y, dim3(tx, 3 * n), b, lds, s, f, tw, n, logn, L);
    hipLaunchKernelGGL(k_fft_z_bins, dim3(nb), b, lds, s, f, tw, n, logn, L, nbins, inv_n6, part);
    hipLaunchKernelGGL(k_spectrum_total, dim3((2 * nbins + 63) / 64), dim3(1024), 0, s, part, nb,
                       2 * nbins, tot);
    if (hipGetLastError() != hipSuccess) return PISOC_ERR_HIP;
    // the totals come back through pageable memory after the stream has drained
    if (hipStreamSynchronize(s) != hipSuccess) return PISOC_ERR_HIP;
    double* host = new (std::nothrow) double[2 * nbins];
    if (!host) return PISOC_ERR_INVALID;
    const bool ok = hipMemcpy(host, tot, sizeof(double) * 2 * nbins, hipMemcpyDeviceToHost) ==
                    hipSuccess;
    if (ok) {
        double e = 0.0, D = 0.0;
        for (int b2 = 0; b2 < nbins; ++b2) {
            h_E[b2] = host[b2];
            e += host[b2];
            D += host[nbins + b2];
        }
        if (h_taylor) *h_taylor = D > 0.0 ? std::sqrt(5.0 * e / D) : 0.0;
        if (h_dsum) *h_dsum = D;
    }
    delete[] host;
    return ok ? PISOC_OK : PISOC_ERR_HIP;
}

pisoc_status pisoc_diag_qcrit(int32_t n, const double* d_u, double* d_q, double* h_means,
                              void* d_ws, size_t ws_bytes, void* hip_stream) {
    if (n < PISOC_MIN_N || n > PISOC_MAX_N || !d_u || !d_q) return PISOC_ERR_INVALID;
    const DiagLayout Ly = diag_layout(n);
    if (!d_ws || ws_bytes < Ly.bytes || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    const size_t N = (size_t)n * n * n;
    double* qpart = reinterpret_cast<double*>(reinterpret_cast<char*>(d_ws) + Ly.qpart);
    double* out = qpart + 2 * kMaxMarch;
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    const double inv_h = (double)n / 6.283185307179586476925286766559;
    const March m = make_march(n, kSY);
    hipLaunchKernelGGL(k_qcrit, m.grid, dim3(kMX, kSY), 0, s, n, m.cz, inv_h, d_u, d_q, qpart);
    if (!h_means) return hipGetLastError() == hipSuccess ? PISOC_OK : PISOC_ERR_HIP;
    hipLaunchKernelGGL(k_qcrit_total, dim3(1), dim3(kBlock), 0, s, qpart, m.blocks, out);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return PISOC_ERR_HIP;
    double t[2];
    if (hipMemcpy(t, out, sizeof(t), hipMemcpyDeviceToHost) != hipSuccess) return PISOC_ERR_HIP;
    h_means[0] = t[0] / (double)N;
    h_means[1] = t[1] / (double)N;
    return PISOC_OK;
}

pisoc_status pisoc_diag_sgs(int32_t n, const double* d_u, double* h_out, void* d_ws,
                            size_t ws_bytes, void* hip_stream) {
    if (n < PISOC_MIN_N || n > PISOC_MAX_N || !d_u || !h_out) return PISOC_ERR_INVALID;
    const DiagLayout Ly = diag_layout(n);
    if (!d_ws || ws_bytes < Ly.bytes || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    const size_t N = (size_t)n * n * n;
    char* ws = reinterpret_cast<char*>(d_ws);
    double* ub = reinterpret_cast<double*>(ws + Ly.field);
    double* part = reinterpret_cast<double*>(ws + Ly.qpart);
    double* out = part + 4 * kMaxMarch;
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    const double inv_h = (double)n / 6.283185307179586476925286766559;
    const March m = make_march(n);
    hipLaunchKernelGGL(k_sgs_filter, m.grid, dim3(kMX, kMY), 0, s, n, m.cz, d_u, ub);
    const March ms = make_march(n, kSY);
    hipLaunchKernelGGL(k_sgs_stats, ms.grid, dim3(kMX, kSY), 0, s, n, ms.cz, inv_h, d_u, ub, part);
    hipLaunchKernelGGL(k_sgs_total, dim3(1), dim3(kBlock), 0, s, part, ms.blocks, out);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return PISOC_ERR_HIP;
    double t[4];
    if (hipMemcpy(t, out, sizeof(t), hipMemcpyDeviceToHost) != hipSuccess) return PISOC_ERR_HIP;
    for (int c = 0; c < 4; ++c) h_out[c] = t[c] / (double)N;
    return PISOC_OK;
}

pisoc_status pisoc_stream_probe(int32_t reads, int32_t writes, int64_t count,
                                const float* const* h_in, float* const* h_out, int32_t blocks,
                                void* hip_stream) {
    if (reads < 1 || reads > kStreamMaxReads || writes < 1 || writes > kStreamMaxWrites || count < 0 ||
        count % 4 != 0 ||
        blocks < 0)
        return PISOC_ERR_INVALID;
    if (count == 0) return PISOC_OK;
    if (!h_in || !h_out) return PISOC_ERR_INVALID;
    StreamPtrs p{};
    for (int r = 0; r < reads; ++r) {
        if (!h_in[r] || reinterpret_cast<uintptr_t>(h_in[r]) % 16 != 0) return PISOC_ERR_INVALID;
        p.in[r] = reinterpret_cast<const f4v*>(h_in[r]);
    }
    for (int w = 0; w < writes; ++w) {
        if (!h_out[w] || reinterpret_cast<uintptr_t>(h_out[w]) % 16 != 0) return PISOC_ERR_INVALID;
        p.out[w] = reinterpret_cast<f4v*>(h_out[w]);
    }
    const size_t n4 = (size_t)count / 4;
    const dim3 g((unsigned)(blocks > 0 ? blocks : kStreamBlocks));
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    kStreamLaunch[reads - 1][writes - 1](g, s, p, n4);
    return hipGetLastError() == hipSuccess ? PISOC_OK : PISOC_ERR_HIP;
}

}  // extern "C"
