// net.hip -- the learned pressure-guess network on gfx950: four periodic
// 3x3x3 convolutions (2 -> 16 -> 16 -> 16 -> 1, ReLU after the first three, no
// biases) evaluated with BF16 operands and FP32 accumulation on the matrix
// cores (v_mfma_f32_16x16x32_bf16 in the 16 -> 16 layers and the weight
// gradients, v_mfma_f32_16x16x16_bf16 in the first and last layer), plus the
// training kernels (data and weight gradients, MSE and residual losses, Adam)
// and the C ABI of the network.
//
// GEMM view of one layer: for 16 consecutive cells along x (one wavefront),
// D[co][cell] = sum over K of A[co][k] B[k][cell] with k = (tap, ci).  A lane
// loads consecutive channels of one neighbour cell, so activations are stored
// channel-last in BF16.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/pisoc.h"
#include "device.hpp"
#include "launch.hpp"
#include "net.hpp"

namespace pisoc {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ inline float bf2f(uint16_t b) {
    uint32_t u = (uint32_t)b << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

__device__ inline int wrapn(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// FP32 -> BF16, round to nearest even, with gfx950's conversion instruction
// (v_cvt_pk_bf16_f32): the same rounding as f2bf for finite values, without
// its branch for NaN.
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
__device__ inline uint32_t bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));
}
__device__ inline uint16_t bf16x1(float a) { return __builtin_bit_cast(uint16_t, (__bf16)a); }

// Every layer marches along z: a wavefront owns 16 cells along x times kRY
// rows along y and walks a chunk of output planes.
constexpr int kRY = 4;
constexpr int kTapBlocks = 7;   // K-blocks of 4 taps (k_conv4_taps)

// The 16 -> 16 layers run on gfx950's K = 32 product
// (v_mfma_f32_16x16x32_bf16, twice the work of the K = 16 form per issue).
// Within one input plane the (kRY + 2) x 3 (row, x shift) items r = 3 iy + q
// are taken two at a time: pair p holds item 2p in lane groups 0-1 and item
// 2p + 1 in groups 2-3, 8 channels (16 bytes) of one cell per lane.  Output row
// oy reads items 3 oy .. 3 oy + 8, the 5 pairs from floor(3 oy / 2) on, whose
// weight operand depends only on the parity c of oy, the pair's slot s in that
// run and dz: 30 operands, held in registers.  60 products per output plane of
// 16 x kRY cells (108 with K = 16), 10 % of their entries the zero halves at
// the ends of odd and even runs.
constexpr int kItems = 3 * (kRY + 2), kPairs = kItems / 2, kSlots = 5;
static_assert(kItems % 2 == 0, "items pair up within a plane");

__device__ inline v4f mfma_k32(v8s a, v8s b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// The 16 -> 16 layer as a z-march.  A wavefront owns 16 cells along x times
// kRY rows along y and walks a chunk of ZC output planes: input plane by input
// plane (ZC + 2 of them, each loaded once, 9 pair items of 16 bytes per
// lane), it issues the products of the three output planes the input plane
// reaches (dz = -1, 0, 1) into a ring of three planes of accumulators, and
// stores an output plane once its last input plane (dz = +1) is done.  The
// weight operands are loaded once per wavefront; each item of the next input
// plane is loaded into its register right after the item's last product, so
// a whole plane of products covers the load.  The plane loop is unrolled in
// full (ZC a template parameter), so that every ring slot and edge test is a
// constant and the loads stay in flight across planes (with run-time tests the
// compiler drained them at every branch: 1.65 against 1.12 ms for the
// network at 256^3).  Against one wavefront per 16 x 4 x 4 tile, which
// reread 6 input planes per 4 output planes and reloaded the weights per
// tile, the layer takes about 290 instead of 480 us at 256^3.
// MASKED (a data gradient): the output channel is zero where the activation
// mask it belongs to is not positive; else ReLU.
template <bool MASKED>
__device__ inline void store_plane_rows(const v4f (&acc)[kRY], uint16_t* __restrict__ out,
                                        const uint16_t* __restrict__ mask, int n, int x, int j0,
                                        int kz, int g) {
#pragma unroll
    for (int oy = 0; oy < kRY; ++oy) {
        const size_t cell = (size_t)x + (size_t)n * ((size_t)(j0 + oy) + (size_t)n * kz);
        v4s m = {0, 0, 0, 0};
        if (MASKED) m = *reinterpret_cast<const v4s*>(mask + cell * 16 + 4 * g);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = acc[oy][e];
            v[e] = (MASKED ? m[e] > 0 : a > 0.f) ? a : 0.f;   // as BF16 bits: > 0 is the sign and not zero
        }
        uint2 q;
        q.x = bf16x2(v[0], v[1]);
        q.y = bf16x2(v[2], v[3]);
        *reinterpret_cast<uint2*>(out + cell * 16 + 4 * g) = q;
    }
}

template <int ZC, bool MASKED>
__global__ void __launch_bounds__(256, 2) k_conv16_zm(int n, int batch,
                                                      const uint16_t* __restrict__ in,
                                                      const v8s* __restrict__ wpp,
                                                      const uint16_t* __restrict__ mask,
                                                      uint16_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int segs = n / 16, nyb = n / kRY, nzc = n / ZC;
    const long nwaves = (long)batch * nzc * nyb * segs;
    if (wave >= nwaves) return;  // whole wavefront; no block barrier below
    const int iseg = (int)(wave % segs);
    long rest = wave / segs;
    const int j0 = (int)(rest % nyb) * kRY;
    rest /= nyb;
    const int k0 = (int)(rest % nzc) * ZC;
    const int b = (int)(rest / nzc);
    const size_t N = (size_t)n * n * n, nn = (size_t)n * n;
    const int m = lane & 15, g = lane >> 4, h = g >> 1;
    v8s B[2][kSlots][3];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
#pragma unroll
            for (int dz = 0; dz < 3; ++dz) B[c][s][dz] = wpp[((c * kSlots + s) * 3 + dz) * 64 + lane];
    // this lane's element offset of each pair item within a plane
    int off[kPairs];
#pragma unroll
    for (int p = 0; p < kPairs; ++p) {
        const int r = 2 * p + h, iy = r / 3, q = r % 3;
        off[p] = (n * wrapn(j0 - 1 + iy, n) + wrapn(iseg * 16 + m + q - 1, n)) * 16 + 8 * (g & 1);
    }
    const uint16_t* inb = in + (size_t)b * N * 16;
    uint16_t* outb = out + (size_t)b * N * 16;
    const uint16_t* maskb = MASKED ? mask + (size_t)b * N * 16 : nullptr;
    auto plane_ptr = [&](int t) { return inb + nn * 16 * (size_t)wrapn(k0 - 1 + t, n); };
    v8s a[kPairs];
    {
        const uint16_t* pb = plane_ptr(0);
#pragma unroll
        for (int p = 0; p < kPairs; ++p) a[p] = *reinterpret_cast<const v8s*>(pb + off[p]);
    }
    v4f acc[3][kRY];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int oy = 0; oy < kRY; ++oy) acc[r][oy] = v4f{0.f, 0.f, 0.f, 0.f};
    // fully unrolled: every plane's output rows and ring slots are constants
#pragma unroll
    for (int t = 0; t < ZC + 2; ++t) {
        const bool more = t + 1 < ZC + 2;
        const uint16_t* pn = plane_ptr(more ? t + 1 : t);
#pragma unroll
        for (int p = 0; p < kPairs; ++p) {
#pragma unroll
            for (int dz = -1; dz <= 1; ++dz) {
                const int oz = t - 1 - dz;   // output plane, ring slot oz mod 3
                if (oz < 0 || oz >= ZC) continue;
#pragma unroll
                for (int oy = 0; oy < kRY; ++oy) {
                    const int s = p - (3 * oy) / 2;
                    if (s < 0 || s >= kSlots) continue;
                    acc[oz % 3][oy] = mfma_k32(B[oy & 1][s][dz + 1], a[p], acc[oz % 3][oy]);
                }
            }
            if (more) a[p] = *reinterpret_cast<const v8s*>(pn + off[p]);
        }
        // output plane t - 2 has had its last input plane (dz = +1)
        if (t >= 2) {
            store_plane_rows<MASKED>(acc[(t - 2) % 3], outb, maskb, n, iseg * 16 + m, j0, k0 + t - 2,
                                     g);
#pragma unroll
            for (int oy = 0; oy < kRY; ++oy) acc[(t - 2) % 3][oy] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    }
}

// The last layer's weights sit in LDS on a zero-padded (dz, dy) grid of [-4, 4]^2.
constexpr int kPadW = 9;   // dy, dz in [-4, 4]

// The last layer as a z-march: a wavefront owns 16 cells along x times kRY
// rows along y and walks ZC output planes.  The matrix columns (output rows of
// the product, weights as the A operand) are the kRY rows of the three output
// planes an input plane reaches, held in a ring: column 4 s + oy is row oy of
// the output plane in slot s (s = plane mod 3; columns 12-15 idle).  Input
// plane by input plane, each two of its (kRY + 2) rows times 3 x shifts are one
// product whose weight operand the lane takes from the padded (dz, dy) grid at
// the offsets of its column; a column whose plane lies outside the chunk reads
// the grid's zeros.  After an input plane the output plane of its dz = +1 taps
// is complete: the lanes of its slot store it and clear their accumulators.
// Each input row is loaded once per plane, into its register right after its
// product (a plane of products covers the load).  y = yscale * output, FP32.
// The row items go into K = 32 products two by two, as in the 16 -> 16 layer: one
// accumulator tuple holds all three planes, so a plane's products form one chain,
// which the pairs halve with the loads and the weights' reads from LDS (33.4 us a
// launch at 128^3 with single items, 25.1 so, the values the same bit for bit; the
// layer's traffic at a large copy's rate takes 16).
template <int ZC>
__global__ void __launch_bounds__(256) k_conv16_final_zm(int n, int batch,
                                                         const uint16_t* __restrict__ in,
                                                         const v4s* __restrict__ wfin,
                                                         float* __restrict__ yout, float yscale) {
    static_assert(kRY == 4, "three planes of kRY rows fit the 16 matrix columns");
    // wl[((dz + 4) kPadW + dy + 4) 3 + q][g]: channels 4g..4g+3 of tap (q - 1, dy, dz)
    __shared__ __align__(16) v4s wl[kPadW * kPadW * 3 * 4];
    for (int i = threadIdx.x; i < kPadW * kPadW * 3 * 4; i += blockDim.x) {
        const int g = i % 4, e = i / 4, q = e % 3, dy = (e / 3) % kPadW - 4, dz = e / (3 * kPadW) - 4;
        const bool reach = dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
        wl[i] = reach ? wfin[((dz + 1) * 9 + (dy + 1) * 3 + q) * 4 + g] : v4s{0, 0, 0, 0};
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int segs = n / 16, nyb = n / kRY, nzc = n / ZC;
    const long nwaves = (long)batch * nzc * nyb * segs;
    if (wave >= nwaves) return;  // whole wavefront; no block barrier below
    const int iseg = (int)(wave % segs);
    long rest = wave / segs;
    const int j0 = (int)(rest % nyb) * kRY;
    rest /= nyb;
    const int k0 = (int)(rest % nzc) * ZC;
    const int b = (int)(rest / nzc);
    const size_t N = (size_t)n * n * n, nn = (size_t)n * n;
    const int m = lane & 15, g = lane >> 4;
    const int col = lane & 15, oy = col % kRY, slot = col / kRY;   // this lane's A row (output column)
    // pair it: the items (input row iy, shift q) 2 it in the lanes' groups 0-1 and
    // 2 it + 1 in groups 2-3, 8 channels of a cell per lane
    const uint16_t* inb = in + (size_t)b * N * 16 + 8 * (g & 1);
    int off[kPairs];
#pragma unroll
    for (int it = 0; it < kPairs; ++it) {
        const int r = 2 * it + (g >> 1), iy = r / 3, q = r % 3;
        off[it] = (n * wrapn(j0 - 1 + iy, n) + wrapn(iseg * 16 + m + q - 1, n)) * 16;
    }
    auto plane_ptr = [&](int t) { return inb + nn * 16 * (size_t)wrapn(k0 - 1 + t, n); };
    v8s a[kPairs];
    {
        const uint16_t* pb = plane_ptr(0);
#pragma unroll
        for (int it = 0; it < kPairs; ++it) a[it] = *reinterpret_cast<const v8s*>(pb + off[it]);
    }
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < ZC + 2; ++t) {
        const bool more = t + 1 < ZC + 2;
        const uint16_t* pn = plane_ptr(more ? t + 1 : t);
        // the output plane of this lane's slot at input plane t: the one of
        // t - 2, t - 1, t congruent to the slot mod 3; its dz = t - 1 - oz, or
        // the grid's zeros (dz = 4) when it is outside the chunk or the slot idle
        const int oz = t - 2 + ((slot - (t - 2) % 3 + 3) % 3);
        const int dz = slot < 3 && oz >= 0 && oz < ZC ? t - 1 - oz : 4;
        const v8s* wb = reinterpret_cast<const v8s*>(wl + (((dz + 4) * kPadW + (3 - oy)) * 3) * 4) + g;
#pragma unroll
        for (int it = 0; it < kPairs; ++it) {
            acc = mfma_k32(wb[4 * it], a[it], acc);
            if (more) a[it] = *reinterpret_cast<const v8s*>(pn + off[it]);
        }
        // output plane t - 2 is complete: lane (g, m) holds rows 4 g + e of
        // cell m, so the lanes of its slot store rows 0..3 and clear them
        if (t >= 2) {
            const int sd = (t - 2) % 3;
            if (g == sd) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const size_t cell = (size_t)(iseg * 16 + m) +
                                        (size_t)n * ((size_t)(j0 + e) + (size_t)n * (k0 + t - 2));
                    yout[(size_t)b * N + cell] = acc[e] * yscale;
                    acc[e] = 0.f;
                }
            }
        }
    }
}

// The first layer (2 input channels, channel-last BF16 [cell][4] input) as a
// z-march like the 16 -> 16 layers.  One K = 16 block per input-row offset
// (dy, dz): lane group g holds the 4 channels of the cell shifted by
// dx = g - 1 (group 3 meets zero weights), so an input row is one 8-byte load
// per lane and the 9 weight operands stay in registers.  A wavefront owns 16
// cells along x times kRY rows along y and walks ZC output planes; each input
// plane's kRY + 2 rows, loaded into their registers right after their last
// product, feed the output rows of the three output planes in reach, held in
// a ring of accumulators.  ReLU, BF16 out.  Against one wavefront per
// 16 x 4 x 4 tile of output rows (36 input rows per 16 output rows) the
// network takes 1.04 instead of 1.07 ms at 256^3.
template <int ZC>
__global__ void __launch_bounds__(256) k_conv4_zm(int n, int batch, const uint16_t* __restrict__ in,
                                                  const v4s* __restrict__ wpk,
                                                  uint16_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int segs = n / 16, nyb = n / kRY, nzc = n / ZC;
    const long nwaves = (long)batch * nzc * nyb * segs;
    if (wave >= nwaves) return;  // whole wavefront; no block barrier below
    const int iseg = (int)(wave % segs);
    long rest = wave / segs;
    const int j0 = (int)(rest % nyb) * kRY;
    rest /= nyb;
    const int k0 = (int)(rest % nzc) * ZC;
    const int b = (int)(rest / nzc);
    const size_t N = (size_t)n * n * n, nn = (size_t)n * n;
    const int m = lane & 15, g = lane >> 4;
    v4s B[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) B[t] = wpk[t * 64 + lane];
    constexpr int kRW = kRY + 2;
    const uint16_t* inb = in + (size_t)b * N * 4;
    const int xo = wrapn(iseg * 16 + m + (g < 3 ? g - 1 : 0), n);   // group 3: weights are zero
    int off[kRW];
#pragma unroll
    for (int iy = 0; iy < kRW; ++iy) off[iy] = (n * wrapn(j0 - 1 + iy, n) + xo) * 4;
    auto plane_ptr = [&](int t) { return inb + nn * 4 * (size_t)wrapn(k0 - 1 + t, n); };
    v4s a[kRW];
    {
        const uint16_t* pb = plane_ptr(0);
#pragma unroll
        for (int iy = 0; iy < kRW; ++iy) a[iy] = *reinterpret_cast<const v4s*>(pb + off[iy]);
    }
    v4f acc[3][kRY];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int oy = 0; oy < kRY; ++oy) acc[r][oy] = v4f{0.f, 0.f, 0.f, 0.f};
    uint16_t* outb = out + (size_t)b * N * 16;
#pragma unroll
    for (int t = 0; t < ZC + 2; ++t) {
        const bool more = t + 1 < ZC + 2;
        const uint16_t* pn = plane_ptr(more ? t + 1 : t);
#pragma unroll
        for (int iy = 0; iy < kRW; ++iy) {
#pragma unroll
            for (int dz = -1; dz <= 1; ++dz) {
                const int oz = t - 1 - dz;   // ring slot oz mod 3
                if (oz < 0 || oz >= ZC) continue;
#pragma unroll
                for (int oy = 0; oy < kRY; ++oy) {
                    const int dy = iy - 1 - oy;
                    if (dy < -1 || dy > 1) continue;
                    acc[oz % 3][oy] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                        B[(dz + 1) * 3 + dy + 1], a[iy], acc[oz % 3][oy], 0, 0, 0);
                }
            }
            if (more) a[iy] = *reinterpret_cast<const v4s*>(pn + off[iy]);
        }
        if (t >= 2) {   // output plane t - 2 has had its last input plane
            store_plane_rows<false>(acc[(t - 2) % 3], outb, nullptr, n, iseg * 16 + m, j0, k0 + t - 2,
                                    g);
#pragma unroll
            for (int oy = 0; oy < kRY; ++oy) acc[(t - 2) % 3][oy] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    }
}

// The first layer of a training step, and MASKED the data gradient of the last:
// a convolution of a channel-last BF16 [cell][4] field with 4 taps to a K-block
// (tap 4 kb + g in lane group g), the grouping the training sums have had all
// along: the z-march above groups the taps of one row instead, and a
// regrouped FP32 sum rounds an activation in 10^5 the other way, which Adam's
// first steps (the sign of each gradient entry) blow up to 1e-3 of the next
// gradient.  A wavefront owns 16 cells along x times kTR rows along y, so that
// its weight operands serve kTR products and 7 kTR loads are in flight
// (one row per wavefront took 25 us for 16 grids of 32^3, this 15).
constexpr int kTR = 4;
template <bool MASKED>
__global__ void __launch_bounds__(256) k_conv4_taps(int n, int batch, const uint16_t* __restrict__ in,
                                                    const v4s* __restrict__ wpk,
                                                    const uint16_t* __restrict__ mask,
                                                    uint16_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int segs = n / 16, nyb = n / kTR;
    if (wave >= (long)batch * n * nyb * segs) return;  // whole wavefront; no block barrier below
    const int iseg = (int)(wave % segs);
    long rest = wave / segs;
    const int j0 = (int)(rest % nyb) * kTR;
    rest /= nyb;
    const int k = (int)(rest % n), b = (int)(rest / n);
    const size_t N = (size_t)n * n * n, nn = (size_t)n * n;
    const int m = lane & 15, g = lane >> 4;
    const uint16_t* inb = in + (size_t)b * N * 4;
    v4s B[kTapBlocks], a[kTR][kTapBlocks];
#pragma unroll
    for (int kb = 0; kb < kTapBlocks; ++kb) B[kb] = wpk[kb * 64 + lane];
#pragma unroll
    for (int kb = 0; kb < kTapBlocks; ++kb) {
        const int tap = 4 * kb + g < 27 ? 4 * kb + g : 26;   // past the last: its weights are zero
        const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
        const uint16_t* pl = inb + (nn * wrapn(k + dz, n) + wrapn(iseg * 16 + m + dx, n)) * 4;
#pragma unroll
        for (int e = 0; e < kTR; ++e)
            a[e][kb] = *reinterpret_cast<const v4s*>(pl + (size_t)n * wrapn(j0 + e + dy, n) * 4);
    }
    v4f acc[kTR];
#pragma unroll
    for (int e = 0; e < kTR; ++e) {
        acc[e] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < kTapBlocks; ++kb)
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(B[kb], a[e][kb], acc[e], 0, 0, 0);
    }
    const size_t off = (size_t)b * N * 16;
    static_assert(kTR == kRY, "store_plane_rows takes kRY rows");
    store_plane_rows<MASKED>(acc, out + off, MASKED ? mask + off : nullptr, n, iseg * 16 + m, j0, k, g);
}

// ---- weight gradients ----
// D[co][(tap, ci)] = sum over the cells of g[cell][co] in[cell + d(tap)][ci]: a
// contraction over the cells, so both matrix operands want 8 consecutive cells
// of one channel per lane, while the fields are channel-last.  A block stages a
// 16 x 8 column of cells plane by plane in LDS with the channels outermost
// (kernels before this loaded every operand entry as a 2-byte gather from
// global memory, 112 loads a lane for 27 products of 16 cells) and marches
// along z over zc planes, a ring of planes in LDS, the next plane's loads in
// flight during the products.  A wavefront owns two rows: the K = 32 cells of a
// product are their 2 x 16 cells, lane group gq holding cells 8 (gq & 1) .. + 7
// of row gq >> 1.  The four wavefronts' FP32 sums are added in FP64 and leave
// as one FP64 partial per block; a block works on every kWgBlocks-th unit
// (column, chunk of planes), so a sum takes no more FP32 additions of products
// than one of 16-cell products with a wavefront per 1/1024 of the cells (from 16^3 to
// 256^3 and 64 grids; it may run over more cells, 32 against 16 for one grid of
// 16^3).  k_wgrad_total adds the partials
// of all layers, 16 slices of blocks at a time (one thread per entry walked them
// all: 245 us a layer).  16 grids of 32^3: 22 us for a 16 -> 16 layer against
// 65, 10 for the first and 9 for the last against 84 and 65, the totals of the
// four layers 9 us against 980.  Bound: the planes' load latency, one plane
// ahead, over 17 planes in turn.
constexpr int kWgX = 16, kWgY = 8;       // cells of a column in x and y
constexpr int kWgBlocks = 512;           // most blocks (partials) per layer
// Units wanted: one 768-thread block per CU for the 16 -> 16 layers (two took as
// long, 21 us, and left twice the partials: their total 11 against 9 us), two of
// 256 threads for the first and last layer (9 against 12 us for the last).
constexpr int kWgUnits16 = 256, kWgUnitsSmall = 512;
struct WgShape {
    int zc, nzc, units, blocks;
};
static WgShape wg_shape(int n, int batch, int want) {
    WgShape w;
    const long cols = (long)batch * (n / kWgX) * (n / kWgY);
    w.nzc = cols >= want ? 1 : (int)std::min<long>(n, (want + cols - 1) / cols);
    w.zc = (n + w.nzc - 1) / w.nzc;
    w.nzc = (n + w.zc - 1) / w.zc;
    w.units = (int)(cols * w.nzc);
    w.blocks = std::min(w.units, kWgBlocks);
    return w;
}
constexpr int kWgBig = 27 * 256, kWgLast = 2 * 256, kWgFirst = 4 * 256;   // entries of a partial

// One 16-channel plane of a column, channels outermost: rows j0 - H .. j0 + 7 + H
// and cells i0 - H .. i0 + 15 + H.  With the halo the rows are 24 entries apart
// (x at entry 8 + x, so that x = 0 and 8 are 16-byte aligned and x = 16 falls
// on the next row's unused entry 0); a channel takes an odd number of 16-byte
// units, so that the 16 channels of a 16-byte read spread over the banks.
template <int H, int THREADS>
struct WgTile {
    static constexpr int kRows = kWgY + 2 * H, kCols = kWgX + 2 * H;
    static constexpr int kPitch = H ? 24 : 16, kOff = H ? 8 : 0;
    static constexpr int kCh = kRows * kPitch + 8;
    static constexpr int kSize = 16 * kCh;
    static constexpr int kJobs = kRows * kCols * 2;      // 8 channels of one cell each
    static constexpr int kPer = (kJobs + THREADS - 1) / THREADS;
    int src[kPer], dst[kPer];   // entry offset in a plane and in the tile (dst < 0: idle)
    v8s val[kPer];
    __device__ void init(int n, int i0, int j0, int tid) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int job = tid + THREADS * q, cell = job >> 1, half = job & 1;
            const int row = cell / kCols, x = cell % kCols - H;
            const bool has = job < kJobs;
            src[q] = has ? (n * wrapn(j0 - H + row, n) + wrapn(i0 + x, n)) * 16 + 8 * half : 0;
            dst[q] = has ? 8 * half * kCh + row * kPitch + kOff + x : -1;
        }
    }
    __device__ void load(const uint16_t* plane) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) val[q] = *reinterpret_cast<const v8s*>(plane + src[q]);
    }
    __device__ void store(uint16_t* tile) const {
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (dst[q] >= 0)
#pragma unroll
                for (int e = 0; e < 8; ++e) tile[dst[q] + e * kCh] = (uint16_t)val[q][e];
    }
};

// The partials of a block: NT tiles of 16 x 16, held NT / G each by the G groups
// of four wavefronts (group w / 4), a group's sums added in FP64 in wavefront
// order.  lds: 4 x 9 x 256 floats.
template <int NT, int G>
__device__ inline void wg_store(const v4f (&acc)[NT / G], float* lds, double* __restrict__ part) {
    constexpr int M = NT / G;
    static_assert(M <= 9, "a group's sums fit the space");
    const int tid = threadIdx.x, lane = tid & 63, wv = (tid >> 6) & 3;
    for (int g = 0; g < G; ++g) {
        __syncthreads();
        if ((tid >> 8) == g)
#pragma unroll
            for (int t = 0; t < M; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)   // lane holds D[4 (lane >> 4) + e][lane & 15]
                    lds[(wv * M + t) * 256 + (4 * (lane >> 4) + e) * 16 + (lane & 15)] = acc[t][e];
        __syncthreads();
        for (int i = tid; i < M * 256; i += 256 * G) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) s += (double)lds[w * M * 256 + i];
            part[((size_t)blockIdx.x * NT + (size_t)g * M) * 256 + i] = s;
        }
    }
}

// 16 -> 16 layer: tile t of the partial is D[co][ci] of tap t.  Twelve
// wavefronts: group dz takes the taps of one dz on the same column.
constexpr int kWg16Threads = 768;
__global__ void __launch_bounds__(kWg16Threads) k_wgrad16(int n, const uint16_t* __restrict__ in,
                                                    const uint16_t* __restrict__ gr, WgShape ws,
                                                    double* __restrict__ part) {
    typedef WgTile<1, kWg16Threads> In;
    typedef WgTile<0, kWg16Threads> Gr;
    constexpr int kLdsIn = 4 * In::kSize, kLds = kLdsIn + 2 * Gr::kSize;
    static_assert(kLds * 2 >= 4 * 9 * 256 * 4, "the partials' sums fit the tiles' space");
    __shared__ __align__(16) uint16_t lds[kLds];
    uint16_t* const ldsg = lds + kLdsIn;
    const int tid = threadIdx.x, lane = tid & 63, wv = (tid >> 6) & 3, dz = tid >> 8;
    const int m = lane & 15, gq = lane >> 4;
    const int r = 2 * wv + (gq >> 1), x0 = 8 * (gq & 1);
    const size_t nn16 = (size_t)n * n * 16;
    const int oa = m * Gr::kCh + r * Gr::kPitch + x0;
    const int ob = m * In::kCh + r * In::kPitch + In::kOff + x0;
    v4f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    const int gx = n / kWgX, gy = n / kWgY;
    for (int u = blockIdx.x; u < ws.units; u += gridDim.x) {
        const int i0 = (u % gx) * kWgX;
        int rest = u / gx;
        const int j0 = (rest % gy) * kWgY;
        rest /= gy;
        const int k0 = (rest % ws.nzc) * ws.zc, b = rest / ws.nzc;
        const int k1 = k0 + ws.zc < n ? k0 + ws.zc : n;
        const uint16_t* inb = in + (size_t)b * n * nn16;
        const uint16_t* grb = gr + (size_t)b * n * nn16;
        In ti;
        Gr tg;
        ti.init(n, i0, j0, tid);
        tg.init(n, i0, j0, tid);
        __syncthreads();   // the last unit's products are done with the tiles
        // plane k0 - 1 + t in ring slot t & 3
        for (int t = 0; t < 3; ++t) {
            ti.load(inb + nn16 * (size_t)wrapn(k0 - 1 + t, n));
            ti.store(lds + t * In::kSize);
        }
        tg.load(grb + nn16 * (size_t)k0);
        tg.store(ldsg);
        __syncthreads();
        for (int t = 0; t < k1 - k0; ++t) {
            // the planes of the next step; past the chunk's end they repeat the last
            const int kn = k0 + t + 1 < k1 ? k0 + t + 1 : k0 + t;
            ti.load(inb + nn16 * (size_t)wrapn(kn + 1, n));
            tg.load(grb + nn16 * (size_t)kn);
            const v8s a = *reinterpret_cast<const v8s*>(ldsg + (t & 1) * Gr::kSize + oa);
            const uint16_t* pl = lds + ((t + dz) & 3) * In::kSize + ob;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const uint16_t* p = pl + dy * In::kPitch;
                typedef uint32_t v4u __attribute__((ext_vector_type(4)));
                const v4u c = *reinterpret_cast<const v4u*>(p);
                const uint32_t lo = p[-1], hi = p[8];
                // the same 8 cells one step to the left and to the right
                const v4u l = {c[0] << 16 | lo, __builtin_amdgcn_alignbit(c[1], c[0], 16),
                               __builtin_amdgcn_alignbit(c[2], c[1], 16),
                               __builtin_amdgcn_alignbit(c[3], c[2], 16)};
                const v4u h = {l[1], l[2], l[3], hi << 16 | c[3] >> 16};
                acc[3 * dy] = mfma_k32(a, __builtin_bit_cast(v8s, l), acc[3 * dy]);
                acc[3 * dy + 1] = mfma_k32(a, __builtin_bit_cast(v8s, c), acc[3 * dy + 1]);
                acc[3 * dy + 2] = mfma_k32(a, __builtin_bit_cast(v8s, h), acc[3 * dy + 2]);
            }
            ti.store(lds + ((t + 3) & 3) * In::kSize);
            tg.store(ldsg + ((t + 1) & 1) * Gr::kSize);
            __syncthreads();
        }
    }
    wg_store<27, 3>(acc, reinterpret_cast<float*>(lds), part);
}

// First and last layer: a 16-channel field and a field of NCH (2 or 1) channels,
// channel-last [cell][4]: D[c][col] = sum over the cells of big[cell][c]
// small[cell + SIGN d(tap)][ch], col = NCH tap + ch.  First layer: the output's
// gradient against the input at + d; last layer: the input against the output's
// gradient at - d.  The small field sits in LDS once per x shift, so that
// every lane's 8 cells are one aligned read.
template <int NCH, int SIGN>
__global__ void __launch_bounds__(256, 2) k_wgrad_small(int n, const uint16_t* __restrict__ big,
                                                        const uint16_t* __restrict__ small,
                                                        WgShape ws, double* __restrict__ part) {
    typedef WgTile<0, 256> Big;
    constexpr int NT = (27 * NCH + 15) / 16, kR = kWgY + 2, kC = kWgX + 2;
    // one plane of the small field: [x shift][channel][row][x], rows 16 entries
    constexpr int kSm = 3 * NCH * kR * kWgX;
    constexpr int kTiles = 2 * Big::kSize + 4 * kSm, kSums = 4 * 9 * 256 * 2;
    __shared__ __align__(16) uint16_t lds[kTiles > kSums ? kTiles : kSums];
    uint16_t* const ldss = lds + 2 * Big::kSize;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, gq = lane >> 4;
    const int r = 2 * wv + (gq >> 1), x0 = 8 * (gq & 1);
    const size_t nn = (size_t)n * n;
    const int oa = m * Big::kCh + r * Big::kPitch + x0;
    // this lane's column of each tile: offset in a plane, plane shift (-1, 0, 1)
    int ob[NT], dzs[NT];
    bool has[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int col = 16 * t + m, tap = col / NCH, ch = col % NCH;
        has[t] = tap < 27;
        const int tp = has[t] ? tap : 13;
        dzs[t] = SIGN * (tp / 9 - 1);
        ob[t] = (((tp % 3) * NCH + ch) * kR + r + 1 + SIGN * ((tp / 3) % 3 - 1)) * kWgX + x0;
    }
    v4f acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    const int gx = n / kWgX, gy = n / kWgY;
    for (int u = blockIdx.x; u < ws.units; u += gridDim.x) {
        const int i0 = (u % gx) * kWgX;
        int rest = u / gx;
        const int j0 = (rest % gy) * kWgY;
        rest /= gy;
        const int k0 = (rest % ws.nzc) * ws.zc, b = rest / ws.nzc;
        const int k1 = k0 + ws.zc < n ? k0 + ws.zc : n;
        const uint16_t* bigb = big + (size_t)b * n * nn * 16;
        const uint16_t* smb = small + (size_t)b * n * nn * 4;
        Big tb;
        tb.init(n, i0, j0, tid);
        // one cell of the small field per thread (rows j0 - 1 .., cells i0 - 1 ..)
        const int row = tid / kC, x = tid % kC - 1;
        const bool job = tid < kR * kC;
        const int src = job ? (n * wrapn(j0 - 1 + row, n) + wrapn(i0 + x, n)) * 4 : 0;
        auto put = [&](v4s v, uint16_t* plane) {
            if (!job) return;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int xs = x - SIGN * (d - 1);   // the copy of shift d holds small at x + SIGN (d - 1)
                if (xs >= 0 && xs < kWgX)
#pragma unroll
                    for (int ch = 0; ch < NCH; ++ch)
                        plane[((d * NCH + ch) * kR + row) * kWgX + xs] = (uint16_t)v[ch];
            }
        };
        auto get = [&](int k) { return *reinterpret_cast<const v4s*>(smb + nn * 4 * (size_t)wrapn(k, n) + src); };
        __syncthreads();
        for (int t = 0; t < 3; ++t) put(get(k0 - 1 + t), ldss + t * kSm);   // ring slot t & 3
        tb.load(bigb + nn * 16 * (size_t)k0);
        tb.store(lds);
        __syncthreads();
        for (int t = 0; t < k1 - k0; ++t) {
            const int kn = k0 + t + 1 < k1 ? k0 + t + 1 : k0 + t;
            const v4s nx = get(kn + 1);
            tb.load(bigb + nn * 16 * (size_t)kn);
            const v8s a = *reinterpret_cast<const v8s*>(lds + (t & 1) * Big::kSize + oa);
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                v8s c = *reinterpret_cast<const v8s*>(ldss + ((t + 1 + dzs[q]) & 3) * kSm + ob[q]);
                if (!has[q]) c = v8s{0, 0, 0, 0, 0, 0, 0, 0};
                acc[q] = mfma_k32(a, c, acc[q]);
            }
            put(nx, ldss + ((t + 3) & 3) * kSm);
            tb.store(lds + ((t + 1) & 1) * Big::kSize);
            __syncthreads();
        }
    }
    wg_store<NT, 1>(acc, reinterpret_cast<float*>(lds), part);
}

// The gradient of every layer from its blocks' partials, in the weights' layout
// [co][ci][27]: 64 entries per block of 1024 threads, the partials in 16
// slices, each summed in block order, the slices added in order.
__global__ void __launch_bounds__(1024) k_wgrad_total(const double* __restrict__ part, int nb16,
                                                      int nbs, float* __restrict__ grad) {
    __shared__ double lds[16][64];
    constexpr int kL[4] = {kWgFirst, kWgBig, kWgBig, kWgLast};
    const int ex = threadIdx.x & 63, sl = threadIdx.x >> 6;
    int e = blockIdx.x * 64 + ex, layer = 0;   // 64 divides every kL
    size_t off = 0;
    int w0 = 0;
#pragma unroll
    for (int l = 0; l < 3; ++l)
        if (layer == l && e >= kL[l]) {
            e -= kL[l];
            off += (size_t)(l == 0 ? nbs : nb16) * kL[l];
            w0 += l == 0 ? 2 * 16 * 27 : 16 * 16 * 27;
            layer = l + 1;
        }
    const int ne = layer == 0 ? kWgFirst : layer == 3 ? kWgLast : kWgBig;
    const int nb = layer == 0 || layer == 3 ? nbs : nb16;
    const int per = (nb + 15) / 16, b0 = sl * per, b1 = b0 + per < nb ? b0 + per : nb;
    const double* p = part + off + e;
    double s = 0.0;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += p[(size_t)b * ne];
    lds[sl][ex] = s;
    __syncthreads();
    if (sl != 0) return;
    s = lds[0][ex];
#pragma unroll
    for (int q = 1; q < 16; ++q) s += lds[q][ex];
    const int tile = e / 256, row = (e % 256) / 16, col = e % 16;
    int idx;
    bool has = true;
    if (layer == 0) {          // rows co, columns 2 tap + ci
        const int c = 16 * tile + col;
        has = c < 54;
        idx = (row * 2 + c % 2) * 27 + c / 2;
    } else if (layer == 3) {   // rows ci, columns tap
        const int c = 16 * tile + col;
        has = c < 27;
        idx = row * 27 + c;
    } else {                   // rows co, columns ci, one tile per tap
        idx = (row * 16 + col) * 27 + tile;
    }
    if (has) grad[w0 + idx] = (float)s;
}

// ---- weight packing ----
// One weight of a layer [co][ci][27] as a convolution's operand: output channel
// o, input channel i of tap t; flip: of the layer's data gradient (the
// transposed layer with the taps mirrored).
__device__ inline float weight_of(const float* __restrict__ w, int cin, int cout, bool flip, int o,
                                  int i, int t) {
    if (!flip) return o < cout && i < cin ? w[((size_t)o * cin + i) * 27 + t] : 0.f;
    return o < cin && i < cout ? w[((size_t)i * cin + o) * 27 + 26 - t] : 0.f;
}

// For k_conv4_zm: one K-block per input-row offset (dy, dz), kb = (dz+1) 3 + (dy+1);
// its K entry 4 g + c holds channel c of the cell dx = g - 1 along x (g = 3 is zero).
__device__ inline v4s pack_rows4(const float* __restrict__ w, int t) {
    const int kb = t / 64, lane = t % 64;
    const int nn = lane & 15, g = lane >> 4;
    const int tap = (kb / 3) * 9 + (kb % 3) * 3 + g;
    v4s v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = (short)f2bf(g < 3 ? weight_of(w, 2, 16, false, nn, e, tap) : 0.f);
    return v;
}

// For k_conv4_taps: K-block kb, lane (n = co, g): the channels of tap 4 kb + g.
__device__ inline v4s pack_taps(const float* __restrict__ w, int cin, int cout, bool flip, int t) {
    const int lane = t % 64, nn = lane & 15, tap = 4 * (t / 64) + (lane >> 4);
    v4s v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = (short)f2bf(tap < 27 ? weight_of(w, cin, cout, flip, nn, e, tap) : 0.f);
    return v;
}

// For k_conv16_zm: operand (c, s, dz) at lane (n = co, g) holds in entry j the
// weight of channel 8 (g & 1) + j for item rr = 2 s + (g >> 1) - c of the
// output row's run, rr = 3 (dy + 1) + dx + 1, zero outside 0..8.
__device__ inline v8s pack_pairs(const float* __restrict__ w, bool flip, int t) {
    const int op = t / 64, lane = t % 64;
    const int dz = op % 3, s = (op / 3) % kSlots, c = op / (3 * kSlots);
    const int co = lane & 15, g = lane >> 4, rr = 2 * s + (g >> 1) - c;
    v8s v;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = (short)f2bf(rr >= 0 && rr < 9
                               ? weight_of(w, 16, 16, flip, co, 8 * (g & 1) + j, dz * 9 + rr)
                               : 0.f);
    return v;
}

// Packed operands: first layer's rows, the last layer's taps (k_conv16_final_zm:
// [tap * 4 + g] = channels 4 g .. 4 g + 3), the 16 -> 16 layers' pairs; for
// training also the first layer's taps and, for the data gradients, the last
// layer's taps and the 16 -> 16 layers' pairs.
constexpr int kRowOps = 9 * 64, kTapOps = kTapBlocks * 64, kFinOps = 27 * 4, kPairOps = 2 * kSlots * 3 * 64;
struct Packed {
    v4s row1[kRowOps];
    v4s fin[kFinOps];
    v8s pair[2][kPairOps];
    v4s taps[2][kTapOps];      // from here on: training only
    v8s bpair[2][kPairOps];
};
static_assert((kRowOps + kFinOps) % 2 == 0 && kTapOps % 2 == 0, "pair operands stay 16-byte aligned");
constexpr int kPackForward = kRowOps + kFinOps + 2 * kPairOps;
constexpr int kPackAll = kPackForward + 2 * kTapOps + 2 * kPairOps;

// Every operand in one launch (one kernel per operand took 11 launches, a
// fifth of the network's time on a 32^3 grid).
__device__ inline void pack_operand(const float* __restrict__ w, Packed* __restrict__ p, int t) {
    const float* w1 = w + 2 * 16 * 27;
    const float* w2 = w1 + 16 * 16 * 27;
    const float* w3 = w2 + 16 * 16 * 27;
    if (t < kRowOps) {
        p->row1[t] = pack_rows4(w, t);
        return;
    }
    if ((t -= kRowOps) < kFinOps) {
        v4s v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (short)f2bf(w3[(size_t)(4 * (t % 4) + e) * 27 + t / 4]);
        p->fin[t] = v;
        return;
    }
    if ((t -= kFinOps) < 2 * kPairOps) {
        const int l = t / kPairOps;
        p->pair[l][t - l * kPairOps] = pack_pairs(l ? w2 : w1, false, t - l * kPairOps);
        return;
    }
    if ((t -= 2 * kPairOps) < 2 * kTapOps) {
        if (t < kTapOps) p->taps[0][t] = pack_taps(w, 2, 16, false, t);
        else p->taps[1][t - kTapOps] = pack_taps(w3, 16, 1, true, t - kTapOps);
        return;
    }
    t -= 2 * kTapOps;
    const int l = t / kPairOps;
    p->bpair[l][t - l * kPairOps] = pack_pairs(l ? w2 : w1, true, t - l * kPairOps);
}

__global__ void __launch_bounds__(256) k_pack(const float* __restrict__ w, Packed* __restrict__ p,
                                              int count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) pack_operand(w, p, t);
}

// The start of a pass in one launch: the first blocks pack the weights (count of
// Packed's operands), the others convert the network's input to channel-last
// BF16 [cell][4] = (x0, x1, 0, 0) from FP32 [cell][2].  Each was a launch of its
// own, 5 us for the pack.
__global__ void __launch_bounds__(256) k_begin(const float* __restrict__ w, Packed* __restrict__ p,
                                               int count, const float* __restrict__ x,
                                               uint16_t* __restrict__ xb, size_t cells) {
    const unsigned nb = (unsigned)(count + 255) / 256;
    if (blockIdx.x < nb) {
        const int t = blockIdx.x * 256 + threadIdx.x;
        if (t < count) pack_operand(w, p, t);
        return;
    }
    size_t i = (size_t)(blockIdx.x - nb) * 256 + threadIdx.x;
    const size_t stride = (size_t)(gridDim.x - nb) * 256;
    for (; i < cells; i += stride) {
        xb[4 * i + 0] = f2bf(x[2 * i + 0]);
        xb[4 * i + 1] = f2bf(x[2 * i + 1]);
        xb[4 * i + 2] = 0;
        xb[4 * i + 3] = 0;
    }
}
static void begin(hipStream_t s, const float* w, Packed* p, int count, const float* x, uint16_t* xb,
                  size_t cells) {
    const unsigned nb = (unsigned)(count + 255) / 256;
    const unsigned lin = (unsigned)std::min<size_t>((cells + 255) / 256, 65536);
    hipLaunchKernelGGL(k_begin, dim3(nb + lin), dim3(256), 0, s, w, p, count, x, xb, cells);
}

// MSE loss partials and the output gradient dy = 2 (y - t) / count as BF16 [cell][4].
__global__ void __launch_bounds__(256) k_mse(const float* __restrict__ y, const float* __restrict__ t,
                                             size_t count, float scale, uint16_t* __restrict__ dy,
                                             double* part) {
    double v[1] = {0.0};
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) {
        const float d = y[i] - t[i];
        v[0] += (double)d * (double)d;
        dy[4 * i + 0] = f2bf(scale * d);
        dy[4 * i + 1] = 0;
        dy[4 * i + 2] = 0;
        dy[4 * i + 3] = 0;
    }
    block_partials<1, 0u>(v, part);
}

// ---- training on the solve's own measure ----
// For one sample with the captured system (b, diag, w) of M x = b and the
// network output g: u = M g, alpha = g.b / g.u (the start rescale of the
// solve), r = b - alpha u and the loss L = |r|^2 / |b|^2, the relative
// residual the solve starts from (invariant to the scale of g and b).  With
// c = g.u:  dL/dg = -(2 / |b|^2) [ (u.r / c) (b - 2 alpha u) + alpha M r ].
// M v = diag v - (1/h^2) sum_f K_f v_nb(f), K_f = I4(w) on face f: the
// pressure operator written with its diagonal.  FP64 arithmetic on the FP32
// network output.
constexpr int kResBlocks = 64;   // blocks per sample (grid kResBlocks x batch)

template <typename V>
__device__ inline double m_offdiag(const double* __restrict__ w, const CellIdx& c, V&& v) {
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) s += i4(w, c, d, 0) * v(c.sh(d, 1)) + i4(w, c, d, -1) * v(c.sh(d, -1));
    return s;
}

__global__ void __launch_bounds__(256) k_res_u(int n, double inv_h2, const double* __restrict__ b,
                                               const double* __restrict__ diag,
                                               const double* __restrict__ w, const float* __restrict__ y,
                                               double* __restrict__ u, double* part) {
    const BlockXYZ bx = block_xyz();
    const size_t N = (size_t)n * n * n, base = (size_t)bx.y * N;
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};   // g.b, g.u, u.b, u.u, b.b
    for (size_t i = (size_t)bx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        const CellIdx c(n, (int)(i % n), (int)((i / n) % n), (int)(i / ((size_t)n * n)), base);
        const size_t P = c.self();
        const double gP = y[P], bP = b[P];
        const double uP = diag[P] * gP - inv_h2 * m_offdiag(w, c, [&](size_t Q) { return (double)y[Q]; });
        u[P] = uP;
        v[0] += gP * bP;
        v[1] += gP * uP;
        v[2] += uP * bP;
        v[3] += uP * uP;
        v[4] += bP * bP;
    }
    block_partials<5, 0u>(v, part);
}

// Per sample (one block each): coef = (alpha, u.r / c, -2 / (|b|^2 batch), its loss).
__global__ void __launch_bounds__(256) k_res_coef(const double* __restrict__ part,
                                                  double* __restrict__ coef) {
    const int sm = blockIdx.x, batch = gridDim.x;
    double t[5];
    reduce_partials_strided<5, 0u>(part, (size_t)kResBlocks * batch, (size_t)sm * kResBlocks,
                                   kResBlocks, t);
    if (threadIdx.x == 0) {
        const double gb = t[0], gu = t[1], ub = t[2], uu = t[3], bb = t[4];
        const bool ok = gu > 0.0 && bb > 0.0;
        const double alpha = ok ? gb / gu : 0.0;
        const double ur = ub - alpha * uu;
        coef[4 * sm + 0] = alpha;
        coef[4 * sm + 1] = ok ? ur / gu : 0.0;
        coef[4 * sm + 2] = ok ? -2.0 / (bb * batch) : 0.0;
        coef[4 * sm + 3] = ok ? (bb - 2.0 * alpha * ub + alpha * alpha * uu) / bb : 1.0;
    }
}

// Output gradient dL/dg as BF16 [cell][4] (channel 0), for the backward pass;
// the first block's first thread also writes the batch mean of the losses,
// added in sample order.
__global__ void __launch_bounds__(256) k_res_dy(int n, double inv_h2, const double* __restrict__ b,
                                                const double* __restrict__ diag,
                                                const double* __restrict__ w,
                                                const double* __restrict__ u,
                                                const double* __restrict__ coef,
                                                uint16_t* __restrict__ dy, double* loss) {
    const BlockXYZ bx = block_xyz();
    const size_t N = (size_t)n * n * n, base = (size_t)bx.y * N;
    const double alpha = coef[4 * bx.y], beta = coef[4 * bx.y + 1], sc = coef[4 * bx.y + 2];
    for (size_t i = (size_t)bx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        const CellIdx c(n, (int)(i % n), (int)((i / n) % n), (int)(i / ((size_t)n * n)), base);
        const size_t P = c.self();
        auto r = [&](size_t Q) { return b[Q] - alpha * u[Q]; };
        const double Mr = diag[P] * r(P) - inv_h2 * m_offdiag(w, c, r);
        const double g = sc * (beta * (b[P] - 2.0 * alpha * u[P]) + alpha * Mr);
        dy[4 * P + 0] = f2bf((float)g);
        dy[4 * P + 1] = 0;
        dy[4 * P + 2] = 0;
        dy[4 * P + 3] = 0;
    }
    if (bx.x == 0 && bx.y == 0 && threadIdx.x == 0) {
        const int batch = gridDim.y;
        double total = 0.0;
        for (int sm = 0; sm < batch; ++sm) total += coef[4 * sm + 3];
        *loss = total / batch;
    }
}

__global__ void k_adam(int nw, float* __restrict__ w, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nw) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------
size_t net_packed_bytes() { return offsetof(Packed, taps); }

void net_pack_forward(hipStream_t s, const float* w32, void* wpk) {
    hipLaunchKernelGGL(k_pack, dim3((kPackForward + 255) / 256), dim3(256), 0, s, w32,
                       reinterpret_cast<Packed*>(wpk), kPackForward);
}

// Output planes per wavefront of the z-marches: the longest chunk (16, 8 or 4
// planes, dividing n) that still gives at least 4096 wavefronts (32 planes
// would spill registers).
static int zm_chunk(int n, int batch) {
    const long per_plane = (long)batch * (n / kRY) * (n / 16);
    for (int zc = 16; zc > 4; zc /= 2)
        if (n % zc == 0 && per_plane * (n / zc) >= 4096) return zc;
    return 4;
}
static unsigned zm_blocks(int n, int batch, int zc) {
    const long waves = (long)batch * (n / zc) * (n / kRY) * (n / 16);
    return (unsigned)((waves + 3) / 4);
}

template <bool MASKED>
static void conv4_taps(hipStream_t s, int n, int batch, const uint16_t* src, const v4s* w,
                       const uint16_t* mask, uint16_t* dst) {
    const long waves = (long)batch * n * (n / kTR) * (n / 16);
    hipLaunchKernelGGL(k_conv4_taps<MASKED>, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, n,
                       batch, src, w, mask, dst);
}
template <bool MASKED>
static void conv16(hipStream_t s, int n, int batch, const uint16_t* src, const v8s* w,
                   const uint16_t* mask, uint16_t* dst) {
    const int zc = zm_chunk(n, batch);
    const dim3 G(zm_blocks(n, batch, zc)), B(256);
    switch (zc) {
    case 16: hipLaunchKernelGGL((k_conv16_zm<16, MASKED>), G, B, 0, s, n, batch, src, w, mask, dst); break;
    case 8: hipLaunchKernelGGL((k_conv16_zm<8, MASKED>), G, B, 0, s, n, batch, src, w, mask, dst); break;
    default: hipLaunchKernelGGL((k_conv16_zm<4, MASKED>), G, B, 0, s, n, batch, src, w, mask, dst); break;
    }
}

// Layers 2 to 4 from the first layer's activations a1 (a3 may be a1).
static void forward_from(hipStream_t s, int n, int batch, const Packed* p, const uint16_t* a1,
                         uint16_t* a2, uint16_t* a3, float* y, float yscale) {
    conv16<false>(s, n, batch, a1, p->pair[0], nullptr, a2);
    conv16<false>(s, n, batch, a2, p->pair[1], nullptr, a3);
    const int zc = zm_chunk(n, batch);
    const dim3 G(zm_blocks(n, batch, zc)), B(256);
    switch (zc) {
    case 16: hipLaunchKernelGGL(k_conv16_final_zm<16>, G, B, 0, s, n, batch, a3, p->fin, y, yscale); break;
    case 8: hipLaunchKernelGGL(k_conv16_final_zm<8>, G, B, 0, s, n, batch, a3, p->fin, y, yscale); break;
    default: hipLaunchKernelGGL(k_conv16_final_zm<4>, G, B, 0, s, n, batch, a3, p->fin, y, yscale); break;
    }
}

void net_forward(hipStream_t s, int n, int batch, const void* wpk, const uint16_t* x4,
                 uint16_t* a, uint16_t* b, float* y, float yscale) {
    const Packed* p = reinterpret_cast<const Packed*>(wpk);
    const int zc = zm_chunk(n, batch);
    const dim3 G(zm_blocks(n, batch, zc)), B(256);
    switch (zc) {
    case 16: hipLaunchKernelGGL(k_conv4_zm<16>, G, B, 0, s, n, batch, x4, p->row1, a); break;
    case 8: hipLaunchKernelGGL(k_conv4_zm<8>, G, B, 0, s, n, batch, x4, p->row1, a); break;
    default: hipLaunchKernelGGL(k_conv4_zm<4>, G, B, 0, s, n, batch, x4, p->row1, a); break;
    }
    forward_from(s, n, batch, p, a, b, a, y, yscale);
}

// ---- training workspace ----
struct NetWs {
    size_t x4, a1, a2, a3, y, g1, g2, dy, wf, part, lpart, ru, rpart, rcoef, total;
    WgShape wg, wgs;   // of the 16 -> 16 layers; of the first and last
    unsigned lblocks;
};

static NetWs net_layout(int n, int batch) {
    NetWs L{};
    const size_t cells = (size_t)batch * n * n * n;
    L.wg = wg_shape(n, batch, kWgUnits16);
    L.wgs = wg_shape(n, batch, kWgUnitsSmall);
    L.lblocks = 1024;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = (off + bytes + 255) / 256 * 256;
        return o;
    };
    L.x4 = take(cells * 4 * 2);
    L.a1 = take(cells * 16 * 2);
    L.a2 = take(cells * 16 * 2);
    L.a3 = take(cells * 16 * 2);
    L.y = take(cells * 4);
    L.g1 = take(cells * 16 * 2);
    L.g2 = take(cells * 16 * 2);
    L.dy = take(cells * 4 * 2);
    L.wf = take(sizeof(Packed));
    L.part = take(((size_t)L.wgs.blocks * (kWgFirst + kWgLast) + (size_t)L.wg.blocks * 2 * kWgBig) *
                  sizeof(double));
    L.lpart = take((size_t)L.lblocks * sizeof(double) + sizeof(double));
    L.ru = take(cells * sizeof(double));
    L.rpart = take((size_t)5 * kResBlocks * batch * sizeof(double));
    L.rcoef = take((size_t)4 * batch * sizeof(double));
    L.total = off;
    return L;
}

}  // namespace pisoc

using namespace pisoc;

static bool net_shape_ok(int32_t n, int32_t batch) {
    return n >= 16 && n <= PISOC_MAX_N && n % 16 == 0 && batch >= 1;
}

extern "C" {

size_t pisoc_net_workspace_bytes(int32_t n, int32_t batch) {
    if (!net_shape_ok(n, batch)) return 0;
    return net_layout(n, batch).total;
}

pisoc_status pisoc_net_forward(int32_t n, int32_t batch, const float* d_w, const float* d_x,
                               float* d_y, void* d_ws, size_t ws_bytes, void* stream) {
    if (!net_shape_ok(n, batch) || !d_w || !d_x || !d_y) return PISOC_ERR_INVALID;
    NetWs L = net_layout(n, batch);
    if (!d_ws || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* ws = reinterpret_cast<char*>(d_ws);
    const size_t cells = (size_t)batch * n * n * n;
    uint16_t* x4 = reinterpret_cast<uint16_t*>(ws + L.x4);
    begin(s, d_w, reinterpret_cast<Packed*>(ws + L.wf), kPackForward, d_x, x4, cells);
    net_forward(s, n, batch, ws + L.wf, x4, reinterpret_cast<uint16_t*>(ws + L.a1),
                reinterpret_cast<uint16_t*>(ws + L.a2), d_y, 1.f);
    return hipGetLastError() == hipSuccess ? PISOC_OK : PISOC_ERR_HIP;
}

// Forward pass of a training step keeping every activation in the
// workspace (y at L.y), after packing the forward and data-gradient weights.
static void grad_forward(hipStream_t s, const NetWs& L, char* ws, int n, int batch, const float* d_w,
                         const float* d_x) {
    auto U = [&](size_t off) { return reinterpret_cast<uint16_t*>(ws + off); };
    const size_t cells = (size_t)batch * n * n * n;
    Packed* p = reinterpret_cast<Packed*>(ws + L.wf);
    begin(s, d_w, p, kPackAll, d_x, U(L.x4), cells);
    conv4_taps<false>(s, n, batch, U(L.x4), p->taps[0], nullptr, U(L.a1));
    forward_from(s, n, batch, p, U(L.a1), U(L.a2), U(L.a3), reinterpret_cast<float*>(ws + L.y), 1.f);
}

// Weight gradient from the output gradient dy (BF16 [cell][4] at L.dy) and
// the activations grad_forward kept.
static void grad_backward(hipStream_t s, const NetWs& L, char* ws, int n, int batch, float* d_grad) {
    auto U = [&](size_t off) { return reinterpret_cast<uint16_t*>(ws + off); };
    const dim3 G(L.wg.blocks), GS(L.wgs.blocks), B(256);
    const Packed* p = reinterpret_cast<const Packed*>(ws + L.wf);
    // partials of layers 1 to 4, one after the other
    double* part1 = reinterpret_cast<double*>(ws + L.part);
    double* part2 = part1 + (size_t)L.wgs.blocks * kWgFirst;
    double* part3 = part2 + (size_t)L.wg.blocks * kWgBig;
    double* part4 = part3 + (size_t)L.wg.blocks * kWgBig;
    // layer 4 (linear), 3, 2, 1
    hipLaunchKernelGGL((k_wgrad_small<1, -1>), GS, B, 0, s, n, U(L.a3), U(L.dy), L.wgs, part4);
    conv4_taps<true>(s, n, batch, U(L.dy), p->taps[1], U(L.a3), U(L.g1));
    hipLaunchKernelGGL(k_wgrad16, G, dim3(kWg16Threads), 0, s, n, U(L.a2), U(L.g1), L.wg, part3);
    conv16<true>(s, n, batch, U(L.g1), p->bpair[1], U(L.a2), U(L.g2));
    hipLaunchKernelGGL(k_wgrad16, G, dim3(kWg16Threads), 0, s, n, U(L.a1), U(L.g2), L.wg, part2);
    conv16<true>(s, n, batch, U(L.g2), p->bpair[0], U(L.a1), U(L.g1));
    hipLaunchKernelGGL((k_wgrad_small<2, 1>), GS, B, 0, s, n, U(L.g1), U(L.x4), L.wgs, part1);
    hipLaunchKernelGGL(k_wgrad_total, dim3((kWgFirst + 2 * kWgBig + kWgLast) / 64), dim3(1024), 0, s,
                       part1, L.wg.blocks, L.wgs.blocks, d_grad);
}

static pisoc_status read_loss(hipStream_t s, const double* loss_dev, double scale, double* h_loss) {
    if (hipGetLastError() != hipSuccess) return PISOC_ERR_HIP;
    if (h_loss) {
        double l = 0.0;
        if (hipMemcpyAsync(&l, loss_dev, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return PISOC_ERR_HIP;
        *h_loss = l * scale;
    }
    return PISOC_OK;
}

pisoc_status pisoc_net_grad(int32_t n, int32_t batch, const float* d_w, const float* d_x,
                            const float* d_t, float* d_grad, double* h_loss, void* d_ws,
                            size_t ws_bytes, void* stream) {
    if (!net_shape_ok(n, batch) || !d_w || !d_x || !d_t || !d_grad) return PISOC_ERR_INVALID;
    NetWs L = net_layout(n, batch);
    if (!d_ws || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* ws = reinterpret_cast<char*>(d_ws);
    const size_t cells = (size_t)batch * n * n * n;
    grad_forward(s, L, ws, n, batch, d_w, d_x);
    // loss and output gradient
    double* lpart = reinterpret_cast<double*>(ws + L.lpart);
    hipLaunchKernelGGL(k_mse, dim3(L.lblocks), dim3(256), 0, s, reinterpret_cast<const float*>(ws + L.y),
                       d_t, cells, (float)(2.0 / (double)cells),
                       reinterpret_cast<uint16_t*>(ws + L.dy), lpart);
    double* loss_dev = lpart + L.lblocks;
    sum_partials(s, lpart, L.lblocks, loss_dev);
    grad_backward(s, L, ws, n, batch, d_grad);
    return read_loss(s, loss_dev, 1.0 / (double)cells, h_loss);
}

pisoc_status pisoc_net_grad_residual(int32_t n, int32_t batch, const float* d_w, const float* d_x,
                                     const double* d_b, const double* d_diag, const double* d_wk,
                                     float* d_grad, double* h_loss, void* d_ws, size_t ws_bytes,
                                     void* stream) {
    if (!net_shape_ok(n, batch) || !d_w || !d_x || !d_b || !d_diag || !d_wk || !d_grad)
        return PISOC_ERR_INVALID;
    NetWs L = net_layout(n, batch);
    if (!d_ws || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(d_ws) % 256) != 0)
        return PISOC_ERR_WORKSPACE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* ws = reinterpret_cast<char*>(d_ws);
    grad_forward(s, L, ws, n, batch, d_w, d_x);
    const double h = 2.0 * M_PI / n, inv_h2 = 1.0 / (h * h);
    double* u = reinterpret_cast<double*>(ws + L.ru);
    double* rpart = reinterpret_cast<double*>(ws + L.rpart);
    double* coef = reinterpret_cast<double*>(ws + L.rcoef);
    double* loss_dev = reinterpret_cast<double*>(ws + L.lpart);
    const dim3 GR(kResBlocks, batch), B(256);
    hipLaunchKernelGGL(k_res_u, GR, B, 0, s, n, inv_h2, d_b, d_diag, d_wk,
                       reinterpret_cast<const float*>(ws + L.y), u, rpart);
    hipLaunchKernelGGL(k_res_coef, dim3(batch), B, 0, s, rpart, coef);
    hipLaunchKernelGGL(k_res_dy, GR, B, 0, s, n, inv_h2, d_b, d_diag, d_wk, u, coef,
                       reinterpret_cast<uint16_t*>(ws + L.dy), loss_dev);
    grad_backward(s, L, ws, n, batch, d_grad);
    return read_loss(s, loss_dev, 1.0, h_loss);
}

pisoc_status pisoc_net_adam(int32_t nw, float* d_w, const float* d_g, float* d_m, float* d_v,
                            int32_t step, float lr, float beta1, float beta2, float eps,
                            void* stream) {
    if (nw < 1 || !d_w || !d_g || !d_m || !d_v || step < 1) return PISOC_ERR_INVALID;
    const float c1 = 1.f - std::pow(beta1, (float)step), c2 = 1.f - std::pow(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((nw + 255) / 256), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), nw, d_w, d_g, d_m, d_v, lr, beta1,
                       beta2, eps, c1, c2);
    return hipGetLastError() == hipSuccess ? PISOC_OK : PISOC_ERR_HIP;
}

}  // extern "C"
