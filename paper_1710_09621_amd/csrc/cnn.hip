// Learned preconditioner: a 4-layer convolutional network with 3^4 kernels acting on the odd-site
// half field of the even-odd system, one s-slice at a time with weights shared over s.
//
// Activations are rows of 32 channels (complex-as-real spin x colour = 24, padded to 32 for the
// matrix cores), row = cb * Ns + s.  The 4D geometry is the checkerboard-compressed lattice
// (xh, y, z, t) with periodic wrap.  Every layer is an implicit GEMM
//     Y[row][n] = b[n] + sum_{tap < 81} sum_{k < 32} X[nbr(row, tap)][k] W[tap][n][k]
// on v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32 accumulation).  The weight gradient is a GEMM
// whose reduction runs over rows.
//
// BF16 operands lie in memory in the order in which the lanes of a wave hold them, units of 16 bytes, so that a load
// instruction reads 1 KB (Ns = 8: pieces of 128 bytes) lane by lane: with the natural order, neighbouring lanes 64
// bytes apart, the L1 needed two accesses for every 64 bytes and bound the convolutions.
//   rows:    per site and group of G = min(16, Ns) slices  [k block of 8 channels][s][8 channels]   (row_unit)
//   sites:   per site  [half of the channels][group of 8 slices][channel % 16][8 slices]           (site_unit)
//   weights: per tap   [half of n][k block][n % 16][8 k]
// FP32 rows (network output, target, gradients) are plain [row][32].
#include <algorithm>

#include "eofa_int.h"
#include "cnn.h"

namespace eofa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short bf16_bits(float f) {
    // round to nearest even
    unsigned u = __builtin_bit_cast(unsigned, f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)(u >> 16);  // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_float(unsigned short h) { return __builtin_bit_cast(float, (unsigned)h << 16); }

// cb-compressed coordinates of a 4D checkerboard index
struct CbGeom {
    int Lxh, Ly, Lz, Lt, Ns;
    int Vh;
};

// unit of the channels 8 kb .. 8 kb + 7 of slice s
__device__ __forceinline__ size_t row_unit(size_t cb, int s, int kb, int Ns) {
    const int G = Ns < 16 ? Ns : 16;
    return cb * Ns * 4 + (s / G) * G * 4 + kb * G + s % G;
}
// unit of the slices s8 .. s8 + 7 (s8 % 8 == 0) of channel c
__device__ __forceinline__ size_t site_unit(size_t cb, int s8, int c, int Ns) {
    return cb * Ns * 4 + ((c >> 4) * (Ns >> 3) + (s8 >> 3)) * 16 + (c & 15);
}
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// sites in y and z of a weight-gradient K step (32 rows at one xh)
__host__ __device__ constexpr int wgrad_yg(int Ns) { return Ns <= 16 ? 2 : 1; }
__host__ __device__ constexpr int wgrad_zg(int Ns) { return Ns == 8 ? 2 : 1; }

// -------------------------------------------------------------------- forward conv
// X: bf16 rows; W: bf16 weights; bias [32] f32 (may be null); Y: bf16 rows or f32 rows.  The weights are the first
// operand, so that a lane's four results are consecutive channels of one row.
// The 16 rows of a matrix-core tile are slices of one site (Ns = 16; Ns = 8: two sites in y; Ns = 32: one half of the
// slices), so a tile's A operand is 1 KB of consecutive memory and the tile of x + dx is the operand of the tap dx at x.
// A wave owns LEN tiles along xh (a whole line: WHOLE, else a segment) on NL neighbouring lines in y, reads the
// operands of one (dt, dz, dy) group of taps per line once (LEN loads, LEN + 2 for a segment) and uses each for the
// three dx: 6 LEN NL MFMAs.  The next group's operands and weights are requested before this group's MFMAs.  Taps are
// added in order, 0 .. 80.  No LDS halo: the operands come from L1 and L2; MFMAs and L1 accesses (14 KB per 48 MFMAs
// of 16 cycles at LEN = 8) are close to balance.  16^3 x 32, Ns = 16: 160 us a layer (174 GFLOP), against 317 us with
// a 4 x 4 x 2 x 2 block and its halo staged in LDS, where every tap re-read its operands.
struct ConvJobs {
    int nx, ny, nz, ns;  // segments, groups of NL lines, z extent, halves of the slices
    int total;
};

template <int LEN, int NL, bool WHOLE, bool OUT_F32>
__global__ __launch_bounds__(256, 2) void k_conv(const unsigned short* __restrict__ X, const unsigned short* __restrict__ W,
                                              const float* __restrict__ bias, void* __restrict__ Y, CbGeom g, ConvJobs jobs,
                                              int relu) {
    constexpr int NF = WHOLE ? LEN : LEN + 2;
    const int lane = threadIdx.x & 63, li = lane & 15, kb = lane >> 4;
    int b = blockIdx.x;
    {   // hardware dispatches workgroup b to XCD b % 8: every XCD takes one contiguous range of the lattice
        const int n = gridDim.x, x = b & 7, i = b >> 3, q = n >> 3, m = n & 7;
        b = x * q + (x < m ? x : m) + i;
    }
    int job = b * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (job >= jobs.total) return;
    const int YT = g.Ns == 8 ? 2 : 1, ny = g.Ly / YT;
    const int js = job % jobs.ns; job /= jobs.ns;
    const int jx = job % jobs.nx; job /= jobs.nx;
    const int jy = job % jobs.ny; job /= jobs.ny;
    const int z = job % jobs.nz, t = job / jobs.nz;
    // the last segment and the last group of lines may overlap the one before (the same values are written twice)
    const int x0 = WHOLE ? 0 : min(jx * LEN, g.Lxh - LEN), y0 = min(jy * NL, ny - NL) * YT;
    const int iy = g.Ns == 8 ? li >> 3 : 0, s = g.Ns == 8 ? li & 7 : js * 16 + li;
    auto wrap = [](int v, int L) { return v < 0 ? v + L : v >= L ? v - L : v; };
    const size_t sx = (size_t)g.Ns * 32;  // one site
    const size_t lo = row_unit(0, s, kb, g.Ns) * 8;
    // operands of the (dt, dz, dy) group tq: f[line][j], xh = x0 + j (WHOLE) or x0 - 1 + j
    auto load_group = [&](int tq, bf16x8 (*f)[NF]) {
        const int dy = tq % 3 - 1, dz = (tq / 3) % 3 - 1, dt = tq / 9 - 1;
        const size_t zt = (size_t)g.Lxh * g.Ly * (wrap(z + dz, g.Lz) + (size_t)g.Lz * wrap(t + dt, g.Lt));
#pragma unroll
        for (int l = 0; l < NL; l++) {
            const unsigned short* p =
                X + (zt + (size_t)g.Lxh * wrap(y0 + l * YT + iy + dy, g.Ly)) * sx + lo;
            if constexpr (WHOLE) {
#pragma unroll
                for (int j = 0; j < LEN; j++) f[l][j] = *(const bf16x8*)(p + j * sx);
            } else {
                f[l][0] = *(const bf16x8*)(p + (x0 == 0 ? g.Lxh - 1 : x0 - 1) * sx);
#pragma unroll
                for (int j = 0; j < LEN; j++) f[l][j + 1] = *(const bf16x8*)(p + (x0 + j) * sx);
                f[l][LEN + 1] = *(const bf16x8*)(p + (x0 + LEN == g.Lxh ? 0 : x0 + LEN) * sx);
            }
        }
    };
    const unsigned short* wl = W + lane * 8;
    auto load_w = [&](int tq, bf16x8 (*w)[2]) {
#pragma unroll
        for (int d = 0; d < 3; d++) {
            w[d][0] = *(const bf16x8*)(wl + (size_t)(3 * tq + d) * 1024);
            w[d][1] = *(const bf16x8*)(wl + (size_t)(3 * tq + d) * 1024 + 512);
        }
    };
    f32x4 acc[NL][LEN][2];
#pragma unroll
    for (int l = 0; l < NL; l++)
#pragma unroll
        for (int j = 0; j < LEN; j++) acc[l][j][0] = acc[l][j][1] = {0, 0, 0, 0};
    bf16x8 f[NL][NF], fn[NL][NF], w[3][2], wn[3][2];
    load_group(0, f);
    load_w(0, w);
    for (int tq = 0; tq < 27; tq++) {
        const int tn = tq < 26 ? tq + 1 : tq;
        load_group(tn, fn);
        load_w(tn, wn);
        __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the MFMAs
#pragma unroll
        for (int d = 0; d < 3; d++)
#pragma unroll
            for (int l = 0; l < NL; l++)
#pragma unroll
                for (int j = 0; j < LEN; j++) {
                    const bf16x8 a = f[l][WHOLE ? (j + d - 1 + LEN) % LEN : j + d];
                    acc[l][j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[d][0], a, acc[l][j][0], 0, 0, 0);
                    acc[l][j][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[d][1], a, acc[l][j][1], 0, 0, 0);
                }
#pragma unroll
        for (int l = 0; l < NL; l++)
#pragma unroll
            for (int j = 0; j < NF; j++) f[l][j] = fn[l][j];
#pragma unroll
        for (int d = 0; d < 3; d++) {
            w[d][0] = wn[d][0];
            w[d][1] = wn[d][1];
        }
    }
    // D layout: lane holds channels 16 h + 4 kb .. + 3 of row li of the tile
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int n = h * 16 + kb * 4;
        const f32x4 bn = bias ? *(const f32x4*)(bias + n) : f32x4{0, 0, 0, 0};
#pragma unroll
        for (int l = 0; l < NL; l++) {
            const size_t c0 = x0 + (size_t)g.Lxh * (y0 + l * YT + iy + (size_t)g.Ly * (z + (size_t)g.Lz * t));
#pragma unroll
            for (int j = 0; j < LEN; j++) {
                f32x4 v = acc[l][j][h] + bn;
                if (relu)
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        if (v[i] < 0.0f) v[i] = 0.0f;
                if constexpr (OUT_F32) {
                    *(f32x4*)((float*)Y + ((c0 + j) * g.Ns + s) * 32 + n) = v;
                } else {
                    const u16x4 o = {bf16_bits(v[0]), bf16_bits(v[1]), bf16_bits(v[2]), bf16_bits(v[3])};
                    *(u16x4*)((unsigned short*)Y + row_unit(c0 + j, s, n >> 3, g.Ns) * 8 + (n & 7)) = o;
                }
            }
        }
    }
}

// -------------------------------------------------------------------- weight gradient
// dW[tap][n][k] = sum_rows dY[row][n] X[nbr(row, tap)][k] from the site-transposed dYT and XT (8 consecutive s of one
// channel are one 16-byte operand: Ns % 8 == 0).  A K step of 32 rows is a column of YG x ZG sites at one xh with all
// or 32 of their slices, and a wave walks such columns along xh for the nine taps (dy, dx) of its (dt, dz): it keeps the
// X operands of xh - 1, xh and xh + 1 at y - 1, y and y + 1 in registers, so a step reads three new X columns and one
// dY column (8 KB, in full cache lines) for 36 MFMAs.  The waves of a workgroup take different lines of its chunk and
// are added up in LDS; part[chunk][tap][32][32] are summed by k_wgrad_reduce.  What the L1 delivers in a step (64 B per
// cycle and CU) takes about as long as its MFMAs.  16^3 x 32, Ns = 16 (173 GFLOP): 175 us a layer; with one (dt, dz, dy)
// per wave, 4 KB for 12 MFMAs, 223 us; with operands gathered per tap from channel-major copies 1199 us.
template <int NS>
__global__ __launch_bounds__(256, 2) void k_conv_wgrad(const unsigned short* __restrict__ dYT,
                                                       const unsigned short* __restrict__ XT, float* __restrict__ part,
                                                       CbGeom g, int nlines) {
    constexpr int YG = wgrad_yg(NS), ZG = wgrad_zg(NS), STEP = 32 * NS;
    __shared__ float sum[36 * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, chunk = blockIdx.x;
    const int li = lane & 15, kb = lane >> 4;
    const int dz = (int)blockIdx.y % 3 - 1, dt = (int)blockIdx.y / 3 - 1;
    // rows of this lane's k block: site (iy, iz) of the column, slices s8 .. s8 + 7
    const int iy = NS == 8 ? kb & 1 : NS == 16 ? kb >> 1 : 0, iz = NS == 8 ? kb >> 1 : 0;
    const int s8 = NS == 16 ? (kb & 1) * 8 : NS == 32 ? kb * 8 : 0;
    const int ny = g.Ly / YG, nz = g.Lz / ZG;
    auto wrap = [](int v, int L) { return v < 0 ? v + L : v >= L ? v - L : v; };
    auto ld = [](const unsigned short* q, bf16x8 f[2]) {
        f[0] = *(const bf16x8*)q;
        f[1] = *(const bf16x8*)(q + 16 * NS);  // the other half of the channels
    };
    f32x4 acc[3][3][2][2];  // [dy][dx][n tile][k tile]
#pragma unroll
    for (int d = 0; d < 9; d++)
#pragma unroll
        for (int k = 0; k < 4; k++) acc[d / 3][d % 3][k >> 1][k & 1] = {0, 0, 0, 0};
    // Chunks of one XCD (workgroup b runs on XCD b % 8) take the lines of one contiguous range in turn, so that what
    // runs at one time reads neighbouring lines: in ranges of their own, half of the L2 accesses missed.
    const int nx = gridDim.x % 8 == 0 ? 8 : 1, xcd = chunk % nx, turn = gridDim.x / nx;
    const int l0 = (int)((long)nlines * xcd / nx), l1 = (int)((long)nlines * (xcd + 1) / nx);
    for (int l = l0 + chunk / nx * 4 + wave; l < l1; l += turn * 4) {
        const int yg = l % ny, r = l / ny, zg = r % nz, t = r / nz;
        const int y = yg * YG + iy, z = zg * ZG + iz;
        const size_t ca = (size_t)g.Lxh * (y + (size_t)g.Ly * (z + (size_t)g.Lz * t));
        const size_t cz = (size_t)g.Lz * wrap(t + dt, g.Lt) + wrap(z + dz, g.Lz);
        const unsigned short* pa = dYT + site_unit(ca, s8, li, NS) * 8;
        const unsigned short* px[3];
#pragma unroll
        for (int e = 0; e < 3; e++)
            px[e] = XT + site_unit((size_t)g.Lxh * (wrap(y + e - 1, g.Ly) + (size_t)g.Ly * cz), s8, li, NS) * 8;
        bf16x8 f0[3][2], f1[3][2], f2[3][2], a[2];
#pragma unroll
        for (int e = 0; e < 3; e++) {
            ld(px[e] + (size_t)(g.Lxh - 1) * STEP, f0[e]);
            ld(px[e], f1[e]);
            ld(px[e] + (size_t)(1 == g.Lxh ? 0 : 1) * STEP, f2[e]);
        }
        ld(pa, a);
        auto mfma = [&](int d, const bf16x8 f[3][2]) {
#pragma unroll
            for (int e = 0; e < 3; e++)
#pragma unroll
                for (int n = 0; n < 2; n++)
#pragma unroll
                    for (int k = 0; k < 2; k++)
                        acc[e][d][n][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[n], f[e][k], acc[e][d][n][k], 0, 0, 0);
        };
        // one step at x: the operands of x - 1 are used first and give way to those of x + 2 (past the end: the line's
        // first ones), which the next step needs last
        auto step = [&](int x, bf16x8 fm[3][2], const bf16x8 fz[3][2], const bf16x8 fp[3][2]) {
            bf16x8 an[2];
            const int xa = x + 1 < g.Lxh ? x + 1 : 0, xf = xa + 1 < g.Lxh ? xa + 1 : 0;
            ld(pa + (size_t)xa * STEP, an);
            mfma(0, fm);
#pragma unroll
            for (int e = 0; e < 3; e++) ld(px[e] + (size_t)xf * STEP, fm[e]);
            __builtin_amdgcn_sched_barrier(0);
            mfma(1, fz);
            mfma(2, fp);
            a[0] = an[0];
            a[1] = an[1];
        };
        int x = 0;
        for (; x + 2 < g.Lxh; x += 3) {
            step(x, f0, f1, f2);
            step(x + 1, f1, f2, f0);
            step(x + 2, f2, f0, f1);
        }
        if (x < g.Lxh) step(x, f0, f1, f2);
        if (x + 1 < g.Lxh) step(x + 1, f1, f2, f0);
    }
    // the four waves' sums in order; the last one writes them out
    for (int w = 0; w < 4; w++) {
        if (wave == w) {
#pragma unroll
            for (int q = 0; q < 36; q++)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int e = q / 12, d = q / 4 % 3, n = q / 2 % 2, k = q % 2;
                    float* c = sum + q * 256 + j * 64 + lane;
                    const float v = w > 0 ? *c + acc[e][d][n][k][j] : acc[e][d][n][k][j];
                    if (w < 3) *c = v;
                    else part[((size_t)chunk * 81 + blockIdx.y * 9 + e * 3 + d) * 1024 + (n * 16 + kb * 4 + j) * 32 + k * 16 + li] = v;
                }
        }
        __syncthreads();
    }
}

// sum over chunks (fixed order, four partial sums) -> g[tap][n][k], masked to the live channels
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* __restrict__ part, int nchunk, float* __restrict__ gw,
                                                      int cin, int cout) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= 81 * 1024) return;
    const int n = (i / 32) % 32, k = i % 32;
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int c = 0;
    for (; c + 3 < nchunk; c += 4)
#pragma unroll
        for (int q = 0; q < 4; q++) s[q] += part[(size_t)(c + q) * 81 * 1024 + i];
    for (; c < nchunk; c++) s[0] += part[(size_t)c * 81 * 1024 + i];
    gw[i] = (n < cout && k < cin) ? (s[0] + s[1]) + (s[2] + s[3]) : 0.0f;
}

// One pass over the output gradient of a layer, d = dY (dY where act > 0 with ReLU): its BF16 rows for the
// backward-data convolution (rows_out, may be null), its site-transposed BF16 copy for the weight gradient, and the
// sums of d over rows in FP64 for the bias gradient, part[block][32].  64 rows per step: four threads a row.
// Bound by memory; as four kernels (ReLU, conversion, transposition, sums) it took 310 us on 1 M rows, now 41 us and 10 us for the last sum.
constexpr int PREP_BLOCKS = 1024;
__global__ __launch_bounds__(256) void k_dy_prep(const float* __restrict__ dY, const unsigned short* __restrict__ act,
                                                 unsigned short* __restrict__ rows_out, unsigned short* __restrict__ dYT,
                                                 double* __restrict__ part, int rows, int Ns) {
    __shared__ union {
        unsigned short tile[32][72];  // 16-byte rows of 8 slices
        double sum[256][8];
    } sh;
    const int row = threadIdx.x >> 2, q = threadIdx.x & 3, c = threadIdx.x >> 3, g8 = threadIdx.x & 7;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int r0 = blockIdx.x * 64; r0 < rows; r0 += gridDim.x * 64) {  // rows is a multiple of 64
        const size_t e = (size_t)(r0 + row) * 32 + q * 8;
        const int cr = (r0 + row) / Ns;
        const size_t u = row_unit(cr, r0 + row - cr * Ns, q, Ns) * 8;
        const f32x4 v0 = *(const f32x4*)(dY + e), v1 = *(const f32x4*)(dY + e + 4);
        float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
        if (act) {
            const u16x8 a = *(const u16x8*)(act + u);
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (bf16_float(a[k]) <= 0.0f) v[k] = 0.0f;
        }
        u16x8 h;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            acc[k] += v[k];
            h[k] = bf16_bits(v[k]);
            sh.tile[q * 8 + k][row] = h[k];
        }
        if (rows_out) *(u16x8*)(rows_out + u) = h;
        __syncthreads();
        const int r8 = r0 + g8 * 8, cb = r8 / Ns;
        *(u16x8*)(dYT + site_unit(cb, r8 - cb * Ns, c, Ns) * 8) = *(const u16x8*)&sh.tile[c][g8 * 8];
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 8; k++) sh.sum[threadIdx.x][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 32) {  // channel n: the 64 threads of its quarter, in order
        const int n = threadIdx.x;
        double t = 0.0;
        for (int r = 0; r < 64; r++) t += sh.sum[r * 4 + (n >> 3)][n & 7];
        part[(size_t)blockIdx.x * 32 + n] = t;
    }
}
// bias gradient: the block partials in a fixed order, 32 lanes per channel's share
__global__ __launch_bounds__(1024) void k_bgrad_fin(const double* __restrict__ part, int nb, float* __restrict__ gb, int cout) {
    __shared__ double red[32][33];
    const int n = threadIdx.x & 31, p = threadIdx.x >> 5;
    double t = 0.0;
    for (int b = p; b < nb; b += 32) t += part[(size_t)b * 32 + n];
    red[p][n] = t;
    __syncthreads();
    if (p == 0) {
        t = 0.0;
        for (int k = 0; k < 32; k++) t += red[k][n];
        gb[n] = (n < cout) ? (float)t : 0.0f;
    }
}

// -------------------------------------------------------------------- elementwise helpers
// bf16 rows -> bf16 sites, 64 rows per workgroup through LDS (16-byte reads and writes)
__global__ __launch_bounds__(256) void k_rows_to_site(const unsigned short* __restrict__ in,
                                                      unsigned short* __restrict__ out, int Ns) {
    __shared__ unsigned short tile[32][72];
    // 64 rows are 256 consecutive units: thread -> (row, k block) in the order of the units
    const int G = Ns < 16 ? Ns : 16, blk = threadIdx.x / (4 * G), w = threadIdx.x % (4 * G), q = w / G, row = blk * G + w % G;
    const int c = threadIdx.x >> 3, g8 = threadIdx.x & 7;
    const size_t r0 = (size_t)blockIdx.x * 64;
    const u16x8 v = *(const u16x8*)(in + r0 * 32 + threadIdx.x * 8);
#pragma unroll
    for (int k = 0; k < 8; k++) tile[q * 8 + k][row] = v[k];
    __syncthreads();
    const size_t r8 = r0 + g8 * 8, cb = r8 / Ns;
    *(u16x8*)(out + site_unit(cb, (int)(r8 - cb * Ns), c, Ns) * 8) = *(const u16x8*)&tile[c][g8 * 8];
}

// bf16 copies of one layer's weights [81][32 n][32 k] in the order of the lanes: the layer itself, and for the
// backward-data convolution Wt[tap][k][n] = W[80 - tap][n][k]
__global__ __launch_bounds__(256) void k_w_pack(const float* __restrict__ w, unsigned short* __restrict__ wb,
                                                unsigned short* __restrict__ wt) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= 81 * 1024) return;
    const int tap = i / 1024, e = i % 1024, kk = e & 7, n = (e >> 9) * 16 + ((e >> 3) & 15), k = ((e >> 7) & 3) * 8 + kk;
    wb[i] = bf16_bits(w[(size_t)tap * 1024 + n * 32 + k]);
    wt[i] = bf16_bits(w[(size_t)(80 - tap) * 1024 + k * 32 + n]);
}

// Adam on the FP32 master parameters
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ gsum, float* __restrict__ m,
                                              float* __restrict__ v, size_t n, float lr, float b1, float b2, float eps,
                                              float c1, float c2, float gscale) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float gi = gsum[i] * gscale;
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// half field [cb][12][Ns] (complex double) -> bf16 rows scaled by sc (24 live channels); a thread writes one unit
__global__ __launch_bounds__(256) void k_half_to_rows(const cd* __restrict__ h, unsigned short* __restrict__ X, int Vh,
                                                      int Ns, const double* __restrict__ scale_ptr, int inv) {
    const double sc = inv ? 1.0 / sqrt(*scale_ptr) : *scale_ptr;
    const int G = Ns < 16 ? Ns : 16, per = 4 * G;
    const size_t n = (size_t)Vh * Ns * 4;
    for (size_t u = (size_t)blockIdx.x * 256 + threadIdx.x; u < n; u += (size_t)gridDim.x * 256) {
        const size_t grp = u / per, cb = grp / (Ns / G);
        const int e = (int)(u - grp * per), kb = e / G, s = (int)(grp - cb * (Ns / G)) * G + e % G;
        u16x8 o = {0, 0, 0, 0, 0, 0, 0, 0};
        if (kb < 3)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const cd z = h[(cb * 12 + kb * 4 + j) * Ns + s];
                o[2 * j] = bf16_bits((float)(sc * z.x));
                o[2 * j + 1] = bf16_bits((float)(sc * z.y));
            }
        *(u16x8*)(X + u * 8) = o;
    }
}

// rows [row][32] f32 -> half field (complex double) times sqrt(*scale) (the norm of the network input)
__global__ __launch_bounds__(256) void k_rows_to_half(const float* __restrict__ Y, cd* __restrict__ h, int Vh, int Ns,
                                                      const double* __restrict__ scale_ptr) {
    const double sc = sqrt(*scale_ptr);
    const size_t n = (size_t)Vh * 12 * Ns;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const int s = (int)(i % Ns);
        const int j = (int)((i / Ns) % 12);
        const size_t cb = i / ((size_t)12 * Ns);
        const size_t row = cb * Ns + s;
        h[i] = {sc * Y[row * 32 + 2 * j], sc * Y[row * 32 + 2 * j + 1]};
    }
}

// dY = (Y - T) * w for the MSE loss; also the partial sums of |Y - T|^2 (T: target rows in f32)
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ Y, const float* __restrict__ T, float* __restrict__ dY,
                                             size_t n, float w, Red red) {
    double s = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float d = Y[i] - T[i];
        dY[i] = d * w;
        s += (double)d * d;
    }
    __shared__ double lds[4];
    finish_sum(red, block_sum256(s, lds));
}

// half field -> f32 rows scaled by 1/sqrt(*scale_ptr) (targets)
__global__ __launch_bounds__(256) void k_half_to_rows_f32(const cd* __restrict__ h, float* __restrict__ T, int Vh, int Ns,
                                                          const double* __restrict__ scale_ptr) {
    const double sc = 1.0 / sqrt(*scale_ptr);
    const size_t n = (size_t)Vh * Ns * 32;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const int c = (int)(i % 32);
        const size_t row = i / 32;
        const int s = (int)(row % Ns);
        const size_t cb = row / Ns;
        float v = 0.0f;
        if (c < 24) {
            const cd z = h[(cb * 12 + (c >> 1)) * Ns + s];
            v = (float)(sc * ((c & 1) ? z.y : z.x));
        }
        T[i] = v;
    }
}

// ==================================================================== launchers
static inline int grid_for(size_t n) {
    size_t b = (n + 255) / 256;
    return (int)(b > 4096 ? 4096 : (b ? b : 1));
}

static CbGeom cbg(const Geom& g, int Ns) { return CbGeom{g.Lxh, g.Ly, g.Lz, g.Lt, Ns, g.Vh}; }


template <int LEN, int NL, bool WHOLE>
static hipError_t conv_launch(const unsigned short* X, const unsigned short* W, const float* bias, void* Y, bool out_f32,
                              const CbGeom& g, int relu, hipStream_t st) {
    const int YT = g.Ns == 8 ? 2 : 1, ny = g.Ly / YT;
    ConvJobs j{WHOLE ? 1 : (g.Lxh + LEN - 1) / LEN, (ny + NL - 1) / NL, g.Lz, g.Ns == 32 ? 2 : 1, 0};
    j.total = j.nx * j.ny * j.nz * j.ns * g.Lt;
    const int wpb = j.total < 1024 ? 1 : 4;  // waves per workgroup: a few waves are spread over the CUs
    const dim3 grid((j.total + wpb - 1) / wpb), block(64 * wpb);
    if (out_f32) hipLaunchKernelGGL((k_conv<LEN, NL, WHOLE, true>), grid, block, 0, st, X, W, bias, Y, g, j, relu);
    else hipLaunchKernelGGL((k_conv<LEN, NL, WHOLE, false>), grid, block, 0, st, X, W, bias, Y, g, j, relu);
    return hipGetLastError();
}

// Tiles per wave by rule: whole lines up to 8 sites, else segments of equal length (5 .. 8); short lines are taken
// 2 or 4 at a time, as far as the y extent goes, so that the weights of a group serve up to 8 tiles.
hipError_t cnn_conv_fwd(const unsigned short* X, const unsigned short* W, const float* bias, void* Y, bool out_f32,
                        const Geom& g, int Ns, int relu, hipStream_t st) {
    if (Ns != 8 && Ns != 16 && Ns != 32) return hipErrorInvalidValue;
    const CbGeom c = cbg(g, Ns);
    // lines taken together: while that leaves two waves per SIMD
    const int lines = c.Ly / (Ns == 8 ? 2 : 1) * c.Lz * c.Lt * (Ns == 32 ? 2 : 1);
    const int ny = std::min(c.Ly / (Ns == 8 ? 2 : 1), std::max(1, lines / 2048));
#define CONV(L, N, WH) return conv_launch<L, N, WH>(X, W, bias, Y, out_f32, c, relu, st)
    switch (c.Lxh) {
    case 1: if (ny >= 4) CONV(1, 4, true); else if (ny >= 2) CONV(1, 2, true); else CONV(1, 1, true);
    case 2: if (ny >= 4) CONV(2, 4, true); else if (ny >= 2) CONV(2, 2, true); else CONV(2, 1, true);
    case 3: if (ny >= 2) CONV(3, 2, true); else CONV(3, 1, true);
    case 4: if (ny >= 2) CONV(4, 2, true); else CONV(4, 1, true);
    case 5: CONV(5, 1, true);
    case 6: CONV(6, 1, true);
    case 7: CONV(7, 1, true);
    case 8: CONV(8, 1, true);
    }
    const int nseg = (c.Lxh + 7) / 8;
    switch ((c.Lxh + nseg - 1) / nseg) {
    case 5: CONV(5, 1, false);
    case 6: CONV(6, 1, false);
    case 7: CONV(7, 1, false);
    default: CONV(8, 1, false);
    }
#undef CONV
}

// chunks of the weight gradient: all their workgroups (9 per chunk, four waves each) fit the chip at once at two per
// CU, and a multiple of 8 keeps the nine workgroups of a chunk on one XCD (workgroup b runs on XCD b % 8)
constexpr int WGRAD_CHUNKS = 56;
static int wgrad_lines(const Geom& g, int Ns) { return g.Ly / wgrad_yg(Ns) * (g.Lz / wgrad_zg(Ns)) * g.Lt; }
int cnn_wgrad_chunks(const Geom& g, int Ns) {
    const int n = std::min((wgrad_lines(g, Ns) + 3) / 4, WGRAD_CHUNKS);
    return n < 8 ? n : n / 8 * 8;
}

hipError_t cnn_wgrad(const unsigned short* dYT, const unsigned short* XT, float* part, float* gw, const Geom& g, int Ns,
                     int cin, int cout, hipStream_t st) {
    const int nlines = wgrad_lines(g, Ns), nchunk = cnn_wgrad_chunks(g, Ns);
    const dim3 grid(nchunk, 9);
    switch (Ns) {
    case 8: hipLaunchKernelGGL(k_conv_wgrad<8>, grid, dim3(256), 0, st, dYT, XT, part, cbg(g, Ns), nlines); break;
    case 16: hipLaunchKernelGGL(k_conv_wgrad<16>, grid, dim3(256), 0, st, dYT, XT, part, cbg(g, Ns), nlines); break;
    case 32: hipLaunchKernelGGL(k_conv_wgrad<32>, grid, dim3(256), 0, st, dYT, XT, part, cbg(g, Ns), nlines); break;
    default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((81 * 1024 + 255) / 256), dim3(256), 0, st, part, nchunk, gw, cin, cout);
    return hipGetLastError();
}

hipError_t cnn_dy_prep(const float* dY, const unsigned short* act, unsigned short* rows_out, unsigned short* dYT,
                       double* part, float* gb, int cout, int rows, int Ns, hipStream_t st) {
    if (rows % 64 || Ns % 8) return hipErrorInvalidValue;
    const int grid = std::min(rows / 64, PREP_BLOCKS);
    hipLaunchKernelGGL(k_dy_prep, dim3(grid), dim3(256), 0, st, dY, act, rows_out, dYT, part, rows, Ns);
    hipLaunchKernelGGL(k_bgrad_fin, dim3(1), dim3(1024), 0, st, part, grid, gb, cout);
    return hipGetLastError();
}

hipError_t cnn_rows_to_site(const unsigned short* in, unsigned short* out, int rows, int Ns, hipStream_t st) {
    if (rows % 64 || Ns % 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rows_to_site, dim3(rows / 64), dim3(256), 0, st, in, out, Ns);
    return hipGetLastError();
}

hipError_t cnn_w_pack(const float* w, unsigned short* wb, unsigned short* wt, hipStream_t st) {
    hipLaunchKernelGGL(k_w_pack, dim3((81 * 1024 + 255) / 256), dim3(256), 0, st, w, wb, wt);
    return hipGetLastError();
}

hipError_t cnn_adam(float* p, const float* g, float* m, float* v, size_t n, float lr, float b1, float b2, float eps,
                    float c1, float c2, float gscale, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1, c2, gscale);
    return hipGetLastError();
}

hipError_t cnn_half_to_rows(const cd* h, unsigned short* X, const Geom& g, int Ns, const double* scale, int inv,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_half_to_rows, dim3(grid_for((size_t)g.Vh * Ns * 4)), dim3(256), 0, st, h, X, g.Vh, Ns, scale, inv);
    return hipGetLastError();
}

hipError_t cnn_half_to_rows_f32(const cd* h, float* T, const Geom& g, int Ns, const double* scale, hipStream_t st) {
    hipLaunchKernelGGL(k_half_to_rows_f32, dim3(grid_for((size_t)g.Vh * Ns * 32)), dim3(256), 0, st, h, T, g.Vh, Ns, scale);
    return hipGetLastError();
}

hipError_t cnn_rows_to_half(const float* Y, cd* h, const Geom& g, int Ns, const double* scale, hipStream_t st) {
    hipLaunchKernelGGL(k_rows_to_half, dim3(grid_for((size_t)g.Vh * 12 * Ns)), dim3(256), 0, st, Y, h, g.Vh, Ns, scale);
    return hipGetLastError();
}

hipError_t cnn_mse(const float* Y, const float* T, float* dY, size_t n, float w, const Red& red, hipStream_t st) {
    const int grid = grid_for(n);
    hipLaunchKernelGGL(k_mse, dim3(grid), dim3(256), 0, st, Y, T, dY, n, w, red);
    return launch_finish(red, (unsigned)grid, st);
}

}  // namespace eofa
