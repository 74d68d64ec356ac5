// Column loads and stores of the hop kernels: cache policy, FP16 columns, reconstruction of scaled columns, canonical
// fields.
#pragma once
#include "eofa_int.h"

namespace eofa {

// Cache policy of the hop's outputs: they are not read again by the same launch, so they bypass the
// caches that hold the re-read neighbour spinors.
template <typename R> __device__ __forceinline__ void st_out(cpx<R>* p, const cpx<R>& v) {
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}
template <typename T> __device__ __forceinline__ void st_raw(T* p, const T& v) { __builtin_nontemporal_store(v, p); }
// The epilogues' site-local inputs (aux, aux2) are read once per launch: nontemporal loads, so that they do not
// displace the re-read neighbour spinors either.
template <typename R> __device__ __forceinline__ cpx<R> ld_once(const cpx<R>* p) {
    return {__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y)};
}

// ---- FP16 storage of a Krylov half field (EOFA_MIXED_FP16): per (cb, s) column the 12 complex
// components as binary16 (re, im) pairs in 3 blocks of 4 (16 bytes, one load per block):
// F[cb][jb < 3][Ns][4 pairs], each column scaled by its own FP32 norm = the largest |real component| of
// its 24 reals, stored after the 12 Vh Ns pairs.  value = norm * half, |half| <= 1.
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));

template <int NS> __device__ __forceinline__ const float* h_norms(const void* f, int Vh) {
    return (const float*)((const h8_t*)f + (size_t)3 * Vh * NS);
}

// NT: nontemporal loads (a column read once per launch)
template <int NS, bool NT = false>
__device__ __forceinline__ void load_h(cpx<float> p[12], const void* __restrict__ f, size_t cb, int s, int Vh) {
    const h8_t* d = (const h8_t*)f + cb * 3 * NS + s;
    const float* np = h_norms<NS>(f, Vh) + cb * NS + s;
    const float n = NT ? __builtin_nontemporal_load(np) : *np;
#pragma unroll
    for (int jb = 0; jb < 3; jb++) {
        const h8_t v = NT ? __builtin_nontemporal_load(d + jb * NS) : d[jb * NS];
#pragma unroll
        for (int k = 0; k < 4; k++) p[4 * jb + k] = {n * (float)v[2 * k], n * (float)v[2 * k + 1]};
    }
}

template <int NS>
__device__ __forceinline__ void store_h(void* __restrict__ f, size_t cb, int s, int Vh, const cpx<float> v[12]) {
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < 12; j++) m = fmaxf(m, fmaxf(fabsf(v[j].x), fabsf(v[j].y)));
    const float inv = m > 0.0f ? 1.0f / m : 0.0f;
    h8_t* d = (h8_t*)f + cb * 3 * NS + s;
#pragma unroll
    for (int jb = 0; jb < 3; jb++) {
        h8_t h;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            h[2 * k] = (_Float16)(v[4 * jb + k].x * inv);
            h[2 * k + 1] = (_Float16)(v[4 * jb + k].y * inv);
        }
        st_raw(d + jb * NS, h);
    }
    st_raw((float*)h_norms<NS>(f, Vh) + cb * NS + s, m);
}

// 12 components of (cb, s) from a field in storage H (FP16 columns) or plain cpx<R>; NT: nontemporal loads
template <int NS, bool H, bool NT = false, typename R>
__device__ __forceinline__ void load_col(cpx<R> p[12], const void* __restrict__ f, size_t cb, int s, int Vh) {
    if constexpr (H) {
        load_h<NS, NT>(p, f, cb, s, Vh);
    } else {
        const cpx<R>* src = (const cpx<R>*)f + cb * 12 * NS + s;
#pragma unroll
        for (int j = 0; j < 12; j++) p[j] = NT ? ld_once(src + j * NS) : src[j * NS];
    }
}

template <int NS, bool H, typename R>
__device__ __forceinline__ void store_col(void* __restrict__ f, size_t cb, int s, int Vh, const cpx<R> v[12]) {
    if constexpr (H) {
        store_h<NS>(f, cb, s, Vh, v);
    } else {
        cpx<R>* dst = (cpx<R>*)f + cb * 12 * NS + s;
#pragma unroll
        for (int j = 0; j < 12; j++) st_out(dst + j * NS, v[j]);
    }
}

// An FP16 column of a field in storage H without its norm (p = raw binary16 values widened) and the norm n.
template <int NS>
__device__ __forceinline__ float load_h_raw(cpx<float> p[12], const void* __restrict__ f, size_t cb, int s, int Vh) {
    const h8_t* d = (const h8_t*)f + cb * 3 * NS + s;
#pragma unroll
    for (int jb = 0; jb < 3; jb++) {
        const h8_t v = d[jb * NS];
#pragma unroll
        for (int k = 0; k < 4; k++) p[4 * jb + k] = {(float)v[2 * k], (float)v[2 * k + 1]};
    }
    return h_norms<NS>(f, Vh)[cb * NS + s];
}

// An FP16 column as loaded: component j is the pair v[j / 4][2 (j % 4)], v[j / 4][2 (j % 4) + 1], times n.
struct HCol { h8_t v[3]; float n; };
template <int NS> __device__ __forceinline__ void load_h_col(HCol& c, const void* __restrict__ f, size_t cb, int s, int Vh) {
    const size_t i = cb * 3 * NS + s;  // one 64-bit offset per column, the same for every field
#pragma unroll
    for (int jb = 0; jb < 3; jb++) c.v[jb] = ((const h8_t*)f)[i + jb * NS];
    const size_t k = cb * NS + s;
    c.n = h_norms<NS>(f, Vh)[k];
}

// project() straight from the binary16 values: a + b as fma(a, 1, b), which the compiler turns into one
// v_fma_mix_f32 on both halves' bits instead of two conversions and an add (the product with 1 is exact, so these are
// the bits of the widened sum).  one: 1.0 in a register that the compiler cannot fold.
// The FP16 hop is bound by vector instructions.  With this and the rotations as operands (add_rotated) at 16^3 x 32,
// Ns = 16, two systems: HM_SITE 100 -> 88 us, HM_SCHUR_W 138 -> 120 us, HM_SCHUR_Q 133 -> 129 us (memory).
template <int MU, int S>
__device__ __forceinline__ void project_hcol(const HCol& c, float one, cpx<float> h[6]) {
    // h_up[k] = up[k] + S (B dn)[k]; the real and imaginary parts of B dn are +- those of one lower component
    auto f = [&](int j, int im) { return (float)c.v[j / 4][2 * (j % 4) + im]; };
    auto add = [&](float a, float b, bool neg) { return __builtin_fmaf(neg ? -b : b, one, a); };
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int dn = 6 + ((MU < 2) ? (k + 3) % 6 : k);  // lower component that meets upper component k
        const bool second = k >= 3;
        if constexpr (MU == 0 || MU == 2) {  // -i dn (both; mu = z: +i on the second spin)
            const bool mi = MU == 0 || !second;  // factor -i, else +i
            h[k].x = add(f(k, 0), f(dn, 1), (S > 0) != mi);
            h[k].y = add(f(k, 1), f(dn, 0), (S > 0) == mi);
        } else {  // mu = y: -dn on the first spin, +dn on the second; mu = t: +dn
            const bool pl = MU == 3 || second;
            h[k].x = add(f(k, 0), f(dn, 0), (S > 0) != pl);
            h[k].y = add(f(k, 1), f(dn, 1), (S > 0) != pl);
        }
    }
}

// reconstruct() of n w: the column norm of an FP16 neighbour folded into the accumulation (one FMA per real
// instead of a multiply on every loaded component and an add)
template <int MU, int S, typename R>
__device__ __forceinline__ void reconstruct_n(cpx<R> acc[12], const cpx<R> w[6], R n) {
    const R sn = S > 0 ? n : -n;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        cpx<R> w0 = w[c], w1 = w[3 + c], t0, t1;  // t = B^dag w
        if constexpr (MU == 0) { t0 = ci(w1); t1 = ci(w0); }
        else if constexpr (MU == 1) { t0 = w1; t1 = cneg(w0); }
        else if constexpr (MU == 2) { t0 = ci(w0); t1 = cneg(ci(w1)); }
        else { t0 = w0; t1 = w1; }
        acc[c].x = fma(n, w0.x, acc[c].x); acc[c].y = fma(n, w0.y, acc[c].y);
        acc[3 + c].x = fma(n, w1.x, acc[3 + c].x); acc[3 + c].y = fma(n, w1.y, acc[3 + c].y);
        acc[6 + c].x = fma(sn, t0.x, acc[6 + c].x); acc[6 + c].y = fma(sn, t0.y, acc[6 + c].y);
        acc[9 + c].x = fma(sn, t1.x, acc[9 + c].x); acc[9 + c].y = fma(sn, t1.y, acc[9 + c].y);
    }
}

// whether the kernel of MODE can write a canonical field
template <int MODE, bool RED> constexpr bool canon_mode() {
    return !RED && (MODE == HM_LIN || MODE == HM_DT || MODE == HM_DW);
}
// canonical index of (s, lex site, j): ((s * V + lex) * 12 + j)
__device__ __forceinline__ void cb_to_lex(const Geom& g, int cb, int par, int& lex) {
    int xh = cb % g.Lxh;
    int r = cb / g.Lxh;
    int y = r % g.Ly; r /= g.Ly;
    int z = r % g.Lz;
    int t = r / g.Lz;
    int x = 2 * xh + ((y + z + t + par) & 1);
    lex = x + g.Lx * (y + g.Ly * (z + g.Lz * t));
}

}  // namespace eofa
