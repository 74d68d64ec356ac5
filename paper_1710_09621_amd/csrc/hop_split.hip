// gfx950 direction-split form of the fused even-odd hop, for lattices whose launch does not fill the chip.
//
// k_hop walks the four directions one after the other in each lane (a fence between them keeps two columns in
// registers), i.e. four dependent memory round trips per launch; on a small lattice, with a few waves per CU,
// those round trips are the whole time of the kernel.  Here a workgroup of four waves owns 64 (site, s) lanes:
// wave mu forms the two link products of direction mu (one round trip for everything the launch reads), hands
// them over in LDS, and wave q then sums the eight terms of spin q in the order of k_hop and applies the epilogue
// to its three colours (the s-operators act on every component by itself).  Every sum has the order of k_hop, so
// the operator is bitwise the same; only the reductions add in another order.  Several systems of a batch run
// side by side (grid y) rather than one after the other.
#include <type_traits>

#include "hop_dev.h"

namespace eofa {

namespace {

// One entry of a site-operator table held in a register: chir_op indexes its tables by s.
template <typename R> struct TabReg {
    R v;
    __device__ __forceinline__ R operator[](int) const { return v; }
};
template <int NS, typename R> struct ChirReg {
    TabReg<R> pre, mid, shf, post, q[ilog2(NS) > 0 ? ilog2(NS) : 1];
};
template <int NS, typename R>
__device__ __forceinline__ void chir_fetch(ChirReg<NS, R>& r, const ChirTab& t, int s) {
    r.pre.v = (R)t.pre[s];
    r.mid.v = (R)t.mid[s];
    r.shf.v = (R)t.shf[s];
    r.post.v = (R)t.post[s];
#pragma unroll
    for (int k = 0; k < ilog2(NS); k++) r.q[k].v = (R)t.q[k][s];
}

// site_op on the three colours of one spin of the upper (up) or lower half
template <int NS, bool DAG, typename R>
__device__ __forceinline__ void site_op_spin(cpx<R> v[3], const ChirReg<NS, R>& t, bool up, int s, int lane) {
    constexpr int SU = DAG ? +1 : -1, ORD = DAG ? 1 : 0;
    if (up) chir_op<NS, SU, ORD, 3>(v, t, s, lane);
    else chir_op<NS, -SU, ORD, 3>(v, t, s, lane);
}

// Neighbours of cb in direction mu (uniform over the wave): nf = x + mu, nk = x - mu.
__device__ __forceinline__ void neighbours_mu(const Geom& g, int cb, int par, int mu, int& nf, int& nk) {
    const int xh = cb % g.Lxh;
    int r = cb / g.Lxh;
    const int y = r % g.Ly;
    r /= g.Ly;
    const int z = r % g.Lz, t = r / g.Lz;
    if (mu == 0) {
        const int odd = (y + z + t + par) & 1;  // x = 2 xh + odd
        nf = cb - xh + (odd ? (xh + 1 == g.Lxh ? 0 : xh + 1) : xh);
        nk = cb - xh + (odd ? xh : (xh == 0 ? g.Lxh - 1 : xh - 1));
        return;
    }
    const int st = mu == 1 ? g.Lxh : mu == 2 ? g.Lxh * g.Ly : g.Lxh * g.Ly * g.Lz;
    const int c = mu == 1 ? y : mu == 2 ? z : t, L = mu == 1 ? g.Ly : mu == 2 ? g.Lz : g.Lt;
    nf = c + 1 == L ? cb - (L - 1) * st : cb + st;
    nk = c == 0 ? cb + (L - 1) * st : cb - st;
}

// The half-spinors of direction MU: hf = (1 + SF gamma) projection of pf, hb = (1 - SF gamma) projection of pb.
template <int MU, int SF, typename R>
__device__ __forceinline__ void project2(const cpx<R> pf[12], const cpx<R> pb[12], cpx<R> hf[6], cpx<R> hb[6]) {
    project<MU, SF>(pf, hf);
    project<MU, -SF>(pb, hb);
}

// acc[c] += S (B^dag w)_l, component l of the lower half of reconstruct(), c the colours: w0, w1 the colour
// vectors of the two spins of w (only the one that enters is read).  n: the column norm of FP16 storage (else 1).
template <int MU, bool FMA, typename R>
__device__ __forceinline__ void add_lower(cpx<R> acc[3], const cpx<R> w[3], int l, R n, bool plus) {
    // B^dag w: mu = x: i w_{1-l}; y: w_1 (l = 0), -w_0 (l = 1); z: i w_0 (l = 0), -i w_1 (l = 1); t: w_l
    const bool neg = (MU == 1 || MU == 2) && l == 1;
    const R c = plus != neg ? n : -n;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const cpx<R> t = (MU == 0 || MU == 2) ? ci(w[k]) : w[k];
        if constexpr (FMA) {
            acc[k].x = fma(c, t.x, acc[k].x);
            acc[k].y = fma(c, t.y, acc[k].y);
        } else {
            acc[k] = plus != neg ? cadd(acc[k], t) : csub(acc[k], t);
        }
    }
}

template <int NS, bool H, typename R>
__device__ __forceinline__ void load_spin(cpx<R> v[3], const void* __restrict__ f, size_t cb, int s, int q, int Vh) {
    if constexpr (H) {
        const float n = h_norms<NS>(f, Vh)[cb * NS + s];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const int j = 3 * q + c;
            const _Float16* d = (const _Float16*)((const h8_t*)f + (cb * 3 + (j >> 2)) * NS + s) + 2 * (j & 3);
            v[c] = {n * (float)d[0], n * (float)d[1]};
        }
    } else {
        const cpx<R>* src = (const cpx<R>*)f + (cb * 12 + 3 * q) * NS + s;
#pragma unroll
        for (int c = 0; c < 3; c++) v[c] = src[c * NS];
    }
}

// Stores spin q of a column.  FP16 columns share one norm per column: the four waves exchange their largest
// component through mx (a workgroup barrier).
template <int NS, bool H, typename R>
__device__ __forceinline__ void store_spin(void* __restrict__ f, size_t cb, int s, int q, int Vh, const cpx<R> v[3],
                                           bool valid, float (*mx)[64]) {
    if constexpr (H) {
        const int lane = threadIdx.x & 63;
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < 3; c++) m = fmaxf(m, fmaxf(fabsf(v[c].x), fabsf(v[c].y)));
        mx[q][lane] = m;
        __syncthreads();
        m = fmaxf(fmaxf(mx[0][lane], mx[1][lane]), fmaxf(mx[2][lane], mx[3][lane]));
        const float inv = m > 0.0f ? 1.0f / m : 0.0f;
        if (valid) {
            typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int c = 0; c < 3; c++) {
                const int j = 3 * q + c;
                const h2_t h = {(_Float16)(v[c].x * inv), (_Float16)(v[c].y * inv)};
                *((h2_t*)((h8_t*)f + (cb * 3 + (j >> 2)) * NS + s) + (j & 3)) = h;
            }
            if (q == 0) ((float*)h_norms<NS>(f, Vh))[cb * NS + s] = m;
        }
    } else if (valid) {
        cpx<R>* dst = (cpx<R>*)f + (cb * 12 + 3 * q) * NS + s;
#pragma unroll
        for (int c = 0; c < 3; c++) dst[c * NS] = v[c];
    }
}

template <int NS, bool DAG, int MODE, bool RED, typename R, bool H>
__global__ __launch_bounds__(256) void k_hop_split(const HopArgsMR<R> a) {
    const int r = blockIdx.y;
    if (a.fin_n && blockIdx.x == gridDim.x - 1) {  // the pending reduction of an earlier launch
        const double* p = a.fin_partials + (size_t)r * a.pstride;
        double* S = a.scal + r * SC_N;
        finish_partials(p, a.fin_n, S, 0, a.fin_epi);
        return;
    }
    const int n = gridDim.x - (a.fin_n ? 1 : 0);
    int b = blockIdx.x;
    {   // hardware dispatches workgroup b to XCD b % 8: every XCD takes one contiguous range of the lattice
        const int x = b & 7, i = b >> 3, q = n >> 3, m = n & 7;
        b = x * q + (x < m ? x : m) + i;
    }
    __shared__ cpx<R> sw[4][2][6][64];  // link products: [mu][forward, backward][component][lane]
    __shared__ float sn[H ? 4 : 1][2][64];
    __shared__ float mx[H ? 2 : 1][4][64];
    __shared__ double lds[4];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int s = lane & (NS - 1);
    int cb = b * (64 / NS) + lane / NS;
    const bool valid = cb < a.g.Vh;
    if (!valid) cb = a.g.Vh - 1;  // keep every lane of a group active for the lane exchanges
    const double done = a.done ? a.done[r * SC_N] : 0.0;  // tested after the barrier: the load overlaps the columns'
    const cpx<R>* in = a.in[r];
    constexpr int SF = DAG ? +1 : -1;
    int nf, nk;
    neighbours_mu(a.g, cb, a.par, w, nf, nk);
    cpx<R> pf[12], pb[12];
    R cf = 1, ck = 1;
    if constexpr (H) {
        cf = load_h_raw<NS>(pf, in, (size_t)nf, s, a.g.Vh);
        ck = load_h_raw<NS>(pb, in, (size_t)nk, s, a.g.Vh);
    } else {
        load_col<NS, false>(pf, in, (size_t)nf, s, 0);
        load_col<NS, false>(pb, in, (size_t)nk, s, 0);
    }
    cpx<R> Uf[9], Ub[9];
#pragma unroll
    for (int k = 0; k < 9; k++) {
        Uf[k] = a.Uown[((size_t)cb * 4 + w) * 9 + k];
        Ub[k] = a.Uoth[((size_t)nk * 4 + w) * 9 + k];
    }
    // what the epilogue of spin w reads, requested with the columns
    const bool up = w < 2;
    constexpr bool SCHUR = MODE == HM_SCHUR_W || MODE == HM_SCHUR_RES;
    constexpr bool OPA = SCHUR || MODE == HM_SITE || MODE == HM_DT, OPB = SCHUR;
    ChirReg<NS, R> tA, tB;
    if constexpr (OPA) chir_fetch<NS, R>(tA, a.opA[r]->h[up ? 0 : 1], s);
    if constexpr (OPB) chir_fetch<NS, R>(tB, a.opB[r]->h[up ? 0 : 1], s);
    cpx<R> ax[3], ax2[3], sf[3];
    const bool aux = SCHUR || MODE == HM_SCHUR_Q || (MODE != HM_DW && a.aux[r] != nullptr);
    if (aux) load_spin<NS, H, R>(ax, a.aux[r], (size_t)cb, s, w, a.g.Vh);
    if constexpr (MODE == HM_SCHUR_Q || MODE == HM_SCHUR_RES) load_spin<NS, false, R>(ax2, a.aux2[r], (size_t)cb, s, w, a.g.Vh);
    if constexpr (MODE == HM_DT || MODE == HM_DW) load_spin<NS, false, R>(sf, a.self, (size_t)cb, s, w, a.g.Vh);
    R alpha = 0;
    if constexpr (MODE == HM_SCHUR_Q) alpha = (R)a.scal[r * SC_N + SC_ALPHA];
    {
        cpx<R> hf[6], hb[6], wv[6];
        switch (w) {
        case 0: project2<0, SF>(pf, pb, hf, hb); break;
        case 1: project2<1, SF>(pf, pb, hf, hb); break;
        case 2: project2<2, SF>(pf, pb, hf, hb); break;
        default: project2<3, SF>(pf, pb, hf, hb); break;
        }
        link_mul<false>(Uf, hf, wv);
#pragma unroll
        for (int k = 0; k < 6; k++) sw[w][0][k][lane] = wv[k];
        link_mul<true>(Ub, hb, wv);
#pragma unroll
        for (int k = 0; k < 6; k++) sw[w][1][k][lane] = wv[k];
        if constexpr (H) { sn[w][0][lane] = cf; sn[w][1][lane] = ck; }
    }
    __syncthreads();
    if (done != 0.0) return;  // uniform over the grid's row
    // spin w of the sum, in the order of the unsplit hop: x, y, z, t, forward before backward
    cpx<R> z[3] = {{0, 0}, {0, 0}, {0, 0}};
    const int l = w & 1;
    auto term = [&](auto MUc, int d) {
        constexpr int MU = decltype(MUc)::value;
        const bool plus = (d == 0) == (SF > 0);  // sign S of (1 + S gamma) in this term
        const int spin = (up || MU >= 2) ? l : 1 - l;
        R nn = 1;
        if constexpr (H) nn = sn[MU][d][lane];
        cpx<R> t[3];
#pragma unroll
        for (int c = 0; c < 3; c++) t[c] = sw[MU][d][3 * spin + c][lane];
        if (up) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                if constexpr (H) { z[c].x = fma(nn, t[c].x, z[c].x); z[c].y = fma(nn, t[c].y, z[c].y); }
                else z[c] = cadd(z[c], t[c]);
            }
        } else {
            add_lower<MU, H>(z, t, l, nn, plus);
        }
    };
    term(std::integral_constant<int, 0>{}, 0); term(std::integral_constant<int, 0>{}, 1);
    term(std::integral_constant<int, 1>{}, 0); term(std::integral_constant<int, 1>{}, 1);
    term(std::integral_constant<int, 2>{}, 0); term(std::integral_constant<int, 2>{}, 1);
    term(std::integral_constant<int, 3>{}, 0); term(std::integral_constant<int, 3>{}, 1);
    // epilogue (the operations of hop_epilogue on this spin)
    double nrm = 0.0;
    cpx<R> v[3];
    if constexpr (MODE == HM_LIN || MODE == HM_SITE) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            v[c] = cscale(a.cz, z[c]);
            if (aux) { v[c].x = fma(a.caux, ax[c].x, v[c].x); v[c].y = fma(a.caux, ax[c].y, v[c].y); }
        }
        if constexpr (MODE == HM_SITE) site_op_spin<NS, DAG>(v, tA, up, s, lane);
    } else if constexpr (SCHUR) {
        site_op_spin<NS, false>(z, tA, up, s, lane);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            v[c].x = fma(a.cz, z[c].x, a.caux * ax[c].x);
            v[c].y = fma(a.cz, z[c].y, a.caux * ax[c].y);
            if constexpr (MODE == HM_SCHUR_RES) v[c] = csub(ax2[c], v[c]);
        }
    } else if constexpr (MODE == HM_SCHUR_Q) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const R qx = fma(a.cz, z[c].x, a.caux * ax[c].x), qy = fma(a.cz, z[c].y, a.caux * ax[c].y);
            v[c].x = fma(-alpha, qx, ax2[c].x);
            v[c].y = fma(-alpha, qy, ax2[c].y);
        }
    } else {
        cpx<R> m[3] = {sf[0], sf[1], sf[2]};
        if constexpr (MODE == HM_DT) site_op_spin<NS, DAG>(m, tA, up, s, lane);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            R tx = a.diag * sf[c].x - (R)0.5 * z[c].x, ty = a.diag * sf[c].y - (R)0.5 * z[c].y;
            if constexpr (MODE == HM_DT) { tx += m[c].x; ty += m[c].y; }
            v[c] = {a.cz * tx, a.cz * ty};
            if (aux) { v[c].x = fma(a.caux, ax[c].x, v[c].x); v[c].y = fma(a.caux, ax[c].y, v[c].y); }
        }
    }
    if (canon_mode<MODE, RED>() && a.canon) {
        int lex;
        cb_to_lex(a.g, cb, a.par, lex);
        cd* d = a.canon + ((a.refl ? NS - 1 - s : s) * 2 * (size_t)a.g.Vh + lex) * 12 + 3 * w;
        const double sg = a.refl && !up ? -1.0 : 1.0;
        if (valid)
#pragma unroll
            for (int c = 0; c < 3; c++) d[c] = {sg * (double)v[c].x, sg * (double)v[c].y};
    } else if (MODE == HM_LIN && a.outf) {
        cpx<float> vf[3];
#pragma unroll
        for (int c = 0; c < 3; c++) vf[c] = {(float)v[c].x, (float)v[c].y};
        store_spin<NS, false>(a.outf, (size_t)cb, s, w, a.g.Vh, vf, valid, mx[0]);
    } else {
        store_spin<NS, H && MODE != HM_SCHUR_Q>(a.out[r], (size_t)cb, s, w, a.g.Vh, v, valid, mx[0]);
    }
    if constexpr (RED) {
#pragma unroll
        for (int c = 0; c < 3; c++) nrm += (double)v[c].x * v[c].x + (double)v[c].y * v[c].y;
    }
    if constexpr (SCHUR) {
        site_op_spin<NS, true>(v, tB, up, s, lane);
        store_spin<NS, H>(a.out2[r], (size_t)cb, s, w, a.g.Vh, v, valid, mx[H ? 1 : 0]);
    }
    if constexpr (RED) {
        const double bs = block_sum256(valid ? nrm : 0.0, lds);
        if (threadIdx.x == 0) a.partials[(size_t)r * a.pstride + blockIdx.x] = bs;
    }
}

}  // namespace

// The split form is the default of a launch of at most kSplitLanes (site, s) lanes, all its systems together: up to
// there k_hop has at most three waves per CU and its four round trips are not hidden.  us per hop, k_hop in
// XCD-contiguous ranges -> split (FP64 / FP32 / FP16 columns):
//   4^4, Ns = 8 (1,024 lanes)            8.8 -> 5.6    7.9 -> 5.2    8.0 -> 5.0
//   8^4, Ns = 8 (16,384)                10.8 -> 7.6    9.1 -> 5.7    9.1 -> 5.3
//   8^3 x 12, Ns = 16 (49,152)          10.8 -> 10.4   9.4 -> 9.3    9.0 -> 7.1
//   8^3 x 16, Ns = 16 (65,536)          11.5 -> 12.6   9.4 -> 10.8   9.0 -> 9.1
// (the split form reads each link once per lane instead of staging it, which shows once the chip is full).
constexpr size_t kSplitLanes = 49152;
bool hop_split(const Geom& g, int Ns, int nr) { return (size_t)g.Vh * Ns * nr <= kSplitLanes; }

int hop_split_blocks(const Geom& g, int Ns) { return (int)(((size_t)g.Vh * Ns + 63) / 64); }

template <typename R>
hipError_t launch_hop_split(int Ns, bool dag, int mode, bool red, const HopArgsMR<R>& a, hipStream_t st, bool half) {
    if (a.nr < 1 || a.nr > NRMAX || !hop_split(a.g, Ns, a.nr)) return hipErrorInvalidValue;
    const int grid = hop_split_blocks(a.g, Ns) + (a.fin_n ? 1 : 0);
#define SPLIT_L(D, M, RD)                                                                                           \
    if constexpr (!hop_has(M, D) || (M == HM_SCHUR_RES && sizeof(R) == 4)) return hipErrorInvalidValue;             \
    else do {                                                                                                            \
        if constexpr (sizeof(R) == 4 && NS >= 8 && (M == HM_SITE || M == HM_SCHUR_W || M == HM_SCHUR_Q)) {           \
            if (half) {                                                                                             \
                hipLaunchKernelGGL((k_hop_split<NS, D, M, M != HM_SITE, R, true>), dim3(grid, a.nr), dim3(256), 0, st, a); \
                break;                                                                                              \
            }                                                                                                       \
        }                                                                                                           \
        if (half) return hipErrorInvalidValue;                                                                      \
        hipLaunchKernelGGL((k_hop_split<NS, D, M, RD, R, false>), dim3(grid, a.nr), dim3(256), 0, st, a);           \
    } while (0)
#define SPLIT_MODES(D)                                                                             \
    switch (mode) {                                                                                \
    case HM_LIN: if (red) SPLIT_L(D, HM_LIN, true); else SPLIT_L(D, HM_LIN, false); break;         \
    case HM_SITE: if (red) SPLIT_L(D, HM_SITE, true); else SPLIT_L(D, HM_SITE, false); break;      \
    case HM_SCHUR_W: SPLIT_L(D, HM_SCHUR_W, true); break;                                          \
    case HM_SCHUR_Q: SPLIT_L(D, HM_SCHUR_Q, true); break;                                          \
    case HM_DT: if (red) SPLIT_L(D, HM_DT, true); else SPLIT_L(D, HM_DT, false); break;            \
    case HM_DW: SPLIT_L(D, HM_DW, false); break;                                                   \
    case HM_SCHUR_RES: SPLIT_L(D, HM_SCHUR_RES, false); break;                                     \
    default: return hipErrorInvalidValue;                                                          \
    }
    switch (Ns) {
    case 4: { constexpr int NS = 4; if (dag) { SPLIT_MODES(true) } else { SPLIT_MODES(false) } break; }
    case 8: { constexpr int NS = 8; if (dag) { SPLIT_MODES(true) } else { SPLIT_MODES(false) } break; }
    case 16: { constexpr int NS = 16; if (dag) { SPLIT_MODES(true) } else { SPLIT_MODES(false) } break; }
    case 32: { constexpr int NS = 32; if (dag) { SPLIT_MODES(true) } else { SPLIT_MODES(false) } break; }
    default: return hipErrorInvalidValue;
    }
#undef SPLIT_MODES
#undef SPLIT_L
    return hipGetLastError();
}
template hipError_t launch_hop_split<double>(int, bool, int, bool, const HopArgsMR<double>&, hipStream_t, bool);
template hipError_t launch_hop_split<float>(int, bool, int, bool, const HopArgsMR<float>&, hipStream_t, bool);

}  // namespace eofa
