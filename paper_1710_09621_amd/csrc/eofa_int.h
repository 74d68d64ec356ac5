// Internal declarations shared by the kernels (kernels.hip) and the host runtime (eofa.cpp).
#pragma once
#include <hip/hip_runtime.h>

#include "eofa_dev.h"

namespace eofa {

enum : int { HM_LIN = 0, HM_SITE = 1, HM_SCHUR_W = 2, HM_SCHUR_Q = 3, HM_DT = 4, HM_DW = 5, HM_SCHUR_RES = 6 };

// Whether a mode exists for the normal (dag = false) or the gamma_5 hop gamma_5 form.
constexpr bool hop_has(int mode, bool dag) {
    return mode == HM_LIN || mode == HM_SITE || mode == HM_DT || dag == (mode == HM_SCHUR_Q);
}

// Order in which workgroups visit the lattice (chosen per lattice by the autotuner).
// The cb index space of one parity is viewed as [t][z][yb] with yb = workgroup index along
// the (xh, y) plane line (nyb workgroups per line).  mode 0: linear.  mode 1: 3D tiles of
// ty x tz x tt workgroups visited tile by tile.  xcd != 0: every XCD (the 8 L2 domains) gets
// one contiguous range of the visiting sequence instead of every 8th workgroup.
// ord = 1 visits each tile with its (z, t) plane fastest and yb slowest.
// mode 3 (single-system FP64 / FP32 hop only): t-walk.  A workgroup owns one segment of 256 / Ns
// sites of a t-slab and walks tt consecutive slabs; the segments form an nyb x (segments / nyb) grid
// and the workgroups that run together on an XCD take a ty x tz patch of it; ord = KB of LDS reserved
// per workgroup (caps the workgroups per CU).  mode 5: mode 3 with the x-direction columns read from LDS,
// for segments that hold whole x-lines.  Mode 6: mode 5 with two lanes per site and slice.  mode 2: the
// direction-split form (hop_split.hip) in XCD-contiguous ranges; the other fields have no meaning.
struct Sched {
    int mode, xcd, ty, tz, tt, nyb, ord;
};
constexpr Sched kSplitSched{2, 1, 1, 1, 1, 1, 0};
inline bool is_twalk(const Sched& sc) { return sc.mode == 3 || sc.mode == 5 || sc.mode == 6; }

template <typename R> struct HopArgs {
    Geom g;
    Sched sc;
    int par;                  // parity of the output sites
    const cpx<R>* in;         // half field of parity 1 - par (the hop input)
    const cpx<R>* Uown;       // packed links of parity par
    const cpx<R>* Uoth;       // packed links of parity 1 - par
    cpx<R>* out;
    cpx<R>* out2;
    const cpx<R>* aux;        // parity par
    const cpx<R>* aux2;       // parity par
    const cpx<R>* self;       // parity par (diagonal term of D_T / D_w)
    cpx<float>* outf;         // HM_LIN: not null: out goes here in FP32 instead
    cd* canon;                // not null: out goes to the output sites of this canonical field instead (hop_canon)
    int refl;                 // canon: gamma_5 R5 on the way, as in launch_unpack5
    const SiteOp* opA;
    const SiteOp* opB;
    R cz, caux, diag;
    const double* scal;       // device scalars (alpha)
    const double* done;       // early-exit flag for graph replays (may be null)
    Red red;
    bool defer;               // leave this launch's partial sums to a later launch (its fin / fin_n)
    Red fin;                  // fin_n > 0: finish the fin_n partial sums that an earlier launch deferred
    unsigned fin_n;
};

// Multi-RHS form of the CG-iteration hops: nr independent systems (own fields, own mass tables,
// own device scalars at scal + r * SC_N) through one launch; the links of each workgroup are
// staged once and reused by all systems; a system whose SC_DONE is set is skipped.
constexpr int NRMAX = 8;
template <typename R> struct HopArgsMR {
    Geom g;
    Sched sc;
    int par, nr;
    int rpb;                // systems per workgroup (set by the launcher)
    const cpx<R>* Uown;
    const cpx<R>* Uoth;
    const cpx<R>* in[NRMAX];
    cpx<R>* out[NRMAX];
    cpx<R>* out2[NRMAX];
    const cpx<R>* aux[NRMAX];
    const cpx<R>* aux2[NRMAX];
    const SiteOp* opA[NRMAX];
    const SiteOp* opB[NRMAX];
    R cz, caux, diag;
    const cpx<R>* self;     // diagonal term of D_T / D_w (one system)
    cpx<float>* outf;       // as in HopArgs (one system)
    cd* canon;
    int refl;
    double* scal;           // nr blocks of SC_N scalars
    const double* done;     // done[r * SC_N] != 0: skip system r (may be null)
    double* partials;       // partials[r * pstride + block]
    int pstride;
    int epi;                // reduction epilogue (EPI_CG_W / EPI_CG_R) for the reducing modes
    bool defer;             // as in HopArgs
    const double* fin_partials;
    unsigned fin_n;
    int fin_epi;
};
// half: FP16-column Krylov fields (R = float; see load_h / store_h in hop_dev.h)
template <typename R> hipError_t launch_hop_mr(int Ns, bool dag, int mode, const HopArgsMR<R>& a, hipStream_t st,
                                               bool half = false);
// The residual's partial sums (n > 0 of system r at partials + r pstride) that the x/p update finishes itself: every
// workgroup adds them up for its beta, the first one writes the scalars.  n = 0: they are finished already.
struct XpFin {
    const double* partials;
    int pstride;
    unsigned n;
};
// n, the partial sums of a system, if an x/p update of Vh Ns lanes is to finish them, else 0
unsigned xp_finishes(unsigned n, size_t lanes, size_t real_bytes, bool half);
// Partial sums that a reducing launch under sc writes per system (for fin_n).
unsigned hop_partials(const Geom& g, int Ns, const Sched& sc);
// direction-split form of the hop (hop_split.hip): whether it is small enough for a launch of nr systems, its workgroups
// per system, and the launch itself (no finishing kernel)
bool hop_split(const Geom& g, int Ns, int nr);
int hop_split_blocks(const Geom& g, int Ns);
template <typename R> hipError_t launch_hop_split(int Ns, bool dag, int mode, bool red, const HopArgsMR<R>& a,
                                                  hipStream_t st, bool half = false);
// FP16 bytes of one half field: 12 Vh Ns (re, im) binary16 pairs + Vh Ns FP32 column norms
inline size_t half_field_bytes_h(const Geom& g, int Ns) { return (size_t)g.Vh * Ns * (12 * 4 + 4); }
// x_r (FP32) += alpha_r p_r ; p_r (FP16 columns) = r_r (FP32) + beta_r p_r unless SC_DONEX is set
hipError_t launch_cg_xp_mr_h(int Ns, int nr, cpx<float>* const* x, void* const* p, cpx<float>* const* r, double* scal,
                             int Vh, const XpFin& fin, hipStream_t st);
hipError_t launch_f2h(int Ns, const cpx<float>* in, void* out, int Vh, hipStream_t st);
hipError_t launch_h2d(int Ns, const void* in, cd* out, int Vh, hipStream_t st);
// x_r += alpha_r p_r ; p_r = r_r + beta_r p_r for the systems whose SC_DONEX is clear
template <typename R> hipError_t launch_cg_xp_mr(int nr, cpx<R>* const* x, cpx<R>* const* p, cpx<R>* const* r,
                                                 double* scal, size_t n, const XpFin& fin, hipStream_t st);

template <typename R> hipError_t launch_hop(int Ns, bool dag, int mode, bool red, const HopArgs<R>& a, hipStream_t st);
int tw_grid(const Geom& g, int Ns, const Sched& sc);
// whether a launch under sc has a form of HM_LIN, HM_DT and HM_DW that writes a canonical field
bool hop_canon(int Ns, const Sched& sc);
Sched block_sched(const Geom& g, int Ns, size_t real_bytes);
// The order of a batch launch of nr systems: the installed one if the batch kernels have it for any number of systems,
// else (null, t-walk, split form) by rule.
inline Sched batch_sched(const Geom& g, int Ns, const Sched* installed, size_t real_bytes, int nr) {
    if (installed && installed->mode < 2) return *installed;
    return hop_split(g, Ns, nr) ? kSplitSched : block_sched(g, Ns, real_bytes);
}
Sched default_sched(const Geom& g, int Ns, size_t real_bytes, bool half);
template <typename R> hipError_t launch_site(int Ns, bool dag, const cpx<R>* in, cpx<R>* out, const SiteOp* op, int Vh,
                                             hipStream_t st);
// x += alpha p ; p = r + beta p unless scal[SC_DONEX] is set
template <typename R> hipError_t launch_cg_xp(cpx<R>* x, cpx<R>* p, const cpx<R>* r, double* scal, size_t n,
                                              const XpFin& fin, hipStream_t st);
template <typename R> hipError_t launch_axpby(R a, const cpx<R>* x, R b, cpx<R>* y, size_t n, const Red* red,
                                              hipStream_t st);
template <typename R> hipError_t launch_norm2(const cpx<R>* x, size_t n, const Red& red, hipStream_t st);
// out[2i] + i out[2i+1] = <v_i, y> (complex, FP64, deterministic), i < nv <= 9; partials >= 2 nv x pstride
hipError_t launch_mdot(const cd* const* v, int nv, const cd* y, size_t n, double* partials, int pstride, double* out,
                       hipStream_t st);
// y += sum_i (cr_i + i ci_i) v_i, nv <= 9
hipError_t launch_maxpy(const cd* const* v, const double* cr, const double* ci, int nv, cd* y, size_t n, hipStream_t st);
// one-block finish of a reduction whose nblocks partials are in r.partials
hipError_t launch_finish(const Red& r, unsigned nblocks, hipStream_t st);
// dst[i] = host_vals[i], i < n <= 64 (values travel as kernel arguments: the host array may die at once)
hipError_t launch_set_vec(double* dst, int n, const double* host_vals, hipStream_t st);
// Terms of the heat-bath combination phi = a0 P_chir eta + sum_l coef[l] out[l] (canonical 4D fields).
constexpr int HB_MAXTERMS = 8;
struct HbTerms {
    const cd* out[HB_MAXTERMS];
    double coef[HB_MAXTERMS];
    double a0;
    int n;
};
// the combination over the n complex elements of a 4D field; |P_chir eta|^2 goes through red
hipError_t launch_hb_combine(const cd* eta, cd* phi, const HbTerms& t, size_t n, int chir, int accumulate,
                             const Red& red, hipStream_t st);
// dst[i] = host_vals[i] for any n, in chunks of 64 values travelling as kernel arguments
hipError_t launch_set_block(double* dst, size_t n, const double* host_vals, hipStream_t st);
// bytes (a multiple of 8) copied from src to dst by a kernel
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st);
// sets S[s_i] = v_i for the slots s_i >= 0 (stream-ordered, no host buffer)
hipError_t launch_scal_set(double* S, int s0, double v0, int s1, double v1, int s2, double v2, hipStream_t st);
// starts a cycle of CG iterations: SC_RR, SC_RR0 and SC_TOL2 set, SC_DONE, SC_DONEX and SC_ITERS cleared
hipError_t launch_scal_arm(double* S, double rr, double rr0, double tol2, hipStream_t st);
// xhi += xlo (first: xhi = xlo), then xlo = 0
hipError_t launch_accum_f(cd* xhi, cpx<float>* xlo, size_t n, bool first, hipStream_t st);
// canonical 5D field -> half[par] (null: that parity is left out) and back (null: zeros)
template <typename R> hipError_t launch_pack5(const cd* canon, cpx<R>* const half[2], const Geom& g, int Ns, int refl,
                                              hipStream_t st);
template <typename R> hipError_t launch_unpack5(const cpx<R>* const half[2], cd* canon, const Geom& g, int Ns, int refl,
                                                hipStream_t st);
// D[par], F[par]: the FP64 and FP32 links of parity par
hipError_t launch_pack_links(const cd* U, cd* const D[2], cpx<float>* const F[2], const Geom& g, double tbc,
                             hipStream_t st);
// an s-space vector travelling as a kernel argument
struct SVec {
    double v[32];
};
// both parities: half[par]
hipError_t launch_source(const cd* phi, cd* const half[2], const Geom& g, int Ns, int chir, const SVec& coef,
                         hipStream_t st);
hipError_t launch_combine(const cd* phi, const cd* const xh[2], cd* out, const Geom& g, int Ns, int chir, double ck,
                          const SVec& Om, int accumulate, const Red& red, hipStream_t st);

// ---- site-local operator tables (sitetab.cpp)
enum SiteKind : int { SK_AINV = 0, SK_AINV_DAG = 1, SK_M = 2, SK_M_DAG = 3, SK_A = 4, SK_A_DAG = 5, SK_OM1L = 6,
                      SK_OM1L_DAG = 7, SK_NKIND = 8 };
// Fill op with the tables of A_T^{-1}, A_T^{-dag}, M, M^T, A, A^T, omega (1 + L) or (1 + L)^T omega for masses
// (mp, mm).
void build_site_op(SiteOp& op, SiteKind kind, int Ns, double m0, const double* omega, double mp, double mm);

}  // namespace eofa
