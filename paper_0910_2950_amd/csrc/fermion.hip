// Fermion-side kernels: the even/odd Wilson hopping term (Dslash) with fused
// Schur-complement and conjugate-gradient epilogues, the reliable-update CG
// driver, the pseudofermion heatbath and the pseudofermion force.
//
// Wilson operator M = 1 - kappa D, D psi(x) = sum_mu [(1 - g_mu) U_mu(x) psi(x+mu)
// + (1 + g_mu) U_mu(x-mu)^+ psi(x-mu)], antiperiodic in t; even/odd Schur
// operator Mhat = 1 - kappa^2 D_eo D_oe on even sites, Mhat^+ = g5 Mhat g5, so
//   Mhat v   : t = D_oe v,      out = v - kappa^2 D_eo t
//   Mhat^+ v : t = D_oe g5 v,   out = v - kappa^2 g5 D_eo t.
// Every Dslash-shaped kernel computes acc = D_{p_out, 1-p_out} [g5] in and the
// epilogue  out = center - kappa^2 [g5] acc  (or out = [g5] acc for a bare hop).
#include <algorithm>
#include <climits>
#include <cmath>

#include "cg_stop.h"
#include "fgi_internal.h"

namespace fgi {

// Threads per block of the Dslash-shaped kernels: at most DBS (launch bounds and
// LDS sizes); the block size in use (64, 128 or 256) is part of the tuned
// schedule, as is the XCD-aware block order.  Helper kernels use DBS.
static const int DBS = 256;
static inline int nblk(long n, int bs) { return (int)((n + bs - 1) / bs); }

// --------------------------------------------------------------- hop sum ---
template <typename R> __device__ __forceinline__ void flip_lower(cx<R> v[4][3]) {
#pragma unroll
    for (int k = 0; k < 3; k++) { v[2][k] = -v[2][k]; v[3][k] = -v[3][k]; }
}

// Round a spinor to FP16 storage with the per-site scale exactly as
// SpinorIO<P16>::store followed by ::load does, in registers.
template <typename R> __device__ __forceinline__ void quantize16(cx<R> v[4][3]) {
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 12; e++) {
        m = fmaxf(m, fabsf(float(v[e / 3][e % 3].re)));
        m = fmaxf(m, fabsf(float(v[e / 3][e % 3].im)));
    }
    float inv = m > 0.f ? 1.0f / m : 0.f;
#pragma unroll
    for (int e = 0; e < 12; e++) {
        cx<R>& a = v[e / 3][e % 3];
        a.re = R(float((_Float16)(float(a.re) * inv)) * m);
        a.im = R(float((_Float16)(float(a.im) * inv)) * m);
    }
}

// p_new = r + beta p_old (explicit FMAs so every kernel rounds identically)
template <typename R>
__device__ __forceinline__ void p_update(const cx<R> r[4][3], cx<R> p[4][3], R beta) {
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) {
            p[i][k].re = fma(beta, p[i][k].re, r[i][k].re);
            p[i][k].im = fma(beta, p[i][k].im, r[i][k].im);
        }
}

// Neighbour spinor loaders used by the hop sum: fetch() issues the raw loads
// of one site, get() converts them to the working precision (the FP16
// conversion and its per-site scale fuse into one mixed-precision FMA) and
// returns the factor the hop applies with its accumulating FMAs (1 here).
template <int PIN, int G5IN, typename R> struct LoadPlain {
    SpinorPtr in;
    typedef RawSp<PIN> Raw;
    __device__ __forceinline__ void fetch(int s, int Vh, Raw& raw) const { fetch_sp<PIN>(in, s, Vh, raw); }
    __device__ __forceinline__ R get(const Raw& raw, cx<R> psi[4][3]) const {
        SpinorIO<PIN, R>::decode(raw, psi);
        if (G5IN) flip_lower(psi);
        return R(1);
    }
};

// The eight hops of D, k = 2 mu + d: d = 0 the forward hop (1 - g_mu) U_mu(x)
// psi(x + mu), d = 1 the backward hop (1 + g_mu) U_mu(x - mu)^+ psi(x - mu).
// Each hop projects to a half spinor, multiplies by the link and accumulates
// the rebuilt spinor times w = (storage scale) x (link unit) x (antiperiodic
// sign in t).
template <int K, int PL, int RECON, bool NT, typename R, typename L>
__device__ __forceinline__ void hop(const Geom& g, int p, int s, const Coord& c, const void* links, const L& load,
                                    cx<R> acc[4][3]) {
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    const int sn = cb_neighbour(g, c, MU, FWD ? +1 : -1);
    cx<R> psi[4][3], h[2][3], uh[2][3];
    typename L::Raw rs;
    load.fetch(sn, g.Vh, rs);
    R w = load.get(rs, psi) * R(link_unit<PL, RECON>());
    spin_proj<MU, FWD ? -1 : +1>(psi, h);
    // the link is loaded after the projection: loads issued any earlier only
    // raise the register count (and lower occupancy on large lattices)
    RawLink<PL, RECON> rl;
    fetch_link<PL, RECON, NT>(links, MU, FWD ? p : 1 - p, FWD ? s : sn, g.Vh, rl);
    const M3<R> u = LinkIO<PL, RECON, R>::decode(rl);
    if constexpr (FWD) {
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int a = 0; a < 3; a++)
                uh[j][a] = cdot3(u.e[a][0], h[j][0], u.e[a][1], h[j][1], u.e[a][2], h[j][2]);
        if (MU == 3 && c.c[3] == g.L[3] - 1) w = -w;
    } else {
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int a = 0; a < 3; a++)
                uh[j][a] = cdot3c(u.e[0][a], h[j][0], u.e[1][a], h[j][1], u.e[2][a], h[j][2]);
        if (MU == 3 && c.c[3] == 0) w = -w;
    }
    spin_recon_acc<MU, FWD ? -1 : +1>(acc, uh, w);
}

template <int PL, int RECON, bool NT, typename R, typename L>
__device__ __forceinline__ void hop_sum(const Geom& g, int p, int s, const void* links, const L& load,
                                        cx<R> acc[4][3]) {
    Coord c = cb_coords(g, p, s);
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) acc[i][k] = {R(0), R(0)};
    hop<0, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<1, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<2, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<3, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<4, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<5, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<6, PL, RECON, NT>(g, p, s, c, links, load, acc);
    hop<7, PL, RECON, NT>(g, p, s, c, links, load, acc);
}

// ------------------------------------------------------------ reductions ---
// No atomics and no grid-scope fences: a reducing kernel writes one partial per
// block (indexed by the block's logical number inside its chain), and the
// kernel after it on the stream sums them in a fixed order (sum_partials), so
// every value is independent of block scheduling and identical wherever it is
// computed.  A last-block-done scheme would need an agent-scope release per
// block, i.e. a write-back of the XCD's L2, which costs several microseconds
// per launch on this part.

// ---------------------------------------------------------- the kernel ---
enum Mode {
    M_HOP = 0,    // out = [g5] acc
    M_SCHUR = 1,  // out = center - kappa^2 [g5] acc          [|out|^2 partials]
    M_CGQ = 2,    // CG: q = p - kappa^2 acc (center p), |q|^2 partials (pAp)
    M_CGX = 3,    // CG: Ap = q - kappa^2 g5 acc; x += alpha p; r -= alpha Ap; |r|^2 partials
    M_RESID = 4,  // r = aux - (center - kappa^2 g5 acc), |r|^2 partials; x = 0 when given
    M_CGS = 5     // CG, Chronopoulos-Gear form: w = q - kappa^2 g5 acc; p = rt + beta p;
                  // s = w + beta s; x += alpha p; r -= alpha s; the hops' copy rt of r;
                  // |r|^2, Re<rt, s>, Re<p, s> partials
};
// With a CG state and partials, an M_HOP launch carries one extra block per
// chain (logical index nb) that sums the M_CGQ partials into st->pAp, or with
// cgs set the three M_CGS partials into the state (cgs_state_update).

struct DArgs {
    Geom g;
    int p_out;
    double kappa2;
    const void* links;
    SpinorPtr in, center, out, aux, x, r;
    double* partial;   // per-block partials written (reducing modes) or read (M_HOP in CG)
    CGState* st;
    int iter;   // absolute index, or the offset from st->base inside a CG batch
    int g5out;
    int gate;   // with st: 0 skip once st->stop_at <= iteration, 1 skip unless st->act
    int xcd;    // XCD-aware block order
    int cgs;    // M_HOP reduction block of the Chronopoulos-Gear form
    SpinorPtr dir, adir;   // M_CGS: p and s = A p, in the precision of x and r
    const void* blk;       // clover kernels: the blocks of the output parity's sites, in the links' precision
    long bstride;          // their stride (V)
};

// The clover term is site-local, so its kernels are the Wilson ones with one
// product by the site's two 6x6 blocks: A_oo^-1 on a hop onto odd sites, A_ee on
// the centre of the Schur-shaped modes.  Both are Hermitian: the upper triangle
// is read and the lower is its conjugate (21 of 36 entries).
template <int PB, typename R> __device__ __forceinline__ cx<R> blk_entry(const void* blk, long stride, int k, int s) {
    if constexpr (PB == P64) {
        const d2 e = ((const d2*)blk)[k * stride + s];
        return {R(e.x), R(e.y)};
    } else {
        const f2 e = ((const f2*)blk)[k * stride + s];
        return {R(e.x), R(e.y)};
    }
}
// y += e x and y += conj(e) x
template <typename R> __device__ __forceinline__ void cfma(cx<R>& y, cx<R> e, cx<R> x) {
    y.re = fma(e.re, x.re, y.re);
    y.re = fma(-e.im, x.im, y.re);
    y.im = fma(e.re, x.im, y.im);
    y.im = fma(e.im, x.re, y.im);
}
// v = A v for a whole site
template <int PB, typename R>
__device__ __forceinline__ void clover_mul(const void* blk, long stride, int s, cx<R> v[4][3]) {
#pragma unroll
    for (int b = 0; b < 2; b++) {
        cx<R> o[6];
#pragma unroll
        for (int r = 0; r < 6; r++) o[r] = {R(0), R(0)};
#pragma unroll
        for (int r = 0; r < 6; r++)
#pragma unroll
            for (int c = r; c < 6; c++) {
                const cx<R> e = blk_entry<PB, R>(blk, stride, b * 36 + r * 6 + c, s);
                if (c == r) {
                    o[r].re = fma(e.re, v[2 * b + c / 3][c % 3].re, o[r].re);
                    o[r].im = fma(e.re, v[2 * b + c / 3][c % 3].im, o[r].im);
                } else {
                    cfma(o[r], e, v[2 * b + c / 3][c % 3]);
                    cfma(o[c], conj(e), v[2 * b + r / 3][r % 3]);
                }
            }
#pragma unroll
        for (int r = 0; r < 6; r++) v[2 * b + r / 3][r % 3] = o[r];
    }
}
// One wave's half block (split kernels): the spin w = 2 b + h of a site holds
// rows 3 h .. 3 h + 2 of block b.
template <int PB, typename R> struct HalfBlk {
    cx<R> e[3][6];
    __device__ __forceinline__ void load(const void* blk, long stride, int s, int w) {
        const int b = w >> 1, r0 = 3 * (w & 1);
#pragma unroll
        for (int k = 0; k < 3; k++)
#pragma unroll
            for (int c = 0; c < 6; c++) {
                const int r = r0 + k;
                const cx<R> v = blk_entry<PB, R>(blk, stride, b * 36 + (c >= r ? r * 6 + c : c * 6 + r), s);
                e[k][c] = c >= r ? v : conj(v);
            }
    }
    __device__ __forceinline__ void mul(const cx<R> v[6], cx<R> o[3]) const {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            o[k] = {R(0), R(0)};
#pragma unroll
            for (int c = 0; c < 6; c++) cfma(o[k], e[k][c], v[c]);
        }
    }
};

// Chronopoulos-Gear form (Chronopoulos and Gear, J. Comput. Appl. Math. 25
// (1989) 153): the operator is applied to the residual, w = A rt with rt the
// residual as the hops read it, and the direction and its image follow by
// recurrence, p_k = rt_k + beta_k p_{k-1}, s_k = w_k + beta_k s_{k-1}, so one
// kernel updates p, s, x and r and the direction update needs no launch of its
// own.  <p_k, A p_k> is not taken from the usual recurrence (it assumes
// rt = r and exact conjugacy, which FP16 storage and reliable updates break)
// but expanded exactly: |Mhat rt_k|^2 + 2 beta Re<rt_k, s_{k-1}> + beta^2
// Re<p_{k-1}, s_{k-1}>, the last two summed by the update kernel before.
// First kernel of iteration k (the reduction block of its hop): the previous
// update's partials |r_k|^2, Re<rt_k, s_{k-1}>, Re<p_{k-1}, s_{k-1}> give
// rr_k, beta_k = rr_k / rr_{k-1} and the correction; the stop test on rr_k.
__device__ __forceinline__ void cgs_state_update(CGState* st, const StateView& S, int iter, const double* part,
                                                 int nb, double* lds) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < nb; k += blockDim.x) {
        v[0] += part[k];
        v[1] += part[nb + k];
        v[2] += part[2 * nb + k];
    }
    block_sum<3>(v, lds);
    if (threadIdx.x == 0) {
        // a select, not S.rr[(iter - 1) & 1]: a run-time index into the state
        // copy makes the compiler place it in LDS, one copy per thread
        const double beta = v[0] / ((iter & 1) ? S.rr[0] : S.rr[1]);
        st->rr[iter & 1] = v[0];
        st->beta = beta;
        st->corr = 2.0 * beta * v[1] + beta * beta * v[2];
        if (v[0] <= S.rr_stop) st->stop_at = iter;
    }
}

// NT: the links are streamed with non-temporal loads (see links_streamed); CL: the clover operator
template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN, bool NT, bool CL>
__device__ __forceinline__ void dslash_body(const DArgs& A, int b, int nb, double* lds) {
    typedef typename Real<PIN == P64 ? P64 : P32>::T R;
    const Geom& g = A.g;
    // Solver state, read up front in one batch of loads (reading each field
    // where it is used puts a memory round trip per branch in front of the
    // data loads).  Of what is used here the same launch writes only stop_at
    // (see cg_leaves).
    StateView S{INT_MAX, 0, 0, 1, {0.0, 0.0}, 0.0, 0.0, 0.0};
    if (A.st) S = load_state(A.st);
    const int iter = S.base + A.iter;
    if (A.st) {  // converged / masked chains no-op
        if (A.gate ? !S.act : cg_leaves(S.stop_at, iter, MODE == M_HOP && A.cgs && b < nb)) return;
        if constexpr (MODE == M_HOP) {
            if (b >= nb) {  // the reduction block: pAp of this iteration, or the CG-form state
                if (A.cgs) {
                    cgs_state_update(A.st, S, iter, A.partial, nb, lds);
                } else if (A.partial) {
                    const double pAp = sum_partials(A.partial, nb, lds);
                    if (threadIdx.x == 0) A.st->pAp = pAp;
                }
                return;
            }
        }
    }
    int s = b * blockDim.x + threadIdx.x;
    double nrm = 0.0, rs = 0.0, ps = 0.0;
    if (s < g.Vh) {
        cx<R> acc[4][3];
        LoadPlain<PIN, G5IN, R> ld{A.in};
        hop_sum<PL, RECON, NT, R>(g, A.p_out, s, A.links, ld, acc);
        if (A.g5out) flip_lower(acc);
        if (MODE == M_HOP) {
            if constexpr (CL) clover_mul<PL, R>(A.blk, A.bstride, s, acc);
            SpinorIO<POUT, R>::store(A.out, s, g.Vh, acc);
        } else {
            cx<R> cen[4][3];
            SpinorIO<PC, R>::load(A.center, s, g.Vh, cen);
            if constexpr (CL) clover_mul<PL, R>(A.blk, A.bstride, s, cen);
            const R k2 = R(A.kappa2);
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int k = 0; k < 3; k++) acc[i][k] = cen[i][k] - k2 * acc[i][k];
            if (MODE == M_SCHUR || MODE == M_CGQ) {
                SpinorIO<POUT, R>::store(A.out, s, g.Vh, acc);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 3; k++)
                        nrm += double(acc[i][k].re) * double(acc[i][k].re) + double(acc[i][k].im) * double(acc[i][k].im);
            } else if (MODE == M_RESID) {
                cx<R> ph[4][3];
                SpinorIO<PC, R>::load(A.aux, s, g.Vh, ph);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        acc[i][k] = ph[i][k] - acc[i][k];
                        nrm += double(acc[i][k].re) * double(acc[i][k].re) + double(acc[i][k].im) * double(acc[i][k].im);
                    }
                SpinorIO<POUT, R>::store(A.out, s, g.Vh, acc);
                if (A.x.v) {
#pragma unroll
                    for (int i = 0; i < 4; i++)
#pragma unroll
                        for (int k = 0; k < 3; k++) acc[i][k] = {R(0), R(0)};
                    SpinorIO<POUT, R>::store(A.x, s, g.Vh, acc);
                }
            } else if (MODE == M_CGX) {
                typedef typename Real<PX>::T RX;
                const RX al = RX(((iter & 1) ? S.rr[1] : S.rr[0]) / S.pAp);
                cx<RX> pv[4][3], xv[4][3], rv[4][3];
                SpinorIO<PC, RX>::load(A.aux, s, g.Vh, pv);  // p has the precision of q
                SpinorIO<PX, RX>::load(A.x, s, g.Vh, xv);
                SpinorIO<PX, RX>::load(A.r, s, g.Vh, rv);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        cx<RX> ap = {RX(acc[i][k].re), RX(acc[i][k].im)};
                        xv[i][k] = xv[i][k] + al * pv[i][k];
                        rv[i][k] = rv[i][k] - al * ap;
                        nrm += double(rv[i][k].re) * double(rv[i][k].re) + double(rv[i][k].im) * double(rv[i][k].im);
                    }
                SpinorIO<PX, RX>::store(A.x, s, g.Vh, xv);
                SpinorIO<PX, RX>::store(A.r, s, g.Vh, rv);
            } else if (MODE == M_CGS) {
                typedef typename Real<PX>::T RX;
                const RX be = RX(S.beta);
                const RX al = RX(((iter & 1) ? S.rr[1] : S.rr[0]) / (S.pAp + S.corr));
                cx<RX> tv[4][3], pv[4][3], sv[4][3], xv[4][3], rv[4][3];
                SpinorIO<PC, RX>::load(A.aux, s, g.Vh, tv);  // rt_k, as the hops read it
                SpinorIO<PX, RX>::load(A.dir, s, g.Vh, pv);
                SpinorIO<PX, RX>::load(A.adir, s, g.Vh, sv);
                SpinorIO<PX, RX>::load(A.x, s, g.Vh, xv);
                SpinorIO<PX, RX>::load(A.r, s, g.Vh, rv);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        const cx<RX> w = {RX(acc[i][k].re), RX(acc[i][k].im)};
                        pv[i][k].re = fma(be, pv[i][k].re, tv[i][k].re);
                        pv[i][k].im = fma(be, pv[i][k].im, tv[i][k].im);
                        sv[i][k].re = fma(be, sv[i][k].re, w.re);
                        sv[i][k].im = fma(be, sv[i][k].im, w.im);
                        xv[i][k] = xv[i][k] + al * pv[i][k];
                        rv[i][k] = rv[i][k] - al * sv[i][k];
                        nrm += double(rv[i][k].re) * double(rv[i][k].re) + double(rv[i][k].im) * double(rv[i][k].im);
                        ps += double(pv[i][k].re) * double(sv[i][k].re) + double(pv[i][k].im) * double(sv[i][k].im);
                    }
                SpinorIO<PX, RX>::store(A.dir, s, g.Vh, pv);
                SpinorIO<PX, RX>::store(A.adir, s, g.Vh, sv);
                SpinorIO<PX, RX>::store(A.x, s, g.Vh, xv);
                SpinorIO<PX, RX>::store(A.r, s, g.Vh, rv);
                if constexpr (PC != PX) {  // the hops' copy of r, and Re<rt, s> with the stored values
                    static_assert(PC == P16, "a separate copy of r is kept for FP16 hops only");
                    SpinorIO<PC, RX>::store(A.aux, s, g.Vh, rv);
                    quantize16(rv);
                }
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 3; k++)
                        rs += double(rv[i][k].re) * double(sv[i][k].re) + double(rv[i][k].im) * double(sv[i][k].im);
            }
        }
    }
    if (MODE == M_HOP || !A.partial) return;
    if constexpr (MODE == M_CGS) {
        double v[3] = {nrm, rs, ps};
        block_sum<3>(v, lds);
        if (threadIdx.x == 0) {
            A.partial[b] = v[0];
            A.partial[nb + b] = v[1];
            A.partial[2 * nb + b] = v[2];
        }
        return;
    }
    double v[1] = {nrm};
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) A.partial[b] = v[0];
}

template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN, bool NT, bool CL>
__global__ void __launch_bounds__(DBS) k_dslash(DArgs A) {
    __shared__ double lds[3 * DBS / 64];
    // site blocks in XCD-aware order (the same order in every kernel of the
    // solver, so a site stays on one XCD); a reduction block comes last
    const int nb = (A.g.Vh + blockDim.x - 1) / blockDim.x;
    const int b = (int)blockIdx.x < nb ? (A.xcd ? xcd_block(blockIdx.x, nb) : (int)blockIdx.x) : blockIdx.x;
    dslash_body<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, NT, CL>(A, b, nb, lds);
}

// ------------------------------------------------ split sites (small lattices) ---
// One thread per site leaves most of the chip idle below a few hundred waves
// (8^4: 32 waves on 1024 SIMDs), and the launch then lasts as long as one
// thread's chain of eight dependent hops.  Here a block's four waves share 64
// sites: wave w takes the two hops along direction w as far as the link times
// half-spinor products, with all its loads in flight together; the products
// meet in LDS and wave w sums spin w of the eight hops and finishes it.  The sum
// runs over the hops in the one-thread order with the same multiply-adds, so a
// site's result has the same bits in FP64 and FP32 (in FP16 the compiler fuses the
// stored numbers' scaling into the projection differently in the two kernels: 3 % of
// the sites of a 12-real hop hold a number stored one step apart, both 3.33e-4 from
// FP64); the block sums of the reductions are grouped differently.
// site_split makes both a property of the lattice and its storage.

// element e = 3 spin + colour of the spinor at s (R the working precision)
template <int P, typename R> __device__ __forceinline__ cx<R> load_elem(const SpinorPtr& f, int s, int Vh, int e, float n) {
    if constexpr (P == P64) {
        const d2 v = ((const d2*)f.v)[(size_t)e * Vh + s];
        return {R(v.x), R(v.y)};
    } else if constexpr (P == P32) {
        const f2 v = ((const f2*)f.v)[((size_t)(e >> 1) * Vh + s) * 2 + (e & 1)];
        return {R(v.x), R(v.y)};
    } else {
        const h2 v = ((const h2*)f.v)[((size_t)(e >> 2) * Vh + s) * 4 + (e & 3)];
        return {R(float(v.x) * n), R(float(v.y) * n)};
    }
}
template <int P> __device__ __forceinline__ float load_norm(const SpinorPtr& f, int s) {
    if constexpr (P == P16) return f.norm[s];
    return 1.0f;
}

// One spin (three colours) of a spinor as one wave of the block holds it.
template <int P, typename R>
__device__ __forceinline__ void load_spin(const SpinorPtr& f, int s, int Vh, int w, cx<R> v[3]) {
    const float n = load_norm<P>(f, s);
#pragma unroll
    for (int k = 0; k < 3; k++) v[k] = load_elem<P, R>(f, s, Vh, 3 * w + k, n);
}

// FP16 storage needs the largest component over the four waves' spins (mx:
// 4 x 64 floats of LDS); every wave of the block calls this together.
template <int P, typename R>
__device__ __forceinline__ void store_spin(const SpinorPtr& f, int s, int Vh, int w, bool live, const cx<R> v[3],
                                           float* mx) {
    if constexpr (P == P16) {
        const int lane = threadIdx.x & 63;
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < 3; k++) m = fmaxf(m, fmaxf(fabsf(float(v[k].re)), fabsf(float(v[k].im))));
        mx[w * 64 + lane] = m;
        __syncthreads();
        m = fmaxf(fmaxf(mx[lane], mx[64 + lane]), fmaxf(mx[128 + lane], mx[192 + lane]));
        if (!live) return;
        const float inv = m > 0.f ? 1.0f / m : 0.f;
        if (w == 0) f.norm[s] = m;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int e = 3 * w + k;
            ((h2*)f.v)[((size_t)(e >> 2) * Vh + s) * 4 + (e & 3)] =
                h2{(_Float16)(float(v[k].re) * inv), (_Float16)(float(v[k].im) * inv)};
        }
    } else {
        if (!live) return;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int e = 3 * w + k;
            if constexpr (P == P64) ((d2*)f.v)[(size_t)e * Vh + s] = d2{double(v[k].re), double(v[k].im)};
            else ((f2*)f.v)[((size_t)(e >> 1) * Vh + s) * 2 + (e & 1)] = f2{float(v[k].re), float(v[k].im)};
        }
    }
}

// U h (FWD) or U^+ h for both rows of a half spinor, into uh[2][3] of one hop
template <bool FWD, typename R>
__device__ __forceinline__ void link_half(const M3<R>& u, const cx<R> h[2][3], cx<R> (*out)[64], int lane) {
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int a = 0; a < 3; a++)
            out[3 * j + a][lane] = FWD ? cdot3(u.e[a][0], h[j][0], u.e[a][1], h[j][1], u.e[a][2], h[j][2])
                                       : cdot3c(u.e[0][a], h[j][0], u.e[1][a], h[j][1], u.e[2][a], h[j][2]);
}

// the link products of both hops along MU, every load issued before any arithmetic
template <int MU, int PIN, int PL, int RECON, int G5IN, typename R>
__device__ __forceinline__ void hop_pair(const Geom& g, int p, int s, const Coord& c, const void* links,
                                         const SpinorPtr& in, cx<R> (*uh)[6][64], int lane) {
    const int sf = cb_neighbour(g, c, MU, +1), sb = cb_neighbour(g, c, MU, -1);
    LoadPlain<PIN, G5IN, R> ld{in};
    typename LoadPlain<PIN, G5IN, R>::Raw rf, rb;
    RawLink<PL, RECON> lf, lb;
    ld.fetch(sf, g.Vh, rf);
    fetch_link<PL, RECON, false>(links, MU, p, s, g.Vh, lf);
    ld.fetch(sb, g.Vh, rb);
    fetch_link<PL, RECON, false>(links, MU, 1 - p, sb, g.Vh, lb);
    cx<R> psi[4][3], h[2][3];
    ld.get(rf, psi);
    spin_proj<MU, -1>(psi, h);
    link_half<true>(LinkIO<PL, RECON, R>::decode(lf), h, uh[2 * MU], lane);
    ld.get(rb, psi);
    spin_proj<MU, +1>(psi, h);
    link_half<false>(LinkIO<PL, RECON, R>::decode(lb), h, uh[2 * MU + 1], lane);
}

// acc += w times spin S of the four-spinor that hop K = 2 MU + d rebuilds from
// its half spinor (the multiply-adds of spin_recon_acc)
template <int S, int K, typename R>
__device__ __forceinline__ void recon_spin(cx<R> acc[3], const cx<R> (*uh)[64], int lane, R w) {
    constexpr int MU = K >> 1;
    constexpr bool NEG = (K & 1) == 0;   // (1 - g_mu), the forward hop
    constexpr int J = S < 2 ? S : ((MU == 0 || MU == 1) ? 3 - S : S - 2);
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cx<R> x = uh[3 * J + c][lane];
        cx<R> y = x;
        if (S >= 2) {
            if (MU == 0) y = NEG ? times_i(x) : times_mi(x);
            else if (MU == 1) y = (S == 2) == NEG ? -x : x;
            else if (MU == 2) y = (S == 2) == NEG ? times_i(x) : times_mi(x);
            else y = NEG ? -x : x;
        }
        acc[c] = axpy(w, y, acc[c]);
    }
}
template <int S, typename R>
__device__ __forceinline__ void sum_spin(cx<R> acc[3], const cx<R> (*uh)[6][64], int lane, R unit, R wf, R wb) {
#pragma unroll
    for (int c = 0; c < 3; c++) acc[c] = {R(0), R(0)};
    recon_spin<S, 0>(acc, uh[0], lane, unit);
    recon_spin<S, 1>(acc, uh[1], lane, unit);
    recon_spin<S, 2>(acc, uh[2], lane, unit);
    recon_spin<S, 3>(acc, uh[3], lane, unit);
    recon_spin<S, 4>(acc, uh[4], lane, unit);
    recon_spin<S, 5>(acc, uh[5], lane, unit);
    recon_spin<S, 6>(acc, uh[6], lane, wf);
    recon_spin<S, 7>(acc, uh[7], lane, wb);
}

// the eight hops' link products: [hop][component][site of the block]
template <typename R> struct SplitLds {
    cx<R> uh[8][6][64];
    float mx[256];
    double red[3 * 4];
};

// spin w of the hop sum (w uniform over the wave); unit carries the link unit,
// the antiperiodic boundary flips the sign of the t hops that cross it
template <typename R>
__device__ __forceinline__ void split_sum(const SplitLds<R>& L, int w, int lane, R unit, const Geom& g, const Coord& c,
                                          int g5out, cx<R> acc[3]) {
    const R wf = c.c[3] == g.L[3] - 1 ? -unit : unit, wb = c.c[3] == 0 ? -unit : unit;
    if (w == 0) sum_spin<0>(acc, L.uh, lane, unit, wf, wb);
    else if (w == 1) sum_spin<1>(acc, L.uh, lane, unit, wf, wb);
    else if (w == 2) sum_spin<2>(acc, L.uh, lane, unit, wf, wb);
    else sum_spin<3>(acc, L.uh, lane, unit, wf, wb);
    if (g5out && w >= 2) {
#pragma unroll
        for (int k = 0; k < 3; k++) acc[k] = -acc[k];
    }
}

// A block's 64 sites of one Dslash-shaped kernel (the modes of dslash_body).
// early: leave before any load when this launch has nothing to do (batched
// launches, where finished chains must not keep the chip busy); otherwise the
// state is only waited for after the hops, its latency hidden behind theirs.
template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN, bool CL>
__device__ __forceinline__ void dslash_split_body(const DArgs& A, int b, int nb, int early,
                                                  SplitLds<typename Real<PIN == P64 ? P64 : P32>::T>& L) {
    typedef typename Real<PIN == P64 ? P64 : P32>::T R;
    typedef typename Real<PX>::T RX;
    const Geom& g = A.g;
    StateView S{INT_MAX, 0, 0, 1, {0.0, 0.0}, 0.0, 0.0, 0.0};
    if (A.st) S = load_state(A.st);
    const int iter = S.base + A.iter;
    const bool idle = A.st && (A.gate ? !S.act : cg_leaves(S.stop_at, iter, MODE == M_HOP && A.cgs && b < nb));
    if (A.st && (early || b >= nb)) {
        if (idle) return;
        if constexpr (MODE == M_HOP) {
            if (b >= nb) {
                if (A.cgs) {
                    cgs_state_update(A.st, S, iter, A.partial, nb, L.red);
                } else if (A.partial) {
                    const double pAp = sum_partials(A.partial, nb, L.red);
                    if (threadIdx.x == 0) A.st->pAp = pAp;
                }
                return;
            }
        }
    }
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s_ = b * SPLIT_SITES + lane;
    const bool live = s_ < g.Vh;
    const int s = live ? s_ : g.Vh - 1;
    const Coord c = cb_coords(g, A.p_out, s);
    // the epilogue's operands, in flight beside the hops'
    cx<R> cen[3], ph[3];
    cx<RX> av[3], xv[3], rv[3], pv[3], sv[3];
    if constexpr (MODE != M_HOP && !CL) load_spin<PC, R>(A.center, s, g.Vh, w, cen);
    [[maybe_unused]] HalfBlk<PL, R> hb;
    [[maybe_unused]] cx<R> six[6];
    if constexpr (CL) {
        hb.load(A.blk, A.bstride, s, w);
        if constexpr (MODE != M_HOP) {
            load_spin<PC, R>(A.center, s, g.Vh, w & 2, six);
            load_spin<PC, R>(A.center, s, g.Vh, w | 1, six + 3);
        }
    }
    if constexpr (MODE == M_RESID) load_spin<PC, R>(A.aux, s, g.Vh, w, ph);
    if constexpr (MODE == M_CGX || MODE == M_CGS) {
        load_spin<PC, RX>(A.aux, s, g.Vh, w, av);
        load_spin<PX, RX>(A.x, s, g.Vh, w, xv);
        load_spin<PX, RX>(A.r, s, g.Vh, w, rv);
    }
    if constexpr (MODE == M_CGS) {
        load_spin<PX, RX>(A.dir, s, g.Vh, w, pv);
        load_spin<PX, RX>(A.adir, s, g.Vh, w, sv);
    }
    if (w == 0) hop_pair<0, PIN, PL, RECON, G5IN, R>(g, A.p_out, s, c, A.links, A.in, L.uh, lane);
    else if (w == 1) hop_pair<1, PIN, PL, RECON, G5IN, R>(g, A.p_out, s, c, A.links, A.in, L.uh, lane);
    else if (w == 2) hop_pair<2, PIN, PL, RECON, G5IN, R>(g, A.p_out, s, c, A.links, A.in, L.uh, lane);
    else hop_pair<3, PIN, PL, RECON, G5IN, R>(g, A.p_out, s, c, A.links, A.in, L.uh, lane);
    __syncthreads();
    if (idle) return;
    const R unit = R(link_unit<PL, RECON>());
    cx<R> acc[3];
    if constexpr (CL && MODE == M_HOP) {   // A_oo^-1 needs both spins of the wave's block
        split_sum<R>(L, w & 2, lane, unit, g, c, A.g5out, six);
        split_sum<R>(L, w | 1, lane, unit, g, c, A.g5out, six + 3);
        hb.mul(six, acc);
    } else {
        split_sum<R>(L, w, lane, unit, g, c, A.g5out, acc);
        if constexpr (CL) hb.mul(six, cen);
    }
    double nrm = 0.0, rs = 0.0, ps = 0.0;
    if constexpr (MODE == M_HOP) {
        store_spin<POUT, R>(A.out, s, g.Vh, w, live, acc, L.mx);
        return;
    } else {
        const R k2 = R(A.kappa2);
#pragma unroll
        for (int k = 0; k < 3; k++) acc[k] = cen[k] - k2 * acc[k];
        if constexpr (MODE == M_SCHUR || MODE == M_CGQ || MODE == M_RESID) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
                if constexpr (MODE == M_RESID) acc[k] = ph[k] - acc[k];
                nrm += double(acc[k].re) * double(acc[k].re) + double(acc[k].im) * double(acc[k].im);
            }
            store_spin<POUT, R>(A.out, s, g.Vh, w, live, acc, L.mx);
            if (MODE == M_RESID && A.x.v) {
#pragma unroll
                for (int k = 0; k < 3; k++) acc[k] = {R(0), R(0)};
                store_spin<POUT, R>(A.x, s, g.Vh, w, live, acc, L.mx);
            }
        } else if constexpr (MODE == M_CGX) {
            const RX al = RX(((iter & 1) ? S.rr[1] : S.rr[0]) / S.pAp);
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const cx<RX> ap = {RX(acc[k].re), RX(acc[k].im)};
                xv[k] = xv[k] + al * av[k];
                rv[k] = rv[k] - al * ap;
                nrm += double(rv[k].re) * double(rv[k].re) + double(rv[k].im) * double(rv[k].im);
            }
            store_spin<PX, RX>(A.x, s, g.Vh, w, live, xv, L.mx);
            store_spin<PX, RX>(A.r, s, g.Vh, w, live, rv, L.mx);
        } else {
            const RX be = RX(S.beta);
            const RX al = RX(((iter & 1) ? S.rr[1] : S.rr[0]) / (S.pAp + S.corr));
#pragma unroll
            for (int k = 0; k < 3; k++) {
                pv[k].re = fma(be, pv[k].re, av[k].re);
                pv[k].im = fma(be, pv[k].im, av[k].im);
                sv[k].re = fma(be, sv[k].re, RX(acc[k].re));
                sv[k].im = fma(be, sv[k].im, RX(acc[k].im));
                xv[k] = xv[k] + al * pv[k];
                rv[k] = rv[k] - al * sv[k];
                nrm += double(rv[k].re) * double(rv[k].re) + double(rv[k].im) * double(rv[k].im);
                ps += double(pv[k].re) * double(sv[k].re) + double(pv[k].im) * double(sv[k].im);
            }
            store_spin<PX, RX>(A.dir, s, g.Vh, w, live, pv, L.mx);
            store_spin<PX, RX>(A.adir, s, g.Vh, w, live, sv, L.mx);
            store_spin<PX, RX>(A.x, s, g.Vh, w, live, xv, L.mx);
            store_spin<PX, RX>(A.r, s, g.Vh, w, live, rv, L.mx);
            if constexpr (PC != PX) {  // the hops' copy of r, and Re<rt, s> with the stored values
                store_spin<PC, RX>(A.aux, s, g.Vh, w, live, rv, L.mx);
                const float m = fmaxf(fmaxf(L.mx[lane], L.mx[64 + lane]), fmaxf(L.mx[128 + lane], L.mx[192 + lane]));
                const float inv = m > 0.f ? 1.0f / m : 0.f;
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    rv[k].re = RX(float((_Float16)(float(rv[k].re) * inv)) * m);
                    rv[k].im = RX(float((_Float16)(float(rv[k].im) * inv)) * m);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; k++) rs += double(rv[k].re) * double(sv[k].re) + double(rv[k].im) * double(sv[k].im);
        }
    }
    if (!A.partial) return;
    if (!live) nrm = rs = ps = 0.0;
    if constexpr (MODE == M_CGS) {
        double v[3] = {nrm, rs, ps};
        block_sum<3>(v, L.red);
        if (threadIdx.x == 0) {
            A.partial[b] = v[0];
            A.partial[nb + b] = v[1];
            A.partial[2 * nb + b] = v[2];
        }
        return;
    }
    double v[1] = {nrm};
    block_sum<1>(v, L.red);
    if (threadIdx.x == 0) A.partial[b] = v[0];
}

template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN, bool CL>
__global__ void __launch_bounds__(256) k_dslash_split(DArgs A) {
    __shared__ SplitLds<typename Real<PIN == P64 ? P64 : P32>::T> L;
    const int nb = (A.g.Vh + SPLIT_SITES - 1) / SPLIT_SITES;
    const int b = (int)blockIdx.x < nb ? (A.xcd ? xcd_block(blockIdx.x, nb) : (int)blockIdx.x) : blockIdx.x;
    dslash_split_body<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, CL>(A, b, nb, 0, L);
}

// one chain's part of a concatenated spinor field / link field
template <int P> __device__ __forceinline__ SpinorPtr spin_off(SpinorPtr p, const ChainDesc& d) {
    if (!p.v) return p;
    SpinorPtr q = p;
    if (P == P64) q.v = (d2*)p.v + 12 * (size_t)d.site0;
    else if (P == P32) q.v = (f4*)p.v + 6 * (size_t)d.site0;
    else {
        q.v = (h8*)p.v + 3 * (size_t)d.site0;
        q.norm = p.norm + d.site0;
    }
    return q;
}

template <int PL, int RECON> __device__ __forceinline__ size_t link_byte_off(const ChainDesc& d) {
    if (PL == P64) return 9 * (size_t)d.link0 * sizeof(d2);
    return (size_t)d.link0 * sloppy_link_bytes(PL, RECON);
}

// One chain's arguments of a batched launch: its own geometry, kappa, solver
// state (base.st[c]) and partials slice.
template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON>
__device__ __forceinline__ DArgs chain_args(const DArgs& base, const ChainDesc& d, int c) {
    DArgs A = base;
    A.g = d.g;
    A.kappa2 = d.kappa * d.kappa;
    A.links = (const char*)base.links + link_byte_off<PL, RECON>(d);
    A.in = spin_off<PIN>(base.in, d);
    A.center = spin_off<PC>(base.center, d);
    A.aux = spin_off<PC>(base.aux, d);
    A.out = spin_off<POUT>(base.out, d);
    A.x = spin_off<MODE == M_RESID ? POUT : PX>(base.x, d);
    A.r = spin_off<PX>(base.r, d);
    A.partial = base.partial ? base.partial + d.blk0[GRID_DS] : nullptr;
    A.st = base.st ? base.st + c : nullptr;
    return A;
}

// batched launch over the chains of one block table (ds_map): nsb site blocks,
// and past them (an M_HOP with partials) the chains' reduction blocks
template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN>
__global__ void __launch_bounds__(DBS) k_dslash_b(DArgs base, const ChainDesc* __restrict__ cd,
                                                  const int2* __restrict__ map, int nsb) {
    __shared__ double lds[3 * DBS / 64];
    const int gb = (int)blockIdx.x < nsb ? (base.xcd ? xcd_block(blockIdx.x, nsb) : (int)blockIdx.x) : blockIdx.x;
    const int2 m = map[gb];
    const ChainDesc& d = cd[m.x];
    const DArgs A = chain_args<MODE, PIN, PC, POUT, PX, PL, RECON>(base, d, m.x);
    dslash_body<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, false, false>(A, m.y, d.nblk[GRID_DS], lds);
}

template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN>
__global__ void __launch_bounds__(256) k_dslash_split_b(DArgs base, const ChainDesc* __restrict__ cd,
                                                        const int2* __restrict__ map, int nsb) {
    __shared__ SplitLds<typename Real<PIN == P64 ? P64 : P32>::T> L;
    const int gb = (int)blockIdx.x < nsb ? (base.xcd ? xcd_block(blockIdx.x, nsb) : (int)blockIdx.x) : blockIdx.x;
    const int2 m = map[gb];
    const ChainDesc& d = cd[m.x];
    const DArgs A = chain_args<MODE, PIN, PC, POUT, PX, PL, RECON>(base, d, m.x);
    dslash_split_body<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, false>(A, m.y, d.nblk[GRID_DS], 1, L);
}

// The iteration's rr, beta or stop (cg_open); block 0 records them for the kernels after it.
__device__ __forceinline__ bool open_iteration(CGState* st, const StateView& S, int iter, const double* partial, int b,
                                               int nb, double* lds, double& beta) {
    return cg_open(
        S, iter, b == 0 && threadIdx.x == 0, [&] { return sum_partials(partial, nb, lds); },
        [&](double rr, double be, bool stop) {
            st->rr[iter & 1] = rr;
            if (stop) st->stop_at = iter;
            else st->beta = be;
        },
        beta);
}

// First kernel of a CG iteration: p = r + beta p, stored in p's precision.
// Later iterations of a run take |r_iter|^2 from the previous M_CGX's
// partials, summed in every block in the same order (so all blocks agree
// bitwise), and beta = rr / rr_prev; block 0 records rr and beta, or the
// stop once rr <= rr_stop, for the kernels after it.  The first iteration of
// a run (start or reliable update) takes the rr and beta it was set up with.
template <int PP, int PX>
__device__ __forceinline__ void cg_p_body(int Vh, SpinorPtr p, SpinorPtr r, CGState* st, const double* partial,
                                          int j, int b, int nb, double* lds) {
    typedef typename Real<PP == P64 ? P64 : P32>::T R;
    // the state and the site's r and p are loaded before anything waits on
    // them, so their latencies overlap with each other and with the partials
    const StateView S = load_state(st);
    const int s = b * blockDim.x + threadIdx.x;
    const int sl = s < Vh ? s : Vh - 1;
    RawSp<PX> rr_raw;
    RawSp<PP> pp_raw;
    fetch_sp<PX>(r, sl, Vh, rr_raw);
    fetch_sp<PP>(p, sl, Vh, pp_raw);
    double beta = 0.0;
    if (!open_iteration(st, S, S.base + j, partial, b, nb, lds, beta)) return;
    if (s >= Vh) return;
    cx<R> rv[4][3], pv[4][3];
    SpinorIO<PX, R>::decode(rr_raw, rv);
    SpinorIO<PP, R>::decode(pp_raw, pv);
    p_update(rv, pv, R(beta));
    SpinorIO<PP, R>::store(p, s, Vh, pv);
}

template <int PP, int PX>
// np: the number of |r|^2 partials (blocks of the M_CGX launch, the same grid)
__global__ void __launch_bounds__(DBS) k_cg_p(int Vh, SpinorPtr p, SpinorPtr r, CGState* st, const double* partial,
                                              int np, int xcd, int j) {
    __shared__ double lds[DBS / 64];
    cg_p_body<PP, PX>(Vh, p, r, st, partial, j, xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x, np, lds);
}

template <int PP, int PX>
__global__ void __launch_bounds__(DBS) k_cg_p_b(const ChainDesc* __restrict__ cd, const int2* __restrict__ map,
                                                SpinorPtr p, SpinorPtr r, CGState* st, const double* partial, int xcd,
                                                int j) {
    __shared__ double lds[DBS / 64];
    const int2 m = map[xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x];
    const ChainDesc& d = cd[m.x];
    cg_p_body<PP, PX>(d.g.Vh, spin_off<PP>(p, d), spin_off<PX>(r, d), st + m.x, partial + d.blk0[GRID_DS], j, m.y,
                      d.nblk[GRID_DS], lds);
}

// The same with a block's four waves sharing 64 sites, one spin each.
template <int PP, int PX>
__device__ __forceinline__ void cg_p_split_body(int Vh, const SpinorPtr& p, const SpinorPtr& r, CGState* st,
                                                const double* partial, int j, int b, int nb, double* lds, float* mx) {
    typedef typename Real<PP == P64 ? P64 : P32>::T R;
    const StateView S = load_state(st);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s_ = b * SPLIT_SITES + (threadIdx.x & 63);
    const bool live = s_ < Vh;
    const int s = live ? s_ : Vh - 1;
    cx<R> rv[3], pv[3];
    load_spin<PX, R>(r, s, Vh, w, rv);
    load_spin<PP, R>(p, s, Vh, w, pv);
    double beta = 0.0;
    if (!open_iteration(st, S, S.base + j, partial, b, nb, lds, beta)) return;
    const R be = R(beta);
#pragma unroll
    for (int k = 0; k < 3; k++) {
        pv[k].re = fma(be, pv[k].re, rv[k].re);
        pv[k].im = fma(be, pv[k].im, rv[k].im);
    }
    store_spin<PP, R>(p, s, Vh, w, live, pv, mx);
}

template <int PP, int PX>
__global__ void __launch_bounds__(256) k_cg_p_split(int Vh, SpinorPtr p, SpinorPtr r, CGState* st,
                                                    const double* partial, int xcd, int j) {
    __shared__ double lds[4];
    __shared__ float mx[256];
    cg_p_split_body<PP, PX>(Vh, p, r, st, partial, j, xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x,
                            gridDim.x, lds, mx);
}

template <int PP, int PX>
__global__ void __launch_bounds__(256) k_cg_p_split_b(const ChainDesc* __restrict__ cd, const int2* __restrict__ map,
                                                      SpinorPtr p, SpinorPtr r, CGState* st, const double* partial,
                                                      int xcd, int j) {
    __shared__ double lds[4];
    __shared__ float mx[256];
    const int2 m = map[xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x];
    const ChainDesc& d = cd[m.x];
    cg_p_split_body<PP, PX>(d.g.Vh, spin_off<PP>(p, d), spin_off<PX>(r, d), st + m.x, partial + d.blk0[GRID_DS], j,
                            m.y, d.nblk[GRID_DS], lds, mx);
}

// Last node of a CG batch: fold the |r|^2 partials of the batch's last
// iteration into the state (so the host sees a finished run at once) and
// move the batch base.  The next batch's first direction update sums the
// same partials again, in the same order, and agrees bitwise.
__device__ __forceinline__ void advance_body(CGState* st, const double* partial, int nb, int n, double* lds) {
    const int it = st->base + n;  // first iteration of the next batch
    if (st->stop_at == INT_MAX) {
        const double rr = sum_partials(partial, nb, lds);
        if (threadIdx.x == 0) {
            st->rr[it & 1] = rr;
            if (rr <= st->rr_stop) st->stop_at = it;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) st->base = it;
}

// seen: the pinned host copy of the state that the host reads at its waits
__global__ void __launch_bounds__(DBS) k_advance(CGState* st, const double* partial, int nb, int n, CGState* seen) {
    __shared__ double lds[DBS / 64];
    advance_body(st, partial, nb, n, lds);
    if (threadIdx.x == 0) *seen = *st;
}

// The scalars of a solve that the host does not have to wait for: tolerances
// in, |phi|^2 and the last true residual out (pinned host memory).
struct CGRun {
    double tol2, ru2;      // tol^2, ru_delta^2 (0: the inner run goes straight to the target)
    const double* bb;      // |phi|^2 on the device
    double* seen;          // host: [0] |phi|^2, [1] |r|^2 of the last true residual
    int maxiter, batch;    // of a batch's chains (cg_cut)
};
__device__ __forceinline__ double inner_stop(const CGRun& C, double rr, double target) {
    const double s = C.ru2 * rr;
    return C.ru2 > 0.0 && s > target ? s : target;
}

// First state of a run: rr0 = |phi|^2, or (part) the |r|^2 of a starting point.
// A zero phi or a starting point within the target leaves a finished run.
__global__ void __launch_bounds__(DBS) k_cg_start(CGState* st, CGRun C, const double* part, int nb) {
    __shared__ double lds[DBS / 64];
    const double rr0 = part ? sum_partials(part, nb, lds) : *C.bb;
    if (threadIdx.x) return;
    const double target = C.tol2 * *C.bb;
    CGState h{};
    h.rr[0] = rr0;
    h.rr[1] = rr0;   // the CG form's first beta divides by it (p = s = 0 there, so its value does not matter)
    h.rr_stop = inner_stop(C, rr0, target);
    const bool there = *C.bb == 0.0 || (part && rr0 <= target) || !isfinite(rr0);
    h.stop_at = there ? 0 : INT_MAX;
    *st = h;
    C.seen[0] = *C.bb;
    C.seen[1] = rr0;
}

// After a true residual at iteration kend: the run continues from it like a
// start that keeps the direction, or is finished.
__global__ void __launch_bounds__(DBS) k_cg_restart(CGState* st, CGRun C, const double* part, int nb, int kend) {
    __shared__ double lds[DBS / 64];
    const double rr = sum_partials(part, nb, lds);
    if (threadIdx.x) return;
    const double target = C.tol2 * *C.bb;
    st->beta = rr / st->rr[(kend - 1) & 1];
    st->rr[kend & 1] = rr;
    st->rr_stop = inner_stop(C, rr, target);
    st->stop_at = rr <= target || !isfinite(rr) ? 0 : INT_MAX;
    st->base = kend;
    st->base0 = kend;
    C.seen[1] = rr;
}

// ---- the chains of a batch, one block each: as above, and each chain's own end
__global__ void __launch_bounds__(DBS) k_cg_start_b(const ChainDesc* __restrict__ cd, CGState* st, CGChain* ch, CGRun C,
                                                    const double* part) {
    __shared__ double lds[DBS / 64];
    const int i = blockIdx.x;
    const double bb = C.bb[i], target = C.tol2 * bb;
    const bool zero = bb == 0.0;
    const double rr0 = part && !zero ? sum_partials(part + cd[i].blk0[GRID_DS], cd[i].nblk[GRID_DS], lds) : bb;
    if (threadIdx.x) return;
    const bool there = zero || (part && rr0 <= target);
    CGState h{};
    h.rr[0] = rr0;
    h.rr_stop = inner_stop(C, rr0, target);
    h.stop_at = there || !isfinite(rr0) ? 0 : INT_MAX;
    st[i] = h;
    CGChain e{};
    e.bb = bb;
    e.rr0 = e.rr = rr0;
    e.status = there ? CH_CONVERGED : isfinite(rr0) ? CH_RUNNING : CH_BAD;
    e.cut = cg_cut(0, C.maxiter, C.batch);
    ch[i] = e;
}

// act: chains whose inner run has ended, or been cut off, take the true residual next
__global__ void __launch_bounds__(DBS) k_advance_b(const ChainDesc* __restrict__ cd, CGState* st, const CGChain* ch,
                                                   const double* partial, int n) {
    __shared__ double lds[DBS / 64];
    const int i = blockIdx.x;
    advance_body(st + i, partial + cd[i].blk0[GRID_DS], cd[i].nblk[GRID_DS], n, lds);
    if (threadIdx.x) return;
    const CGState& s = st[i];
    st[i].act = ch[i].status == CH_RUNNING && (s.stop_at <= s.base || s.base >= ch[i].cut);
}

// Unless all running chains have ended their inner runs (or one was cut off), hold
// the true residual back: the chains that wait keep in step with the few that need
// some iterations more.
__global__ void __launch_bounds__(DBS) k_cg_hold_b(int nc, CGState* st, const CGChain* ch) {
    int open = 0, cut = 0;
    for (int i = threadIdx.x; i < nc; i += DBS) {
        const bool running = ch[i].status == CH_RUNNING;
        open |= running && !st[i].act;
        cut |= st[i].act && st[i].stop_at > st[i].base;
    }
    open = __syncthreads_or(open);
    cut = __syncthreads_or(cut);
    if (!open || cut) return;
    for (int i = threadIdx.x; i < nc; i += DBS) st[i].act = 0;
}

// seen: the pinned host copy of states and chains that the host reads once a round
__global__ void __launch_bounds__(DBS) k_cg_restart_b(const ChainDesc* __restrict__ cd, CGState* st, CGChain* ch, CGRun C,
                                                      const double* part, CGSeen* seen) {
    __shared__ double lds[DBS / 64];
    const int i = blockIdx.x;
    CGState s = st[i];
    CGChain e = ch[i];
    const double rr = s.act ? sum_partials(part + cd[i].blk0[GRID_DS], cd[i].nblk[GRID_DS], lds) : 0.0;
    if (threadIdx.x) return;
    if (s.act) {
        const double target = C.tol2 * e.bb;
        const int kend = s.stop_at <= s.base ? s.stop_at : s.base;
        e.rr = rr;
        e.iters = kend;
        s.act = 0;
        if (!isfinite(rr) || rr <= target || kend >= C.maxiter) {
            e.status = !isfinite(rr) ? CH_BAD : rr <= target ? CH_CONVERGED : CH_CUT;
            s.stop_at = 0;   // no iteration runs from now on
        } else {
            e.updates++;
            e.cut = cg_cut(kend, C.maxiter, C.batch);
            s.beta = rr / s.rr[(kend - 1) & 1];
            s.rr[kend & 1] = rr;
            s.rr_stop = inner_stop(C, rr, target);
            s.stop_at = INT_MAX;
            s.base = kend;
            s.base0 = kend;
        }
        st[i] = s;
        ch[i] = e;
    }
    seen[i].s = s;
    seen[i].h = e;
}

// act: the chains with (zero) or without a zero right-hand side
__global__ void k_cg_mask_b(int nc, CGState* st, const double* bb, int zero) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nc) st[i].act = (bb[i] == 0.0) == (zero != 0);
}

// conversion between storage precisions (through FP64 registers)
template <int PA, int PB>
__global__ void k_convert(int Vh, SpinorPtr a, SpinorPtr b) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= Vh) return;
    cx<double> v[4][3];
    SpinorIO<PA, double>::load(a, s, Vh, v);
    SpinorIO<PB, double>::store(b, s, Vh, v);
}

// y(FP64) += x(PX)
template <int PX>
__global__ void k_add_to64(int Vh, SpinorPtr x, SpinorPtr y) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= Vh) return;
    cx<double> a[4][3], b[4][3];
    SpinorIO<PX, double>::load(x, s, Vh, a);
    SpinorIO<P64, double>::load(y, s, Vh, b);
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) b[i][k] = b[i][k] + a[i][k];
    SpinorIO<P64, double>::store(y, s, Vh, b);
}

// The three partials an M_CGS launch leaves (|r|^2, Re<rt, s>, Re<p, s>) for
// the vectors as they stand: the start of a Chronopoulos-Gear run and each
// reliable update, so the next iteration's first kernel finds them as after
// any other iteration.  Blocks of the solver's block size, indexed linearly.
template <int PP, int PX>
__global__ void __launch_bounds__(DBS) k_cgs_partials(int Vh, SpinorPtr r, SpinorPtr rt, SpinorPtr p, SpinorPtr sv,
                                                      double* partial) {
    __shared__ double lds[3 * DBS / 64];
    typedef typename Real<PX>::T RX;
    const int nb = gridDim.x, b = blockIdx.x;
    const int s = b * blockDim.x + threadIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    if (s < Vh) {
        cx<RX> rv[4][3], tv[4][3], pv[4][3], w[4][3];
        SpinorIO<PX, RX>::load(r, s, Vh, rv);
        SpinorIO<PP, RX>::load(rt, s, Vh, tv);
        SpinorIO<PX, RX>::load(p, s, Vh, pv);
        SpinorIO<PX, RX>::load(sv, s, Vh, w);
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                v[0] += double(rv[i][k].re) * double(rv[i][k].re) + double(rv[i][k].im) * double(rv[i][k].im);
                v[1] += double(tv[i][k].re) * double(w[i][k].re) + double(tv[i][k].im) * double(w[i][k].im);
                v[2] += double(pv[i][k].re) * double(w[i][k].re) + double(pv[i][k].im) * double(w[i][k].im);
            }
    }
    block_sum<3>(v, lds);
    if (threadIdx.x == 0) {
        partial[b] = v[0];
        partial[nb + b] = v[1];
        partial[2 * nb + b] = v[2];
    }
}


__global__ void k_zero(size_t n, double* p) {
    size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 0.0;
}

__global__ void k_norm2_partials(int Vh, const d2* __restrict__ v, double* partial) {
    __shared__ double lds[DBS / 64];
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    double a[1] = {0.0};
    if (s < Vh) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            d2 e = v[(size_t)k * Vh + s];
            a[0] += e.x * e.x + e.y * e.y;
        }
    }
    block_sum<1>(a, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = a[0];
}

// Re phi^+ X - |eta|^2 per even site, block partials
__global__ void k_pf_density(int Vh, const d2* __restrict__ phi, const d2* __restrict__ X, const d2* __restrict__ eta,
                             double* partial) {
    __shared__ double lds[DBS / 64];
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    double a[1] = {0.0};
    if (s < Vh) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            d2 f = phi[(size_t)k * Vh + s], x = X[(size_t)k * Vh + s];
            a[0] += f.x * x.x + f.y * x.y;
            if (eta) {
                d2 e = eta[(size_t)k * Vh + s];
                a[0] -= e.x * e.x + e.y * e.y;
            }
        }
    }
    block_sum<1>(a, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = a[0];
}

// ----------------------------------------------------- fermion force ------
// For S = phi^+ (Mhat^+ Mhat)^-1 phi and full-lattice X = (X_e, D_oe X_e),
// Y = (Mhat X_e, g5 D_oe g5 Mhat X_e):  F_mu(x) = kappa^2 bc TA(U_mu(x) C) with
//   C = sum_k h-_k(X(x+mu)) h-_k(Y(x))^+ + h+_k(Y(x+mu)) h+_k(X(x))^+,
// h-/h+ the two independent spin components of (1 -/+ g_mu) (colour vectors),
// bc = -1 on the time boundary link.
// C(A, B) of the link (mu, x) for full-lattice vectors A, B (parity p site s,
// its forward neighbour sn of the other parity)
// A full-lattice field as its two parity halves seen from one site: `here`
// the half of the site's parity, `there` the other (its neighbours').  Chosen
// by selects once per thread: an array of the two indexed by the run-time
// parity would make the compiler keep a copy per thread in LDS.
struct PairAt {
    SpinorPtr here, there;
};
__device__ __forceinline__ PairAt pair_at(SpinorPtr even, SpinorPtr odd, int p) {
    return PairAt{p ? odd : even, p ? even : odd};
}

template <int MU>
__device__ __forceinline__ M3<double> outer_c(const Geom& g, int s, int sn, const PairAt& A, const PairAt& B) {
    cx<double> a[4][3], h1[2][3], h2[2][3], h3[2][3], h4[2][3];
    SpinorIO<P64, double>::load(A.there, sn, g.Vh, a);
    spin_proj<MU, -1>(a, h1);
    SpinorIO<P64, double>::load(B.here, s, g.Vh, a);
    spin_proj<MU, -1>(a, h2);
    SpinorIO<P64, double>::load(B.there, sn, g.Vh, a);
    spin_proj<MU, +1>(a, h3);
    SpinorIO<P64, double>::load(A.here, s, g.Vh, a);
    spin_proj<MU, +1>(a, h4);
    M3<double> C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
            C.e[i][j] = mulc(h1[0][i], h2[0][j]) + mulc(h1[1][i], h2[1][j]) + mulc(h3[0][i], h4[0][j]) +
                        mulc(h3[1][i], h4[1][j]);
    return C;
}

template <int MU>
__device__ __forceinline__ void ff_add(const Geom& g, int p, int s, const Coord& c, const M3<double>& W, double coef,
                                       double* F) {
    double x[8];
    ta_components(W, x);
    double f = coef * ((MU == 3 && c.c[3] == g.L[3] - 1) ? -1.0 : 1.0);
    double* o = F + (size_t)((MU * 2 + p) * 8) * g.Vh + s;
#pragma unroll
    for (int k = 0; k < 8; k++) o[(size_t)k * g.Vh] += f * x[k];
}

template <int MU>
__device__ __forceinline__ void ff_link(const Geom& g, int p, int s, const Coord& c, const d2* U,
                                        const PairAt& X, const PairAt& Y, double coef, double* F) {
    int sn = cb_neighbour(g, c, MU, +1);
    M3<double> C = outer_c<MU>(g, s, sn, X, Y);
    ff_add<MU>(g, p, s, c, m3_mul(gauge_load(U, MU, p, s, g.Vh), C), coef, F);
}

__global__ void __launch_bounds__(256) k_fermion_force(Geom g, const d2* __restrict__ U, SpinorPtr Xe, SpinorPtr Xo,
                                                      SpinorPtr Ye, SpinorPtr Yo, double coef, double* __restrict__ F,
                                                      int xcd) {
    int t = slab_thread(g.Vh, 2, xcd);
    if (t >= g.V) return;
    int p = t / g.Vh, s = t % g.Vh;
    Coord c = cb_coords(g, p, s);
    const PairAt X = pair_at(Xe, Xo, p), Y = pair_at(Ye, Yo, p);
    ff_link<0>(g, p, s, c, U, X, Y, coef, F);
    ff_link<1>(g, p, s, c, U, X, Y, coef, F);
    ff_link<2>(g, p, s, c, U, X, Y, coef, F);
    ff_link<3>(g, p, s, c, U, X, Y, coef, F);
}

// Derivative along V of the force kappa^2 bc TA(U C(X, Y)) (Section 4's
// Leibniz rule on the force): the vectors move to dX, dY and the link U to
// V U, so per link
//   J += coef bc TA( U [C(dX, Y) + C(X, dY)] + V U C(X, Y) ).
template <int MU>
__device__ __forceinline__ void ff_tangent_link(const Geom& g, int p, int s, const Coord& c, const d2* U,
                                                const double* Vd, const PairAt& X, const PairAt& Y,
                                                const PairAt& dX, const PairAt& dY, double coef,
                                                double* J) {
    int sn = cb_neighbour(g, c, MU, +1);
    M3<double> C1 = outer_c<MU>(g, s, sn, dX, Y);
    M3<double> C2 = outer_c<MU>(g, s, sn, X, dY);
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) C1.e[i][j] = C1.e[i][j] + C2.e[i][j];
    M3<double> u = gauge_load(U, MU, p, s, g.Vh);
    double v[8];
    mom_load(Vd, MU, p, s, g.Vh, v);
    M3<double> W0 = m3_mul(alg_matrix(v), m3_mul(u, outer_c<MU>(g, s, sn, X, Y)));
    M3<double> W = m3_mul(u, C1);
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) W.e[i][j] = W.e[i][j] + W0.e[i][j];
    ff_add<MU>(g, p, s, c, W, coef, J);
}

__global__ void __launch_bounds__(256) k_fermion_force_tangent(Geom g, const d2* __restrict__ U,
                                                              const double* __restrict__ Vd, SpinorPtr Xe,
                                                              SpinorPtr Xo, SpinorPtr Ye, SpinorPtr Yo, SpinorPtr dXe,
                                                              SpinorPtr dXo, SpinorPtr dYe, SpinorPtr dYo, double coef,
                                                              double* __restrict__ J, int xcd) {
    int t = slab_thread(g.Vh, 2, xcd);
    if (t >= g.V) return;
    int p = t / g.Vh, s = t % g.Vh;
    Coord c = cb_coords(g, p, s);
    const PairAt X = pair_at(Xe, Xo, p), Y = pair_at(Ye, Yo, p), dX = pair_at(dXe, dXo, p), dY = pair_at(dYe, dYo, p);
    ff_tangent_link<0>(g, p, s, c, U, Vd, X, Y, dX, dY, coef, J);
    ff_tangent_link<1>(g, p, s, c, U, Vd, X, Y, dX, dY, coef, J);
    ff_tangent_link<2>(g, p, s, c, U, Vd, X, Y, dX, dY, coef, J);
    ff_tangent_link<3>(g, p, s, c, U, Vd, X, Y, dX, dY, coef, J);
}

// out = a x + b [g5] y on FP64 even/odd vectors (out may alias x or y)
__global__ void k_sp_lincomb(int Vh, double a, const d2* x, double b, const d2* y, int g5y, d2* out) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= Vh) return;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const double by = (g5y && k >= 6) ? -b : b;
        d2 u = x[(size_t)k * Vh + s], v = y[(size_t)k * Vh + s];
        out[(size_t)k * Vh + s] = d2{a * u.x + by * v.x, a * u.y + by * v.y};
    }
}

// ------------------------------------------------- batched small kernels ---
// chain of the calling block in a Vh-sized batched grid and its local site
#define FGI_CHAIN_SITE(cd, nc)                                             \
    const int c_ = find_chain(cd, nc, blockIdx.x, GRID_VH);                \
    const ChainDesc& d = cd[c_];                                           \
    const int s = (blockIdx.x - d.blk0[GRID_VH]) * blockDim.x + threadIdx.x

template <int PA, int PB>
__global__ void k_convert_b(const ChainDesc* __restrict__ cd, int nc, SpinorPtr a, SpinorPtr b) {
    FGI_CHAIN_SITE(cd, nc);
    if (s >= d.g.Vh) return;
    cx<double> v[4][3];
    SpinorIO<PA, double>::load(spin_off<PA>(a, d), s, d.g.Vh, v);
    SpinorIO<PB, double>::store(spin_off<PB>(b, d), s, d.g.Vh, v);
}

template <int PX>
__global__ void k_add_to64_b(const ChainDesc* __restrict__ cd, int nc, const CGState* st, SpinorPtr x, SpinorPtr y) {
    FGI_CHAIN_SITE(cd, nc);
    if (s >= d.g.Vh || !st[c_].act) return;
    cx<double> a[4][3], b[4][3];
    SpinorIO<PX, double>::load(spin_off<PX>(x, d), s, d.g.Vh, a);
    SpinorPtr yy = spin_off<P64>(y, d);
    SpinorIO<P64, double>::load(yy, s, d.g.Vh, b);
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) b[i][k] = b[i][k] + a[i][k];
    SpinorIO<P64, double>::store(yy, s, d.g.Vh, b);
}

// zero the spinors of the chains with act set
template <int P>
__global__ void k_zero_spinor_b(const ChainDesc* __restrict__ cd, int nc, const CGState* st, SpinorPtr v) {
    FGI_CHAIN_SITE(cd, nc);
    if (s >= d.g.Vh || !st[c_].act) return;
    cx<double> z[4][3];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) z[i][k] = {0.0, 0.0};
    SpinorIO<P, double>::store(spin_off<P>(v, d), s, d.g.Vh, z);
}

__global__ void k_norm2_partials_b(const ChainDesc* __restrict__ cd, int nc, const d2* __restrict__ v,
                                   double* __restrict__ partial) {
    __shared__ double lds[DBS / 64];
    FGI_CHAIN_SITE(cd, nc);
    const d2* w = v + 12 * (size_t)d.site0;
    double a[1] = {0.0};
    if (s < d.g.Vh) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            d2 e = w[(size_t)k * d.g.Vh + s];
            a[0] += e.x * e.x + e.y * e.y;
        }
    }
    block_sum<1>(a, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = a[0];
}

__global__ void k_pf_density_b(const ChainDesc* __restrict__ cd, int nc, const d2* __restrict__ phi,
                               const d2* __restrict__ X, const d2* __restrict__ eta, double* __restrict__ partial) {
    __shared__ double lds[DBS / 64];
    FGI_CHAIN_SITE(cd, nc);
    const size_t o = 12 * (size_t)d.site0;
    const int Vh = d.g.Vh;
    double a[1] = {0.0};
    if (s < Vh) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            d2 f = phi[o + (size_t)k * Vh + s], x = X[o + (size_t)k * Vh + s];
            a[0] += f.x * x.x + f.y * x.y;
            if (eta) {
                d2 e = eta[o + (size_t)k * Vh + s];
                a[0] -= e.x * e.x + e.y * e.y;
            }
        }
    }
    block_sum<1>(a, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = a[0];
}

// batched fermion force: coef times kappa_c^2 for chain c (Y_e = Mhat X_e form)
__global__ void __launch_bounds__(256) k_fermion_force_b(const ChainDesc* __restrict__ cd, int nc,
                                                        const d2* __restrict__ U, SpinorPtr Xe, SpinorPtr Xo,
                                                        SpinorPtr Ye, SpinorPtr Yo, double coef,
                                                        double* __restrict__ F) {
    const int c_ = find_chain(cd, nc, blockIdx.x, GRID_V);
    const ChainDesc& d = cd[c_];
    const Geom& g = d.g;
    const int t = (blockIdx.x - d.blk0[GRID_V]) * blockDim.x + threadIdx.x;
    if (t >= g.V) return;
    int p = t / g.Vh, s = t % g.Vh;
    Coord c = cb_coords(g, p, s);
    const PairAt X = pair_at(spin_off<P64>(Xe, d), spin_off<P64>(Xo, d), p);
    const PairAt Y = pair_at(spin_off<P64>(Ye, d), spin_off<P64>(Yo, d), p);
    const d2* u = U + 9 * d.link0;
    double* f = F + 8 * d.link0;
    const double cf = coef * d.kappa * d.kappa;
    ff_link<0>(g, p, s, c, u, X, Y, cf, f);
    ff_link<1>(g, p, s, c, u, X, Y, cf, f);
    ff_link<2>(g, p, s, c, u, X, Y, cf, f);
    ff_link<3>(g, p, s, c, u, X, Y, cf, f);
}

// ------------------------------------------------------- host launchers ---
static SpinorPtr sp(const void* v, float* norm = nullptr) { return SpinorPtr{(void*)v, norm}; }

// Links are streamed (non-temporal loads) when the whole link field of the
// operator is larger than the L2 caches together (8 XCDs x 4 MB): then they
// cannot stay cached between launches anyway, and streaming them keeps the
// neighbour spinors in L2.  Smaller fields are reused from L2 across the CG's
// kernels, so they are loaded normally.  Batched launches always load them
// normally (batches are many small lattices).
static const double kL2Bytes = 32.0 * (1 << 20);
static int links_streamed(const FermionOp& op, long nlinks) {
    const double per = op.prec == P64 ? 144 : (double)sloppy_link_bytes(op.prec, op.recon);
    return per * (double)nlinks > kL2Bytes ? 1 : 0;
}

// blocks (= partials) of the Dslash-shaped kernels on a lattice
static int ds_blocks(const Ctx& c, int Vh) { return nblk(Vh, ds_sites(c, Vh)); }

template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN, bool CL>
static void launch_dslash_rec(Ctx& c, const FermionOp& op, DArgs& a) {
    // an M_HOP inside CG (state and partials) carries the pAp reduction block
    const int extra = (MODE == M_HOP && a.st && a.partial) ? 1 : 0;
    if (site_split(c, a.g.Vh)) {
        hipLaunchKernelGGL((k_dslash_split<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, CL>),
                           dim3(nblk(a.g.Vh, SPLIT_SITES) + extra), dim3(256), 0, c.stream, a);
        return;
    }
    const dim3 nb(nblk(a.g.Vh, c.ds_bs) + extra), bs(c.ds_bs);
    if (links_streamed(op, 4L * a.g.V))
        hipLaunchKernelGGL((k_dslash<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, true, CL>), nb, bs, 0, c.stream, a);
    else hipLaunchKernelGGL((k_dslash<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN, false, CL>), nb, bs, 0, c.stream, a);
}

// op.blk selects the clover kernels: A_oo^-1 on hops onto odd sites, A_ee on the
// centre of the other modes
template <int MODE, int PIN, int PC, int POUT, int PX, int G5IN>
static void launch_dslash(Ctx& c, const FermionOp& op, DArgs& a) {
    a.xcd = c.ds_xcd;
    if (op.blk) {
        if constexpr (PIN != P16 && MODE != M_CGS) {
            if (MODE == M_HOP && a.p_out != 1) throw Error(-1, "a clover hop goes onto odd sites");   // A_ee there
            a.bstride = a.g.V;
            a.blk = (const char*)op.blk + (size_t)a.p_out * a.g.Vh * (op.prec == P64 ? sizeof(d2) : sizeof(f2));
            if constexpr (PIN == P64) {
                if (op.prec != P64) throw Error(-1, "FP64 spinors need FP64 links");
                launch_dslash_rec<MODE, PIN, PC, POUT, PX, P64, 18, G5IN, true>(c, op, a);
            } else {
                if (op.prec != P32) throw Error(-1, "the clover kernels take FP64 or FP32 links");
                if (op.recon == 18) launch_dslash_rec<MODE, PIN, PC, POUT, PX, P32, 18, G5IN, true>(c, op, a);
                else launch_dslash_rec<MODE, PIN, PC, POUT, PX, P32, 12, G5IN, true>(c, op, a);
            }
            FGI_LAUNCH_CHECK();
            return;
        }
        throw Error(-1, "no clover kernel for this storage");
    }
    if constexpr (PIN == P64) {
        if (op.prec != P64) throw Error(-1, "FP64 spinors need FP64 links");
        launch_dslash_rec<MODE, PIN, PC, POUT, PX, P64, 18, G5IN, false>(c, op, a);
    } else {
        if (op.prec == P32 && op.recon == 18) launch_dslash_rec<MODE, PIN, PC, POUT, PX, P32, 18, G5IN, false>(c, op, a);
        else if (op.prec == P32) launch_dslash_rec<MODE, PIN, PC, POUT, PX, P32, 12, G5IN, false>(c, op, a);
        else if (op.prec == P16 && op.recon == 18) launch_dslash_rec<MODE, PIN, PC, POUT, PX, P16, 18, G5IN, false>(c, op, a);
        else if (op.prec == P16) launch_dslash_rec<MODE, PIN, PC, POUT, PX, P16, 12, G5IN, false>(c, op, a);
        else throw Error(-1, "sloppy spinors need sloppy links");
    }
    FGI_LAUNCH_CHECK();
}

static DArgs base_args(const FermionOp& op, int p_out) {
    DArgs a{};
    a.g = *op.g;
    a.p_out = p_out;
    a.kappa2 = op.kappa * op.kappa;
    a.links = op.links;
    return a;
}

static CGState* dev_state(Ctx& c) { return (CGState*)c.state.get(sizeof(CGState)); }

void dslash(Ctx& c, const FermionOp& op, int out_parity, int prec_in, SpinorPtr in, int prec_out, SpinorPtr out) {
    DArgs a = base_args(op, out_parity);
    a.in = in;
    a.out = out;
    if (prec_in == P64 && prec_out == P64) launch_dslash<M_HOP, P64, P64, P64, P64, 0>(c, op, a);
    else if (prec_in == P32 && prec_out == P32) launch_dslash<M_HOP, P32, P32, P32, P32, 0>(c, op, a);
    else if (prec_in == P16 && prec_out == P16) launch_dslash<M_HOP, P16, P16, P16, P32, 0>(c, op, a);
    else throw Error(-1, "dslash: unsupported precision pair");
}

void mhat(Ctx& c, const FermionOp& op, int prec, SpinorPtr in_e, SpinorPtr tmp_o, SpinorPtr out_e, int dagger) {
    if (prec != P64) throw Error(-1, "mhat: FP64 only");
    DArgs a = base_args(op, 1);
    a.in = in_e;
    a.out = tmp_o;
    if (dagger) launch_dslash<M_HOP, P64, P64, P64, P64, 1>(c, op, a);
    else launch_dslash<M_HOP, P64, P64, P64, P64, 0>(c, op, a);
    DArgs b = base_args(op, 0);
    b.in = tmp_o;
    b.center = in_e;
    b.out = out_e;
    b.g5out = dagger;
    launch_dslash<M_SCHUR, P64, P64, P64, P64, 0>(c, op, b);
}

void pf_heatbath(Ctx& c, const FermionOp& op64, const d2* eta, d2* phi) {
    d2* t = (d2*)c.tmp_o.get(sizeof(d2) * 12 * (size_t)op64.g->Vh);
    mhat(c, op64, P64, sp(eta), sp(t), sp(phi), 1);
}

void spinor_copy(Ctx& c, const Geom& g, const d2* src, d2* dst) {
    FGI_HIP(hipMemcpyAsync(dst, src, sizeof(d2) * 12 * (size_t)g.Vh, hipMemcpyDeviceToDevice, c.stream));
}

int pf_density_partials(Ctx& c, const Geom& g, const d2* phi, const d2* X, const d2* eta, double* partial) {
    int nb = nblk(g.Vh, DBS);
    hipLaunchKernelGGL(k_pf_density, dim3(nb), dim3(DBS), 0, c.stream, g.Vh, phi, X, eta, partial);
    FGI_LAUNCH_CHECK();
    return nb;
}

// F += coef * TA(U C(X, Y)) with X = (X_e, D_oe X_e), Y = (Y_e, g5 D_oe g5 Y_e):
// the derivative -d/dt of 2 Re[Y^+ D X] / 2 per link (coef carries the kappas)
void fermion_force_xy(Ctx& c, const FermionOp& op64, const d2* Xe, const d2* Ye, double* F, double coef) {
    const Geom& g = *op64.g;
    size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    d2* Xo = (d2*)c.Xo.get(n);
    d2* Yo = (d2*)c.Yo.get(n);
    dslash(c, op64, 1, P64, sp(Xe), P64, sp(Xo));          // X_o = D_oe X_e
    {                                                       // Y_o = g5 D_oe g5 Y_e
        DArgs a = base_args(op64, 1);
        a.in = sp(Ye);
        a.out = sp(Yo);
        a.g5out = 1;
        launch_dslash<M_HOP, P64, P64, P64, P64, 1>(c, op64, a);
    }
    hipLaunchKernelGGL(k_fermion_force, dim3(slab_blocks(g.Vh, 2, 256, c.ds_xcd)), dim3(256), 0, c.stream, g,
                       (const d2*)op64.links, sp(Xe), sp(Xo), sp(Ye), sp(Yo), coef, F, c.ds_xcd);
    FGI_LAUNCH_CHECK();
}

// pseudofermion force of phi^+ (Mhat^+ Mhat)^-1 phi at op64.kappa: Y_e = Mhat X_e
void fermion_force(Ctx& c, const FermionOp& op64, const d2* Xe, double* F, double coef) {
    const Geom& g = *op64.g;
    size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    d2* Ye = (d2*)c.Ye.get(n);
    d2* t = (d2*)c.tmp_o.get(n);
    mhat(c, op64, P64, sp(Xe), sp(t), sp(Ye), 0);
    fermion_force_xy(c, op64, Xe, Ye, F, coef * op64.kappa * op64.kappa);
}

// ------------------------------------------------ force gradient (Section 4) ---
// J_V[F_F] = d/dt F_F(exp(tV) U) for S = phi^+ A^-1 phi, A = Mhat^+ Mhat.
// With dD the hopping term on the tangent links V U (opW):
//   dMhat = -kappa^2 (dD_eo D_oe + D_eo dD_oe),
//   Z = d_V X_e = -A^-1 (dMhat^+ Y_e + Mhat^+ dMhat X_e),   Y_e = Mhat X_e,
//   dX = (Z, dD_oe X_e + D_oe Z),
//   dY = (dMhat X_e + Mhat Z, g5 dD_oe g5 Y_e + g5 D_oe g5 dY_e),
//   J += coef kappa^2 bc TA(U [C(dX, Y) + C(X, dY)] + V U C(X, Y)).
namespace {
void lincomb(Ctx& c, const Geom& g, double a, const d2* x, double b, const d2* y, int g5y, d2* out) {
    hipLaunchKernelGGL(k_sp_lincomb, dim3(nblk(g.Vh, DBS)), dim3(DBS), 0, c.stream, g.Vh, a, x, b, y, g5y, out);
    FGI_LAUNCH_CHECK();
}
// out_o = [g5] D_oe g5 in_e  (the odd half of the Y vectors)
void hop_g5(Ctx& c, const FermionOp& op, const d2* in, d2* out, int g5out) {
    DArgs a = base_args(op, 1);
    a.in = sp(in);
    a.out = sp(out);
    a.g5out = g5out;
    launch_dslash<M_HOP, P64, P64, P64, P64, 1>(c, op, a);
}
}  // namespace

void fermion_tangent_rhs(Ctx& c, const FermionOp& op64, const FermionOp& opW, const d2* Xe, d2* rhs) {
    const Geom& g = *op64.g;
    const size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    const double k2 = op64.kappa * op64.kappa;
    d2 *Ye = (d2*)c.Ye.get(n), *Yo = (d2*)c.Yo.get(n), *Xo = (d2*)c.Xo.get(n);
    d2 *to = (d2*)c.tmp_o.get(n), *te = (d2*)c.tmp_e.get(n);
    d2 *dmx = (d2*)c.tg_dmx.get(n), *dxo = (d2*)c.tg_dxo.get(n), *dye = (d2*)c.tg_dye.get(n);
    d2* dyo = (d2*)c.tg_dyo.get(n);
    mhat(c, op64, P64, sp(Xe), sp(to), sp(Ye), 0);            // Y_e = Mhat X_e
    dslash(c, op64, 1, P64, sp(Xe), P64, sp(Xo));             // X_o = D_oe X_e
    hop_g5(c, op64, Ye, Yo, 1);                                // Y_o = g5 D_oe g5 Y_e
    // dMhat X_e = -kappa^2 (dD_eo X_o + D_eo dD_oe X_e)
    dslash(c, opW, 1, P64, sp(Xe), P64, sp(dxo));             // dD_oe X_e (first part of dX_o)
    dslash(c, op64, 0, P64, sp(dxo), P64, sp(te));
    dslash(c, opW, 0, P64, sp(Xo), P64, sp(dmx));
    lincomb(c, g, -k2, te, -k2, dmx, 0, dmx);
    // dMhat^+ Y_e = -kappa^2 g5 (dD_eo D_oe g5 Y_e + D_eo dD_oe g5 Y_e), with D_oe g5 Y_e = g5 Y_o
    hop_g5(c, opW, Ye, dyo, 0);                                // dD_oe g5 Y_e (g5 of it: first part of dY_o)
    dslash(c, op64, 0, P64, sp(dyo), P64, sp(dye));            // D_eo dD_oe g5 Y_e
    {
        DArgs a = base_args(opW, 0);                           // dD_eo g5 Y_o
        a.in = sp(Yo);
        a.out = sp(te);
        launch_dslash<M_HOP, P64, P64, P64, P64, 1>(c, opW, a);
    }
    lincomb(c, g, 1.0, te, 1.0, dye, 0, te);
    mhat(c, op64, P64, sp(dmx), sp(to), sp(rhs), 1);          // Mhat^+ dMhat X_e
    lincomb(c, g, -1.0, rhs, k2, te, 1, rhs);                  // -(Mhat^+ dMhat X_e + dMhat^+ Y_e)
}

void fermion_force_tangent(Ctx& c, const FermionOp& op64, const FermionOp& opW, const double* Vd, const d2* Xe,
                           const d2* Z, double* J, double coef) {
    const Geom& g = *op64.g;
    const size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    d2 *Ye = (d2*)c.Ye.get(n), *Yo = (d2*)c.Yo.get(n), *Xo = (d2*)c.Xo.get(n);
    d2* to = (d2*)c.tmp_o.get(n);
    d2 *dmx = (d2*)c.tg_dmx.get(n), *dxo = (d2*)c.tg_dxo.get(n), *dye = (d2*)c.tg_dye.get(n);
    d2* dyo = (d2*)c.tg_dyo.get(n);
    dslash(c, op64, 1, P64, sp(Z), P64, sp(to));               // dX_o = dD_oe X_e + D_oe Z
    lincomb(c, g, 1.0, dxo, 1.0, to, 0, dxo);
    mhat(c, op64, P64, sp(Z), sp(to), sp(dye), 0);             // dY_e = dMhat X_e + Mhat Z
    lincomb(c, g, 1.0, dye, 1.0, dmx, 0, dye);
    hop_g5(c, op64, dye, to, 1);                               // dY_o = g5 D_oe g5 dY_e + g5 dD_oe g5 Y_e
    lincomb(c, g, 1.0, to, 1.0, dyo, 1, dyo);
    hipLaunchKernelGGL(k_fermion_force_tangent, dim3(slab_blocks(g.Vh, 2, 256, c.ds_xcd)), dim3(256), 0, c.stream, g,
                       (const d2*)op64.links, Vd, sp(Xe), sp(Xo), sp(Ye), sp(Yo), sp(Z), sp(dxo), sp(dye), sp(dyo),
                       coef * op64.kappa * op64.kappa, J, c.ds_xcd);
    FGI_LAUNCH_CHECK();
}

static void zero_spinor(Ctx& c, const Geom& g, void* v, int prec);

// d_V chi for chi = Mhat^+ phi at op64.kappa: out_e = dMhat^+ in_e =
// -kappa^2 g5 (dD_eo D_oe + D_eo dD_oe) g5 in_e, dD the hopping term on the
// tangent links of opW (uses tmp_o, tmp_e and the hs_t1 scratch)
void dmhat_dag_apply(Ctx& c, const FermionOp& op64, const FermionOp& opW, const d2* in_e, d2* out_e) {
    const Geom& g = *op64.g;
    const size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    const double k2 = op64.kappa * op64.kappa;
    d2 *to = (d2*)c.tmp_o.get(n), *te = (d2*)c.tmp_e.get(n), *t1 = (d2*)c.hs_t1.get(n);
    hop_g5(c, op64, in_e, to, 0);                              // D_oe g5 in
    {
        DArgs a = base_args(opW, 0);                           // dD_eo D_oe g5 in
        a.in = sp(to);
        a.out = sp(te);
        launch_dslash<M_HOP, P64, P64, P64, P64, 0>(c, opW, a);
    }
    hop_g5(c, opW, in_e, t1, 0);                               // dD_oe g5 in
    dslash(c, op64, 0, P64, sp(t1), P64, sp(out_e));           // D_eo dD_oe g5 in
    lincomb(c, g, 0.0, out_e, -k2, te, 0, te);                 // -k2 dD_eo D_oe g5 in
    lincomb(c, g, -k2, out_e, 1.0, te, 0, out_e);              // -k2 (... + D_eo dD_oe g5 in)
    lincomb(c, g, 0.0, out_e, 1.0, out_e, 1, out_e);           // g5
}

// J += coef bc TA(U [C(dX, Y) + C(X, dY)] + V U C(X, Y)) for the bilinear force
// of fermion_force_xy with X = (X_e, D_oe X_e), Y = (Y_e, g5 D_oe g5 Y_e), when
// X_e moves by dX_e and Y_e is fixed: dX = (dX_e, dD_oe X_e + D_oe dX_e),
// dY = (0, g5 dD_oe g5 Y_e)
void fermion_force_xy_tangent(Ctx& c, const FermionOp& op64, const FermionOp& opW, const double* Vd, const d2* Xe,
                              const d2* Ye, const d2* dXe, double* J, double coef) {
    const Geom& g = *op64.g;
    const size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    d2 *xo = (d2*)c.hs_xo.get(n), *yo = (d2*)c.hs_yo.get(n), *dxo = (d2*)c.hs_dxo.get(n);
    d2 *dyo = (d2*)c.hs_dyo.get(n), *zero = (d2*)c.hs_zero.get(n), *t1 = (d2*)c.hs_t1.get(n);
    zero_spinor(c, g, zero, P64);
    dslash(c, op64, 1, P64, sp(Xe), P64, sp(xo));               // X_o = D_oe X_e
    hop_g5(c, op64, Ye, yo, 1);                                 // Y_o = g5 D_oe g5 Y_e
    dslash(c, opW, 1, P64, sp(Xe), P64, sp(dxo));               // dD_oe X_e
    dslash(c, op64, 1, P64, sp(dXe), P64, sp(t1));              // + D_oe dX_e
    lincomb(c, g, 1.0, dxo, 1.0, t1, 0, dxo);
    hop_g5(c, opW, Ye, dyo, 1);                                 // dY_o = g5 dD_oe g5 Y_e
    hipLaunchKernelGGL(k_fermion_force_tangent, dim3(slab_blocks(g.Vh, 2, 256, c.ds_xcd)), dim3(256), 0, c.stream, g,
                       (const d2*)op64.links, Vd, sp(Xe), sp(xo), sp(Ye), sp(yo), sp(dXe), sp(dxo), sp(zero), sp(dyo),
                       coef, J, c.ds_xcd);
    FGI_LAUNCH_CHECK();
}

void spinor_lincomb(Ctx& c, const Geom& g, double a, const d2* x, double b, const d2* y, int g5y, d2* out) {
    lincomb(c, g, a, x, b, y, g5y, out);
}

// F += coef * TA(U C(X, Y)) for given odd halves X_o, Y_o (operators whose odd
// reconstruction is not D_oe alone)
void fermion_force_xyo(Ctx& c, const FermionOp& op64, const d2* Xe, const d2* Xo, const d2* Ye, const d2* Yo,
                       double* F, double coef) {
    const Geom& g = *op64.g;
    hipLaunchKernelGGL(k_fermion_force, dim3(slab_blocks(g.Vh, 2, 256, c.ds_xcd)), dim3(256), 0, c.stream, g,
                       (const d2*)op64.links, sp(Xe), sp(Xo), sp(Ye), sp(Yo), coef, F, c.ds_xcd);
    FGI_LAUNCH_CHECK();
}

// out_o = [g5] A_oo^-1 D_oe g5 in_e (FP64; no A_oo^-1 without op64.blk)
void hop_oe_g5(Ctx& c, const FermionOp& op64, const d2* in_e, d2* out_o, int g5out) { hop_g5(c, op64, in_e, out_o, g5out); }

// ---------------------------------------------------------------- CG ------
// |v|^2 into the device scalar out
static void norm2(Ctx& c, const Geom& g, const d2* v, double* out) {
    double* part = partial_buf(c, g);
    int nb = nblk(g.Vh, DBS);
    hipLaunchKernelGGL(k_norm2_partials, dim3(nb), dim3(DBS), 0, c.stream, g.Vh, v, part);
    FGI_LAUNCH_CHECK();
    final_sum(c, part, nb, out);
}

// r = phi - Mhat^+ Mhat X in FP64, stored in r's precision PR, and its |r|^2
// partials (returns their number); x0: a vector of the same precision to clear
template <int PR>
static int true_residual(Ctx& c, const FermionOp& op64, const d2* phi, const d2* X, SpinorPtr r, SpinorPtr x0) {
    const Geom& g = *op64.g;
    size_t n = sizeof(d2) * 12 * (size_t)g.Vh;
    d2* t = (d2*)c.tmp_o.get(n);
    d2* q = (d2*)c.cg_q.get(n);
    mhat(c, op64, P64, sp(X), sp(t), sp(q), 0);  // q = Mhat X
    DArgs a = base_args(op64, 1);                // t = D_oe g5 q
    a.in = sp(q);
    a.out = sp(t);
    launch_dslash<M_HOP, P64, P64, P64, P64, 1>(c, op64, a);
    DArgs b = base_args(op64, 0);                // r = phi - (q - k^2 g5 D_eo t)
    b.in = sp(t);
    b.center = sp(q);
    b.aux = sp(phi);
    b.out = r;
    b.x = x0;
    b.g5out = 1;
    b.partial = partial_buf(c, g);
    launch_dslash<M_RESID, P64, P64, PR, P64, 0>(c, op64, b);
    return ds_blocks(c, g.Vh);
}

struct CGVecs {
    SpinorPtr x, r, p, q, t;  // x, r in PX; p, q, t in PP
    SpinorPtr pf, sf, rt;     // Chronopoulos-Gear form: p, s = A p in PX; rt, the hops' r, in PP (r itself if PP = PX)
};

// One CG iteration on A = Mhat^+ Mhat: a direction update and four
// Dslash-shaped kernels; the iteration index is st->base + j so a captured
// batch can be replayed.
//   rr = sum of the previous |r|^2 partials, beta, stop test; p = r + beta p
//   t = D_oe p
//   q = p - k^2 D_eo t; |q|^2 partials
//   t = D_oe g5 q; pAp = sum of the |q|^2 partials  [one extra block]
//   Ap = q - k^2 g5 D_eo t; x += alpha p; r -= alpha Ap; |r|^2 partials
// Each reduction's partials are consumed by the next kernel that reads them,
// before the next reduction writes, so one buffer serves both.
template <int PP, int PX>
static void cg_iteration(Ctx& c, const FermionOp& ops, const CGVecs& v, int j) {
    CGState* st = dev_state(c);
    double* part = partial_buf(c, *ops.g);
    const int Vh = ops.g->Vh;
    if (site_split(c, Vh))
        hipLaunchKernelGGL((k_cg_p_split<PP, PX>), dim3(ds_blocks(c, Vh)), dim3(256), 0, c.stream, Vh, v.p, v.r, st,
                           (const double*)part, c.ds_xcd, j);
    else
        hipLaunchKernelGGL((k_cg_p<PP, PX>), dim3(nblk(Vh, c.ds_bs)), dim3(c.ds_bs), 0, c.stream, Vh, v.p, v.r, st,
                           (const double*)part, nblk(Vh, c.ds_bs), c.ds_xcd, j);
    FGI_LAUNCH_CHECK();
    {
        DArgs a = base_args(ops, 1);
        a.in = v.p;
        a.out = v.t;
        a.st = st;
        a.iter = j;
        launch_dslash<M_HOP, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = v.p;
        a.out = v.q;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_CGQ, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 1);
        a.in = v.q;
        a.out = v.t;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_HOP, PP, PP, PP, PX, 1>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = v.q;
        a.aux = v.p;
        a.x = v.x;
        a.r = v.r;
        a.g5out = 1;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_CGX, PP, PP, PP, PX, 0>(c, ops, a);
    }
}

// One iteration in the Chronopoulos-Gear form: four Dslash-shaped kernels.
//   t = D_oe rt; rr, beta and the <p, A p> correction from the partials  [one extra block]
//   q = rt - k^2 D_eo t; |q|^2 partials
//   t = D_oe g5 q; |q|^2 summed into pAp  [one extra block]
//   w = q - k^2 g5 D_eo t; p = rt + beta p; s = w + beta s; x += alpha p; r -= alpha s;
//   rt; |r|^2, Re<rt, s>, Re<p, s> partials
template <int PP, int PX>
static void cg_iteration_cgs(Ctx& c, const FermionOp& ops, const CGVecs& v, int j) {
    CGState* st = dev_state(c);
    double* part = partial_buf(c, *ops.g);
    {
        DArgs a = base_args(ops, 1);
        a.in = v.rt;
        a.out = v.t;
        a.partial = part;
        a.cgs = 1;
        a.st = st;
        a.iter = j;
        launch_dslash<M_HOP, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = v.rt;
        a.out = v.q;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_CGQ, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 1);
        a.in = v.q;
        a.out = v.t;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_HOP, PP, PP, PP, PX, 1>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = v.q;
        a.aux = v.rt;
        a.x = v.x;
        a.r = v.r;
        a.dir = v.pf;
        a.adir = v.sf;
        a.g5out = 1;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash<M_CGS, PP, PP, PP, PX, 0>(c, ops, a);
    }
}

// the M_CGS partials of the vectors as they stand (start of a run, reliable update)
template <int PP, int PX>
static void cgs_partials(Ctx& c, const Geom& g, const CGVecs& v) {
    hipLaunchKernelGGL((k_cgs_partials<PP, PX>), dim3(ds_blocks(c, g.Vh)), dim3(ds_sites(c, g.Vh)), 0, c.stream, g.Vh, v.r,
                       v.rt, v.pf, v.sf, partial_buf(c, g));
    FGI_LAUNCH_CHECK();
}

// B iterations then the batch's closing reduction and base += B, on c.stream
template <int PP, int PX>
static void cg_batch_eager(Ctx& c, const FermionOp& ops, const CGVecs& v, int B) {
    for (int j = 0; j < B; j++) {
        if (c.cg_form && !ops.blk) cg_iteration_cgs<PP, PX>(c, ops, v, j);
        else cg_iteration<PP, PX>(c, ops, v, j);
    }
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(DBS), 0, c.stream, dev_state(c), (const double*)partial_buf(c, *ops.g),
                       ds_blocks(c, ops.g->Vh), B, c.host_state);
    FGI_LAUNCH_CHECK();
}

// N bare hops t = D_oe g5 q on the solve's live operator and vectors (the
// sample that times the Dslash kernel; t is scratch, q is only read)
template <int PP, int PX>
static void hop_sample_eager(Ctx& c, const FermionOp& ops, const CGVecs& v, int N) {
    for (int j = 0; j < N; j++) {
        DArgs a = base_args(ops, 1);
        a.in = v.q;
        a.out = v.t;
        launch_dslash<M_HOP, PP, PP, PP, PX, 1>(c, ops, a);
    }
}

// Capture `body` on the private capture stream into an instantiated graph,
// cached under `key`.
template <typename Body>
static GraphEntry& cached_graph(Ctx& c, const std::string& key, Body body) {
    for (auto& e : c.graphs)
        if (e.key == key) return e;
    if (!c.cap_stream) FGI_HIP(hipStreamCreateWithFlags(&c.cap_stream, hipStreamNonBlocking));
    if (c.graphs.size() >= 24) {
        hipGraphExecDestroy(c.graphs.front().exec);
        c.graphs.erase(c.graphs.begin());
    }
    GraphEntry e;
    e.key = key;
    hipStream_t saved = c.stream;
    c.stream = c.cap_stream;
    hipGraph_t graph = nullptr;
    try {
        FGI_HIP(hipStreamBeginCapture(c.cap_stream, hipStreamCaptureModeRelaxed));
        body();
        FGI_HIP(hipStreamEndCapture(c.cap_stream, &graph));
        FGI_HIP(hipGraphInstantiate(&e.exec, graph, nullptr, nullptr, 0));
        FGI_HIP(hipGraphDestroy(graph));
    } catch (...) {
        c.stream = saved;
        hipStreamEndCapture(c.cap_stream, &graph);
        if (graph) hipGraphDestroy(graph);
        throw;
    }
    c.stream = saved;
    c.graphs.push_back(e);
    c.graph_captures++;
    return c.graphs.back();
}

template <int PP, int PX>
static std::string graph_key(const char* what, Ctx& c, const FermionOp& ops, const CGVecs& v, int n) {
    char key[512];
    snprintf(key, sizeof key, "%s/%d/%d/%p/%p/%.17g/%d/%d/%d/%d/%d/%d/%d/%p/%p/%p/%p/%p/%p/%p/%p/%d/%d/%d/%d/%p/%p/%p/%p",
             what, PP, PX, ops.links, ops.blk, ops.kappa, ops.prec, ops.recon, ops.g->L[0], ops.g->L[1], ops.g->L[2],
             ops.g->L[3], ops.g->Vh, v.x.v, v.r.v, v.p.v, v.q.v, v.t.v, (void*)v.p.norm, (void*)dev_state(c),
             (void*)partial_buf(c, *ops.g), n, c.ds_bs, c.ds_xcd, c.cg_form, v.pf.v, v.sf.v, v.rt.v,
             (void*)v.rt.norm);
    return key;
}

template <int PA, int PB>
static void convert(Ctx& c, const Geom& g, SpinorPtr a, SpinorPtr b) {
    hipLaunchKernelGGL((k_convert<PA, PB>), dim3(nblk(g.Vh, DBS)), dim3(DBS), 0, c.stream, g.Vh, a, b);
    FGI_LAUNCH_CHECK();
}

void convert_spinor(Ctx& c, const Geom& g, int pa, SpinorPtr a, int pb, SpinorPtr b) {
    if (pa == P64 && pb == P32) convert<P64, P32>(c, g, a, b);
    else if (pa == P64 && pb == P16) convert<P64, P16>(c, g, a, b);
    else if (pa == P32 && pb == P64) convert<P32, P64>(c, g, a, b);
    else if (pa == P16 && pb == P64) convert<P16, P64>(c, g, a, b);
    else if (pa == P64 && pb == P64) convert<P64, P64>(c, g, a, b);
    else throw Error(-1, "convert_spinor: unsupported pair");
}

static void zero_spinor(Ctx& c, const Geom& g, void* v, int prec) {
    size_t n = prec == P64 ? 24 * (size_t)g.Vh : (prec == P32 ? 12 * (size_t)g.Vh : 0);
    if (prec == P16) throw Error(-1, "zero_spinor: FP16");
    hipLaunchKernelGGL(k_zero, dim3(nblk((long)n, 256)), dim3(256), 0, c.stream, n, (double*)v);
    FGI_LAUNCH_CHECK();
}

// s = A p at a reliable update of the Chronopoulos-Gear form, from p as the
// hops read it: with FP16 hops p is first rounded to FP16 storage (in q) and
// kept that way, so s stays the image of the p that x is moved along.
template <int PP, int PX>
static void cgs_refresh_s(Ctx& c, const FermionOp& ops, const CGVecs& v) {
    const Geom& g = *ops.g;
    SpinorPtr pin = v.pf;
    if constexpr (PP != PX) {
        convert<PX, PP>(c, g, v.pf, v.q);
        convert<PP, PX>(c, g, v.q, v.pf);
        pin = v.q;
    }
    {
        DArgs a = base_args(ops, 1);
        a.in = pin;
        a.out = v.t;
        launch_dslash<M_HOP, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = pin;
        a.out = v.q;   // M pin, in place when pin is q (each site reads only its own centre)
        launch_dslash<M_SCHUR, PP, PP, PP, PX, 0>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 1);
        a.in = v.q;
        a.out = v.t;
        launch_dslash<M_HOP, PP, PP, PP, PX, 1>(c, ops, a);
    }
    {
        DArgs a = base_args(ops, 0);
        a.in = v.t;
        a.center = v.q;
        a.out = v.sf;
        a.g5out = 1;
        launch_dslash<M_SCHUR, PP, PP, PX, PX, 0>(c, ops, a);
    }
}

// guess: X holds the starting point on entry (else CG starts from zero); the
// run then begins like a reliable update, from the true residual phi - A X,
// and stops on |phi - A X| <= tol |phi| as always.
template <int PP, int PX>
static CGResult cg_run(Ctx& c, const FermionOp& op64, const FermionOp& ops, const d2* phi, d2* X, double tol,
                       int maxiter, bool guess) {
    const Geom& g = *op64.g;
    const size_t n64 = sizeof(d2) * 12 * (size_t)g.Vh;
    CGResult res{0, 0, 0.0, 0};
    CGState* st = dev_state(c);
    double* scal = (double*)c.scal.get(sizeof(double) * 64);
    norm2(c, g, phi, scal);
    const double drop = ru_drop(c, PP);
    const CGRun run{tol * tol, PX == P64 ? 0.0 : drop * drop, scal, c.host_scal, maxiter, c.cg_batch};
    d2* r64 = (d2*)c.cg_r.get(n64);
    auto start = [&](const double* part, int nb) {
        hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(DBS), 0, c.stream, st, run, part, nb);
        FGI_LAUNCH_CHECK();
    };
    if (guess) {
        const int nb = true_residual<P64>(c, op64, phi, X, sp(r64), SpinorPtr{});
        start(partial_buf(c, g), nb);
    } else {
        zero_spinor(c, g, X, P64);
        start(nullptr, 0);
    }
    const d2* r_start = guess ? r64 : phi;
    CGVecs v{};   // every field null until set: the graph key reads them all
    float* norms = (float*)c.s_norms.get(sizeof(float) * 4 * (size_t)g.Vh);
    if (PX == P64) {
        if (!guess) spinor_copy(c, g, phi, r64);
        v.x = sp(X);
        v.r = sp(r64);
        v.p = sp(c.cg_p.get(n64));
        v.q = sp(c.cg_q.get(n64));
        v.t = sp(c.s_t.get(n64));
        spinor_copy(c, g, r_start, (d2*)v.p.v);
    } else {
        size_t nx = sizeof(float) * 24 * (size_t)g.Vh;
        size_t np = PP == P32 ? nx : sizeof(_Float16) * 24 * (size_t)g.Vh;
        v.x = sp(c.s_x.get(nx));
        v.r = sp(c.s_r.get(nx));
        v.p = sp(c.s_p.get(np), norms);
        v.q = sp(c.s_q.get(np), norms + g.Vh);
        v.t = sp(c.s_t.get(np), norms + 2 * (size_t)g.Vh);
        zero_spinor(c, g, v.x.v, P32);
        convert<P64, PX>(c, g, sp(r_start), v.r);
        convert<P64, PP>(c, g, sp(r_start), v.p);
    }
    partial_buf(c, g);  // allocate before any capture
    const bool cgs = c.cg_form != 0 && !ops.blk;
    if (cgs) {  // Chronopoulos-Gear form: p = s = 0, rt = r, and the partials its first iteration sums
        const size_t nx = PX == P64 ? n64 : sizeof(float) * 24 * (size_t)g.Vh;
        v.pf = sp(c.s_pf.get(nx));
        v.sf = sp(c.s_sf.get(nx));
        zero_spinor(c, g, v.pf.v, PX);
        zero_spinor(c, g, v.sf.v, PX);
        if constexpr (PP == PX) {
            v.rt = v.r;
        } else {
            v.rt = sp(c.s_rt.get(sizeof(_Float16) * 24 * (size_t)g.Vh), norms + 3 * (size_t)g.Vh);
            convert<PX, PP>(c, g, v.r, v.rt);
        }
        cgs_partials<PP, PX>(c, g, v);
    }
    const bool prof = c.profile && (c.profile_prec < 0 || c.profile_prec == PP);
    const int B = c.cg_batch;
    GraphEntry* ge = nullptr;
    if (c.use_graphs)
        ge = &cached_graph(c, graph_key<PP, PX>("cg", c, ops, v, B), [&] { cg_batch_eager<PP, PX>(c, ops, v, B); });
    // The host launches as many iterations as the decay of |r|^2 so far says the
    // inner run still needs, then waits once for the state that k_advance leaves
    // in pinned memory; a run whose end is not the solve's goes on from its true
    // residual without the host (k_cg_restart).  Fixed batches of 8 left a third
    // of the launches empty where a run takes ten iterations, and each run
    // waited twice.  The iterates do not depend on the counts.
    int k = 0, base0 = 0;   // iterations launched so far; start of the current inner run
    const int whole = op64.blk ? 1 : B;
    int kcap = cg_cut(0, maxiter, whole);   // where an unfinished run is cut off
    int n = std::min(std::min(B, 8), kcap);
    double rr_first = 0.0;
    const bool fp64_next = PX != P64 && op64.blk;   // the caller goes on in FP64 (clover_cg_mp)
    auto broken = [&](CGBreak how) {
        res.broke = how;
        return res;
    };
    for (;;) {
        for (int left = n; left > 0;) {
            const int m = std::min(left, B);
            if (ge && m == B) FGI_HIP(hipGraphLaunch(ge->exec, c.stream));
            else cg_batch_eager<PP, PX>(c, ops, v, m);
            left -= m;
        }
        FGI_HIP(hipStreamSynchronize(c.stream));
        const CGState hs = *c.host_state;
        const double bb = c.host_scal[0], rr_true = c.host_scal[1], target = tol * tol * bb;
        if (!std::isfinite(rr_true)) {
            if (base0 && fp64_next) return broken(CG_BROKE_LOST);
            throw Error(-4, guess && !base0 ? "CG: non-finite residual of the starting point" : "CG: non-finite residual");
        }
        if (bb == 0.0) {   // phi = 0: the solution is 0, whatever the start
            if (guess) zero_spinor(c, g, X, P64);
            res.converged = 1;
            return res;
        }
        if ((guess || base0) && rr_true <= target) {   // the last true residual was there already
            res.converged = 1;
            res.rel_resid = std::sqrt(rr_true / bb);
            if (!base0) return res;
            res.reliable_updates--;
            break;
        }
        if (rr_first == 0.0) rr_first = rr_true;
        const int kend = hs.stop_at <= k + n ? hs.stop_at : k + n;
        const bool inner_done = hs.stop_at <= kend;
        k = kend;
        const double now = hs.rr[kend & 1];
        if (!std::isfinite(now)) {
            res.iters = kend;
            res.rel_resid = std::sqrt(rr_true / bb);   // X is as the last true residual found it
            if (fp64_next) return broken(CG_BROKE_KEPT);
            throw Error(-4, "CG: non-finite residual");
        }
        double stop = hs.rr_stop;
        if (inner_done || kend >= kcap) {
            if (PX != P64) {
                hipLaunchKernelGGL((k_add_to64<PX>), dim3(nblk(g.Vh, DBS)), dim3(DBS), 0, c.stream, g.Vh, v.x, sp(X));
                FGI_LAUNCH_CHECK();
            }
            // reliable update: continue from the true residual, keep the direction
            const int nb = true_residual<PX>(c, op64, phi, X, v.r, PX == P64 ? SpinorPtr{} : v.x);
            hipLaunchKernelGGL(k_cg_restart, dim3(1), dim3(DBS), 0, c.stream, st, run,
                               (const double*)partial_buf(c, g), nb, kend);
            FGI_LAUNCH_CHECK();
            res.iters = kend;
            if (stop <= target || kend >= maxiter) {   // the solve should end here: look before launching more
                FGI_HIP(hipStreamSynchronize(c.stream));
                const double rr = c.host_scal[1];
                res.rel_resid = std::sqrt(rr / bb);
                if (!std::isfinite(rr)) {
                    if (fp64_next) return broken(CG_BROKE_LOST);
                    throw Error(-4, "CG: non-finite residual");
                }
                if (rr <= target) {
                    res.converged = 1;
                    break;
                }
                if (kend >= maxiter) break;
            }
            res.reliable_updates++;
            if (cgs) {  // the hops' copy of the new r, s = A p afresh, and the partials
                if constexpr (PP != PX) convert<PX, PP>(c, g, v.r, v.rt);
                cgs_refresh_s<PP, PX>(c, ops, v);
                cgs_partials<PP, PX>(c, g, v);
            }
            base0 = kend;
            kcap = cg_cut(kend, maxiter, whole);
            stop = std::max(run.ru2 * now, target);
        }
        const double need = std::log(stop / now) / (std::log(now / rr_first) / kend);
        n = !(need > 0.0) || need > 1e6 ? B : need > 12.0 ? (int)std::min(0.9 * need, 64.0) : (int)std::ceil(need);
        n = std::min(n, kcap - k);
    }
    if (prof) {
        // live sample of the bare hop: N back-to-back launches between two events
        const int N = 16;
        if (c.ev_pool.empty()) {
            for (int i = 0; i < 2; i++) {
                hipEvent_t e;
                FGI_HIP(hipEventCreate(&e));
                c.ev_pool.push_back(e);
            }
        }
        GraphEntry* hg = nullptr;
        if (c.use_graphs)
            hg = &cached_graph(c, graph_key<PP, PX>("hop", c, ops, v, N), [&] { hop_sample_eager<PP, PX>(c, ops, v, N); });
        FGI_HIP(hipEventRecord(c.ev_pool[0], c.stream));
        if (hg) FGI_HIP(hipGraphLaunch(hg->exec, c.stream));
        else hop_sample_eager<PP, PX>(c, ops, v, N);
        FGI_HIP(hipEventRecord(c.ev_pool[1], c.stream));
        FGI_HIP(hipEventSynchronize(c.ev_pool[1]));
        float ms = 0.f;
        FGI_HIP(hipEventElapsedTime(&ms, c.ev_pool[0], c.ev_pool[1]));
        c.dslash_ms += ms;
        c.dslash_launches += N;
        c.dslash_sites += (long)N * g.Vh;
    }
    return res;
}

// ====================================================== batched chains ======
template <int MODE, int PIN, int PC, int POUT, int PX, int PL, int RECON, int G5IN>
static void launch_dslash_b_rec(Ctx& c, const Batch& B, DArgs& a) {
    // an M_HOP inside CG (states and partials) carries one pAp reduction block per chain
    const bool red = MODE == M_HOP && a.st && a.partial;
    for (int k = 0; k < 2; k++) {
        const int nsb = B.ds_blk[k];
        if (!nsb) continue;
        const dim3 nb(nsb + (red ? B.ds_nc[k] : 0));
        if (k == DS_SPLIT)
            hipLaunchKernelGGL((k_dslash_split_b<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN>), nb, dim3(256), 0,
                               c.stream, a, B.cd, B.ds_map[k], nsb);
        else
            hipLaunchKernelGGL((k_dslash_b<MODE, PIN, PC, POUT, PX, PL, RECON, G5IN>), nb, dim3(c.ds_bs), 0, c.stream,
                               a, B.cd, B.ds_map[k], nsb);
    }
}

template <int MODE, int PIN, int PC, int POUT, int PX, int G5IN>
static void launch_dslash_b(Ctx& c, const Batch& B, const FermionOp& op, DArgs& a) {
    a.xcd = c.ds_xcd;
    if constexpr (PIN == P64) {
        launch_dslash_b_rec<MODE, PIN, PC, POUT, PX, P64, 18, G5IN>(c, B, a);
    } else {
        if (op.prec == P32 && op.recon == 18) launch_dslash_b_rec<MODE, PIN, PC, POUT, PX, P32, 18, G5IN>(c, B, a);
        else if (op.prec == P32) launch_dslash_b_rec<MODE, PIN, PC, POUT, PX, P32, 12, G5IN>(c, B, a);
        else if (op.recon == 18) launch_dslash_b_rec<MODE, PIN, PC, POUT, PX, P16, 18, G5IN>(c, B, a);
        else launch_dslash_b_rec<MODE, PIN, PC, POUT, PX, P16, 12, G5IN>(c, B, a);
    }
    FGI_LAUNCH_CHECK();
}

static DArgs base_args_b(const FermionOp& op, int p_out) {
    DArgs a{};
    a.p_out = p_out;
    a.links = op.links;
    return a;
}

#define FGI_B_LAUNCH(kernel, grid) \
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(DBS), 0, c.stream

// out = Mhat in (dagger: Mhat^+) for every chain (gated by st[c].act when st given)
static void mhat_b(Ctx& c, const Batch& B, const FermionOp& op64, const d2* in, d2* tmp, d2* out, int dagger,
                   CGState* st) {
    DArgs a = base_args_b(op64, 1);
    a.in = sp(in);
    a.out = sp(tmp);
    a.st = st;
    a.gate = 1;
    if (dagger) launch_dslash_b<M_HOP, P64, P64, P64, P64, 1>(c, B, op64, a);
    else launch_dslash_b<M_HOP, P64, P64, P64, P64, 0>(c, B, op64, a);
    DArgs b = base_args_b(op64, 0);
    b.in = sp(tmp);
    b.center = sp(in);
    b.out = sp(out);
    b.g5out = dagger;
    b.st = st;
    b.gate = 1;
    launch_dslash_b<M_SCHUR, P64, P64, P64, P64, 0>(c, B, op64, b);
}

void pf_heatbath_b(Ctx& c, const Batch& B, const FermionOp& op64, const d2* eta, d2* phi) {
    d2* t = (d2*)c.tmp_o.get(sizeof(d2) * 12 * (size_t)B.sites);
    mhat_b(c, B, op64, eta, t, phi, 1, nullptr);
}

void fermion_force_b(Ctx& c, const Batch& B, const FermionOp& op64, const d2* Xe, double* F, double coef) {
    size_t n = sizeof(d2) * 12 * (size_t)B.sites;
    d2* Xo = (d2*)c.Xo.get(n);
    d2* Ye = (d2*)c.Ye.get(n);
    d2* Yo = (d2*)c.Yo.get(n);
    d2* t = (d2*)c.tmp_o.get(n);
    {
        DArgs a = base_args_b(op64, 1);
        a.in = sp(Xe);
        a.out = sp(Xo);
        launch_dslash_b<M_HOP, P64, P64, P64, P64, 0>(c, B, op64, a);
    }
    mhat_b(c, B, op64, Xe, t, Ye, 0, nullptr);
    {
        DArgs a = base_args_b(op64, 1);
        a.in = sp(Ye);
        a.out = sp(Yo);
        a.g5out = 1;
        launch_dslash_b<M_HOP, P64, P64, P64, P64, 1>(c, B, op64, a);
    }
    hipLaunchKernelGGL(k_fermion_force_b, dim3(B.nblk[GRID_V]), dim3(256), 0, c.stream, B.cd, B.nc,
                       (const d2*)op64.links, sp(Xe), sp(Xo), sp(Ye), sp(Yo), coef, F);
    FGI_LAUNCH_CHECK();
}

void pf_density_b(Ctx& c, const Batch& B, const d2* phi, const d2* X, const d2* eta, double* partial, double* out) {
    hipLaunchKernelGGL(k_pf_density_b, dim3(B.nblk[GRID_VH]), dim3(DBS), 0, c.stream, B.cd, B.nc, phi, X, eta, partial);
    FGI_LAUNCH_CHECK();
    final_sums_b(c, B, partial, GRID_VH, out);
}

// true_residual for the chains with act set
template <int PR>
static void true_residual_b(Ctx& c, const Batch& B, const FermionOp& op64, const d2* phi, const d2* X, SpinorPtr r,
                            SpinorPtr x0, CGState* st) {
    size_t n = sizeof(d2) * 12 * (size_t)B.sites;
    d2* t = (d2*)c.tmp_o.get(n);
    d2* q = (d2*)c.cg_q.get(n);
    mhat_b(c, B, op64, X, t, q, 0, st);
    DArgs a = base_args_b(op64, 1);
    a.in = sp(q);
    a.out = sp(t);
    a.st = st;
    a.gate = 1;
    launch_dslash_b<M_HOP, P64, P64, P64, P64, 1>(c, B, op64, a);
    DArgs b = base_args_b(op64, 0);
    b.in = sp(t);
    b.center = sp(q);
    b.aux = sp(phi);
    b.out = r;
    b.x = x0;
    b.g5out = 1;
    b.partial = partial_buf(c, B);
    b.st = st;
    b.gate = 1;
    launch_dslash_b<M_RESID, P64, P64, PR, P64, 0>(c, B, op64, b);
}

template <int PP, int PX>
static void cg_iteration_b(Ctx& c, const Batch& B, const FermionOp& ops, const CGVecs& v, int j, CGState* st) {
    double* part = partial_buf(c, B);
    if (B.ds_blk[DS_SPLIT])
        hipLaunchKernelGGL((k_cg_p_split_b<PP, PX>), dim3(B.ds_blk[DS_SPLIT]), dim3(256), 0, c.stream, B.cd,
                           B.ds_map[DS_SPLIT], v.p, v.r, st, (const double*)part, c.ds_xcd, j);
    if (B.ds_blk[DS_PLAIN])
        hipLaunchKernelGGL((k_cg_p_b<PP, PX>), dim3(B.ds_blk[DS_PLAIN]), dim3(c.ds_bs), 0, c.stream, B.cd,
                           B.ds_map[DS_PLAIN], v.p, v.r, st, (const double*)part, c.ds_xcd, j);
    FGI_LAUNCH_CHECK();
    {
        DArgs a = base_args_b(ops, 1);
        a.in = v.p;
        a.out = v.t;
        a.st = st;
        a.iter = j;
        launch_dslash_b<M_HOP, PP, PP, PP, PX, 0>(c, B, ops, a);
    }
    {
        DArgs a = base_args_b(ops, 0);
        a.in = v.t;
        a.center = v.p;
        a.out = v.q;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash_b<M_CGQ, PP, PP, PP, PX, 0>(c, B, ops, a);
    }
    {
        DArgs a = base_args_b(ops, 1);
        a.in = v.q;
        a.out = v.t;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash_b<M_HOP, PP, PP, PP, PX, 1>(c, B, ops, a);
    }
    {
        DArgs a = base_args_b(ops, 0);
        a.in = v.t;
        a.center = v.q;
        a.aux = v.p;
        a.x = v.x;
        a.r = v.r;
        a.g5out = 1;
        a.partial = part;
        a.st = st;
        a.iter = j;
        launch_dslash_b<M_CGX, PP, PP, PP, PX, 0>(c, B, ops, a);
    }
}

template <int PP, int PX>
static void cg_batch_b(Ctx& c, const Batch& B, const FermionOp& ops, const CGVecs& v, int nit, CGState* st,
                       const CGChain* ch) {
    for (int j = 0; j < nit; j++) cg_iteration_b<PP, PX>(c, B, ops, v, j, st);
    hipLaunchKernelGGL(k_advance_b, dim3(B.nc), dim3(DBS), 0, c.stream, B.cd, st, ch,
                       (const double*)partial_buf(c, B), nit);
    FGI_LAUNCH_CHECK();
}

// All chains of the batch solved together: every kernel covers every chain,
// each chain with its own CG state; chains stop on their own and take their
// reliable updates in masked steps.
//
// A round is half as many iterations again as the slowest chain's inner run still
// needs by its decay so far, one masked true residual for the chains that the
// device finds at their end, and one wait.  While a chain's inner run goes on, all
// true residuals are held back (k_cg_hold_b), so that the chains enter their next
// inner runs together.  Out of step, a round ends for one chain or another every
// time, and the launches past a chain's end cost its blocks' exit; holding back for
// one round only lets large chains drift apart.  Rounds of a fixed batch with the
// masks set by the host -> held for one round -> held:
//   16^3x32 thermalised at beta 5.6, kappa 0.1575, FG n = 16 in FP16 storage with
//   fixed-point links (s): 2 chains 2.17 -> 2.42 -> 2.05, 8 chains 8.33 -> 8.91 ->
//   7.79, where one chain alone takes 1.05;
//   links exp(0.45 X), kappa 0.15 to 0.157 (ms): 96 chains of 4^4 to 8^3x16 in FP16
//   storage 158 -> 120 -> 119, 24 in FP32 117 -> 69.5 -> 63.8, 24 in FP64 118 -> 81.2
//   -> 80.9, 12 with fixed-point links 96.6 -> 73.5 -> 73.4, 3 in FP16 45 -> 33.1 -> 32.2.
// The iterates do not depend on the counts.
template <int PP, int PX>
static std::vector<CGResult> cg_run_b(Ctx& c, const Batch& B, const FermionOp& op64, const FermionOp& ops,
                                      const d2* phi, d2* X, double tol, int maxiter, bool guess) {
    const int nc = B.nc;
    const double drop = ru_drop(c, PP);
    const size_t n64 = sizeof(d2) * 12 * (size_t)B.sites;
    std::vector<CGResult> res(nc, CGResult{0, 0, 0.0, 0});
    double* part = partial_buf(c, B);
    double* bb = (double*)c.bscal.get(sizeof(double) * nc);
    CGState* st = (CGState*)c.bstate.get((sizeof(CGState) + sizeof(CGChain)) * nc);
    CGChain* ch = (CGChain*)(st + nc);
    const CGRun run{tol * tol, PX == P64 ? 0.0 : drop * drop, bb, nullptr, maxiter, c.cg_batch};
    hipLaunchKernelGGL(k_norm2_partials_b, dim3(B.nblk[GRID_VH]), dim3(DBS), 0, c.stream, B.cd, nc, phi, part);
    FGI_LAUNCH_CHECK();
    final_sums_b(c, B, part, GRID_VH, bb);
    if (!guess) zero_doubles(c, (double*)X, 24 * (size_t)B.sites);
    d2* r64 = (d2*)c.cg_r.get(n64);
    if (guess) {  // every chain with a nonzero right-hand side starts from its true residual
        const dim3 nb(nblk(nc, DBS)), bs(DBS);
        hipLaunchKernelGGL(k_cg_mask_b, nb, bs, 0, c.stream, nc, st, (const double*)bb, 1);
        FGI_B_LAUNCH((k_zero_spinor_b<P64>), B.nblk[GRID_VH]), B.cd, nc, st, sp(X));   // phi = 0: the solution is 0
        hipLaunchKernelGGL(k_cg_mask_b, nb, bs, 0, c.stream, nc, st, (const double*)bb, 0);
        FGI_LAUNCH_CHECK();
        true_residual_b<P64>(c, B, op64, phi, X, sp(r64), SpinorPtr{}, st);
    }
    hipLaunchKernelGGL(k_cg_start_b, dim3(nc), dim3(DBS), 0, c.stream, B.cd, st, ch, run,
                       guess ? (const double*)part : nullptr);
    FGI_LAUNCH_CHECK();
    CGVecs v{};
    float* norms = (float*)c.s_norms.get(sizeof(float) * 3 * (size_t)B.sites);
    const d2* r_start = guess ? r64 : phi;
    if (PX == P64) {
        if (!guess) FGI_HIP(hipMemcpyAsync(r64, phi, n64, hipMemcpyDeviceToDevice, c.stream));
        v.x = sp(X);
        v.r = sp(r64);
        v.p = sp(c.cg_p.get(n64));
        v.q = sp(c.cg_q.get(n64));
        v.t = sp(c.s_t.get(n64));
        FGI_HIP(hipMemcpyAsync(v.p.v, r_start, n64, hipMemcpyDeviceToDevice, c.stream));
    } else {
        size_t nx = sizeof(float) * 24 * (size_t)B.sites;
        size_t np = PP == P32 ? nx : sizeof(_Float16) * 24 * (size_t)B.sites;
        v.x = sp(c.s_x.get(nx));
        v.r = sp(c.s_r.get(nx));
        v.p = sp(c.s_p.get(np), norms);
        v.q = sp(c.s_q.get(np), norms + B.sites);
        v.t = sp(c.s_t.get(np), norms + 2 * (size_t)B.sites);
        zero_doubles(c, (double*)v.x.v, 12 * (size_t)B.sites);
        FGI_B_LAUNCH((k_convert_b<P64, PX>), B.nblk[GRID_VH]), B.cd, nc, sp(r_start), v.r);
        FGI_B_LAUNCH((k_convert_b<P64, PP>), B.nblk[GRID_VH]), B.cd, nc, sp(r_start), v.p);
        FGI_LAUNCH_CHECK();
    }
    const int Bi = c.cg_batch;
    GraphEntry* ge = nullptr;
    if (c.use_graphs) {
        // the grid sizes are baked into the graph (the chain table is read at run time)
        char key[400];
        snprintf(key, sizeof key, "bcg/%d/%d/%p/%d/%d/%d/%d/%d/%p/%p/%ld/%p/%p/%p/%p/%p/%p/%p/%p/%p/%d/%d/%d", PP, PX,
                 ops.links, ops.prec, ops.recon, nc, B.ds_blk[0], B.ds_blk[1], (void*)B.ds_map[0], (void*)B.ds_map[1],
                 B.sites, (void*)B.cd, v.x.v, v.r.v, v.p.v,
                 v.q.v, v.t.v, (void*)v.p.norm, (void*)st, (void*)part, Bi, c.ds_bs, c.ds_xcd);
        ge = &cached_graph(c, key, [&] { cg_batch_b<PP, PX>(c, B, ops, v, Bi, st, ch); });
    }
    for (int n = std::min(Bi, 8); n > 0;) {
        for (int left = n; left > 0;) {
            const int m = std::min(left, Bi);
            if (ge && m == Bi) FGI_HIP(hipGraphLaunch(ge->exec, c.stream));
            else cg_batch_b<PP, PX>(c, B, ops, v, m, st, ch);
            left -= m;
        }
        hipLaunchKernelGGL(k_cg_hold_b, dim3(1), dim3(DBS), 0, c.stream, nc, st, (const CGChain*)ch);
        if (PX != P64) {
            FGI_B_LAUNCH((k_add_to64_b<PX>), B.nblk[GRID_VH]), B.cd, nc, st, v.x, sp(X));
            FGI_LAUNCH_CHECK();
        }
        true_residual_b<PX>(c, B, op64, phi, X, v.r, PX == P64 ? SpinorPtr{} : v.x, st);
        hipLaunchKernelGGL(k_cg_restart_b, dim3(nc), dim3(DBS), 0, c.stream, B.cd, st, ch, run, (const double*)part,
                           c.host_bseen);
        FGI_LAUNCH_CHECK();
        FGI_HIP(hipStreamSynchronize(c.stream));
        n = 0;
        int room = INT_MAX;
        for (int i = 0; i < nc; i++) {
            const CGState& s = c.host_bseen[i].s;
            const CGChain& e = c.host_bseen[i].h;
            if (e.status == CH_BAD)
                throw Error(-4, guess && !e.iters ? "batched CG: non-finite residual of the starting point"
                                                  : "batched CG: non-finite residual");
            if (e.status != CH_RUNNING) continue;
            if (s.stop_at <= s.base) continue;   // ended and held back
            const double now = s.rr[s.base & 1];
            if (!std::isfinite(now)) throw Error(-4, "batched CG: non-finite residual");
            const double need = std::log(s.rr_stop / now) / (std::log(now / e.rr0) / s.base);
            n = std::max(n, !(need > 0.0) || need > 1e6 ? Bi : (int)std::min(std::ceil(1.5 * need), 64.0));
            room = std::min(room, e.cut - s.base);   // no chain past its cut-off
        }
        n = std::min(n, room);
    }
    for (int i = 0; i < nc; i++) {
        const CGChain& e = c.host_bseen[i].h;
        res[i] = CGResult{e.iters, e.status == CH_CONVERGED, e.bb > 0 ? std::sqrt(e.rr / e.bb) : 0.0, e.updates};
    }
    return res;
}

std::vector<CGResult> cg_solve_b(Ctx& c, const Batch& B, const FermionOp& op64, const FermionOp& ops, int sprec,
                                 const d2* phi, d2* X, double tol, int maxiter, bool guess) {
    if ((size_t)B.nc > c.host_b_cap) {
        if (c.host_bseen) hipHostFree(c.host_bseen);
        c.host_bseen = nullptr;
        c.host_b_cap = 0;
        FGI_HIP(hipHostMalloc((void**)&c.host_bseen, sizeof(CGSeen) * B.nc, hipHostMallocDefault));
        c.host_b_cap = B.nc;
    }
    if (sprec == P64) return cg_run_b<P64, P64>(c, B, op64, op64, phi, X, tol, maxiter, guess);
    if (sprec == P32) return cg_run_b<P32, P32>(c, B, op64, ops, phi, X, tol, maxiter, guess);
    return cg_run_b<P16, P32>(c, B, op64, ops, phi, X, tol, maxiter, guess);
}

CGResult cg_solve(Ctx& c, const FermionOp& op64, const FermionOp& ops, int sprec, const d2* phi, d2* X, double tol,
                  int maxiter, bool guess) {
    if (sprec == P64) return cg_run<P64, P64>(c, op64, op64, phi, X, tol, maxiter, guess);
    if (sprec == P32) return cg_run<P32, P32>(c, op64, ops, phi, X, tol, maxiter, guess);
    return cg_run<P16, P32>(c, op64, ops, phi, X, tol, maxiter, guess);
}

// ============================================ t-decomposed hopping term ======
// One GPU's share of a lattice split over GPUs in t: its local sub-lattice is
// an ordinary (L0, L1, L2, Lt) checkerboard, and the hops across its two
// t-faces go through halo buffers instead of the local field.  Face sites form
// one contiguous range of F = Vh / Lt checkerboard indices per t slice (t is
// the slowest coordinate), and the site (x, y, z) of the t = 0 face and of the
// t = Lt - 1 face share the face index f = s - t F, also across neighbouring
// ranks (Lt even keeps the local and global parities equal).
//
// The pack kernel forms, for an input field of parity p_in, what each
// neighbour rank needs from this one:
//   to_lo[f] = sign_lo (1 - g4) psi(x, t = 0)                (projected half spinor)
//   to_hi[f] = sign_hi U_t(x)^+ (1 + g4) psi(x, t = Lt - 1)   (already carried by its link)
// as 2 x 3 complex numbers in the working precision R.  The rank below reads
// our to_lo as its from_hi, the rank above our to_hi as its from_lo.  The
// signs carry the antiperiodic boundary: -1 on the lowest rank's to_lo and on
// the highest rank's to_hi, +1 elsewhere.  The halo hop then applies exactly
// the arithmetic of the local kernel's t hops (the link product of the forward
// hop, the spin reconstruction of both), so a decomposed hop is bitwise the
// hop of the whole lattice.
struct HaloArgs {
    Geom g;
    int p;       // output parity (hop) or input parity (pack)
    int s0, s1;  // hop: output sites s0 <= s < s1, or with faces the two face slices
    int faces;
    const void* links;
    SpinorPtr in, out;
    const void* lo;  // hop: from_lo (backward t hops at t = 0);  pack: to_lo
    const void* hi;  // hop: from_hi (forward t hops at t = Lt-1); pack: to_hi
    double sign_lo, sign_hi;
};

template <typename R> struct HaloT;
template <> struct HaloT<double> { typedef d2 T; };
template <> struct HaloT<float> { typedef f2 T; };

// component k = 3 j + a of face entry f: SoA over the F face sites
template <typename R>
__device__ __forceinline__ void halo_store(void* buf, int F, int f, const cx<R> v[2][3], R sign) {
    typedef typename HaloT<R>::T T;
    T* b = (T*)buf;
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int a = 0; a < 3; a++) b[(size_t)(3 * j + a) * F + f] = T{sign * v[j][a].re, sign * v[j][a].im};
}

template <typename R>
__device__ __forceinline__ void halo_load(const void* buf, int F, int f, cx<R> v[2][3]) {
    typedef typename HaloT<R>::T T;
    const T* b = (const T*)buf;
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const T x = b[(size_t)(3 * j + a) * F + f];
            v[j][a] = {x.x, x.y};
        }
}

template <int PIN, int PL, int RECON>
__global__ void __launch_bounds__(DBS) k_halo_pack(HaloArgs A) {
    typedef typename Real<PIN == P64 ? P64 : P32>::T R;
    const Geom& g = A.g;
    const int F = g.Vh / g.L[3];
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    LoadPlain<PIN, 0, R> ld{A.in};
    cx<R> psi[4][3], h[2][3];
    {   // t = 0: the forward hop of the rank below lands here
        typename LoadPlain<PIN, 0, R>::Raw rs;
        ld.fetch(f, g.Vh, rs);
        const R w = ld.get(rs, psi);
        spin_proj<3, -1>(psi, h);
        halo_store<R>(const_cast<void*>(A.lo), F, f, h, w * R(A.sign_lo));
    }
    {   // t = Lt - 1: the backward hop of the rank above, link product included
        const int s = (g.L[3] - 1) * F + f;
        typename LoadPlain<PIN, 0, R>::Raw rs;
        ld.fetch(s, g.Vh, rs);
        const R w = ld.get(rs, psi);
        spin_proj<3, +1>(psi, h);
        RawLink<PL, RECON> rl;
        fetch_link<PL, RECON, false>(A.links, 3, A.p, s, g.Vh, rl);
        const M3<R> u = LinkIO<PL, RECON, R>::decode(rl);
        cx<R> uh[2][3];
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int a = 0; a < 3; a++)
                uh[j][a] = cdot3c(u.e[0][a], h[j][0], u.e[1][a], h[j][1], u.e[2][a], h[j][2]);
        halo_store<R>(const_cast<void*>(A.hi), F, f, uh, w * R(A.sign_hi) * R(link_unit<PL, RECON>()));
    }
}

template <int PIN, int POUT, int PL, int RECON>
__global__ void __launch_bounds__(DBS) k_dslash_halo(HaloArgs A) {
    typedef typename Real<PIN == P64 ? P64 : P32>::T R;
    const Geom& g = A.g;
    const int F = g.Vh / g.L[3];
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    // faces: threads 0..F-1 take the t = 0 slice, F..2F-1 the t = Lt-1 slice
    const int s = A.faces ? (i < F ? i : g.Vh - 2 * F + i) : A.s0 + i;
    if (A.faces ? i >= 2 * F : s >= A.s1) return;
    const int p = A.p;
    LoadPlain<PIN, 0, R> ld{A.in};
    const Coord c = cb_coords(g, p, s);
    cx<R> acc[4][3];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) acc[i][k] = {R(0), R(0)};
    hop<0, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    hop<1, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    hop<2, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    hop<3, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    hop<4, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    hop<5, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    if (c.c[3] == g.L[3] - 1) {  // forward t hop: the projected spinor of the rank above
        cx<R> h[2][3];
        halo_load<R>(A.hi, F, s - (g.L[3] - 1) * F, h);
        RawLink<PL, RECON> rl;
        fetch_link<PL, RECON, false>(A.links, 3, p, s, g.Vh, rl);
        const M3<R> u = LinkIO<PL, RECON, R>::decode(rl);
        cx<R> uh[2][3];
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int a = 0; a < 3; a++)
                uh[j][a] = cdot3(u.e[a][0], h[j][0], u.e[a][1], h[j][1], u.e[a][2], h[j][2]);
        spin_recon_acc<3, -1>(acc, uh, R(link_unit<PL, RECON>()));
    } else {
        hop<6, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    }
    if (c.c[3] == 0) {  // backward t hop: the link product of the rank below
        cx<R> uh[2][3];
        halo_load<R>(A.lo, F, s, uh);
        spin_recon_acc<3, +1>(acc, uh, R(1));
    } else {
        hop<7, PL, RECON, false>(g, p, s, c, A.links, ld, acc);
    }
    SpinorIO<POUT, R>::store(A.out, s, g.Vh, acc);
}

size_t halo_bytes(const Geom& g, int prec) {
    return (size_t)6 * (g.Vh / g.L[3]) * (prec == P64 ? sizeof(d2) : sizeof(f2));
}

template <int PIN, int POUT>
static void halo_launch(Ctx& c, const FermionOp& op, HaloArgs& a, bool pack) {
    const int n = pack ? a.g.Vh / a.g.L[3] : (a.faces ? 2 * (a.g.Vh / a.g.L[3]) : a.s1 - a.s0);
    if (n <= 0) return;
    const int nb = nblk(n, DBS);
#define FGI_HALO_K(PL_, RC_)                                                                                   \
    do {                                                                                                         \
        if (pack) hipLaunchKernelGGL((k_halo_pack<PIN, PL_, RC_>), dim3(nb), dim3(DBS), 0, c.stream, a);         \
        else hipLaunchKernelGGL((k_dslash_halo<PIN, POUT, PL_, RC_>), dim3(nb), dim3(DBS), 0, c.stream, a);      \
    } while (0)
    if constexpr (PIN == P64) {
        FGI_HALO_K(P64, 18);
    } else {
        if (op.prec == P32 && op.recon == 18) FGI_HALO_K(P32, 18);
        else if (op.prec == P32) FGI_HALO_K(P32, 12);
        else if (op.prec == P16 && op.recon == 18) FGI_HALO_K(P16, 18);
        else if (op.prec == P16) FGI_HALO_K(P16, 12);
        else throw Error(-1, "sloppy spinors need sloppy links");
    }
#undef FGI_HALO_K
    FGI_LAUNCH_CHECK();
}

static HaloArgs halo_args(const FermionOp& op) {
    HaloArgs a{};
    a.g = *op.g;
    a.links = op.links;
    return a;
}

void halo_pack(Ctx& c, const FermionOp& op, int prec, int in_parity, SpinorPtr in, double sign_lo, double sign_hi,
               void* to_lo, void* to_hi) {
    HaloArgs a = halo_args(op);
    a.p = in_parity;
    a.in = in;
    a.lo = to_lo;
    a.hi = to_hi;
    a.sign_lo = sign_lo;
    a.sign_hi = sign_hi;
    if (prec == P64) halo_launch<P64, P64>(c, op, a, true);
    else if (prec == P32) halo_launch<P32, P32>(c, op, a, true);
    else halo_launch<P16, P16>(c, op, a, true);
}

// part: 0 every site, 1 the interior (1 <= t <= Lt - 2), 2 the two face slices (one launch)
void dslash_halo(Ctx& c, const FermionOp& op, int prec, int out_parity, SpinorPtr in, SpinorPtr out,
                 const void* from_lo, const void* from_hi, int part) {
    HaloArgs a = halo_args(op);
    a.p = out_parity;
    a.in = in;
    a.out = out;
    a.lo = from_lo;
    a.hi = from_hi;
    const int F = a.g.Vh / a.g.L[3];
    auto run = [&](int s0, int s1, int faces) {
        a.s0 = s0;
        a.s1 = s1;
        a.faces = faces;
        if (prec == P64) halo_launch<P64, P64>(c, op, a, false);
        else if (prec == P32) halo_launch<P32, P32>(c, op, a, false);
        else halo_launch<P16, P16>(c, op, a, false);
    };
    if (part == 0) run(0, a.g.Vh, 0);
    else if (part == 1) run(F, a.g.Vh - F, 0);
    else if (a.g.L[3] == 2) run(0, a.g.Vh, 0);  // both slices are faces
    else run(0, 0, 1);
}

}  // namespace fgi
