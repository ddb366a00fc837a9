// Gauge-side kernels: layout conversion, Hamiltonian densities, the Wilson
// gauge (staple) force and its tangent (the force gradient along a field),
// the exact su(3) link update and reunitarisation.  FP64 throughout.
#include "fgi_coord.h"
#include "fgi_internal.h"

namespace fgi {

static inline int nblocks(long n, int bs) { return (int)((n + bs - 1) / bs); }
static const int BS = 256;

// ---------------------------------------------------------------- layout ---
// User links and momenta are [mu][site] records of NE entries (links 9 complex,
// momenta 8 doubles).  A block moves 256 records: it meets user memory in one
// contiguous stretch and each parity's planes in runs of 128, with the transpose
// in LDS.  (Sites 2q and 2q + 1 are checkerboard index q of the two parities.)
// Bound by memory; a thread per record of one parity fetched every line once per
// parity.  32^3x64: links in 690 -> 492 us, momenta out 401 -> 211, the rate of
// a copy.
template <typename T, int NE, int PAD>
__device__ __forceinline__ void pack_records(const Geom& g, T* __restrict__ user, T* __restrict__ in, int to_internal,
                                             int blk, T* lds) {
    constexpr int ROW = NE + PAD;
    const int t = threadIdx.x, r0 = blk * 256, n = min(256, 4 * g.V - r0);   // first record, records
    // this thread's record in the planes
    const int p = t >> 7, q = (r0 >> 1) + (t & 127), mu = q / g.Vh, s = q - mu * g.Vh;
    const bool live = 2 * (t & 127) < n;
    const int rec = 2 * (t & 127) + (live ? cb_coords(g, p, s).c[0] & 1 : 0);
    T* pl = in + (size_t)((mu * 2 + p) * NE) * g.Vh + s;
    T* us = user + (size_t)r0 * NE;
    T v[NE];
    if (to_internal) {
#pragma unroll
        for (int j = 0; j < NE; j++)
            if (t + 256 * j < n * NE) v[j] = us[t + 256 * j];
#pragma unroll
        for (int j = 0; j < NE; j++) {
            const int e = t + 256 * j;
            if (e < n * NE) lds[(e / NE) * ROW + e % NE] = v[j];
        }
        __syncthreads();
        if (!live) return;
#pragma unroll
        for (int k = 0; k < NE; k++) pl[(size_t)k * g.Vh] = lds[rec * ROW + k];
    } else {
        if (live) {
#pragma unroll
            for (int k = 0; k < NE; k++) v[k] = pl[(size_t)k * g.Vh];
#pragma unroll
            for (int k = 0; k < NE; k++) lds[rec * ROW + k] = v[k];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NE; j++) {
            const int e = t + 256 * j;
            if (e < n * NE) us[e] = lds[(e / NE) * ROW + e % NE];
        }
    }
}
// The same by a thread per record of one parity, without the exchange.
template <typename T, int NE>
__device__ __forceinline__ void pack_record(const Geom& g, T* __restrict__ user, T* __restrict__ in, int to_internal,
                                            int t) {
    if (t >= 4 * g.V) return;
    const int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    const Coord c = cb_coords(g, p, s);
    const int i = c.c[0] + g.L[0] * (c.c[1] + g.L[1] * (c.c[2] + g.L[2] * c.c[3]));
    T* pl = in + (size_t)(r * NE) * g.Vh + s;
    T* us = user + ((size_t)mu * g.V + i) * NE;
    T v[NE];
    if (to_internal) {
#pragma unroll
        for (int k = 0; k < NE; k++) v[k] = us[k];
#pragma unroll
        for (int k = 0; k < NE; k++) pl[(size_t)k * g.Vh] = v[k];
    } else {
#pragma unroll
        for (int k = 0; k < NE; k++) v[k] = pl[(size_t)k * g.Vh];
#pragma unroll
        for (int k = 0; k < NE; k++) us[k] = v[k];
    }
}
// One block's 256 records either way.
template <bool EX, typename T, int NE, int PAD>
__device__ __forceinline__ void pack_block(const Geom& g, T* user, T* in, int to_internal, int blk, T* lds) {
    if (EX) pack_records<T, NE, PAD>(g, user, in, to_internal, blk, lds);
    else pack_record<T, NE>(g, user, in, to_internal, blk * 256 + (int)threadIdx.x);
}
constexpr int PACK_LINK_LDS = 256 * 9, PACK_MOM_LDS = 256 * 9;   // elements; a momentum row is padded to 9

template <bool EX>
__global__ void __launch_bounds__(256) k_pack_gauge(Geom g, const d2* user, d2* U, int to_internal) {
    __shared__ d2 lds[EX ? PACK_LINK_LDS : 1];
    pack_block<EX, d2, 9, 0>(g, (d2*)user, U, to_internal, blockIdx.x, lds);
}

template <bool EX>
__global__ void __launch_bounds__(256) k_pack_mom(Geom g, const double* user, double* P, int to_internal) {
    __shared__ double lds[EX ? PACK_MOM_LDS : 1];
    pack_block<EX, double, 8, 1>(g, (double*)user, P, to_internal, blockIdx.x, lds);
}

// user even spinor: entry k (= checkerboard index of the k-th even site) holds [4][3] complex
__device__ __forceinline__ void pack_even_body(const Geom& g, const d2* __restrict__ user, d2* __restrict__ X,
                                               int to_internal, int s) {
    if (s >= g.Vh) return;
    if (to_internal) {
#pragma unroll
        for (int k = 0; k < 12; k++) X[(size_t)k * g.Vh + s] = user[(size_t)s * 12 + k];
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) ((d2*)user)[(size_t)s * 12 + k] = X[(size_t)k * g.Vh + s];
    }
}

__global__ void k_pack_even(Geom g, const d2* __restrict__ user, d2* __restrict__ X, int to_internal) {
    pack_even_body(g, user, X, to_internal, blockIdx.x * blockDim.x + threadIdx.x);
}

// A call's inputs in one launch: nl blocks of links, nm of momenta, the rest of the
// even spinor.  Small calls last as long as their launches: Mhat at 8^4, four
// launches instead of five, 25 -> 21 us, the fermion force 52 -> 39 us (its split
// hops included).
template <bool EX>
__global__ void __launch_bounds__(256) k_pack_inputs(Geom g, const d2* U, d2* u, const double* P, double* pm,
                                                     const d2* X, d2* x, int nl, int nm) {
    __shared__ d2 lds[EX ? PACK_LINK_LDS : 1];
    const int b = blockIdx.x;
    if (b < nl) pack_block<EX, d2, 9, 0>(g, (d2*)U, u, 1, b, lds);
    else if (b < nl + nm) pack_block<EX, double, 8, 1>(g, (double*)P, pm, 1, b - nl, (double*)lds);
    else pack_even_body(g, X, x, 1, (b - nl - nm) * 256 + (int)threadIdx.x);
}

// batched: field 0 links, 1 momenta, 2 even spinor (the chain's user pointer)
template <bool EX>
__global__ void __launch_bounds__(256) k_pack_b(const ChainDesc* __restrict__ cd, int nc, void* internal, int field,
                                                int to_internal) {
    __shared__ d2 lds[EX ? PACK_LINK_LDS : 1];
    const int kind = field == 2 ? GRID_VH : GRID_4V;
    const int c = find_chain(cd, nc, blockIdx.x, kind);
    const ChainDesc& d = cd[c];
    const int b = blockIdx.x - d.blk0[kind];
    if (field == 0) pack_block<EX, d2, 9, 0>(d.g, (d2*)d.user_U, (d2*)internal + 9 * d.link0, to_internal, b, lds);
    else if (field == 1)
        pack_block<EX, double, 8, 1>(d.g, (double*)d.user_P, (double*)internal + 8 * d.link0, to_internal, b, (double*)lds);
    else
        pack_even_body(d.g, (const d2*)d.user_eta, (d2*)internal + 12 * d.site0, to_internal, b * 256 + (int)threadIdx.x);
}

// Which way.  On a lattice that the L2s hold, a thread per record leaves each plane's
// stretch in the L2 of the XCD whose block reads it next (blocks in linear order), and
// waits for no barrier; above, every line's second fetch costs more.  Whole calls,
// exchange -> direct (us): reunitarise 8^4 26.4 -> 24.6, 8x8x16x16 33.2 -> 29.0, 12^4 35.2 ->
// 35.4, 12^3x24 40.5 -> 46.7; link update 8^3x16 37.9 -> 34.0, 12^4 43.1 -> 44.7, 16^4
// 70.3 -> 76.1.  Momenta alone: kinetic term (in) 16^3x8 33.6 -> 31.3, 16^4 37.6 -> 33.5,
// 10x14x22x26 39.7 -> 40.6; gauge force (out) 8^4 30.5 -> 29.5, 8^3x16 35.1 -> 36.3.
// Links alone go direct up to twice the line where the planes are whole rounds of the
// eight XCDs (2048 sites): action 16^3x8 46.5 -> 43.2.
constexpr int PACK_DIRECT_MAX_V = 16384, PACK_MOM_IN_MAX_V = 65536, PACK_MOM_OUT_MAX_V = 4096;
static bool whole_rounds(const Geom& g) { return g.Vh % 2048 == 0; }
static bool exchange_links(const Geom& g, int to_internal) {
    return g.V > (to_internal && whole_rounds(g) ? 2 * PACK_DIRECT_MAX_V : PACK_DIRECT_MAX_V);
}
static bool exchange_mom(const Geom& g, int to_internal) {
    return g.V > (to_internal ? PACK_MOM_IN_MAX_V : PACK_MOM_OUT_MAX_V);
}
static void launch_pack_gauge(Ctx& c, const Geom& g, const void* user, d2* U, int to_internal) {
    const dim3 nb(nblocks(4L * g.V, BS)), bs(BS);
    if (exchange_links(g, to_internal)) hipLaunchKernelGGL(k_pack_gauge<true>, nb, bs, 0, c.stream, g, (const d2*)user, U, to_internal);
    else hipLaunchKernelGGL(k_pack_gauge<false>, nb, bs, 0, c.stream, g, (const d2*)user, U, to_internal);
    FGI_LAUNCH_CHECK();
}
static void launch_pack_mom(Ctx& c, const Geom& g, const double* user, double* P, int to_internal) {
    const dim3 nb(nblocks(4L * g.V, BS)), bs(BS);
    if (exchange_mom(g, to_internal)) hipLaunchKernelGGL(k_pack_mom<true>, nb, bs, 0, c.stream, g, user, P, to_internal);
    else hipLaunchKernelGGL(k_pack_mom<false>, nb, bs, 0, c.stream, g, user, P, to_internal);
    FGI_LAUNCH_CHECK();
}

void pack_gauge(Ctx& c, const Geom& g, const void* user, d2* U) { launch_pack_gauge(c, g, user, U, 1); }
// links, and where given momenta and an even spinor
void pack_inputs(Ctx& c, const Geom& g, const void* U, d2* u, const double* P, double* pm, const void* X, d2* x) {
    const int nl = nblocks(4L * g.V, BS), nm = P ? nl : 0, nx = X ? nblocks(g.Vh, BS) : 0;
    const dim3 nb(nl + nm + nx), bs(BS);
    if (g.V > PACK_DIRECT_MAX_V)
        hipLaunchKernelGGL(k_pack_inputs<true>, nb, bs, 0, c.stream, g, (const d2*)U, u, P, pm, (const d2*)X, x, nl, nm);
    else
        hipLaunchKernelGGL(k_pack_inputs<false>, nb, bs, 0, c.stream, g, (const d2*)U, u, P, pm, (const d2*)X, x, nl, nm);
    FGI_LAUNCH_CHECK();
}
void unpack_gauge(Ctx& c, const Geom& g, const d2* U, void* user) { launch_pack_gauge(c, g, user, (d2*)U, 0); }
void pack_mom(Ctx& c, const Geom& g, const double* user, double* P) { launch_pack_mom(c, g, user, P, 1); }
void unpack_mom(Ctx& c, const Geom& g, const double* P, double* user) { launch_pack_mom(c, g, user, (double*)P, 0); }
void pack_even_spinor(Ctx& c, const Geom& g, const void* user, d2* X) {
    hipLaunchKernelGGL(k_pack_even, dim3(nblocks(g.Vh, BS)), dim3(BS), 0, c.stream, g, (const d2*)user, X, 1);
    FGI_LAUNCH_CHECK();
}
void unpack_even_spinor(Ctx& c, const Geom& g, const d2* X, void* user) {
    hipLaunchKernelGGL(k_pack_even, dim3(nblocks(g.Vh, BS)), dim3(BS), 0, c.stream, g, (const d2*)user, (d2*)X, 0);
    FGI_LAUNCH_CHECK();
}

// sloppy copies of the FP64 master gauge field
__device__ __forceinline__ void make_sloppy_body(const Geom& g, const d2* __restrict__ U, void* __restrict__ out,
                                                 int prec, int recon, int t) {
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh;  // r = mu * 2 + p
    const d2* in = U + (size_t)(r * 9) * g.Vh + s;
    cx<double> e[9];
#pragma unroll
    for (int k = 0; k < 9; k++) {
        const d2 v = in[(size_t)k * g.Vh];
        e[k] = {v.x, v.y};
    }
    store_sloppy_link(out, prec, recon, r, s, g.Vh, e);
}

__global__ void k_make_sloppy(Geom g, const d2* __restrict__ U, void* __restrict__ out, int prec, int recon) {
    make_sloppy_body(g, U, out, prec, recon, blockIdx.x * blockDim.x + threadIdx.x);
}

// byte offset of a chain's sloppy links in the concatenated sloppy field
__device__ __forceinline__ size_t sloppy_byte_off(const ChainDesc& d, int prec, int recon) {
    return (size_t)d.link0 * sloppy_link_bytes(prec, recon);
}

__global__ void k_make_sloppy_b(const ChainDesc* __restrict__ cd, int nc, const d2* __restrict__ U,
                                void* __restrict__ out, int prec, int recon) {
    const int c = find_chain(cd, nc, blockIdx.x, GRID_4V);
    const ChainDesc& d = cd[c];
    make_sloppy_body(d.g, U + 9 * d.link0, (char*)out + sloppy_byte_off(d, prec, recon), prec, recon,
                     (blockIdx.x - d.blk0[GRID_4V]) * blockDim.x + threadIdx.x);
}

void make_sloppy(Ctx& c, const Geom& g, const d2* U, void* sloppy, int prec, int recon) {
    hipLaunchKernelGGL(k_make_sloppy, dim3(nblocks(4L * g.V, BS)), dim3(BS), 0, c.stream, g, U, sloppy, prec, recon);
    FGI_LAUNCH_CHECK();
}

// ----------------------------------------------------------- densities ---
// h(x) = beta sum_{mu<nu} (1 - ReTr[U_mu(x) U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+]/3)
//        + 1/2 sum_mu |p_mu(x)|^2
__device__ __forceinline__ void ham_density_body(const Geom& g, double beta, const d2* __restrict__ U,
                                                 const double* __restrict__ P, double* __restrict__ h, int t) {
    if (t >= g.V) return;
    int p = t / g.Vh, s = t % g.Vh;
    Coord c = cb_coords(g, p, s);
    double acc = 0.0;
#pragma unroll 1
    for (int mu = 0; mu < (U ? 4 : 0); mu++) {
        M3<double> umu = gauge_load(U, mu, p, s, g.Vh);
        int smu = cb_neighbour(g, c, mu, +1);
#pragma unroll 1
        for (int nu = mu + 1; nu < 4; nu++) {
            int snu = cb_neighbour(g, c, nu, +1);
            M3<double> a = m3_mul(umu, gauge_load(U, nu, 1 - p, smu, g.Vh));
            M3<double> b = m3_mul(gauge_load(U, nu, p, s, g.Vh), gauge_load(U, mu, 1 - p, snu, g.Vh));
            double tr = 0.0;
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) tr += a.e[i][j].re * b.e[i][j].re + a.e[i][j].im * b.e[i][j].im;
            acc += 1.0 - tr / 3.0;
        }
    }
    acc *= beta;
    if (P) {
        double kin = 0.0;
        for (int mu = 0; mu < 4; mu++) {
            double x[8];
            mom_load(P, mu, p, s, g.Vh, x);
#pragma unroll
            for (int a = 0; a < 8; a++) kin += x[a] * x[a];
        }
        acc += 0.5 * kin;
    }
    h[t] = acc;
}

__global__ void __launch_bounds__(256) k_ham_density(Geom g, double beta, const d2* __restrict__ U, const double* __restrict__ P,
                              double* __restrict__ h, int xcd) {
    ham_density_body(g, beta, U, P, h, slab_thread(g.Vh, 2, xcd));
}

// bscale multiplies each chain's beta (1 - 8 c1 for the plaquettes of the improved action)
__global__ void __launch_bounds__(256) k_ham_density_b(const ChainDesc* __restrict__ cd, int nc, const d2* __restrict__ U,
                                const double* __restrict__ P, double* __restrict__ h, double bscale) {
    const int c = find_chain(cd, nc, blockIdx.x, GRID_V);
    const ChainDesc& d = cd[c];
    ham_density_body(d.g, d.beta * bscale, U ? U + 9 * d.link0 : nullptr, P ? P + 8 * d.link0 : nullptr, h + d.vol0,
                     (blockIdx.x - d.blk0[GRID_V]) * blockDim.x + threadIdx.x);
}

void rect_density_add(Ctx& c, const Geom& g, double bc1, const d2* U, double* h);

// Order of the density kernel: linear where the fields lie in the L2s as the layout
// kernels' blocks left them: the momenta up to 65536 sites, and links whose planes are
// whole rounds of the XCDs unless the rectangles read them too.  Linear -> slabs (us): kinetic term 8x8x16x16 30.4 -> 31.8,
// 16^3x8 31.3 -> 33.8, 12^3x24 34.8 -> 34.7; action 8^3x16 38.7 -> 39.6, 16^3x8 43.2 ->
// 47.2, 16^4 52.6 -> 52.7, 16^3x32 91.9 -> 84.3; 12^3x8 45.2 -> 43.2, 12^3x24 51.5 -> 47.6.
static int density_order(const Ctx& c, const Geom& g, const d2* U, double c1) {
    if (g.V <= PACK_MOM_IN_MAX_V && (!U || (whole_rounds(g) && c1 == 0.0))) return 0;
    return slab_order(c, g);
}

void ham_density(Ctx& c, const Geom& g, double beta, const d2* U, const double* P, double* h, double c1) {
    const int xcd = density_order(c, g, U, c1);
    hipLaunchKernelGGL(k_ham_density, dim3(slab_blocks(g.Vh, 2, BS, xcd)), dim3(BS), 0, c.stream, g,
                       beta * (1.0 - 8.0 * c1), U, P, h, xcd);
    FGI_LAUNCH_CHECK();
    if (c1 != 0.0 && U) rect_density_add(c, g, beta * c1, U, h);
}

__global__ void k_diff_partials(int n, const double* __restrict__ h1, const double* __restrict__ h0,
                                double* __restrict__ partial) {
    __shared__ double lds[16];
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    double v[1] = {0.0};
    if (t < n) v[0] = h0 ? h1[t] - h0[t] : h1[t];
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// partial[blk0 + b] = sum over chain-local block b of (h1 - h0) on the chain's V sites
__global__ void k_diff_partials_b(const ChainDesc* __restrict__ cd, int nc, const double* __restrict__ h1,
                                  const double* __restrict__ h0, double* __restrict__ partial) {
    __shared__ double lds[16];
    const int c = find_chain(cd, nc, blockIdx.x, GRID_V);
    const ChainDesc& d = cd[c];
    const int t = (blockIdx.x - d.blk0[GRID_V]) * blockDim.x + threadIdx.x;
    double v[1] = {0.0};
    if (t < d.g.V) v[0] = h0 ? h1[d.vol0 + t] - h0[d.vol0 + t] : h1[d.vol0 + t];
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// out[c] = fixed-order sum of chain c's partials (one block per chain)
__global__ void k_final_sum_b(const ChainDesc* __restrict__ cd, const double* __restrict__ partial, int kind,
                              double* __restrict__ out) {
    __shared__ double lds[16];
    const ChainDesc& d = cd[blockIdx.x];
    double s = sum_partials(partial + d.blk0[kind], d.nblk[kind], lds);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

int diff_partials(Ctx& c, int n, const double* h1, const double* h0, double* partial) {
    int nb = nblocks(n, BS);
    hipLaunchKernelGGL(k_diff_partials, dim3(nb), dim3(BS), 0, c.stream, n, h1, h0, partial);
    FGI_LAUNCH_CHECK();
    return nb;
}

__global__ void k_final_sum(const double* __restrict__ partial, int n, double* __restrict__ out) {
    __shared__ double lds[16];
    double s = sum_partials(partial, n, lds);
    if (threadIdx.x == 0) *out = s;
}

void final_sum(Ctx& c, const double* partial, int n, double* out) {
    hipLaunchKernelGGL(k_final_sum, dim3(1), dim3(BS), 0, c.stream, partial, n, out);
    FGI_LAUNCH_CHECK();
}

// ------------------------------------------------------------- force -----
// Staple sum A_mu(x) = sum_{nu != mu} [U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
//                                     + U_nu(x+mu-nu)^+ U_mu(x-nu)^+ U_nu(x-nu)];
// the part of S_G holding U_mu(x) is -beta/3 ReTr(U_mu(x) A_mu(x)), so
// F_mu(x) = -e S = -(beta/6) TA(U_mu(x) A_mu(x)).
//
// The improved action adds c1 times the six rectangle staples per nu.  They are
// the two plaquette staples with one of their three links replaced by that link's
// own staple pointing outwards: the upper one, a b^+ c^+ (a = U_nu(x+mu), b =
// U_mu(x+nu), c = U_nu(x)), with a by a' = U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^+,
// b by b' = U_nu(x+nu) U_mu(x+2nu) U_nu(x+mu+nu)^+ or c by c' = U_mu(x-mu)^+
// U_nu(x-mu) U_mu(x-mu+nu); the lower one, (e d)^+ f, alike.  So
//   f0 a b^+ c^+ + f1 (a' b^+ c^+ + a b'^+ c^+ + a b^+ c'^+)
//     = [f0 a b^+ + f1 (a' b^+ + a b'^+)] c^+ + f1 (a b^+) c'^+,
// eleven products for a half, the plaquette included.
struct ForceCoef { double f0, f1; };   // of the plaquette and of the rectangle staples

// the upper (UP) or lower plaquette staple of link (MU, x) in the (MU, nu) plane
template <int MU, bool UP>
__device__ __forceinline__ M3<double> staple(const Geom& g, const d2* __restrict__ U, const Coord& c, int p, int s,
                                             int nu) {
    const Coord cm = cb_shift(g, c, MU, +1);
    if (UP) {   // U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
        const int sm = cb_index(g, cm), sn = cb_neighbour(g, c, nu, +1);
        return m3_mul_nd(m3_mul_nd(gauge_load(U, nu, 1 - p, sm, g.Vh), gauge_load(U, MU, 1 - p, sn, g.Vh)),
                         gauge_load(U, nu, p, s, g.Vh));
    }
    // (U_mu(x-nu) U_nu(x+mu-nu))^+ U_nu(x-nu)
    const int sb = cb_neighbour(g, c, nu, -1), smb = cb_neighbour(g, cm, nu, -1);
    return m3_mul_dn(m3_mul(gauge_load(U, MU, 1 - p, sb, g.Vh), gauge_load(U, nu, p, smb, g.Vh)),
                     gauge_load(U, nu, 1 - p, sb, g.Vh));
}

// One of the three turns of a half of the improved staples, added to A; T is
// carried from turn to turn.  Turn 0: T = f0 a b^+, A += f1 (a b^+) c'^+; turn 1:
// T += f1 a b'^+; turn 2: T += f1 a' b^+, A += T c^+ (the lower half alike).  The
// turns are blocks of a rolled loop: only A and T live across them (the links they
// share are loaded again), so a turn's five matrices fit two waves per SIMD; as one
// straight piece the compiler hoists the loads and spills 3 KB a lane.
template <int MU, bool UP>
__device__ __forceinline__ void rect_turn(const Geom& g, const d2* __restrict__ U, const Coord& c, int p, int s, int nu,
                                          int turn, const ForceCoef& k, M3<double>& A, M3<double>& T) {
    const int o = 1 - p;
    const Coord cm = cb_shift(g, c, MU, +1);
    // a load the compiler cannot take for one it has made before: the links that the
    // turns share, kept live from turn to turn, would spill
    auto ld = [&](int mu, int par, int site) {
        asm volatile("" : "+v"(site));
        return gauge_load(U, mu, par, site, g.Vh);
    };
    M3<double> l;
    if (UP) {
        const int sm = cb_index(g, cm), sn = cb_neighbour(g, c, nu, +1);
        if (turn == 0) {          // c' = U_mu(x-mu)^+ U_nu(x-mu) U_mu(x-mu+nu)
            const Coord cl = cb_shift(g, c, MU, -1);
            const int sl = cb_index(g, cl);
            l = m3_mul(m3_mul_dn(ld(MU, o, sl), ld(nu, o, sl)),
                       ld(MU, p, cb_neighbour(g, cl, nu, +1)));
            m3_scale(l, k.f1);
            T = m3_mul_nd(ld(nu, o, sm), ld(MU, o, sn));
            m3_acc(A, m3_mul_nd(T, l));
            m3_scale(T, k.f0);
        } else if (turn == 1) {   // b' = U_nu(x+nu) U_mu(x+2nu) U_nu(x+mu+nu)^+
            const int s2n = cb_neighbour(g, cb_shift(g, c, nu, +1), nu, +1), smn = cb_neighbour(g, cm, nu, +1);
            l = m3_mul_nd(m3_mul(ld(nu, o, sn), ld(MU, p, s2n)),
                          ld(nu, p, smn));
            m3_scale(l, k.f1);
            m3_acc(T, m3_mul_nd(ld(nu, o, sm), l));
        } else {                  // a' = U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^+
            const int s2m = cb_neighbour(g, cm, MU, +1), smn = cb_neighbour(g, cm, nu, +1);
            l = m3_mul_nd(m3_mul(ld(MU, o, sm), ld(nu, p, s2m)),
                          ld(MU, p, smn));
            m3_scale(l, k.f1);
            m3_acc(T, m3_mul_nd(l, ld(MU, o, sn)));
            m3_acc(A, m3_mul_nd(T, ld(nu, p, s)));
        }
    } else {
        const Coord cb = cb_shift(g, c, nu, -1), cmb = cb_shift(g, cm, nu, -1);
        const int sb = cb_index(g, cb), smb = cb_index(g, cmb);
        if (turn == 0) {          // f' = U_mu(x-nu-mu)^+ U_nu(x-nu-mu) U_mu(x-mu)
            const Coord cl = cb_shift(g, c, MU, -1);
            const int slb = cb_neighbour(g, cl, nu, -1);
            l = m3_mul(m3_mul_dn(ld(MU, p, slb), ld(nu, p, slb)),
                       ld(MU, o, cb_index(g, cl)));
            m3_scale(l, k.f1);
            T = m3_mul(ld(MU, o, sb), ld(nu, p, smb));
            m3_acc(A, m3_mul_dn(T, l));
            m3_scale(T, k.f0);
        } else if (turn == 1) {   // e' = U_nu(x-2nu)^+ U_mu(x-2nu) U_nu(x-2nu+mu)
            const int s2b = cb_neighbour(g, cb, nu, -1), sm2b = cb_neighbour(g, cmb, nu, -1);
            l = m3_mul(m3_mul_dn(ld(nu, p, s2b), ld(MU, p, s2b)),
                       ld(nu, o, sm2b));
            m3_scale(l, k.f1);
            m3_acc(T, m3_mul(l, ld(nu, p, smb)));
        } else {                  // d' = U_mu(x+mu-nu) U_nu(x+2mu-nu) U_mu(x+mu)^+
            const int s2mb = cb_neighbour(g, cmb, MU, +1);
            l = m3_mul_nd(m3_mul(ld(MU, p, smb), ld(nu, o, s2mb)),
                          ld(MU, o, cb_index(g, cm)));
            m3_scale(l, k.f1);
            m3_acc(T, m3_mul(ld(MU, o, sb), l));
            m3_acc(A, m3_mul_dn(T, ld(nu, o, sb)));
        }
    }
}

// s, as a value the compiler cannot recognise as one it has used before
__device__ __forceinline__ int again(int s) {
    asm volatile("" : "+v"(s));
    return s;
}

// The same half as three turns of rect_turn, in one piece: one wave of a split
// link has nothing else to do while it waits, so the loads of a turn overlap the
// products of the last (force and update, turns -> piece, us: 4^4 25.5 -> 18.4,
// 8^3x16 60.7 -> 40.5; over the six halves of an unsplit link the turns are the
// faster, 16^3x32 409 -> 382, 32^3x64 8068 -> 7617).  again() marks links that are
// loaded again because, kept live, they would spill.
template <int MU, bool UP>
__device__ __forceinline__ M3<double> rect_half(const Geom& g, const d2* __restrict__ U, const Coord& c, int p, int s,
                                                int nu, const ForceCoef& k) {
    const int o = 1 - p;
    const Coord cm = cb_shift(g, c, MU, +1);
    const Coord cl = cb_shift(g, c, MU, -1);
    M3<double> A, T;
    if (UP) {
        const int sm = again(cb_index(g, cm)), sn = cb_neighbour(g, c, nu, +1), sl = again(cb_index(g, cl));
        const Coord cmn = cb_shift(g, cm, nu, +1);
        const int smn = cb_index(g, cmn);
        M3<double> l = m3_mul(m3_mul_dn(gauge_load(U, MU, o, sl, g.Vh), gauge_load(U, nu, o, sl, g.Vh)),
                              gauge_load(U, MU, p, cb_neighbour(g, cl, nu, +1), g.Vh));
        m3_scale(l, k.f1);
        T = m3_mul_nd(gauge_load(U, nu, o, sm, g.Vh), gauge_load(U, MU, o, sn, g.Vh));
        A = m3_mul_nd(T, l);
        m3_scale(T, k.f0);
        __builtin_amdgcn_sched_barrier(0);
        const int s2n = cb_neighbour(g, cb_shift(g, c, nu, +1), nu, +1);
        l = m3_mul_nd(m3_mul(gauge_load(U, nu, o, sn, g.Vh), gauge_load(U, MU, p, s2n, g.Vh)),
                      gauge_load(U, nu, p, smn, g.Vh));
        m3_scale(l, k.f1);
        m3_acc(T, m3_mul_nd(gauge_load(U, nu, o, again(sm), g.Vh), l));
        __builtin_amdgcn_sched_barrier(0);
        const int s2m = cb_neighbour(g, cm, MU, +1);
        l = m3_mul_nd(m3_mul(gauge_load(U, MU, o, again(sm), g.Vh), gauge_load(U, nu, p, s2m, g.Vh)),
                      gauge_load(U, MU, p, smn, g.Vh));
        m3_scale(l, k.f1);
        m3_acc(T, m3_mul_nd(l, gauge_load(U, MU, o, again(sn), g.Vh)));
        m3_acc(A, m3_mul_nd(T, gauge_load(U, nu, p, again(s), g.Vh)));
    } else {
        const Coord cb = cb_shift(g, c, nu, -1), cmb = cb_shift(g, cm, nu, -1), clb = cb_shift(g, cl, nu, -1);
        const int sm = again(cb_index(g, cm)), sb = cb_index(g, cb), smb = cb_index(g, cmb), slb = cb_index(g, clb);
        M3<double> l = m3_mul(m3_mul_dn(gauge_load(U, MU, p, slb, g.Vh), gauge_load(U, nu, p, slb, g.Vh)),
                              gauge_load(U, MU, o, again(cb_index(g, cl)), g.Vh));
        m3_scale(l, k.f1);
        T = m3_mul(gauge_load(U, MU, o, sb, g.Vh), gauge_load(U, nu, p, smb, g.Vh));
        A = m3_mul_dn(T, l);
        m3_scale(T, k.f0);
        __builtin_amdgcn_sched_barrier(0);
        const int s2b = cb_neighbour(g, cb, nu, -1), sm2b = cb_neighbour(g, cmb, nu, -1);
        l = m3_mul(m3_mul_dn(gauge_load(U, nu, p, s2b, g.Vh), gauge_load(U, MU, p, s2b, g.Vh)),
                   gauge_load(U, nu, o, sm2b, g.Vh));
        m3_scale(l, k.f1);
        m3_acc(T, m3_mul(l, gauge_load(U, nu, p, again(smb), g.Vh)));
        __builtin_amdgcn_sched_barrier(0);
        const int s2mb = cb_neighbour(g, cmb, MU, +1);
        l = m3_mul_nd(m3_mul(gauge_load(U, MU, p, again(smb), g.Vh), gauge_load(U, nu, o, s2mb, g.Vh)),
                      gauge_load(U, MU, o, sm, g.Vh));
        m3_scale(l, k.f1);
        m3_acc(T, m3_mul(gauge_load(U, MU, o, again(sb), g.Vh), l));
        m3_acc(A, m3_mul_dn(T, gauge_load(U, nu, o, again(sb), g.Vh)));
    }
    return A;
}

// one link U_mu(x); MU known at compile time (every block of the force
// launch holds links of one direction, so the switch below does not diverge)
template <int MU, bool IMP>
__device__ __forceinline__ void gauge_force_link(const Geom& g, double f, const ForceCoef& k, const d2* __restrict__ U,
                                                 double* __restrict__ F, int accumulate, int s, int p, int r) {
    const Coord c = cb_coords(g, p, s);
    M3<double> A = m3_zero<double>();
    if constexpr (IMP) {
        M3<double> T = m3_zero<double>();
#pragma unroll 1
        for (int j = 0; j < 18; j++) {
            const int h = j / 3, turn = j - 3 * h, nu = (h >> 1) + ((h >> 1) >= MU);
            if (h & 1) rect_turn<MU, false>(g, U, c, p, s, nu, turn, k, A, T);
            else rect_turn<MU, true>(g, U, c, p, s, nu, turn, k, A, T);
        }
    } else {
#pragma unroll 1
        for (int nu = 0; nu < 4; nu++) {
            if (nu == MU) continue;
            m3_acc(A, staple<MU, true>(g, U, c, p, s, nu));
            m3_acc(A, staple<MU, false>(g, U, c, p, s, nu));
        }
    }
    M3<double> W = m3_mul(gauge_load(U, MU, p, s, g.Vh), A);
    double x[8];
    ta_components(W, x);
    double* o = F + (size_t)(r * 8) * g.Vh + s;
#pragma unroll
    for (int a = 0; a < 8; a++) {
        double v = f * x[a];
        o[(size_t)a * g.Vh] = accumulate ? o[(size_t)a * g.Vh] + v : v;
    }
}

template <bool IMP>
__device__ __forceinline__ void gauge_force_body(const Geom& g, double f, const ForceCoef& k, const d2* __restrict__ U,
                                                 double* __restrict__ F, int accumulate, int t) {
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    switch (mu) {
    case 0: gauge_force_link<0, IMP>(g, f, k, U, F, accumulate, s, p, r); break;
    case 1: gauge_force_link<1, IMP>(g, f, k, U, F, accumulate, s, p, r); break;
    case 2: gauge_force_link<2, IMP>(g, f, k, U, F, accumulate, s, p, r); break;
    default: gauge_force_link<3, IMP>(g, f, k, U, F, accumulate, s, p, r); break;
    }
}

// f multiplies TA(U A); with IMP the staples carry k.f0 and k.f1.  With IMP bound by
// FP64 VALU at two waves per SIMD: 67 products a link, 1.3e4 flops, 20 TFLOP/s at
// 16^3x32.  A plaquette launch and one of the 18 rectangle staples, paired on the
// steps they share, read links twice and F back: force and update at 16^3x32 487 ->
// 381 us, 32^3x64 9.93 -> 7.66 ms.  Storing the link staples that the rectangles
// share needs fewer products and lost to the traffic (581 us).
template <bool IMP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_gauge_force(Geom g, double f, ForceCoef k, const d2* __restrict__ U, double* __restrict__ F, int accumulate, int xcd) {
    gauge_force_body<IMP>(g, f, k, U, F, accumulate, slab_thread(g.Vh, 8, xcd));
}

// Small lattices: one thread per link leaves the chip idle (4^4: 16 waves) and
// the launch lasts as long as one thread's thirteen dependent products.  Here a
// block's six waves share 64 links of one (mu, parity): wave w forms staple
// w & 1 of the w / 2-th plane, the six staples meet in LDS and are summed in the
// one-thread order, and four waves form the entries of U A that their force
// components need.  Without the rectangles: the same operations in the same order
// as unsplit, the same bits.
struct GaugeSplitLds {
    cx<double> st[6][9][64];
    cx<double> A[9][64];
};

template <int MU, bool IMP>
__device__ __forceinline__ void gauge_force_split_link(const Geom& g, double f, const ForceCoef& kf,
                                                       const d2* __restrict__ U, double* __restrict__ F, int accumulate,
                                                       int s, bool live, int p, int r, GaugeSplitLds& L) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = w >> 1, nu = k + (k >= MU);
    const Coord c = cb_coords(g, p, s);
    M3<double> S;
    if constexpr (IMP) {
        if (w & 1) S = rect_half<MU, false>(g, U, c, p, s, nu, kf);
        else S = rect_half<MU, true>(g, U, c, p, s, nu, kf);
    } else {
        if (w & 1) S = staple<MU, false>(g, U, c, p, s, nu);
        else S = staple<MU, true>(g, U, c, p, s, nu);
    }
    const M3<double> u = gauge_load(U, MU, p, s, g.Vh);
#pragma unroll
    for (int e = 0; e < 9; e++) L.st[w][e][lane] = S.e[e / 3][e % 3];
    __syncthreads();
    for (int e = w; e < 9; e += 6) {
        cx<double> a = {0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 6; j++) a = a + L.st[j][e][lane];
        L.A[e][lane] = a;
    }
    __syncthreads();
    if (w > 3 || !live) return;
    auto W = [&](int i, int j) {
        return u.e[i][0] * L.A[j][lane] + u.e[i][1] * L.A[3 + j][lane] + u.e[i][2] * L.A[6 + j][lane];
    };
    double* o = F + (size_t)(r * 8) * g.Vh + s;
    auto put = [&](int a, double x) {
        const double v = f * x;
        o[(size_t)a * g.Vh] = accumulate ? o[(size_t)a * g.Vh] + v : v;
    };
    // the components of ta_components, from the entries they are made of
    if (w == 0) {
        const cx<double> a = W(0, 1), b = W(1, 0);
        put(0, a.im + b.im);
        put(1, a.re - b.re);
    } else if (w == 1) {
        const cx<double> a = W(0, 2), b = W(2, 0);
        put(3, a.im + b.im);
        put(4, a.re - b.re);
    } else if (w == 2) {
        const cx<double> a = W(1, 2), b = W(2, 1);
        put(5, a.im + b.im);
        put(6, a.re - b.re);
    } else {
        const double a = W(0, 0).im, b = W(1, 1).im, d = W(2, 2).im;
        put(2, a - b);
        put(7, 0.57735026918962576451 * (a + b - 2.0 * d));
    }
}

template <bool IMP>
__device__ __forceinline__ void gauge_force_split_block(const Geom& g, double f, const ForceCoef& k,
                                                        const d2* __restrict__ U, double* __restrict__ F,
                                                        int accumulate, int B, GaugeSplitLds& L) {
    const int r = B & 7, p = r & 1, s_ = (B >> 3) * 64 + (threadIdx.x & 63);
    const bool live = s_ < g.Vh;
    const int s = live ? s_ : g.Vh - 1;
    switch (r >> 1) {
    case 0: gauge_force_split_link<0, IMP>(g, f, k, U, F, accumulate, s, live, p, r, L); break;
    case 1: gauge_force_split_link<1, IMP>(g, f, k, U, F, accumulate, s, live, p, r, L); break;
    case 2: gauge_force_split_link<2, IMP>(g, f, k, U, F, accumulate, s, live, p, r, L); break;
    default: gauge_force_split_link<3, IMP>(g, f, k, U, F, accumulate, s, live, p, r, L); break;
    }
}

template <bool IMP>
__global__ void __launch_bounds__(384) k_gauge_force_split(Geom g, double f, ForceCoef k, const d2* __restrict__ U,
                                                          double* __restrict__ F, int accumulate, int xcd) {
    __shared__ GaugeSplitLds L;
    gauge_force_split_block<IMP>(g, f, k, U, F, accumulate, xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x, L);
}

// the chains of a batch that take the split kernel (GRID_GS)
template <bool IMP>
__global__ void __launch_bounds__(384) k_gauge_force_split_b(const ChainDesc* __restrict__ cd, int nc,
                                                            const d2* __restrict__ U, double* __restrict__ F,
                                                            double coef, double c1, int accumulate) {
    __shared__ GaugeSplitLds L;
    const int c = find_chain(cd, nc, blockIdx.x, GRID_GS);
    const ChainDesc& d = cd[c];
    gauge_force_split_block<IMP>(d.g, -d.beta / 6.0 * coef, ForceCoef{1.0 - 8.0 * c1, c1}, U + 9 * d.link0,
                                 F + 8 * d.link0, accumulate, blockIdx.x - d.blk0[GRID_GS], L);
}

template <bool IMP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_gauge_force_b(const ChainDesc* __restrict__ cd, int nc, const d2* __restrict__ U, double* __restrict__ F, double coef,
                double c1, int accumulate) {
    const int c = find_chain(cd, nc, blockIdx.x, GRID_4V);
    const ChainDesc& d = cd[c];
    if (d.nblk[GRID_GS]) return;   // it has the split kernel
    gauge_force_body<IMP>(d.g, -d.beta / 6.0 * coef, ForceCoef{1.0 - 8.0 * c1, c1}, U + 9 * d.link0, F + 8 * d.link0,
                          accumulate, (blockIdx.x - d.blk0[GRID_4V]) * blockDim.x + threadIdx.x);
}

void gauge_force(Ctx& c, const Geom& g, double beta, const d2* U, double* F, double coef, int accumulate, double c1) {
    const double f = -beta / 6.0 * coef;
    const ForceCoef k{1.0 - 8.0 * c1, c1};
    if (g.V <= GAUGE_SPLIT_MAX_V) {
        const dim3 nb(8 * nblocks(g.Vh, 64)), bs(384);
        if (c1 != 0.0) hipLaunchKernelGGL(k_gauge_force_split<true>, nb, bs, 0, c.stream, g, f, k, U, F, accumulate, c.ds_xcd);
        else hipLaunchKernelGGL(k_gauge_force_split<false>, nb, bs, 0, c.stream, g, f, k, U, F, accumulate, c.ds_xcd);
    } else {
        const dim3 nb(slab_blocks(g.Vh, 8, BS, c.ds_xcd)), bs(BS);
        if (c1 != 0.0) hipLaunchKernelGGL(k_gauge_force<true>, nb, bs, 0, c.stream, g, f, k, U, F, accumulate, c.ds_xcd);
        else hipLaunchKernelGGL(k_gauge_force<false>, nb, bs, 0, c.stream, g, f, k, U, F, accumulate, c.ds_xcd);
    }
    FGI_LAUNCH_CHECK();
}

// Tangent of the gauge force along a field of su(3) elements V:
// d/dt F_G(exp(tV) U) at t = 0.  Each link moves as dU = V U, dU^+ = -U^+ V;
// the product rule is applied factor by factor to U_mu(x) A_mu(x).
__device__ __forceinline__ M3<double> valg(const double* Vd, int mu, int p, int s, int Vh) {
    double x[8];
    mom_load(Vd, mu, p, s, Vh, x);
    return alg_matrix(x);
}

// mode 0: J = coef * d/dt F_G(exp(tV) U)
// mode 1: J = coef * (Hessian of S_G in the chart exp(omega) U at omega = 0) V
//         = coef * (-J_V[F_G] + [V, F_G] / 2)   (per link commutator)
__global__ void __launch_bounds__(256) k_gauge_tangent(Geom g, double beta, const d2* __restrict__ U,
                                                      const double* __restrict__ Vd, double* __restrict__ J,
                                                      double coef, int accumulate, int mode, int xcd) {
    int t = slab_thread(g.Vh, 8, xcd);
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    Coord c = cb_coords(g, p, s);
    // indexed coordinates here (cb_neighbour_ix): with selects this kernel
    // spills more and runs 3 % slower than with the compiler's LDS copy
    int s_pmu = cb_neighbour_ix(g, c, mu, +1);
    Coord cpm = c;
    cpm.c[mu] = (c.c[mu] + 1) % g.L[mu];
    M3<double> A = m3_zero<double>(), dA = m3_zero<double>();
#pragma unroll 1
    for (int nu = 0; nu < 4; nu++) {
        if (nu == mu) continue;
        int s_pnu = cb_neighbour_ix(g, c, nu, +1);
        int s_mnu = cb_neighbour_ix(g, c, nu, -1);
        int s_pmu_mnu = cb_neighbour_ix(g, cpm, nu, -1);
        {   // upper staple a b^+ c^+
            M3<double> a = gauge_load(U, nu, 1 - p, s_pmu, g.Vh);
            M3<double> b = gauge_load(U, mu, 1 - p, s_pnu, g.Vh);
            M3<double> cc = gauge_load(U, nu, p, s, g.Vh);
            M3<double> da = m3_mul(valg(Vd, nu, 1 - p, s_pmu, g.Vh), a);
            M3<double> db = m3_mul(valg(Vd, mu, 1 - p, s_pnu, g.Vh), b);
            M3<double> dc = m3_mul(valg(Vd, nu, p, s, g.Vh), cc);
            M3<double> bc = m3_mul_nd(m3_dag(b), cc);  // b^+ c^+
            m3_acc(A, m3_mul(a, bc));
            m3_acc(dA, m3_mul(da, bc));
            m3_acc(dA, m3_mul_nd(m3_mul_nd(a, db), cc));
            m3_acc(dA, m3_mul_nd(m3_mul_nd(a, b), dc));
        }
        {   // lower staple d^+ e^+ f
            M3<double> d = gauge_load(U, nu, p, s_pmu_mnu, g.Vh);
            M3<double> e = gauge_load(U, mu, 1 - p, s_mnu, g.Vh);
            M3<double> f = gauge_load(U, nu, 1 - p, s_mnu, g.Vh);
            M3<double> dd = m3_mul(valg(Vd, nu, p, s_pmu_mnu, g.Vh), d);
            M3<double> de = m3_mul(valg(Vd, mu, 1 - p, s_mnu, g.Vh), e);
            M3<double> df = m3_mul(valg(Vd, nu, 1 - p, s_mnu, g.Vh), f);
            M3<double> ed = m3_mul(e, d);  // (d^+ e^+)^+
            m3_acc(A, m3_mul_dn(ed, f));
            m3_acc(dA, m3_mul_dn(m3_mul(e, dd), f));
            m3_acc(dA, m3_mul_dn(m3_mul(de, d), f));
            m3_acc(dA, m3_mul_dn(ed, df));
        }
    }
    M3<double> u = gauge_load(U, mu, p, s, g.Vh);
    M3<double> vl = valg(Vd, mu, p, s, g.Vh);
    M3<double> du = m3_mul(vl, u);
    M3<double> dW = m3_mul(du, A);
    m3_acc(dW, m3_mul(u, dA));
    double x[8];
    ta_components(dW, x);
    double* o = J + (size_t)(r * 8) * g.Vh + s;
    const double f = -beta / 6.0;
    if (mode == 1) {
        // F = f TA(U A) as a matrix; [V, F] components
        double fx[8];
        ta_components(m3_mul(u, A), fx);
#pragma unroll
        for (int a = 0; a < 8; a++) fx[a] *= f;
        M3<double> Fm = alg_matrix(fx);
        M3<double> C = m3_mul(vl, Fm);
        M3<double> D = m3_mul(Fm, vl);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) C.e[i][j] = C.e[i][j] - D.e[i][j];
        double cx8[8];
        ta_components(C, cx8);
#pragma unroll
        for (int a = 0; a < 8; a++) x[a] = -f * x[a] + 0.5 * cx8[a];
    } else {
#pragma unroll
        for (int a = 0; a < 8; a++) x[a] = f * x[a];
    }
#pragma unroll
    for (int a = 0; a < 8; a++) {
        double v = coef * x[a];
        o[(size_t)a * g.Vh] = accumulate ? o[(size_t)a * g.Vh] + v : v;
    }
}

void rect_tangent(Ctx& c, const Geom& g, double beta, double c1, const d2* U, const double* Vd, double* J,
                  double coef, int mode);

void gauge_force_tangent(Ctx& c, const Geom& g, double beta, const d2* U, const double* Vd, double* J, double coef,
                         int accumulate, int mode, double c1) {
    hipLaunchKernelGGL(k_gauge_tangent, dim3(slab_blocks(g.Vh, 8, BS, c.ds_xcd)), dim3(BS), 0, c.stream, g, beta, U,
                       Vd, J, coef * (1.0 - 8.0 * c1), accumulate, mode, c.ds_xcd);
    FGI_LAUNCH_CHECK();
    if (c1 != 0.0) rect_tangent(c, g, beta, c1, U, Vd, J, coef, mode);
}

// ------------------------------------------------- rectangle (2x1) terms ---
// Improved gauge action
//   S_G = beta sum_x [c0 sum_{mu<nu} (1 - ReTr P_{mu nu}(x)/3) + c1 sum_{mu!=nu} (1 - ReTr R_{mu nu}(x)/3)],
// c0 = 1 - 8 c1, R_{mu nu}(x) the rectangle two links along mu and one along nu
// (c1 = -1/12: tree-level Symanzik, Luscher and Weisz 1985; c1 = -0.331:
// Iwasaki).  Everything is linear in (c0, c1): the plaquette kernels above run
// with their coefficient scaled by c0 and the kernels below add the c1 part.

// The 18 rectangle staples of link (mu, x) are the 5-link paths from x + mu
// back to x that close a 2x1 rectangle through U_mu(x); per nu != mu, six
// shapes, written as steps (+-1: along +-mu, +-2: along +-nu):
//   two long along mu, +nu side, U_mu(x) the first or the second mu link;
//   the same on the -nu side; two long along nu on the +nu and -nu sides.
__constant__ int RECT_SHAPES[6][5] = {{1, 2, -1, -1, -2}, {2, -1, -1, -2, 1}, {1, -2, -1, -1, 2},
                                      {-2, -1, -1, 2, 1},  {2, 2, -1, -2, -2}, {-2, -2, -1, 2, 2}};

// One factor of a path walked from y: a step along +d multiplies U_d(y) and
// moves to y + d; a step along -d moves to y - d and multiplies U_d(y)^+.
// With TAN, dl is the derivative of the factor along V (V U, or -U^+ V).
template <bool TAN>
__device__ __forceinline__ M3<double> path_factor(const Geom& g, const d2* __restrict__ U,
                                                  const double* __restrict__ Vd, Coord& y, int d, int fwd,
                                                  M3<double>& dl) {
    if (!fwd) coord_step(g, y, d, 0);
    const int par = coord_parity(y), s = cb_index(g, y);
    const M3<double> u = gauge_load(U, d, par, s, g.Vh);
    if (TAN) {
        const M3<double> v = valg(Vd, d, par, s, g.Vh);
        if (fwd) {
            dl = m3_mul(v, u);
        } else {
            dl = m3_mul_dn(u, v);
            m3_scale(dl, -1.0);
        }
    }
    if (fwd) coord_step(g, y, d, 1);
    return fwd ? u : m3_dag(u);
}

// A = sum of the 18 rectangle staples of link (mu, x); with TAN, dA = its
// derivative along V by the product rule, factor by factor.
template <bool TAN>
__device__ __forceinline__ void rect_staples(const Geom& g, const d2* __restrict__ U, const double* __restrict__ Vd,
                                             const Coord& c, int mu, M3<double>& A, M3<double>& dA) {
    A = m3_zero<double>();
    if (TAN) dA = m3_zero<double>();
#pragma unroll 1
    for (int nu = 0; nu < 4; nu++) {
        if (nu == mu) continue;
#pragma unroll 1
        for (int k = 0; k < 6; k++) {
            Coord y = c;
            coord_step(g, y, mu, 1);
            M3<double> P, D, dl;
#pragma unroll 1
            for (int j = 0; j < 5; j++) {
                const int st = RECT_SHAPES[k][j];
                const int d = (st == 1 || st == -1) ? mu : nu;
                const M3<double> f = path_factor<TAN>(g, U, Vd, y, d, st > 0, dl);
                if (j == 0) {
                    P = f;
                    if (TAN) D = dl;
                } else {
                    if (TAN) {
                        D = m3_mul(D, f);
                        m3_acc(D, m3_mul(P, dl));
                    }
                    P = m3_mul(P, f);
                }
            }
            m3_acc(A, P);
            if (TAN) m3_acc(dA, D);
        }
    }
}

// h(x) += bc1 sum_{mu != nu} (1 - ReTr R_{mu nu}(x) / 3), with
// ReTr R = ReTr(a b^+), a = U_mu(x) U_mu(x+mu) U_nu(x+2mu), b = U_nu(x) U_mu(x+nu) U_mu(x+mu+nu)
__device__ __forceinline__ void rect_density_body(const Geom& g, double bc1, const d2* __restrict__ U,
                                                  double* __restrict__ h, int t) {
    if (t >= g.V) return;
    const int p = t / g.Vh, s = t % g.Vh;
    const Coord c = cb_coords(g, p, s);
    double acc = 0.0;
#pragma unroll 1
    for (int mu = 0; mu < 4; mu++) {
        Coord xm = c;
        coord_step(g, xm, mu, 1);
        Coord x2m = xm;
        coord_step(g, x2m, mu, 1);
        const M3<double> aa = m3_mul(gauge_load(U, mu, p, s, g.Vh), link_at(g, U, mu, xm));
#pragma unroll 1
        for (int nu = 0; nu < 4; nu++) {
            if (nu == mu) continue;
            Coord xn = c, xmn = xm;
            coord_step(g, xn, nu, 1);
            coord_step(g, xmn, nu, 1);
            const M3<double> a = m3_mul(aa, link_at(g, U, nu, x2m));
            const M3<double> b = m3_mul(m3_mul(gauge_load(U, nu, p, s, g.Vh), link_at(g, U, mu, xn)),
                                        link_at(g, U, mu, xmn));
            double tr = 0.0;
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) tr += a.e[i][j].re * b.e[i][j].re + a.e[i][j].im * b.e[i][j].im;
            acc += 1.0 - tr / 3.0;
        }
    }
    h[t] += bc1 * acc;
}

__global__ void __launch_bounds__(256) k_rect_density(Geom g, double bc1, const d2* __restrict__ U,
                                                     double* __restrict__ h, int xcd) {
    rect_density_body(g, bc1, U, h, slab_thread(g.Vh, 2, xcd));
}

// batched chains: chain c adds its beta * c1 times its rectangle sum
__global__ void __launch_bounds__(256) k_rect_density_b(const ChainDesc* __restrict__ cd, int nc, double c1,
                                                       const d2* __restrict__ U, double* __restrict__ h) {
    const int c = find_chain(cd, nc, blockIdx.x, GRID_V);
    const ChainDesc& d = cd[c];
    rect_density_body(d.g, d.beta * c1, U + 9 * d.link0, h + d.vol0,
                      (blockIdx.x - d.blk0[GRID_V]) * blockDim.x + threadIdx.x);
}

void rect_density_add(Ctx& c, const Geom& g, double bc1, const d2* U, double* h) {
    const int xcd = slab_order(c, g);
    hipLaunchKernelGGL(k_rect_density, dim3(slab_blocks(g.Vh, 2, BS, xcd)), dim3(BS), 0, c.stream, g, bc1, U, h, xcd);
    FGI_LAUNCH_CHECK();
}

// J += coef * (mode 0: J_V[F_R]; mode 1: -J_V[F_R] + [V, F_R] / 2) for the
// rectangle part F_R = -(beta c1 / 6) TA(U A^R) of the force
__device__ __forceinline__ void rect_tangent_body(const Geom& g, double bc1, const d2* __restrict__ U,
                                                  const double* __restrict__ Vd, double* __restrict__ J, double coef,
                                                  int mode, int t) {
    if (t >= 4 * g.V) return;
    const int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    const Coord c = cb_coords(g, p, s);
    M3<double> A, dA;
    rect_staples<true>(g, U, Vd, c, mu, A, dA);
    const M3<double> u = gauge_load(U, mu, p, s, g.Vh);
    const M3<double> vl = valg(Vd, mu, p, s, g.Vh);
    M3<double> dW = m3_mul(m3_mul(vl, u), A);
    m3_acc(dW, m3_mul(u, dA));
    double x[8];
    ta_components(dW, x);
    const double f = -bc1 / 6.0;
    if (mode == 1) {
        double fx[8];
        ta_components(m3_mul(u, A), fx);
#pragma unroll
        for (int a = 0; a < 8; a++) fx[a] *= f;
        const M3<double> Fm = alg_matrix(fx);
        M3<double> C = m3_mul(vl, Fm);
        const M3<double> D = m3_mul(Fm, vl);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) C.e[i][j] = C.e[i][j] - D.e[i][j];
        double cx8[8];
        ta_components(C, cx8);
#pragma unroll
        for (int a = 0; a < 8; a++) x[a] = -f * x[a] + 0.5 * cx8[a];
    } else {
#pragma unroll
        for (int a = 0; a < 8; a++) x[a] = f * x[a];
    }
    double* o = J + (size_t)(r * 8) * g.Vh + s;
#pragma unroll
    for (int a = 0; a < 8; a++) o[(size_t)a * g.Vh] += coef * x[a];
}

// Up to one wave per SIMD (16384 sites) the kernel keeps its registers; above, two
// waves per SIMD are held, for 108 B a lane of scratch.  Free -> two waves (us): 4^4
// 151 -> 174, 8^4 160 -> 185, 12^3x8 190 -> 225, 8x8x16x16 184 -> 212; 12^4 335 -> 320,
// 10x12x14x16 348 -> 335, 14^3x20 661 -> 643; from 16^4 on within 3 % either way.
constexpr int RECT_TANGENT_ONE_WAVE_V = 16384;
__global__ void __launch_bounds__(256) k_rect_tangent_small(Geom g, double bc1, const d2* __restrict__ U,
                                                           const double* __restrict__ Vd, double* __restrict__ J,
                                                           double coef, int mode, int xcd) {
    rect_tangent_body(g, bc1, U, Vd, J, coef, mode, slab_thread(g.Vh, 8, xcd));
}
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_rect_tangent(Geom g, double bc1, const d2* __restrict__ U, const double* __restrict__ Vd, double* __restrict__ J,
               double coef, int mode, int xcd) {
    rect_tangent_body(g, bc1, U, Vd, J, coef, mode, slab_thread(g.Vh, 8, xcd));
}

void rect_tangent(Ctx& c, const Geom& g, double beta, double c1, const d2* U, const double* Vd, double* J,
                  double coef, int mode) {
    const dim3 nb(slab_blocks(g.Vh, 8, BS, c.ds_xcd)), bs(BS);
    if (g.V <= RECT_TANGENT_ONE_WAVE_V)
        hipLaunchKernelGGL(k_rect_tangent_small, nb, bs, 0, c.stream, g, beta * c1, U, Vd, J, coef, mode, c.ds_xcd);
    else
        hipLaunchKernelGGL(k_rect_tangent, nb, bs, 0, c.stream, g, beta * c1, U, Vd, J, coef, mode, c.ds_xcd);
    FGI_LAUNCH_CHECK();
}

// ------------------------------------------------------------ updates ----
// Lattices of at most SERIES_MAX_V sites take the exponential's series.  It is the
// faster on every lattice (a leapfrog step, closed form -> series, us: 4^4 14.4 ->
// 9.3, 8x4x8x8 15.4 -> 10.0; 8^3x6 16.7 -> 11.5, 8^3x16 23.7 -> 18.2, 16^3x32 137.4 ->
// 133.9), where an update lasts as long as one wave's chain of transcendental calls
// most of all.  The line is not one of speed: the two differ in the last bits, and
// above it the links keep those that the benchmark's seeded thermalisation, and the
// calibration measured on its field, start from.
constexpr int SERIES_MAX_V = 2048;
template <bool SERIES>
__device__ __forceinline__ void link_update_body(const Geom& g, double h, const double* __restrict__ X,
                                                 const d2* __restrict__ src, d2* __restrict__ dst,
                                                 void* __restrict__ sloppy, int prec, int recon, int t) {
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    double x[8];
    mom_load(X, mu, p, s, g.Vh, x);
#pragma unroll
    for (int a = 0; a < 8; a++) x[a] *= h;
    M3<double> E = SERIES ? su3_exp_series(alg_matrix(x)) : su3_exp(alg_matrix(x));
    M3<double> u = m3_mul(E, gauge_load(src, mu, p, s, g.Vh));
    gauge_store(dst, mu, p, s, g.Vh, u);
    if (sloppy) {
        cx<double> e[9];
#pragma unroll
        for (int k = 0; k < 9; k++) e[k] = u.e[k / 3][k % 3];
        store_sloppy_link(sloppy, prec, recon, r, s, g.Vh, e);
    }
}

template <bool SERIES>
__global__ void __launch_bounds__(256) k_link_update(Geom g, double h, const double* __restrict__ X, const d2* __restrict__ src,
                              d2* __restrict__ dst, void* __restrict__ sloppy, int prec, int recon) {
    link_update_body<SERIES>(g, h, X, src, dst, sloppy, prec, recon, blockIdx.x * blockDim.x + threadIdx.x);
}

// the chains of one kind (SERIES: at most SERIES_MAX_V sites)
template <bool SERIES>
__global__ void __launch_bounds__(256) k_link_update_b(const ChainDesc* __restrict__ cd, int nc, double h, const double* __restrict__ X,
                                const d2* __restrict__ src, d2* __restrict__ dst, void* __restrict__ sloppy, int prec,
                                int recon) {
    const int c = find_chain(cd, nc, blockIdx.x, GRID_4V);
    const ChainDesc& d = cd[c];
    if (SERIES != (d.g.V <= SERIES_MAX_V)) return;
    link_update_body<SERIES>(d.g, h, X + 8 * d.link0, src + 9 * d.link0, dst + 9 * d.link0,
                     sloppy ? (char*)sloppy + sloppy_byte_off(d, prec, recon) : nullptr, prec, recon,
                     (blockIdx.x - d.blk0[GRID_4V]) * blockDim.x + threadIdx.x);
}

void link_update(Ctx& c, const Geom& g, double h, const double* X, const d2* src, d2* dst, void* sloppy, int prec,
                 int recon) {
    if (g.V <= SERIES_MAX_V)   // blocks of one wave: more of the chip
        hipLaunchKernelGGL(k_link_update<true>, dim3(nblocks(4L * g.V, 64)), dim3(64), 0, c.stream, g, h, X, src, dst,
                           sloppy, prec, recon);
    else
        hipLaunchKernelGGL(k_link_update<false>, dim3(nblocks(4L * g.V, BS)), dim3(BS), 0, c.stream, g, h, X, src, dst,
                           sloppy, prec, recon);
    FGI_LAUNCH_CHECK();
}

// W_l = V_l U_l: the derivative of exp(t V_l) U_l at t = 0.  The hopping term
// is linear in each link and its adjoint, and d(U^+) = (V U)^+, so the
// hopping term on W is the derivative of D along V (Section 4, e_j acting
// on the fermion kernel).
__global__ void k_tangent_links(Geom g, const double* __restrict__ Vd, const d2* __restrict__ U,
                                d2* __restrict__ W) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    double x[8];
    mom_load(Vd, mu, p, s, g.Vh, x);
    gauge_store(W, mu, p, s, g.Vh, m3_mul(alg_matrix(x), gauge_load(U, mu, p, s, g.Vh)));
}

void tangent_links(Ctx& c, const Geom& g, const double* Vd, const d2* U, d2* W) {
    hipLaunchKernelGGL(k_tangent_links, dim3(nblocks(4L * g.V, BS)), dim3(BS), 0, c.stream, g, Vd, U, W);
    FGI_LAUNCH_CHECK();
}

__global__ void k_axpy(long n, double a, const double* __restrict__ x, double* __restrict__ y) {
    long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] += a * x[t];
}

void mom_axpy(Ctx& c, const Geom& g, double a, const double* x, double* y) {
    long n = 4L * 2 * 8 * g.Vh;
    hipLaunchKernelGGL(k_axpy, dim3(nblocks(n, BS)), dim3(BS), 0, c.stream, n, a, x, y);
    FGI_LAUNCH_CHECK();
}

__global__ void k_dot_partials(long n, const double* __restrict__ x, const double* __restrict__ y,
                               double* __restrict__ partial) {
    __shared__ double lds[16];
    long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    double v[1] = {t < n ? x[t] * y[t] : 0.0};
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

int dot_partials(Ctx& c, long n, const double* x, const double* y, double* partial) {
    int nb = nblocks(n, BS);
    hipLaunchKernelGGL(k_dot_partials, dim3(nb), dim3(BS), 0, c.stream, n, x, y, partial);
    FGI_LAUNCH_CHECK();
    return nb;
}

__global__ void k_zero_d(size_t n, double* __restrict__ p) {
    size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 0.0;
}

void zero_doubles(Ctx& c, double* p, size_t n) {
    hipLaunchKernelGGL(k_zero_d, dim3(nblocks((long)n, BS)), dim3(BS), 0, c.stream, n, p);
    FGI_LAUNCH_CHECK();
}

// Gram-Schmidt on rows 0 and 1, row 2 = conj(row0 x row1)
__device__ __forceinline__ void reunitarize_body(const Geom& g, d2* __restrict__ U, int t) {
    if (t >= 4 * g.V) return;
    int s = t % g.Vh, r = t / g.Vh, p = r & 1, mu = r >> 1;
    M3<double> u = gauge_load(U, mu, p, s, g.Vh);
    double n0 = 0;
    for (int j = 0; j < 3; j++) n0 += u.e[0][j].re * u.e[0][j].re + u.e[0][j].im * u.e[0][j].im;
    n0 = 1.0 / sqrt(n0);
    for (int j = 0; j < 3; j++) u.e[0][j] = n0 * u.e[0][j];
    cx<double> d = {0, 0};
    for (int j = 0; j < 3; j++) d = d + cmul(u.e[0][j], u.e[1][j]);
    for (int j = 0; j < 3; j++) u.e[1][j] = u.e[1][j] - d * u.e[0][j];
    double n1 = 0;
    for (int j = 0; j < 3; j++) n1 += u.e[1][j].re * u.e[1][j].re + u.e[1][j].im * u.e[1][j].im;
    n1 = 1.0 / sqrt(n1);
    for (int j = 0; j < 3; j++) u.e[1][j] = n1 * u.e[1][j];
    recon_row2(u);
    gauge_store(U, mu, p, s, g.Vh, u);
}

__global__ void k_reunitarize(Geom g, d2* __restrict__ U) {
    reunitarize_body(g, U, blockIdx.x * blockDim.x + threadIdx.x);
}

void reunitarize(Ctx& c, const Geom& g, d2* U) {
    hipLaunchKernelGGL(k_reunitarize, dim3(nblocks(4L * g.V, BS)), dim3(BS), 0, c.stream, g, U);
    FGI_LAUNCH_CHECK();
}

__global__ void __launch_bounds__(256) k_exp_batch(int n, const double* __restrict__ p, double h, d2* __restrict__ out) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    double x[8];
    for (int a = 0; a < 8; a++) x[a] = h * p[(size_t)t * 8 + a];
    M3<double> E = su3_exp(alg_matrix(x));
    for (int k = 0; k < 9; k++) out[(size_t)t * 9 + k] = d2{E.e[k / 3][k % 3].re, E.e[k / 3][k % 3].im};
}

void exp_su3_batch(Ctx& c, int n, const double* p, double h, void* out) {
    hipLaunchKernelGGL(k_exp_batch, dim3(nblocks(n, BS)), dim3(BS), 0, c.stream, n, p, h, (d2*)out);
    FGI_LAUNCH_CHECK();
}

// ------------------------------------------------------ batched launchers ---
void pack_b(Ctx& c, const Batch& B, void* internal, int field, int to_internal) {
    int nb = field == 2 ? B.nblk[GRID_VH] : B.nblk[GRID_4V];
    if (B.vol > PACK_DIRECT_MAX_V)
        hipLaunchKernelGGL(k_pack_b<true>, dim3(nb), dim3(BS), 0, c.stream, B.cd, B.nc, internal, field, to_internal);
    else
        hipLaunchKernelGGL(k_pack_b<false>, dim3(nb), dim3(BS), 0, c.stream, B.cd, B.nc, internal, field, to_internal);
    FGI_LAUNCH_CHECK();
}

void make_sloppy_b(Ctx& c, const Batch& B, const d2* U, void* sloppy, int prec, int recon) {
    hipLaunchKernelGGL(k_make_sloppy_b, dim3(B.nblk[GRID_4V]), dim3(BS), 0, c.stream, B.cd, B.nc, U, sloppy, prec, recon);
    FGI_LAUNCH_CHECK();
}

void ham_density_b(Ctx& c, const Batch& B, const d2* U, const double* P, double* h, double c1) {
    hipLaunchKernelGGL(k_ham_density_b, dim3(B.nblk[GRID_V]), dim3(BS), 0, c.stream, B.cd, B.nc, U, P, h,
                       1.0 - 8.0 * c1);
    FGI_LAUNCH_CHECK();
    if (c1 != 0.0 && U) {
        hipLaunchKernelGGL(k_rect_density_b, dim3(B.nblk[GRID_V]), dim3(BS), 0, c.stream, B.cd, B.nc, c1, U, h);
        FGI_LAUNCH_CHECK();
    }
}

void diff_sums_b(Ctx& c, const Batch& B, const double* h1, const double* h0, double* partial, double* out) {
    hipLaunchKernelGGL(k_diff_partials_b, dim3(B.nblk[GRID_V]), dim3(BS), 0, c.stream, B.cd, B.nc, h1, h0, partial);
    FGI_LAUNCH_CHECK();
    final_sums_b(c, B, partial, GRID_V, out);
}

void final_sums_b(Ctx& c, const Batch& B, const double* partial, int kind, double* out) {
    hipLaunchKernelGGL(k_final_sum_b, dim3(B.nc), dim3(BS), 0, c.stream, B.cd, partial, kind, out);
    FGI_LAUNCH_CHECK();
}

template <bool IMP>
static void launch_gauge_force_b(Ctx& c, const Batch& B, const d2* U, double* F, double coef, int accumulate, double c1) {
    if (B.nblk[GRID_GS])
        hipLaunchKernelGGL(k_gauge_force_split_b<IMP>, dim3(B.nblk[GRID_GS]), dim3(384), 0, c.stream, B.cd, B.nc, U, F,
                           coef, c1, accumulate);
    if (B.gauge_plain)
        hipLaunchKernelGGL(k_gauge_force_b<IMP>, dim3(B.nblk[GRID_4V]), dim3(BS), 0, c.stream, B.cd, B.nc, U, F, coef, c1,
                           accumulate);
    FGI_LAUNCH_CHECK();
}

void gauge_force_b(Ctx& c, const Batch& B, const d2* U, double* F, double coef, int accumulate, double c1) {
    if (c1 != 0.0) launch_gauge_force_b<true>(c, B, U, F, coef, accumulate, c1);
    else launch_gauge_force_b<false>(c, B, U, F, coef, accumulate, c1);
}

void link_update_b(Ctx& c, const Batch& B, double h, const double* X, const d2* src, d2* dst, void* sloppy, int prec,
                   int recon) {
    if (B.min_vol <= SERIES_MAX_V)
        hipLaunchKernelGGL(k_link_update_b<true>, dim3(B.nblk[GRID_4V]), dim3(BS), 0, c.stream, B.cd, B.nc, h, X, src,
                           dst, sloppy, prec, recon);
    if (B.max_vol > SERIES_MAX_V)
        hipLaunchKernelGGL(k_link_update_b<false>, dim3(B.nblk[GRID_4V]), dim3(BS), 0, c.stream, B.cd, B.nc, h, X, src,
                           dst, sloppy, prec, recon);
    FGI_LAUNCH_CHECK();
}

}  // namespace fgi
