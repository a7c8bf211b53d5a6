// dd_force.hip -- derivative of L = |D^{-1} phi|^2 with respect to the gauge
// links and to c_SW: the fermion-force bilinear of the operator of the
// appendix, D = 1 + C - kappa H.
//
// With psi = D^{-1} phi and chi = D^{-dagger} psi (D^dagger = gamma_5 D gamma_5),
// dL = -2 Re <chi| dD psi>.  Per link U_mu(n) the kernels build the 3x3 matrix
// W_mu(n) with dL = Re sum tr(dU_mu(n) W_mu(n)):
//
//   hop:    W += 2 kappa phase_mu(n) ( [(1 - gamma_mu) psi(n+mu)] chi(n)^dagger
//                                    + ( [(1 + gamma_mu) psi(n)] chi(n+mu)^dagger )^dagger )
//           (outer products over colour, summed over spin);
//   clover: C = i kappa c_SW sum_{mu<nu} sigma_{mu nu} (x) F_{mu nu},
//           F = (Q - Q^dagger)/8, gives dL = Re sum tr(dQ_{mu nu}(n) Y_{mu nu}(n)) with
//           Y = (-i kappa c_SW / 4)(Lambda + Lambda^dagger), anti-Hermitian, and
//           Lambda_{ba} = sum_{alpha beta} sigma_{alpha beta} psi_{b beta} conj(chi_{a alpha}).
//           Every plaquette through the link contributes: for the closed path
//           U Z2 Z3 Z4 (corners d1 = n, d2 = n+mu, d3, d4) the derivative with
//           respect to U is  Y(d2) Z2 Z3 Z4 + Z2 Y(d3) Z3 Z4 + Z2 Z3 Y(d4) Z4 + Z2 Z3 Z4 Y(d1),
//           with Y of the plane taken with the sign of the orientation: + for the
//           plaquette n -> n+mu -> n+mu+nu -> n+nu when mu < nu, and the sign
//           flips with nu > mu and for the plaquette on the -nu side.  Six
//           plaquettes per link (two per other direction), each seen from its
//           four corners: the 24 leaves a link enters.
//   c_SW:   dL/dc_SW = -2 Re <chi| (C / c_SW) psi> = 2 kappa sum_{n, mu<nu} Im tr(F_{mu nu} Lambda_{mu nu}).
//
// Output per link: G = W^dagger, the gradient dL/dRe U + i dL/dIm U entry by
// entry, or (su(3) form) the traceless Hermitian F_mu(n) = (i/2)(X - X^dagger)
// - tr/3, X = U W, with dL = tr(omega F) for U -> exp(i omega) U.
//
// Two kernels: k_force_y brings psi and chi into the internal layout and computes Y for the
// six planes of every site (FP64, FORCE_Y_ELEMS double2 per site, block-major like every other
// field) and the c_SW sum; k_force_w gathers per link.  Both in FP64.
//
// What bounds them (24^4, 332 k sites): k_force_y moves 1.8 kB per site, 605 MB, in 116 us,
// 5.2 TB/s (with psi and chi packed by kernels of their own and Y stored as full 3x3 matrices
// the three took 204 us).  k_force_w takes 550 to 570 us.  Its arithmetic, 5100 FP64 instructions per
// wavefront, would take 170 us, and the data it cannot do without 90 us; what bounds it is the
// vector-memory address path of the CUs: a wavefront loads 303 entries of 16 bytes per lane (6.4 GB
// over the launch), and the address units are busy in 74 % of the cycles, the VALU in 44 %; the 7.4 GB
// that the L2 serves (13 TB/s) are a third of its rate, and requests do not wait for it.  The 64
// sites x 4 directions of a workgroup share their lines in the L2 while they are there; in
// an earlier form the four directions were four passes over the lattice, with nine more
// entries per Y, 512 registers (one wavefront per SIMD instead of two) and every complex
// multiply-add in three instructions instead of two: 1404 us.
#include <mutex>

#include "dd_device.h"
#include "dd_gauge.h"
#include "dd_launch.h"

namespace dd {

// Work field of the force for the entry point that allocates nothing: a fixed
// file-scope device array (each GPU holds its own copy, at its own address, until
// the process ends).  Host code never passes `scratch` itself to a kernel -- on the
// host that name is only a stand-in -- but the device address looked up below.
static __device__ __align__(256) unsigned char scratch[FORCE_SCRATCH_BYTES];

hipError_t force_scratch_address(void **ptr)
{
    // once per device, with that device current
    static std::mutex mu;
    static void *addr[MAX_DEVICES] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

// chiral components of a spinor: u[blk][s][c] = psi_s + (-1)^blk psi_{s+2}
// (the rotation P = [[1, 1], [1, -1]] / sqrt 2 without the 1/sqrt 2)
DD_INL void chiral(const Spinor<double> &p, cx<double> (&u)[2][2][3])
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            u[0][s][c] = p.v[s][c] + p.v[s + 2][c];
            u[1][s][c] = p.v[s][c] - p.v[s + 2][c];
        }
}

// Y of one plane is anti-Hermitian: stored as its upper entries (0,1), (0,2), (1,2) and the
// imaginary parts of its diagonal, five double2 (80 of the 144 bytes of a full 3x3)
struct AntiH {
    cx<double> u[3];
    double d[3];
};

DD_INL void load_y(const Geom &g, const double2 *Y, long long i, int plane, AntiH &M)
{
    const double2 *p = Y + elem(g, (int)(i >> g.lbvol), (int)(i & (g.bvol - 1)), FORCE_Y_ELEMS, plane * 5);
    double2 t[5];
#pragma unroll
    for (int e = 0; e < 5; ++e) t[e] = p[(long long)e << g.lbvol];
#pragma unroll
    for (int e = 0; e < 3; ++e) M.u[e] = {t[e].x, t[e].y};
    M.d[0] = t[3].x;
    M.d[1] = t[3].y;
    M.d[2] = t[4].x;
}

DD_INL void store_y(const Geom &g, double2 *Y, int l, int s, int plane, const AntiH &M)
{
    double2 *p = Y + elem(g, l, s, FORCE_Y_ELEMS, plane * 5);
    const long long n = g.bvol;
#pragma unroll
    for (int e = 0; e < 3; ++e) p[e * n] = make_double2(M.u[e].re, M.u[e].im);
    p[3 * n] = make_double2(M.d[0], M.d[1]);
    p[4 * n] = make_double2(M.d[2], 0.0);
}

DD_INL void load_canonical(const double2 *src, long long n, Spinor<double> &x)
{
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double2 t = src[n * 12 + c * 4 + a];
            x.v[a][c] = {t.x, t.y};
        }
}

// psi and chi into the internal layout (for k_force_w), Y of the six planes per site and, where
// asked, dL/dc_SW:
//   CSW 0: not asked; 1 (c_SW != 0): from the clover blocks already built, -(2 / c_SW) Re <chi| C psi>,
//   with C = Q diag(N+, N-) Q - 1 taken block by block in the chiral components,
//   Q u = (u_+, u_-): <chi| C psi> = sum_b u_b(chi)^dagger (N_b - 1/2) u_b(psi);
//   2 (c_SW = 0, no clover to read it from): from the field strength, 2 kappa sum Im tr(F Lambda).
// One instantiation each: with all three in one kernel every call paid for the registers of the
// field strength (512 and scratch, one wavefront per SIMD).
template <int CSW>
__global__ void __launch_bounds__(BLAS_WG, CSW == 2 ? 1 : 2)
    k_force_y(Geom g, const double2 *psi_can, const double2 *chi_can, SpinorField<0> psi, SpinorField<0> chi,
              const double2 *u64, const double2 *clov, SigmaBlocks sig, double kcsw, double kappa, double csw, double2 *Y,
              double *partials)
{
    double v[1] = {0.0};
    for (long long i = (long long)blockIdx.x * BLAS_WG + threadIdx.x; i < g.V; i += (long long)gridDim.x * BLAS_WG) {
        Site st;
        decode(g, i, st);
        const int l = st.l, s = st.s;
        const long long n = lex_index(g, st);
        cx<double> up[2][2][3], ux[2][2][3];
        {
            Spinor<double> p;
            load_canonical(psi_can, n, p);
            psi.store(g, l, s, p);
            chiral(p, up);
            load_canonical(chi_can, n, p);
            chi.store(g, l, s, p);
            chiral(p, ux);
        }
        if (CSW == 1) {
            double re = 0.0;
            int sl = s;
            asm volatile("" : "+v"(sl) : "v"(ux[1][1][2].re));  // ... and the first block's behind psi and chi
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                cx<double> w[6];
                const cx<double> *u = &up[b][0][0];
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const double2 d = clov[elem(g, l, sl, 36, b * 18 + j)];
                    w[2 * j] = (d.x - 0.5) * u[2 * j];
                    w[2 * j + 1] = (d.y - 0.5) * u[2 * j + 1];
                }
#pragma unroll
                for (int r = 0; r < 6; ++r)
#pragma unroll
                    for (int c = r + 1; c < 6; ++c) {
                        const double2 t = clov[elem(g, l, sl, 36, b * 18 + 3 + upper_index(r, c))];
                        const cx<double> h = {t.x, t.y};
                        w[r] = cmac(w[r], h, u[c]);
                        w[c] = cmacc(w[c], h, u[r]);
                    }
#pragma unroll
                for (int r = 0; r < 6; ++r) re += cmulc((&ux[b][0][0])[r], w[r]).re;
                // the second block's loads stay behind the first block: both at once take 144 VGPRs
                asm volatile("" : "+v"(sl) : "v"(re));
            }
            v[0] -= (2.0 / csw) * re;
        }
        // sigma = P u P with u = diag(sig blocks), P symmetric: the bilinear in the chiral components
        // carries a factor 1/2; stores Y = (-i kcsw / 4)(lam + lam^dagger) of the plane
        auto plane_y = [&](int plane, cx<double> (&lam)[3][3]) {
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) lam[b][a] = {0.0, 0.0};
#pragma unroll
            for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                for (int s1 = 0; s1 < 2; ++s1)
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2) {
                        const cx<double> sg = {0.5 * sig.re[plane][blk][s1][s2], 0.5 * sig.im[plane][blk][s1][s2]};
                        if (sg.re == 0.0 && sg.im == 0.0) continue;
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            const cx<double> t = sg * up[blk][s2][b];
#pragma unroll
                            for (int a = 0; a < 3; ++a) lam[b][a] = cmacc(lam[b][a], ux[blk][s1][a], t);
                        }
                    }
            const double f = 0.25 * kcsw;
            AntiH y;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                y.d[b] = -f * (lam[b][b].re + lam[b][b].re);
#pragma unroll
                for (int a = b + 1; a < 3; ++a) {
                    const cx<double> h = lam[b][a] + conj(lam[a][b]);
                    y.u[b + a - 1] = {f * h.im, -f * h.re};
                }
            }
            store_y(g, Y, l, s, plane, y);
        };
        cx<double> lam[3][3];
        if constexpr (CSW != 2) {
#pragma unroll 1
            for (int plane = 0; plane < 6; ++plane) plane_y(plane, lam);
        } else {
            int plane = 0;
            for (int mu = 0; mu < 4; ++mu)
                for (int nu = mu + 1; nu < 4; ++nu, ++plane) {
                    plane_y(plane, lam);
                    Mat3<double> F;
                    field_strength(g, u64, i, mu, nu, F);
                    cx<double> tr = {0.0, 0.0};
#pragma unroll
                    for (int a = 0; a < 3; ++a)
#pragma unroll
                        for (int b = 0; b < 3; ++b) tr = cmac(tr, F.m[a][b], lam[b][a]);
                    v[0] += 2.0 * kappa * tr.im;
                }
        }
    }
    if (CSW != 0) wg_reduce_store<1>(v, partials);
}

// entry (i, k), i != k
DD_INL cx<double> off_diag(const AntiH &M, int i, int k)
{
    return i < k ? M.u[i + k - 1] : cx<double>{-M.u[i + k - 1].re, M.u[i + k - 1].im};
}

// element (i, k) of A or of A^dagger
template <bool DAG> DD_INL cx<double> el(const Mat3<double> &A, int i, int k)
{
    return DAG ? conj(A.m[k][i]) : A.m[i][k];
}

// W += f sum_k conj(a[k][col]) b[k][row] over the two spins of two half spinors: the spin
// trace of an outer product of two projected spinors
DD_INL void half_outer(const Half<double> &a, const Half<double> &b, cx<double> f, Mat3<double> &W)
{
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const cx<double> s = cmacc(cmulc(a.v[0][c], b.v[0][r]), a.v[1][c], b.v[1][r]);
            W.m[r][c] = cmac(W.m[r][c], f, s);
        }
}

DD_INL int plane_index(int a, int b)  // a < b
{
    return a == 0 ? b - 1 : (a == 1 ? b + 1 : 5);
}

// A site with its block coordinates packed (two to a word), for steps in a direction that is known
// only at run time (uniform in the wavefront): shifts and kernel arguments read at a uniform index
// instead of indexed local arrays, which would be put into scratch memory or LDS.
struct SiteP {
    int l, s;
    unsigned long long B01, B23;
};

// the neighbour in direction mu (dir = +1 or -1); wrap: the hop crosses the lattice edge
DD_INL SiteP stepp(const Geom &g, const SiteP &a, int mu, int dir, bool &wrap)
{
    const int b = g.b[mu], sh = g.sh[mu], NB = g.NB[mu];
    const int c = ((a.s >> sh) & (b - 1)) + dir, B = (int)((mu < 2 ? a.B01 : a.B23) >> (32 * (mu & 1)));
    const int db = c < 0 ? -1 : c >= b ? 1 : 0;  // blocks moved
    int nB = B + db;
    wrap = nB < 0 || nB >= NB;
    nB = nB < 0 ? nB + NB : nB >= NB ? nB - NB : nB;
    SiteP r;
    r.l = a.l + (nB - B) * g.bstride[mu];
    r.s = a.s + ((dir - db * b) << sh);
    const unsigned long long d = (unsigned long long)(long long)(nB - B) << (32 * (mu & 1));
    r.B01 = a.B01 + (mu < 2 ? d : 0);
    r.B23 = a.B23 + (mu < 2 ? 0 : d);
    return r;
}

// The derivative of the plaquette through U_mu(n) in the (mu, nu) plane on the SD side, with Y of
// that plane at its corners: for the closed path U B C D (corners d1 = n, d2 = n + mu, d3, d4),
//   W += sgn [ Y2 B C D + B Y3 C D + B C Y4 D + B C D Y1 ] = sgn [ E_B (C D) + B (C E_D) ],
//   E_B = Y2 B + B Y3,  E_D = Y4 D + D Y1.
// C = U_mu(.)^dagger always; B is daggered on the -nu side and D on the +nu side.  E_D is formed
// once, C is read row by row into C D and C E_D, and E_B row by row into W, so at most five 3x3
// matrices are live (a 3x3 takes 36 VGPRs).
template <int SD>
DD_INL void staple_force(const Geom &g, const double2 *u64, const double2 *Y, const Geom &gu, const SiteP &si, const SiteP &sj, int mu,
                         int nu, int plane, double sgn, Mat3<double> &W)
{
    constexpr bool DB = SD < 0, DD = SD > 0;
    bool wrap;
    const SiteP ns = stepp(gu, si, nu, SD, wrap), js = stepp(gu, sj, nu, SD, wrap);
    auto index = [&](const SiteP &a) { return ((long long)a.l << g.lbvol) + a.s; };
    const long long i = index(si), j = index(sj);
    const long long n_s = index(ns), j_s = index(js);  // n + sd nu, n + mu + sd nu
    Mat3<double> T, T2;                        // C D and C E_D
    {
        Mat3<double> L, E;
        AntiH Y1, Y4;
        load_link64(g, u64, SD > 0 ? i : n_s, nu, L);  // D = U_nu(n)^dagger, or U_nu(n - nu)
        load_y(g, Y, i, plane, Y1);
        load_y(g, Y, n_s, plane, Y4);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const cx<double> x = el<DD>(L, a, b);
                const double d = Y4.d[a] + Y1.d[b];
                cx<double> s = {-d * x.im, d * x.re};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (k != a) s = cmac(s, off_diag(Y4, a, k), el<DD>(L, k, b));
                    if (k != b) s = cmac(s, el<DD>(L, a, k), off_diag(Y1, k, b));
                }
                E.m[a][b] = s;
            }
        Mat3<double> C;
        load_link64(g, u64, n_s, mu, C);  // C = U_mu(n + sd nu)^dagger
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                cx<double> s = el<true>(C, a, 0) * el<DD>(L, 0, b), s2 = el<true>(C, a, 0) * E.m[0][b];
#pragma unroll
                for (int k = 1; k < 3; ++k) {
                    s = cmac(s, el<true>(C, a, k), el<DD>(L, k, b));
                    s2 = cmac(s2, el<true>(C, a, k), E.m[k][b]);
                }
                T.m[a][b] = s;
                T2.m[a][b] = s2;
            }
    }
    Mat3<double> B;
    AntiH Y2, Y3;
    load_y(g, Y, j, plane, Y2);
    load_link64(g, u64, SD > 0 ? j : j_s, nu, B);  // B = U_nu(n + mu), or U_nu(n + mu - nu)^dagger
    load_y(g, Y, j_s, plane, Y3);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cx<double> e[3];  // row a of E_B
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const cx<double> x = el<DB>(B, a, b);
            const double d = Y2.d[a] + Y3.d[b];
            cx<double> s = {-d * x.im, d * x.re};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (k != a) s = cmac(s, off_diag(Y2, a, k), el<DB>(B, k, b));
                if (k != b) s = cmac(s, el<DB>(B, a, k), off_diag(Y3, k, b));
            }
            e[b] = s;
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            cx<double> s = e[0] * T.m[0][b], s2 = el<DB>(B, a, 0) * T2.m[0][b];
#pragma unroll
            for (int k = 1; k < 3; ++k) {
                s = cmac(s, e[k], T.m[k][b]);
                s2 = cmac(s2, el<DB>(B, a, k), T2.m[k][b]);
            }
            s = s + s2;
            W.m[a][b] = {fma_(sgn, s.re, W.m[a][b].re), fma_(sgn, s.im, W.m[a][b].im)};
        }
    }
}

// the hop term: k2 = 2 kappa phase times the spin traces of
//   [(1 - gamma_mu) psi(n+mu)] chi(n)^dagger  and  ([(1 + gamma_mu) psi(n)] chi(n+mu)^dagger)^dagger,
// each the trace over the two projected spins (1 -+ gamma_mu is twice a projector: the trace
// equals sum_k conj(P chi)_k (P psi)_k for mu < 3, half of it for mu = 3, where the projection
// carries the factor 2: k2 = kappa phase there)
template <int MU>
DD_INL void hop_force(const Geom &g, const SpinorField<0> &psi, const SpinorField<0> &chi, const SiteP &si,
                      const SiteP &sj, cx<double> k2, Mat3<double> &W)
{
    Spinor<double> p;
    Half<double> hp, hx;
    psi.load(g, sj.l, sj.s, p);
    project(MU, +1, p, hp);     // P^- psi(n+mu)
    chi.load(g, si.l, si.s, p);
    project(MU, +1, p, hx);     // P^- chi(n)
    half_outer(hx, hp, k2, W);  // W[b][a] += k2 sum conj(hx_a) hp_b
    psi.load(g, si.l, si.s, p);
    project(MU, -1, p, hp);     // P^+ psi(n)
    chi.load(g, sj.l, sj.s, p);
    project(MU, -1, p, hx);     // P^+ chi(n+mu)
    half_outer(hp, hx, k2, W);  // W[b][a] += k2 sum conj(hp_a) hx_b
}

// A workgroup takes 64 consecutive sites, wavefront mu the links in direction mu; writes the
// canonical [4][Lt][Lz][Ly][Lx][3][3].  B > 0: the block shape is B^4, known at compile time.
template <int B>
__global__ void __launch_bounds__(256, 2) k_force_w(Geom gin, SpinorField<0> psi, SpinorField<0> chi, const double2 *u64,
                                                 const double2 *Y, Phase4 ph, double kappa, int su3, double2 *out)
{
    const Geom g = fixed_shape<B>(gin);
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long i = (long long)xcd_remap(blockIdx.x, gridDim.x) * 64 + (threadIdx.x & 63);
    if (i >= g.V) return;
    Site st;
    decode(g, i, st);
    const SiteP si{st.l, st.s, (unsigned long long)st.B[0] | (unsigned long long)st.B[1] << 32,
                   (unsigned long long)st.B[2] | (unsigned long long)st.B[3] << 32};
    bool wrap;
    const SiteP sj = stepp(gin, si, mu, +1, wrap);

    Mat3<double> W;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) W.m[a][b] = {0.0, 0.0};
    {
        const cx<double> phase = wrap ? cx<double>{ph.re[mu], ph.im[mu]} : cx<double>{1.0, 0.0};
        const cx<double> k2 = ((mu == 3 ? 1.0 : 2.0) * kappa) * phase;
        switch (mu) {
        case 0: hop_force<0>(g, psi, chi, si, sj, k2, W); break;
        case 1: hop_force<1>(g, psi, chi, si, sj, k2, W); break;
        case 2: hop_force<2>(g, psi, chi, si, sj, k2, W); break;
        default: hop_force<3>(g, psi, chi, si, sj, k2, W); break;
        }
    }

    // ---- clover term: the six plaquettes through the link, staple by staple
    if (Y) {
#pragma unroll 1
        for (int nu = 0; nu < 4; ++nu) {
            if (nu == mu) continue;
            const int plane = mu < nu ? plane_index(mu, nu) : plane_index(nu, mu);
            const double orient = mu < nu ? 1.0 : -1.0;
            staple_force<+1>(g, u64, Y, gin, si, sj, mu, nu, plane, orient, W);
            staple_force<-1>(g, u64, Y, gin, si, sj, mu, nu, plane, -orient, W);
        }
    }

    // ---- output
    Mat3<double> O;
    if (su3) {
        Mat3<double> U, X;
        load_link64(g, u64, i, mu, U);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                cx<double> t = U.m[a][0] * W.m[0][b];
#pragma unroll
                for (int k = 1; k < 3; ++k) t = cmac(t, U.m[a][k], W.m[k][b]);
                X.m[a][b] = t;
            }
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                cx<double> d = X.m[a][b] - conj(X.m[b][a]);
                O.m[a][b] = {-0.5 * d.im, 0.5 * d.re};  // (i/2) d
            }
        const double tr = (O.m[0][0].re + O.m[1][1].re + O.m[2][2].re) / 3.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) O.m[a][a].re -= tr;
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) O.m[a][b] = conj(W.m[b][a]);
    }
    const long long n = lex_index(g, st);
    double2 *dst = out + ((long long)mu * g.V + n) * 9;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) dst[a * 3 + b] = make_double2(O.m[a][b].re, O.m[a][b].im);
}

hipError_t launch_force(const Geom &g, hipStream_t st, const ForceArgs &a)
{
    const int nwg = blas_grid_sites(g);
    auto ky = !a.partials ? k_force_y<0> : a.csw != 0.0 ? k_force_y<1> : k_force_y<2>;
    hipLaunchKernelGGL(ky, dim3(nwg), dim3(BLAS_WG), 0, st, g, (const double2 *)a.psi_can, (const double2 *)a.chi_can,
                       SpinorField<0>{(double2 *)a.psi}, SpinorField<0>{(double2 *)a.chi}, (const double2 *)a.u64, (const double2 *)a.clov64, a.sig, a.kcsw,
                       a.kappa, a.csw, (double2 *)a.y, a.partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.partials) {
        e = launch_finalize(st, a.partials, nwg, 1, a.dcsw);
        if (e != hipSuccess) return e;
    }
    const bool cube4 = g.b[0] == 4 && g.b[1] == 4 && g.b[2] == 4 && g.b[3] == 4;
    hipLaunchKernelGGL((cube4 ? k_force_w<4> : k_force_w<0>), dim3((unsigned)((g.V + 63) / 64)), dim3(256), 0, st, g,
                       SpinorField<0>{(double2 *)a.psi}, SpinorField<0>{(double2 *)a.chi}, (const double2 *)a.u64,
                       a.kcsw != 0.0 ? (const double2 *)a.y : nullptr, a.phase, a.kappa, a.su3, (double2 *)a.out);
    return hipGetLastError();
}

}  // namespace dd
