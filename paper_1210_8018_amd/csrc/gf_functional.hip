// The differentiable functional: F of Eq. 1 as a function of gauge
// parameters, F_U[g] = 1/(12 V) sum_x sum_mu Re Tr[g(x) U_mu(x) g^dag(x+mu)]
// with g(x) = exp(i sum_a lambda_a omega_a(x)), and its gradients with respect
// to omega and to the links. Single configuration (slot 0).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gf_device.h"
#include "gf_internal.h"

namespace gfk {

namespace {

// Q = sum_a omega_a lambda_a (hermitian, traceless) and Q^2.
struct Herm {
    double a, b, c;           // diagonal
    double2 q01, q02, q12;    // upper triangle; the lower one is its conjugate
};

__device__ __forceinline__ double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }

__device__ __forceinline__ Herm herm_of(const double w[8])
{
    const double r3 = 0.57735026918962576451;
    Herm Q;
    Q.a = w[2] + w[7] * r3;
    Q.b = -w[2] + w[7] * r3;
    Q.c = -2.0 * w[7] * r3;
    Q.q01 = make_double2(w[0], -w[1]);
    Q.q02 = make_double2(w[3], -w[4]);
    Q.q12 = make_double2(w[5], -w[6]);
    return Q;
}

__device__ __forceinline__ Herm herm_square(const Herm &Q)
{
    const double n01 = cabs2(Q.q01), n02 = cabs2(Q.q02), n12 = cabs2(Q.q12);
    Herm S;
    S.a = Q.a * Q.a + n01 + n02;
    S.b = Q.b * Q.b + n01 + n12;
    S.c = Q.c * Q.c + n02 + n12;
    S.q01 = cfmac(Q.q02, Q.q12, cscale(Q.q01, Q.a + Q.b));
    S.q02 = cfma(Q.q01, Q.q12, cscale(Q.q02, Q.a + Q.c));
    S.q12 = ccfma(Q.q01, Q.q02, cscale(Q.q12, Q.b + Q.c));
    return S;
}

// exp(i Q) = f0 + f1 Q + f2 Q^2: Q^3 = p Q + d (Cayley and Hamilton, Tr Q = 0)
// with p = Tr Q^2 / 2 and d = det Q reduces every power. The coefficients of
// Q / 2^j come from the Taylor series, summed from its last term with Q
// (s0 + s1 Q + s2 Q^2) = d s2 + (s0 + p s2) Q + s1 Q^2, and exp(2 Z) = exp(Z)^2
// is taken on the coefficients, so that no matrix product is needed beyond
// Q^2. DERIV: also the derivatives with respect to p and d.
//
// At most kCoefDoublings times: where two eigenvalues of Q nearly agree, the
// coefficients grow as 2^j and their derivatives as 8^j with the number j of
// doublings, and cancel in what they multiply. Beyond that the matrix itself
// is squared. Errors near lambda_8, rms, |omega| = 150 and 450: exp 3.1e-14 and
// 7e-14 (doublings throughout 7e-13 and 8e-12, the matrix series 6e-14 and
// 2e-13), dF/domega 5e-14 and 2e-13 (2e-12 and 2e-10; 8e-14 and 4e-13). With
// four doublings neither is above the matrix series in any direction at any
// size tried (|omega| 0.1 to 450), and omega of standard deviation 0.6 needs
// no more (24^4, standard deviation 0.6 as before; 6: k_fg_backward 114 -> 125
// us, k_expg 16 -> 20).
struct ExpCoef {
    double2 f[3];   // of 1, Q, Q^2 of the scaled Q
    double2 fp[3];  // derivatives with respect to p ...
    double2 fd[3];  // ... and d of the scaled Q
};

constexpr int kCoefDoublings = 4;
constexpr int kExpTerms = 16;  // |Q| <= 1/2 (scaled): the first term left out is below 1e-18

__device__ __forceinline__ double2 times_i(double2 a, double s) { return make_double2(-s * a.y, s * a.x); }

template <bool DERIV>
__device__ __forceinline__ void exp_coef(ExpCoef &E, double p, double d, int j)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) E.f[k] = E.fp[k] = E.fd[k] = cz();
    E.f[0].x = 1.0;
#pragma unroll
    for (int n = kExpTerms; n >= 1; --n) {
        const double r = 1.0 / (double)n;
        double2 *f = E.f, *fp = E.fp, *fd = E.fd;
        const double2 t0 = cscale(f[2], d), t1 = make_double2(f[0].x + p * f[2].x, f[0].y + p * f[2].y), t2 = f[1];
        if constexpr (DERIV) {
            const double2 p0 = cscale(fp[2], d);
            const double2 p1 = make_double2(fp[0].x + f[2].x + p * fp[2].x, fp[0].y + f[2].y + p * fp[2].y);
            const double2 p2 = fp[1];
            const double2 d0 = make_double2(f[2].x + d * fd[2].x, f[2].y + d * fd[2].y);
            const double2 d1 = make_double2(fd[0].x + p * fd[2].x, fd[0].y + p * fd[2].y);
            const double2 d2 = fd[1];
            fp[0] = times_i(p0, r);
            fp[1] = times_i(p1, r);
            fp[2] = times_i(p2, r);
            fd[0] = times_i(d0, r);
            fd[1] = times_i(d1, r);
            fd[2] = times_i(d2, r);
        }
        f[0] = times_i(t0, r);
        f[0].x += 1.0;
        f[1] = times_i(t1, r);
        f[2] = times_i(t2, r);
    }
    for (int k = 0; k < j; ++k) {
        const double2 a = E.f[0], b = E.f[1], c = E.f[2];
        const double2 aa = cmul(a, a), ab = cmul(a, b), bc = cmul(b, c), cc = cmul(c, c);
        const double2 g2 = cadd(cmul(b, b), cscale(cmul(a, c), 2.0));
        if constexpr (DERIV) {
            // derivative of the square's coefficients (below) along a change
            // (da, db, dc) of the coefficients
            const auto along = [&](double2 *v) {
                const double2 da = v[0], db = v[1], dc = v[2];
                const double2 dbc = cfma(b, dc, cmul(db, c)), dcc = cmul(c, dc);  // d(bc), d(cc)/2
                const double2 v0 = cadd(cmul(a, da), cscale(dbc, d));
                const double2 v1 = cadd(cfma(b, da, cmul(a, db)), cadd(cscale(dbc, p), cscale(dcc, d)));
                const double2 v2 = cadd(cfma(a, dc, cfma(c, da, cmul(b, db))), cscale(dcc, p));
                v[0] = cscale(v0, 2.0);
                v[1] = cscale(v1, 2.0);
                v[2] = cscale(v2, 2.0);
            };
            along(E.fp);
            E.fp[1] = cadd(E.fp[1], cscale(bc, 2.0));
            E.fp[2] = cadd(E.fp[2], cc);
            along(E.fd);
            E.fd[0] = cadd(E.fd[0], cscale(bc, 2.0));
            E.fd[1] = cadd(E.fd[1], cc);
        }
        E.f[0] = cadd(aa, cscale(bc, 2.0 * d));
        E.f[1] = cadd(cscale(cadd(ab, cscale(bc, p)), 2.0), cscale(cc, d));
        E.f[2] = cadd(g2, cscale(cc, p));
    }
}

// The scaled Q = Q / 2^j (|Q| <= 1/2 in the Frobenius norm), its square and
// invariants, and j.
struct Scaled {
    Herm Q, Q2;
    double p, d;
    int j;
};

// j: the smallest with |Q| <= 2^j / 2.
__device__ __forceinline__ int doublings(const double w[8])
{
    double n = 0.0;
#pragma unroll
    for (int a = 0; a < 8; ++a) n += w[a] * w[a];
    n = sqrt(2.0 * n);  // Tr Q^2 = 2 sum_a omega_a^2
    int j = 0;
    while (n > 0.5 && j < 60) {
        n *= 0.5;
        ++j;
    }
    return j;
}

__device__ __forceinline__ Scaled scaled_of(const double w[8])
{
    Scaled s;
    s.j = doublings(w);
    const double sc = ldexp(1.0, -s.j);
    double v[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) v[a] = w[a] * sc;
    s.Q = herm_of(v);
    s.Q2 = herm_square(s.Q);
    const Herm &Q = s.Q;
    s.p = 0.5 * (s.Q2.a + s.Q2.b + s.Q2.c);
    const double2 t = cmul(Q.q01, Q.q12);
    s.d = Q.a * (Q.b * Q.c - cabs2(Q.q12)) - Q.b * cabs2(Q.q02) - Q.c * cabs2(Q.q01) +
          2.0 * (t.x * Q.q02.x + t.y * Q.q02.y);
    return s;
}

// f0 + f1 Q + f2 Q^2, rows 0 and 1 (row 2 of a special unitary matrix is
// conj(r0 x r1)).
__device__ __forceinline__ M3 exp_rows(const ExpCoef &E, const Herm &Q, const Herm &S)
{
    const double2 f0 = E.f[0], f1 = E.f[1], f2 = E.f[2];
    const auto diag = [&](double q, double s) {
        return make_double2(f0.x + f1.x * q + f2.x * s, f0.y + f1.y * q + f2.y * s);
    };
    M3 m;
    m.e[0] = diag(Q.a, S.a);
    m.e[4] = diag(Q.b, S.b);
    m.e[1] = cfma(f2, S.q01, cmul(f1, Q.q01));
    m.e[2] = cfma(f2, S.q02, cmul(f1, Q.q02));
    m.e[3] = cfmac(f2, S.q01, cmulc(f1, Q.q01));
    m.e[5] = cfma(f2, S.q12, cmul(f1, Q.q12));
    return m;
}

// exp of the unscaled Q (|Q| = 2^j |scaled Q|, j > kCoefDoublings) from rows 0
// and 1 after kCoefDoublings doublings, projected to SU(3): a squaring doubles
// the distance from it.
__device__ __forceinline__ void square_up(M3 &m, int j)
{
    m3_row2(m);
    for (int k = kCoefDoublings; k < j; ++k) m = m3_mul(m, m);
    m3_reunit(m);
}

__device__ __forceinline__ void load_omega(const double *__restrict__ om, int V, int s, double w[8])
{
#pragma unroll
    for (int a = 0; a < 8; ++a) w[a] = om[(size_t)a * V + s];
}

// g(x) = exp(i sum_a lambda_a omega_a(x)) in two-row form into the
// configuration's g buffer. Bound by memory (64 + 96 B per site): 24^4
// 12 us (4.3 TB/s); by 18 terms of the matrix series and three rows 47 us.
__global__ __launch_bounds__(kSiteBlock) void k_expg(const Cfg *__restrict__ cfgs, const double *__restrict__ omega)
{
    const Cfg &C = cfgs[0];
    const int s = blockIdx.x * kSiteBlock + threadIdx.x;
    if (s >= C.V) return;
    double w[8];
    load_omega(omega, C.V, s, w);
    const Scaled q = scaled_of(w);
    ExpCoef E;
    exp_coef<false>(E, q.p, q.d, min(q.j, kCoefDoublings));
    M3 g = exp_rows(E, q.Q, q.Q2);
    if (q.j > kCoefDoublings) square_up(g, q.j);
    m3_store12(C.g, C.V, s, g);
}

// Work-item of a t-walk: kSiteBlock consecutive sites of the (x, y, z) volume
// (nb3 such sets), tch t-slices.
struct Walk {
    int s3, t0, f[3], b[3];  // site, first slice, spatial neighbours (offsets within a slice)
    bool inside;
};

__device__ __forceinline__ Walk walk_of(const Cfg &C, int blk, int nb3, int tch)
{
    Walk w;
    const int tc = blk / nb3;
    w.t0 = tc * tch;
    w.s3 = (blk - tc * nb3) * kSiteBlock + threadIdx.x;
    w.inside = w.s3 < C.V3;
    const int Lx = C.dims[0], Ly = C.dims[1], Lz = C.dims[2], V2 = C.V2;
    const int r = w.s3 / Lx, x = w.s3 - r * Lx, z = r / Ly, y = r - z * Ly;
    w.f[0] = (x + 1 == Lx) ? w.s3 - (Lx - 1) : w.s3 + 1;
    w.f[1] = (y + 1 == Ly) ? w.s3 - (Ly - 1) * Lx : w.s3 + Lx;
    w.f[2] = (z + 1 == Lz) ? w.s3 - (Lz - 1) * V2 : w.s3 + V2;
    w.b[0] = (x == 0) ? w.s3 + (Lx - 1) : w.s3 - 1;
    w.b[1] = (y == 0) ? w.s3 + (Ly - 1) * Lx : w.s3 - Lx;
    w.b[2] = (z == 0) ? w.s3 + (Lz - 1) * V2 : w.s3 - V2;
    return w;
}

// a += b c
__device__ __forceinline__ void m3_acc(M3 &a, const M3 &b, const M3 &c)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) a.e[i * 3 + j] = cfma(b.e[i * 3 + k], c.e[k * 3 + j], a.e[i * 3 + j]);
}

// Re Tr[w gf^dag] = sum_ij Re(w_ij conj(gf_ij))
__device__ __forceinline__ double re_tr_dag(const M3 &w, const M3 &gf, double acc)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        acc = fma(w.e[k].x, gf.e[k].x, acc);
        acc = fma(w.e[k].y, gf.e[k].y, acc);
    }
    return acc;
}

// Per-block partial sums of sum_mu Re Tr[g(x) U_mu(x) g^dag(x+mu)] (Eq. 1),
// two doubles per block. A block walks tch t-slices; g(x + t) of one is g(x)
// of the next. Bound by memory (576 B of links and 96 of g per site): 24^4
// 34 us (6.6 TB/s); a site per work-item and three-row g 62 us.
__global__ __launch_bounds__(kSiteBlock) void k_fg_partials(const Cfg *__restrict__ cfgs, int nb3, int tch)
{
    __shared__ dd red[2 * (kSiteBlock / 64)];
    const Cfg &C = cfgs[0];
    const int V = C.V, Lt = C.dims[3];
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const Walk w = walk_of(C, blk, nb3, tch);
    dd sum = {0.0, 0.0}, zero = {0.0, 0.0};
    if (w.inside) {
        const double2 *__restrict__ G = C.g, *__restrict__ U = C.U;
        M3 gx = m3_load12(G, V, w.s3 + C.V3 * w.t0);
        for (int t = w.t0; t < w.t0 + tch; ++t) {
            const int ts = C.V3 * t, tn = C.V3 * (t + 1 == Lt ? 0 : t + 1);
            double acc = 0.0;
#pragma unroll
            for (int mu = 0; mu < 4; ++mu) {
                M3 u;
#pragma unroll
                for (int k = 0; k < 9; ++k) u.e[k] = ld_stream(U + (size_t)(9 * mu + k) * V + w.s3 + ts);
                const M3 gf = m3_load12(G, V, mu < 3 ? w.f[mu < 3 ? mu : 0] + ts : w.s3 + tn);
                acc = re_tr_dag(m3_mul(gx, u), gf, acc);
                if (mu == 3) gx = gf;
            }
            sum = dd_add(sum, dd{acc, 0.0});
        }
    }
    block_sum2(sum, zero, red);
    if (threadIdx.x == 0) {
        double *p = C.partials + (size_t)blk * 2;
        p[0] = sum.hi;
        p[1] = sum.lo;
    }
}

// Sum of the partial pairs of every block, times `scale`, to *out.
__global__ __launch_bounds__(256) void k_sum_partials(const Cfg *__restrict__ cfgs, int nblk, double scale,
                                                      double *__restrict__ out)
{
    __shared__ dd red[2 * (256 / 64)];
    const Cfg &C = cfgs[0];
    dd f = {0.0, 0.0}, z = {0.0, 0.0};
    for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
        const double *p = C.partials + (size_t)i * 2;
        f = dd_add(f, dd{p[0], p[1]});
    }
    block_sum2(f, z, red);
    if (threadIdx.x == 0) *out = (f.hi + f.lo) * scale;
}

// Tr(Q M) for hermitian Q: sum_ij Q_ij M_ji
__device__ __forceinline__ double2 tr_herm(const Herm &Q, const M3 &m)
{
    double2 t = make_double2(Q.a * m.e[0].x + Q.b * m.e[4].x + Q.c * m.e[8].x,
                             Q.a * m.e[0].y + Q.b * m.e[4].y + Q.c * m.e[8].y);
    t = cfma(Q.q01, m.e[3], t);
    t = ccfma(Q.q01, m.e[1], t);
    t = cfma(Q.q02, m.e[6], t);
    t = ccfma(Q.q02, m.e[2], t);
    t = cfma(Q.q12, m.e[7], t);
    return ccfma(Q.q12, m.e[5], t);
}

__device__ __forceinline__ M3 herm_full(const Herm &Q)
{
    M3 m;
    m.e[0] = make_double2(Q.a, 0.0);
    m.e[4] = make_double2(Q.b, 0.0);
    m.e[8] = make_double2(Q.c, 0.0);
    m.e[1] = Q.q01;
    m.e[2] = Q.q02;
    m.e[5] = Q.q12;
    m.e[3] = cconj(Q.q01);
    m.e[6] = cconj(Q.q02);
    m.e[7] = cconj(Q.q12);
    return m;
}

// dF/domega_a(x) = Re Tr[(dg/domega_a) Sigma] scale for the staple sum Sigma.
// With g = f0 + f1 Q + f2 Q^2 and f_i functions of p and d,
//   dg/domega_a = f1 lambda_a + f2 (Q lambda_a + lambda_a Q)
//               + Tr(Q lambda_a) sum_i fp_i Q^i + Tr(Q^2 lambda_a) sum_i fd_i Q^i
// (dp = Tr(Q lambda_a), dd = Tr(adj(Q) lambda_a), adj(Q) = Q^2 - p, Tr lambda_a
// = 0), so it is Re Tr(lambda_a M) with M = f1 Sigma + f2 (Sigma Q + Q Sigma)
// + Bp Q + Bd Q^2, Bp = sum_i fp_i Tr(Q^i Sigma) and Bd alike. Everything in
// the scaled Q, whose derivative is 2^-j lambda_a. A squaring of the matrix, g
// = h^2, turns Re Tr[dg Sigma] into Re Tr[dh (h Sigma + Sigma h)]; the h of
// all squarings commute, so that they can be taken from the smallest on.
__device__ __forceinline__ void omega_gradient(double w[8], M3 &Sig, double scale, double *__restrict__ out, int V,
                                               int s)
{
    if (doublings(w) > kCoefDoublings) {
        const Scaled q = scaled_of(w);
        ExpCoef E;
        exp_coef<false>(E, q.p, q.d, kCoefDoublings);
        M3 h = exp_rows(E, q.Q, q.Q2);
        m3_reunit(h);
        for (int k = kCoefDoublings; k < q.j; ++k) {
            M3 a = m3_mul(h, Sig);
            m3_fence(a);
            m3_acc(a, Sig, h);
            m3_fence(a);
            Sig = a;
            h = m3_mul(h, h);
            m3_fence(h);
        }
        // Q is formed again below, not kept beside all of the above (spilled)
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(w[a]));
    }
    const Scaled q = scaled_of(w);
    ExpCoef E;
    exp_coef<true>(E, q.p, q.d, min(q.j, kCoefDoublings));
    const double2 t0 = cadd(cadd(Sig.e[0], Sig.e[4]), Sig.e[8]), t1 = tr_herm(q.Q, Sig), t2 = tr_herm(q.Q2, Sig);
    const double2 Bp = cfma(E.fp[2], t2, cfma(E.fp[1], t1, cmul(E.fp[0], t0)));
    const double2 Bd = cfma(E.fd[2], t2, cfma(E.fd[1], t1, cmul(E.fd[0], t0)));
    const M3 Q = herm_full(q.Q), S = herm_full(q.Q2);
    const M3 A = m3_add(m3_mul(Sig, Q), m3_mul(Q, Sig));
    M3 m;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        m.e[k] = cfma(Bd, S.e[k], cfma(Bp, Q.e[k], cfma(E.f[2], A.e[k], cmul(E.f[1], Sig.e[k]))));
    // Re Tr(lambda_a M)
    const double r3 = 0.57735026918962576451, sc = scale * ldexp(1.0, -q.j);
    out[s] = sc * (m.e[1].x + m.e[3].x);
    out[(size_t)1 * V + s] = sc * (m.e[3].y - m.e[1].y);
    out[(size_t)2 * V + s] = sc * (m.e[0].x - m.e[4].x);
    out[(size_t)3 * V + s] = sc * (m.e[2].x + m.e[6].x);
    out[(size_t)4 * V + s] = sc * (m.e[6].y - m.e[2].y);
    out[(size_t)5 * V + s] = sc * (m.e[5].x + m.e[7].x);
    out[(size_t)6 * V + s] = sc * (m.e[7].y - m.e[5].y);
    out[(size_t)7 * V + s] = sc * r3 * (m.e[0].x + m.e[4].x - 2.0 * m.e[8].x);
}

// acc + (a b)^dag
__device__ __forceinline__ void add_dag(M3 &acc, const M3 &m)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            acc.e[i * 3 + j].x += m.e[j * 3 + i].x;
            acc.e[i * 3 + j].y -= m.e[j * 3 + i].y;
        }
}

// Gradients of Eq. 1 with g = exp(i omega.lambda):
//   dF/domega (omega_gradient) with
//   Sigma(x) = sum_mu [U_mu(x) g^dag(x+mu) + (g(x-mu) U_mu(x-mu))^dag], and
//   dF/dRe U_mu(x) + i dF/dIm U_mu(x) = g^dag(x) g(x+mu) / (12 V).
// A block walks tch t-slices: g(x + t) of one slice is g(x) of the next, and
// g(x - t) U_t(x - t) of a slice is formed in the one before.
//
// What bounds it: memory (links in and out, 1152 B, and 224 of g and omega per
// site): 24^4 108 us (4.2 TB/s, two waves per SIMD); a site per work-item and the derivative of the
// exponential by 18 terms of the matrix series (54 products) 197 us.
template <bool DOM, bool DU>
__global__ __launch_bounds__(kSiteBlock, 2) void k_fg_backward(const Cfg *__restrict__ cfgs, int nb3, int tch,
                                                               const double *__restrict__ omega, double scale,
                                                               double *__restrict__ d_omega, double2 *__restrict__ d_U)
{
    const Cfg &C = cfgs[0];
    const int V = C.V, Lt = C.dims[3];
    const Walk w = walk_of(C, xcd_remap(blockIdx.x, gridDim.x), nb3, tch);
    if (!w.inside) return;
    const double2 *G = C.g, *U = C.U;
    M3 gx = m3_load12(G, V, w.s3 + C.V3 * w.t0);
    M3 gu;  // g(x - t) U_t(x - t)
    if constexpr (DOM) {
        const int sp = w.s3 + C.V3 * (w.t0 == 0 ? Lt - 1 : w.t0 - 1);
        gu = m3_mul(m3_load12(G, V, sp), m3_load(U + (size_t)27 * V, V, sp));
    }
    for (int t = w.t0; t < w.t0 + tch; ++t) {
        const int ts = C.V3 * t, s = w.s3 + ts;
        M3 Sig = m3_zero();
        if constexpr (DOM) add_dag(Sig, gu);
        M3 gn;
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const double2 *Um = U + (size_t)mu * 9 * V;
            const M3 gf = m3_load12(G, V, mu < 3 ? w.f[mu < 3 ? mu : 0] + ts
                                                 : w.s3 + C.V3 * (t + 1 == Lt ? 0 : t + 1));
            if constexpr (DU) {
                const M3 dU = m3_scale(m3_dag_mul(gx, gf), scale);
#pragma unroll
                for (int k = 0; k < 9; ++k) st_stream(d_U + (size_t)(9 * mu + k) * V + s, dU.e[k]);
            }
            if constexpr (DOM) {
                const M3 u = m3_load(Um, V, s);
                Sig = m3_add(Sig, m3_mul_dag(u, gf));
                m3_fence(Sig);
                if (mu < 3) {
                    const int sb = w.b[mu < 3 ? mu : 0] + ts;
                    add_dag(Sig, m3_mul(m3_load12(G, V, sb), m3_load(Um, V, sb)));
                    m3_fence(Sig);
                } else {
                    gu = m3_mul(gx, u);
                    m3_fence(gu);
                }
            }
            if (mu == 3) gn = gf;
        }
        if constexpr (DOM) {
            double om[8];
            load_omega(omega, V, s, om);
            omega_gradient(om, Sig, scale, d_omega, V, s);
        }
        gx = gn;
    }
}

}  // namespace

hipError_t launch_functional_g(const Launch &L, int nblk_site, const MarchPlan &m, const double *omega, double scale,
                               double *out)
{
    const int nblk = m.nb3 * (m.Lt / m.tch);
    hipLaunchKernelGGL(k_expg, dim3(nblk_site), dim3(kSiteBlock), 0, L.stream, L.cfgs, omega);
    hipLaunchKernelGGL(k_fg_partials, dim3(nblk), dim3(kSiteBlock), 0, L.stream, L.cfgs, m.nb3, m.tch);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, L.stream, L.cfgs, nblk, scale, out);
    return hipGetLastError();
}

hipError_t launch_functional_g_backward(const Launch &L, int nblk_site, const MarchPlan &m, const double *omega,
                                        double scale, double *d_omega, double2 *d_U)
{
    const dim3 grid(m.nb3 * (m.Lt / m.tch)), blk(kSiteBlock);
    hipLaunchKernelGGL(k_expg, dim3(nblk_site), blk, 0, L.stream, L.cfgs, omega);
    if (d_omega && d_U)
        hipLaunchKernelGGL((k_fg_backward<true, true>), grid, blk, 0, L.stream, L.cfgs, m.nb3, m.tch, omega, scale,
                           d_omega, d_U);
    else if (d_omega)
        hipLaunchKernelGGL((k_fg_backward<true, false>), grid, blk, 0, L.stream, L.cfgs, m.nb3, m.tch, omega, scale,
                           d_omega, d_U);
    else
        hipLaunchKernelGGL((k_fg_backward<false, true>), grid, blk, 0, L.stream, L.cfgs, m.nb3, m.tch, omega, scale,
                           d_omega, d_U);
    return hipGetLastError();
}

}  // namespace gfk
