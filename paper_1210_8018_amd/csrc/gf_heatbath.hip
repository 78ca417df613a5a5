// Input generator on the GPU: thermalised SU(3) configurations of the Wilson
// action S = beta sum_P (1 - Re Tr U_P / 3), the kind of configuration the
// paper gauge-fixes (section 3, beta = 5.8 to 6.2). Cabibbo-Marinari
// pseudo-heatbath over the SU(2) subgroups (0,1), (0,2), (1,2) with
// Kennedy-Pendleton draws, microcanonical overrelaxation, Philox4x32-10
// random numbers with one counter per draw (Salmon et al., SC 2011). The
// draw-to-counter assignment and the order of updates follow one published
// definition so that a CPU implementation reproduces the same configuration.
// Also the average plaquette.
#include <hip/hip_runtime.h>

#include "gf_device.h"
#include "gf_internal.h"

namespace gfk {

namespace {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;
constexpr int kHbMaxAttempts = 64;  // Kennedy-Pendleton attempts per draw
constexpr int kHbDirectionSlot = 255;

struct U4 {
    uint32_t v[4];
};

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                            uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += kPhiloxW0;
            k1 += kPhiloxW1;
        }
        const uint32_t hi0 = __umulhi(kPhiloxM0, c0), lo0 = kPhiloxM0 * c0;
        const uint32_t hi1 = __umulhi(kPhiloxM1, c2), lo1 = kPhiloxM1 * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    U4 o;
    o.v[0] = c0;
    o.v[1] = c1;
    o.v[2] = c2;
    o.v[3] = c3;
    return o;
}

// A 32-bit draw as a uniform number in (0, 1].
__device__ __forceinline__ double unit_open0(uint32_t u) { return ((double)u + 1.0) * (1.0 / 4294967296.0); }

// Draw `slot` (attempt j, or the direction) of subgroup k of the update of
// U_mu(site) in heatbath sweep n: counter (site, mu + 4k + 16 slot, n lo, n hi).
__device__ __forceinline__ U4 hb_draw(int site, int mu, int k, int slot, long long n, uint32_t k0, uint32_t k1)
{
    return philox4x32_10((uint32_t)site, (uint32_t)(mu + 4 * k + 16 * slot),
                         (uint32_t)((unsigned long long)n & 0xffffffffull), (uint32_t)((unsigned long long)n >> 32),
                         k0, k1);
}

constexpr double kTwoPi = 6.28318530717958647692;

// x in SU(2) with density exp(a x0) (Haar measure): x0 by Kennedy-Pendleton
// rejection from sqrt(1 - x0^2) e^(a x0), the vector part uniform on its
// sphere. false if no attempt is accepted within the cap (x untouched).
__device__ bool kp_draw(double a, int site, int mu, int k, long long n, uint32_t k0, uint32_t k1, double x[4])
{
    for (int j = 0; j < kHbMaxAttempts; ++j) {
        const U4 r = hb_draw(site, mu, k, j, n, k0, k1);
        const double r1 = unit_open0(r.v[0]), r2 = unit_open0(r.v[1]), r3 = unit_open0(r.v[2]),
                     r4 = unit_open0(r.v[3]);
        const double c = cos(kTwoPi * r2);
        const double lam2 = -(log(r1) + c * c * log(r3)) / (2.0 * a);
        if (r4 * r4 <= 1.0 - lam2) {
            x[0] = 1.0 - 2.0 * lam2;
            const U4 d = hb_draw(site, mu, k, kHbDirectionSlot, n, k0, k1);
            const double ct = 2.0 * unit_open0(d.v[0]) - 1.0, phi = kTwoPi * unit_open0(d.v[1]);
            const double rad = sqrt(fmax(0.0, 1.0 - x[0] * x[0]));
            const double st = sqrt(fmax(0.0, 1.0 - ct * ct));
            x[1] = rad * st * cos(phi);
            x[2] = rad * st * sin(phi);
            x[3] = rad * ct;
            return true;
        }
    }
    return false;
}

// The generator works on a copy of the links in the workspace, split by site
// parity so that the sites of one class are consecutive: [4][9][V], the sites
// of parity p (of x + y + z + t) in the half p of every plane, in
// lexicographic order, x halved. The copy takes the two two-row link buffers
// (768 bytes per site for 576 needed), which hold nothing between calls.
__device__ __forceinline__ double2 *hb_links(const Cfg &C) { return C.U12[0]; }

// What a class reads and writes: the caller's array (a call of one sweep of a
// small lattice), the copy as the caller's full matrices (the first of several
// sweeps), the copy in two-row form.
enum HbForm : int { kHbCaller, kHbFull, kHbTwoRow };

// Element s of the copy: site of parity par, (xh, row) = (x / 2, y + Ly (z + Lz t)).
struct HbGeom {
    int half, V2h, V3h;  // Lx / 2 sites of a parity per row; per xy-plane; per (x, y, z) volume
};

// A link of the copy. FULL: all nine elements, the caller's matrices (a
// call's first sweep). Otherwise two rows, the third rebuilt: every link is
// then one that m3_reunit has projected, whose third row is m3_row2 of the
// other two, so both forms give the same matrix bit for bit. The element
// offset within a plane is an unsigned 32-bit byte count (16 V < 2^32 for
// every V the library takes), so the plane's address stays in scalar
// registers.
template <bool FULL>
__device__ __forceinline__ M3 hb_load(const double2 *base, int V, int s)
{
    M3 m;
    const uint32_t off = (uint32_t)s * 16u;
#pragma unroll
    for (int k = 0; k < (FULL ? 9 : 6); ++k)
        m.e[k] = *(const double2 *)((const char *)(base + (size_t)k * V) + off);
    return m;
}

// Index in a half of the copy of the neighbour one step along MU (STEP = +1
// or -1) of the site (xh, c[1], c[2], c[3]) with x = 2 xh + odd, flat index i:
// along y, z and t the neighbour keeps x and so xh; along x it keeps xh or
// moves it by one, as x is odd or even. `odd` of the neighbour: 1 - odd along
// x (c[] and odd are updated by the caller).
template <int MU, int STEP>
__device__ __forceinline__ int hb_hop(const HbGeom &G, const int *L, const int (&c)[4], int odd, int i)
{
    if constexpr (MU == 0) {
        if constexpr (STEP > 0) {
            if (!odd) return i;
            return (c[0] + 1 == G.half) ? i - (G.half - 1) : i + 1;
        } else {
            if (odd) return i;
            return (c[0] == 0) ? i + (G.half - 1) : i - 1;
        }
    } else {
        const int st = MU == 1 ? G.half : MU == 2 ? G.V2h : G.V3h;
        if constexpr (STEP > 0)
            return (c[MU] + 1 == L[MU]) ? i - (L[MU] - 1) * st : i + st;
        else
            return (c[MU] == 0) ? i + (L[MU] - 1) * st : i - st;
    }
}

// Where the half of a parity begins, and the element of index i there whose x
// is 2 xh + odd (the caller's array is not split: 2 i + odd).
template <HbForm F>
__device__ __forceinline__ int hb_half(int V, int par)
{
    return F == kHbCaller || !par ? 0 : V / 2;
}
template <HbForm F>
__device__ __forceinline__ int hb_element(int i, int odd)
{
    return F == kHbCaller ? 2 * i + odd : i;
}

// The three links of one staple of direction NU of U_MU(s): the upper one
// U_nu(s+mu) U_mu^dag(s+nu) U_nu^dag(s), or (LOWER) U_nu^dag(s+mu-nu)
// U_mu^dag(s-nu) U_nu(s-nu). i: index of s in the half `par`; ip: of s + mu
// in the other half. s + nu and s - nu are of the other parity, s + mu - nu
// of the parity of s.
struct Staple {
    M3 a, b, c;
};

template <HbForm F, int MU, int NU, bool LOWER>
__device__ __forceinline__ Staple load_staple(const double2 *U, const HbGeom &G, const int *L, int V, int par,
                                              const int (&c)[4], int odd, int i, int ip)
{
    constexpr bool FULL = F != kHbTwoRow;
    const double2 *own = U + hb_half<F>(V, par);
    const double2 *oth = U + hb_half<F>(V, 1 - par);
    const double2 *ownn = own + (size_t)NU * 9 * V, *othn = oth + (size_t)NU * 9 * V, *othm = oth + (size_t)MU * 9 * V;
    Staple S;
    if constexpr (!LOWER) {
        S.a = hb_load<FULL>(othn, V, hb_element<F>(ip, MU == 0 ? 1 - odd : odd));
        S.b = hb_load<FULL>(othm, V, hb_element<F>(hb_hop<NU, +1>(G, L, c, odd, i), NU == 0 ? 1 - odd : odd));
        S.c = hb_load<FULL>(ownn, V, hb_element<F>(i, odd));
    } else {
        const int im = hb_hop<NU, -1>(G, L, c, odd, i);
        // s + mu: x is odd there where it is not at s (mu = x), else as at s
        int cp[4] = {c[0], c[1], c[2], c[3]};
        int oddp = odd;
        if constexpr (MU == 0) {
            cp[0] = !odd ? c[0] : (c[0] + 1 == G.half ? 0 : c[0] + 1);
            oddp = 1 - odd;
        } else {
            cp[MU] = (c[MU] + 1 == L[MU]) ? 0 : c[MU] + 1;
        }
        const int em = hb_element<F>(im, NU == 0 ? 1 - odd : odd);
        S.a = hb_load<FULL>(ownn, V, hb_element<F>(hb_hop<NU, -1>(G, L, cp, oddp, ip), NU == 0 ? 1 - oddp : oddp));
        S.b = hb_load<FULL>(othm, V, em);
        S.c = hb_load<FULL>(othn, V, em);
    }
    return S;
}

// Adds a staple to the sum A: U_MU(s) A is the sum of the six plaquettes
// through the link.
template <bool FULL, bool LOWER>
__device__ __forceinline__ void add_staple(M3 &A, Staple &S)
{
    if constexpr (!FULL) {
        m3_row2(S.a);
        m3_row2(S.b);
        m3_row2(S.c);
    }
    if constexpr (!LOWER)
        A = m3_add(A, m3_mul_dag(m3_mul_dag(S.a, S.b), S.c));
    else
        A = m3_add(A, m3_mul(m3_mul(m3_dag(S.a), m3_dag(S.b)), S.c));
    m3_fence(A);
}

// One Cabibbo-Marinari update of u against staple sum A: for each subgroup
// (p, q), the part of the 2x2 block of u A proportional to SU(2) is
// nk V (V in SU(2)); u <- r u with r = X V^dag, X drawn with density
// exp((2 beta / 3) nk x0) (mode 0, heatbath), or r = V^dag V^dag (mode 1,
// overrelaxation, which keeps Re Tr(u A)). Then Gram-Schmidt.
__device__ void cm_update(M3 &u, const M3 &A, double beta, int mode, int site, int mu, long long n, uint32_t k0,
                          uint32_t k1)
{
    const int sub[3][2] = {{0, 1}, {0, 2}, {1, 2}};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int p = sub[k][0], q = sub[k][1];
        const M3 W = m3_mul(u, A);
        const double2 al = cscale(cadd(W.e[p * 3 + p], cconj(W.e[q * 3 + q])), 0.5);
        const double2 be = cscale(csub(W.e[p * 3 + q], cconj(W.e[q * 3 + p])), 0.5);
        const double det = al.x * al.x + al.y * al.y + be.x * be.x + be.y * be.y;
        if (!(det > 1e-300)) continue;
        const double nk = sqrt(det);
        const double2 v00 = make_double2(al.x / nk, al.y / nk), v01 = make_double2(be.x / nk, be.y / nk);
        // V^dag
        const double2 d00 = cconj(v00), d01 = make_double2(-v01.x, -v01.y), d10 = cconj(v01), d11 = v00;
        double2 r00, r01, r10, r11;
        if (mode == 0) {
            double x[4];
            if (!kp_draw(2.0 * beta / 3.0 * nk, site, mu, k, n, k0, k1, x)) continue;
            const double2 x00 = make_double2(x[0], x[3]), x01 = make_double2(x[2], x[1]);
            const double2 x10 = make_double2(-x[2], x[1]), x11 = make_double2(x[0], -x[3]);
            r00 = cadd(cmul(x00, d00), cmul(x01, d10));
            r01 = cadd(cmul(x00, d01), cmul(x01, d11));
            r10 = cadd(cmul(x10, d00), cmul(x11, d10));
            r11 = cadd(cmul(x10, d01), cmul(x11, d11));
        } else {
            r00 = cadd(cmul(d00, d00), cmul(d01, d10));
            r01 = cadd(cmul(d00, d01), cmul(d01, d11));
            r10 = cadd(cmul(d10, d00), cmul(d11, d10));
            r11 = cadd(cmul(d10, d01), cmul(d11, d11));
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double2 up = u.e[p * 3 + j], uq = u.e[q * 3 + j];
            u.e[p * 3 + j] = cadd(cmul(r00, up), cmul(r01, uq));
            u.e[q * 3 + j] = cadd(cmul(r10, up), cmul(r11, uq));
        }
    }
    m3_reunit(u);
}

// Updates every U_MU(s) with x + y + z + t = par (mod 2); these links are
// independent (their staples hold only other directions and other-parity
// sites). Work-items take these sites in slabs of zc xy-planes (hb_slab):
// within a slab in lexicographic order, then the next slab. MODE 0: heatbath,
// 1: overrelaxation.
//
// What bounds it: memory. A class reads every link of the other three
// directions and half of U_MU, in two-row form 384 B per lattice site at
// least, and writes 48; at 32^4 it reads 610 (L2 serves the second use of a
// link to the sites in flight only) and takes 107 us, with 2900 VALU
// instructions per wave (40 us of issue) beside it. In lexicographic order
// all through it read 660 to 730 and took 114 to 118 us (hb_slab). The steps
// to that form: reading the caller's array (three rows, the other parity's
// elements between this one's in every cache line) 432 us; the parity-split
// copy with the loads of all six staples issued first (spilled) 200; one
// staple at a time (m3_fence) 124 (three waves per SIMD); the next staple's
// loads in flight 117 (two waves per SIMD); blocks not renumbered by XCD 132.
template <HbForm F, int MODE, int MU>
__global__ __launch_bounds__(kSiteBlock, 2) void k_heatbath(const Cfg *__restrict__ cfgs, int par, double beta,
                                                         uint32_t k0, uint32_t k1, long long n, int zc)
{
    constexpr bool FULL = F != kHbTwoRow;
    const Cfg &C = cfgs[0];
    const int V = C.V;
    const int w = xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (w >= V / 2) return;
    const int L[4] = {C.dims[0], C.dims[1], C.dims[2], C.dims[3]};
    const HbGeom G = {L[0] / 2, C.V2 / 2, C.V3 / 2};
    int c[4];
    const int p = w / G.V2h, q = w - p * G.V2h;  // xy-plane of a parity, site in it
    c[1] = q / G.half;
    c[0] = q - c[1] * G.half;
    const int slab = p / (zc * L[3]), z0 = slab * zc, zn = min(zc, L[2] - z0), pz = p - z0 * L[3];
    c[3] = pz / zn;
    c[2] = z0 + pz - c[3] * zn;
    const int row = c[1] + L[1] * (c[2] + L[2] * c[3]), i = c[0] + G.half * row;
    const int odd = (c[1] + c[2] + c[3] + par) & 1;
    const int s = 2 * c[0] + odd + L[0] * row;
    double2 *U = F == kHbCaller ? C.U : hb_links(C);
    const int ip = hb_hop<MU, +1>(G, L, c, odd, i);
    M3 A = m3_zero();
    constexpr int N0 = MU == 0 ? 1 : 0, N1 = MU <= 1 ? 2 : 1, N2 = MU <= 2 ? 3 : 2;
#define GF_LOAD(NU_, LO_) load_staple<F, MU, NU_, LO_>(U, G, L, V, par, c, odd, i, ip)
    if constexpr (FULL) {
        Staple S = GF_LOAD(N0, false);
        add_staple<FULL, false>(A, S);
        S = GF_LOAD(N0, true);
        add_staple<FULL, true>(A, S);
        S = GF_LOAD(N1, false);
        add_staple<FULL, false>(A, S);
        S = GF_LOAD(N1, true);
        add_staple<FULL, true>(A, S);
        S = GF_LOAD(N2, false);
        add_staple<FULL, false>(A, S);
        S = GF_LOAD(N2, true);
        add_staple<FULL, true>(A, S);
    } else {  // each staple's links loaded while the one before is formed
        Staple S0 = GF_LOAD(N0, false);
        Staple S1 = GF_LOAD(N0, true);
        add_staple<FULL, false>(A, S0);
        S0 = GF_LOAD(N1, false);
        add_staple<FULL, true>(A, S1);
        S1 = GF_LOAD(N1, true);
        add_staple<FULL, false>(A, S0);
        S0 = GF_LOAD(N2, false);
        add_staple<FULL, true>(A, S1);
        S1 = GF_LOAD(N2, true);
        add_staple<FULL, false>(A, S0);
        add_staple<FULL, true>(A, S1);
    }
#undef GF_LOAD
    double2 *Um = U + (size_t)MU * 9 * V + hb_half<F>(V, par);
    const int e = hb_element<F>(i, odd);
    M3 u = hb_load<FULL>(Um, V, e);
    if constexpr (!FULL) m3_row2(u);
    cm_update(u, A, beta, MODE, s, MU, n, k0, k1);
    if constexpr (FULL)
        m3_store(Um, V, e, u);
    else
        m3_store12(Um, V, e, u);
}

// Index in the generator's copy of the caller's site s.
__device__ __forceinline__ int hb_index(const Cfg &C, int s)
{
    int c[4];
    site_coords(C.dims, s, c);
    const int par = (c[0] + c[1] + c[2] + c[3]) & 1;
    return (par ? C.V / 2 : 0) + (s - c[0]) / 2 + c[0] / 2;
}

// Caller's links -> the generator's copy.
__global__ __launch_bounds__(kSiteBlock) void k_hb_pack(const Cfg *__restrict__ cfgs)
{
    const Cfg &C = cfgs[0];
    const int V = C.V;
    const int s = blockIdx.x * kSiteBlock + threadIdx.x;
    if (s >= V) return;
    const int i = hb_index(C, s);
    double2 *__restrict__ dst = hb_links(C);
    const double2 *__restrict__ src = C.U;
#pragma unroll
    for (int k = 0; k < 36; ++k) dst[(size_t)k * V + i] = ld_stream(src + (size_t)k * V + s);
}

// The generator's copy -> the caller's links, third rows rebuilt (what the
// projection of the last sweep gave).
__global__ __launch_bounds__(kSiteBlock) void k_hb_unpack(const Cfg *__restrict__ cfgs)
{
    const Cfg &C = cfgs[0];
    const int V = C.V;
    const int s = blockIdx.x * kSiteBlock + threadIdx.x;
    if (s >= V) return;
    const int i = hb_index(C, s);
    const double2 *__restrict__ src = hb_links(C);
    double2 *__restrict__ dst = C.U;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) m3_store(dst + (size_t)mu * 9 * V, V, s, m3_load12(src + (size_t)mu * 9 * V, V, i));
}

// acc + Re Tr U_mu(x) U_nu(x+mu) U_mu^dag(x+nu) U_nu^dag(x): the scalar
// product of two products of two links, a row at a time.
__device__ __forceinline__ double plaq_pair(const M3 &um, const M3 &un, const M3 &un_mu, const M3 &um_nu, double acc)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double2 a = cmul(um.e[i * 3], un_mu.e[j]), b = cmul(un.e[i * 3], um_nu.e[j]);
            a = cfma(um.e[i * 3 + 1], un_mu.e[3 + j], a);
            b = cfma(un.e[i * 3 + 1], um_nu.e[3 + j], b);
            a = cfma(um.e[i * 3 + 2], un_mu.e[6 + j], a);
            b = cfma(un.e[i * 3 + 2], um_nu.e[6 + j], b);
            acc = fma(a.x, b.x, acc);
            acc = fma(a.y, b.y, acc);
        }
    return acc;
}

// Per-block compensated sums of the six plaquettes Re Tr U_P of each site,
// into partials[2 b], partials[2 b + 1]. A block takes kSiteBlock consecutive
// sites of the (x, y, z) volume (nb3 such sets) through tch t-slices. The
// (i, t) plaquettes are completed one slice late, with the next slice's own
// links, so that every block reads a slice's links in the same slice of its
// walk as the blocks of its neighbours.
//
// What bounds it: memory. It cannot read less than the 576 B per site of the
// links; at 32^4 it reads 1140 (the z neighbours of a slice, more than L2
// holds apart) in 183 us, 6.5 TB/s. Before: two whole matrices loaded per
// plaquette of every site and three products each, 440 us; own links once and
// two products, one site per work-item without the walk, 251 us (1690 B per
// site); the walk with the next slice's links kept for its own plaquettes 245
// us (its neighbours read them a slice later, from memory).
__global__ __launch_bounds__(kSiteBlock, 2) void k_plaquette(const Cfg *__restrict__ cfgs, int nb3, int tch)
{
    __shared__ dd red[2 * (kSiteBlock / 64)];
    const Cfg &C = cfgs[0];
    const int V = C.V;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int tc = blk / nb3;
    const int s3 = (blk - tc * nb3) * kSiteBlock + threadIdx.x;
    dd sum = {0.0, 0.0}, zero = {0.0, 0.0};
    if (s3 < C.V3) {
        const int Lx = C.dims[0], Ly = C.dims[1], Lz = C.dims[2], Lt = C.dims[3];
        const int r = s3 / Lx, x = s3 - r * Lx, z = r / Ly, y = r - z * Ly;
        int f[3];  // forward neighbours in x, y, z
        f[0] = (x + 1 == Lx) ? s3 - (Lx - 1) : s3 + 1;
        f[1] = (y + 1 == Ly) ? s3 - (Ly - 1) * Lx : s3 + Lx;
        f[2] = (z + 1 == Lz) ? s3 - (Lz - 1) * C.V2 : s3 + C.V2;
        const double2 *U = C.U;
        const double2 *Ut = U + (size_t)27 * V;
        const int t0 = tc * tch;
        M3 m[3];  // U_t^dag(x, t) U_i(x, t) U_t(x + i, t) of the slice before
        for (int t = t0; t <= t0 + tch; ++t) {
            const int ts = C.V3 * (t == Lt ? 0 : t);
            double acc = 0.0;
            M3 u[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                u[i] = hb_load<true>(U + (size_t)i * 9 * V, V, s3 + ts);
                if (t > t0)  // the (i, t) plaquettes of the slice before
#pragma unroll
                    for (int k = 0; k < 9; ++k) {
                        acc = fma(m[i].e[k].x, u[i].e[k].x, acc);
                        acc = fma(m[i].e[k].y, u[i].e[k].y, acc);
                    }
            }
            if (t < t0 + tch) {
                asm volatile("" : "+v"(acc)::"memory");
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = i + 1; j < 3; ++j) {
                        acc = plaq_pair(u[i], u[j], hb_load<true>(U + (size_t)j * 9 * V, V, f[i] + ts),
                                        hb_load<true>(U + (size_t)i * 9 * V, V, f[j] + ts), acc);
                        asm volatile("" : "+v"(acc)::"memory");  // the next pair's loads after this one's products
                    }
                const M3 ut = hb_load<true>(Ut, V, s3 + ts);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    m[i] = m3_dag_mul(ut, m3_mul(u[i], hb_load<true>(Ut, V, f[i] + ts)));
                    m3_fence(m[i]);
                }
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

__global__ __launch_bounds__(256) void k_sum_plaquette(const Cfg *__restrict__ cfgs, int nblk, double *__restrict__ out)
{
    __shared__ dd red[2 * (256 / 64)];
    const Cfg &C = cfgs[0];
    dd f = {0.0, 0.0}, z = {0.0, 0.0};
    for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
        const double *p = C.partials + (size_t)i * 2;
        f = dd_add(f, dd{p[0], p[1]});
    }
    block_sum2(f, z, red);
    if (threadIdx.x == 0) *out = (f.hi + f.lo) / (18.0 * (double)C.V);
}

// z-planes of k_heatbath's slabs. An XCD has some 16384 sites of a class in
// flight; numbered a t-slice after the other, where a t-slice holds that many
// none of them finds a link that another loads as its t-neighbour. Numbered
// slab by slab, t ahead of the slab, they are a tile of several z and several
// t, best as long in z as in t (16384 sites of a parity / sites of an
// xy-plane planes, its root), but not under six planes: the t beside the tile
// are the ones loaded just before. A heatbath and four overrelaxation sweeps,
// us, without slabs and in slabs of 3, 4, 6, 8, 16: 24^4 1937, 1838, 1834,
// 1816, 1834, 1881; 32^4 5886, 5694, 5549, 5536, 5583, 5822; 36 x 18 x 24 x
// 54 4679, 4522, 4440, 4454, 4469, 4525; 48^4 33967, 28592, 28603, 27403,
// 28231, 29607; 64^3 x 16 27266, 23499, 23200, 23204, 22865, 26442; 16^2 x
// 64^2 5704, 5789, 6322, 5713, 5474, 5456 (this one's planes are of 128
// sites: 11). A lattice whose sites are in flight at once needs no slabs:
// 16^3 x 32 728 without, 749 in slabs of 4.
int hb_slab(const int *dims)
{
    const int V2h = dims[0] / 2 * dims[1];
    if ((long long)V2h * dims[2] * dims[3] <= 8 * 16384) return dims[2];
    const double nz = fmax(6.0, sqrt(16384.0 / V2h));
    const int k = (int)(dims[2] / nz + 0.5);
    return k <= 1 ? dims[2] : (dims[2] + k - 1) / k;
}

// One sweep, in place in the caller's array (form kHbCaller) or in the copy.
hipError_t heatbath_sweep(const Launch &L, const int *dims, int mode, HbForm form, double beta, uint64_t seed, long long n)
{
    const int V = dims[0] * dims[1] * dims[2] * dims[3], zc = hb_slab(dims);
    // single waves as work-groups where work-groups of four would not give
    // each CU one
    const int nt = V / 2 >= 256 * kSiteBlock ? kSiteBlock : 64;
    const dim3 grid((V / 2 + nt - 1) / nt), blk(nt);
    const uint32_t k0 = (uint32_t)(seed & 0xffffffffull), k1 = (uint32_t)(seed >> 32);
#define GF_HB(F_, MODE_, MU_)                                                                                    \
    for (int par = 0; par < 2; ++par)                                                                               \
        hipLaunchKernelGGL((k_heatbath<F_, MODE_, MU_>), grid, blk, 0, L.stream, L.cfgs, par, beta, k0, k1, n, zc);
#define GF_HB4(F_, MODE_) GF_HB(F_, MODE_, 0) GF_HB(F_, MODE_, 1) GF_HB(F_, MODE_, 2) GF_HB(F_, MODE_, 3)
    if (form == kHbCaller) {
        GF_HB4(kHbCaller, 0)
    } else if (form == kHbFull) {
        GF_HB4(kHbFull, 0)
    } else if (mode == 0) {
        GF_HB4(kHbTwoRow, 0)
    } else {
        GF_HB4(kHbTwoRow, 1)
    }
#undef GF_HB4
#undef GF_HB
    return hipGetLastError();
}

// A call of one heatbath sweep works in place up to this many sites: the two
// launches of the copy cost more than the sweep gains (us of such a call, in
// place and with the copy: 4^4 148 and 162, 8^4 152 and 175, 12^4 162 and 182,
// 16^4 215 and 219; 16^3 x 32 356 and 299, 24^4 944 and 745).
constexpr int kHbInPlace = 65536;

}  // namespace

hipError_t launch_heatbath(const Launch &L, const int *dims, int nblk, double beta, int n_sweeps, int n_or, uint64_t seed,
                           long long sweep0)
{
    if (n_sweeps <= 0) return hipSuccess;
    const int V = dims[0] * dims[1] * dims[2] * dims[3];
    if (n_sweeps == 1 && n_or == 0 && V <= kHbInPlace) return heatbath_sweep(L, dims, 0, kHbCaller, beta, seed, sweep0);
    hipLaunchKernelGGL(k_hb_pack, dim3(nblk), dim3(kSiteBlock), 0, L.stream, L.cfgs);
    hipError_t e = hipGetLastError();
    for (int i = 0; i < n_sweeps && e == hipSuccess; ++i) {
        e = heatbath_sweep(L, dims, 0, i == 0 ? kHbFull : kHbTwoRow, beta, seed, sweep0 + i);
        for (int r = 0; r < n_or && e == hipSuccess; ++r) e = heatbath_sweep(L, dims, 1, kHbTwoRow, beta, seed, 0);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_hb_unpack, dim3(nblk), dim3(kSiteBlock), 0, L.stream, L.cfgs);
    return hipGetLastError();
}

hipError_t launch_plaquette(const Launch &L, const MarchPlan &m, double *out)
{
    const int nblk = m.nb3 * (m.Lt / m.tch);
    hipLaunchKernelGGL(k_plaquette, dim3(nblk), dim3(kSiteBlock), 0, L.stream, L.cfgs, m.nb3, m.tch);
    hipLaunchKernelGGL(k_sum_plaquette, dim3(1), dim3(256), 0, L.stream, L.cfgs, nblk, out);
    return hipGetLastError();
}

}  // namespace gfk
