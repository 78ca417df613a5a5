// Transform passes for extents up to 64 (2^a 3^b) whose radix stages run in
// registers: a line of L = G1 G2 points takes one round of G1-point
// transforms and (L > 12, L != 16) one of G2-point transforms, each in the
// registers of a work-item, instead of one LDS round trip per radix 2, 3, 4
// or 8 stage as in the LDS-staged passes of gf_kernels.hip (which keep the
// extents above 64). The (x, y) pass, the (z, t) pass (plain, or forward, K(p),
// backward), and 1D z and t passes for (z, t) planes too large to hold more
// than an xy-site or two of. A work-group takes one tile of one field, so
// that small lattices still give every CU work.
//
// In FP32 the butterflies and twiddles are those of the Stockham radix
// sequence 3, ..., 8, ..., 4 or 2 of the LDS-staged passes (a group fuses
// consecutive stages), so that both give the same values bit for bit; FP64
// lines of 16, 36 and 48 points take other radices, which need fewer registers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "gf_device.h"
#include "gf_internal.h"
#include "gf_transform.h"

namespace gfk {

namespace {

constexpr int kAnyThreads = 256;

// Radices of a group of G points, in the order of the stages it fuses.
template <int G>
struct Radices {
    static constexpr int r1 = G == 6 ? 3 : G == 9 ? 3 : G == 12 ? 3 : G == 16 ? 8 : G;
    static constexpr int r2 = G / r1;
};

// Component-wise copy: whole-vector assignments keep an array of vectors out
// of registers.
template <typename T2>
__device__ __forceinline__ void put2(T2 &d, const T2 &v)
{
    d.x = v.x;
    d.y = v.y;
}

template <int R, typename T2>
__device__ __forceinline__ void dft_r(T2 (&a)[R], int sign)
{
    if constexpr (R == 2)
        dft2(a);
    else if constexpr (R == 3)
        dft3(a, sign);
    else if constexpr (R == 4)
        dft4(a, sign);
    else
        dft8(a, sign);
}

template <int SIGN, typename T2>
__device__ __forceinline__ T2 twiddled(T2 v, T2 w)
{
    if constexpr (SIGN > 0) w.y = -w.y;
    return t_mul(v, w);
}

// Two fused Stockham stages of radix R1 and R2 (1: none) on the G = R1 R2
// elements v[m] = x[j + m L/G] of a line of L = NS G REST points whose first
// NS points' worth of stages are done: kk = j mod NS. On return v[q] is
// output (j - kk) G + kk + q NS. tw[e] = exp(-2 pi i e / L).
template <int R1, int R2, int NS, int REST, int SIGN, typename T2>
__device__ __forceinline__ void group(T2 (&v)[R1 * R2], const T2 *tw, int kk)
{
#pragma unroll
    for (int m2 = 0; m2 < R2; ++m2) {
        T2 a[R1];
#pragma unroll
        for (int m1 = 0; m1 < R1; ++m1) {
            put2(a[m1], v[m2 + R2 * m1]);
            if (NS > 1 && m1 > 0) put2(a[m1], twiddled<SIGN>(a[m1], tw[m1 * kk * (R2 * REST)]));
        }
        dft_r<R1>(a, SIGN);
#pragma unroll
        for (int q1 = 0; q1 < R1; ++q1) put2(v[m2 + R2 * q1], a[q1]);
    }
    if constexpr (R2 > 1) {
        T2 o[R1 * R2];
#pragma unroll
        for (int q1 = 0; q1 < R1; ++q1) {
            T2 b[R2];
#pragma unroll
            for (int m2 = 0; m2 < R2; ++m2) {
                put2(b[m2], v[m2 + R2 * q1]);
                if (m2 > 0 && (NS > 1 || q1 > 0)) put2(b[m2], twiddled<SIGN>(b[m2], tw[m2 * (kk + q1 * NS) * REST]));
            }
            dft_r<R2>(b, SIGN);
#pragma unroll
            for (int q2 = 0; q2 < R2; ++q2) put2(o[q1 + R1 * q2], b[q2]);
            }
#pragma unroll
        for (int q = 0; q < R1 * R2; ++q) put2(v[q], o[q]);
    }
}

// The same group with its radices (and so the fused stages) in the opposite
// order.
template <int G, int NS, int REST, int SIGN, typename T2>
__device__ __forceinline__ void group_reversed(T2 (&v)[G], const T2 *tw, int kk)
{
    if constexpr (Radices<G>::r2 == 1)
        group<G, 1, NS, REST, SIGN>(v, tw, kk);
    else
        group<Radices<G>::r2, Radices<G>::r1, NS, REST, SIGN>(v, tw, kk);
}

template <int L, typename T2>
__host__ __device__ constexpr int g1_of() { return any_g1(L, std::is_same<T2, double2>::value); }
// slot of a line in which a forward transform leaves frequency f
template <int L, typename T2>
__device__ __forceinline__ int slot_of(int f)
{
    constexpr int G1 = g1_of<L, T2>(), G2 = L / G1;
    return (f % G1) * G2 + f / G1;
}

// Items of a phase: `npen` lines times the groups of a line.
struct Item {
    int pen, j;
};
__device__ __forceinline__ Item item_of(int b, FastDiv fpen, int npen)
{
    const int j = fdiv(b, fpen);
    return {b - j * npen, j};
}

// Element i of an array whose byte offsets fit 32 bits (a field: 16 V < 2^32
// for every V the library takes): base in scalar registers, one offset
// register per access.
template <typename T>
__device__ __forceinline__ T &at32(T *base, unsigned i)
{
    return *(T *)((char *)base + i * (unsigned)sizeof(T));
}

// Where the lines of a phase are. In LDS, slot l of line `pen` is at
// line(pen)[l ls]; in memory element i is at src / dst [off(pen) + i gs]
// (stored only where ok(pen)).
template <typename T2, typename Line, typename Off, typename Ok>
struct Lines {
    const T2 *src;
    T2 *dst;
    int ls;
    unsigned gs;
    Line line;
    Off off;
    Ok ok;
};
template <typename T2, typename Line, typename Off, typename Ok>
__device__ __forceinline__ Lines<T2, Line, Off, Ok> lines_of(const T2 *src, T2 *dst, int ls, unsigned gs, Line line,
                                                             Off off, Ok ok)
{
    return {src, dst, ls, gs, line, off, ok};
}

// N elements i0, i0 + di, ... of a line from or to memory; slots from or to LDS.
template <int N, typename T2, typename IO>
__device__ __forceinline__ void mem_get(T2 (&v)[N], const IO &io, int pen, int i0, int di)
{
    const unsigned o = io.off(pen) + (unsigned)i0 * io.gs, d = (unsigned)di * io.gs;
#pragma unroll
    for (int m = 0; m < N; ++m) put2(v[m], at32(io.src, o + m * d));
}
template <int N, typename T2, typename IO>
__device__ __forceinline__ void mem_put(const T2 (&v)[N], const IO &io, int pen, int i0, int di)
{
    if (!io.ok(pen)) return;
    const unsigned o = io.off(pen) + (unsigned)i0 * io.gs, d = (unsigned)di * io.gs;
#pragma unroll
    for (int m = 0; m < N; ++m) put2(at32(io.dst, o + m * d), v[m]);
}
template <int N, typename T2, typename IO, typename SlotOf>
__device__ __forceinline__ void lds_get(T2 (&v)[N], const IO &io, int pen, SlotOf slot)
{
    const T2 *p = io.line(pen);
#pragma unroll
    for (int m = 0; m < N; ++m) put2(v[m], p[slot(m) * io.ls]);
}
template <int N, typename T2, typename IO, typename SlotOf>
__device__ __forceinline__ void lds_put(const T2 (&v)[N], const IO &io, int pen, SlotOf slot)
{
    T2 *p = io.line(pen);
#pragma unroll
    for (int m = 0; m < N; ++m) put2(p[slot(m) * io.ls], v[m]);
}

// One axis of `npen` lines of L points, SIGN -1 or +1, from memory (INM) or
// LDS to memory (OUTM) or LDS. A work-item reads and writes the same slots of
// a line, so the only barrier is the one between two groups; with two groups
// result f ends in slot slot_of(f). Elements read from LDS sit in their
// natural slots, or (PERM) where such a pass has left them: result t then
// ends in slot slot_of(slot_of(t)). ROWS: the lines are contiguous in memory;
// 16 lines times the groups of a line are consecutive items, so that a wave
// reads runs of 64 / 16 or more elements of each.
template <int L, int SIGN, bool INM, bool OUTM, bool PERM, bool ROWS = false, typename T2, typename IO>
__device__ __forceinline__ void axis_pass(const T2 *tw, int npen, const IO &io)
{
    constexpr int G1 = g1_of<L, T2>(), G2 = L / G1;
    const FastDiv fpen = fast_div(npen), f16 = fast_div(G2);
    const auto place = [](int l) __attribute__((always_inline)) { return PERM ? slot_of<L, T2>(l) : l; };
    const int items = ROWS ? ((npen + 15) & ~15) * G2 : npen * G2;
    for (int b = threadIdx.x; b < items; b += kAnyThreads) {
        Item it;
        if constexpr (ROWS) {
            const int g = fdiv(b >> 4, f16);
            it.j = (b >> 4) - g * G2;
            it.pen = 16 * g + (b & 15);
            if (it.pen >= npen) continue;
        } else {
            it = item_of(b, fpen, npen);
        }
        const auto own = [&](int m) __attribute__((always_inline)) { return place(it.j + m * G2); };
        T2 v[G1];
        if constexpr (INM)
            mem_get(v, io, it.pen, it.j, G2);
        else
            lds_get(v, io, it.pen, own);
        group<Radices<G1>::r1, Radices<G1>::r2, 1, G2, SIGN>(v, tw, 0);
        if constexpr (G2 == 1 && OUTM)
            mem_put(v, io, it.pen, 0, 1);
        else
            lds_put(v, io, it.pen, own);
    }
    if constexpr (G2 > 1) {
        __syncthreads();
        for (int b = threadIdx.x; b < npen * G1; b += kAnyThreads) {
            const Item it = item_of(b, fpen, npen);
            const auto own = [&](int m) __attribute__((always_inline)) { return place(it.j * G2 + m); };
            T2 v[G2];
            lds_get(v, io, it.pen, own);
            group<Radices<G2>::r1, Radices<G2>::r2, G1, 1, SIGN>(v, tw, it.j);
            if constexpr (OUTM)
                mem_put(v, io, it.pen, it.j, G1);
            else
                lds_put(v, io, it.pen, own);
        }
    }
}

// Forward transform, multiplication by K, backward transform of `npen` lines.
// K of frequency f of a line at km[koff(pen) + f ks]. The backward transform
// takes the radix sequence forwards, or (CENTRE) backwards: its first group
// is then the forward transform's last, on the same elements, and the scaling
// sits between the two in registers. In LDS, result t ends in slot t if
// CENTRE or one group, else in slot_of(slot_of(t)).
template <int L, bool CENTRE, bool INM, bool OUTM, typename T2, typename T, typename KOff, typename IO>
__device__ __forceinline__ void axis_scaled(const T2 *tw, int npen, const T *km, KOff koff, unsigned ks, const IO &io)
{
    constexpr int G1 = g1_of<L, T2>(), G2 = L / G1;
    const FastDiv fpen = fast_div(npen);
    const auto scale = [&](auto &v, int pen, int f0, int df) __attribute__((always_inline)) {
        const unsigned o = koff(pen) + (unsigned)f0 * ks, d = (unsigned)df * ks;
#pragma unroll
        for (int q = 0; q < (int)(sizeof(v) / sizeof(T2)); ++q) {
            const T k = at32(km, o + q * d);
            v[q].x *= k;
            v[q].y *= k;
        }
    };
    const auto natural = [](int m) __attribute__((always_inline)) { return m; };
    if constexpr (G2 == 1) {
        for (int b = threadIdx.x; b < npen; b += kAnyThreads) {
            T2 v[L];
            if constexpr (INM)
                mem_get(v, io, b, 0, 1);
            else
                lds_get(v, io, b, natural);
            group<Radices<L>::r1, Radices<L>::r2, 1, 1, -1>(v, tw, 0);
            scale(v, b, 0, 1);
            if constexpr (CENTRE)
                group_reversed<L, 1, 1, +1>(v, tw, 0);
            else
                group<Radices<L>::r1, Radices<L>::r2, 1, 1, +1>(v, tw, 0);
            if constexpr (OUTM)
                mem_put(v, io, b, 0, 1);
            else
                lds_put(v, io, b, natural);
        }
    } else {
        for (int b = threadIdx.x; b < npen * G2; b += kAnyThreads) {
            const Item it = item_of(b, fpen, npen);
            const auto own = [&](int m) __attribute__((always_inline)) { return it.j + m * G2; };
            T2 v[G1];
            if constexpr (INM)
                mem_get(v, io, it.pen, it.j, G2);
            else
                lds_get(v, io, it.pen, own);
            group<Radices<G1>::r1, Radices<G1>::r2, 1, G2, -1>(v, tw, 0);
            lds_put(v, io, it.pen, own);
        }
        __syncthreads();
        for (int b = threadIdx.x; b < npen * G1; b += kAnyThreads) {
            const Item it = item_of(b, fpen, npen);
            const auto own = [&](int m) __attribute__((always_inline)) { return it.j * G2 + m; };
            T2 v[G2];
            lds_get(v, io, it.pen, own);
            group<Radices<G2>::r1, Radices<G2>::r2, G1, 1, -1>(v, tw, it.j);
            scale(v, it.pen, it.j, G1);
            // backwards: stages G2 then G1, the first on elements j + q G1
            if constexpr (CENTRE) group_reversed<G2, 1, G1, +1>(v, tw, 0);
            lds_put(v, io, it.pen, own);
        }
        __syncthreads();
        if constexpr (CENTRE) {
            // output (j, q) of the first backward group is element j G2 + q of
            // the intermediate line, in that slot: the second takes j + m G2
            for (int b = threadIdx.x; b < npen * G2; b += kAnyThreads) {
                const Item it = item_of(b, fpen, npen);
                const auto own = [&](int m) __attribute__((always_inline)) { return it.j + m * G2; };
                T2 v[G1];
                lds_get(v, io, it.pen, own);
                group_reversed<G1, G2, 1, +1>(v, tw, it.j);
                if constexpr (OUTM)
                    mem_put(v, io, it.pen, it.j, G2);
                else
                    lds_put(v, io, it.pen, own);
            }
        } else {
            axis_pass<L, +1, false, OUTM, true>(tw, npen, io);
        }
    }
}

// Calls f with the length as a compile-time constant (uniform over the block).
template <typename F>
__device__ __forceinline__ void with_length(int L, F f)
{
    switch (L) {
#define GF_CASE(L_) \
    case L_: f(std::integral_constant<int, L_>{}); break;
        GF_CASE(2) GF_CASE(3) GF_CASE(4) GF_CASE(6) GF_CASE(8) GF_CASE(9) GF_CASE(12) GF_CASE(16)
        GF_CASE(18) GF_CASE(24) GF_CASE(27) GF_CASE(32) GF_CASE(36) GF_CASE(48) GF_CASE(54) GF_CASE(64)
#undef GF_CASE
    default: break;
    }
}

template <typename T2>
__device__ __forceinline__ void fill_twiddles(T2 *dst, const Cfg &C, int axis)
{
    const T2 *__restrict__ src = (const T2 *)C.tw + C.tw_off[axis];
    for (int e = threadIdx.x; e < C.dims[axis]; e += kAnyThreads) dst[e] = src[e];
}

// Index whose element sits in slot l after `passes` two-group passes.
__device__ __forceinline__ int slot_index(int L, int g1, int l, int passes)
{
    const int g2 = L / g1;
    if (g2 == 1) return l;
    for (int k = 0; k < passes; ++k) l = (l % g2) * g1 + l / g2;
    return l;
}

// (x, y) transform of the planes of a tile of one field (the caller's in place;
// the iteration's: x_pass_in, x_pass_out).
// Tile: xyQ consecutive xy-planes (fewer in a configuration's last tile),
// element (x, y, q) at x + Xp (y + Ly q), Xp = Lx or Lx + 1, odd: the lanes of
// an x-line access (consecutive rows) fall on distinct LDS banks.
// take_reg: also the configurations whose iteration runs this pass in
// registers throughout (k_fft_xy_reg). fold: as in k_fft_xy.
//
// What bounds it: latency of memory with five waves per SIMD (its waves wait
// for it 70 % of their lives; no LDS bank conflicts). 36^4 FP64 56 us forward
// and 43 back (3.8 and 5.0 TB/s; LDS-staged 92 and 105), 12^4 10 and 8 us
// (19 and 21: 21 work-groups of four fields each). At four waves per SIMD 36^4
// took 54 and 48 us; with the x-lines staged through LDS 71 and 55.
template <typename T2, int SIGN>
__global__ __launch_bounds__(kAnyThreads, 5) void k_fft_xy_any(const Cfg *__restrict__ cfgs, const Batch *__restrict__ B,
                                                            void *fields_override, int respect_done, int nf,
                                                            int take_reg, int fold)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int ntiles = B->off_xy[B->n] * nf;
    if ((int)blockIdx.x >= ntiles) {
        const Cfg &R = cfgs[B->idx[blockIdx.x - ntiles]];
        if (R.ctrl->done) return;
        finalize_config(R, R.nblk_march, 1, fold == 2, (dd *)smem);
        return;
    }
    const int rb = xcd_remap(blockIdx.x, ntiles);
    const int tile = rb / nf, f = rb - tile * nf;
    const int c = find_cfg(B->off_xy, B->n, tile);
    const Cfg &C = cfgs[B->idx[c]];
    if (respect_done && C.ctrl->done) return;
    if (!C.xy_any || (C.xy_reg && !take_reg)) return;  // another pass takes it
    const int Lx = C.dims[0], Ly = C.dims[1], V2 = C.V2;
    const int q0 = (tile - B->off_xy[c]) * C.xyQ;
    const int nq = min(C.xyQ, C.dims[2] * C.dims[3] - q0);
    const int Xp = Lx | 1, rows = Ly * nq;
    T2 *buf = (T2 *)smem;
    T2 *twx = buf + Xp * Ly * C.xyQ, *twy = twx + Lx;
    const size_t o = (size_t)f * C.V + (size_t)q0 * V2;
    const T2 *src = x_pass_in<T2>(C, fields_override, SIGN) + o;
    T2 *dst = x_pass_out<T2>(C, fields_override, SIGN) + o;
    // x-lines of two groups come from memory into registers; whole ones
    // through LDS, where each work-item takes a line
    const int g1x = any_g1(Lx, std::is_same<T2, double2>::value);
    if (g1x == Lx) {
        const FastDiv fl = fast_div(Lx);
        for (int i = threadIdx.x; i < rows * Lx; i += kAnyThreads) {
            const int r = fdiv(i, fl);
            put2(buf[i + r * (Xp - Lx)], src[i]);
        }
    }
    fill_twiddles(twx, C, 0);
    fill_twiddles(twy, C, 1);
    __syncthreads();
    const auto all = [](int) __attribute__((always_inline)) { return true; };
    const auto xio = lines_of<T2>(
        src, dst, 1, 1u, [&](int r) __attribute__((always_inline)) { return buf + r * Xp; },
        [&](int r) __attribute__((always_inline)) { return (unsigned)(r * Lx); }, all);
    with_length(Lx, [&](auto l) __attribute__((always_inline)) {
        constexpr int L = decltype(l)::value;
        constexpr bool two = g1_of<L, T2>() != L;
        axis_pass<L, SIGN, two, false, false, two>(twx, rows, xio);
    });
    __syncthreads();
    // y-lines: line (slot of x, plane q), x fastest
    const FastDiv fx = fast_div(Lx);
    const auto yio = lines_of<T2>(
        src, dst, Xp, (unsigned)Lx,
        [&](int pen) __attribute__((always_inline)) {
            const int q = fdiv(pen, fx);
            return buf + (pen - q * Lx) + Xp * Ly * q;
        },
        [&](int pen) __attribute__((always_inline)) {
            const int q = fdiv(pen, fx);
            return (unsigned)(slot_index(Lx, g1x, pen - q * Lx, 1) + V2 * q);
        },
        all);
    with_length(Ly, [&](auto l) __attribute__((always_inline)) {
        axis_pass<decltype(l)::value, SIGN, false, true, false>(twy, Lx * nq, yio);
    });
}

// (z, t) pass of a tile of one field: ztP (a power of two) consecutive
// xy-sites (fewer valid ones in a ragged last tile) times the (z, t) plane,
// element (p, z, t) at p + P z + Tp t. MODE -1 / +1: plain transform; 0:
// forward, K(p), backward. The elements come from memory into the registers
// of the z-lines' first group and leave from those of the last group.
//
// What bounds it: memory and L2 for rows of P elements (64 to 128 bytes), and
// on small lattices the chain of its few phases. Scaled, FP64: 36^4 84 us (2.7
// TB/s; LDS-staged 214), 36 x 18 x 24 x 54 47 (133, rows of one element), 12^4
// 8.6 (46: nine tiles, four fields each one after the other, 13 round trips
// through LDS instead of 3), 8^4 7.5 (30).
template <typename T2, int MODE>
__global__ __launch_bounds__(kAnyThreads, 4) void k_fft_zt_any(const Cfg *__restrict__ cfgs, const Batch *__restrict__ B,
                                                            void *fields_override, int respect_done, int nf)
{
    using T = typename Cx<T2>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    const int rb = xcd_remap(blockIdx.x, gridDim.x);
    const int tile = rb / nf, f = rb - tile * nf;
    const int c = find_cfg(B->off_zt, B->n, tile);
    const Cfg &C = cfgs[B->idx[c]];
    if (respect_done && C.ctrl->done) return;
    if (!C.zt_any || (MODE == 0 && C.zt_reg)) return;  // another pass takes it
    const int P = C.ztP, lp = ilog2(P), Lz = C.dims[2], Lt = C.dims[3], V2 = C.V2;
    const int Tp = P * Lz + C.ztPad;
    const int i0 = (tile - B->off_zt[c]) * P, np = min(P, V2 - i0);
    T2 *buf = (T2 *)smem;
    T2 *twz = buf + Tp * Lt, *twt = twz + Lz;
    fill_twiddles(twz, C, 2);
    fill_twiddles(twt, C, 3);
    T2 *__restrict__ g = zt_pass<T2>(C, fields_override) + (size_t)f * C.V + i0;
    __syncthreads();
    // z-lines: line (p, t); t-lines: line (p, slot of z). Lanes past a ragged
    // tile's last site read it again and store nothing.
    constexpr bool f64 = std::is_same<T2, double2>::value;
    const int g1z = any_g1(Lz, f64), g1t = any_g1(Lt, f64);
    const unsigned vz = (unsigned)V2, vt = (unsigned)V2 * (unsigned)Lz;
    const auto ok = [&](int pen) __attribute__((always_inline)) { return (pen & (P - 1)) < np; };
    const auto site = [&](int pen) __attribute__((always_inline)) { return (unsigned)min(pen & (P - 1), np - 1); };
    const auto zline = [&](int pen) __attribute__((always_inline)) { return buf + (pen & (P - 1)) + Tp * (pen >> lp); };
    const auto tline = [&](int pen) __attribute__((always_inline)) { return buf + pen; };
    const auto zin = lines_of<T2>(
        g, g, P, vz, zline, [&](int pen) __attribute__((always_inline)) { return site(pen) + (unsigned)(pen >> lp) * vt; },
        ok);
    with_length(Lz, [&](auto l) __attribute__((always_inline)) {
        axis_pass<decltype(l)::value, (MODE > 0 ? 1 : -1), true, false, false>(twz, P * Lt, zin);
    });
    __syncthreads();
    // memory offset of a t-line: its z, or kz, from its slot
    const auto toff = [&](int pen) __attribute__((always_inline)) {
        return site(pen) + (unsigned)slot_index(Lz, g1z, pen >> lp, 1) * vz;
    };
    const auto tio = lines_of<T2>(g, g, Tp, vt, tline, toff, ok);
    if constexpr (MODE != 0) {
        with_length(Lt, [&](auto l) __attribute__((always_inline)) {
            axis_pass<decltype(l)::value, MODE, false, true, false>(twt, P * Lz, tio);
        });
        return;
    }
    const T *__restrict__ Km = (const T *)C.kmom + i0;
    // the backward t transform takes its stages backwards in FP64, and in FP32
    // where the LDS-staged pass for powers of two did (Lt = 2, 4, 16, 32), so
    // that an FP32 transform keeps its rounding
    const bool centre = f64 || (is_p2(Lz) && is_p2(Lt) && Lt != 8 && Lt != 64);
    if (centre) {
        with_length(Lt, [&](auto l) __attribute__((always_inline)) {
            constexpr int L = decltype(l)::value;
            if constexpr (std::is_same<T2, double2>::value || L == 2 || L == 4 || L == 16 || L == 32)
                axis_scaled<L, true, false, false>(twt, P * Lz, Km, toff, vt, tio);
        });
    } else {
        if constexpr (!std::is_same<T2, double2>::value)
            with_length(Lt, [&](auto l) __attribute__((always_inline)) {
                axis_scaled<decltype(l)::value, false, false, false>(twt, P * Lz, Km, toff, vt, tio);
            });
    }
    __syncthreads();
    const auto zout = lines_of<T2>(
        g, g, P, vz, zline,
        [&](int pen) __attribute__((always_inline)) {
            return site(pen) + (unsigned)(centre ? pen >> lp : slot_index(Lt, g1t, pen >> lp, 2)) * vt;
        },
        ok);
    with_length(Lz, [&](auto l) __attribute__((always_inline)) {
        axis_pass<decltype(l)::value, +1, false, true, true>(twz, P * Lt, zout);
    });
}

// One 1D pass along z (axis 2) or t (axis 3): any_line_width(L) lines of one
// field per work-group, consecutive in memory apart from the axis (a ragged
// last group clamped), their elements from memory into the first group's
// registers and back from the last's. MODE -1 / +1: plain; 0 (t): forward,
// K(p), backward. Bound by memory: 36^4 FP64 37, 50 and 37 us (z, t scaled,
// z; 5.8, 4.6, 5.8 TB/s; staged in LDS 70, 115 and 68).
template <typename T2, int MODE>
__global__ __launch_bounds__(kAnyThreads, 4) void k_fft_line_any(const Cfg *__restrict__ cfgs,
                                                              const Batch *__restrict__ B, int axis,
                                                              void *fields_override, int respect_done, int nf)
{
    using T = typename Cx<T2>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    const int rb = xcd_remap(blockIdx.x, gridDim.x);
    const int *off = B->off_lany[axis - 2];
    const int tile = rb / nf, f = rb - tile * nf;
    const int c = find_cfg(off, B->n, tile);
    const Cfg &C = cfgs[B->idx[c]];
    if (respect_done && C.ctrl->done) return;
    const int Ll = C.dims[axis], NL = any_line_width(Ll, std::is_same<T2, double2>::value);
    const int nlines = C.V / Ll;
    const int l0 = (tile - off[c]) * NL, nl = min(NL, nlines - l0);
    const unsigned S = axis == 2 ? (unsigned)C.V2 : (unsigned)C.V3;
    // line l of the axis starts at l (t-lines), or at (l mod V2) + V3 (l / V2)
    const FastDiv fv2 = fast_div(C.V2);
    T2 *buf = (T2 *)smem;
    T2 *tw = buf + (any_g1(Ll, std::is_same<T2, double2>::value) == Ll ? 0 : NL * Ll);
    fill_twiddles(tw, C, axis);
    T2 *__restrict__ g = zt_pass<T2>(C, fields_override) + (size_t)f * C.V;
    const T *__restrict__ Km = (const T *)C.kmom;
    __syncthreads();
    const auto start = [&](int pen) __attribute__((always_inline)) {
        const int l = l0 + min(pen, nl - 1);
        if (axis == 3) return (unsigned)l;
        const int t = fdiv(l, fv2);
        return (unsigned)(l - t * C.V2) + (unsigned)t * (unsigned)C.V3;
    };
    const auto io = lines_of<T2>(
        g, g, NL, S, [&](int pen) __attribute__((always_inline)) { return buf + pen; }, start,
        [&](int pen) __attribute__((always_inline)) { return pen < nl; });
    with_length(Ll, [&](auto l) __attribute__((always_inline)) {
        constexpr int L = decltype(l)::value;
        if constexpr (MODE != 0)
            axis_pass<L, MODE, true, true, false>(tw, NL, io);
        else
            axis_scaled<L, std::is_same<T2, double2>::value, true, true>(tw, NL, Km, start, S, io);
    });
}

template <typename T2>
hipError_t run_xy_any(const Launch &L, int sign, void *fo, int nf, int rd, int take_reg, int fold)
{
    const dim3 grid(L.total_xy_tiles * nf + (fold ? L.ncfg : 0));
    const size_t sh = std::max((size_t)L.xy_any_elems * sizeof(T2), (size_t)(2 * (kAnyThreads / 64) * sizeof(dd)));
    if (sign < 0)
        hipLaunchKernelGGL((k_fft_xy_any<T2, -1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, fo, rd, nf,
                           take_reg, fold);
    else
        hipLaunchKernelGGL((k_fft_xy_any<T2, +1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, fo, rd, nf,
                           take_reg, fold);
    return hipGetLastError();
}

template <typename T2>
hipError_t run_zt_any(const Launch &L, int mode, int sign, void *fo, int nf, int rd)
{
    const dim3 grid(L.total_zt_tiles * nf);
    const size_t sh = (size_t)L.zt_any_elems * sizeof(T2);
    if (mode == 1)
        hipLaunchKernelGGL((k_fft_zt_any<T2, 0>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, fo, rd, nf);
    else if (sign < 0)
        hipLaunchKernelGGL((k_fft_zt_any<T2, -1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, fo, rd, nf);
    else
        hipLaunchKernelGGL((k_fft_zt_any<T2, +1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, fo, rd, nf);
    return hipGetLastError();
}

template <typename T2>
hipError_t run_line_any(const Launch &L, int axis, int mode, int sign, void *fo, int nf, int rd)
{
    const dim3 grid(L.total_lany[axis - 2] * nf);
    const size_t sh = (size_t)L.lany_elems[axis - 2] * sizeof(T2);
    if (mode == 1)
        hipLaunchKernelGGL((k_fft_line_any<T2, 0>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, axis, fo,
                           rd, nf);
    else if (sign < 0)
        hipLaunchKernelGGL((k_fft_line_any<T2, -1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, axis, fo,
                           rd, nf);
    else
        hipLaunchKernelGGL((k_fft_line_any<T2, +1>), grid, dim3(kAnyThreads), sh, L.stream, L.cfgs, L.batch, axis, fo,
                           rd, nf);
    return hipGetLastError();
}

template <typename T2>
hipError_t set_lds_any()
{
    const int bytes = 144 * 1024;  // the largest tile: 8 xy-sites x 32 x 32 of a register (z, t) pass, FP64
    const void *k[] = {(const void *)k_fft_xy_any<T2, -1>,   (const void *)k_fft_xy_any<T2, +1>,
                       (const void *)k_fft_zt_any<T2, 0>,    (const void *)k_fft_zt_any<T2, -1>,
                       (const void *)k_fft_zt_any<T2, +1>,   (const void *)k_fft_line_any<T2, 0>,
                       (const void *)k_fft_line_any<T2, -1>, (const void *)k_fft_line_any<T2, +1>};
    for (const void *f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_fft_xy_any(const Launch &L, int sign, void *fields_override, int nfields, int respect_done, int take_reg,
                             int fold)
{
    return L.fp32 ? run_xy_any<float2>(L, sign, fields_override, nfields, respect_done, take_reg, fold)
                  : run_xy_any<double2>(L, sign, fields_override, nfields, respect_done, take_reg, fold);
}

hipError_t launch_fft_zt_any(const Launch &L, int mode, int sign, void *fields_override, int nfields, int respect_done)
{
    return L.fp32 ? run_zt_any<float2>(L, mode, sign, fields_override, nfields, respect_done)
                  : run_zt_any<double2>(L, mode, sign, fields_override, nfields, respect_done);
}

hipError_t launch_fft_line_any(const Launch &L, int axis, int mode, int sign, void *fields_override, int nfields,
                               int respect_done)
{
    return L.fp32 ? run_line_any<float2>(L, axis, mode, sign, fields_override, nfields, respect_done)
                  : run_line_any<double2>(L, axis, mode, sign, fields_override, nfields, respect_done);
}

hipError_t set_lds_limits_any()
{
    const hipError_t e = set_lds_any<double2>();
    return e != hipSuccess ? e : set_lds_any<float2>();
}

}  // namespace gfk
