// Shared by the transform kernels: small DFTs of either precision, and the
// final reduction of an update, which rides on a transform pass.
#pragma once

#include "gf_device.h"
#include "gf_internal.h"

namespace gfk {

// ============================================================ reductions + stopping rule
// Sum the block partials of one configuration in a fixed order (the whole
// block takes part), F = sum/(12 V) (Eq. 1), theta = sum/(3 V) (Eq. 4); with
// count_iter, count the update, record the history, flip the link buffer if
// asked and evaluate the stopping rule theta <= eps.
// The partial sums are taken kReduceLanes at a time in a fixed order, each 64
// of these lanes by one wave; a work-group of fewer waves takes them in turn,
// one of more leaves the others idle: every caller forms the same sums bit
// for bit.
constexpr int kReduceLanes = 256;

// Whether the iteration after update `it` also projects the links.
__device__ __forceinline__ int next_reunit(const Cfg &C, long long it)
{
    return C.reunit_every > 0 && (it + 1) % (long long)C.reunit_every == 0;
}

// red: 2 kReduceLanes / 64 entries
static __device__ __forceinline__ void finalize_config(const Cfg &C, int nparts, int count_iter, int flip, dd *red)
{
    Ctrl *ct = C.ctrl;
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    for (int w = threadIdx.x >> 6; w < kReduceLanes / 64; w += nw) {
        dd f = {0.0, 0.0}, t = {0.0, 0.0};
        for (int i = 64 * w + lane; i < nparts; i += kReduceLanes) {
            const double *p = C.partials + (size_t)i * 4;
            f = dd_add(f, dd{p[0], p[1]});
            t = dd_add(t, dd{p[2], p[3]});
        }
        f = wave_sum(f);
        t = wave_sum(t);
        if (lane == 0) {
            red[2 * w] = f;
            red[2 * w + 1] = t;
        }
    }
    __syncthreads();
    dd f = red[0], t = red[1];
    for (int k = 1; k < kReduceLanes / 64; ++k) {
        f = dd_add(f, red[2 * k]);
        t = dd_add(t, red[2 * k + 1]);
    }
    if (threadIdx.x == 0) {
        const double F = (f.hi + f.lo) / (12.0 * (double)C.V);
        const double th = (t.hi + t.lo) / (3.0 * (double)C.V);
        ct->F = F;
        ct->theta = th;
        long long it = ct->iter;
        if (count_iter) {
            it += 1;
            ct->iter = it;
            if (flip) ct->cur ^= 1;
            ct->ru_now = next_reunit(C, it);
        }
        ct->hist[it % kHist][0] = F;
        ct->hist[it % kHist][1] = th;
        if (count_iter) {
            int d = kRunning;
            if (!isfinite(F) || !isfinite(th))
                d = kNonFinite;
            else if (!(th > ct->eps))
                d = kConverged;
            else if (it >= ct->max_iter)
                d = kMaxIter;
            ct->done = d;
        }
    }
}

// ============================================================ the fields of a pass
// Fields the caller gave (gf_fft) are transformed in place. In an iteration
// the forward pass over x reads Delta from `fields` and writes to `work`, the
// passes along y, z and t work there in place, and the backward pass over x
// writes Delta~ to `fields2` (for large lattices the same buffer as `work`). So
// Delta stays in `fields` until the next update or measurement, and neither a
// pass launched ahead for a configuration that turns out to have stopped nor a
// stage call (gf_gauge) between two iterating calls spoils what the next update
// starts from. An iteration takes as long as with a transform in place in
// `fields` (32^4 FP64 254.8 us for 255.9, 36^4 496 for 502), or less where the
// buffer is a third one (16^3 x 32 52.8 for 54.9).
template <typename T2>
__device__ __forceinline__ T2 *zt_pass(const Cfg &C, void *fields_override)
{
    return (T2 *)(fields_override ? fields_override : (void *)C.work);
}
template <typename T2>
__device__ __forceinline__ const T2 *x_pass_in(const Cfg &C, void *fields_override, int sign)
{
    return (const T2 *)(fields_override ? fields_override : sign < 0 ? (void *)C.fields : (void *)C.work);
}
template <typename T2>
__device__ __forceinline__ T2 *x_pass_out(const Cfg &C, void *fields_override, int sign)
{
    return (T2 *)(fields_override ? fields_override : sign < 0 ? (void *)C.work : (void *)C.fields2);
}

// ============================================================ small DFTs
template <typename T2>
struct Cx;
template <>
struct Cx<double2> {
    using T = double;
    __device__ static double2 mk(double a, double b) { return make_double2(a, b); }
};
template <>
struct Cx<float2> {
    using T = float;
    __device__ static float2 mk(float a, float b) { return make_float2(a, b); }
};

template <typename T2>
__device__ __forceinline__ T2 t_add(T2 a, T2 b)
{
    T2 r;
    r.x = a.x + b.x;
    r.y = a.y + b.y;
    return r;
}
template <typename T2>
__device__ __forceinline__ T2 t_sub(T2 a, T2 b)
{
    T2 r;
    r.x = a.x - b.x;
    r.y = a.y - b.y;
    return r;
}
template <typename T2>
__device__ __forceinline__ T2 t_mul(T2 a, T2 b)
{
    T2 r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}
// multiply by sign * i
template <typename T2>
__device__ __forceinline__ T2 t_mul_si(T2 a, int sign)
{
    T2 r;
    if (sign < 0) {
        r.x = a.y;
        r.y = -a.x;
    } else {
        r.x = -a.y;
        r.y = a.x;
    }
    return r;
}

// r-point DFTs, b_q = sum_m a_m exp(sign 2 pi i m q / r), in place.
template <typename T2>
__device__ __forceinline__ void dft2(T2 *a)
{
    T2 t = a[0];
    a[0] = t_add(t, a[1]);
    a[1] = t_sub(t, a[1]);
}

template <typename T2>
__device__ __forceinline__ void dft3(T2 *a, int sign)
{
    using T = typename Cx<T2>::T;
    const T h = (T)0.86602540378443864676;  // sqrt(3)/2
    T2 s = t_add(a[1], a[2]);
    T2 d = t_sub(a[1], a[2]);
    T2 b0 = t_add(a[0], s);
    T2 m;
    m.x = a[0].x - (T)0.5 * s.x;
    m.y = a[0].y - (T)0.5 * s.y;
    // exp(sign 2 pi i/3) = -1/2 + sign i h: b1 = m + sign i h d, b2 = m - sign i h d
    T2 r = t_mul_si(d, sign);
    r.x *= h;
    r.y *= h;
    a[0] = b0;
    a[1] = t_add(m, r);
    a[2] = t_sub(m, r);
}

template <typename T2>
__device__ __forceinline__ void dft4r(T2 &a0, T2 &a1, T2 &a2, T2 &a3, int sign)
{
    const T2 s02 = t_add(a0, a2), d02 = t_sub(a0, a2);
    const T2 s13 = t_add(a1, a3), d13 = t_mul_si(t_sub(a1, a3), sign);
    a0 = t_add(s02, s13);
    a2 = t_sub(s02, s13);
    a1 = t_add(d02, d13);
    a3 = t_sub(d02, d13);
}

template <typename T2>
__device__ __forceinline__ void dft4(T2 *a, int sign)
{
    dft4r(a[0], a[1], a[2], a[3], sign);
}

template <typename T2>
__device__ __forceinline__ void dft8(T2 *a, int sign)
{
    using T = typename Cx<T2>::T;
    const T r2 = (T)0.70710678118654752440;
    T2 e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
    T2 o0 = a[1], o1 = a[3], o2 = a[5], o3 = a[7];
    dft4r(e0, e1, e2, e3, sign);
    dft4r(o0, o1, o2, o3, sign);
    // w^q, w = exp(sign 2 pi i / 8): w^1 = (1 + sign i) r2, w^2 = sign i, w^3 = (-1 + sign i) r2
    T2 t1, t3;
    {
        const T2 si = t_mul_si(o1, sign);
        t1.x = (o1.x + si.x) * r2;
        t1.y = (o1.y + si.y) * r2;
    }
    const T2 t2 = t_mul_si(o2, sign);
    {
        const T2 si = t_mul_si(o3, sign);
        t3.x = (si.x - o3.x) * r2;
        t3.y = (si.y - o3.y) * r2;
    }
    a[0] = t_add(e0, o0);
    a[4] = t_sub(e0, o0);
    a[1] = t_add(e1, t1);
    a[5] = t_sub(e1, t1);
    a[2] = t_add(e2, t2);
    a[6] = t_sub(e2, t2);
    a[3] = t_add(e3, t3);
    a[7] = t_sub(e3, t3);
}

}  // namespace gfk
