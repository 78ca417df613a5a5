// The (z, t) part of an FP64 update on lattices with 64 slices along both:
// forward z and t transforms, K(p), backward t and z transforms in one pass.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gf_device.h"
#include "gf_internal.h"
#include "gf_transform.h"

namespace gfk {
namespace {

constexpr int kN = 64;  // points of a line
constexpr int kP = 4;   // xy-sites of a tile

__device__ __forceinline__ double2 conj_if(double2 w, int sign) { return sign < 0 ? w : make_double2(w.x, -w.y); }

// exp(sign 2 pi i m / 16) of the 4 * 4 split, m = n0 k0.
__device__ __forceinline__ double2 w16(int m, int sign)
{
    const double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, r2 = 0.70710678118654752440;
    const double2 w = m == 1 ? make_double2(c1, s1)
                    : m == 2 ? make_double2(r2, r2)
                    : m == 3 ? make_double2(s1, c1)
                    : m == 4 ? make_double2(0.0, 1.0)
                    : m == 6 ? make_double2(-r2, r2)
                             : make_double2(-c1, -s1);
    return make_double2(w.x, sign < 0 ? -w.y : w.y);
}

// Forward 16-point DFT in place, 16 = 4 * 4; output k0 + 4 k1 is left at
// 4 k0 + k1, where the backward one takes it from.
__device__ __forceinline__ void dft16_fwd(double2 (&v)[16])
{
#pragma unroll
    for (int n0 = 0; n0 < 4; ++n0) {
        dft4r(v[n0], v[n0 + 4], v[n0 + 8], v[n0 + 12], -1);
#pragma unroll
        for (int k0 = 1; k0 < 4; ++k0)
            if (n0 > 0) v[n0 + 4 * k0] = t_mul(v[n0 + 4 * k0], w16(n0 * k0, -1));
    }
#pragma unroll
    for (int k0 = 0; k0 < 4; ++k0) dft4r(v[4 * k0], v[4 * k0 + 1], v[4 * k0 + 2], v[4 * k0 + 3], -1);
}

__device__ __forceinline__ void dft16_bwd(double2 (&v)[16])
{
#pragma unroll
    for (int k0 = 0; k0 < 4; ++k0) dft4r(v[4 * k0], v[4 * k0 + 1], v[4 * k0 + 2], v[4 * k0 + 3], +1);
#pragma unroll
    for (int n0 = 0; n0 < 4; ++n0) {
#pragma unroll
        for (int k0 = 1; k0 < 4; ++k0)
            if (n0 > 0) v[n0 + 4 * k0] = t_mul(v[n0 + 4 * k0], w16(n0 * k0, +1));
        dft4r(v[n0], v[n0 + 4], v[n0 + 8], v[n0 + 12], +1);
    }
}

// Element at a 32-bit byte offset (16 V < 2^32 for every V the library takes).
__device__ __forceinline__ double2 &at(double2 *base, unsigned bytes) { return *(double2 *)((char *)base + bytes); }
__device__ __forceinline__ double at(const double *base, unsigned bytes)
{
    return *(const double *)((const char *)base + bytes);
}

// Order between a wave's own LDS accesses, which the hardware keeps.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A work-group takes kP = 4 xy-sites of one field (64-byte rows): 4 planes of
// 64 x 64, 256 KB, which stay in registers from the load to the store, 32
// elements per work-item. LDS (130 KB) only passes elements on: along z,
// 64 = 8 * 8, between the eight lanes of a wave that share a (site, t); along
// t, 64 = 4 * 16, the 4 in registers, through a half of the tile at a time to
// work-items that hold all 16, scale by K(p) and go back the same way.
//
// Against three 1D passes (z; t, K(p), t; z) it reads and writes the fields
// once instead of three times. What bounds it: one such work-group fills a
// CU, so that its loads and stores (475 us of the fields' 2.1 GB at 64^4) and
// its arithmetic and LDS traffic (140 and 100 us) share the time but for what
// other CUs hide. Measured, FP64, us: 64^4 660 (1D passes 1318), 48 x 32 x
// 64^2 267 (378), 16^2 x 64^2 38 (80), 8^2 x 64^2 31 (46). Tiles of two
// sites, two work-groups per CU: 1182 at 64^4 (32-byte rows); barriers that
// leave loads in flight 745 against 705; K(p) loaded when it is needed 742
// against 705. Consecutive work-groups are the fields of a tile (they share
// K(p)), or the tiles of a field where a plane is a multiple of 64 KB, as the
// rows of a tile then fall on the same memory channels: 64^4 708 against 660,
// 48 x 32 x 64^2 267 against 282.
__global__ __launch_bounds__(128 * kP, 2) void k_fft_zt64(const Cfg *__restrict__ cfgs, int respect_done, int nf)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Cfg &C = cfgs[0];
    if (respect_done && C.ctrl->done) return;
    constexpr int P = kP, LP = 2;  // P = 2^LP
    const int rb = xcd_remap(blockIdx.x, gridDim.x);
    int f, tile;
    if (C.V2 % 4096 == 0) {
        const int nt = gridDim.x / nf;
        f = rb / nt, tile = rb - f * nt;
    } else {
        tile = rb / nf, f = rb - tile * nf;
    }
    const unsigned V2 = C.V2;
    const int i0 = tile * P, np = min(P, C.V2 - i0);
    double2 *buf = (double2 *)smem;           // [2][16][64][P]
    double2 *tw = buf + 2 * 16 * kN * P;      // exp(-2 pi i m / 64)
    const int p = threadIdx.x & (P - 1), a = (threadIdx.x >> LP) & 7, tt = threadIdx.x >> (LP + 3);
    const double2 *__restrict__ src = (const double2 *)C.tw + C.tw_off[2];
    if (threadIdx.x < kN) tw[threadIdx.x] = src[threadIdx.x];
    const int ps = min(p, np - 1);  // a ragged tile's lanes past its last site read it again and store nothing
    double2 *__restrict__ g = (double2 *)C.work + (size_t)f * C.V + i0;
    unsigned go = (V2 * (unsigned)(a + kN * tt) + ps) * 16u;
    double2 d[4][8];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int m = 0; m < 8; ++m) d[j][m] = at(g, go + V2 * (unsigned)(8 * m + kN * 16 * j) * 16u);
    __syncthreads();
    // exchange of a between the lanes of one (p, t): within a wave
    double2 *xw = buf + (threadIdx.x >> 6) * (64 / (8 * P)) * 8 * 9 * P + ((threadIdx.x & 63) >> (LP + 3)) * 8 * 9 * P + p;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        dft8(d[j], -1);
#pragma unroll
        for (int k = 0; k < 8; ++k) xw[k * 9 * P + a * P] = k ? t_mul(d[j][k], tw[a * k]) : d[j][k];
        wave_order();
#pragma unroll
        for (int m = 0; m < 8; ++m) d[j][m] = xw[a * 9 * P + m * P];
        wave_order();
        dft8(d[j], -1);  // kz = a + 8 q
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        dft4r(d[0][q], d[1][q], d[2][q], d[3][q], -1);
#pragma unroll
        for (int k = 1; k < 4; ++k) d[k][q] = t_mul(d[k][q], tw[tt * k]);
    }
    __syncthreads();
    const int kz = (threadIdx.x >> LP) & 63, b = threadIdx.x >> (LP + 6);
    double2 *col = buf + ((b * 16) * kN + kz) * P + p;
    double2 *row = buf + (tt * kN + a) * P + p;
    const double *__restrict__ K = (const double *)C.kmom + i0;
    const unsigned ko = (V2 * (unsigned)(kz + kN * b) + ps) * 8u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        double K16[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)  // kt = 2 h + b + 4 r
            K16[r] = at(K, ko + V2 * (unsigned)(kN * (2 * h + 4 * r)) * 8u);
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int q = 0; q < 8; ++q) row[(bb * 16 * kN + 8 * q) * P] = d[2 * h + bb][q];
        __syncthreads();
        double2 e[16];
#pragma unroll
        for (int n = 0; n < 16; ++n) e[n] = col[n * kN * P];
        dft16_fwd(e);
#pragma unroll
        for (int k0 = 0; k0 < 4; ++k0)
#pragma unroll
            for (int k1 = 0; k1 < 4; ++k1) {
                e[4 * k0 + k1].x *= K16[k0 + 4 * k1];
                e[4 * k0 + k1].y *= K16[k0 + 4 * k1];
            }
        dft16_bwd(e);
#pragma unroll
        for (int n = 0; n < 16; ++n) col[n * kN * P] = e[n];
        __syncthreads();
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int q = 0; q < 8; ++q) d[2 * h + bb][q] = row[(bb * 16 * kN + 8 * q) * P];
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
#pragma unroll
        for (int k = 1; k < 4; ++k) d[k][q] = t_mul(d[k][q], conj_if(tw[tt * k], +1));
        dft4r(d[0][q], d[1][q], d[2][q], d[3][q], +1);
        if (q & 1) wave_order();
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        asm volatile("" : "+v"(go));  // offsets formed again, not kept from the loads
        dft8(d[j], +1);
#pragma unroll
        for (int n = 0; n < 8; ++n) xw[n * 9 * P + a * P] = n ? t_mul(d[j][n], conj_if(tw[a * n], +1)) : d[j][n];
        wave_order();
#pragma unroll
        for (int m = 0; m < 8; ++m) d[j][m] = xw[a * 9 * P + m * P];
        wave_order();
        dft8(d[j], +1);  // z = a + 8 m
        if (p < np)
#pragma unroll
            for (int m = 0; m < 8; ++m) at(g, go + V2 * (unsigned)(8 * m + kN * 16 * j) * 16u) = d[j][m];
    }
}

constexpr size_t kLds = (2 * 16 * kN * kP + kN) * sizeof(double2);

}  // namespace

hipError_t launch_fft_zt64(const Launch &L, int V2, int nf, int respect_done)
{
    hipLaunchKernelGGL(k_fft_zt64, dim3((V2 + kP - 1) / kP * nf), dim3(128 * kP), kLds, L.stream, L.cfgs, respect_done, nf);
    return hipGetLastError();
}

hipError_t set_lds_limits_zt64()
{
    return hipFuncSetAttribute((const void *)k_fft_zt64, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
}

}  // namespace gfk
