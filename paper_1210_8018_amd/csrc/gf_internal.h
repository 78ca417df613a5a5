// Internal structures shared by the kernels (gf_kernels.hip) and the host
// runtime (gf_runtime.hip). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gfk {

// Device pointers of the configuration table carry the global address space
// in the device code of the kernel sources (those that include gf_device.h),
// so that accesses through them are global (not flat) memory instructions:
// flat accesses also count as LDS operations, and every wait for LDS would
// then wait for them as well. The layout is the same (64-bit pointers).
#if defined(__HIP_DEVICE_COMPILE__) && defined(GF_KERNEL_SOURCE)
#define GF_GLOBAL __attribute__((address_space(1)))
#else
#define GF_GLOBAL
#endif

constexpr int kMaxCfg = 64;        // configurations per batch context
constexpr int kHist = 256;         // device ring of (F, theta) per configuration
constexpr int kSiteBlock = 256;    // work-items per site-parallel block
constexpr int kFftThreads = 256;   // work-items per transform tile
constexpr int kMaxStages = 8;      // radix stages per axis
constexpr int kFields = 4;         // packed transform fields per site
constexpr int kTileElems2D = 4096; // largest LDS tile (elements) of the 2D passes


enum : int { kRunning = 0, kConverged = 1, kMaxIter = 2, kNonFinite = 3 };

// Transform lines held in registers (k_fft_line, k_fft_xy_reg,
// k_fft_xy_inv_reg): lengths 16 and 24 over two lanes of a wave, 32, 48 and
// 64 over four; each length is its own kernel instance, marked by a bit.
__host__ __device__ constexpr bool line_len_ok(int L) { return L == 16 || L == 24 || L == 32 || L == 48 || L == 64; }
__host__ __device__ constexpr int line_lanes(int L) { return L >= 32 ? 4 : 2; }
__host__ __device__ constexpr int line_len_bit(int L) { return L == 16 ? 0 : L == 24 ? 1 : L == 32 ? 2 : L == 48 ? 3 : 4; }
// planes per tile of the register (x, y) passes: a tile stays within 4096
// elements (the LDS-staged inverse pass serves the same tiles)
__host__ __device__ constexpr int xy_reg_planes_for(int L) { return L == 16 ? 8 : L == 24 ? 4 : L == 32 ? 2 : 1; }
// (z, t) plane shapes of the register (z, t) passes, one instance each:
// 32 x 32 (k_fft_zt_reg), 16 x 16, 24 x 24, 16 x 32, 48 x 48
// (k_fft_zt_lines); -1 none
__host__ __device__ constexpr int zt_shape_bit(int Lz, int Lt)
{
    return (Lz == 16 && Lt == 16)   ? 0
           : (Lz == 24 && Lt == 24) ? 1
           : (Lz == 32 && Lt == 32) ? 2
           : (Lz == 16 && Lt == 32) ? 3
           : (Lz == 48 && Lt == 48) ? 4
                                    : -1;
}

// Lines of gf_fft_any.hip: lengths up to 64, each a group of any_g1 points
// and (where that is not the whole line) one of L / any_g1 points, run in the
// registers of a work-item. The groups are consecutive stages of the radix
// sequence 3, ..., 8, ..., 4 or 2 (FP64: also 4 4, 3 2 3 2 and 3 2 8, whose
// groups need fewer registers).
__host__ __device__ constexpr bool any_len_ok(int L)
{
    return L == 2 || L == 3 || L == 4 || L == 6 || L == 8 || L == 9 || L == 12 || L == 16 || L == 18 || L == 24 ||
           L == 27 || L == 32 || L == 36 || L == 48 || L == 54 || L == 64;
}
__host__ __device__ constexpr int any_g1(int L, bool f64)
{
    return f64 && L == 16                                  ? 4
           : f64 && (L == 36 || L == 48)                   ? 6
           : (L <= 12 || L == 16)                          ? L
           : (L == 18 || L == 24 || L == 27 || L == 48)    ? 3
           : (L == 32 || L == 64)                          ? 8
                                                           : 9;
}
// lines per work-group of the 1D passes: 256 where a work-item takes a whole
// line, else as many as keep 4 FP64 tiles of the longest lines in LDS
__host__ __device__ constexpr int any_line_width(int L, bool f64) { return any_g1(L, f64) == L ? 256 : 32; }

// Transform schedules: which passes make up the 4D transform, scaling and
// inverse (the scaling is always fused into the pass that completes the
// forward transform).
enum : int {
    kSchedAuto = 0,
    kSched1D = 1,    // x, y, z, t+scale, z, y, x (1D passes) + gauge
    kSchedXY1D = 2,  // xy, z, t+scale, z, xy^-1+gauge
    kSchedXYZT = 3,  // xy, zt+scale, xy^-1+gauge
    kSchedCount = 4
};

// Device control block of one configuration. Written only by device code
// (the arming and reduction kernels), read back by the host per chunk.
struct Ctrl {
    double eps;          // stop once theta <= eps
    double F, theta;     // latest measurement
    long long iter;      // updates since init
    long long max_iter;  // absolute cap on iter
    int done;            // kRunning / kConverged / kMaxIter / kNonFinite
    int cur;             // current two-row link buffer, U12[cur]
    int ru_now;          // the coming iteration also projects the new links
    int in_caller;       // the current links are the caller's array U (full 3x3), not U12[cur]
    int pad2;
    double hist[kHist][2];  // (F, theta) after update k at slot k % kHist
};

// One axis of a 1D transform pass: tiles of P pencils of length L, elements
// of a pencil spaced S apart in memory.
struct FftAxis {
    int L, S, P;
    int ntile;        // tiles per field
    int inner_chunks; // S / P for axes > 0
    int nstage;
    int radix[kMaxStages];
};

struct Cfg {
    int dims[4];
    int V;
    int V2;               // Lx * Ly
    int V3;               // Lx * Ly * Lz
    int nblk_site;        // site blocks of kSiteBlock
    int nb3;              // blocks over the (x, y, z) volume
    int tile[3];          // (x, y, z) extent of one block's sites; tile[0] = 0: kSiteBlock consecutive sites
    int ntile[3];         // tiles along x, y, z (tile mode)
    int nch;              // walks along t: block tc of a site set takes slices [tc Lt / nch, (tc + 1) Lt / nch)
    int nblk_march;       // nb3 * nch: blocks of the marching kernels
    GF_GLOBAL double2 *U;        // links [4][3][3][V] (the caller's array)
    GF_GLOBAL double2 *U12[2];   // two-row links [4][2][3][V], two buffers (workspace)
    GF_GLOBAL float2 *U12f[2];   // the same two link buffers in single-precision storage (link_prec 1)
    GF_GLOBAL float2 *g12f;      // two-row g in single-precision storage
    GF_GLOBAL void *fields;      // Delta of the last measurement or update, packed fields [4][V], double2 or float2
    GF_GLOBAL void *work;        // its transform [4][V], between the passes (may be fields2)
    GF_GLOBAL void *fields2;     // the filtered fields Delta~ [4][V] read by the fused pass
    GF_GLOBAL double2 *g;        // gauge field [3][3][V]
    GF_GLOBAL double *partials;  // [nblk_march or nblk_site][4]: (F hi, F lo, theta hi, theta lo)
    GF_GLOBAL Ctrl *ctrl;
    GF_GLOBAL const double *sin2;  // 4 sin^2(pi n / L_mu), axis mu at sin2 + sin2_off[mu]
    int sin2_off[4];
    GF_GLOBAL const void *tw;    // twiddles exp(-2 pi i e / L_mu), axis mu at tw + tw_off[mu]
    int tw_off[4];
    double kfac;          // (alpha / 2) * p2max / V
    GF_GLOBAL void *kmom;        // K(p) per momentum site [V], double (FP64 transform) or float (FP32)
    int reunit_every;
    FftAxis ax[4];
    int xyQ, nxy;         // xy pass: Q consecutive xy-planes per tile, nxy tiles per field
    int ztP, nzt;         // zt pass: P consecutive xy-sites per tile, nzt tiles per field
    int xyPad;            // LDS elements added to every x-row of an xy tile (bank spreading)
    int ztPad;            // LDS elements added to every t-plane of a zt tile
    int zt_reg;           // the scaled (z, t) pass runs in registers: k_fft_zt_reg (32 x 32), k_fft_zt_lines (the others)
    int xy_reg;           // the iteration's (x, y) passes run in k_fft_xy_reg / k_fft_xy_inv_reg (Lx = Ly = 16 to 64)
    int xy_any, zt_any;   // the 2D passes run in k_fft_xy_any / k_fft_zt_any where not in the above
    int lany[2];          // the 1D z / t passes run in k_fft_line_any
    int line[2];          // the 1D z (line[0]) / t (line[1]) passes run in k_fft_line (that extent 16 to 64)
};

// Block-to-configuration maps for every launch shape of a batch: entry e
// covers configuration idx[e], blocks [off[e], off[e + 1]).
struct Batch {
    int n;
    int idx[kMaxCfg];
    int off_site[kMaxCfg + 1];
    int off_march[kMaxCfg + 1];
    int off_fft[4][kMaxCfg + 1];
    int off_xy[kMaxCfg + 1];
    int off_zt[kMaxCfg + 1];
    int off_lany[2][kMaxCfg + 1];  // k_fft_line_any work-groups per field of the z and t passes
    int off_line[2][kMaxCfg + 1];  // k_fft_line units (64 / line_lanes xy-sites x 4 lines) of the z and t passes
};

struct Launch {
    const Cfg *cfgs;      // device array
    const Batch *batch;   // device struct
    int total_site_blocks;
    int total_march_blocks;
    int march_pair;       // the fused pass takes two site sets per block (512 work-items): 0 never,
                          // 1 always, 2 with single-precision link storage only
    int total_fft_tiles[4];
    int total_xy_tiles;
    int total_zt_tiles;
    int xy_cap, zt_cap;            // 2D tile capacity variant (1024, 2048 or 4096 elements)
    int xy_th, zt_th;              // work-group size of the 2D passes (capacity / elements per work-item)
    int xy_fpb, zt_fpb;            // fields per work-group of the 2D passes (the next one prefetched)
    int xy_p2, zt_p2;              // some configuration has power-of-two extents in that pass
    int xy_gen, zt_gen;            // some configuration has not
    int ax_p2[4], ax_gen[4];       // same for the 1D passes of each axis
    int xy_tw2, xy_tw_total;       // LDS twiddle layout of the xy pass: y table offset, entries
    int zt_tw2, zt_tw_total;       // same for the zt pass
    int zt_reg_any;                // scaled zt pass: some configuration in k_fft_zt_reg / k_fft_zt_lines
    int xy_any, zt_any;            // some configuration has k_fft_xy_any / k_fft_zt_any passes
    int zt64;                      // one configuration, whose 1D z and t passes of an update run as k_fft_zt64
    int xy_any_it, zt_any_it;      // ... in the iteration (not in the register passes there)
    int xy_any_elems, zt_any_elems;  // LDS elements of their tiles and twiddles
    int total_lany[2], lany_elems[2];  // work-groups per field and LDS elements of k_fft_line_any
    int zt_reg_groups;             // work-groups per tile of k_fft_zt_reg (1, 2 or 4: fields split among them)
    int zt_reg_p;                  // xy-sites per tile of k_fft_zt_reg / k_fft_zt_lines (2, 4 or 8)
    int zt_m;                      // (z, t) plane shapes of the register passes present (bits zt_shape_bit)
    int xy_reg_any;                // iteration's xy passes: some configuration in the register ones
    int xy_reg_groups;             // work-groups per tile of the register xy passes
    int xy_m;                      // their plane sizes present (bits line_len_bit)
    int total_line[2];             // k_fft_line units of the z and t passes (0: no configuration has them)
    int line_m[2];                 // line lengths among them (bits line_len_bit)
    int max_lds_elems;    // 1D passes: largest P * L
    int fp32;             // transform precision
    int fused;            // iterations use the fused update + divergence kernel
    int link_f32;         // links and g held in single-precision two-row storage (this phase)
    int ncfg;
    hipStream_t stream;
};

hipError_t launch_arm(const Launch &L, int ncfg, double eps, long long add_iters, int reset_iter);
// the same for configuration k alone
hipError_t launch_arm_one(const Launch &L, int k, double eps, long long add_iters, int reset_iter);
hipError_t launch_delta(const Launch &L, int respect_done, double2 *full_delta);
hipError_t launch_reduce(const Launch &L, int ncfg, int count_iter, int respect_done);
hipError_t launch_fft_axis(const Launch &L, int axis, int sign, int mode, void *fields_override,
                           int nfields, int respect_done);
// fold_reduce: the pass also does the final reduction of the previous update
// (in place of launch_reduce after it).
hipError_t launch_fft_xy(const Launch &L, int sign, void *fields_override, int nfields, int respect_done,
                         int fold_reduce = 0);
hipError_t launch_fft_xy_inv_gauge(const Launch &L, int respect_done, double2 *g_override);
hipError_t launch_fft_zt(const Launch &L, int mode, int sign, void *fields_override, int nfields, int respect_done);
hipError_t launch_fft_zt_scale(const Launch &L, int respect_done);
hipError_t set_lds_limits();
// gf_fft_any.hip. take_reg: also configurations whose
// iteration runs this pass in k_fft_xy_reg / k_fft_xy_inv_reg
hipError_t launch_fft_xy_any(const Launch &L, int sign, void *fields_override, int nfields, int respect_done, int take_reg,
                             int fold);
hipError_t launch_fft_zt_any(const Launch &L, int mode, int sign, void *fields_override, int nfields, int respect_done);
hipError_t launch_fft_line_any(const Launch &L, int axis, int mode, int sign, void *fields_override, int nfields,
                               int respect_done);
hipError_t set_lds_limits_any();
hipError_t launch_fft_zt64(const Launch &L, int V2, int nf, int respect_done);
hipError_t set_lds_limits_zt64();
// any_only: for the configurations whose inverse (x, y) pass k_fft_xy_any took
hipError_t launch_gauge(const Launch &L, int respect_done, double2 *g_override, int any_only = 0);
hipError_t launch_update(const Launch &L, int respect_done, const double2 *g_override);
// Where the fused pass of an update takes the old links from and puts the
// new ones: the two-row buffers, or the caller's array
// for the first update of a call (old links) or the last of a gf_step call
// (new links).
enum : int { kLinksBuffers = 0, kLinksFromCaller = 1, kLinksToCaller = 2 };
// reunit: some listed configuration projects its links in this update (the
// instance for those runs too)
hipError_t launch_update_delta(const Launch &L, int link_io, int reunit);
// in_caller: the first update reads the caller's links; else they are copied
// to binary32 two-row buffer 0
hipError_t launch_begin_call(const Launch &L, int in_caller, double eps, long long add_iters);
hipError_t launch_momentum_table(const Launch &L);
// reads every configuration's two-row link buffers (cache eviction before a timed pass)
hipError_t launch_touch_links(const Launch &L);
// n_sweeps times a heatbath sweep (numbers from sweep0) and n_or
// overrelaxation sweeps of the caller's links
hipError_t launch_heatbath(const Launch &L, const int *dims, int nblk, double beta, int n_sweeps, int n_or, uint64_t seed,
                           long long sweep0);
// Walks of the plaquette and of the functional: nb3 sets of kSiteBlock
// consecutive sites of the (x, y, z) volume, tch t-slices (a divisor of Lt)
// per block.
struct MarchPlan {
    int nb3, tch, Lt;
};
hipError_t launch_plaquette(const Launch &L, const MarchPlan &m, double *out);
hipError_t launch_unpack_links(const Launch &L);
// gf_functional.hip (two doubles of partials per walk block)
hipError_t launch_functional_g(const Launch &L, int nblk_site, const MarchPlan &m, const double *omega, double scale,
                               double *out);
// d_omega or d_U may be null
hipError_t launch_functional_g_backward(const Launch &L, int nblk_site, const MarchPlan &m, const double *omega,
                                        double scale, double *d_omega, double2 *d_U);

}  // namespace gfk
