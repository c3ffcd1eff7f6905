// Launchers of the tendency-kernel configurations and the macro that
// builds a registry list.  Included by one translation unit per field type.
#pragma once

#include "kl_internal.hpp"
#include "stencil.hpp"
#include "stencil_zl.hpp"
#include "stencil_step.hpp"
#include "stencil_rf.hpp"
#include "stencil_les.hpp"
#include "stencil_les_zl.hpp"
#include "stencil_les_rf.hpp"

#include <algorithm>

namespace kl {

inline unsigned cdivu(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

template <typename T>
StencilArgs<T> device_args(const HostArgs &h)
{
    StencilArgs<T> a;
    a.itot = h.itot;
    a.jtot = h.jtot;
    a.ktot = h.ktot;
    a.kw0 = h.kw0;
    a.bc = h.bc;
    a.off = h.off;
    a.js = h.js;
    a.ks = h.ks;
    a.dxi = (T)h.dxi;
    a.dyi = (T)h.dyi;
    a.visc = (T)h.visc;
    a.dt = (T)h.dt;
    a.dzi = (const T *)h.dzi;
    a.dzhi = (const T *)h.dzhi;
    a.ut = (T *)h.ut;
    a.vt = (T *)h.vt;
    a.wt = (T *)h.wt;
    a.u = (const T *)h.u;
    a.v = (const T *)h.v;
    a.w = (const T *)h.w;
    a.nbx = a.nby = a.nbz = 1;
    a.evisc = (const T *)h.evisc;
    a.rf_cpr = a.rf_rows = a.rf_kb = 0;
    a.x_fill = 0;
    return a;
}

// 1-D grids only: total threads must fit the 32-bit grid size.
inline bool grid_fits(uint64_t blocks, uint64_t threads) { return blocks * threads < (1ull << 32); }

template <typename T, int KERNEL>
hipError_t launch_plain(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, 256);
    a.nby = h.jtot;
    a.nbz = h.ktot;
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 256)) return hipErrorInvalidConfiguration;
    if (KERNEL == KL_KERNEL_ADVEC_U)
        hipLaunchKernelGGL(advec_u_plain<T>, dim3((unsigned)nb), dim3(256), 0, s, a);
    else if (KERNEL == KL_KERNEL_DIFF_UVW)
        hipLaunchKernelGGL(diff_uvw_plain<T>, dim3((unsigned)nb), dim3(256), 0, s, a);
    else if (KERNEL == KL_KERNEL_ADVEC_U_2I5)
        hipLaunchKernelGGL(advec_u_2i5_plain<T>, dim3((unsigned)nb), dim3(256), 0, s, a);
    else if (KERNEL == KL_KERNEL_ADVEC_DIFF)
        hipLaunchKernelGGL(advec_diff_plain<T>, dim3((unsigned)nb), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(diff_smag_plain<T>, dim3((unsigned)nb), dim3(256), 0, s, a);
    return hipGetLastError();
}

// The default configuration of the fused pass onto tendencies that start at zero.
template <typename T>
hipError_t launch_plain_fresh(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, 256);
    a.nby = h.jtot;
    a.nbz = h.ktot;
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((advec_diff_plain<T, true>), dim3((unsigned)nb), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename T, int KERNEL, int VX, int BX, int BY, int KB, int XCD, int NT = 0, int WPE = 1>
hipError_t launch_zc(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)BX * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, BX * BY)) return hipErrorInvalidConfiguration;
    if (KERNEL == KL_KERNEL_ADVEC_U)
        hipLaunchKernelGGL((advec_u_zc<T, VX, BX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(BX, BY), 0, s, a);
    else
        hipLaunchKernelGGL((diff_uvw_zc<T, VX, BX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(BX, BY), 0, s, a);
    return hipGetLastError();
}

template <typename T, int KERNEL, int VX, int BY, int KB, int XCD, int NT = 0, int WPE = 1>
hipError_t launch_zl(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    if (KERNEL == KL_KERNEL_ADVEC_U)
        hipLaunchKernelGGL((advec_u_zl<T, VX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    else
        hipLaunchKernelGGL((diff_uvw_zl<T, VX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    return hipGetLastError();
}

template <typename T, int KERNEL, int VX, int BY, int KB, int NT = 0, int WPE = 1>
hipError_t launch_zl_batch(const void *descs, const void *tiles, int ntiles, int nblocks, int *queue, hipStream_t s)
{
    if (KERNEL == KL_KERNEL_ADVEC_U)
        hipLaunchKernelGGL((advec_u_zl_batch<T, VX, BY, KB, NT, WPE>), dim3(nblocks), dim3(64, BY), 0, s,
                           (const StencilArgs<T> *)descs, (const int4 *)tiles, ntiles, queue);
    else
        hipLaunchKernelGGL((diff_uvw_zl_batch<T, VX, BY, KB, NT, WPE>), dim3(nblocks), dim3(64, BY), 0, s,
                           (const StencilArgs<T> *)descs, (const int4 *)tiles, ntiles, queue);
    return hipGetLastError();
}

template <typename T, int KERNEL, int VX, int BY, int KB, int NT = 0, int WPE = 1>
int zl_batch_occupancy()
{
    int n = 0;
    hipError_t e;
    if (KERNEL == KL_KERNEL_ADVEC_U)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, advec_u_zl_batch<T, VX, BY, KB, NT, WPE>, 64 * BY, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, diff_uvw_zl_batch<T, VX, BY, KB, NT, WPE>, 64 * BY, 0);
    return e == hipSuccess && n > 0 ? n : 1;
}

template <typename T, int VX, int BY, int KB, int XCD, int NT = 0, int WPE = 1, int MODE = FUSE_STEP>
hipError_t launch_step(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((step_zl<T, VX, BY, KB, XCD, NT, WPE, MODE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && (MODE & FUSE_NOYZ)) e = launch_fill_yz_images(h, h.ut, h.vt, h.wt, s);
    return e;
}

template <typename T, int VX, int BY, int KB, int NT = 0, int WPE = 1, int MODE = FUSE_STEP>
hipError_t launch_step_batch(const void *descs, const void *tiles, int ntiles, int nblocks, int *queue,
                             hipStream_t s)
{
    hipLaunchKernelGGL((step_zl_batch<T, VX, BY, KB, NT, WPE, MODE>), dim3(nblocks), dim3(64, BY), 0, s,
                       (const StencilArgs<T> *)descs, (const int4 *)tiles, ntiles, queue);
    return hipGetLastError();
}

template <typename T, int VX, int BY, int KB, int NT = 0, int WPE = 1, int MODE = FUSE_STEP>
int step_batch_occupancy()
{
    int n = 0;
    const hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, step_zl_batch<T, VX, BY, KB, NT, WPE, MODE>, 64 * BY, 0);
    return e == hipSuccess && n > 0 ? n : 1;
}

// Row-flattened tiles.  Tendencies stream past the caches when the arrays of a
// call exceed the memory-side cache (256 MB): 301x203x151 FP32 diff_uvw (221 MB)
// 57 us cached, 60 streamed; 320x320x160 (393 MB) 115 cached, 95 streamed.
template <typename T, int V, int MODE, int THREADS>
hipError_t launch_rf(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.rf_cpr = rf_chunks(h.itot, V);
    a.rf_rows = rf_rows(h.jtot, a.rf_cpr, THREADS);
    a.nby = (int)cdivu(h.jtot, a.rf_rows);
    a.rf_kb = rf_levels(a.nby, h.ktot, THREADS);
    a.nbz = (int)cdivu(h.ktot, a.rf_kb);
    const uint64_t nb = (uint64_t)a.nby * a.nbz;
    a.nbx = a.nby % 8 == 0 ? a.nby : (int)nb;
    const int threads = (std::max(a.rf_rows, 2) * a.rf_cpr + 63) / 64 * 64;
    if (!grid_fits(nb, threads) || threads > THREADS) return hipErrorInvalidConfiguration;
    const size_t lds = rf_lds_bytes(a.rf_cpr, a.rf_rows);
    constexpr int arrays = (MODE & RF_DIFF) ? 6 : 4;
    if ((double)arrays * h.itot * h.jtot * h.ktot * sizeof(T) > 256e6)
        hipLaunchKernelGGL((rf_kernel<T, V, MODE, 1, THREADS>), dim3((unsigned)nb), dim3(threads), lds, s, a);
    else
        hipLaunchKernelGGL((rf_kernel<T, V, MODE, 0, THREADS>), dim3((unsigned)nb), dim3(threads), lds, s, a);
    return hipGetLastError();
}

template <typename T, int V, int MODE, int THREADS, int NT = 1>
hipError_t launch_rf_batch(const void *descs, const void *tiles, int ntiles, int nblocks, int *queue, hipStream_t s)
{
    hipLaunchKernelGGL((rf_batch<T, V, MODE, NT, THREADS>), dim3(nblocks), dim3(THREADS),
                       THREADS == 256 ? RF_LDS_256 : RF_LDS_512, s, (const StencilArgs<T> *)descs, (const int4 *)tiles,
                       ntiles, queue);
    return hipGetLastError();
}

template <typename T, int V, int MODE, int THREADS>
int rf_batch_occupancy()
{
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, rf_batch<T, V, MODE, 1, THREADS>, THREADS,
                                                                      THREADS == 256 ? RF_LDS_256 : RF_LDS_512);
    return e == hipSuccess && n > 0 ? n : 1;
}

// The paper's schemes; tendencies are streamed past the memory-side cache where
// a call's arrays do not fit it (256 MB), as in launch_rf.
template <typename T, int V, int KERNEL>
hipError_t launch_les_rf(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    const LesRfShape sh = les_rf_shape(KERNEL, h.itot, h.jtot, V);
    a.rf_cpr = sh.W;
    a.rf_rows = sh.R;
    a.nbx = (int)cdivu(rf_chunks(h.itot, V), sh.W);
    a.nby = (int)cdivu(h.jtot, sh.R);
    a.rf_kb = les_rf_levels(a.nbx * a.nby, h.ktot);
    a.nbz = (int)cdivu(h.ktot, a.rf_kb);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, sh.threads) || sh.threads > 512) return hipErrorInvalidConfiguration;
    constexpr int arrays = KERNEL == KL_KERNEL_ADVEC_U_2I5 ? 4 : 7;
    const bool nt = (double)arrays * h.itot * h.jtot * h.ktot * sizeof(T) > 256e6;
    const dim3 grid((unsigned)nb), block(sh.threads);
    if (KERNEL == KL_KERNEL_ADVEC_U_2I5) {
        if (nt)
            hipLaunchKernelGGL((advec_u_2i5_rf<T, V, 1>), grid, block, sh.lds, s, a);
        else
            hipLaunchKernelGGL((advec_u_2i5_rf<T, V, 0>), grid, block, sh.lds, s, a);
    } else {
        if (nt)
            hipLaunchKernelGGL((diff_smag_rf<T, V, 1>), grid, block, sh.lds, s, a);
        else
            hipLaunchKernelGGL((diff_smag_rf<T, V, 0>), grid, block, sh.lds, s, a);
    }
    return hipGetLastError();
}

// The row-flattened tile shape of a grid in a persistent kernel of configuration v.
template <typename T>
void batch_shape(const Variant &v, const kl_grid_t *g, int rf_kb, StencilArgs<T> &a)
{
    if (v.family != FAMILY_RF) return;
    const TileShape t = batch_tiles(v, g, rf_kb);
    a.rf_cpr = rf_chunks(g->itot, v.vx);
    a.rf_rows = t.by;
    a.rf_kb = t.kb;
}

// diff_uvw as three single-component passes (u, then v, then w) of the LDS
// z-march: the same values and arithmetic, three read/write streams in
// flight at a time instead of nine.
template <typename T, int VX, int BY, int KB, int XCD, int NT = 0>
hipError_t launch_zl_split(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((diff_uvw_zl<T, VX, BY, KB, XCD, NT, 1, 1>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    hipLaunchKernelGGL((diff_uvw_zl<T, VX, BY, KB, XCD, NT, 1, 2>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    hipLaunchKernelGGL((diff_uvw_zl<T, VX, BY, KB, XCD, NT, 1, 4>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    return hipGetLastError();
}

template <typename T, int VX, int BY, int KB, int XCD, int NT = 0, int WPE = 1, int PAIR = 0, int YS = 0>
hipError_t launch_advec5_zl(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    if (PAIR)
        hipLaunchKernelGGL((advec_u_2i5_zlp<T, VX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    else
        hipLaunchKernelGGL((advec_u_2i5_zl<T, VX, BY, KB, XCD, NT, WPE, YS>), dim3((unsigned)nb), dim3(64, BY), 0, s,
                           a);
    return hipGetLastError();
}

template <typename T, int VX, int BY, int KB, int XCD, int NT = 0, int HL = 1>
hipError_t launch_advec5_zr(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((advec_u_2i5_zr<T, VX, BY, KB, XCD, NT, 1, HL>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    return hipGetLastError();
}

template <typename T, int VX, int BY, int KB, int XCD, int NT = 0, int WPE = 1, int RING = 0>
hipError_t launch_smag_zl(const HostArgs &h, hipStream_t s)
{
    StencilArgs<T> a = device_args<T>(h);
    a.nbx = (int)cdivu(h.itot, (int64_t)64 * VX);
    a.nby = (int)cdivu(h.jtot, BY);
    a.nbz = (int)cdivu(h.ktot, KB);
    const uint64_t nb = (uint64_t)a.nbx * a.nby * a.nbz;
    if (!grid_fits(nb, 64 * BY)) return hipErrorInvalidConfiguration;
    if constexpr (RING)
        hipLaunchKernelGGL((diff_smag_zr<T, VX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    else
        hipLaunchKernelGGL((diff_smag_zl<T, VX, BY, KB, XCD, NT, WPE>), dim3((unsigned)nb), dim3(64, BY), 0, s, a);
    return hipGetLastError();
}

}  // namespace kl

#define KL_STR2(x) #x
#define KL_STR(x) KL_STR2(x)

// One z-marching configuration entry.
#define KL_ZC(T, DT, KERN, VX, BX, BY, KB, XCD)                                                   \
    Variant{"zc_v" KL_STR(VX) "_b" KL_STR(BX) "x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD), \
            KERN, DT, FAMILY_ZC, VX, BX, BY, KB, XCD, &launch_zc<T, KERN, VX, BX, BY, KB, XCD>, nullptr, \
            nullptr}

#define KL_ZC_XCD(T, DT, KERN, VX, BX, BY, KB) \
    KL_ZC(T, DT, KERN, VX, BX, BY, KB, 0), KL_ZC(T, DT, KERN, VX, BX, BY, KB, 1)

#define KL_ZC_KB(T, DT, KERN, VX, BX, BY) \
    KL_ZC_XCD(T, DT, KERN, VX, BX, BY, 16), KL_ZC_XCD(T, DT, KERN, VX, BX, BY, 64)

#define KL_ZC_BLOCKS(T, DT, KERN, VX)                                           \
    KL_ZC_KB(T, DT, KERN, VX, 64, 1), KL_ZC_KB(T, DT, KERN, VX, 64, 4),          \
        KL_ZC_KB(T, DT, KERN, VX, 128, 2), KL_ZC_KB(T, DT, KERN, VX, 256, 1)

// One LDS-staged z-marching configuration entry (block 64 x BY).
#define KL_ZL(T, DT, KERN, VX, BY, KB, XCD)                                                   \
    Variant{"zl_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD), KERN, DT, \
            FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_zl<T, KERN, VX, BY, KB, XCD>,             \
            &launch_zl_batch<T, KERN, VX, BY, KB>, &zl_batch_occupancy<T, KERN, VX, BY, KB>}

#define KL_ZL_XCD(T, DT, KERN, VX, BY, KB) KL_ZL(T, DT, KERN, VX, BY, KB, 0), KL_ZL(T, DT, KERN, VX, BY, KB, 1)

#define KL_ZL_KB(T, DT, KERN, VX, BY)                                                \
    KL_ZL_XCD(T, DT, KERN, VX, BY, 32), KL_ZL_XCD(T, DT, KERN, VX, BY, 64), \
        KL_ZL_XCD(T, DT, KERN, VX, BY, 128)

#define KL_ZL_BLOCKS(T, DT, KERN, VX) \
    KL_ZL_KB(T, DT, KERN, VX, 4), KL_ZL_KB(T, DT, KERN, VX, 8), KL_ZL_KB(T, DT, KERN, VX, 16)

// Extra configurations: streaming tendencies (NT), slab-local XCD order and
// a waves-per-SIMD floor (WPE), named ..._x<XCD>_nt<NT>_w<WPE>.
#define KL_ZLX(T, DT, KERN, VX, BY, KB, XCD, NT, WPE)                                                 \
    Variant{"zl_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT)     \
            "_w" KL_STR(WPE),                                                                         \
            KERN, DT, FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_zl<T, KERN, VX, BY, KB, XCD, NT, WPE>,   \
            &launch_zl_batch<T, KERN, VX, BY, KB, NT, WPE>, &zl_batch_occupancy<T, KERN, VX, BY, KB, NT, WPE>}

#define KL_ZCX(T, DT, KERN, VX, BX, BY, KB, XCD, NT, WPE)                                              \
    Variant{"zc_v" KL_STR(VX) "_b" KL_STR(BX) "x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt"    \
            KL_STR(NT) "_w" KL_STR(WPE),                                                              \
            KERN, DT, FAMILY_ZC, VX, BX, BY, KB, XCD, &launch_zc<T, KERN, VX, BX, BY, KB, XCD, NT, WPE>, \
            nullptr, nullptr}

#define KL_ZLX_SET(T, DT, KERN, VX)                                                                     \
    KL_ZLX(T, DT, KERN, VX, 8, 32, 2, 0, 1), KL_ZLX(T, DT, KERN, VX, 8, 32, 2, 1, 1),                  \
        KL_ZLX(T, DT, KERN, VX, 8, 32, 0, 1, 1), KL_ZLX(T, DT, KERN, VX, 8, 128, 2, 0, 1),             \
        KL_ZLX(T, DT, KERN, VX, 8, 128, 2, 1, 1), KL_ZLX(T, DT, KERN, VX, 8, 128, 0, 1, 1),            \
        KL_ZLX(T, DT, KERN, VX, 8, 32, 0, 0, 4), KL_ZLX(T, DT, KERN, VX, 8, 32, 2, 1, 4),              \
        KL_ZLX(T, DT, KERN, VX, 4, 64, 2, 1, 1), KL_ZLX(T, DT, KERN, VX, 16, 64, 2, 1, 1)

#define KL_NT2_SET(T, DT, KERN, VX)                                                                     \
    KL_ZLX(T, DT, KERN, VX, 4, 64, 2, 2, 1), KL_ZLX(T, DT, KERN, VX, 4, 128, 2, 1, 1),                 \
        KL_ZLX(T, DT, KERN, VX, 4, 128, 2, 2, 1), KL_ZLX(T, DT, KERN, VX, 4, 256, 2, 1, 1),            \
        KL_ZLX(T, DT, KERN, VX, 8, 64, 2, 1, 1), KL_ZLX(T, DT, KERN, VX, 8, 64, 2, 2, 1),              \
        KL_ZLX(T, DT, KERN, VX, 4, 64, 0, 1, 1), KL_ZCX(T, DT, KERN, VX, 64, 4, 16, 2, 2, 1),          \
        KL_ZCX(T, DT, KERN, VX, 64, 2, 16, 2, 1, 1), KL_ZCX(T, DT, KERN, VX, 64, 8, 16, 2, 1, 1)

#define KL_ZCX_SET(T, DT, KERN, VX)                                                                     \
    KL_ZCX(T, DT, KERN, VX, 64, 4, 16, 2, 0, 1), KL_ZCX(T, DT, KERN, VX, 64, 4, 16, 2, 1, 1),          \
        KL_ZCX(T, DT, KERN, VX, 64, 4, 16, 0, 1, 1), KL_ZCX(T, DT, KERN, VX, 64, 4, 32, 0, 1, 1)

// Fused-step configurations (kernel KL_KERNEL_STEP).
#define KL_ST(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"step_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),    \
            KL_KERNEL_STEP, DT, FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_step<T, VX, BY, KB, XCD, NT>,     \
            &launch_step_batch<T, VX, BY, KB, NT>, &step_batch_occupancy<T, VX, BY, KB, NT>}

// The same with a register cap of 512 / WPE per lane (WPE waves per SIMD)
// and the ring options of MODE (FUSE_HALO3, FUSE_RING6), named by TAG.
#define KL_STW(T, DT, VX, BY, KB, XCD, NT, WPE, MODE, TAG)                                               \
    Variant{"step_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT)     \
            "_w" KL_STR(WPE) TAG,                                                                        \
            KL_KERNEL_STEP, DT, FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_step<T, VX, BY, KB, XCD, NT, WPE, MODE>, \
            &launch_step_batch<T, VX, BY, KB, NT, WPE, MODE>, &step_batch_occupancy<T, VX, BY, KB, NT, WPE, MODE>}

// A fused step whose y and z ghost cells are refilled by a second kernel
// (FUSE_NOYZ).  Its persistent form (served ticks) is the same tile writing
// those ghost cells itself, which gives the same bits without a refill
// launch per tick.
#define KL_STY(T, DT, VX, BY, KB, XCD, NT, MODE, TAG)                                                    \
    Variant{"step_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT)     \
            "_w1" TAG,                                                                                   \
            KL_KERNEL_STEP, DT, FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_step<T, VX, BY, KB, XCD, NT, 1, (MODE) | FUSE_NOYZ>, \
            &launch_step_batch<T, VX, BY, KB, NT, 1, MODE>, &step_batch_occupancy<T, VX, BY, KB, NT, 1, MODE>}

#define KL_ST_SET(T, DT, VX)                                                                             \
    KL_ST(T, DT, VX, 8, 32, 0, 0), KL_ST(T, DT, VX, 4, 64, 2, 1), KL_ST(T, DT, VX, 8, 32, 2, 1),         \
        KL_ST(T, DT, VX, 4, 128, 2, 1), KL_ST(T, DT, VX, 8, 64, 0, 1), KL_ST(T, DT, VX, 4, 32, 0, 0),    \
        KL_ST(T, DT, VX, 4, 8, 0, 0), KL_ST(T, DT, VX, 4, 16, 0, 0), KL_ST(T, DT, VX, 8, 8, 0, 0),       \
        KL_ST(T, DT, VX, 2, 16, 0, 0)

// Fused advec_u + diff_uvw configurations (kernel KL_KERNEL_ADVEC_DIFF): the
// fused-step tile accumulating into the tendencies.
#define KL_AD(T, DT, VX, BY, KB, XCD, NT)                                                                 \
    Variant{"ad_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),      \
            KL_KERNEL_ADVEC_DIFF, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                    \
            &launch_step<T, VX, BY, KB, XCD, NT, 1, FUSE_PAIR>, &launch_step_batch<T, VX, BY, KB, NT, 1, FUSE_PAIR>, \
            &step_batch_occupancy<T, VX, BY, KB, NT, 1, FUSE_PAIR>,                                       \
            &launch_step<T, VX, BY, KB, XCD, NT, 1, FUSE_PAIR | FUSE_FRESH>,                              \
            &launch_step_batch<T, VX, BY, KB, NT, 1, FUSE_PAIR | FUSE_FRESH>,                             \
            &step_batch_occupancy<T, VX, BY, KB, NT, 1, FUSE_PAIR | FUSE_FRESH>}

#define KL_ADW(T, DT, VX, BY, KB, XCD, NT, WPE, MODE, TAG)                                               \
    Variant{"ad_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT)       \
            "_w" KL_STR(WPE) TAG,                                                                        \
            KL_KERNEL_ADVEC_DIFF, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                    \
            &launch_step<T, VX, BY, KB, XCD, NT, WPE, FUSE_PAIR | (MODE)>,                                \
            &launch_step_batch<T, VX, BY, KB, NT, WPE, FUSE_PAIR | (MODE)>,                               \
            &step_batch_occupancy<T, VX, BY, KB, NT, WPE, FUSE_PAIR | (MODE)>,                            \
            &launch_step<T, VX, BY, KB, XCD, NT, WPE, FUSE_PAIR | FUSE_FRESH | (MODE)>,                   \
            &launch_step_batch<T, VX, BY, KB, NT, WPE, FUSE_PAIR | FUSE_FRESH | (MODE)>,                  \
            &step_batch_occupancy<T, VX, BY, KB, NT, WPE, FUSE_PAIR | FUSE_FRESH | (MODE)>}

#define KL_AD_SET(T, DT, VX)                                                                             \
    KL_AD(T, DT, VX, 4, 8, 0, 0), KL_AD(T, DT, VX, 8, 8, 0, 0), KL_AD(T, DT, VX, 4, 32, 0, 0),           \
        KL_AD(T, DT, VX, 8, 32, 0, 0), KL_AD(T, DT, VX, 8, 32, 2, 1), KL_AD(T, DT, VX, 4, 64, 2, 1),     \
        KL_AD(T, DT, VX, 8, 64, 2, 1), KL_AD(T, DT, VX, 4, 128, 2, 1), KL_AD(T, DT, VX, 8, 128, 2, 1),   \
        KL_AD(T, DT, VX, 8, 256, 2, 1), KL_AD(T, DT, VX, 4, 256, 2, 1)

// Top-down slab order (XCD = 3) for a kernel that follows another sweep.
#define KL_REV_SET(T, DT, KERN, VX)                                                                     \
    KL_ZLX(T, DT, KERN, VX, 4, 64, 3, 1, 1), KL_ZLX(T, DT, KERN, VX, 4, 128, 3, 1, 1),                 \
        KL_ZLX(T, DT, KERN, VX, 4, 256, 3, 1, 1), KL_ZLX(T, DT, KERN, VX, 8, 32, 3, 1, 1),             \
        KL_ZLX(T, DT, KERN, VX, 8, 128, 3, 1, 1), KL_ZLX(T, DT, KERN, VX, 4, 128, 3, 0, 1)

// Waves-per-SIMD floors of 3 and 4 on the top-down slab configurations
// (fewer registers, more waves in flight).
#define KL_OCC_SET(T, DT, KERN, VX)                                                                     \
    KL_ZLX(T, DT, KERN, VX, 4, 256, 3, 1, 3), KL_ZLX(T, DT, KERN, VX, 4, 256, 3, 1, 4),                \
        KL_ZLX(T, DT, KERN, VX, 4, 128, 3, 1, 3), KL_ZLX(T, DT, KERN, VX, 4, 64, 3, 1, 4)

// Short z-marches for small grids (more tiles, shorter chains).
#define KL_SMALL_SET(T, DT, KERN, VX)                                                                   \
    KL_ZLX(T, DT, KERN, VX, 4, 8, 0, 0, 1), KL_ZLX(T, DT, KERN, VX, 4, 16, 0, 0, 1),                   \
        KL_ZLX(T, DT, KERN, VX, 8, 8, 0, 0, 1), KL_ZLX(T, DT, KERN, VX, 8, 16, 0, 1, 1)

// advec_u_2i5 LDS z-march configurations, named a5_v<VX>_b64x<BY>_k<KB>_x<XCD>_nt<NT>.
// The pair-unrolled march, named a5p_...
#define KL_A5P(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"a5p_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),       \
            KL_KERNEL_ADVEC_U_2I5, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                     \
            &launch_advec5_zl<T, VX, BY, KB, XCD, NT, 1, 1>, nullptr, nullptr}

// advec_u_2i5 with each y face evaluated once (shared through LDS), named
// a5s_v<VX>_b64x<BY>_k<KB>_x<XCD>_nt<NT>.
#define KL_A5S(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"a5s_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),       \
            KL_KERNEL_ADVEC_U_2I5, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                     \
            &launch_advec5_zl<T, VX, BY, KB, XCD, NT, 1, 0, 1>, nullptr, nullptr}

// The parity-slot march (no register copies at the end of a level), named a5r_...
#define KL_A5R(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"a5r_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),       \
            KL_KERNEL_ADVEC_U_2I5, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                     \
            &launch_advec5_zr<T, VX, BY, KB, XCD, NT>, nullptr, nullptr}

// The same with the u halo rows loaded HL levels ahead, named a5r_..._h<HL>.
#define KL_A5RH(T, DT, VX, BY, KB, XCD, NT, HL)                                                             \
    Variant{"a5r_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT)        \
            "_h" KL_STR(HL),                                                                                \
            KL_KERNEL_ADVEC_U_2I5, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                     \
            &launch_advec5_zr<T, VX, BY, KB, XCD, NT, HL>, nullptr, nullptr}

#define KL_A5(T, DT, VX, BY, KB, XCD, NT)                                                                   \
    Variant{"a5_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),        \
            KL_KERNEL_ADVEC_U_2I5, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                     \
            &launch_advec5_zl<T, VX, BY, KB, XCD, NT>, nullptr, nullptr}

// diff_smag LDS z-march configurations, named s2_v<VX>_b64x<BY>_k<KB>_x<XCD>_nt<NT>.
#define KL_S2(T, DT, VX, BY, KB, XCD, NT)                                                                   \
    Variant{"s2_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),        \
            KL_KERNEL_DIFF_SMAG, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                       \
            &launch_smag_zl<T, VX, BY, KB, XCD, NT>, nullptr, nullptr}

// diff_smag with the parity-slot march, named s2r_v<VX>_b64x<BY>_k<KB>_x<XCD>_nt<NT>.
#define KL_S2R(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"s2r_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),       \
            KL_KERNEL_DIFF_SMAG, DT, FAMILY_ZL, VX, 64, BY, KB, XCD,                                       \
            &launch_smag_zl<T, VX, BY, KB, XCD, NT, 1, 1>, nullptr, nullptr}

// diff_uvw split into per-component passes, named zl3_v<VX>_b64x<BY>_k<KB>_x<XCD>_nt<NT>.
#define KL_ZL3(T, DT, VX, BY, KB, XCD, NT)                                                                  \
    Variant{"zl3_v" KL_STR(VX) "_b64x" KL_STR(BY) "_k" KL_STR(KB) "_x" KL_STR(XCD) "_nt" KL_STR(NT),       \
            KL_KERNEL_DIFF_UVW, DT, FAMILY_ZL, VX, 64, BY, KB, XCD, &launch_zl_split<T, VX, BY, KB, XCD, NT>, \
            nullptr, nullptr}

// Row-flattened configurations, named rf_t<block threads>; they size their
// tiles to the grid themselves.
#define KL_RF(T, DT, KERN, V, MODE, THREADS)                                                                \
    Variant{"rf_t" KL_STR(THREADS), KERN, DT, FAMILY_RF, V, THREADS, 1, 0, 0, &launch_rf<T, V, MODE, THREADS>, nullptr, \
            nullptr}

#define KL_RFB(T, DT, KERN, V, MODE, THREADS)                                                               \
    Variant{"rf_t" KL_STR(THREADS), KERN, DT, FAMILY_RF, V, THREADS, 1, 0, 0, &launch_rf<T, V, MODE, THREADS>, \
            &launch_rf_batch<T, V, MODE, THREADS>, &rf_batch_occupancy<T, V, MODE, THREADS>,                \
            &launch_rf<T, V, (MODE) | RF_FRESH, THREADS>, &launch_rf_batch<T, V, (MODE) | RF_FRESH, THREADS>, \
            &rf_batch_occupancy<T, V, (MODE) | RF_FRESH, THREADS>, &launch_rf_batch<T, V, MODE, THREADS, 0>}

#define KL_RFL(T, DT, KERN, V)                                                                              \
    Variant{"rf_t512", KERN, DT, FAMILY_RF, V, 512, 1, 0, 0, &launch_les_rf<T, V, KERN>, nullptr, nullptr}

#define KL_RF_SET(T, DT, V)                                                                                 \
    switch (kernel) {                                                                                       \
    case KL_KERNEL_ADVEC_U:                                                                                 \
        out.push_back(KL_RF(T, DT, KL_KERNEL_ADVEC_U, V, RF_ADVEC, 256));                                   \
        out.push_back(KL_RF(T, DT, KL_KERNEL_ADVEC_U, V, RF_ADVEC, 512));                                   \
        break;                                                                                              \
    case KL_KERNEL_DIFF_UVW:                                                                                \
        out.push_back(KL_RF(T, DT, KL_KERNEL_DIFF_UVW, V, RF_DIFF, 256));                                   \
        out.push_back(KL_RF(T, DT, KL_KERNEL_DIFF_UVW, V, RF_DIFF, 512));                                   \
        break;                                                                                              \
    case KL_KERNEL_ADVEC_DIFF:                                                                              \
        out.push_back(KL_RFB(T, DT, KL_KERNEL_ADVEC_DIFF, V, RF_ADVEC | RF_DIFF, 256));                     \
        out.push_back(KL_RFB(T, DT, KL_KERNEL_ADVEC_DIFF, V, RF_ADVEC | RF_DIFF, 512));                     \
        break;                                                                                              \
    case KL_KERNEL_STEP:                                                                                    \
        out.push_back(KL_RFS(T, DT, V, 256));                                                               \
        out.push_back(KL_RFS(T, DT, V, 512));                                                               \
        break;                                                                                              \
    case KL_KERNEL_ADVEC_U_2I5: out.push_back(KL_RFL(T, DT, KL_KERNEL_ADVEC_U_2I5, V)); break;              \
    case KL_KERNEL_DIFF_SMAG: out.push_back(KL_RFL(T, DT, KL_KERNEL_DIFF_SMAG, V)); break;                  \
    default: break;                                                                                         \
    }

#define KL_RFS(T, DT, V, THREADS)                                                                           \
    Variant{"rf_t" KL_STR(THREADS), KL_KERNEL_STEP, DT, FAMILY_RF, V, THREADS, 1, 0, 0,                     \
            &launch_rf<T, V, RF_ADVEC | RF_DIFF | RF_STEP, THREADS>,                                        \
            &launch_rf_batch<T, V, RF_ADVEC | RF_DIFF | RF_STEP, THREADS>,                                  \
            &rf_batch_occupancy<T, V, RF_ADVEC | RF_DIFF | RF_STEP, THREADS>, nullptr, nullptr, nullptr,    \
            &launch_rf_batch<T, V, RF_ADVEC | RF_DIFF | RF_STEP, THREADS, 0>}
