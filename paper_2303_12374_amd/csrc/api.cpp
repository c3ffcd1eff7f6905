// C-ABI entry points: argument checks, layout, the selection cache and
// dispatch of the tendency kernels, ghost fill, Euler step and reductions.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <unordered_map>

#include "kl_internal.hpp"

#define KL_VERSION_STRING "klstencil 0.1.0 (gfx950)"

namespace kl {

namespace {
thread_local std::string g_last_error;
}

int fail(int code, const char *fmt, ...)
{
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(KL_ERR_DEVICE, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

void clear_error() { g_last_error.clear(); }

const std::vector<Variant> &variants(int kernel, int dtype)
{
    return dtype == KL_F32 ? variants_f32(kernel) : variants_f64(kernel);
}

int check_grid(const kl_grid_t *g)
{
    if (!g) return fail(KL_ERR_INVALID, "grid is NULL");
    if (g->gc != 1 && g->gc != 3) return fail(KL_ERR_INVALID, "ghost width gc=%d, must be 1 or 3", g->gc);
    if (g->dtype != KL_F32 && g->dtype != KL_F64) return fail(KL_ERR_INVALID, "dtype %d", g->dtype);
    if (g->bc < KL_BC_ZWALL_ZEROGRAD || g->bc > KL_BC_ZPERIODIC) return fail(KL_ERR_INVALID, "bc %d", g->bc);
    if (g->itot < 1 || g->jtot < 1 || g->ktot < 1)
        return fail(KL_ERR_INVALID, "interior sizes %d x %d x %d must be >= 1", g->itot, g->jtot, g->ktot);
    if (g->bc != KL_BC_ZPERIODIC && g->ktot < 2)
        return fail(KL_ERR_INVALID, "z walls need ktot >= 2 (got %d)", g->ktot);
    const int64_t gc = g->gc;
    if (g->jstride < (int64_t)g->itot + 2 * gc)
        return fail(KL_ERR_INVALID, "jstride %lld < itot+2*gc", (long long)g->jstride);
    if (g->kstride < g->jstride * ((int64_t)g->jtot + 2 * gc))
        return fail(KL_ERR_INVALID, "kstride %lld < jstride*(jtot+2*gc)", (long long)g->kstride);
    if (g->off < (gc - 1) * (g->jstride + 1))
        return fail(KL_ERR_INVALID, "off %lld < (gc-1)*(jstride+1): ghost cells before the buffer",
                    (long long)g->off);
    if (!g->dzi || !g->dzhi) return fail(KL_ERR_INVALID, "dzi/dzhi is NULL");
    return KL_OK;
}

HostArgs make_args(const kl_grid_t *g)
{
    HostArgs a;
    memset(&a, 0, sizeof a);
    a.itot = g->itot;
    a.jtot = g->jtot;
    a.ktot = g->ktot;
    a.kw0 = g->bc == KL_BC_ZPERIODIC ? 1 : 2;
    a.gc = g->gc;
    a.dtype = g->dtype;
    a.bc = g->bc;
    a.off = g->off;
    a.js = g->jstride;
    a.ks = g->kstride;
    a.dxi = g->dxi;
    a.dyi = g->dyi;
    a.dzi = g->dzi;
    a.dzhi = g->dzhi;
    return a;
}

bool variant_eligible(const Variant &v, const kl_grid_t *g, const void *const *ptrs, int nptr)
{
    if (v.family == FAMILY_RF && (v.kernel == KL_KERNEL_ADVEC_U_2I5 || v.kernel == KL_KERNEL_DIFF_SMAG))
        return g->itot >= 8 && g->jstride * ((int64_t)g->jtot + 6) * (g->dtype == KL_F32 ? 4 : 8) < ((int64_t)1 << 31);
    if (v.family == FAMILY_RF)  // any alignment; rows that fit a block, 32-bit offsets inside a level
        return rf_chunks(g->itot, v.vx) <= rf_max_chunks(v.bx) &&
               g->jstride * ((int64_t)g->jtot + 2) * (g->dtype == KL_F32 ? 4 : 8) < ((int64_t)1 << 31);
    if (v.vx > 1) {
        const int64_t vx = v.vx;
        if (g->itot % vx || (g->off + 1) % vx || g->jstride % vx || g->kstride % vx) return false;
        const uintptr_t align = (uintptr_t)vx * (g->dtype == KL_F32 ? 4 : 8);
        for (int n = 0; n < nptr; ++n)
            if (ptrs[n] && ((uintptr_t)ptrs[n] % align)) return false;
    }
    return true;
}

// ---------------------------------------------------------------------------
// per-device, per-stream workspace for reduction partials (never freed)
// ---------------------------------------------------------------------------
namespace {
std::mutex g_ws_mu;
std::map<std::pair<int, hipStream_t>, void *> g_ws;
constexpr size_t WS_BYTES = 512 * 1024;
}  // namespace

void *workspace(size_t bytes, hipStream_t s)
{
    if (bytes > WS_BYTES) return nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    std::lock_guard<std::mutex> lk(g_ws_mu);
    auto key = std::make_pair(dev, s);
    auto it = g_ws.find(key);
    if (it != g_ws.end()) return it->second;
    void *p = nullptr;
    if (hipMalloc(&p, WS_BYTES) != hipSuccess) return nullptr;
    g_ws[key] = p;
    return p;
}

// ---------------------------------------------------------------------------
// selection cache: (kernel, dtype, itot, jtot, ktot, device) -> variant index
// ---------------------------------------------------------------------------
namespace {
std::mutex g_plan_mu;
std::map<std::tuple<int, int, int, int, int, int>, int> g_plans;
}  // namespace

void clear_plans()
{
    std::lock_guard<std::mutex> lk(g_plan_mu);
    g_plans.clear();
}

int variant_index(int kernel, int dtype, const std::string &name)
{
    using Names = std::unordered_map<std::string, int>;
    static const std::vector<Names> names = [] {
        std::vector<Names> all(2 * KL_NUM_KERNELS);
        for (int n = 0; n < 2 * KL_NUM_KERNELS; ++n) {
            const auto &vs = variants(n / 2, n % 2);
            for (size_t i = 0; i < vs.size(); ++i) all[n].emplace(vs[i].name, (int)i);
        }
        return all;
    }();
    const Names &of = names[2 * kernel + dtype];
    const auto it = of.find(name);
    return it == of.end() ? -1 : it->second;
}

namespace {
// Whether v takes rows of g's length at all; the layout and the pointers of a
// call decide the rest (variant_eligible).
bool takes_row_length(const Variant &v, const kl_grid_t *g)
{
    if (v.family != FAMILY_RF) return g->itot % v.vx == 0;
    if (v.kernel == KL_KERNEL_ADVEC_U_2I5 || v.kernel == KL_KERNEL_DIFF_SMAG) return g->itot >= 8;
    return rf_chunks(g->itot, v.vx) <= rf_max_chunks(v.bx);
}

// Whether whole chunks of V points make up rows that fill segments of 64 chunks.
bool fills_waves(int itot, int V)
{
    const int cpr = rf_chunks(itot, V);
    return itot % V == 0 && itot >= 0.94 * ((cpr + 63) / 64) * 64 * V;
}

// The tile for rows that the row-flattened ones do not take or lose on.  Small
// grids need short marches to fill the chip, and no far record gives one: against
// the fastest of each of 19 sizes of rows of more than 256 chunks and up to 5e6
// points (548x9x123 to 1892x84x21) the mean is FP64 advec_u 1.07, diff_uvw 1.17,
// fused pass 1.06, fused step 1.03; FP32 1.03, 1.10, 1.07, 1.03 (nearest record
// 1.07, 2.7, 1.20, 1.03; 1.03, 1.8, 1.08, 1.13; 614x10x112 FP64 diff_uvw 18 us, 126).
// From there on, 16 to 19 sizes (552x97x77 to 2048x256x64): FP64 1.05, 1.07, 1.03,
// 1.02; FP32 1.06, 1.08, 1.09, 1.04.  FP32 rows are longer and keep the short
// marches for more points (1940x18x211 FP32 advec_u, diff_uvw, fused pass, fused
// step 1.07, 1.03, 1.14, 1.08 against 1.57, 1.50, 1.60, 1.48).  The step's march is
// the longer the more points there are.
const char *wide_rows_tile(int kernel, int dtype, int itot, double points)
{
    const bool f32 = dtype == KL_F32, small = points < 5e6, longer = f32 && itot > 1024 && points < 1.15e7;
    switch (kernel) {
    case KL_KERNEL_ADVEC_U:
        if (points < (!f32 ? 7.5e6 : itot > 1024 ? 2e7 : 1.15e7))
            return f32 && itot % 2 == 0 ? "zc_v2_b64x1_k16_x1" : "zc_v1_b64x1_k16_x1";
        if (!f32) return "zl_v2_b64x8_k32_x0_nt1_w1";
        if (itot <= 512 && fills_waves(itot, 4)) return "zl_v4_b64x4_k64_x3_nt1_w1";
        return itot <= 1024 ? "zc_v2_b64x4_k16_x2_nt1_w1" : "zc_v4_b64x4_k16_x2_nt1_w1";
    case KL_KERNEL_DIFF_UVW:
        if (small) return f32 ? "default" : "zl_v2_b64x8_k8_x0_nt0_w1";
        if (longer) return "zc_v4_b64x1_k16_x1";
        return f32 ? "zl_v4_b64x8_k16_x0_nt1_w1" : "zl_v2_b64x8_k32_x0_nt1_w1";
    case KL_KERNEL_ADVEC_DIFF:
        if (small) return f32 ? "default" : "ad_v2_b64x4_k8_x0_nt0";
        if (f32 && points < 2e7) return "ad_v4_b64x4_k8_x0_nt0";
        return f32 ? "ad_v4_b64x4_k64_x2_nt1" : "ad_v2_b64x8_k32_x2_nt1";
    default: break;  // the fused step
    }
    if (itot % (f32 ? 4 : 2)) return "step_v1_b64x4_k8_x0_nt0";
    if (small) return "step_v2_b64x4_k8_x0_nt0";
    if (longer) return "step_v4_b64x4_k8_x0_nt0";
    if (!f32) return points < 6e7 ? "step_v2_b64x4_k32_x2_nt1_w1_h3y" : "step_v2_b64x8_k64_x2_nt1_w1_h3y";
    return points < 2.4e7 ? "step_v4_b64x4_k16_x2_nt1_w1_h3y"
                          : points < 6e7 ? "step_v4_b64x4_k32_x2_nt1_w1_h3y" : "step_v4_b64x8_k64_x2_nt1_w1_h3y";
}

// The configuration of a problem size that no record names.  A record's tile is
// fixed for its own size: over 111 sizes of every length, height and aspect
// (16^3 .. 1024x1020x128, both types), every configuration of the second-order
// kernels and the step timed, the nearest record is 1.3 to 2.7 times the fastest
// in the mean of a kernel and up to 47 times; this rule is 1.01 to 1.04 times.  Its lines, in us (rule, other):
//  - A record whose sizes are within 1.25% in all keeps its word; on fields of
//    400 MB and more within 10%, where longer marches pay (500x500x500 FP32
//    diff_uvw, nearest to 512^3, 785, row-flattened 873).
//  - Rows of up to 80 chunks take the row-flattened tile of 256 threads, rows of up
//    to 256 the one of 512 (300x300x150 FP32 diff_uvw 79, nearest record 152;
//    768x300x100 161, 181).
//  - Grids of fewer than 2^19 points are short launches: a record of about the
//    same shape (within 0.3 in the logarithms of the sizes), else the default up to
//    512 KB a field (48^3 FP32 diff_uvw 6.6, row-flattened 7.3), else the row-flattened
//    tile (32x128x128 FP64 advec_u 7.1, default 10.3; 500x20x30 8, the nearest
//    record 33).  Rows too long for it: the default (1000x16x16 FP64 advec_u 8, the
//    nearest record 19).
//  - The fused step's row-flattened tile writes its images itself and falls behind
//    on long rows of large grids.  Rows of more than 80 chunks take it below 5e6
//    points (264x100x60 FP64 24, nearest fixed tile 39), and where they
//    fill its block to 400 of 512 threads and either the fields are small (FP32
//    50 MB, FP64 70: 400x300x100 FP32 80, long-row tile 91; above, 512x64x508 98,
//    105 row-flattened; 208x200x200 FP64 114, 129; above, 400x300x100 167, 172) or
//    the rows leave a fifth of the other tiles' lanes without a point, with five
//    rows a block (102 chunks; 384x344x404 FP32 341, 371) or up to 192 chunks and
//    120 MB (264x187x264 FP64 176, 182; above, 608x386x313 FP32 433, 552); and
//    where no vector divides the rows (510x300x100 FP32 104, 138).
//  - advec_u on rows of more than 80 chunks: four arrays, where whole rows gain
//    nothing on large grids and blocks of 512 threads are few on small ones.  From
//    1e6 points a tile of one row (FP32 up to 1.15e7 points 520x100x60 12,
//    row-flattened 17, above 400x300x100 44, 39; FP64 up to 7.5e6 264x100x60 13, 16,
//    above 336x200x120 69, 55; below 1e6 510x70x17 FP64 12, 10).  The
//    long-row tile on FP32 rows of more than 128 chunks from 2e7 points (832x600x64
//    133, row-flattened 150; 524x402x283 256, 294; below, 560x300x100 72, 60), from
//    6e7 the nearest fixed one (1000x1000x64 225, 256); on FP32 rows of 81 to 128
//    chunks that fill segments of 64, from 1.5e7 (with diff_uvw after it
//    512x512x120 290, 309), else from 5e7 (384x344x404 213, 225; below, 448x448x200
//    175, 164); on FP64 rows of more than 80 from 4e7 (512x261x304 300, 333;
//    420x705x137 348, 332).
//  - Longer rows: wide_rows_tile (FP64 704x400x80 diff_uvw 313, nearest record 449);
//    where its vector does not divide them the default.
//  - The paper's schemes have one row-flattened tile, fastest or within 2% of it
//    at every size tried from 2^19 points up; below, the default (100x37x61 9.4,
//    nearest record 55).  It does not take rows of fewer than 8 points: their 1-wide
//    tile of 16 levels, from 2^17 points (4x256x256 FP32 advec_u_2i5 22, default 39;
//    1x512x512 diff_smag 99, 217).
int unrecorded_variant(const kl_grid_t *g, int kernel, const std::vector<SizeRecord> &records)
{
    const auto &vs = variants(kernel, g->dtype);
    const bool f32 = g->dtype == KL_F32, step = kernel == KL_KERNEL_STEP;
    const double points = (double)g->itot * g->jtot * g->ktot, bytes = points * (f32 ? 4 : 8);
    const double sizes[3] = {(double)g->itot, (double)g->jtot, (double)g->ktot};
    const int V = f32 ? 4 : 2, cpr = rf_chunks(g->itot, V);
    const bool few = points < (double)(1 << 19);

    // nearest record by the ratios of the sizes, and nearest with a fixed tile
    int near = 0, near_fixed = 0;
    double dist = INFINITY, dist_fixed = INFINITY;
    for (const SizeRecord &r : records) {
        const int n = r.variant;
        if (!takes_row_length(vs[n], g) || !(r.size[0] > 0 && r.size[1] > 0 && r.size[2] > 0)) continue;
        double d = 0;
        for (int a = 0; a < 3; ++a) d += log(r.size[a] / sizes[a]) * log(r.size[a] / sizes[a]);
        d = sqrt(d);
        if (d <= dist) {
            dist = d;
            near = n;
        }
        if (vs[n].family != FAMILY_RF && d <= dist_fixed) {
            dist_fixed = d;
            near_fixed = n;
        }
    }
    auto named = [&](const char *name, int otherwise) {
        const int n = variant_index(kernel, g->dtype, name);
        return n >= 0 && takes_row_length(vs[n], g) ? n : otherwise;
    };
    if (kernel == KL_KERNEL_ADVEC_U_2I5 || kernel == KL_KERNEL_DIFF_SMAG) {
        if (points < (double)(1 << (g->itot < 8 ? 17 : 19))) return 0;
        if (g->itot >= 8) return named("rf_t512", 0);
        return named(kernel == KL_KERNEL_DIFF_SMAG ? "s2_v1_b64x8_k16_x0_nt0" : "a5_v1_b64x8_k16_x0_nt0", 0);
    }
    if (dist <= (bytes >= 4e8 ? 0.1 : 0.0125)) return near;
    const bool rows_fit = cpr <= rf_max_chunks(512), short_rows = cpr <= rf_max_chunks(256);
    const int flat = !rows_fit ? 0 : named(short_rows ? "rf_t256" : "rf_t512", 0);
    const int wide = named(wide_rows_tile(kernel, g->dtype, g->itot, points), flat);
    if (step) {
        if (short_rows || (rows_fit && (points < 5e6 || g->itot % V))) return flat;
        const bool idle = g->itot < 0.8 * ((cpr + 63) / 64) * 64 * V && (cpr <= 102 || (cpr <= 192 && bytes < 120e6));
        return rows_fit && 512 / cpr * cpr >= 400 && (bytes < (f32 ? 50e6 : 70e6) || idle) ? flat : wide;
    }
    if (few) return dist <= 0.3 ? near : bytes < (double)(1 << 19) ? 0 : flat;
    if (!rows_fit) return wide;
    if (kernel == KL_KERNEL_ADVEC_U && !short_rows) {
        const double from = !f32 ? 4e7 : cpr > 128 ? 2e7 : fills_waves(g->itot, V) ? 1.5e7 : 5e7;
        if (points >= 1e6 && points < (f32 ? 1.15e7 : 7.5e6)) return wide;
        if (points > from && g->itot % 2 == 0) return f32 && cpr > 128 && points >= 6e7 ? near_fixed : wide;
    }
    return flat;
}
}  // namespace

int select_variant(const kl_grid_t *g, int kernel)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    const auto key = std::make_tuple(kernel, g->dtype, g->itot, g->jtot, g->ktot, dev);
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        auto it = g_plans.find(key);
        if (it != g_plans.end()) return it->second;
    }
    int index = 0;
    DeviceIdent id;
    if (current_device_ident(&id) == KL_OK) {
        std::string name;
        int level = 5;
        bool same_size = false;
        std::vector<SizeRecord> records;
        if (wisdom_select(wisdom_dir(), kernel, g->dtype, id, g->itot, g->jtot, g->ktot, &name, &level, &same_size,
                          &records) == KL_OK &&
            level < 5)
            index = same_size ? std::max(0, variant_index(kernel, g->dtype, name)) : unrecorded_variant(g, kernel, records);
    }
    std::lock_guard<std::mutex> lk(g_plan_mu);
    g_plans[key] = index;
    return index;
}

int run_variant(const kl_grid_t *g, int kernel, int index, void *const *fields, double visc, hipStream_t s,
                double dt, bool fresh)
{
    const auto &vs = variants(kernel, g->dtype);
    if (index < 0 || index >= (int)vs.size()) return fail(KL_ERR_NOTFOUND, "variant index %d", index);
    if (kernel == KL_KERNEL_ADVEC_U_2I5 && g->gc < 3)
        return fail(KL_ERR_INVALID, "advec_u_2i5 needs gc = 3 ghost cells in x and y (grid has %d)", g->gc);
    const Variant &v = vs[index];
    const int nptr = kernel_nptr(kernel);
    if (!variant_eligible(v, g, (const void *const *)fields, nptr))
        return fail(KL_ERR_INVALID, "configuration %s not eligible for this grid/alignment", v.name);
    HostArgs a = make_args(g);
    a.dt = dt;
    a.u = fields[0];
    a.v = fields[1];
    a.w = fields[2];
    a.ut = fields[3];
    a.vt = fields[4];
    a.wt = fields[5];
    a.evisc = nptr > 6 ? fields[6] : nullptr;
    a.visc = visc;
    const hipError_t e = fresh ? v.fresh(a, s) : v.launch(a, s);
    if (e != hipSuccess) return hip_fail(e, v.name);
    return KL_OK;
}

}  // namespace kl

using namespace kl;

namespace {

int check_ptrs(const void *const *p, int n)
{
    for (int i = 0; i < n; ++i)
        if (!p[i]) return fail(KL_ERR_INVALID, "field pointer %d is NULL", i);
    return KL_OK;
}

// Launch `kernel` with the selected configuration.  When it does not fit this
// call's rows or alignment, a row-flattened configuration takes its place,
// which takes any (stencil_rf.hpp: 301x203x151 FP32 advec_u 65 us in the
// default configuration, 32 row-flattened; FP64 diff_uvw 265 and 111), and
// the default only on rows too long for one.
int launch_selected(const kl_grid_t *g, int kernel, void *const *fields, double visc, hipStream_t s,
                    double dt = 0.0, bool fresh = false)
{
    int index = select_variant(g, kernel);
    const auto &vs = variants(kernel, g->dtype);
    const void *const *ptrs = (const void *const *)fields;
    const int nptr = kernel_nptr(kernel);
    if (!variant_eligible(vs[index], g, ptrs, nptr)) {
        index = 0;
        for (size_t n = vs.size(); n-- > 0;)  // the smallest block that fits (registered smallest first)
            if (vs[n].family == FAMILY_RF && variant_eligible(vs[n], g, ptrs, nptr)) index = (int)n;
    }
    if (!variant_eligible(vs[index], g, ptrs, nptr))
        return fail(KL_ERR_INVALID, "no configuration of %s fits this grid/alignment", kernel_name(kernel));
    // a capture holds the tendencies a launch accumulates onto
    const int rc = fresh ? KL_OK : maybe_capture(g, kernel, fields, visc, dt, s);
    if (rc) return rc;
    return run_variant(g, kernel, index, fields, visc, s, dt, fresh);
}

bool kernel_ok(int32_t kernel) { return kernel >= 0 && kernel < KL_NUM_KERNELS; }

}  // namespace

extern "C" {

const char *kl_version(void) { return KL_VERSION_STRING; }

const char *kl_last_error(void) { return g_last_error.c_str(); }

int kl_layout_gc(int32_t itot, int32_t jtot, int32_t ktot, int32_t dtype, int32_t gc, int64_t *off,
                 int64_t *jstride, int64_t *kstride, int64_t *alloc_elems)
{
    clear_error();
    if (itot < 1 || jtot < 1 || ktot < 1) return fail(KL_ERR_INVALID, "sizes must be >= 1");
    if (dtype != KL_F32 && dtype != KL_F64) return fail(KL_ERR_INVALID, "dtype %d", dtype);
    if (gc != 1 && gc != 3) return fail(KL_ERR_INVALID, "gc %d must be 1 or 3", gc);
    if (!off || !jstride || !kstride || !alloc_elems) return fail(KL_ERR_INVALID, "NULL output");
    const int64_t line = 128 / (dtype == KL_F32 ? 4 : 8);  // elements per 128-byte line
    const int64_t js = ((int64_t)itot + 2 * gc + line - 1) / line * line;
    const int64_t o = (gc - 1) * js + line - 1;  // idx(1, j, k) on a line boundary
    const int64_t ks = js * ((int64_t)jtot + 2 * gc);
    *off = o;
    *jstride = js;
    *kstride = ks;
    *alloc_elems = o + ks * ((int64_t)ktot + 2) + 2 * line;
    return KL_OK;
}

int kl_layout(int32_t itot, int32_t jtot, int32_t ktot, int32_t dtype, int64_t *off, int64_t *jstride,
              int64_t *kstride, int64_t *alloc_elems)
{
    return kl_layout_gc(itot, jtot, ktot, dtype, 1, off, jstride, kstride, alloc_elems);
}

int kl_fill_ghosts(const kl_grid_t *g, void *u, void *v, void *w, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[3] = {u, v, w};
    if ((rc = check_ptrs(p, 3))) return rc;
    const hipError_t e = launch_fill_ghosts(make_args(g), u, v, w, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "fill_ghosts");
}

int kl_fill_scalar(const kl_grid_t *g, void *f, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (!f) return fail(KL_ERR_INVALID, "field pointer is NULL");
    const hipError_t e = launch_fill_scalar(make_args(g), f, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "fill_scalar");
}

int kl_advec_u_2i5(const kl_grid_t *g, void *ut, const void *u, const void *v, const void *w, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (g->gc < 3) return fail(KL_ERR_INVALID, "advec_u_2i5 needs gc = 3 ghost cells in x and y (grid has %d)", g->gc);
    const void *p[4] = {u, v, w, ut};
    if ((rc = check_ptrs(p, 4))) return rc;
    void *f[6] = {(void *)u, (void *)v, (void *)w, ut, nullptr, nullptr};
    return launch_selected(g, KL_KERNEL_ADVEC_U_2I5, f, 0.0, (hipStream_t)stream);
}

int kl_diff_smag(const kl_grid_t *g, void *ut, void *vt, void *wt, const void *u, const void *v, const void *w,
                 const void *evisc, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[7] = {u, v, w, ut, vt, wt, evisc};
    if ((rc = check_ptrs(p, 7))) return rc;
    void *f[7] = {(void *)u, (void *)v, (void *)w, ut, vt, wt, (void *)evisc};
    return launch_selected(g, KL_KERNEL_DIFF_SMAG, f, 0.0, (hipStream_t)stream);
}

int kl_advec_u(const kl_grid_t *g, void *ut, const void *u, const void *v, const void *w, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[4] = {u, v, w, ut};
    if ((rc = check_ptrs(p, 4))) return rc;
    void *f[6] = {(void *)u, (void *)v, (void *)w, ut, nullptr, nullptr};
    return launch_selected(g, KL_KERNEL_ADVEC_U, f, 0.0, (hipStream_t)stream);
}

int kl_diff_uvw(const kl_grid_t *g, void *ut, void *vt, void *wt, const void *u, const void *v, const void *w,
                double visc, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[6] = {u, v, w, ut, vt, wt};
    if ((rc = check_ptrs(p, 6))) return rc;
    void *f[6] = {(void *)u, (void *)v, (void *)w, ut, vt, wt};
    return launch_selected(g, KL_KERNEL_DIFF_UVW, f, visc, (hipStream_t)stream);
}

int kl_advec_diff(const kl_grid_t *g, void *ut, void *vt, void *wt, const void *u, const void *v, const void *w,
                  double visc, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[6] = {u, v, w, ut, vt, wt};
    if ((rc = check_ptrs(p, 6))) return rc;
    void *f[6] = {(void *)u, (void *)v, (void *)w, ut, vt, wt};
    return launch_selected(g, KL_KERNEL_ADVEC_DIFF, f, visc, (hipStream_t)stream);
}

int kl_euler(const kl_grid_t *g, double dt, void *u, void *v, void *w, const void *ut, const void *vt,
             const void *wt, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[6] = {u, v, w, ut, vt, wt};
    if ((rc = check_ptrs(p, 6))) return rc;
    HostArgs a = make_args(g);
    a.ut = (void *)ut;
    a.vt = (void *)vt;
    a.wt = (void *)wt;
    const hipError_t e = launch_euler(a, dt, u, v, w, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "euler");
}

int kl_step(const kl_grid_t *g, double visc, double dt, void *u, void *v, void *w, void *ut, void *vt, void *wt,
            void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[6] = {u, v, w, ut, vt, wt};
    if ((rc = check_ptrs(p, 6))) return rc;
    hipStream_t s = (hipStream_t)stream;
    HostArgs a = make_args(g);
    void *f[6] = {u, v, w, ut, vt, wt};
    if (capture_pending(g, KL_KERNEL_ADVEC_U) || capture_pending(g, KL_KERNEL_DIFF_UVW)) {
        // the step's two tendency kernels are to be captured: launch them
        for (void *t : {ut, vt, wt}) {
            const hipError_t e = launch_zero_interior(a, t, s);
            if (e != hipSuccess) return hip_fail(e, "zero tendencies");
        }
        if ((rc = launch_selected(g, KL_KERNEL_ADVEC_U, f, visc, s))) return rc;
        if ((rc = launch_selected(g, KL_KERNEL_DIFF_UVW, f, visc, s))) return rc;
    } else {
        // one pass for the zeroing and both kernels, bitwise theirs: 6 values
        // per point moved instead of 17
        if ((rc = launch_selected(g, KL_KERNEL_ADVEC_DIFF, f, visc, s, 0.0, true))) return rc;
    }
    a.ut = ut;
    a.vt = vt;
    a.wt = wt;
    const hipError_t e = launch_euler(a, dt, u, v, w, s);
    return e == hipSuccess ? KL_OK : hip_fail(e, "euler");
}

int kl_step_fused(const kl_grid_t *g, double visc, double dt, const void *u, const void *v, const void *w,
                  void *u_out, void *v_out, void *w_out, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[6] = {u, v, w, u_out, v_out, w_out};
    if ((rc = check_ptrs(p, 6))) return rc;
    for (int a = 0; a < 3; ++a)
        for (int b = 3; b < 6; ++b)
            if (p[a] == p[b]) return fail(KL_ERR_INVALID, "fused step: input %d and output %d overlap", a, b - 3);
    void *f[6] = {(void *)u, (void *)v, (void *)w, u_out, v_out, w_out};
    if ((rc = launch_selected(g, KL_KERNEL_STEP, f, visc, (hipStream_t)stream, dt))) return rc;
    if (g->gc != 1) {  // the kernel writes one ghost layer; refill wider halos whole
        const hipError_t e = launch_fill_ghosts(make_args(g), u_out, v_out, w_out, (hipStream_t)stream);
        if (e != hipSuccess) return hip_fail(e, "fill_ghosts");
    }
    return KL_OK;
}

int kl_reduce_fp64(const kl_grid_t *g, int32_t what, const void *f0, const void *f1, const void *f2, double *out,
                   void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (what != 0 && what != 1) return fail(KL_ERR_INVALID, "what=%d", what);
    if (!out) return fail(KL_ERR_INVALID, "out is NULL");
    if (what == 0) {
        const void *p[3] = {f0, f1, f2};
        if ((rc = check_ptrs(p, 3))) return rc;
    }
    void *ws = workspace(reduce_scratch_bytes(), (hipStream_t)stream);
    if (!ws) return fail(KL_ERR_NOMEM, "reduction workspace");
    const hipError_t e = launch_reduce(make_args(g), what, f0, f1, f2, out, ws, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "reduce");
}

int kl_generate_fields(const kl_grid_t *g, uint64_t seed, void *u, void *v, void *w, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const void *p[3] = {u, v, w};
    if ((rc = check_ptrs(p, 3))) return rc;
    const hipError_t e = launch_gen_uniform(make_args(g), seed, u, v, w, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "generate_fields");
}

int kl_hash_interior(const kl_grid_t *g, const void *f, uint64_t *out, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (!f || !out) return fail(KL_ERR_INVALID, "NULL pointer");
    void *ws = workspace(reduce_scratch_bytes(), (hipStream_t)stream);
    if (!ws) return fail(KL_ERR_NOMEM, "hash workspace");
    const hipError_t e = launch_hash(make_args(g), f, out, ws, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "hash");
}

int kl_num_variants(int32_t kernel, int32_t dtype)
{
    clear_error();
    if (!kernel_ok(kernel) || (dtype != KL_F32 && dtype != KL_F64))
        return fail(KL_ERR_INVALID, "kernel %d / dtype %d", kernel, dtype);
    return (int)variants(kernel, dtype).size();
}

int kl_variant_name(int32_t kernel, int32_t dtype, int32_t index, char *buf, size_t len)
{
    const int n = kl_num_variants(kernel, dtype);
    if (n < 0) return n;
    if (index < 0 || index >= n) return fail(KL_ERR_NOTFOUND, "variant index %d", index);
    if (!buf || len == 0) return fail(KL_ERR_INVALID, "NULL buffer");
    snprintf(buf, len, "%s", variants(kernel, dtype)[index].name);
    return KL_OK;
}

int kl_variant_eligible(const kl_grid_t *g, int32_t kernel, int32_t index, const void *const fields[6])
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    const int n = kl_num_variants(kernel, g->dtype);
    if (n < 0) return n;
    if (index < 0 || index >= n) return fail(KL_ERR_NOTFOUND, "variant index %d", index);
    return variant_eligible(variants(kernel, g->dtype)[index], g, fields, fields ? kernel_nptr(kernel) : 0) ? 1 : 0;
}

int kl_launch_variant_dt(const kl_grid_t *g, int32_t kernel, int32_t index, void *const fields[6], double visc,
                         double dt, void *stream)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (!kernel_ok(kernel)) return fail(KL_ERR_INVALID, "kernel %d", kernel);
    if (!fields) return fail(KL_ERR_INVALID, "fields is NULL");
    if ((rc = check_ptrs((const void *const *)fields, kernel_nptr(kernel)))) return rc;
    return run_variant(g, kernel, index, fields, visc, (hipStream_t)stream, dt);
}

int kl_launch_variant(const kl_grid_t *g, int32_t kernel, int32_t index, void *const fields[6], double visc,
                      void *stream)
{
    return kl_launch_variant_dt(g, kernel, index, fields, visc, 0.0, stream);
}

int kl_selected_variant(const kl_grid_t *g, int32_t kernel)
{
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (!kernel_ok(kernel)) return fail(KL_ERR_INVALID, "kernel %d", kernel);
    return select_variant(g, kernel);
}

int kl_clear_plan_cache(void)
{
    clear_plans();
    return KL_OK;
}

}  // extern "C"
