// Row-flattened z-marching tiles of the second-order kernels, for rows of any
// length at any alignment.
//
// The other z-march tiles give a wave one row segment of 64 VX points, which
// leaves most lanes idle on rows that do not fill it (32 of 256 points, or
// 45 of 256 in the second segment of a 301-point row) and needs 16-byte
// aligned rows.  Here a block owns R whole rows (its rows times their chunks
// fill the block), a row is cpr chunks of V points, and thread t takes chunk
// t % cpr of row t / cpr, so a wave may hold several rows or parts of two.
// Loads and stores are 16 bytes wide at element alignment; the last chunk of a
// row may be partial (its loads run into the row's ghost cells and at most
// V - 2 elements further, its stores are per point).
//
// Per level, as in the other tiles: z neighbours from a 4-slot register ring
// (level k+3 requested at level k), x and y neighbours from LDS, one barrier.
// A whole row is in LDS, so the periodic x neighbours are there too and no x
// edge is loaded.  u and v have two planes;
// w has three and is staged one level ahead, because advec_u needs its left
// neighbour at level k+1.  The two halo rows are loaded by the first 2 cpr
// threads (u, v one level ahead, w two); the other threads' halo load is one
// address for all and lands in a spare slot, so that every load is issued and
// consumed on every path and the compiler's waits stay exact.
//
// Bound by HBM from about 10^7 points (301x203x151 FP32, 517 MB for the pair:
// 5.9 TB/s), below that by latency: blocks of 256 threads at up to 222 VGPRs
// and 52 KB of LDS, two or three per CU.  Measured against the fastest of the
// other tiles (us): advec_u 301x203x151 FP32 65 -> 32, FP64 133 -> 66;
// diff_uvw 320x320x160 FP32 151 -> 94, 301x203x151 FP64 268 -> 113; fused pass
// 128^3 FP64 32 -> 29; fused step, two buffers in turn, 128^3 FP32 23 -> 17, 256^3
// 102 -> 99.  Rows of more than 256 chunks are left to the other tiles, which split
// them in x, and some shorter ones (unrecorded_variant in api.cpp).
//
// The per-point functions are those of stencil.hpp: results are bitwise those
// of every other configuration.
#pragma once

#include "stencil_step.hpp"

namespace kl {

enum { RF_ADVEC = 1, RF_DIFF = 2, RF_FRESH = 4, RF_STEP = 8 };

// Store the first `n` of a chunk's V values.
template <int NT, typename T, int V>
__device__ __forceinline__ void rf_store(T *p, const T (&x)[V], int n)
{
    if (n == V) {
        if constexpr (NT)
            ustore_nt<T, V>(p, x);
        else
            ustore<T, V>(p, x);
    } else {
#pragma unroll
        for (int m = 0; m < V - 1; ++m)
            if (m < n) p[m] = x[m];
    }
}

// The n-th of a chunk's values (n in [1, V]).  Nested comparisons of scalars:
// a chain of equalities over the array is turned into an indexed access,
// which puts the array into scratch memory.
template <typename T, int V>
__device__ __forceinline__ T rf_nth(const T (&x)[V], int n)
{
    if constexpr (V == 4) {
        const T x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
        const T lo = n > 1 ? x1 : x0, hi = n > 3 ? x3 : x2;
        return n > 2 ? hi : lo;
    } else {
        static_assert(V == 2, "chunks of 16 bytes");
        const T x0 = x[0], x1 = x[1];
        return n > 1 ? x1 : x0;
    }
}

// The z ghost cells whose source is a chunk of new values (n points at
// (i0.., j, k) of field `fld`), with their x and y images; first and last
// levels only.
template <typename T, int V>
__device__ __forceinline__ void rf_z_images(T *f, const StencilArgs<T> &a, int fld, int i0, int j, int k, int n,
                                            const T (&val)[V])
{
    auto put = [&](int jj, int kk, int sign) __attribute__((always_inline)) {
        T *row = f + a.off + (int64_t)jj * a.js + (int64_t)kk * a.ks;
        T x[V];
#pragma unroll
        for (int m = 0; m < V; ++m) x[m] = sign == 0 ? T(0) : (sign < 0 ? -val[m] : val[m]);
        rf_store<0, T, V>(row + i0, x, n);
        if (i0 == 1) row[a.itot + 1] = x[0];
        if (i0 + V > a.itot) row[0] = rf_nth<T, V>(x, n);
    };
    const int kt = a.ktot;
    // z images (level, sign), at most two besides w's level 0; level k: none
    int z1 = k, s1 = 1, z2 = k, s2 = 1;
    if (a.bc == KL_BC_ZPERIODIC) {
        if (k == kt) z1 = 0;
        if (k == 1) z2 = kt + 1;
    } else if (fld < 2) {
        if (k == 1) z1 = 0;
        if (k == kt) z2 = kt + 1;
    } else {
        const int sw = a.bc == KL_BC_ZWALL_ZEROGRAD ? 1 : 0;  // w's wall faces
        if (k == 2) { z1 = 1; s1 = sw; }
        if (k == kt) { z2 = kt + 1; s2 = sw; }
    }
    const bool z0 = a.bc != KL_BC_ZPERIODIC && fld == 2 && k == 2;
    const int s0 = a.bc == KL_BC_ZWALL_ZEROGRAD ? 1 : -1;
    for (int y = 0; y < 3; ++y) {
        if ((y == 1 && j != 1) || (y == 2 && j != a.jtot)) continue;
        const int jj = y == 0 ? j : (y == 1 ? a.jtot + 1 : 0);
        if (z1 != k) put(jj, z1, s1);
        if (z2 != k) put(jj, z2, s2);
        if (z0) put(jj, 0, s0);
    }
}

// Row block ty (a.rf_rows rows of a.rf_cpr chunks), level slab tz (a.rf_kb levels).
// XF (batched pass): with a.x_fill the x ghost columns of the inputs are
// written too, from the row ends in registers.  In rows of whole chunks no tile
// uses a ghost column (row ends are their own x neighbours), so they need not
// be there before, and a fill that leaves them out skips three lines per row
// and field, two of them read (a partial last chunk has the ghost column as
// its last point's neighbour: such grids are filled before).  56 grids FP32,
// fill, pass and sums: 689 -> 619 us.
template <typename T, int V, int MODE, int NT, bool XF = false>
__device__ __forceinline__ void rf_tile(const StencilArgs<T> &a, int ty, int tz, T *lds)
{
    constexpr bool ADV = (MODE & RF_ADVEC) != 0, DIF = (MODE & RF_DIFF) != 0;
    constexpr bool STEP = (MODE & RF_STEP) != 0, ACC = !STEP && (MODE & RF_FRESH) == 0;
    constexpr int NTD = DIF ? 3 : 1;  // tendencies (or new fields) of a point
    __syncthreads();                  // a block may run tiles back to back
    const int cpr = a.rf_cpr, R = a.rf_rows;
    const int t = (int)threadIdx.x;
    const int j0 = 1 + ty * R;
    const int nv = min(R, a.jtot - j0 + 1);
    const int k0 = 1 + tz * a.rf_kb, k1 = min(k0 + a.rf_kb, a.ktot + 1);
    const int row_t = t / cpr, c = t - row_t * cpr;
    const bool own = row_t < nv;
    const int row = min(row_t, nv - 1);  // threads without a row repeat one of the last
    const int i0 = 1 + c * V;
    const int n_own = own ? min(V, a.itot - c * V) : 0;  // points stored
    const int64_t ks = a.ks;
    const int js = (int)a.js;

    // 32-bit offsets from the uniform base (column 0 of row j0 - 1)
    const int64_t base = a.off + (int64_t)(j0 - 1) * a.js;
    const int o_own = (row + 1) * js + i0;
    const int side = t >= cpr;
    const bool halo = t < 2 * cpr;
    const int hc = t - side * cpr;
    const int o_x = halo ? (side ? (nv + 1) * js : 0) + 1 + hc * V : 1;
    auto at = [&](T *f, int l, int o) { return boff(f + base + (int64_t)l * ks, (uint32_t)o * (uint32_t)sizeof(T)); };
    auto cat = [&](const T *f, int l, int o) {
        return boff(f + base + (int64_t)l * ks, (uint32_t)o * (uint32_t)sizeof(T));
    };

    // LDS: element offsets inside a plane; the x neighbours of the row's ends
    // are the row's other end
    const int S = V * cpr, spare = (R + 2) * S, PS = spare + 64 * V;
    const int l_row = (row + 1) * S, l_own = l_row + c * V;
    const int l_x = halo ? (side ? (nv + 1) * S : 0) + hc * V : spare + (t & 63) * V;
    const int l_left = l_row + (c == 0 ? a.itot : c * V) - 1;
    const int l_right = l_row + (c == cpr - 1 ? 0 : (c + 1) * V);
    T *pu[2] = {lds, lds + PS}, *pv[2] = {lds + 2 * PS, lds + 3 * PS};
    T *pw0 = lds + 4 * PS, *pw1 = lds + 5 * PS, *pw2 = lds + 6 * PS;  // w: levels k, k+1, next

    const T *F[3] = {a.u, a.v, a.w};
    T *O[3] = {a.ut, a.vt, a.wt};
    const T dxi = a.dxi, dyi = a.dyi, dxi2 = a.dxi * a.dxi, dyi2 = a.dyi * a.dyi, visc = a.visc, dt = a.dt;
    const int kw0 = a.kw0, kt = a.ktot;

    T Rg[4][3][V];              // field ring: slot s % 4 holds level kk + s
    T X[2][3][V];               // halo chunk by level parity
    T Q[ACC ? 2 : 1][NTD][V];   // tendencies by level parity
    // halo rows are never used at level ktot + 1: clamped to ktot, so that the
    // wide loads of the last ghost row stay inside the field
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        uload<T, V>(Rg[3][f], cat(F[f], k0 - 1, o_own));
        uload<T, V>(Rg[0][f], cat(F[f], k0, o_own));
        uload<T, V>(Rg[1][f], cat(F[f], k0 + 1, o_own));
        uload<T, V>(Rg[2][f], cat(F[f], min(k0 + 2, k1), o_own));
        uload<T, V>(X[0][f], cat(F[f], k0, o_x));
    }
    if constexpr (DIF) uload<T, V>(X[1][2], cat(F[2], min(k0 + 1, kt), o_x));
#pragma unroll
    for (int f = 0; f < NTD; ++f)
        if constexpr (ACC) {
            if constexpr (NT)
                uload_nt<T, V>(Q[0][f], cat(O[f], k0, o_own));
            else
                uload<T, V>(Q[0][f], cat(O[f], k0, o_own));
        }
    // w of level k0
    vstore<T, V>(pw0 + l_own, Rg[0][2]);
    if constexpr (DIF) vstore<T, V>(pw0 + l_x, X[0][2]);
    vm_drain();

    for (int kk = k0;; kk += 4) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = kk + s;
            if (k >= k1) return;
            const int p = s & 1, q = p ^ 1;
            T(&b)[3][V] = Rg[(s + 3) & 3];
            T(&cc)[3][V] = Rg[s & 3];
            T(&tp)[3][V] = Rg[(s + 1) & 3];
            // halo chunks of u, v at level k+1 and w at level k+2, tendencies of level k+1
            uload<T, V>(X[q][0], cat(F[0], min(k + 1, kt), o_x));
            uload<T, V>(X[q][1], cat(F[1], min(k + 1, kt), o_x));
            // rows of level k (u, v) and k+1 (w) into LDS
            vstore<T, V>(pu[p] + l_own, cc[0]);
            vstore<T, V>(pu[p] + l_x, X[p][0]);
            vstore<T, V>(pv[p] + l_own, cc[1]);
            vstore<T, V>(pv[p] + l_x, X[p][1]);
            vstore<T, V>(pw1 + l_own, tp[2]);
            if constexpr (DIF) {
                vstore<T, V>(pw1 + l_x, X[q][2]);
                uload<T, V>(X[p][2], cat(F[2], min(k + 2, kt), o_x));
            }
            if constexpr (ACC) {
#pragma unroll
                for (int f = 0; f < NTD; ++f) {
                    if constexpr (NT)
                        uload_nt<T, V>(Q[q][f], cat(O[f], k + 1, o_own));
                    else
                        uload<T, V>(Q[q][f], cat(O[f], k + 1, o_own));
                }
            }
            __syncthreads();
            T un[V], us[V], vn[V];
            vload<T, V>(un, pu[p] + l_own + S);
            vload<T, V>(us, pu[p] + l_own - S);
            vload<T, V>(vn, pv[p] + l_own + S);
            const T ul = pu[p][l_left], ur = pu[p][l_right];
            const T vl = pv[p][l_left], wl = pw0[l_left];
            T vnl = T(0), wtl = T(0);
            if constexpr (ADV) {
                vnl = pv[p][l_left + S];
                wtl = pw1[l_left];
            }
            T vs[V], wn[V], ws[V], vr = T(0), wr = T(0);
            if constexpr (DIF) {
                vload<T, V>(vs, pv[p] + l_own - S);
                vload<T, V>(wn, pw0 + l_own + S);
                vload<T, V>(ws, pw0 + l_own - S);
                vr = pv[p][l_right];
                wr = pw0[l_right];
            }
            const T dzik = kload(a.dzi, k), dzikm1 = kload(a.dzi, k - 1), dzhik = kload(a.dzhi, k),
                    dzhik1 = kload(a.dzhi, k + 1);
            T res[NTD][V];
#pragma unroll
            for (int n = 0; n < V; ++n) {
                const T uw = n == 0 ? ul : cc[0][n - 1], ue = n == V - 1 ? ur : cc[0][n + 1];
                const T v_w = n == 0 ? vl : cc[1][n - 1], w_w = n == 0 ? wl : cc[2][n - 1];
                T tu = ACC ? Q[p][0][n] : T(0);
                if constexpr (ADV) {
                    const T v_nw = n == 0 ? vnl : vn[n - 1], w_tw = n == 0 ? wtl : tp[2][n - 1];
                    tu = tu + advec_u_point<T>(cc[0][n], ue, uw, un[n], us[n], tp[0][n], b[0][n], v_w, cc[1][n], v_nw,
                                               vn[n], w_w, cc[2][n], w_tw, tp[2][n], dxi, dyi, dzik);
                }
                if constexpr (DIF) {
                    const T v_e = n == V - 1 ? vr : cc[1][n + 1], w_e = n == V - 1 ? wr : cc[2][n + 1];
                    tu = tu + diff_c_point<T>(cc[0][n], ue, uw, un[n], us[n], tp[0][n], b[0][n], dxi2, dyi2, dzik,
                                              dzhik1, dzhik, visc);
                    const T tv = (ACC ? Q[p][1 % NTD][n] : T(0)) + diff_c_point<T>(cc[1][n], v_e, v_w, vn[n], vs[n], tp[1][n],
                                                                             b[1][n], dxi2, dyi2, dzik, dzhik1, dzhik, visc);
                    // w below its first level: formed, not accumulated (zero where it starts at zero)
                    const T dw = diff_w_point<T>(cc[2][n], w_e, w_w, wn[n], ws[n], tp[2][n], b[2][n], dxi2, dyi2,
                                                 dzik, dzikm1, dzhik, visc);
                    const T tw = ACC ? Q[p][2 % NTD][n] + dw : (STEP || k >= kw0 ? T(0) + dw : T(0));
                    res[1 % NTD][n] = STEP ? euler_value<T>(cc[1][n], dt, tv) : tv;
                    res[2 % NTD][n] = STEP ? euler_value<T>(cc[2][n], dt, tw) : tw;
                }
                res[0][n] = STEP ? euler_value<T>(cc[0][n], dt, tu) : tu;
            }
            if constexpr (ACC) {
#pragma unroll
                for (int f = 0; f < NTD; ++f) settle(Q[p][f]);
            }
            if constexpr (XF) {
                if (a.x_fill && own) {
#pragma unroll
                    for (int f = 0; f < 3; ++f) {
                        T *level = const_cast<T *>(F[f]) + base + (int64_t)k * ks;
                        if (c == 0) *boff(level, (uint32_t)(o_own + a.itot) * (uint32_t)sizeof(T)) = cc[f][0];
                        if (c == cpr - 1)
                            *boff(level, (uint32_t)(o_own - i0) * (uint32_t)sizeof(T)) = rf_nth<T, V>(cc[f], n_own);
                    }
                }
            }
            if (own) {
                if constexpr (STEP) {
                    // the point, its x images, and the same on the y image's
                    // row: edge blocks then cost a few stores more, where a
                    // general image path made them the launch's last to end
                    const int j = j0 + row;
                    auto put = [&](T *f, int o, const T(&x)[V]) __attribute__((always_inline)) {
                        T *row0 = f + a.off + (int64_t)k * ks;
                        rf_store<NT, T, V>(boff(row0, (uint32_t)o * (uint32_t)sizeof(T)), x, n_own);
                        if (c == 0) *boff(row0, (uint32_t)(o + a.itot) * (uint32_t)sizeof(T)) = x[0];
                        if (c == cpr - 1)
                            *boff(row0, (uint32_t)(o - i0) * (uint32_t)sizeof(T)) = rf_nth<T, V>(x, n_own);
                    };
#pragma unroll
                    for (int f = 0; f < 3; ++f) {
                        if (f == 2 && k < kw0) continue;
                        put(O[f], j * js + i0, res[f % NTD]);
                        if (j == 1) put(O[f], (a.jtot + 1) * js + i0, res[f % NTD]);
                        if (j == a.jtot) put(O[f], i0, res[f % NTD]);
                    }
                    if (k <= 2 || k == kt) {
#pragma unroll
                        for (int f = 0; f < 3; ++f)
                            if (f < 2 || k >= kw0) rf_z_images<T, V>(O[f], a, f, i0, j, k, n_own, res[f % NTD]);
                    }
                } else {
#pragma unroll
                    for (int f = 0; f < NTD; ++f)
                        if (!ACC || f < 2 || k >= kw0) rf_store<NT, T, V>(at(O[f], k, o_own), res[f], n_own);
                }
            }
            const int l3 = min(k + 3, k1);
#pragma unroll
            for (int f = 0; f < 3; ++f) uload<T, V>(b[f], cat(F[f], l3, o_own));
            T *x = pw0;
            pw0 = pw1;
            pw1 = pw2;
            pw2 = x;
        }
    }
}

// One block per tile.  Tiles y fastest, then z; each XCD takes a contiguous
// part of every a.nbx consecutive tiles (a slab of levels when its row blocks
// divide by the 8 XCDs, else the whole list), so neighbouring row blocks
// share their halo rows in one L2.
template <typename T, int V, int MODE, int NT, int THREADS>
__global__ __launch_bounds__(THREADS, 2) void rf_kernel(StencilArgs<T> a)
{
    extern __shared__ __align__(16) unsigned char rf_lds[];
    const unsigned L = (unsigned)a.nbx, s = blockIdx.x / L;
    const unsigned b = s * L + xcd_remap(blockIdx.x - s * L, L);
    const unsigned tz = b / (unsigned)a.nby;
    rf_tile<T, V, MODE, NT>(a, (int)(b - tz * (unsigned)a.nby), (int)tz, reinterpret_cast<T *>(rf_lds));
}

// Persistent form: tile = (grid, -, ty, tz).  A block's first tile takes no ticket,
// which on small grids is a good part of the walk (64 grids of 16^3 FP32 24 -> 20
// us) and puts the tiles where the list says (spread_tiles).  The z-march tiles draw
// it: their lists keep neighbours together, and blocks do not start in order (256^3
// FP32 fused pass drawn 109, not drawn 117).
template <typename T, int V, int MODE, int NT, int THREADS>
__global__ __launch_bounds__(THREADS, 2) void rf_batch(const StencilArgs<T> *__restrict__ grids,
                                                       const int4 *__restrict__ tiles, int ntiles, int *queue)
{
    extern __shared__ __align__(16) unsigned char rf_lds[];
    for (int n = next_tile<true>(queue, -1); n < ntiles; n = next_tile<true>(queue, n)) {
        const int4 tl = tiles[n];
        const StencilArgs<T> a = global_args(grids[tl.x]);
        rf_tile<T, V, MODE, NT, (MODE & RF_STEP) == 0>(a, tl.z, tl.w, reinterpret_cast<T *>(rf_lds));
    }
    walk_done(queue);
}

}  // namespace kl
