// Row-flattened z-marching tiles of the paper's schemes (advec_u_2i5,
// diff_smag), for rows of any length at any alignment.
//
// As in stencil_rf.hpp a block owns R rows of W chunks of V points (16 bytes,
// loads and stores at element alignment) and thread t takes chunk t % W of row
// t / W; here the rows may be cut into segments of equal width, because the
// halos in y (six rows of u for the fifth-order faces, two rows of four
// fields for the stress) ask for tall blocks.  Everything around the block's
// own chunks - halo rows, the chunks beyond the segment's ends - is a list of
// chunks, one per thread: each thread loads one and writes it to LDS.  At the
// ends of a row those chunks are the row's own other end (x is periodic), so
// no x ghost line is fetched.  A partial last chunk loads the row's ghost
// cells in its place; its stores are per point.
//
// LDS holds rows of 16-byte chunks, so a thread reads its neighbours' chunks
// whole: nine 16-byte reads and three scalars per level for advec_u_2i5 at
// V = 4, where the wave-per-row tiles (stencil_les_zl.hpp) read about 40
// scalars; twelve and thirteen for diff_smag, against about 130.
//
// Bound by memory traffic at 256^3 and up, by the load-to-barrier chain of a
// level below.  us before (fastest other configuration that takes the grid)
// and with these tiles: advec_u_2i5 512^3 FP32 545 -> 470 (5 values a point moved:
// 5.7 TB/s), 256^3 FP32 70 -> 57, FP64 131 -> 118,
// 301x203x151 FP32 unpadded 91 -> 39, 128^3 FP32 19 -> 12; diff_smag 512^3 FP32
// 993 -> 913 (10 values a point: 5.9 TB/s), FP64 1902 -> 1873, 301x203x151 FP32
// unpadded 250 -> 75, 128^3 FP32 33 -> 19.
//
// The per-face functions are those of stencil_les.hpp: results are bitwise
// those of every other configuration.
#pragma once

#include "stencil_les.hpp"
#include "stencil_rf.hpp"

namespace kl {

// Segment sx, row block ty of a block's tile.
template <int V>
struct LesRfTile {
    int W, R, i0w, Wl, j0, nv, k0, k1;  // chunks and rows per block, first column, chunks and rows here, levels
    int row, c, i0, n_own;              // the thread's row and chunk (clamped), first column, points it stores
    bool last;                          // the segment ends the row

    template <typename T>
    __device__ __forceinline__ LesRfTile(const StencilArgs<T> &a, int sx, int ty, int tz)
    {
        W = a.rf_cpr;
        R = a.rf_rows;
        const int t = (int)threadIdx.x;
        i0w = 1 + sx * W * V;
        const int width = min(W * V, a.itot - i0w + 1);
        Wl = (width + V - 1) / V;
        last = i0w + width > a.itot;
        j0 = 1 + ty * R;
        nv = min(R, a.jtot - j0 + 1);
        k0 = 1 + tz * a.rf_kb;
        k1 = min(k0 + a.rf_kb, a.ktot + 1);
        const int row_t = t / W, c_t = t - row_t * W;
        row = min(row_t, nv - 1);
        c = min(c_t, Wl - 1);
        i0 = i0w + c * V;
        n_own = row_t < nv && c_t < Wl ? min(V, a.itot - i0 + 1) : 0;
    }
    // First column of the n columns left of the segment, and of those right of
    // its last chunk: the row's other end where the segment ends the row.
    __device__ __forceinline__ int left_of(int itot, int n) const { return (i0w == 1 ? itot + 1 : i0w) - n; }
    __device__ __forceinline__ int right_of(int itot) const { return i0w + Wl * V - (last ? itot : 0); }
};

// Tile order as rf_kernel's: x fastest, then y, then z.
template <typename T>
__device__ __forceinline__ void les_rf_tile_of(const StencilArgs<T> &a, int &sx, int &ty, int &tz)
{
    const unsigned S = (unsigned)(a.nbx * a.nby), L = (S & 7u) == 0 ? S : S * (unsigned)a.nbz;
    const unsigned s = blockIdx.x / L;
    const unsigned b = s * L + xcd_remap(blockIdx.x - s * L, L);
    const unsigned r = b / (unsigned)a.nbx;
    sx = (int)(b - r * (unsigned)a.nbx);
    tz = (int)(r / (unsigned)a.nby);
    ty = (int)(r - (unsigned)tz * (unsigned)a.nby);
}

// ---------------------------------------------------------------------------
// advec_u_2i5.  LDS per level parity: u rows j0-3 .. j0+nv+2 with 4 columns on
// each side, v rows j0 .. j0+nv and w rows j0 .. j0+nv-1 (level k+1) with a
// chunk on the left, a spare chunk per lane.
// ---------------------------------------------------------------------------
template <typename T, int V, int NT>
__global__ __launch_bounds__(512, 2) void advec_u_2i5_rf(StencilArgs<T> a)
{
    constexpr int HC = 4 / V;  // chunks of the 4 halo columns
    extern __shared__ __align__(16) unsigned char les_lds[];
    int sx, ty, tz;
    les_rf_tile_of(a, sx, ty, tz);
    const LesRfTile<V> g(a, sx, ty, tz);
    const int W = g.W, R = g.R, nv = g.nv, k0 = g.k0, k1 = g.k1, kt = a.ktot;
    const int SU = W * V + 8, SV = (W + 1) * V;
    const int oV = (R + 6) * SU, oW = oV + (R + 1) * SV, oS = oW + R * SV, PB = oS + 64 * V;
    T *lds = reinterpret_cast<T *>(les_lds);
    const int t = (int)threadIdx.x, lane = t & 63;
    const int64_t ks = a.ks;
    const int js = (int)a.js;

    // own chunk: 32-bit offset from the uniform base (column 0 of row j0)
    const int64_t base = a.off + (int64_t)g.j0 * a.js;
    const uint32_t o_own = (uint32_t)(g.row * js + g.i0) * (uint32_t)sizeof(T);
    const T *u = a.u + base, *v = a.v + base, *w = a.w + base;
    T *ut = a.ut + base;
    const int lu = (g.row + 3) * SU + 4 + g.c * V, lv = oV + g.row * SV + V + g.c * V, lw = lv + (oW - oV);

    // the thread's extra chunk
    const T *xp = u + 1;          // level 0 of its source
    int lx = oS + lane * V;       // where it goes
    {
        int e = t;
        const int n_row = 6 * W, n_edge = 2 * HC * (R + 6);
        if (e < n_row) {  // u halo rows
            const int h = e / W, c = e - h * W, rho = h < 3 ? h : nv + h;
            if (c < g.Wl) {
                xp = u + (int64_t)(rho - 3) * js + g.i0w + c * V;
                lx = rho * SU + 4 + c * V;
            }
        } else if ((e -= n_row) < n_edge) {  // u beyond the segment's ends
            const int rho = e / (2 * HC), s = e - rho * 2 * HC;
            if (rho < nv + 6) {
                xp = u + (int64_t)(rho - 3) * js +
                     (s < HC ? g.left_of(a.itot, 4) + s * V : g.right_of(a.itot) + (s - HC) * V);
                lx = rho * SU + (s < HC ? s * V : 4 + g.Wl * V + (s - HC) * V);
            }
        } else if ((e -= n_edge) < W) {  // v's north row
            if (e < g.Wl) {
                xp = v + (int64_t)nv * js + g.i0w + e * V;
                lx = oV + nv * SV + V + e * V;
            }
        } else if ((e -= W) < R + 1) {  // v left of the segment
            if (e <= nv) {
                xp = v + (int64_t)e * js + g.left_of(a.itot, V);
                lx = oV + e * SV;
            }
        } else if ((e -= R + 1) < nv) {  // w left of the segment, a level up
            xp = w + (int64_t)e * js + g.left_of(a.itot, V) + ks;
            lx = oW + e * SV;
        }
    }

    auto at = [&](const T *f, int l) __attribute__((always_inline)) { return boff(f + (int64_t)l * ks, o_own); };
    T S[6][V];       // u(k-2) .. u(k+3) of the own chunk
    T UN[2][V];      // window tops in flight
    T X[2][V];       // extra chunk
    T VO[2][V], WR[2][V], UT[2][V], FB[V];
#pragma unroll
    for (int m = 0; m < 6; ++m) uload<T, V>(S[m], at(u, min(max(k0 - 2 + m, 0), kt + 1)));
    {
        T ub3[V], w0[V];
        uload<T, V>(ub3, at(u, max(k0 - 3, 0)));
        uload<T, V>(w0, at(w, k0));
        const T wl = w[(int64_t)k0 * ks + (int64_t)g.row * js + (g.i0 == 1 ? a.itot : g.i0 - 1)];
#pragma unroll
        for (int n = 0; n < V; ++n)
            FB[n] = flux_z_2i5(mid(n == 0 ? wl : w0[n - 1], w0[n]), ub3[n], S[0][n], S[1][n], S[2][n], S[3][n], S[4][n],
                               k0, kt);
    }
    auto load = [&](int q, int k) __attribute__((always_inline)) {  // level k's operands besides the window
        uload<T, V>(X[q], xp + (int64_t)k * ks);
        uload<T, V>(VO[q], at(v, k));
        uload<T, V>(WR[q], at(w, k + 1));
        if constexpr (NT)
            uload_nt<T, V>(UT[q], at(ut, k));
        else
            uload<T, V>(UT[q], at(ut, k));
    };
    load(0, k0);
    uload<T, V>(UN[1], at(u, min(k0 + 4, kt + 1)));
    const T dxi = a.dxi, dyi = a.dyi;
    vm_drain();

    for (int kk = k0;; kk += 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = kk + p, q = p ^ 1;
            if (k >= k1) return;
            load(q, min(k + 1, k1 - 1));
            uload<T, V>(UN[p], at(u, min(k + 5, kt + 1)));
            T *pl = lds + p * PB;
            vstore<T, V>(pl + lu, S[2]);
            vstore<T, V>(pl + lv, VO[p]);
            vstore<T, V>(pl + lw, WR[p]);
            vstore<T, V>(pl + lx, X[p]);
            __syncthreads();
            T FX[V + 1];
            {
                T ux[V + 8];  // columns -4 .. V+3 from the chunk's first
#pragma unroll
                for (int h = 0; h < HC; ++h) {
                    T c4[V];
                    vload<T, V>(c4, pl + lu - 4 + h * V);
#pragma unroll
                    for (int n = 0; n < V; ++n) ux[h * V + n] = c4[n];
                    vload<T, V>(c4, pl + lu + V + h * V);
#pragma unroll
                    for (int n = 0; n < V; ++n) ux[4 + V + h * V + n] = c4[n];
                }
#pragma unroll
                for (int n = 0; n < V; ++n) ux[4 + n] = S[2][n];
#pragma unroll
                for (int f = 0; f <= V; ++f)
                    FX[f] = flux5(mid(ux[f + 3], ux[f + 4]), ux[f + 1], ux[f + 2], ux[f + 3], ux[f + 4], ux[f + 5], ux[f + 6]);
            }
            T y[6][V], vn[V];  // u rows -3, -2, -1, +1, +2, +3; v's north row
#pragma unroll
            for (int m = 0; m < 6; ++m) vload<T, V>(y[m], pl + lu + (m < 3 ? m - 3 : m - 2) * SU);
            vload<T, V>(vn, pl + lv + SV);
            const T vnl = pl[lv + SV - 1], vl = pl[lv - 1], wl = pl[lw - 1];
            const T dzik = kload(a.dzi, k);
            T res[V];
#pragma unroll
            for (int n = 0; n < V; ++n) {
                const T vnf = mid(n == 0 ? vnl : vn[n - 1], vn[n]), vsf = mid(n == 0 ? vl : VO[p][n - 1], VO[p][n]);
                const T fn = flux5(vnf, y[1][n], y[2][n], S[2][n], y[3][n], y[4][n], y[5][n]);
                const T fs = flux5(vsf, y[0][n], y[1][n], y[2][n], S[2][n], y[3][n], y[4][n]);
                const T ft = flux_z_2i5(mid(n == 0 ? wl : WR[p][n - 1], WR[p][n]), S[0][n], S[1][n], S[2][n], S[3][n],
                                        S[4][n], S[5][n], k + 1, kt);
                res[n] = UT[p][n] + advec_2i5_combine(FX[n + 1], FX[n], fn, fs, ft, FB[n], dxi, dyi, dzik);
                FB[n] = ft;
            }
            settle(UT[p]);
            if (g.n_own) rf_store<NT, T, V>(boff(ut + (int64_t)k * ks, o_own), res, g.n_own);
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int n = 0; n < V; ++n) S[m][n] = S[m + 1][n];
#pragma unroll
            for (int n = 0; n < V; ++n) S[5][n] = UN[q][n];
        }
    }
}

// ---------------------------------------------------------------------------
// diff_smag.  LDS: three planes of levels in rotation (k, k+1 read, the third
// refilled with level k+2 at the end of level k), each holding rows j0-1 ..
// j0+nv of u, v, w and the eddy viscosity with a chunk on each side, and a
// spare chunk per lane.  Level l's rows are loaded at level l-3 (l-2 in 8-byte
// types) and written at level l-2.  The operands on level k-1 are carried in
// registers, in 4-byte types the own ones of level k too.
// ---------------------------------------------------------------------------
template <typename T, int V, int NT>
__global__ __launch_bounds__(512, 2) void diff_smag_rf(StencilArgs<T> a)
{
    // slots of staged rows: two hold a level's rows while the next one's load;
    // in 8-byte types the second slot's registers would spill
    constexpr int NS = sizeof(T) == 4 ? 2 : 1;
    // whether the own operands of level k+1 stay in registers for the next
    // level, or are read from LDS again (same reason)
    constexpr bool CARRY = sizeof(T) == 4;
    extern __shared__ __align__(16) unsigned char les_lds[];
    int sx, ty, tz;
    les_rf_tile_of(a, sx, ty, tz);
    const LesRfTile<V> g(a, sx, ty, tz);
    const int W = g.W, R = g.R, nv = g.nv, k0 = g.k0, k1 = g.k1, kt = a.ktot;
    const int SW = (W + 2) * V, FP = (R + 2) * SW, oS = 4 * FP, PB = oS + 64 * V;
    T *lds = reinterpret_cast<T *>(les_lds);
    const int t = (int)threadIdx.x, lane = t & 63;
    const int64_t ks = a.ks;
    const int js = (int)a.js;
    const int64_t base = a.off + (int64_t)g.j0 * a.js;
    const uint32_t o_own = (uint32_t)(g.row * js + g.i0) * (uint32_t)sizeof(T);
    const T *F[4] = {a.u + base, a.v + base, a.w + base, a.evisc + base};
    T *O[3] = {a.ut + base, a.vt + base, a.wt + base};
    const int lo = (g.row + 1) * SW + V + g.c * V;  // own chunk in a field's plane

    // the thread's extra chunk; the north halo row is not read on level ktot+1
    // (its wide loads could leave a field with one ghost layer there)
    const T *xp = F[0] + 1;
    int lx = oS + lane * V;
    bool north = false;
    {
        int e = t;
        const int n_row = 8 * W, n_edge = 8 * (R + 2);
        int f = 0, rho = 0, col = 1, pos = -1;
        if (e < n_row) {  // halo rows of the four fields
            const int h = e / W, c = e - h * W;
            f = h >> 1;
            rho = h & 1 ? nv + 1 : 0;
            col = g.i0w + c * V;
            pos = c < g.Wl ? V + c * V : -1;
        } else if ((e -= n_row) < n_edge) {  // beyond the segment's ends
            const int r = e >> 3, s = e & 7;
            f = s >> 1;
            rho = r;
            col = s & 1 ? g.right_of(a.itot) : g.left_of(a.itot, V);
            pos = r <= nv + 1 ? (s & 1 ? V + g.Wl * V : 0) : -1;
        }
        if (pos >= 0) {
            const T *p = f == 0 ? F[0] : (f == 1 ? F[1] : (f == 2 ? F[2] : F[3]));
            xp = p + (int64_t)(rho - 1) * js + col;
            lx = f * FP + rho * SW + pos;
            north = rho == nv + 1;
        }
    }

    auto at = [&](const T *f, int l) __attribute__((always_inline)) { return boff(f + (int64_t)l * ks, o_own); };
    T G[NS][4][V], X[NS][V];  // staged own chunks and extra chunk
    T TT[3][V];
    auto load = [&](int q, int l) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 4; ++f) uload<T, V>(G[q][f], at(F[f], l));
        uload<T, V>(X[q], xp + (int64_t)(north ? min(l, kt) : l) * ks);
    };
    auto stage = [&](int q, T *pl) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 4; ++f) vstore<T, V>(pl + f * FP + lo, G[q][f]);
        vstore<T, V>(pl + lx, X[q]);
    };
    T *pb = lds, *pc = lds + PB, *pp = lds + 2 * PB;  // levels k-1 (to be refilled), k, k+1
    const T dxi = a.dxi, dyi = a.dyi;

    load(0, k0 - 1);
    stage(0, pb);
    load(NS - 1, k0);
    stage(NS - 1, pc);
    load(0, k0 + 1);
    if (NS == 2) load(1, min(k0 + 2, k1));

    // carried from level to level: own chunks and neighbours of level k, and
    // the operands of level k-1
    T uc[V], vc[V], wc[V], ec[V], ws[V], es[V], wl, el;
    T bu[V], bur, bv[V], bvn[V], be[V], bel, ber, bes[V], ben[V];
    SmagFace<T> BU[V], BV[V];
    T BW[V];
    __syncthreads();
    {
        const T dzhik = kload(a.dzhi, k0);
        const T *b0 = pb + lo, *b1 = pb + FP + lo, *b2 = pb + 2 * FP + lo, *b3 = pb + 3 * FP + lo;
        T bw[V];
        vload<T, V>(bu, b0);
        bur = b0[V];
        vload<T, V>(bv, b1);
        vload<T, V>(bvn, b1 + SW);
        vload<T, V>(bw, b2);
        vload<T, V>(be, b3);
        bel = b3[-1];
        ber = b3[V];
        vload<T, V>(bes, b3 - SW);
        vload<T, V>(ben, b3 + SW);
        const T *c0 = pc + lo, *c1 = pc + FP + lo, *c2 = pc + 2 * FP + lo, *c3 = pc + 3 * FP + lo;
        vload<T, V>(uc, c0);
        vload<T, V>(vc, c1);
        vload<T, V>(wc, c2);
        vload<T, V>(ec, c3);
        vload<T, V>(ws, c2 - SW);
        vload<T, V>(es, c3 - SW);
        wl = c2[-1];
        el = c3[-1];
#pragma unroll
        for (int n = 0; n < V; ++n) {
            const T ebw = n == 0 ? bel : be[n - 1], ew = n == 0 ? el : ec[n - 1], ww = n == 0 ? wl : wc[n - 1];
            BU[n] = smag_u_zface<T>(ebw, be[n], ew, ec[n], uc[n], bu[n], wc[n], ww, dxi, dzhik);
            BV[n] = smag_v_zface<T>(bes[n], be[n], es[n], ec[n], vc[n], bv[n], wc[n], ws[n], dyi, dzhik);
            BW[n] = smag_w_zcenter<T>(be[n], wc[n], bw[n]);
        }
    }
    stage(0, pp);
    vm_drain();

    for (int kk = k0;; kk += 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = kk + p, q = p ^ 1;
            if (k >= k1) return;
            __syncthreads();  // level k+1 visible, level k-1 no longer read
            // the tendencies of level k, then the rows of level k+3 (k+2 with
            // one slot; clamped at the end of the tile, where they are unused)
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                if constexpr (NT)
                    uload_nt<T, V>(TT[f], at(O[f], k));
                else
                    uload<T, V>(TT[f], at(O[f], k));
            }
            load(NS == 2 ? p : 0, min(k + NS + 1, k1));

            const T *c0 = pc + lo, *c1 = pc + FP + lo, *c2 = pc + 2 * FP + lo, *c3 = pc + 3 * FP + lo;
            const T *t0 = pp + lo, *t1 = pp + FP + lo, *t2 = pp + 2 * FP + lo, *t3 = pp + 3 * FP + lo;
            if constexpr (!CARRY) {
                vload<T, V>(uc, c0);
                vload<T, V>(vc, c1);
                vload<T, V>(wc, c2);
                vload<T, V>(ec, c3);
                vload<T, V>(es, c3 - SW);
                el = c3[-1];
            }
            // the faces at the top of the level, then the horizontal terms:
            // separate phases, so that their operands need not be held together
            T ut[V], vt[V], wt[V], wts[V], et[V], ets[V];
            vload<T, V>(ut, t0);
            vload<T, V>(vt, t1);
            vload<T, V>(wt, t2);
            vload<T, V>(wts, t2 - SW);
            vload<T, V>(et, t3);
            vload<T, V>(ets, t3 - SW);
            const T wtl = t2[-1], etl = t3[-1];
            const T dzik = kload(a.dzi, k), dzikm1 = kload(a.dzi, k - 1), dzhik = kload(a.dzhi, k),
                    dzhik1 = kload(a.dzhi, k + 1);
            SmagFace<T> tu[V], tv[V];
            T tw[V];
#pragma unroll
            for (int n = 0; n < V; ++n) {
                const T ew = n == 0 ? el : ec[n ? n - 1 : 0];
                const T etw = n == 0 ? etl : et[n ? n - 1 : 0], wtw = n == 0 ? wtl : wt[n ? n - 1 : 0];
                tu[n] = smag_u_zface<T>(ew, ec[n], etw, et[n], ut[n], uc[n], wt[n], wtw, dxi, dzhik1);
                tv[n] = smag_v_zface<T>(es[n], ec[n], ets[n], et[n], vt[n], vc[n], wt[n], wts[n], dyi, dzhik1);
                tw[n] = smag_w_zcenter<T>(ec[n], wt[n], wc[n]);
            }
            if constexpr (!CARRY) {
                __builtin_amdgcn_sched_barrier(0);
                vload<T, V>(ws, c2 - SW);
                wl = c2[-1];
            }
            T un[V], us[V], vn[V], vs[V], wn[V], en[V];
            vload<T, V>(un, c0 + SW);
            vload<T, V>(us, c0 - SW);
            vload<T, V>(vn, c1 + SW);
            vload<T, V>(vs, c1 - SW);
            vload<T, V>(wn, c2 + SW);
            vload<T, V>(en, c3 + SW);
            const T ul = c0[-1], ur = c0[V], usr = c0[V - SW];
            const T vl = c1[-1], vr = c1[V], vnl = c1[SW - 1];
            const T wr = c2[V];
            const T er = c3[V], enl = c3[SW - 1], esl = c3[-SW - 1], esr = c3[V - SW];
            T o0[V], o1[V], o2[V];
#pragma unroll
            for (int n = 0; n < V; ++n) {
                const bool f = n == 0, z = n == V - 1;
                const T uw = f ? ul : uc[n ? n - 1 : 0], ue = z ? ur : uc[z ? n : n + 1], use = z ? usr : us[z ? n : n + 1];
                const T vw = f ? vl : vc[n ? n - 1 : 0], ve = z ? vr : vc[z ? n : n + 1], vnw = f ? vnl : vn[n ? n - 1 : 0];
                const T ww = f ? wl : wc[n ? n - 1 : 0], we = z ? wr : wc[z ? n : n + 1];
                const T ew = f ? el : ec[n ? n - 1 : 0], ee = z ? er : ec[z ? n : n + 1], enw = f ? enl : en[n ? n - 1 : 0];
                const T esw = f ? esl : es[n ? n - 1 : 0], ese = z ? esr : es[z ? n : n + 1];
                const T b_ue = z ? bur : bu[z ? n : n + 1], b_ew = f ? bel : be[n ? n - 1 : 0], b_ee = z ? ber : be[z ? n : n + 1];
                o0[n] = TT[0][n] + smag_uv_total<T>(smag_u_xy<T>(uc[n], ue, uw, un[n], us[n], vn[n], vnw, vc[n], vw, ec[n],
                                                                 ew, en[n], enw, es[n], esw, dxi, dyi),
                                                    tu[n], BU[n], dzik);
                o1[n] = TT[1][n] + smag_uv_total<T>(smag_v_xy<T>(vc[n], ve, vw, vn[n], vs[n], ue, use, uc[n], us[n], ec[n],
                                                                 es[n], ee, ese, ew, esw, dxi, dyi),
                                                    tv[n], BV[n], dzik);
                o2[n] = TT[2][n] + smag_w_total<T>(smag_w_xy<T>(wc[n], we, ww, wn[n], ws[n], ue, b_ue, uc[n], bu[n], vn[n],
                                                                bvn[n], vc[n], bv[n], ec[n], be[n], ee, b_ee, ew, b_ew,
                                                                en[n], ben[n], es[n], bes[n], dxi, dyi, dzhik),
                                                   tw[n], BW[n], dzik, dzikm1, dzhik);
                BU[n] = tu[n];
                BV[n] = tv[n];
                BW[n] = tw[n];
            }
#pragma unroll
            for (int f = 0; f < 3; ++f) settle(TT[f]);
            if (g.n_own) {
                rf_store<NT, T, V>(boff(O[0] + (int64_t)k * ks, o_own), o0, g.n_own);
                rf_store<NT, T, V>(boff(O[1] + (int64_t)k * ks, o_own), o1, g.n_own);
                if (k >= a.kw0) rf_store<NT, T, V>(boff(O[2] + (int64_t)k * ks, o_own), o2, g.n_own);
            }
            // the level moves down
            bur = ur;
            bel = el;
            ber = er;
            if constexpr (CARRY) {
                wl = wtl;
                el = etl;
            }
#pragma unroll
            for (int n = 0; n < V; ++n) {
                bu[n] = uc[n];
                bv[n] = vc[n];
                bvn[n] = vn[n];
                be[n] = ec[n];
                bes[n] = es[n];
                ben[n] = en[n];
                if constexpr (CARRY) {
                    uc[n] = ut[n];
                    vc[n] = vt[n];
                    wc[n] = wt[n];
                    ec[n] = et[n];
                    ws[n] = wts[n];
                    es[n] = ets[n];
                }
            }
            stage(NS == 2 ? q : 0, pb);  // level k+2 over level k-1
            T *x = pb;
            pb = pc;
            pc = pp;
            pp = x;
        }
    }
}

}  // namespace kl
