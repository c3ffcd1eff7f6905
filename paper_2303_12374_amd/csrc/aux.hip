// Auxiliary kernels: ghost fill, fused Euler update + ghost refill, interior
// zeroing, FP64 reductions, bit hash and the device-side field generator.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "kl_internal.hpp"
#include "stencil.hpp"

namespace kl {
namespace {

struct Dims {
    int itot, jtot, ktot, bc;
    int64_t off, js, ks;
    int gc;  // ghost cells per side in x and y
};

inline Dims dims_of(const HostArgs &a) { return Dims{a.itot, a.jtot, a.ktot, a.bc, a.off, a.js, a.ks, a.gc}; }

__device__ __forceinline__ int64_t at(const Dims &d, int i, int j, int k)
{
    return d.off + i + (int64_t)j * d.js + (int64_t)k * d.ks;
}

// Interior index of which periodic index p (p >= 1 - gc) is the image.
__device__ __forceinline__ int wrap_n(int p, int n)
{
    int q = (p - 1) % n;
    if (q < 0) q += n;
    return q + 1;
}
__device__ __forceinline__ int wrap_i(const Dims &d, int i) { return wrap_n(i, d.itot); }
__device__ __forceinline__ int wrap_j(const Dims &d, int j) { return wrap_n(j, d.jtot); }

// Source level and factor of level k of field f (0 u, 1 v, 2 w) under the
// boundary rule; factor 0 means the cell is set to zero.
__device__ __forceinline__ int src_k(const Dims &d, int f, int k, int &sign)
{
    sign = 1;
    const int kt = d.ktot;
    if (d.bc == KL_BC_ZPERIODIC) return k == 0 ? kt : (k == kt + 1 ? 1 : k);
    if (f < 2) return k == 0 ? 1 : (k == kt + 1 ? kt : k);
    if (d.bc == KL_BC_ZWALL_ZEROGRAD) return (k == 0 || k == 1) ? 2 : (k == kt + 1 ? kt : k);
    // no penetration
    if (k == 1 || k == kt + 1) {
        sign = 0;
        return 2;
    }
    if (k == 0) {
        sign = -1;
        return 2;
    }
    return k;
}

// One thread per ghost cell (region R0: the whole planes k = 0 and ktot+1;
// R1: the 2 gc ghost rows of levels 1..ktot; R2: the 2 gc ghost columns of
// the interior rows of levels 1..ktot; R3: the interior of plane k = 1, for
// w in wall modes).  Every source cell is an interior cell that no thread
// writes, so the cells can be filled in any order.  kind[f] is the z rule
// of field f (0 and 1: the u/v rule, 2: the w rule); a NULL field is skipped.
// The cell index math is 32-bit: the launchers refuse grids with 2^32 or
// more ghost cells (64-bit divisions cost tens of instructions each).
// r3_wide: region R3 spans the x ghost columns of plane k = 1 too (for a
// refill that skips R2, whose columns at k = 1 belong to w's wall plane).
template <typename T>
__device__ __forceinline__ void fill_cell(const Dims &d, T *u, T *v, T *w, int k0, int k1, int k2, int64_t n0_,
                                          int64_t n1_, int64_t n2_, int64_t n3_, int64_t t_, bool r3_wide = false)
{
    const uint32_t n0 = (uint32_t)n0_, n01 = (uint32_t)(n0_ + n1_), n012 = (uint32_t)(n0_ + n1_ + n2_),
                   nall = (uint32_t)(n0_ + n1_ + n2_ + n3_);
    if (t_ >= (int64_t)nall) return;
    const uint32_t t = (uint32_t)t_;
    const int gc = d.gc;
    const uint32_t ic = (uint32_t)(d.itot + 2 * gc), plane = ic * (uint32_t)(d.jtot + 2 * gc);
    const uint32_t g2 = 2u * (uint32_t)gc;
    int i, j, k;
    bool w_only = false;
    if (t < n0) {
        const uint32_t p = t < plane ? t : t - plane;
        k = t < plane ? 0 : d.ktot + 1;
        j = (int)(p / ic) + 1 - gc;
        i = (int)(p % ic) + 1 - gc;
    } else if (t < n01) {
        const uint32_t q = t - n0;
        const uint32_t r = q / ic;  // ghost row index over (level, row)
        i = (int)(q % ic) + 1 - gc;
        k = 1 + (int)(r / g2);
        const int jr = (int)(r % g2);
        j = jr < gc ? 1 - gc + jr : d.jtot + 1 + (jr - gc);
    } else if (t < n012) {
        const uint32_t q = t - n01;
        const int c = (int)(q % g2);
        const uint32_t rest = q / g2;
        j = 1 + (int)(rest % (uint32_t)d.jtot);
        k = 1 + (int)(rest / (uint32_t)d.jtot);
        i = c < gc ? 1 - gc + c : d.itot + 1 + (c - gc);
    } else {
        const uint32_t q = t - n012;
        const uint32_t rw = r3_wide ? ic : (uint32_t)d.itot;
        k = 1;
        j = 1 + (int)(q / rw);
        i = 1 + (int)(q % rw) - (r3_wide ? gc : 0);
        w_only = true;
    }
    const int si = wrap_i(d, i), sj = wrap_j(d, j);
    const int64_t dst = at(d, i, j, k);
    T *f3[3] = {u, v, w};
    const int kind[3] = {k0, k1, k2};
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        T *p = f3[f];
        if (!p || (w_only && kind[f] != 2)) continue;
        int sign;
        const int sk = src_k(d, kind[f], k, sign);
        p[dst] = sign == 0 ? T(0) : (sign < 0 ? -p[at(d, si, sj, sk)] : p[at(d, si, sj, sk)]);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void fill_ghosts_kernel(Dims d, T *u, T *v, T *w, int k0, int k1, int k2,
                                                         int64_t n0, int64_t n1, int64_t n2, int64_t n3,
                                                         bool r3_wide)
{
    fill_cell<T>(d, u, v, w, k0, k1, k2, n0, n1, n2, n3, (int64_t)blockIdx.x * 256 + threadIdx.x, r3_wide);
}

// Ghost fill of the velocity fields of many grids in one launch: block b
// fills cells [256 lb, 256 lb + 256) of grid job g, (g, lb) = blocks[b];
// the same cell map and copies as the single-grid fill.
struct FillJob {
    Dims d;
    void *u, *v, *w;
    int64_t n0, n1, n2, n3;
};

template <typename T>
__global__ __launch_bounds__(256) void fill_ghosts_batch_kernel(const FillJob *__restrict__ jobs,
                                                               const int2 *__restrict__ blocks)
{
    const int2 b = blocks[blockIdx.x];
    const FillJob j = jobs[b.x];
    fill_cell<T>(j.d, as_global((T *)j.u), as_global((T *)j.v), as_global((T *)j.w), 0, 1, 2, j.n0, j.n1, j.n2,
                 j.n3, (int64_t)b.y * 256 + threadIdx.x);
}

template <typename T>
__global__ __launch_bounds__(256) void zero_interior_kernel(Dims d, T *f, int nbx)
{
    unsigned b = blockIdx.x;
    const int bx = b % nbx;
    b /= nbx;
    const int j = 1 + (int)(b % d.jtot);
    const int k = 1 + (int)(b / d.jtot);
    const int i = 1 + bx * 256 + (int)threadIdx.x;
    if (i > d.itot) return;
    f[at(d, i, j, k)] = T(0);
}

// ---------------------------------------------------------------------------
// Rows cut into pieces, for the kernels that stream the interior in memory
// order (reductions, Euler update).  A piece is up to R rows of one level; a
// row is cpr chunks of V consecutive points, the last one moved back so that
// it ends at itot (its first `ov` points repeat the chunk before it and are
// masked).  The loads are 16 bytes wide at element alignment, so any itot >= V
// and any layout takes the same path.  The level is one per piece, which
// leaves one 32-bit multiplication per chunk for the row index and one
// metric read per piece.
// ---------------------------------------------------------------------------
struct RowPieces {
    uint32_t cpr;    // chunks per row
    uint32_t magic;  // (e * magic) >> 32 = e / cpr for e < R * cpr (0 when R = 1: row 0)
    uint32_t ov;     // repeated points of a row's last chunk
    uint32_t R, ng;  // rows per piece, pieces per level
    uint32_t np;     // pieces
};

// e / cpr by multiplication with the rounded-up reciprocal is exact while
// e * cpr < 2^32; here e < 2^14, and cpr <= 2^13 where a piece has two rows.
RowPieces row_pieces(const HostArgs &a, int V, int64_t chunks_per_piece)
{
    RowPieces r;
    r.cpr = (uint32_t)((a.itot + V - 1) / V);
    r.ov = r.cpr * (uint32_t)V - (uint32_t)a.itot;
    r.R = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(a.jtot, std::min<int64_t>(chunks_per_piece, 1 << 14) / r.cpr));
    r.magic = r.R == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + r.cpr - 1) / r.cpr);
    r.ng = ((uint32_t)a.jtot + r.R - 1) / r.R;
    r.np = r.ng * (uint32_t)a.ktot;
    return r;
}

// The Euler update's blocks, a chunk per thread: the rows that fit 256 threads,
// or one row of up to 512 chunks, or an equal part of a longer one.  Whole waves,
// so that those of a row that starts on a cache line store whole lines.  (Longer
// rows in 256 threads, us; one point per thread, chunks in a loop, now:
// 2048x4x64 FP64 10.2, 15.1, 7.9; 1500x200x100 FP64 unpadded 398, 465, 411;
// 1024x500x64 FP64 450, 426, 400; 560x300x100 FP64 238, 209, 201.  Blocks of
// 256 cut out of one row, or out of several in a run: 560x300x100 240, 207;
// 526x359x388 FP64, now 898, 926 in a loop, 1000 in a run.)
struct EulerBlocks {
    RowPieces rp;
    uint32_t threads, nseg;  // per block; blocks per piece
};

EulerBlocks euler_blocks(const HostArgs &a, int V)
{
    EulerBlocks b;
    b.rp = row_pieces(a, V, 256);
    b.threads = 256;
    b.nseg = 1;
    if (b.rp.cpr > 256) {
        b.nseg = (b.rp.cpr + 511) / 512;
        b.threads = ((b.rp.cpr + b.nseg - 1) / b.nseg + 63) / 64 * 64;
    }
    return b;
}

// Points per 16-byte chunk, or 1 for rows narrower than that.
inline int row_chunk(const HostArgs &a)
{
    const int V = a.dtype == KL_F32 ? 4 : 2;
    return a.itot >= V ? V : 1;
}

// Chunk e of a piece of n chunks: its row and first column (0-based) in the
// piece, and the first of its V points that counts (V: none, for a thread
// beyond the piece's end).
template <int V>
struct Chunk {
    int row, col, lo;
    __device__ Chunk() {}
    __device__ __forceinline__ Chunk(const RowPieces &rp, uint32_t e, uint32_t n)
    {
        const uint32_t ec = e < n ? e : n - 1;
        const uint32_t r = rp.cpr == 1 ? ec : __umulhi(ec, rp.magic);
        const uint32_t c = ec - r * rp.cpr;
        const uint32_t ov = V > 1 && c == rp.cpr - 1 ? rp.ov : 0u;
        row = (int)r;
        col = (int)(c * (uint32_t)V - ov);
        lo = e < n ? (int)ov : V;
    }
};

// ---------------------------------------------------------------------------
// Forward Euler, f += dt * ft, with the ghost refill: the thread that updates
// a chunk also writes every ghost cell whose source is in it (the inverse of
// the fill map; needs itot, jtot >= gc, so that every ghost cell is the image
// of one interior cell by one shift).
//
// Bound by HBM: 6 values read and 3 written per point.  One chunk per thread
// and 256 a piece: the blocks then sweep memory in order (pieces of 2048
// chunks ran 10-20% slower).  The tendencies are read for the last time and
// stream past the caches.  The images cost a branch that only the pieces and
// chunks on a face take.  Against one point per thread (and a second kernel
// for the outer layers of a three-layer halo): 256^3 FP32 158 -> 85 us, gc = 3
// 176 -> 95; 512x512x256 FP32 592 -> 413 us (5.9 TB/s), FP64 1055 -> 825;
// 301x203x151 FP32 137 -> 52 us.
// ---------------------------------------------------------------------------
// Store the points n >= lo of a chunk at (i0 .., j, k), and their x images.
template <typename T, int V, int NT = 0>
__device__ __forceinline__ void put_chunk(const Dims &d, T *p, int i0, int j, int k, int lo, const T (&val)[V])
{
    T *row = p + at(d, 0, j, k);
    if (lo == 0) {
        if constexpr (NT)
            ustore_nt<T, V>(row + i0, val);
        else
            ustore<T, V>(row + i0, val);
    } else {
#pragma unroll
        for (int n = 0; n < V; ++n)
            if (n >= lo) row[i0 + n] = val[n];
    }
    if (i0 <= d.gc || i0 + V - 1 > d.itot - d.gc) {
#pragma unroll
        for (int n = 0; n < V; ++n) {
            const int i = i0 + n;
            if (n >= lo && i <= d.gc) row[d.itot + i] = val[n];
            if (n >= lo && i > d.itot - d.gc) row[i - d.itot] = val[n];
        }
    }
}

template <typename T, int V, int NT>
__device__ __forceinline__ void euler_chunk(const Dims &d, T *p, int f, int i0, int j, int k,
                                            int lo, const T (&val)[V])
{
    put_chunk<T, V, NT>(d, p, i0, j, k, lo, val);
    const int kt = d.ktot;
    if (j > d.gc && j <= d.jtot - d.gc && k > 2 && k < kt) return;
    // z images with their factors
    int zk[4], zs[4], nz = 1;
    zk[0] = k;
    zs[0] = 1;
    if (d.bc == KL_BC_ZPERIODIC) {
        if (k == kt) { zk[nz] = 0; zs[nz++] = 1; }
        if (k == 1) { zk[nz] = kt + 1; zs[nz++] = 1; }
    } else if (f < 2) {
        if (k == 1) { zk[nz] = 0; zs[nz++] = 1; }
        if (k == kt) { zk[nz] = kt + 1; zs[nz++] = 1; }
    } else if (d.bc == KL_BC_ZWALL_ZEROGRAD) {
        if (k == 2) { zk[nz] = 0; zs[nz++] = 1; zk[nz] = 1; zs[nz++] = 1; }
        if (k == kt) { zk[nz] = kt + 1; zs[nz++] = 1; }
    } else {
        if (k == 2) { zk[nz] = 0; zs[nz++] = -1; zk[nz] = 1; zs[nz++] = 0; }
        if (k == kt) { zk[nz] = kt + 1; zs[nz++] = 0; }
    }
    for (int a = 0; a < nz; ++a) {
        T v[V];
#pragma unroll
        for (int n = 0; n < V; ++n) v[n] = zs[a] == 0 ? T(0) : (zs[a] < 0 ? -val[n] : val[n]);
        if (a > 0) put_chunk<T, V>(d, p, i0, j, zk[a], lo, v);
        if (j <= d.gc) put_chunk<T, V>(d, p, i0, d.jtot + j, zk[a], lo, v);
        if (j > d.jtot - d.gc) put_chunk<T, V>(d, p, i0, j - d.jtot, zk[a], lo, v);
    }
}

// Block b: part b % nseg of piece b / nseg (256 threads: a whole piece).
template <typename T, int V, int NT, int THREADS>
__global__ __launch_bounds__(THREADS) void euler_kernel(Dims d, RowPieces rp, uint32_t nseg, T dt, int kw0, T *u, T *v,
                                                   T *w, const T *ut, const T *vt, const T *wt)
{
    const uint32_t pc = THREADS == 256 ? blockIdx.x : blockIdx.x / nseg;
    const uint32_t e = THREADS == 256 ? threadIdx.x : (blockIdx.x - pc * nseg) * blockDim.x + threadIdx.x;
    const int k = 1 + (int)(pc / rp.ng);
    const uint32_t j0 = (pc % rp.ng) * rp.R;
    const uint32_t left = (uint32_t)d.jtot - j0;
    const uint32_t n = (left < rp.R ? left : rp.R) * rp.cpr;
    if (e >= n) return;
    T *f3[3] = {u, v, w};
    const T *t3[3] = {ut, vt, wt};
    const int64_t base = at(d, 1, 1 + (int)j0, k);
    const Chunk<V> c(rp, e, n);
    const int64_t o = base + (int64_t)c.row * d.js + c.col;
    T x[3][V], y[3][V];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        if constexpr (NT)
            uload_nt<T, V>(x[f], f3[f] + o);
        else
            uload<T, V>(x[f], f3[f] + o);
        uload_nt<T, V>(y[f], t3[f] + o);
    }
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        if (f == 2 && k < kw0) continue;
        T val[V];
#pragma unroll
        for (int i = 0; i < V; ++i) val[i] = euler_value<T>(x[f][i], dt, y[f][i]);
        euler_chunk<T, V, NT>(d, f3[f], f, 1 + c.col, 1 + (int)j0 + c.row, k, c.lo, val);
    }
}

// ---------------------------------------------------------------------------
// FP64 checksums (sum, sum of squares, largest magnitude of each field).  Pass
// 1: block b of nb sums pieces b, b + nb, ...; a thread takes every RT-th chunk
// of a piece, RM in flight at a time; partials are combined by a fixed tree
// (lanes, then waves).  Pass 2 reduces the nb partials in one block the same
// way.  No atomics, and the mapping depends only on the grid, so the result is
// bitwise reproducible.
//
// Bound by HBM (one read of the fields) down to about 10^7 points, below that
// by the two launches.  Two chunks of three fields keep 6 16-byte loads in
// flight per thread (the nine sums need the registers: four chunks took 134 and
// were slower), and 1024 chunks a piece still give a 128^3 grid 512 blocks; at
// most RED_MAXB blocks (8 per CU) keep pass 2 to a few loads per thread.
// Against 4096 blocks of scattered rows, a division per point and row, and a
// tree over LDS (us): 512^3 FP32 311 -> 284, 128^3 26 -> 12, 301x203x151 FP32
// (one point per load before) 102 -> 28.
// ---------------------------------------------------------------------------
constexpr int RB = 4096;   // pass-1 blocks of the hash, and the scratch's partial count
constexpr int RT = 256;    // threads per block
constexpr int RQ = 9;      // values per partial
constexpr int RED_MAXB = 2048;
constexpr int SUM_P = 4;   // batched sums: partials per group of waves
constexpr int RT2 = 512;   // threads of pass 2
static_assert(RED_MAXB <= RB, "the reductions' partials fit the scratch");

constexpr int RM = 2;      // chunks in flight per thread
__device__ constexpr bool is_max(int q) { return q % 3 == 2; }

struct RedPlan {
    RowPieces rp;
    int nb;  // pass-1 blocks
};

RedPlan red_plan(const HostArgs &a)
{
    RedPlan p;
    const int V = row_chunk(a);
    const int64_t total = (int64_t)((a.itot + V - 1) / V) * a.jtot * a.ktot;
    p.rp = row_pieces(a, V, std::min<int64_t>(4096, std::max<int64_t>(1024, total / RED_MAXB)));
    p.nb = (int)std::min<uint32_t>(RED_MAXB, p.rp.np);
    return p;
}

// Conservation sums: points per load, partials, and waves per partial (those of
// the slots that own rows; a block of RT threads takes 4 / waves groups of partials).
int sum_rows_chunk(const HostArgs &a, const void *f0, const void *f1, const void *f2)
{
    const int V = a.dtype == KL_F32 ? 4 : 2;
    const bool aligned = a.itot % V == 0 && (a.off + 1) % V == 0 && a.js % V == 0 && a.ks % V == 0 &&
                         ((uintptr_t)f0 | (uintptr_t)f1 | (uintptr_t)f2) % 16 == 0;
    return aligned ? V : 1;
}
int sum_rows_blocks(const HostArgs &a) { return (int)std::min<int64_t>(RB, (int64_t)a.jtot * a.ktot); }
int sum_rows_waves(const HostArgs &a, int V)
{
    const int cpr = a.itot / V;
    if (cpr >= RT) return RT / 64;
    const int64_t slots = ((int64_t)a.jtot * a.ktot + RB - 1) / RB, threads = std::min<int64_t>(RT / cpr, slots) * cpr;
    return threads <= 64 ? 1 : threads <= 128 ? 2 : 4;
}

// Reduce acc over the block's NT threads; thread q < RQ writes value q to
// out[q * stride].
template <int NT>
__device__ __forceinline__ void block_tree(double (&acc)[RQ], double *out, int64_t stride)
{
    constexpr int NQ = RQ, NW = NT / 64;
    __shared__ double sh[NW][NQ];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double o = __shfl_down(acc[q], (unsigned)s, 64);
            acc[q] = is_max(q) ? fmax(acc[q], o) : acc[q] + o;
        }
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[wave][q] = acc[q];
    __syncthreads();
    if ((int)threadIdx.x < NQ) {
        const int q = (int)threadIdx.x;
        double r = sh[0][q];
        for (int w = 1; w < NW; ++w) r = q % 3 == 2 ? fmax(r, sh[w][q]) : r + sh[w][q];
        out[q * stride] = r;
    }
}

// Pass-1 block b of nb; its partial value q goes to partial[q * nb + b].
template <typename T, int V>
__global__ __launch_bounds__(RT) void reduce_pass1(Dims d, RedPlan pl, const T *f0, const T *f1, const T *f2,
                                                  double *partial)
{
    const RowPieces &rp = pl.rp;
    const T *f3[3] = {f0, f1, f2};
    double acc[RQ];
    T mx[3] = {T(0), T(0), T(0)};  // the largest |f| so far, exact in T
#pragma unroll
    for (int q = 0; q < RQ; ++q) acc[q] = 0.0;
    for (uint32_t p = blockIdx.x; p < rp.np; p += (uint32_t)pl.nb) {
        const int k = 1 + (int)(p / rp.ng);
        const uint32_t j0 = (p % rp.ng) * rp.R;
        const uint32_t left = (uint32_t)d.jtot - j0;
        const uint32_t n = (left < rp.R ? left : rp.R) * rp.cpr;
        const int64_t base = at(d, 1, 1 + (int)j0, k);
        for (uint32_t e0 = threadIdx.x; e0 < n; e0 += RM * RT) {
            T x[RM][3][V];
            int lo[RM];
#pragma unroll
            for (int m = 0; m < RM; ++m) {
                const Chunk<V> c(rp, e0 + m * RT, n);
                const int64_t o = base + (int64_t)c.row * d.js + c.col;
                lo[m] = c.lo;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    if (f3[f] == nullptr) {
#pragma unroll
                        for (int i = 0; i < V; ++i) x[m][f][i] = T(0);
                    } else {
                        uload<T, V>(x[m][f], f3[f] + o);
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < RM; ++m)
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        const T xi = i < lo[m] ? T(0) : x[m][f][i];
                        const double y = (double)xi;
                        acc[3 * f] += y;
                        acc[3 * f + 1] = tfma(y, y, acc[3 * f + 1]);
                        mx[f] = tmax(mx[f], tabs(xi));
                    }
        }
    }
#pragma unroll
    for (int f = 0; f < 3; ++f) acc[3 * f + 2] = (double)mx[f];
    block_tree<RT>(acc, partial + blockIdx.x, pl.nb);
}

// Pass 2 over nb partials (value q of block b at partial[q * nb + b]).
__global__ __launch_bounds__(RT2) void reduce_pass2(const double *partial, int nb, double *out)
{
    double acc[RQ];
#pragma unroll
    for (int q = 0; q < RQ; ++q) acc[q] = 0.0;
#pragma unroll
    for (int m = 0; m < RED_MAXB / RT2; ++m) {
        const int b = m * RT2 + (int)threadIdx.x;
        if (b < nb)
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                const double y = partial[(int64_t)q * nb + b];
                acc[q] = is_max(q) ? fmax(acc[q], y) : acc[q] + y;
            }
    }
    block_tree<RT2>(acc, out, 1);
}

// Conservation sums.  Where they vanish (momentum tendencies of the flux-form
// schemes, z periodic) the digits of the result are the rounding of this very
// order of additions, so the order is fixed: row r = (j, k) pairs belongs to
// partial r % RB, a row's points in chunks of V (16 bytes where rows and fields
// are aligned to it, else one point) to the RT threads of that partial, slot s
// of rpp = RT / cpr taking every rpp-th of its rows; each point is weighted,
// then added; the threads' sums are combined by halving.
//
// Bound by HBM at 256^3, by the two launches below.  Only threads and partials
// that own rows are launched (partials of one or two waves share a block), four
// rows are in flight per thread, and the tree is one exchange between waves and
// shuffles.  Against 4096 blocks of 256, two rows in flight and nine values
// over LDS (us): 512^3 FP32 351 -> 274 (5.9 TB/s), 128^3 27 -> 12,
// 301x203x151 FP32 (one point per load) 102 -> 37; FP64 256^3 110 -> 76,
// 301x203x151 69 -> 40.  In a batch the rows of a partial are few, so a group
// of waves takes four partials at once: 56 grids FP32, 0.2 million partials,
// the whole graph 807 us with one per block, 715 with one per group, 646 with
// four.

// Sums of NP values of acc over each group of gw waves (1, 2 or 4) of a block of
// RT threads; partial p of the group goes to out + p if p < n.
template <int NP>
__device__ __forceinline__ void sum_tree(double (&acc)[NP][3], int gw, double *out, int n, int64_t stride)
{
    __shared__ double sh[RT / 64][3 * NP][64];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    if (gw > 1) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) sh[wave][3 * p + q][lane] = acc[p][q];
        __syncthreads();
        if (wave & (gw - 1)) return;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int e = 3 * p + q;
                const double w1 = sh[wave + 1][e][lane], w2 = gw > 2 ? sh[(wave + 2) & 3][e][lane] : 0.0,
                             w3 = gw > 2 ? sh[(wave + 3) & 3][e][lane] : 0.0;
                acc[p][q] = (acc[p][q] + w2) + (w1 + w3);
            }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[p][q] += __shfl_down(acc[p][q], (unsigned)s, 64);
    if (lane == 0)
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (p < n)
#pragma unroll
                for (int q = 0; q < 3; ++q) out[q * stride + p] = acc[p][q];
}

// The block's partials, from b0: NP for each group of gw waves (one where a row
// has RT chunks or more), four rows in flight.
template <typename T, int V, int NP>
__device__ __forceinline__ void sum_rows(const Dims &d, int kw0, const T *f0, const T *f1, const T *f2, const T *dzi,
                                         const T *dzhi, int b0, int nb, int gw, double *partial)
{
    const int t = (int)threadIdx.x & (64 * gw - 1);
    const int cpr = d.itot / V;
    const bool wide = cpr >= RT;  // one partial per block
    const uint32_t b = (uint32_t)(b0 + (int)threadIdx.x / (64 * gw) * NP);
    const uint32_t nrows = (uint32_t)d.jtot * (uint32_t)d.ktot, jt = (uint32_t)d.jtot;  // below 2^31
    const T *f3[3] = {f0, f1, f2};
    double acc[NP][3];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q) acc[p][q] = 0.0;
    auto load = [&](T (&x)[3][V], uint32_t r, int c) {
        const int64_t o = at(d, 1 + c * V, 1 + (int)(r % jt), 1 + (int)(r / jt));
#pragma unroll
        for (int f = 0; f < 3; ++f) vload<T, V>(x[f], f3[f] + o);
    };
    auto add = [&](double (&a)[3], const T (&x)[3][V], uint32_t r) {
        const int k = 1 + (int)(r / jt);
        const double wz = 1.0 / (double)dzi[k], wzh = 1.0 / (double)dzhi[k];
#pragma unroll
        for (int n = 0; n < V; ++n) {
            a[0] += (double)x[0][n] * wz;
            a[1] += (double)x[1][n] * wz;
            if (k >= kw0) a[2] += (double)x[2][n] * wzh;
        }
    };
    if (!wide) {
        const int rpp = RT / cpr, slot = t / cpr, c = t % cpr;
        const uint32_t step = (uint32_t)rpp * RB;
        constexpr int M = 4 / NP;
        if (slot < rpp)
            for (uint32_t r = b + (uint32_t)slot * RB; r < nrows; r += M * step) {
                T x[M][NP][3][V];
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int p = 0; p < NP; ++p) load(x[m][p], min(r + m * step + p, nrows - 1), c);
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        if (r + m * step + p < nrows) add(acc[p], x[m][p], r + m * step + p);
            }
    } else {  // pairs of rows, chunk by chunk
        uint32_t r = b;
        for (; r + RB < nrows; r += 2 * RB)
            for (int c = t; c < cpr; c += 2 * RT) {
                const bool two = c + RT < cpr;
                const int c2 = two ? c + RT : c;
                T x[4][3][V];
                load(x[0], r, c);
                load(x[1], r + RB, c);
                load(x[2], r, c2);
                load(x[3], r + RB, c2);
                add(acc[0], x[0], r);
                add(acc[0], x[1], r + RB);
                if (two) {
                    add(acc[0], x[2], r);
                    add(acc[0], x[3], r + RB);
                }
            }
        if (r < nrows)
            for (int c = t; c < cpr; c += RT) {
                T x[3][V];
                load(x, r, c);
                add(acc[0], x, r);
            }
    }
    sum_tree<NP>(acc, gw, partial + b, wide ? 1 : nb - (int)b, nb);
}

template <typename T, int V>
__global__ __launch_bounds__(RT) void sum_rows_pass1(Dims d, int kw0, const T *f0, const T *f1, const T *f2,
                                                    const T *dzi, const T *dzhi, int nb, int gw, double *partial)
{
    sum_rows<T, V, 1>(d, kw0, f0, f1, f2, dzi, dzhi, (int)blockIdx.x * (4 / gw), nb, gw, partial);
}

// Pass 2 by one block: thread t sums partials t, t + RT, ...
__device__ __forceinline__ void sum_rows_final(const double *partial, int nb, double *out)
{
    double acc[1][3] = {{0.0, 0.0, 0.0}};
#pragma unroll
    for (int m = 0; m < RB / RT; ++m) {
        const int b = m * RT + (int)threadIdx.x;
#pragma unroll
        for (int q = 0; q < 3; ++q) acc[0][q] += b < nb ? partial[(int64_t)q * nb + b] : 0.0;
    }
    sum_tree<1>(acc, RT / 64, out, 1, 1);
}

__global__ __launch_bounds__(RT) void sum_rows_pass2(const double *partial, int nb, double *out)
{
    sum_rows_final(partial, nb, out);
}

// Conservation sums of many grids in two launches: pass-1 block blockIdx.x is
// block b of job g, (g, b) = blocks[blockIdx.x], into that job's own partials;
// pass 2 reduces each grid's partials in one block.  Per grid the rows,
// blocks and trees are those of the single-grid reduction, so each grid's
// sums are bitwise those of kl_reduce_fp64.
struct SumJob {
    Dims d;
    int kw0, nb, gw;
    int64_t first;  // the job's first partial
    const void *f0, *f1, *f2, *dzi, *dzhi;
};

template <typename T, int V>
__global__ __launch_bounds__(RT) void sums_batch_pass1(const SumJob *__restrict__ jobs,
                                                      const int2 *__restrict__ blocks, double *partials)
{
    const int2 gb = blocks[blockIdx.x];
    const SumJob j = jobs[gb.x];
    sum_rows<T, V, SUM_P>(j.d, j.kw0, as_global((const T *)j.f0), as_global((const T *)j.f1),
                          as_global((const T *)j.f2), as_global((const T *)j.dzi), as_global((const T *)j.dzhi), gb.y, j.nb, j.gw, partials + j.first);
}

__global__ __launch_bounds__(RT) void sums_batch_pass2(const longlong2 *__restrict__ slots, const double *partials,
                                                       double *out)
{
    const longlong2 sl = slots[blockIdx.x];  // first partial and number of blocks of this grid
    sum_rows_final(partials + sl.x, (int)sl.y, out + 3 * (int64_t)blockIdx.x);
}

// Bit hash: sum over interior cells (mod 2^64) of SplitMix64(bits ^ cell key).
__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

template <typename T>
__device__ __forceinline__ uint64_t bits_of(T x)
{
    if constexpr (sizeof(T) == 8) {
        return (uint64_t)__double_as_longlong(x);
    } else {
        return (uint64_t)(uint32_t)__float_as_uint(x);
    }
}

template <typename T>
__global__ __launch_bounds__(RT) void hash_pass1(Dims d, const T *f, uint64_t *partial)
{
    uint64_t acc = 0;
    const int64_t nrows = (int64_t)d.jtot * d.ktot;
    for (int64_t r = blockIdx.x; r < nrows; r += RB) {
        const int j = 1 + (int)(r % d.jtot);
        const int k = 1 + (int)(r / d.jtot);
        const int64_t base = at(d, 0, j, k);
        for (int i = 1 + (int)threadIdx.x; i <= d.itot; i += RT) {
            const uint64_t key = (uint64_t)i + ((uint64_t)j << 21) + ((uint64_t)k << 42);
            acc += mix64(bits_of<T>(f[base + i]) ^ mix64(key));
        }
    }
    __shared__ uint64_t sh[RT];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = RT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(RT) void hash_pass2(const uint64_t *partial, uint64_t *out)
{
    uint64_t acc = 0;
    for (int b = threadIdx.x; b < RB; b += RT) acc += partial[b];
    __shared__ uint64_t sh[RT];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = RT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

// Device generator of the served initial state: U[-1,1) noise from the
// counter-based SplitMix64 recipe plus the mean flow (1, 0.5, 0), rounded to
// the field type.  Counter of interior point (i-1, j-1, k-1) of field f:
// ((seed*8 + f) << 40) + (i-1) + itot*((j-1) + jtot*(k-1)).
template <typename T>
__global__ __launch_bounds__(256) void gen_uniform_kernel(Dims d, uint64_t seed, T *u, T *v, T *w, int nbx)
{
    unsigned b = blockIdx.x;
    const int bx = b % nbx;
    b /= nbx;
    const int j = 1 + (int)(b % d.jtot);
    const int k = 1 + (int)(b / d.jtot);
    const int i = 1 + bx * 256 + (int)threadIdx.x;
    if (i > d.itot) return;
    const int64_t c = at(d, i, j, k);
    const uint64_t cnt = (uint64_t)(i - 1) + (uint64_t)d.itot * ((uint64_t)(j - 1) + (uint64_t)d.jtot * (uint64_t)(k - 1));
    const double mean[3] = {1.0, 0.5, 0.0};
    T *f3[3] = {u, v, w};
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        const uint64_t key = ((seed * 8u + (uint64_t)f) << 40) + cnt;
        const double r = (double)(mix64(key) >> 11) * 0x1.0p-53;
        f3[f][c] = (T)((2.0 * r - 1.0) + mean[f]);
    }
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

size_t reduce_scratch_bytes() { return (size_t)RB * RQ * sizeof(double); }

namespace {
hipError_t fill_launch(const HostArgs &a, void *u, void *v, void *w, int k0, int k1, int k2, bool w_faces,
                       hipStream_t s, bool x_columns = true)
{
    const Dims d = dims_of(a);
    const int64_t gc = a.gc;
    const int64_t ic = a.itot + 2 * gc, jc = a.jtot + 2 * gc;
    const int64_t n0 = 2 * ic * jc, n1 = 2 * gc * ic * a.ktot;
    const int64_t n2 = x_columns ? 2 * gc * (int64_t)a.jtot * a.ktot : 0;  // region R2 (x ghost columns)
    // R3 (w's plane k = 1 in wall modes) with its x ghost columns when R2 is skipped
    const int64_t n3 = (w_faces && a.bc != KL_BC_ZPERIODIC) ? (x_columns ? a.itot : ic) * (int64_t)a.jtot : 0;
    if (n0 + n1 + n2 + n3 >= ((int64_t)1 << 32)) return hipErrorInvalidValue;  // 32-bit cell index
    const unsigned nb = cdiv(n0 + n1 + n2 + n3, 256);
    if (a.dtype == KL_F32)
        hipLaunchKernelGGL(fill_ghosts_kernel<float>, dim3(nb), dim3(256), 0, s, d, (float *)u, (float *)v,
                           (float *)w, k0, k1, k2, n0, n1, n2, n3, !x_columns);
    else
        hipLaunchKernelGGL(fill_ghosts_kernel<double>, dim3(nb), dim3(256), 0, s, d, (double *)u,
                           (double *)v, (double *)w, k0, k1, k2, n0, n1, n2, n3, !x_columns);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_fill_ghosts(const HostArgs &a, void *u, void *v, void *w, hipStream_t s)
{
    return fill_launch(a, u, v, w, 0, 1, 2, true, s);
}

hipError_t launch_fill_yz_images(const HostArgs &a, void *u, void *v, void *w, hipStream_t s)
{
    return fill_launch(a, u, v, w, 0, 1, 2, true, s, false);
}

hipError_t launch_fill_scalar(const HostArgs &a, void *f, hipStream_t s)
{
    return fill_launch(a, f, nullptr, nullptr, 0, 0, 0, false, s);
}

namespace {
// Above this size of u, v and w together they are streamed past the caches:
// the memory-side cache holds 256 MB, and fields that fit are still there
// when the next kernel reads them (256^3 FP32, 201 MB: 86 us cached, 104
// streamed; 512x512x256 FP32, 805 MB: 507 us cached, 397 streamed).
constexpr double EULER_CACHED_BYTES = 256e6;

template <typename T, int V, int NT>
void euler_go(const HostArgs &a, const Dims &d, const EulerBlocks &b, double dt, void *u, void *v, void *w, hipStream_t s)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(b.rp.np * b.nseg), dim3(b.threads), 0, s, d, b.rp, b.nseg, (T)dt, a.kw0, (T *)u,
                           (T *)v, (T *)w, (const T *)a.ut, (const T *)a.vt, (const T *)a.wt);
    };
    if (b.threads > 256)  // only rows of more than 256 chunks
        go(euler_kernel<T, V, NT, 512>);
    else
        go(euler_kernel<T, V, NT, 256>);
}
}  // namespace

hipError_t launch_euler(const HostArgs &a, double dt, void *u, void *v, void *w, hipStream_t s)
{
    // grids narrower than their halo: update with one ghost layer, refill all of them after
    const bool narrow = a.itot < a.gc || a.jtot < a.gc;
    Dims d = dims_of(a);
    if (narrow) d.gc = 1;
    if ((int64_t)a.jtot * a.ktot >= ((int64_t)1 << 31)) return hipErrorInvalidValue;  // 32-bit piece index
    const int V = row_chunk(a);
    const EulerBlocks b = euler_blocks(a, V);
    const bool nt = 3.0 * a.itot * a.jtot * a.ktot * (a.dtype == KL_F32 ? 4 : 8) > EULER_CACHED_BYTES;
    if (a.dtype == KL_F32)
        V == 4 ? (nt ? euler_go<float, 4, 1>(a, d, b, dt, u, v, w, s) : euler_go<float, 4, 0>(a, d, b, dt, u, v, w, s))
               : euler_go<float, 1, 0>(a, d, b, dt, u, v, w, s);
    else
        V == 2 ? (nt ? euler_go<double, 2, 1>(a, d, b, dt, u, v, w, s) : euler_go<double, 2, 0>(a, d, b, dt, u, v, w, s))
               : euler_go<double, 1, 0>(a, d, b, dt, u, v, w, s);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && narrow ? launch_fill_ghosts(a, u, v, w, s) : e;
}

hipError_t launch_zero_interior(const HostArgs &a, void *f, hipStream_t s)
{
    const Dims d = dims_of(a);
    const int nbx = (int)cdiv(a.itot, 256);
    const unsigned nb = (unsigned)nbx * a.jtot * a.ktot;
    if (a.dtype == KL_F32)
        hipLaunchKernelGGL(zero_interior_kernel<float>, dim3(nb), dim3(256), 0, s, d, (float *)f, nbx);
    else
        hipLaunchKernelGGL(zero_interior_kernel<double>, dim3(nb), dim3(256), 0, s, d, (double *)f, nbx);
    return hipGetLastError();
}

namespace {
template <typename T, int V>
void sums_go(const HostArgs &a, int nb, const void *f0, const void *f1, const void *f2, double *partial,
             hipStream_t s)
{
    const int gw = sum_rows_waves(a, V);
    hipLaunchKernelGGL((sum_rows_pass1<T, V>), dim3(cdiv(nb, 4 / gw)), dim3(RT), 0, s, dims_of(a), a.kw0,
                       (const T *)f0, (const T *)f1, (const T *)f2, (const T *)a.dzi, (const T *)a.dzhi, nb, gw,
                       partial);
}

template <typename T, int V>
void launch_pass1(const HostArgs &a, const RedPlan &pl, const void *f0, const void *f1, const void *f2,
                  double *partial, hipStream_t s)
{
    hipLaunchKernelGGL((reduce_pass1<T, V>), dim3(pl.nb), dim3(RT), 0, s, dims_of(a), pl, (const T *)f0,
                       (const T *)f1, (const T *)f2, partial);
}
}  // namespace

hipError_t launch_reduce(const HostArgs &a, int what, const void *f0, const void *f1, const void *f2,
                         double *out, void *scratch, hipStream_t s)
{
    double *partial = (double *)scratch;
    if ((int64_t)a.jtot * a.ktot >= ((int64_t)1 << 31)) return hipErrorInvalidValue;  // 32-bit piece index
    if (what == 0) {
        const int V = sum_rows_chunk(a, f0, f1, f2), nb = sum_rows_blocks(a);
        if (a.dtype == KL_F32)
            V == 4 ? sums_go<float, 4>(a, nb, f0, f1, f2, partial, s)
                   : sums_go<float, 1>(a, nb, f0, f1, f2, partial, s);
        else
            V == 2 ? sums_go<double, 2>(a, nb, f0, f1, f2, partial, s)
                   : sums_go<double, 1>(a, nb, f0, f1, f2, partial, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(sum_rows_pass2, dim3(1), dim3(RT), 0, s, (const double *)partial, nb, out);
        return hipGetLastError();
    }
    const RedPlan pl = red_plan(a);
    const bool vec = row_chunk(a) > 1;
    if (a.dtype == KL_F32) {
        if (vec)
            launch_pass1<float, 4>(a, pl, f0, f1, f2, partial, s);
        else
            launch_pass1<float, 1>(a, pl, f0, f1, f2, partial, s);
    } else {
        if (vec)
            launch_pass1<double, 2>(a, pl, f0, f1, f2, partial, s);
        else
            launch_pass1<double, 1>(a, pl, f0, f1, f2, partial, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_pass2, dim3(1), dim3(RT2), 0, s, (const double *)partial, pl.nb, out);
    return hipGetLastError();
}

// ---- batched ghost fill and conservation sums (used by the batched form) ----

size_t fill_job_bytes() { return sizeof(FillJob); }

int64_t fill_cell_count(const HostArgs &a)
{
    const int64_t gc = a.gc;
    const int64_t ic = a.itot + 2 * gc, jc = a.jtot + 2 * gc;
    return 2 * ic * jc + 2 * gc * ic * a.ktot + 2 * gc * (int64_t)a.jtot * a.ktot +
           (a.bc != KL_BC_ZPERIODIC ? (int64_t)a.itot * a.jtot : 0);
}

void append_fill_job(const HostArgs &a, void *u, void *v, void *w, bool x_columns, std::vector<char> &jobs,
                     std::vector<int2> &blocks)
{
    const int64_t gc = a.gc;
    const int64_t ic = a.itot + 2 * gc, jc = a.jtot + 2 * gc;
    FillJob j;
    j.d = dims_of(a);
    j.u = u;
    j.v = v;
    j.w = w;
    j.n0 = 2 * ic * jc;
    j.n1 = 2 * gc * ic * a.ktot;
    j.n2 = x_columns ? 2 * gc * (int64_t)a.jtot * a.ktot : 0;
    j.n3 = a.bc != KL_BC_ZPERIODIC ? (int64_t)a.itot * a.jtot : 0;  // the velocity fill: w's wall faces
    const int job = (int)(jobs.size() / sizeof(FillJob));
    const char *p = (const char *)&j;
    jobs.insert(jobs.end(), p, p + sizeof j);
    const unsigned nb = cdiv(j.n0 + j.n1 + j.n2 + j.n3, 256);
    for (unsigned b = 0; b < nb; ++b) blocks.push_back(make_int2(job, (int)b));
}

hipError_t launch_fill_batch(int dtype, const void *jobs, const void *blocks, int nblocks, hipStream_t s)
{
    if (nblocks <= 0) return hipSuccess;
    if (dtype == KL_F32)
        hipLaunchKernelGGL(fill_ghosts_batch_kernel<float>, dim3(nblocks), dim3(256), 0, s, (const FillJob *)jobs,
                           (const int2 *)blocks);
    else
        hipLaunchKernelGGL(fill_ghosts_batch_kernel<double>, dim3(nblocks), dim3(256), 0, s, (const FillJob *)jobs,
                           (const int2 *)blocks);
    return hipGetLastError();
}

size_t sum_job_bytes() { return sizeof(SumJob); }

bool sums_vectorized(const HostArgs &a, const void *ut, const void *vt, const void *wt)
{
    return sum_rows_chunk(a, ut, vt, wt) > 1;
}

void append_sum_job(const HostArgs &a, const void *ut, const void *vt, const void *wt, std::vector<char> &jobs,
                    std::vector<int2> &blocks, std::vector<longlong2> &slots, int64_t *npartials)
{
    const int job = (int)(jobs.size() / sizeof(SumJob));
    SumJob j;
    memset(&j, 0, sizeof j);
    j.d = dims_of(a);
    j.nb = sum_rows_blocks(a);
    const int V = sum_rows_chunk(a, ut, vt, wt), per = a.itot / V >= RT ? 1 : 4 / sum_rows_waves(a, V) * SUM_P;
    j.gw = sum_rows_waves(a, V);
    j.kw0 = a.kw0;
    j.first = *npartials;
    j.f0 = ut;
    j.f1 = vt;
    j.f2 = wt;
    j.dzi = a.dzi;
    j.dzhi = a.dzhi;
    for (int b = 0; b < j.nb; b += per) blocks.push_back(make_int2(job, b));
    longlong2 sl;
    sl.x = j.first;
    sl.y = j.nb;
    slots.push_back(sl);
    *npartials += 3 * (int64_t)j.nb;
    const char *p = (const char *)&j;
    jobs.insert(jobs.end(), p, p + sizeof j);
}

hipError_t launch_sums_batch(int dtype, bool vec, const void *jobs, const void *blocks, int nblocks, double *partials,
                             hipStream_t s)
{
    if (nblocks <= 0) return hipSuccess;
    const dim3 grid((unsigned)nblocks);
    const SumJob *j = (const SumJob *)jobs;
    const int2 *bl = (const int2 *)blocks;
    if (dtype == KL_F32) {
        if (vec)
            hipLaunchKernelGGL((sums_batch_pass1<float, 4>), grid, dim3(RT), 0, s, j, bl, partials);
        else
            hipLaunchKernelGGL((sums_batch_pass1<float, 1>), grid, dim3(RT), 0, s, j, bl, partials);
    } else {
        if (vec)
            hipLaunchKernelGGL((sums_batch_pass1<double, 2>), grid, dim3(RT), 0, s, j, bl, partials);
        else
            hipLaunchKernelGGL((sums_batch_pass1<double, 1>), grid, dim3(RT), 0, s, j, bl, partials);
    }
    return hipGetLastError();
}

hipError_t launch_sums_finish(const void *slots, const double *partials, int nslots, double *out, hipStream_t s)
{
    if (nslots <= 0) return hipSuccess;
    hipLaunchKernelGGL(sums_batch_pass2, dim3((unsigned)nslots), dim3(RT), 0, s, (const longlong2 *)slots, partials,
                       out);
    return hipGetLastError();
}

hipError_t launch_hash(const HostArgs &a, const void *f, uint64_t *out, void *scratch, hipStream_t s)
{
    const Dims d = dims_of(a);
    uint64_t *partial = (uint64_t *)scratch;
    if (a.dtype == KL_F32)
        hipLaunchKernelGGL(hash_pass1<float>, dim3(RB), dim3(RT), 0, s, d, (const float *)f, partial);
    else
        hipLaunchKernelGGL(hash_pass1<double>, dim3(RB), dim3(RT), 0, s, d, (const double *)f, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(hash_pass2, dim3(1), dim3(RT), 0, s, (const uint64_t *)partial, out);
    return hipGetLastError();
}

hipError_t launch_gen_uniform(const HostArgs &a, uint64_t seed, void *u, void *v, void *w, hipStream_t s)
{
    const Dims d = dims_of(a);
    const int nbx = (int)cdiv(a.itot, 256);
    const unsigned nb = (unsigned)nbx * a.jtot * a.ktot;
    if (a.dtype == KL_F32)
        hipLaunchKernelGGL(gen_uniform_kernel<float>, dim3(nb), dim3(256), 0, s, d, seed, (float *)u,
                           (float *)v, (float *)w, nbx);
    else
        hipLaunchKernelGGL(gen_uniform_kernel<double>, dim3(nb), dim3(256), 0, s, d, seed, (double *)u,
                           (double *)v, (double *)w, nbx);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Reductions without allocation.  The pass-1 partials go to a fixed array in
// device memory that the code object brings with it, so the call needs no
// hipMalloc.  Each device holds its own copy until the process ends; its
// address is looked up once per device, with that device current.  In host
// code `scratch` names a host-side stand-in, so only the looked-up address is
// ever handed to a kernel.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[RB * RQ];
constexpr size_t NOALLOC_SCRATCH_BYTES = sizeof(double) * RB * RQ;  // 288 KiB
constexpr int NOALLOC_MAX_DEVICES = 64;

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES];
}  // namespace

}  // namespace kl

extern "C" int kl_reduce_fp64_noalloc(const kl_grid_t *g, int32_t what, const void *f0, const void *f1,
                                      const void *f2, double *out, void *stream)
{
    using namespace kl;
    clear_error();
    int rc = check_grid(g);
    if (rc) return rc;
    if (what != 0 && what != 1) return fail(KL_ERR_INVALID, "what=%d", what);
    if (!out) return fail(KL_ERR_INVALID, "out is NULL");
    if (what == 0 && (!f0 || !f1 || !f2)) return fail(KL_ERR_INVALID, "conservation sums need ut, vt, wt");
    // the partial count is fixed (one row of RQ values per pass-1 block), not
    // a function of the grid; refuse if it ever outgrew the array
    if (reduce_scratch_bytes() > NOALLOC_SCRATCH_BYTES)
        return fail(KL_ERR_INVALID, "reduction needs %zu B of scratch, the fixed array holds %zu B",
                    reduce_scratch_bytes(), NOALLOC_SCRATCH_BYTES);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES)
        return fail(KL_ERR_INVALID, "device %d beyond the %d the fixed scratch table covers", dev,
                    NOALLOC_MAX_DEVICES);
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            e = hipGetSymbolAddress(&g_scratch_ptr[dev], HIP_SYMBOL(scratch));
            if (e != hipSuccess) {
                g_scratch_ptr[dev] = nullptr;
                return hip_fail(e, "hipGetSymbolAddress(scratch)");
            }
        }
        ptr = g_scratch_ptr[dev];
    }
    e = launch_reduce(make_args(g), what, f0, f1, f2, out, ptr, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : hip_fail(e, "reduce_noalloc");
}
