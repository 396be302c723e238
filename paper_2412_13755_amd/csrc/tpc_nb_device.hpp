#pragma once
// Neighbour finding between adjacent pad rows (gfx950): per-segment device
// functions, used by the stage kernels and by the persistent kernel.
//
// Exact definition (the result every enumeration must reproduce): for each
// cluster h of row r in [1, R-2], the pair (d in row r-1, u in row r+1) that
// passes the position windows and the second-difference cuts with the
// smallest q = dy*dy + dz*dz, ties to the smaller u id, then the smaller d id.
// Every floating-point operation is one single-precision rounding: the
// functions below carry "fp contract(off)" and the stage file is compiled
// with -ffp-contract=off, so no multiply-add is fused.
//
// Design: one workgroup per h-row (frame, sector, row) segment.  It bins its
// two neighbouring rows, of up to TPC_LDS_ROW clusters each, into LDS on one
// y-z cell grid sized from the data (the row pair is read once, coalesced,
// and every candidate access is an LDS access); every thread lists the
// clusters of either row in its own cluster's window, and the pairs of a
// wavefront's lists are then scored 64 at a time (mix_query_seg).
//
// Dense rows (a neighbouring row of more than TPC_LDS_ROW clusters, as in a
// continuous-readout time frame with ~10^4 clusters per pad row): the h-row
// and both neighbouring rows are first counting-sorted by z alone into a
// global copy (nb_bin_seg).  The query workgroup then walks its h-row in
// slabs of consecutive sorted clusters (nearby z); a slab's window in z
// selects a contiguous range of each neighbouring row's sorted copy, which
// is binned into LDS exactly as a small row pair, and the slab's clusters
// are searched there.  A slab whose ranges exceed the LDS is halved; a
// slab of the smallest size that still does not fit is searched directly
// in the global sorted copies.  The cells scanned are derived from the
// window and cut intervals with a safety margin (see best_pair), so they
// over-cover the candidates and the exact predicates decide.
#include "tpc_internal.hpp"

namespace tpc_nb {


// Cell index of coordinate v on an axis of n cells starting at v0, 1/edge iw
// (iw = 0 when n = 1).  Monotonic non-decreasing in v; NaN and values below
// the axis go to cell 0, values beyond it (+inf too) to cell n - 1.
// Branch-free: fmaxf returns the number when the other operand is NaN.
__device__ inline int cell_coord(float v, float v0, float iw, int n) {
#pragma clang fp contract(off)
    float c = (v - v0) * iw;
    c = fmaxf(c, 0.0f);
    c = fminf(c, (float)(n - 1));
    return (int)c;                                  // floor for c >= 0
}

// Grid of one row: cell edges >= edge x the window (1.01 by default), at
// most min(n, cap) cells.  ext = (ymin, ymax, zmin, zmax) of the finite
// coordinates.
__device__ inline SegGrid row_grid(float ymin, float ymax, float zmin, float zmax, int n, int cap,
                                   float win_y, float win_z, float edge = 1.01f) {
#pragma clang fp contract(off)
    if (!(ymin <= ymax)) { ymin = 0.f; ymax = 0.f; }
    if (!(zmin <= zmax)) { zmin = 0.f; zmax = 0.f; }
    const int c = n < cap ? n : cap;
    const float ry = ymax - ymin, rz = zmax - zmin;
    const float fz = rz / (edge * win_z), fy = ry / (edge * win_y);
    const int nzmax = fz >= (float)c ? c : (fz >= 1.0f ? (int)fz : 1);
    const int nymax = fy >= (float)c ? c : (fy >= 1.0f ? (int)fy : 1);
    const int nz = nzmax;
    int ny = c / nz;
    if (ny > nymax) ny = nymax;
    if (ny < 1) ny = 1;
    SegGrid g = {ymin, zmin, ny > 1 ? (float)ny / ry : 0.f, nz > 1 ? (float)nz / rz : 0.f, ny, nz, 0, 0};
    return g;
}

// Finite extent of clusters [a, b) (whole workgroup; contains barriers).
__device__ inline void row_extent(const float *__restrict__ y, const float *__restrict__ z, int a, int b,
                                  float (*red)[TPC_BLOCK / TPC_WAVE], float ext[4]) {
    float ymin = INFINITY, ymax = -INFINITY, zmin = INFINITY, zmax = -INFINITY;
    for (int i = a + (int)threadIdx.x; i < b; i += TPC_BLOCK) {
        const float yv = y[i], zv = z[i];
        if (isfinite(yv)) { ymin = fminf(ymin, yv); ymax = fmaxf(ymax, yv); }
        if (isfinite(zv)) { zmin = fminf(zmin, zv); zmax = fmaxf(zmax, zv); }
    }
    ymin = wave_min(ymin); ymax = wave_max(ymax);
    zmin = wave_min(zmin); zmax = wave_max(zmax);
    const int wid = threadIdx.x / TPC_WAVE, lane = threadIdx.x & (TPC_WAVE - 1);
    __syncthreads();
    if (lane == 0) { red[0][wid] = ymin; red[1][wid] = ymax; red[2][wid] = zmin; red[3][wid] = zmax; }
    __syncthreads();
    ymin = red[0][0]; ymax = red[1][0]; zmin = red[2][0]; zmax = red[3][0];
    for (int w = 1; w < TPC_BLOCK / TPC_WAVE; ++w) {
        ymin = fminf(ymin, red[0][w]); ymax = fmaxf(ymax, red[1][w]);
        zmin = fminf(zmin, red[2][w]); zmax = fmaxf(zmax, red[3][w]);
    }
    ext[0] = ymin; ext[1] = ymax; ext[2] = zmin; ext[3] = zmax;
}

// Finite z extent of clusters [a, b) (whole workgroup; contains barriers).
__device__ inline void row_zextent(const float *__restrict__ z, int a, int b, float (*red)[TPC_BLOCK / TPC_WAVE],
                                   float &zlo, float &zhi) {
    float zmin = INFINITY, zmax = -INFINITY;
    for (int i = a + (int)threadIdx.x; i < b; i += TPC_BLOCK) {
        const float zv = z[i];
        if (isfinite(zv)) { zmin = fminf(zmin, zv); zmax = fmaxf(zmax, zv); }
    }
    zmin = wave_min(zmin);
    zmax = wave_max(zmax);
    const int wid = threadIdx.x / TPC_WAVE, lane = threadIdx.x & (TPC_WAVE - 1);
    __syncthreads();
    if (lane == 0) { red[0][wid] = zmin; red[1][wid] = zmax; }
    __syncthreads();
    zmin = red[0][0];
    zmax = red[1][0];
    for (int w = 1; w < TPC_BLOCK / TPC_WAVE; ++w) {
        zmin = fminf(zmin, red[0][w]);
        zmax = fmaxf(zmax, red[1][w]);
    }
    zlo = zmin;
    zhi = zmax;
}

// Counting sort of clusters [a, b) by cell of grid g (whole workgroup;
// contains barriers).  Writes y, z, global id in cell order to
// dy/dz/did[obase + k] and cell starts cs[c] = obase + first position of
// cell c, cs[cells] = obase + n.  cnt: LDS scratch of >= cells ints.
__device__ inline void row_sort(const float *__restrict__ y, const float *__restrict__ z, int a, int b,
                                const SegGrid &g, int *cnt, int *scan_sh, float *dy, float *dz, int32_t *did,
                                int32_t *cs, int obase) {
#pragma clang fp contract(off)
    const int tid = threadIdx.x;
    const int cells = g.ny * g.nz;
    for (int c = tid; c < cells; c += TPC_BLOCK) cnt[c] = 0;
    __syncthreads();
    for (int i = a + tid; i < b; i += TPC_BLOCK) {
        const int c = cell_coord(y[i], g.y0, g.iwy, g.ny) * g.nz + cell_coord(z[i], g.z0, g.iwz, g.nz);
        atomicAdd(&cnt[c], 1);
    }
    __syncthreads();
    // exclusive scan: each thread owns a contiguous run of cells
    const int per = (cells + TPC_BLOCK - 1) / TPC_BLOCK;
    const int c0 = tid * per;
    int c1 = c0 + per;
    if (c1 > cells) c1 = cells;
    int local = 0;
    for (int c = c0; c < c1; ++c) local += cnt[c];
    int total;
    int run = block_exclusive_scan(local, scan_sh, &total);
    for (int c = c0; c < c1; ++c) {
        const int v = cnt[c];
        cnt[c] = obase + run;         // becomes the scatter cursor
        cs[c] = obase + run;
        run += v;
    }
    if (tid == 0) cs[cells] = obase + (b - a);
    __syncthreads();
    for (int i = a + tid; i < b; i += TPC_BLOCK) {
        const float yv = y[i], zv = z[i];
        const int c = cell_coord(yv, g.y0, g.iwy, g.ny) * g.nz + cell_coord(zv, g.z0, g.iwz, g.nz);
        const int slot = atomicAdd(&cnt[c], 1);
        dy[slot] = yv;
        dz[slot] = zv;
        did[slot] = i;
    }
    __syncthreads();
}

// Rows of at most this many clusters are binned in LDS by the query
// workgroup itself; an h-row with a larger neighbouring row is dense.
#define TPC_LDS_ROW 1024

__device__ inline int seg_size(const int32_t *off, int s) { return off[s + 1] - off[s]; }

// Is `seg` a non-empty interior h-row with a neighbouring row of more than
// TPC_LDS_ROW clusters (searched in slabs over the z-sorted rows)?
__device__ inline bool dense_hrow(const int32_t *off, int seg, int n_rows) {
    const int r = seg % n_rows;
    if (r == 0 || r == n_rows - 1 || seg_size(off, seg) == 0) return false;
    return seg_size(off, seg - 1) > TPC_LDS_ROW || seg_size(off, seg + 1) > TPC_LDS_ROW;
}

// Grid of a row in z alone: min(n, cap) cells of equal length over the
// finite z extent (ny = 1, so every y falls in the one cell column).
__device__ inline SegGrid zrow_grid(float zmin, float zmax, int n, int cap) {
#pragma clang fp contract(off)
    if (!(zmin <= zmax)) { zmin = 0.f; zmax = 0.f; }
    const int c = n < cap ? n : cap;
    const float rz = zmax - zmin;
    const int nz = (rz > 0.f && c > 1) ? c : 1;
    return SegGrid{0.f, zmin, 0.f, nz > 1 ? (float)nz / rz : 0.f, 1, nz, 0, 0};
}

// Counting sort of clusters [a, b) by cell of grid g through an LDS
// permutation (whole workgroup; contains barriers): the same cell order as
// row_sort, but the scatter writes 16-bit local indices into LDS and the
// sorted copy is then written in position order (coalesced stores, reads
// gathered from the row), so no partially written cache lines go to HBM.
// n = b - a <= TPC_BIN_PERM.  g has one cell column (a zrow_grid, ny = 1),
// so the cell is z's alone and y is read only by the final gather.
#ifndef TPC_BIN_PERM
#define TPC_BIN_PERM 17408   // 51 KB of LDS: three binning workgroups per CU
#endif
__device__ inline void row_sort_perm(const float *__restrict__ y, const float *__restrict__ z, int a, int b,
                                     const SegGrid &g, int *cnt, int *scan_sh, uint16_t *perm,
                                     float *__restrict__ dy, float *__restrict__ dz, int32_t *__restrict__ did,
                                     int32_t *__restrict__ cs, int obase) {
#pragma clang fp contract(off)
    const int tid = threadIdx.x;
    const int cells = g.ny * g.nz;
    for (int c = tid; c < cells; c += TPC_BLOCK) cnt[c] = 0;
    __syncthreads();
    for (int i = a + tid; i < b; i += TPC_BLOCK) atomicAdd(&cnt[cell_coord(z[i], g.z0, g.iwz, g.nz)], 1);
    __syncthreads();
    const int per = (cells + TPC_BLOCK - 1) / TPC_BLOCK;
    const int c0 = tid * per;
    int c1 = c0 + per;
    if (c1 > cells) c1 = cells;
    int local = 0;
    for (int c = c0; c < c1; ++c) local += cnt[c];
    int total;
    int run = block_exclusive_scan(local, scan_sh, &total);
    for (int c = c0; c < c1; ++c) {
        const int v = cnt[c];
        cnt[c] = run;                 // becomes the scatter cursor
        cs[c] = obase + run;
        run += v;
    }
    if (tid == 0) cs[cells] = obase + (b - a);
    __syncthreads();
    for (int i = a + tid; i < b; i += TPC_BLOCK) {
        const int c = cell_coord(z[i], g.z0, g.iwz, g.nz);
        perm[atomicAdd(&cnt[c], 1)] = (uint16_t)(i - a);
    }
    __syncthreads();
    // the gathers through the permutation are random within the row: z
    // first, then y, so that a workgroup's reads span one row array at a
    // time (the rows in flight on an XCD then miss its L2 less)
    for (int k = tid; k < b - a; k += TPC_BLOCK) {
        const int i = a + perm[k];
        dz[obase + k] = z[i];
        did[obase + k] = i;
    }
    __syncthreads();
    for (int k = tid; k < b - a; k += TPC_BLOCK) dy[obase + k] = y[a + perm[k]];
    __syncthreads();
}

// z-sorted global copy of segment `seg`, made only when it is a dense h-row
// or a neighbouring row of one (whole workgroup; contains barriers; L: LDS
// scratch).  With PERM the sort goes through an LDS permutation (rows of up
// to TPC_BIN_PERM clusters; larger rows scatter directly).
struct BinLds {
    int cnt[TPC_CELL_CAP];
    float red[4][TPC_BLOCK / TPC_WAVE];
    int scan_sh[TPC_BLOCK / TPC_WAVE];
};
struct BinLdsPerm : BinLds {
    uint16_t perm[TPC_BIN_PERM];
};

// Does segment `seg` need a z-sorted copy (a dense h-row or a neighbouring
// row of one)?
__device__ inline bool nb_bin_needed(const int32_t *off, int seg, int n_rows) {
    const int r = seg % n_rows;
    return dense_hrow(off, seg, n_rows) || (r >= 1 && dense_hrow(off, seg - 1, n_rows)) ||
           (r <= n_rows - 2 && dense_hrow(off, seg + 1, n_rows));
}

template <class LDS>
__device__ inline void nb_bin_seg(int seg, int n_rows, const int32_t *__restrict__ off,
                                  const float *__restrict__ y, const float *__restrict__ z, float win_y,
                                  float win_z, SegGrid *__restrict__ grid, int32_t *__restrict__ cstart,
                                  float *__restrict__ sy, float *__restrict__ sz,
                                  int32_t *__restrict__ sid, LDS &L) {
#pragma clang fp contract(off)
    int *cnt = L.cnt;
    float (*red)[TPC_BLOCK / TPC_WAVE] = L.red;
    int *scan_sh = L.scan_sh;
    if (!nb_bin_needed(off, seg, n_rows)) return;
    __syncthreads();                 // LDS reuse across calls in a persistent loop
    const int a = off[seg], b = off[seg + 1], n = b - a;
    const int base = a + seg;
    if (n == 0) {
        if (threadIdx.x == 0) {
            SegGrid g = {0.f, 0.f, 0.f, 0.f, 0, 0, 0, 0};
            grid[seg] = g;
            cstart[base] = a;
        }
        return;
    }
    float zlo, zhi;
    row_zextent(z, a, b, red, zlo, zhi);
    const SegGrid g = zrow_grid(zlo, zhi, n, TPC_CELL_CAP);
    if (threadIdx.x == 0) grid[seg] = g;
    if constexpr (sizeof(LDS) >= sizeof(BinLdsPerm)) {
        if (n <= TPC_BIN_PERM) {
            row_sort_perm(y, z, a, b, g, cnt, scan_sh, L.perm, sy, sz, sid, cstart + base, a);
            return;
        }
    }
    row_sort(y, z, a, b, g, cnt, scan_sh, sy, sz, sid, cstart + base, a);
}

struct Best {
    float q;
    int32_t u, d;
};

// Lexicographic (q, u, d) order against the best so far (none yet: u < 0).
__device__ inline bool better(float q, int32_t u, int32_t d, const Best &b) {
    const bool tie = q == b.q;
    return (b.u < 0) | (q < b.q) | (tie & (u < b.u)) | (tie & (u == b.u) & (d < b.d));
}

// Best (up, down) pair for cluster (yh, zh) in the cell-sorted up row (UY,
// UZ, UI, UCS, gu) and down row (D...).  UCS[c] indexes the first cluster of
// cell c in UY/UZ/UI; a stored id k stands for cluster ubase + k (dbase + k
// in the down row).  Every operation is one single-precision rounding, and
// the predicates are evaluated on exactly the operands of the definition.
// The down row lies A rows below h and the up row B rows above (A, B in
// {1, 2}): with ay = y_u - y_h and by = y_h - y_d (z likewise) a pair passes
// |ay| <= B win, |by| <= A win and |dy| <= cut for the second difference
// dy = g (ay / B - by / A), g = 2 / (A + B), scored by q = dy*dy + dz*dz.
// At A = B = 1 every scale factor is exactly 1 and dy = ay - by, the
// adjacent-row definition; B win, ay / B and by / A are exact for the other
// distances (powers of two) and g = 2/3 is the rounded constant.
//
// Enumeration: the down-row clusters in h's window are collected first (up
// to TPC_NB_DLIST in registers); then every up-row cluster in the window is
// paired with that list.  If more down clusters are in the window, each up
// candidate instead scans the down-row cells that overlap the cut interval
// around its straight-line prediction c = h - (A / B)(u - h), of half-width
// A (A + B) / 2 cut.  Cells scanned are those overlapping the window (or
// cut) interval widened by a margin m far above the rounding of the
// predicates and of c; as cell_coord is monotonic, every cluster that can
// pass the exact predicates is visited.  A cluster h with a non-finite
// coordinate fails every window, so it is skipped.
#define TPC_NB_DLIST 8

template <int A = 1, int B = 1, class FP, class IP, class CP>
__device__ __forceinline__ Best best_pair(float yh, float zh, FP UY, FP UZ, IP UI, CP UCS, const SegGrid &gu,
                                 int32_t ubase, FP DY, FP DZ, IP DI, CP DCS, const SegGrid &gd,
                                 int32_t dbase, float win_y, float win_z, float cut_y, float cut_z) {
#pragma clang fp contract(off)
    static_assert(A >= 1 && A <= 2 && B >= 1 && B <= 2, "partners one or two rows away");
    constexpr float fa = (float)A, fb = (float)B;
    constexpr float g = 2.0f / (float)(A + B);
    constexpr float kw = A > B ? fa : fb;              // widest window, in windows
    constexpr float kc = (float)(A * (A + B)) / 2.0f;  // cut interval of the down row, in cuts
    constexpr float rab = fa / fb;                     // prediction slope of the down row
    Best best = {0.f, -1, -1};
    if (gu.ny <= 0 || gd.ny <= 0 || !isfinite(yh) || !isfinite(zh)) return best;
    const float my = 1e-5f * (fabsf(yh) + kw * win_y + kc * cut_y) + 1e-6f;
    const float mz = 1e-5f * (fabsf(zh) + kw * win_z + kc * cut_z) + 1e-6f;
    const float wdy = fa * win_y + my, wdz = fa * win_z + mz;
    const float wuy = fb * win_y + my, wuz = fb * win_z + mz;
    const float ky = kc * cut_y + my, kz = kc * cut_z + mz;
    // down clusters in the window (by / A kept)
    float lb[TPC_NB_DLIST][2];
    int32_t ld[TPC_NB_DLIST];
#pragma unroll
    for (int j = 0; j < TPC_NB_DLIST; ++j) { lb[j][0] = 0.f; lb[j][1] = 0.f; ld[j] = -1; }
    int nd = 0;
    {
        const int y0 = cell_coord(yh - wdy, gd.y0, gd.iwy, gd.ny), y1 = cell_coord(yh + wdy, gd.y0, gd.iwy, gd.ny);
        const int z0 = cell_coord(zh - wdz, gd.z0, gd.iwz, gd.nz), z1 = cell_coord(zh + wdz, gd.z0, gd.iwz, gd.nz);
        for (int iy = y0; iy <= y1; ++iy) {
            const int e0 = DCS[iy * gd.nz + z0];
            const int e1 = DCS[iy * gd.nz + z1 + 1];
            for (int kd = e0; kd < e1; ++kd) {
                const float by = yh - DY[kd];
                const float bz = zh - DZ[kd];
                if (!(fabsf(by) <= fa * win_y && fabsf(bz) <= fa * win_z)) continue;
                const int32_t d = dbase + (int32_t)DI[kd];
                const float sy = by / fa, sz = bz / fa;
#pragma unroll
                for (int j = 0; j < TPC_NB_DLIST; ++j)
                    if (nd == j) { lb[j][0] = sy; lb[j][1] = sz; ld[j] = d; }
                ++nd;
            }
        }
    }
    if (nd == 0) return best;
    const bool listed = nd <= TPC_NB_DLIST;
    const int yu0 = cell_coord(yh - wuy, gu.y0, gu.iwy, gu.ny), yu1 = cell_coord(yh + wuy, gu.y0, gu.iwy, gu.ny);
    const int zu0 = cell_coord(zh - wuz, gu.z0, gu.iwz, gu.nz), zu1 = cell_coord(zh + wuz, gu.z0, gu.iwz, gu.nz);
    for (int iyu = yu0; iyu <= yu1; ++iyu) {
        const int ue0 = UCS[iyu * gu.nz + zu0];
        const int ue1 = UCS[iyu * gu.nz + zu1 + 1];
        for (int ku = ue0; ku < ue1; ++ku) {
            const float ay = UY[ku] - yh;
            const float az = UZ[ku] - zh;
            if (!(fabsf(ay) <= fb * win_y && fabsf(az) <= fb * win_z)) continue;
            const int32_t u = ubase + (int32_t)UI[ku];
            const float ty = ay / fb, tz = az / fb;
            if (listed) {
#pragma unroll
                for (int j = 0; j < TPC_NB_DLIST; ++j) {
                    const float ey = ty - lb[j][0];
                    const float ez = tz - lb[j][1];
                    const float dy = g * ey;
                    const float dz = g * ez;
                    if (j < nd && fabsf(dy) <= cut_y && fabsf(dz) <= cut_z) {
                        const float qy = dy * dy;
                        const float qz = dz * dz;
                        const float q = qy + qz;
                        if (better(q, u, ld[j], best)) { best.q = q; best.u = u; best.d = ld[j]; }
                    }
                }
                continue;
            }
            const float cy = yh - rab * ay, cz = zh - rab * az;
            const int yd0 = cell_coord(cy - ky, gd.y0, gd.iwy, gd.ny);
            const int yd1 = cell_coord(cy + ky, gd.y0, gd.iwy, gd.ny);
            const int zd0 = cell_coord(cz - kz, gd.z0, gd.iwz, gd.nz);
            const int zd1 = cell_coord(cz + kz, gd.z0, gd.iwz, gd.nz);
            for (int iyd = yd0; iyd <= yd1; ++iyd) {
                const int de0 = DCS[iyd * gd.nz + zd0];
                const int de1 = DCS[iyd * gd.nz + zd1 + 1];
                for (int kd = de0; kd < de1; ++kd) {
                    const float by = yh - DY[kd];
                    const float bz = zh - DZ[kd];
                    if (!(fabsf(by) <= fa * win_y && fabsf(bz) <= fa * win_z)) continue;
                    const float ey = ty - by / fa;
                    const float ez = tz - bz / fa;
                    const float dy = g * ey;
                    const float dz = g * ez;
                    if (!(fabsf(dy) <= cut_y && fabsf(dz) <= cut_z)) continue;
                    const float qy = dy * dy;
                    const float qz = dz * dz;
                    const float q = qy + qz;
                    const int32_t d = dbase + (int32_t)DI[kd];
                    if (better(q, u, d, best)) { best.q = q; best.u = u; best.d = d; }
                }
            }
        }
    }
    return best;
}

// LDS form of the row pair of a dense row's slab: both ranges of up to ROW
// clusters each, with finer cells than the global form (up to 4 per cluster,
// CELLS per row) so that the cells around h hold few candidates.
template <int ROW, int CELLS>
struct PairLdsT {
    float y[2 * ROW + 1], z[2 * ROW + 1];
    uint16_t rel[2 * ROW];                  // cluster id minus its row's first id
    alignas(16) uint32_t cs[CELLS];         // cell starts of both rows (< CELLS each), concatenated, two to a word
    float red[8][TPC_BLOCK / TPC_WAVE];
    int scan_sh[TPC_BLOCK / TPC_WAVE];
};

// Bins a down row of n0 clusters and an up row of n1 clusters with one LDS
// counting sort over the concatenated cell range (whole workgroup; contains
// barriers).  src(k, y, z, rel) gives cluster k of the pair (the down row
// first) and its id relative to its row's first cluster.  On return the
// down row occupies cells [0, C0) with grid gd, the up row cells C0 + [0, C1)
// with grid gu, and cell c holds positions [cs[c], cs[c+1]) of y/z/rel.
// Cell edges are at least edge_d (down row) and edge_u (up row) windows.
__device__ inline int pair_cell(float yv, float zv, const SegGrid &g) {
    return cell_coord(yv, g.y0, g.iwy, g.ny) * g.nz + cell_coord(zv, g.z0, g.iwz, g.nz);
}

template <int CELLS>
__device__ inline SegGrid pair_grid(float ymin, float ymax, float zmin, float zmax, int n, float win_y,
                                    float win_z, float edge) {
    if (n == 0) return SegGrid{0.f, 0.f, 0.f, 0.f, 0, 0, 0, 0};
    const int cap = 4 * n < CELLS ? 4 * n : CELLS - 1;
    return row_grid(ymin, ymax, zmin, zmax, cap, cap, win_y, win_z, edge);
}

// Two position ranges of the z-sorted copies (sy, sz, sid): [pa0, pa0 + n0)
// of the down row, whose first cluster id is base0, then [pa1, ...) of the
// up row (base1).
struct SortedPairSrc {
    const float *sy, *sz;
    const int32_t *sid;
    int pa0, n0, pa1, base0, base1;
    __device__ void operator()(int k, float &vy, float &vz, uint16_t &rel) const {
        const int p = k < n0 ? pa0 + k : pa1 + (k - n0);
        vy = sy[p];
        vz = sz[p];
        rel = (uint16_t)(sid[p] - (k < n0 ? base0 : base1));
    }
};

template <int ROW, int CELLS, class Src>
__device__ __forceinline__ void pair_bin(const Src &src, int n0, int n1, float win_y, float win_z, float edge_d,
                                float edge_u,
                                PairLdsT<ROW, CELLS> &L, SegGrid &gd, SegGrid &gu, int &C0) {
#pragma clang fp contract(off)
    constexpr int PT = 2 * ROW / TPC_BLOCK;      // row-pair clusters per thread
    constexpr int PC = CELLS / TPC_BLOCK;        // cell words per thread
    static_assert(PC % 4 == 0, "cell words in 16-byte groups");
    static_assert(2 * ROW < 65536, "16-bit cell starts");
    auto bump = [&](int c) {                     // cs[c]++, the value before
        const int sh = 16 * (c & 1);
        return (int)((atomicAdd(&L.cs[c >> 1], 1u << sh) >> sh) & 0xFFFFu);
    };
    const int tid = threadIdx.x;
    const int nt = n0 + n1;
    // both rows are read once, into registers (one global round trip); the
    // groups of TPC_BLOCK clusters that the pair does not reach are skipped
    // by the whole workgroup
    float vy[PT], vz[PT];
    uint16_t vr[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int k = tid + j * TPC_BLOCK;
        vy[j] = 0.f;
        vz[j] = 0.f;
        vr[j] = 0;
        if (j * TPC_BLOCK < nt && k < nt) src(k, vy[j], vz[j], vr[j]);
    }
    int4 *cs4 = reinterpret_cast<int4 *>(L.cs) + tid * (PC / 4);
#pragma unroll
    for (int q = 0; q < PC / 4; ++q) cs4[q] = make_int4(0, 0, 0, 0);
    // finite extents of both rows
    float e[8] = {INFINITY, -INFINITY, INFINITY, -INFINITY, INFINITY, -INFINITY, INFINITY, -INFINITY};
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        if (j * TPC_BLOCK >= nt) break;
        const int k = tid + j * TPC_BLOCK;
        const bool fy = k < nt && isfinite(vy[j]), fz = k < nt && isfinite(vz[j]);
        if (k < n0) {
            if (fy) { e[0] = fminf(e[0], vy[j]); e[1] = fmaxf(e[1], vy[j]); }
            if (fz) { e[2] = fminf(e[2], vz[j]); e[3] = fmaxf(e[3], vz[j]); }
        } else {
            if (fy) { e[4] = fminf(e[4], vy[j]); e[5] = fmaxf(e[5], vy[j]); }
            if (fz) { e[6] = fminf(e[6], vz[j]); e[7] = fmaxf(e[7], vz[j]); }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = (j & 1) ? wave_max(e[j]) : wave_min(e[j]);
    const int wid = tid / TPC_WAVE, lane = tid & (TPC_WAVE - 1);
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) L.red[j][wid] = e[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float v = L.red[j][0];
#pragma unroll
        for (int w = 1; w < TPC_BLOCK / TPC_WAVE; ++w)
            v = (j & 1) ? fmaxf(v, L.red[j][w]) : fminf(v, L.red[j][w]);
        e[j] = v;
    }
    gd = pair_grid<CELLS>(e[0], e[1], e[2], e[3], n0, win_y, win_z, edge_d);
    gu = pair_grid<CELLS>(e[4], e[5], e[6], e[7], n1, win_y, win_z, edge_u);
    C0 = gd.ny * gd.nz;
    // count cell c into cs[c + 2]
    int cell[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        cell[j] = 0;
        if (j * TPC_BLOCK >= nt) break;
        const int k = tid + j * TPC_BLOCK;
        const SegGrid g = k < n0 ? gd : gu;
        cell[j] = (k < n0 ? 0 : C0) + pair_cell(vy[j], vz[j], g);
        if (k < nt) bump(cell[j] + 2);
    }
    __syncthreads();
    // inclusive scan: cs[c + 1] = first position of cell c (the counts of
    // cells below c are in cs[2 .. c + 1]).  Each thread takes PC words of
    // the array as they lie, whatever the number of cells: 16-byte accesses
    // and no loop (a run per thread, word by word, conflicted on the banks).
    uint32_t w[PC];
    uint32_t local = 0;                          // (its halves' sums do not overflow: 2 ROW clusters)
#pragma unroll
    for (int q = 0; q < PC / 4; ++q) {
        const int4 v = cs4[q];
        w[4 * q] = (uint32_t)v.x;
        w[4 * q + 1] = (uint32_t)v.y;
        w[4 * q + 2] = (uint32_t)v.z;
        w[4 * q + 3] = (uint32_t)v.w;
        local += w[4 * q] + w[4 * q + 1] + w[4 * q + 2] + w[4 * q + 3];
    }
    int total;
    uint32_t run = (uint32_t)block_exclusive_scan((int)((local & 0xFFFFu) + (local >> 16)), L.scan_sh, &total);
#pragma unroll
    for (int q = 0; q < PC; ++q) {
        const uint32_t lo = run + (w[q] & 0xFFFFu);
        run = lo + (w[q] >> 16);
        w[q] = lo | run << 16;
    }
#pragma unroll
    for (int q = 0; q < PC / 4; ++q)
        cs4[q] = make_int4((int)w[4 * q], (int)w[4 * q + 1], (int)w[4 * q + 2], (int)w[4 * q + 3]);
    __syncthreads();
    // scatter; the cursor of cell c moves from its start to its end, which
    // leaves cs[c] = start of cell c for every c in [0, C]
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        if (j * TPC_BLOCK >= nt) break;
        const int k = tid + j * TPC_BLOCK;
        if (k < nt) {
            const int slot = bump(cell[j] + 1);
            L.y[slot] = vy[j];
            L.z[slot] = vz[j];
            L.rel[slot] = vr[j];
        }
    }
    __syncthreads();
}

// Does h-row `seg` (an interior, non-empty row) have neighbour rows that fit
// the small mixed LDS form (mix_query_seg)?
#define TPC_MIX_N 1152
__device__ inline bool small_pair(const int32_t *off, int seg) {
    const int n0 = seg_size(off, seg - 1), n1 = seg_size(off, seg + 1);
    return n0 <= TPC_LDS_ROW && n1 <= TPC_LDS_ROW && n0 + n1 <= TPC_MIX_N;
}

// The first and the last row of a sector have no triplets: writes that, and
// returns whether `seg` is one (whole workgroup).
__device__ inline bool inner_row(int seg, int n_rows) {
    const int r = seg % n_rows;
    return r > 0 && r < n_rows - 1;
}
__device__ inline bool edge_row(int seg, const int32_t *off, int n_rows, int32_t *up, int32_t *dn) {
    if (inner_row(seg, n_rows)) return false;
    for (int i = off[seg] + threadIdx.x; i < off[seg + 1]; i += TPC_BLOCK) { up[i] = -1; dn[i] = -1; }
    return true;
}

// Is `seg` an h-row that the small mixed form does not take (of the large
// form, or dense)?
__device__ inline bool rest_hrow(const int32_t *off, int seg, int n_rows) {
    const int r = seg % n_rows;
    return r > 0 && r < n_rows - 1 && seg_size(off, seg) > 0 && !small_pair(off, seg);
}

// Tunables of the dense-row search: h clusters per slab (the slab's
// clusters are consecutive in the z-sorted h-row), the smallest slab before
// the global fallback, the row-pair LDS size of a slab, and the LDS cell
// edges of a slab's down and up rows in windows (the down row is only
// searched around predictions, in boxes of twice the cuts; the up row in
// windows).
#ifndef TPC_NB_SLAB
#define TPC_NB_SLAB 512
#endif
#define TPC_NB_LIST 19        // (as many as four workgroups per CU leave room for)
#ifndef TPC_NB_SLAB_MIN
#define TPC_NB_SLAB_MIN 64
#endif
#ifndef TPC_NB_DENSE_ROW
#define TPC_NB_DENSE_ROW 1024
#endif
#ifndef TPC_NB_DENSE_CELLS
#define TPC_NB_DENSE_CELLS 2048
#endif
#ifndef TPC_NB_DENSE_EDGE_D
#define TPC_NB_DENSE_EDGE_D 0.18f
#endif
#ifndef TPC_NB_DENSE_EDGE_U
#define TPC_NB_DENSE_EDGE_U 0.25f
#endif
// LDS of a dense-row workgroup: the slab's row pair and the slab's results
// (up id << 16 | down id relative to their rows, all ones for none), which
// are written out once the slab is searched.
template <int ROW, int CELLS>
struct DenseLdsT : PairLdsT<ROW, CELLS> {
    uint32_t res[TPC_NB_SLAB];
    uint16_t list[TPC_NB_LIST][TPC_BLOCK];   // per thread: up clusters in its windows, to be searched from
};
using DenseLds = DenseLdsT<TPC_NB_DENSE_ROW, TPC_NB_DENSE_CELLS>;

// Positions [x, y) of the z-sorted copy of a row (grid g, cell starts cs)
// that hold every cluster with z in [lo, hi] (whole cells: cell_coord is
// monotonic, so a cluster with z in the interval lies in a cell between
// those of lo and hi).
__device__ inline int2 zrange(const SegGrid &g, const int32_t *cs, float lo, float hi) {
    if (g.ny <= 0) return make_int2(0, 0);
    const int c0 = cell_coord(lo, g.z0, g.iwz, g.nz), c1 = cell_coord(hi, g.z0, g.iwz, g.nz);
    return make_int2(cs[c0], cs[c1 + 1]);
}

// Search of one slab (clusters [pb, pb + pn) of the h-row's z-sorted copy)
// whose row pair is binned in L (whole workgroup): the result of
// best_pair<1, 1> for every cluster h, by the same single-precision
// operations on a pruned set of candidates.  A lane takes clusters h of the
// slab in turn (consecutive lanes, consecutive positions: nearby z) and walks
// the up-row cells of h's window; for every u in the window it scans the
// down-row cells of the box around the prediction 2h - u.  Once a passing
// triplet of score q* is known the box half-widths shrink from the cuts to
// sqrt(q*) (1 + 1e-4) plus the rounding margin: a down cluster outside has
// |dy| or |dz| above sqrt(q*), so fl(dy^2) + fl(dz^2) > q* (rounding is
// monotonic and both squares are >= 0) and it can neither beat nor tie the
// best, whose lexicographic order (q, then u id, then d id) is kept
// exactly.
//
// A thread has two clusters of the slab.  Bound by vector instructions, so
// the walk over a window's up clusters and the searches of their boxes are
// loops of their own, each iteration of which does what most lanes need: the
// walk reads two candidates and lists those in the window (up to TPC_NB_LIST,
// an LDS column per thread); then each round of the search, for a lane whose
// box is exhausted, sets up the next listed cluster's, steps to a row of
// cells with candidates, and scores two of them.  (One flat loop over both,
// in which every lane went through the window test, the box set-up and the
// row steps: 14.0 ms of a continuous-readout frame's 6.4 10^7 clusters, now
// 10.6.)  A window's rows of cells are walked from h's own outwards: a track
// moves little in y from one pad row to the next, so its partner, after
// which the boxes are small, comes among the first.  A down candidate c at
// t = (y_c - y_h, z_c - z_h) is scored with d_y = a_y + t_y, equal (rounding
// included) to a_y - (y_h - y_d) since fl(y_h - y_d) = -fl(y_d - y_h).  The
// best so far is one 64-bit key (bits of q, then the up and down ids, 16
// bits each), so the lexicographic order is one unsigned comparison (q >= 0,
// whose bit patterns order as its values) and the test carries no branches.
//
// Cell ranges are computed in cell units: the window's or the prediction's
// cell coordinate is (y_h - y0) iw (minus a_y iw for the prediction), its
// half-width (w + m) iw plus e = 1e-6 (|y0| iw + 1) cells, where w is the
// window or min(cut, sqrt(q*) (1 + 1e-4)).  These products round
// differently from cell_coord at the range's edge by a few units of 2^-24
// of (|y_h| + |y0| + w) iw, which m (1e-5 of |y_h| + window + cut) and e
// cover, so every cluster that can pass lies in the cells scanned.  The
// square root of the box set-up is the hardware estimate (a few ulp at
// most; a denormal q* may give 0, which only shrinks the box to its
// rounding margin, still far above sqrt(q*)): the 1e-4 widening covers it.
__device__ inline int cell_in(float c, float nmax) { return (int)__builtin_amdgcn_fmed3f(c, 0.0f, nmax); }

template <int ROW, int CELLS>
__device__ __forceinline__ void slab_search(int pb, int pn, const float *__restrict__ sy, const float *__restrict__ sz,
                                   const int32_t *__restrict__ sid, int32_t baseu, int32_t based,
                                   const SegGrid &gu, const SegGrid &gd, int C0, float win_y, float win_z,
                                   float cut_y, float cut_z, int32_t *__restrict__ up,
                                   int32_t *__restrict__ dn, DenseLdsT<ROW, CELLS> &L) {
#pragma clang fp contract(off)
    static_assert(TPC_NB_SLAB == 2 * TPC_BLOCK, "two clusters of the slab per thread");
    static_assert(2 * ROW <= 2048, "11-bit positions");
    typedef uint16_t __attribute__((may_alias)) cell16;
    const float *Y = L.y, *Z = L.z;
    const uint16_t *R = L.rel;
    const cell16 *DCS = reinterpret_cast<const cell16 *>(L.cs), *UCS = DCS + C0;
    const bool grids = gu.ny > 0 && gd.ny > 0;
    constexpr uint64_t NONE = (0x7F800000ull << 32) | 0xFFFFFFFFull;
    const float edy = 1e-6f * (fabsf(gd.y0) * gd.iwy + 1.0f), edz = 1e-6f * (fabsf(gd.z0) * gd.iwz + 1.0f);
    const float euy = 1e-6f * (fabsf(gu.y0) * gu.iwy + 1.0f), euz = 1e-6f * (fabsf(gu.z0) * gu.iwz + 1.0f);
    const float dny = (float)(gd.ny - 1), dnz = (float)(gd.nz - 1);
    const float uny = (float)(gu.ny - 1), unz = (float)(gu.nz - 1);
    const float wcy = win_y + cut_y, wcz = win_z + cut_z;
    const int tid = threadIdx.x;
    float yv[2], zv[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int j = tid + s * TPC_BLOCK;
        yv[s] = j < pn ? sy[pb + j] : NAN;
        zv[s] = j < pn ? sz[pb + j] : NAN;
    }
    uint64_t best = NONE;
    int cur = 0, n = 0;                           // whose best it is; entries in the list
    float yh = yv[0], zh = zv[0];
    auto result = [&](int s) { L.res[tid + s * TPC_BLOCK] = best != NONE ? (uint32_t)best : 0xFFFFFFFFu; };
    // the listed up clusters' boxes in the down row
    auto search = [&]() {
        float my = 0.f, mz = 0.f, hy = 0.f, hz = 0.f, ay = 0.f, az = 0.f;
        uint32_t urs = 0;
        int i = 0, yd = 0, yd1 = -1, zd0 = 0, zd1 = 0, kd = 0, e1 = 0;
        while (__ballot(kd < e1 || yd < yd1 || i < n)) {
            if (kd == e1) {
                if (yd >= yd1 && i < n) {
                    const uint32_t e = L.list[i++][tid];
                    if ((int)(e >> 15) != cur) {  // the second cluster's first
                        result(0);
                        best = NONE;
                        cur = 1;
                        yh = yv[1];
                        zh = zv[1];
                    }
                    const int c = (int)(e & 2047u);
                    ay = Y[c] - yh;
                    az = Z[c] - zh;
                    urs = (uint32_t)R[c] << 16;
                    my = __builtin_fmaf(fabsf(yh) + wcy, 1e-5f, 1e-6f);
                    mz = __builtin_fmaf(fabsf(zh) + wcz, 1e-5f, 1e-6f);
                    hy = (yh - gd.y0) * gd.iwy;
                    hz = (zh - gd.z0) * gd.iwz;
                    // down clusters around the prediction h - (u - h)
                    const float r = __builtin_amdgcn_sqrtf(__uint_as_float((uint32_t)(best >> 32))) * 1.0001f;
                    const float py = __builtin_fmaf(-ay, gd.iwy, hy), pz = __builtin_fmaf(-az, gd.iwz, hz);
                    const float ky = __builtin_fmaf(fminf(cut_y, r) + my, gd.iwy, edy);
                    const float kz = __builtin_fmaf(fminf(cut_z, r) + mz, gd.iwz, edz);
                    yd = cell_in(py - ky, dny);
                    yd1 = cell_in(py + ky, dny);
                    zd0 = cell_in(pz - kz, dnz);
                    zd1 = cell_in(pz + kz, dnz);
                    const int row = __mul24(yd, gd.nz);
                    kd = DCS[row + zd0];
                    e1 = DCS[row + zd1 + 1];
                }
            }
            while (kd == e1 && yd < yd1) {
                ++yd;
                const int row = __mul24(yd, gd.nz);
                kd = DCS[row + zd0];
                e1 = DCS[row + zd1 + 1];
            }
            // (two per round: boxes hold few, and the rounds are what costs)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (kd < e1) {
                    const int c = kd++;
                    const float ty = Y[c] - yh;
                    const float tz = Z[c] - zh;
                    const uint32_t rr = R[c];
                    const float dy = ay + ty;
                    const float dz = az + tz;
                    const float qy = dy * dy;
                    const float qz = dz * dz;
                    const float q = qy + qz;
                    const uint64_t key = ((uint64_t)__float_as_uint(q) << 32) | (uint64_t)(urs | rr);
                    // bitwise, not short-circuit, conjunctions: no branches in the test
                    const bool win = (int)(fabsf(ty) <= win_y) & (int)(fabsf(tz) <= win_z) & (int)(fabsf(dy) <= cut_y) &
                                     (int)(fabsf(dz) <= cut_z) & (int)(key < best);
                    best = win ? key : best;
                }
            }
        }
        n = 0;
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        // the up clusters in the window of the thread's s-th cluster
        const float y = yv[s], z = zv[s];
        int ic = 0, nabove = 0, it = 0, it1 = -1, zc0 = 0, zc1 = 0, k = 0, k1 = 0;
        if (grids && isfinite(y) && isfinite(z)) {
            const float my = __builtin_fmaf(fabsf(y) + wcy, 1e-5f, 1e-6f);
            const float mz = __builtin_fmaf(fabsf(z) + wcz, 1e-5f, 1e-6f);
            const float uy = (y - gu.y0) * gu.iwy, uz = (z - gu.z0) * gu.iwz;
            const float wy = __builtin_fmaf(win_y + my, gu.iwy, euy);
            const float wz = __builtin_fmaf(win_z + mz, gu.iwz, euz);
            // rows from h's own up, then from the one below it down
            ic = cell_in(uy, uny);
            nabove = cell_in(uy + wy, uny) - ic;
            it1 = nabove + ic - cell_in(uy - wy, uny);
            zc0 = cell_in(uz - wz, unz);
            zc1 = cell_in(uz + wz, unz);
            const int row = __mul24(ic, gu.nz);
            k = UCS[row + zc0];
            k1 = UCS[row + zc1 + 1];
        }
        while (true) {
            while (__ballot((k < k1 || it < it1) && n < TPC_NB_LIST)) {
                if (n == TPC_NB_LIST) continue;
                if (k == k1 && it < it1) {
                    ++it;
                    const int row = __mul24(ic + (it <= nabove ? it : nabove - it), gu.nz);
                    k = UCS[row + zc0];
                    k1 = UCS[row + zc1 + 1];
                }
                if (k < k1) {                     // (two are read at once, whether or not the row has both)
                    const float a0 = Y[k] - y, b0 = Z[k] - z, a1 = Y[k + 1] - y, b1 = Z[k + 1] - z;
                    if ((int)(fabsf(a0) <= win_y) & (int)(fabsf(b0) <= win_z))
                        L.list[n++][tid] = (uint16_t)(k | s << 15);
                    ++k;
                    if (k < k1 && n < TPC_NB_LIST) {
                        if ((int)(fabsf(a1) <= win_y) & (int)(fabsf(b1) <= win_z))
                            L.list[n++][tid] = (uint16_t)(k | s << 15);
                        ++k;
                    }
                }
            }
            if (!__ballot(k < k1 || it < it1)) break;
            search();
        }
    }
    search();
    result(cur);
    if (cur == 0) {
        best = NONE;
        result(1);
    }
    // results in the slab's order (ids read coalesced; the search loop
    // issues no global store, whose completion its waits for the next
    // cluster's loads would also wait for)
    __syncthreads();
    for (int p = threadIdx.x; p < pn; p += TPC_BLOCK) {
        const uint32_t r = L.res[p];
        const int32_t h = sid[pb + p];
        up[h] = r == 0xFFFFFFFFu ? -1 : baseu + (int32_t)(r >> 16);
        dn[h] = r == 0xFFFFFFFFu ? -1 : based + (int32_t)(r & 0xFFFFu);
    }
}

// Start of part k of a dense h-row of n z-sorted clusters searched in
// `parts` parts by different workgroups: k / parts of it, rounded down to
// whole slabs (part parts ends at n).
__device__ inline int dense_split(int n, int k, int parts) {
    return k >= parts ? n : (int)((int64_t)n * k / parts) / TPC_NB_SLAB * TPC_NB_SLAB;
}

// Dense h-row `seg` (whole workgroup; contains barriers): slabs of
// consecutive clusters of its z-sorted copy.  A partner of h passes the
// window test only if its z lies within win_z of z_h (the difference is one
// rounding), so the neighbouring rows' clusters with z in the slab's finite
// z extent widened by win_z and a margin far above that rounding hold every
// candidate; their positions form one range of each z-sorted copy.  Both
// ranges are binned into LDS and the slab searched there (slab_search); a
// slab whose ranges do not fit is halved, and at TPC_NB_SLAB_MIN clusters it
// is searched in the global copies instead.  The outcome does not depend
// on which superset of the candidates is searched.
template <int ROW, int CELLS>
__device__ __forceinline__ void nb_dense_seg(int seg, const int32_t *__restrict__ off, int32_t n_rows, float win_y,
                                    float win_z, float cut_y, float cut_z, const SegGrid *__restrict__ grid,
                                    const int32_t *__restrict__ cstart, const float *__restrict__ sy,
                                    const float *__restrict__ sz, const int32_t *__restrict__ sid,
                                    int32_t *__restrict__ up, int32_t *__restrict__ dn,
                                    DenseLdsT<ROW, CELLS> &L, int part = 0, int parts = 1) {
#pragma clang fp contract(off)
    if (!dense_hrow(off, seg, n_rows)) return;
    const int tid = threadIdx.x;
    const int a = off[seg], n = off[seg + 1] - a;
    const int lo = dense_split(n, part, parts), hi = dense_split(n, part + 1, parts);
    const int sd = seg - 1, su = seg + 1;
    const int based = off[sd], baseu = off[su];
    const SegGrid gdg = grid[sd], gug = grid[su];
    const int32_t *csd = cstart + based + sd;
    const int32_t *csu = cstart + baseu + su;
    // relative ids are 16-bit in the keys and in LDS (at most 65534, so a
    // result is never all ones)
    const bool rel_ok = seg_size(off, sd) <= 65535 && seg_size(off, su) <= 65535;
    int P = TPC_NB_SLAB;
    for (int p0 = lo; p0 < hi;) {
        const int pn = hi - p0 < P ? hi - p0 : P;
        float lo = INFINITY, hi = -INFINITY;
        for (int k = tid; k < pn; k += TPC_BLOCK) {
            const float zv = sz[a + p0 + k];
            if (isfinite(zv)) { lo = fminf(lo, zv); hi = fmaxf(hi, zv); }
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        __syncthreads();             // the previous slab's search is done with L
        if ((tid & (TPC_WAVE - 1)) == 0) {
            L.red[0][tid / TPC_WAVE] = lo;
            L.red[1][tid / TPC_WAVE] = hi;
        }
        __syncthreads();
        lo = L.red[0][0];
        hi = L.red[1][0];
        for (int w = 1; w < TPC_BLOCK / TPC_WAVE; ++w) {
            lo = fminf(lo, L.red[0][w]);
            hi = fmaxf(hi, L.red[1][w]);
        }
        __syncthreads();             // everyone has read L.red
        int2 rd = make_int2(0, 0), ru = make_int2(0, 0);
        if (lo <= hi) {
            const float m = 1e-5f * (fmaxf(fabsf(lo), fabsf(hi)) + win_z + cut_z) + 1e-6f;
            const float w = win_z + m;
            rd = zrange(gdg, csd, lo - w, hi + w);
            ru = zrange(gug, csu, lo - w, hi + w);
        }
        const int nd = rd.y - rd.x, nu = ru.y - ru.x;
        const bool fits = rel_ok && nd <= ROW && nu <= ROW;
        if (!fits && P > TPC_NB_SLAB_MIN) {
            P >>= 1;
            continue;
        }
        if (fits) {
            SegGrid gd, gu;
            int C0;
            pair_bin(SortedPairSrc{sy, sz, sid, rd.x, nd, ru.x, based, baseu}, nd, nu, win_y, win_z,
                     TPC_NB_DENSE_EDGE_D, TPC_NB_DENSE_EDGE_U, L, gd, gu, C0);
            slab_search(a + p0, pn, sy, sz, sid, baseu, based, gu, gd, C0, win_y, win_z, cut_y, cut_z, up, dn,
                        L);
        } else {
            for (int k = tid; k < pn; k += TPC_BLOCK) {
                const int p = a + p0 + k;
                const Best bt = best_pair(sy[p], sz[p], sy, sz, sid, csu, gug, 0, sy, sz, sid, csd, gdg, 0,
                                          win_y, win_z, cut_y, cut_z);
                const int32_t h = sid[p];
                up[h] = bt.u;
                dn[h] = bt.d;
            }
        }
        p0 += pn;
        P = TPC_NB_SLAB;
    }
    __syncthreads();                 // LDS reuse across calls in a persistent loop
}

// The two neighbouring rows of an h-row (at most N clusters together) binned
// together: one cell grid, one cell order, so that a cluster's window is one
// set of cells.
#define TPC_MIX_WORDS 32      // words of 64 pairs taken in a round

// Are windows of the nt clusters of a row pair of extents ry, rz searched by
// boxes of the cuts (mix_wave), in cells made for that?  Where more than most
// overflow the lists (clusters spread evenly) and a box is far smaller than a
// window.  Event of 10^4 tracks, windows of 10 cm (20 clusters): 0.83 -> 0.58
// ms, of 40 cm 18 -> 1.7 ms; with cuts of half the window the boxes lose
// (0.99 -> 1.15 ms).
__device__ inline bool mix_boxes(int nt, float ry, float rz, int list, float win_y, float win_z, float cut_y,
                                 float cut_z) {
    const float a = fmaxf(ry, win_y), b = fmaxf(rz, win_z);
    return (float)nt * fminf(a, 2.0f * win_y) * fminf(b, 2.0f * win_z) > 1.5f * (float)list * a * b &&
           fminf(win_y, cut_y) * fminf(win_z, cut_z) < 0.125f * win_y * win_z;
}

template <int N, int CELLS, int LIST_>
struct MixLdsT {
    static constexpr int LIST = LIST_;
    float2 p[N + 1];                                // (y, z) in cell order
    uint16_t id[N + 1];                             // position in the down row, or n0 + position in the up row
    alignas(16) uint16_t cs[CELLS];                 // cell starts
    union {
        alignas(16) uint32_t cnt[CELLS];            // while binning
        uint16_t list[LIST][TPC_BLOCK];             // per thread: clusters in its window, by position in p
    } u;
    unsigned long long best[TPC_BLOCK];
    unsigned long long starts[TPC_BLOCK / TPC_WAVE][TPC_MIX_WORDS];
    int red[4][TPC_BLOCK / TPC_WAVE];
    int scan_sh[TPC_BLOCK / TPC_WAVE];
};
using MixLds = MixLdsT<TPC_MIX_N, 1024, 16>;            // 24 KB: six workgroups per CU
using MixLdsL = MixLdsT<2 * TPC_LDS_ROW, 2048, 24>;     // 39 KB: four

// Orders of the LDS accesses within a wavefront (the hardware keeps them in
// order; this keeps the compiler from moving them).
__device__ inline void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Bins both neighbouring rows of an h-row into L (whole workgroup; contains
// barriers): the clusters of [ra0, ra0 + n0) and [ra1, ra1 + nt - n0).  The
// grid covers the finite extents of both rows; how it divides them decides
// no result, so its divisions are hardware reciprocals.
template <int N, int CELLS, int LIST>
__device__ inline SegGrid mix_bin(const float *__restrict__ y, const float *__restrict__ z, int ra0, int n0, int ra1,
                                  int nt, float win_y, float win_z, float cut_y, float cut_z,
                                  MixLdsT<N, CELLS, LIST> &L) {
#pragma clang fp contract(off)
    constexpr int PT = (N + TPC_BLOCK - 1) / TPC_BLOCK;
    constexpr int Q = CELLS / (4 * TPC_BLOCK);      // groups of four cells per thread
    static_assert(CELLS == 4 * Q * TPC_BLOCK, "cells in groups of four per thread");
    static_assert(N < 65535, "16-bit positions");
    const int tid = threadIdx.x;
    float vy[PT], vz[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int k = tid + j * TPC_BLOCK;
        vy[j] = NAN;
        vz[j] = NAN;
        if (j * TPC_BLOCK < nt && k < nt) {
            const int i = k < n0 ? ra0 + k : ra1 + (k - n0);
            vy[j] = y[i];
            vz[j] = z[i];
        }
    }
    int4 *cnt4 = reinterpret_cast<int4 *>(L.u.cnt) + tid * Q;
#pragma unroll
    for (int q = 0; q < Q; ++q) cnt4[q] = make_int4(0, 0, 0, 0);
    // extents as integers of the same order: min y, min -y, min z, min -z
    auto ordered = [](float v) {
        const int i = __float_as_int(v);
        return i ^ ((i >> 31) & 0x7FFFFFFF);
    };
    constexpr int TOP = 0x7FFFFFFF;
    int e[4] = {TOP, TOP, TOP, TOP};
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        if (j * TPC_BLOCK >= nt) break;
        const int oy = ordered(vy[j]), oz = ordered(vz[j]);
        const bool fy = isfinite(vy[j]), fz = isfinite(vz[j]);
        e[0] = min(e[0], fy ? oy : TOP);
        e[1] = min(e[1], fy ? ~oy : TOP);
        e[2] = min(e[2], fz ? oz : TOP);
        e[3] = min(e[3], fz ? ~oz : TOP);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = lane63_min(e[j]);
    const int wid = tid / TPC_WAVE, lane = tid & (TPC_WAVE - 1);
    if (lane == TPC_WAVE - 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) L.red[j][wid] = e[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[j] = L.red[j][0];
#pragma unroll
        for (int w = 1; w < TPC_BLOCK / TPC_WAVE; ++w) e[j] = min(e[j], L.red[j][w]);
    }
    auto back = [](int o) { return __int_as_float(o ^ ((o >> 31) & 0x7FFFFFFF)); };
    const float ymin = back(e[0]), ymax = back(~e[1]), zmin = back(e[2]), zmax = back(~e[3]);
    // up to four cells per cluster of the larger row, edges of at least the
    // window
    const int nm = n0 > nt - n0 ? n0 : nt - n0;
    const int cap = 4 * nm < CELLS - 2 ? 4 * nm : CELLS - 2;
    const float fc = (float)cap, ry = ymax - ymin, rz = zmax - zmin;
    float fz = rz * (0.99f * __builtin_amdgcn_rcpf(win_z)), fy = ry * (0.99f * __builtin_amdgcn_rcpf(win_y));
    float fcz = fc;
    // (what follows from the windows and cuts is formed anew for each row pair:
    // kept across a workgroup's segments it took registers from the search,
    // 200 frames 1271 -> 1299 us, 1279 so)
    float wy = win_y, wz = win_z, cy = cut_y, cz = cut_z;
    asm volatile("" : "+s"(wy), "+s"(wz), "+s"(cy), "+s"(cz));
    if (mix_boxes(nt, ry, rz, LIST, wy, wz, cy, cz)) {
        // most windows are searched by boxes: edges of at least the smaller of
        // window and cut, as many in y as windows and the rest in z
        fcz = fc * __builtin_amdgcn_rcpf(fmaxf(1.0f, fminf(fy, fc)));
        fz = rz * (0.99f * __builtin_amdgcn_rcpf(fminf(wz, cz)));
        fy = ry * (0.99f * __builtin_amdgcn_rcpf(fminf(wy, cy)));
    }
    const int nz = fz >= fcz ? max((int)fcz, 1) : (fz >= 1.0f ? (int)fz : 1);
    int ny = (int)(fc * __builtin_amdgcn_rcpf((float)nz));
    if (ny * nz > cap) --ny;
    ny = fy >= (float)ny ? ny : (fy >= 1.0f ? (int)fy : 1);
    if (ny < 1) ny = 1;
    const SegGrid g = {ymin, zmin, ny > 1 ? (float)ny * __builtin_amdgcn_rcpf(ry) : 0.f,
                       nz > 1 ? (float)nz * __builtin_amdgcn_rcpf(rz) : 0.f, ny, nz, 0, 0};
    int cell[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        cell[j] = 0;
        if (j * TPC_BLOCK >= nt) break;
        cell[j] = pair_cell(vy[j], vz[j], g);
        if (tid + j * TPC_BLOCK < nt) atomicAdd(&L.u.cnt[cell[j]], 1u);
    }
    __syncthreads();
    // exclusive scan, the same cells per thread whatever their number (at
    // most CELLS - 2, so the word behind the last cell's is the total)
    int4 c[Q];
    int sum = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        c[q] = cnt4[q];
        sum += c[q].x + c[q].y + c[q].z + c[q].w;
    }
    int total;
    int run = block_exclusive_scan(sum, L.scan_sh, &total);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b0 = run, b1 = b0 + c[q].x, b2 = b1 + c[q].y, b3 = b2 + c[q].z;
        run = b3 + c[q].w;
        cnt4[q] = make_int4(b0, b1, b2, b3);
        reinterpret_cast<uint2 *>(L.cs)[tid * Q + q] =
            make_uint2((uint32_t)b0 | (uint32_t)b1 << 16, (uint32_t)b2 | (uint32_t)b3 << 16);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        if (j * TPC_BLOCK >= nt) break;
        const int k = tid + j * TPC_BLOCK;
        if (k < nt) {
            const uint32_t slot = atomicAdd(&L.u.cnt[cell[j]], 1u);
            L.p[slot] = make_float2(vy[j], vz[j]);
            L.id[slot] = (uint16_t)k;
        }
    }
    __syncthreads();
    return g;
}

struct PairKey {
    unsigned long long key;
    int owner;
};

// Key of the pair (up position ku, down position kd) of the h-cluster
// (yh, zh), smaller for the better pair: bits of q, then the ids.  All ones
// if the pair fails the cuts.  By the operations of the definition.
template <class LDS>
__device__ inline unsigned long long mix_key(float yh, float zh, int ku, int kd, const LDS &L, float cut_y,
                                             float cut_z) {
#pragma clang fp contract(off)
    const float2 u = L.p[ku], d = L.p[kd];
    const uint32_t ids = (uint32_t)L.id[ku] << 16 | L.id[kd];
    const float dy = (u.x - yh) - (yh - d.x), dz = (u.y - zh) - (zh - d.y);
    const float qy = dy * dy, qz = dz * dz;
    const float q = qy + qz;
    const bool pass = (int)(fabsf(dy) <= cut_y) & (int)(fabsf(dz) <= cut_z);
    return pass ? ((unsigned long long)__float_as_uint(q) << 32) | ids : ~0ull;
}

// Best pair of cluster (yh, zh) by a whole wavefront, into *best (its key so
// far, an LDS word), nd down and nu up clusters being in its window: these
// are compacted into the wavefront's part of the lists, and their pairs
// taken 64 at a time.  Beyond TPC_MIX_PAIRS pairs only the up clusters are
// listed, and each lane takes one at a time and searches the cells of the box
// around the prediction 2h - u, whose half-widths shrink from the cuts to the
// best pair's distance (slab_search has the reasons): where windows hold
// hundreds, mix_bin's cells are as small as the cuts, and a box holds a few.
// (Windows of 80 cm, event of 10^4 tracks: 42 ms of all pairs, 2.3 so.)
#define TPC_MIX_PAIRS 1024
template <class LDS>
__device__ inline void mix_wave(float yh, float zh, int n0, int nd, int nu, const SegGrid &g, LDS &L, float win_y,
                                float win_z, float cut_y, float cut_z, float my, float mz, unsigned long long *best) {
#pragma clang fp contract(off)
    constexpr int CAP = LDS::LIST * TPC_WAVE;
    static_assert(TPC_LDS_ROW <= CAP, "the up clusters of a window fit");
    const int lane = threadIdx.x & (TPC_WAVE - 1), base = threadIdx.x - lane;
    auto at = [&](int e) -> uint16_t & { return L.u.list[e / TPC_WAVE][base + e % TPC_WAVE]; };
    const int y0 = cell_coord(yh - (win_y + my), g.y0, g.iwy, g.ny);
    const int y1 = cell_coord(yh + (win_y + my), g.y0, g.iwy, g.ny);
    const int z0 = cell_coord(zh - (win_z + mz), g.z0, g.iwz, g.nz);
    const int z1 = cell_coord(zh + (win_z + mz), g.z0, g.iwz, g.nz);
    const bool fine = fmaxf(win_y * g.iwy, win_z * g.iwz) > 1.5f;      // made for boxes
    const bool all = nd + nu <= CAP && (!fine || nd * nu <= TPC_MIX_PAIRS);
    unsigned long long b = ~0ull;
    if (nd == 0 || nu == 0) return;
    int id0 = 0, iu0 = 0;                            // listed so far
    for (int iy = y0; iy <= y1; ++iy) {
        const int e = L.cs[iy * g.nz + z1 + 1];
        for (int k0 = L.cs[iy * g.nz + z0]; k0 < e; k0 += TPC_WAVE) {
            const int k = k0 + lane;
            bool down = false, upper = false;
            if (k < e) {
                const bool in = fabsf(L.p[k].x - yh) <= win_y && fabsf(L.p[k].y - zh) <= win_z;
                const int id = L.id[k];
                down = all && in && id < n0;
                upper = in && id >= n0;
            }
            const uint64_t bd = __ballot(down), bu = __ballot(upper);
            if (down) at(id0 + lanes_below(bd)) = (uint16_t)k;
            if (upper) at(CAP - 1 - iu0 - lanes_below(bu)) = (uint16_t)k;
            id0 += __popcll(bd);
            iu0 += __popcll(bu);
        }
    }
    wave_fence();
    if (all) {
        const float inv = __builtin_amdgcn_rcpf((float)nd);
        for (int t = lane; t < nd * nu; t += TPC_WAVE) {
            // t / nd: the error of the product is far below the 0.5 / nd to
            // the next integer
            const int iu = (int)(((float)t + 0.5f) * inv);
            const unsigned long long key = mix_key(yh, zh, at(CAP - 1 - iu), at(t - iu * nd), L, cut_y, cut_z);
            b = key < b ? key : b;
        }
    } else {
        float r = INFINITY;                          // no better pair is further off in y or z
        for (int t0 = 0; t0 < nu; t0 += TPC_WAVE) {
            if (t0 + lane < nu) {
                const int ku = at(CAP - 1 - (t0 + lane));
                const float2 u = L.p[ku];
                const uint32_t up = (uint32_t)L.id[ku] << 16;
                const float ay = u.x - yh, az = u.y - zh;
                const float cy = yh - ay, cz = zh - az, ky = fminf(cut_y, r) + my, kz = fminf(cut_z, r) + mz;
                const int yd1 = cell_coord(cy + ky, g.y0, g.iwy, g.ny), zd1 = cell_coord(cz + kz, g.z0, g.iwz, g.nz);
                const int zd0 = cell_coord(cz - kz, g.z0, g.iwz, g.nz);
                for (int iy = cell_coord(cy - ky, g.y0, g.iwy, g.ny); iy <= yd1; ++iy) {
                    const int e = L.cs[iy * g.nz + zd1 + 1];
                    for (int k = L.cs[iy * g.nz + zd0]; k < e; ++k) {
                        const float2 d = L.p[k];
                        const uint32_t id = L.id[k];
                        const float by = yh - d.x, bz = zh - d.y;
                        const float dy = ay - by, dz = az - bz;
                        const float qy = dy * dy, qz = dz * dz;
                        const float q = qy + qz;
                        const unsigned long long key = ((unsigned long long)__float_as_uint(q) << 32) | (up | id);
                        const bool win = (int)((int)id < n0) & (int)(fabsf(by) <= win_y) & (int)(fabsf(bz) <= win_z) &
                                         (int)(fabsf(dy) <= cut_y) & (int)(fabsf(dz) <= cut_z) & (int)(key < b);
                        b = win ? key : b;
                    }
                }
            }
            const int q = __builtin_amdgcn_readlane(lane63_min(b == ~0ull ? 0x7F800000 : (int)(b >> 32)), TPC_WAVE - 1);
            r = __builtin_amdgcn_sqrtf(__int_as_float(q)) * 1.0001f;
        }
    }
    if (b != ~0ull) atomicMin(best, b);
    wave_fence();
}

// Best triplet of every cluster of h-row `seg` whose neighbouring rows hold
// at most N clusters together (whole workgroup; contains barriers).
//
// Bound by vector instructions, most of which a loop per cluster spends on
// lanes that wait: with two clusters of either row in a window on average,
// the busiest lane of a wavefront has five times the mean number of pairs.
// So a lane only lists the clusters in its window (down from the front of
// its list, up from the back), and the pairs of all lanes are then dealt
// out 64 at a time: lane starts are set as bits of a mask, a lane finds its
// pair's owner by counting bits, and the owner's best key is a 64-bit LDS
// minimum.  Windows of more than LIST clusters go to mix_wave: with 16 of
// them 0.03 % at 230 clusters per row and 1.3 % at 460, where they begin to
// cost; the large form's 24 leave few up to its 1024.  (Left to their own
// lanes, by boxes around the predictions, such windows cost more up to 100
// clusters of either row in them: for the large rows of an event of 3 10^4
// tracks 865 us against 378.)
template <int N, int CELLS, int LIST>
__device__ __forceinline__ void mix_query_seg(int seg, const int32_t *__restrict__ off, const float *__restrict__ y,
                                              const float *__restrict__ z, float win_y, float win_z, float cut_y,
                                              float cut_z, int32_t *__restrict__ up, int32_t *__restrict__ dn,
                                              MixLdsT<N, CELLS, LIST> &L) {
#pragma clang fp contract(off)
    static_assert(LIST <= 24 && TPC_WAVE == 64, "14 bits of pair starts; nd * nd * nu < 2^12");
    const int a = off[seg], b = off[seg + 1], ra0 = off[seg - 1], n0 = a - ra0, nt = n0 + off[seg + 2] - b;
    const int tid = threadIdx.x, lane = tid & (TPC_WAVE - 1), wid = tid / TPC_WAVE;
    // the first h of each thread is loaded together with the row pair
    float yh = 0.f, zh = 0.f;
    if (a + tid < b) {
        yh = y[a + tid];
        zh = z[a + tid];
    }
    const SegGrid g = mix_bin(y, z, ra0, n0, b, nt, win_y, win_z, cut_y, cut_z, L);
    for (int i0 = a + wid * TPC_WAVE; i0 < b; i0 += TPC_BLOCK) {
        const int i = i0 + lane;
        if (i0 >= a + TPC_BLOCK && i < b) {
            yh = y[i];
            zh = z[i];
        }
        const float my = 1e-5f * (fabsf(yh) + win_y + cut_y) + 1e-6f;
        const float mz = 1e-5f * (fabsf(zh) + win_z + cut_z) + 1e-6f;
        int nd = 0, nu = 0;
        if (i < b && isfinite(yh) && isfinite(zh)) {
            const float wy = win_y + my, wz = win_z + mz;
            const int y0 = cell_coord(yh - wy, g.y0, g.iwy, g.ny), y1 = cell_coord(yh + wy, g.y0, g.iwy, g.ny);
            const int z0 = cell_coord(zh - wz, g.z0, g.iwz, g.nz), z1 = cell_coord(zh + wz, g.z0, g.iwz, g.nz);
            int row = __mul24(y0, g.nz), k = L.cs[row + z0], e = L.cs[row + z1 + 1];
            for (int iy = y0; iy <= y1; ++iy) {
                // (the next row's range; of the last one again, not used)
                row += iy < y1 ? g.nz : 0;
                const int kn = L.cs[row + z0], en = L.cs[row + z1 + 1];
                auto take = [&](const float2 &c, int side, int q) {
                    if (!((int)(fabsf(c.x - yh) <= win_y) & (int)(fabsf(c.y - zh) <= win_z) & (int)(q < e))) return;
                    const int s = side >= n0;
                    if (nd + nu < LIST) L.u.list[s ? LIST - 1 - nu : nd][tid] = (uint16_t)q;
                    nu += s;
                    nd += 1 - s;
                };
                // two at a time, the sides read with the coordinates: the
                // chain of LDS reads is what a wavefront waits for
                for (; k < e; k += 2) {
                    const float2 c0 = L.p[k], c1 = L.p[k + 1];
                    const int s0 = L.id[k], s1 = L.id[k + 1];
                    take(c0, s0, k);
                    take(c1, s1, k + 1);
                }
                k = kn;
                e = en;
            }
        }
        const bool listed = nd + nu <= LIST;
        const int P = listed ? nd * nu : 0;
        const int inc = lane_scan(P), S = inc - P;
        const int total = __builtin_amdgcn_readlane(inc, TPC_WAVE - 1);
        L.best[tid] = ~0ull;
        if (total > 0) {
            // what a pair needs of its owner, in the order of the owners
            const uint64_t has = __ballot(P > 0);
            const int below = lanes_below(has);
            const int rank = 4 * (P > 0 ? below : __popcll(has) + lane - below);
            // nd divides j < nd nu by a product: ceil(2^12 / nd) is off by
            // less than 1, the product by less than j / 2^12 < 1 / nd
            const int m = (int)(4096.0f * __builtin_amdgcn_rcpf((float)nd)) + 1;
            const int pw = __builtin_amdgcn_ds_permute(rank, (int)((uint32_t)S | (uint32_t)nd << 14 | (uint32_t)m << 19));
            const int py = __builtin_amdgcn_ds_permute(rank, __float_as_int(yh));
            const int pz = __builtin_amdgcn_ds_permute(rank, __float_as_int(zh));
            const int pl = __builtin_amdgcn_ds_permute(rank, tid);
            for (int r0 = 0; r0 < total; r0 += TPC_MIX_WORDS * TPC_WAVE) {
                if (lane < TPC_MIX_WORDS) L.starts[wid][lane] = 0;
                wave_fence();
                if (P > 0 && S >= r0 && S < r0 + TPC_MIX_WORDS * TPC_WAVE)
                    atomicOr(&L.starts[wid][(S - r0) >> 6], 1ull << (S & 63));
                wave_fence();
                // all words of the mask at once, one per lane
                const unsigned long long words = L.starts[wid][lane % TPC_MIX_WORDS];
                int before = __popcll(__ballot(P > 0 && S < r0)) - 1;
                auto pair = [&](int t0) {
                    const int q = (t0 - r0) / TPC_WAVE;
                    const uint64_t M = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(words >> 32), q) << 32 |
                                       (uint32_t)__builtin_amdgcn_readlane((int)words, q);
                    const int r = 4 * (before + (int)(M & 1) + lanes_below(M >> 1));
                    before += __popcll(M);
                    const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute(r, pw);
                    const float oy = __int_as_float(__builtin_amdgcn_ds_bpermute(r, py));
                    const float oz = __int_as_float(__builtin_amdgcn_ds_bpermute(r, pz));
                    const int owner = __builtin_amdgcn_ds_bpermute(r, pl);
                    // (beyond the last pair: its owner's first)
                    const int j = t0 + lane < total ? t0 + lane - (int)(w & 0x3FFFu) : 0, n = (int)(w >> 14) & 31;
                    const int iu = __mul24(j, (int)(w >> 19)) >> 12, id = j - __mul24(iu, n);
                    const int kd = L.u.list[id][owner], ku = L.u.list[LIST - 1 - iu][owner];
                    return PairKey{mix_key(oy, oz, ku, kd, L, cut_y, cut_z), owner};
                };
                // two pairs per lane in flight
                const int end = total - r0 < TPC_MIX_WORDS * TPC_WAVE ? total : r0 + TPC_MIX_WORDS * TPC_WAVE;
                for (int t0 = r0; t0 < end; t0 += 2 * TPC_WAVE) {
                    const PairKey k0 = pair(t0);
                    PairKey k1 = {~0ull, 0};
                    if (t0 + TPC_WAVE < end) k1 = pair(t0 + TPC_WAVE);
                    if (k0.key != ~0ull) atomicMin(&L.best[k0.owner], k0.key);
                    if (k1.key != ~0ull) atomicMin(&L.best[k1.owner], k1.key);
                }
                wave_fence();
            }
        }
        // the others by the whole wavefront, one after the other
        for (uint64_t over = __ballot(!listed); over != 0; over &= over - 1) {
            const int l = __builtin_ctzll(over);
            auto of = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
            float wy = win_y, wz = win_z, cy = cut_y, cz = cut_z;
            asm volatile("" : "+s"(wy), "+s"(wz), "+s"(cy), "+s"(cz));      // (as in mix_bin)
            mix_wave(of(yh), of(zh), n0, __builtin_amdgcn_readlane(nd, l), __builtin_amdgcn_readlane(nu, l), g, L, wy, wz,
                     cy, cz, of(my), of(mz), &L.best[tid - lane + l]);
        }
        if (i < b) {
            const unsigned long long best = L.best[tid];
            const bool found = best != ~0ull;
            up[i] = found ? b + (int32_t)((uint32_t)best >> 16) - n0 : -1;
            dn[i] = found ? ra0 + (int32_t)(best & 0xFFFFu) : -1;
        }
        wave_fence();
    }
}

// Items of [0, n) that workgroup b of G takes and that pass `pick`, into
// `list` (its own, at most TPC_BLOCK of the items b, b + G, ... from `from` on
// at a time); returns how many.  Whole workgroup; contains barriers.  One
// test per thread: a workgroup that walks over its items one after the other
// waits for their row offsets each time.
template <class Pick>
__device__ inline int pick_items(int from, int b, int G, int n, const Pick &pick, int *list, int *count) {
    __syncthreads();
    if (threadIdx.x == 0) *count = 0;
    __syncthreads();
    const int64_t i = b + (int64_t)G * (from + (int)threadIdx.x);
    if (i < n && pick((int)i)) list[atomicAdd(count, 1)] = (int)i;
    __syncthreads();
    return *count;
}

// Best triplet of every cluster of h-row `seg` whose neighbouring rows hold
// at most 64 clusters together, by one wavefront without LDS or barriers:
// lane k holds the k-th of them, every lane tests its cluster's window
// against all (a bit each), and scores the few pairs of its bits.  Rows this
// small are many (half of 64 uneven frames' 350 000 segments) and cost what
// launching a workgroup and its barriers cost: 2.5 -> 1 ns per segment.
#define TPC_TINY_N 64
__device__ inline bool tiny_pair(const int32_t *off, int seg) {
    return off[seg] - off[seg - 1] + off[seg + 2] - off[seg + 1] <= TPC_TINY_N;
}

__device__ inline void tiny_query_wave(int seg, const int32_t *__restrict__ off, const float *__restrict__ y,
                                       const float *__restrict__ z, float win_y, float win_z, float cut_y,
                                       float cut_z, int32_t *__restrict__ up, int32_t *__restrict__ dn) {
#pragma clang fp contract(off)
    static_assert(TPC_TINY_N == TPC_WAVE, "a cluster per lane, a bit each");
    const int lane = threadIdx.x & (TPC_WAVE - 1);
    const int ra0 = off[seg - 1], a = off[seg], b = off[seg + 1], n0 = a - ra0, nt = n0 + off[seg + 2] - b;
    float yh = 0.f, zh = 0.f, cy = 0.f, cz = 0.f;
    if (a + lane < b) {
        yh = y[a + lane];
        zh = z[a + lane];
    }
    if (lane < nt) {
        const int k = lane < n0 ? ra0 + lane : b + lane - n0;
        cy = y[k];
        cz = z[k];
    }
    const uint64_t downs = n0 < 64 ? (1ull << n0) - 1 : ~0ull;
    for (int i0 = a; i0 < b; i0 += TPC_WAVE) {
        const int i = i0 + lane;
        if (i0 > a && i < b) {
            yh = y[i];
            zh = z[i];
        }
        uint32_t bits[2] = {0, 0};
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            for (int k = 32 * w; k < nt && k < 32 * w + 32; ++k) {
                const float ky = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cy), k));
                const float kz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cz), k));
                const bool in = (int)(fabsf(ky - yh) <= win_y) & (int)(fabsf(kz - zh) <= win_z);
                bits[w] |= in ? 1u << (k & 31) : 0u;
            }
        }
        // (a non-finite h is in no window)
        const uint64_t m = i < b ? (uint64_t)bits[1] << 32 | bits[0] : 0ull;
        const uint64_t md = m & downs;
        uint64_t mu = md ? m & ~downs : 0ull, d = md;
        unsigned long long best = ~0ull;
        while (__ballot(mu != 0)) {              // (every lane stays active for the exchanges)
            const int ku = mu ? __builtin_ctzll(mu) : 0, kd = mu ? __builtin_ctzll(d) : 0;
            auto of = [](int k, float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * k, __float_as_int(v))); };
            const float uy = of(ku, cy), uz = of(ku, cz), vy = of(kd, cy), vz = of(kd, cz);
            const float dy = (uy - yh) - (yh - vy), dz = (uz - zh) - (zh - vz);
            const float qy = dy * dy, qz = dz * dz;
            const float q = qy + qz;
            const bool pass = (int)(mu != 0) & (int)(fabsf(dy) <= cut_y) & (int)(fabsf(dz) <= cut_z);
            const unsigned long long key = ((unsigned long long)__float_as_uint(q) << 32) | (uint32_t)(ku << 16 | kd);
            best = pass && key < best ? key : best;
            d &= d - 1;
            if (d == 0) {
                d = md;
                mu &= mu - 1;
            }
        }
        if (i < b) {
            const bool found = best != ~0ull;
            up[i] = found ? b + (int32_t)((uint32_t)best >> 16) - n0 : -1;
            dn[i] = found ? ra0 + (int32_t)(best & 0xFFFFu) : -1;
        }
    }
}

}  // namespace tpc_nb
