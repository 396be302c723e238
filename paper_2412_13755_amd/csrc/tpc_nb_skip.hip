// Neighbours across a missing pad row (gfx950).  After the adjacent-row
// search, each cluster it left without partners looks for them up to two
// rows away: the best pair spanning three rows ((A, B) = (1, 2) or (2, 1)
// rows below/above), else the best spanning four ((2, 2)); the exact
// predicates and the ordering are those of best_pair.  A cluster that has
// an adjacent-row triplet keeps it, so only the unlinked ones are queried --
// a tenth to a quarter of the clusters, spread over every row (noise, track
// ends, the clusters beside a missing one), thirty to sixty per row.
//
//  skip_seg    one workgroup per h-row whose partner rows hold at most
//              SKIP_ROW_MAX clusters each, taking the row's clusters in
//              chunks of SKIP_Q; rows in ascending order over all sectors,
//              so that the inner rows, which hold the most clusters, do not
//              trail.  A chunk's unlinked clusters with finite coordinates
//              (the others cannot link) go to LDS, ranked by z (the longer
//              axis: fewer of them in a window of it); every thread streams
//              clusters of the four partner rows (coalesced) and finds the
//              queries in its window by a binary search over the ranked z
//              -- exact, since rounding is monotonic, so the z predicate
//              |fl(z_h - z_c)| <= w holds on a contiguous run of ranks --
//              once to count each query's candidates per row, then, for as
//              many queries as the LDS pool holds the candidates of, once
//              more to store them (row position and coordinates) in
//              exact-size lists; the (down, up) pairs of all these queries
//              are then dealt out over the workgroup and scored from LDS with
//              the exact arithmetic of best_pair.  (A query whose candidates
//              alone exceed the pool scans the two rows instead.)
//  skip_prep, skip_query
//              the h-rows with a larger partner row: global cell-sorted
//              copies of the rows they need, their unlinked clusters in one
//              list, one thread per listed cluster running best_pair in the
//              sorted copies.
#include "tpc_nb_device.hpp"
#include "tpc_nb_skip.hpp"

namespace {

// Best pair across one missing row for cluster (hy, hz): (1, 2) and (2, 1)
// compete by (q, u, d); (2, 2) only if neither passes.  d1, u1, d2, u2 are
// the rows r-1, r+1, r-2, r+2 (d2 only if lo2, u2 only if hi2).
template <class V>
__device__ inline tpc_nb::Best skip_pair(float hy, float hz, const V &d1, const V &u1, const V &d2,
                                         const V &u2, bool lo2, bool hi2, float win_y, float win_z,
                                         float cut_y, float cut_z) {
    tpc_nb::Best bt = {0.f, -1, -1};
    if (hi2)
        bt = tpc_nb::best_pair<1, 2>(hy, hz, u2.y, u2.z, u2.i, u2.cs, u2.g, u2.base, d1.y, d1.z, d1.i, d1.cs,
                                     d1.g, d1.base, win_y, win_z, cut_y, cut_z);
    if (lo2) {
        const tpc_nb::Best c = tpc_nb::best_pair<2, 1>(hy, hz, u1.y, u1.z, u1.i, u1.cs, u1.g, u1.base, d2.y,
                                                       d2.z, d2.i, d2.cs, d2.g, d2.base, win_y, win_z,
                                                       cut_y, cut_z);
        if (c.u >= 0 && tpc_nb::better(c.q, c.u, c.d, bt)) bt = c;
    }
    if (bt.u < 0 && lo2 && hi2)
        bt = tpc_nb::best_pair<2, 2>(hy, hz, u2.y, u2.z, u2.i, u2.cs, u2.g, u2.base, d2.y, d2.z, d2.i, d2.cs,
                                     d2.g, d2.base, win_y, win_z, cut_y, cut_z);
    return bt;
}

// A cell-sorted row as best_pair reads it (global copy: stored ids are
// global cluster ids, base 0).
struct RowView {
    const float *y, *z;
    const int32_t *i;
    const int32_t *cs;
    SegGrid g;
    int32_t base;
};

__device__ inline RowView row_view(const SkipWs &w, const int32_t *off, int s) {
    return RowView{w.nb.sy, w.nb.sz, w.nb.sid, w.nb.cstart + off[s] + s, w.nb.grid[s], 0};
}

#define SKIP_ROW_MAX 1024      // partner rows up to this size: skip_seg
#define SKIP_Q 256             // clusters of a row, so queries, per skip_seg pass
#define SKIP_POOL 2048         // window candidates of one pass, all queries and rows

// Cluster range of row r + dr of h-row seg's (frame, sector); empty if that
// row is outside the sector.
__device__ inline void partner_row(const int32_t *off, int seg, int r, int n_rows, int dr, int &a, int &b) {
    const int rr = r + dr;
    if (rr < 0 || rr >= n_rows) {
        a = b = 0;
        return;
    }
    a = off[seg + dr];
    b = off[seg + dr + 1];
}

// Does interior h-row seg have a partner row too large for skip_seg?
__device__ inline bool skip_large(const int32_t *off, int seg, int n_rows) {
    const int r = seg % n_rows;
    if (r < 1 || r > n_rows - 2) return false;
    int m = 0;
    for (int dr = -2; dr <= 2; ++dr) {
        if (dr == 0) continue;
        int a, b;
        partner_row(off, seg, r, n_rows, dr, a, b);
        m = b - a > m ? b - a : m;
    }
    return m > SKIP_ROW_MAX;
}

// Cell-sorted copy of every row that a large h-row needs; the unlinked
// clusters of large h-rows appended to the list.
__global__ void __launch_bounds__(TPC_BLOCK)
skip_prep(const int32_t *__restrict__ off, int32_t NR, int32_t n_rows, const float *__restrict__ y,
          const float *__restrict__ z, float win_y, float win_z, const int32_t *__restrict__ up, SkipWs w) {
    __shared__ tpc_nb::BinLds L;
    __shared__ int base_sh, list[TPC_BLOCK], listed;
    auto large = [&](int seg, int r) { return skip_large(off, seg, n_rows) && (r >= 2 || r <= n_rows - 3); };
    auto needed = [&](int seg, int r) {               // by an h-row up to two rows from it
        bool need = false;
        for (int k = -2; k <= 2; ++k) {
            const int rh = r + k;
            if (k != 0 && rh >= 1 && rh <= n_rows - 2) need = need || skip_large(off, seg + k, n_rows);
        }
        return need;
    };
    for (int from = 0; blockIdx.x + (int64_t)gridDim.x * from < NR; from += TPC_BLOCK) {
        const int m = tpc_nb::pick_items(from, blockIdx.x, gridDim.x, NR, [&](int s) {
            return needed(s, s % n_rows) || large(s, s % n_rows);
        }, list, &listed);
        for (int j = 0; j < m; ++j) {
            const int seg = list[j], r = seg % n_rows;
            const int a = off[seg], b = off[seg + 1], n = b - a;
            __syncthreads();                          // LDS reuse
            if (needed(seg, r)) {
                const int cbase = a + seg;
                if (n == 0) {
                    if (threadIdx.x == 0) {
                        w.nb.grid[seg] = SegGrid{0.f, 0.f, 0.f, 0.f, 0, 0, 0, 0};
                        w.nb.cstart[cbase] = a;
                    }
                } else {
                    float ext[4];
                    tpc_nb::row_extent(y, z, a, b, L.red, ext);
                    const SegGrid g =
                        tpc_nb::row_grid(ext[0], ext[1], ext[2], ext[3], n, TPC_CELL_CAP, win_y, win_z);
                    if (threadIdx.x == 0) w.nb.grid[seg] = g;
                    tpc_nb::row_sort(y, z, a, b, g, L.cnt, L.scan_sh, w.nb.sy, w.nb.sz, w.nb.sid, w.nb.cstart + cbase,
                                     a);
                }
            }
            if (!large(seg, r)) continue;
            for (int c0 = a; c0 < b; c0 += TPC_BLOCK) {
                const int h = c0 + (int)threadIdx.x;
                const int unl = h < b && up[h] < 0;
                int cnt;
                const int pos = block_exclusive_scan(unl, L.scan_sh, &cnt);
                if (threadIdx.x == 0 && cnt > 0) base_sh = atomicAdd(w.count, cnt);
                __syncthreads();
                if (unl) w.list[base_sh + pos] = make_int2(h, seg);
                __syncthreads();
            }
        }
    }
}

__global__ void __launch_bounds__(TPC_BLOCK)
skip_query(const int32_t *__restrict__ off, int32_t n_rows, const float *__restrict__ y,
           const float *__restrict__ z, float win_y, float win_z, float cut_y, float cut_z, SkipWs w,
           int32_t *up, int32_t *dn) {
    const int count = *w.count;
    for (int i = blockIdx.x * TPC_BLOCK + threadIdx.x; i < count; i += gridDim.x * TPC_BLOCK) {
        const int2 e = w.list[i];
        const int32_t h = e.x;
        const int seg = e.y;
        const int r = seg % n_rows;
        const bool lo2 = r >= 2, hi2 = r <= n_rows - 3;
        const RowView d1 = row_view(w, off, seg - 1), u1 = row_view(w, off, seg + 1);
        const RowView d2 = lo2 ? row_view(w, off, seg - 2) : d1;
        const RowView u2 = hi2 ? row_view(w, off, seg + 2) : u1;
        const tpc_nb::Best bt = skip_pair(y[h], z[h], d1, u1, d2, u2, lo2, hi2, win_y, win_z, cut_y, cut_z);
        if (bt.u >= 0) {
            up[h] = bt.u;
            dn[h] = bt.d;
        }
    }
}

// Scores pair (d, u) for h exactly as best_pair does (the windows already
// passed) and keeps the better one.
template <int A, int B>
__device__ inline void score_pair(float hy, float hz, float yu, float zu, int32_t u, float yd, float zd,
                                  int32_t d, float cut_y, float cut_z, tpc_nb::Best &best) {
#pragma clang fp contract(off)
    constexpr float fa = (float)A, fb = (float)B;
    constexpr float g = 2.0f / (float)(A + B);
    const float ay = yu - hy, az = zu - hz;
    const float by = hy - yd, bz = hz - zd;
    const float ty = ay / fb, tz = az / fb;
    const float sy = by / fa, sz = bz / fa;
    const float ey = ty - sy;
    const float ez = tz - sz;
    const float dy = g * ey;
    const float dz = g * ez;
    if (!(fabsf(dy) <= cut_y && fabsf(dz) <= cut_z)) return;
    const float qy = dy * dy;
    const float qz = dz * dz;
    const float q = qy + qz;
    if (tpc_nb::better(q, u, d, best)) { best.q = q; best.u = u; best.d = d; }
}

// Every pair of the down row [d0, d1) (A rows below) and up row [u0, u1)
// (B rows above) inside the windows: the exact scan for an overflowing list.
template <int A, int B>
__device__ inline void scan_rows(float hy, float hz, const float *__restrict__ y, const float *__restrict__ z,
                                 int d0, int d1, int u0, int u1, float win_y, float win_z, float cut_y,
                                 float cut_z, tpc_nb::Best &best) {
#pragma clang fp contract(off)
    constexpr float fa = (float)A, fb = (float)B;
    for (int u = u0; u < u1; ++u) {
        const float yu = y[u], zu = z[u];
        const float ay = yu - hy, az = zu - hz;
        if (!(fabsf(ay) <= fb * win_y && fabsf(az) <= fb * win_z)) continue;
        for (int d = d0; d < d1; ++d) {
            const float yd = y[d], zd = z[d];
            const float by = hy - yd, bz = hz - zd;
            if (!(fabsf(by) <= fa * win_y && fabsf(bz) <= fa * win_z)) continue;
            score_pair<A, B>(hy, hz, yu, zu, u, yd, zd, d, cut_y, cut_z, best);
        }
    }
}

struct SegLds {
    float qy[SKIP_Q], qz[SKIP_Q];
    int32_t qh[SKIP_Q];
    float rz[SKIP_Q];                    // query z in ascending order
    int32_t rq[SKIP_Q];                  // ... and the query at each rank
    int32_t cnt[4 * SKIP_Q];             // candidates of (query q, row k) at 4 q + k
    int32_t cur[4 * SKIP_Q];             // cursors of the fill pass
    int32_t tot[SKIP_Q + 1];             // prefix of the queries' candidates
    int32_t pre[SKIP_Q];                 // prefix of the queries' pairs
    unsigned long long best[SKIP_Q];     // key of the best pair: bits of q, up id, down id (relative, 16 bits)
    float2 p[SKIP_POOL];                 // candidate coordinates
    uint16_t pool[SKIP_POOL];            // candidate positions within the partner row
    int scan_sh[TPC_BLOCK / TPC_WAVE];
};

// The queries in [q0, q1) whose window holds partner-row cluster (cy, cz):
// counted (FILL = false) or stored at the cursors (FILL = true).  Queries are
// ranked by z; fl(hz - cz) does not decrease with hz, so the ones passing
// |fl(hz - cz)| <= wz are a run of ranks, found by a binary search for its
// first member.  The predicates are those of best_pair: hz - cz for a row
// below (bz = z_h - z_d), cz - hz for a row above (az = z_u - z_h), whose
// magnitudes are equal.
template <bool FILL>
__device__ inline void window_hits(SegLds &L, int nq, int q0, int q1, int k, int rel, float cy, float cz, float wy,
                                   float wz) {
#pragma clang fp contract(off)
    int lo = 0, hi = nq;                     // first rank with hz - cz >= -wz
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (L.rz[mid] - cz >= -wz) hi = mid;
        else lo = mid + 1;
    }
    for (int j = lo; j < nq; ++j) {
        const float hz = L.rz[j];
        const float dz = k < 2 ? hz - cz : cz - hz;
        if (!(fabsf(dz) <= wz)) break;
        const int q = L.rq[j];
        const float hy = L.qy[q];
        const float dy = k < 2 ? hy - cy : cy - hy;
        if (fabsf(dy) <= wy && (!FILL || (q >= q0 && q < q1))) {
            if (FILL) {
                const int slot = atomicAdd(&L.cur[4 * q + k], 1);
                L.pool[slot] = (uint16_t)rel;
                L.p[slot] = make_float2(cy, cz);
            } else {
                atomicAdd(&L.cnt[4 * q + k], 1);
            }
        }
    }
}

// All clusters of the partner rows: the rows below, [ra[0] or ra[1], rb[1]),
// then those above, [ra[2], rb[2] or rb[3]), both without a gap; four clusters
// per thread are read at once.
template <bool FILL>
__device__ inline void window_pass(SegLds &L, int nq, int q0, int q1, const int ra[4], const int rb[4], bool lo2,
                                   bool hi2, const float *__restrict__ y, const float *__restrict__ z, float win_y,
                                   float win_z) {
#pragma clang fp contract(off)
    constexpr int U = 4;
    const int d0 = lo2 ? ra[0] : ra[1], nd = rb[1] - d0, nt = nd + (hi2 ? rb[3] : rb[2]) - ra[2];
    for (int i0 = threadIdx.x; i0 < nt; i0 += U * TPC_BLOCK) {
        float cy[U], cz[U];
        int c[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = i0 + j * TPC_BLOCK;
            c[j] = i < nd ? d0 + i : ra[2] + (i - nd);
            cy[j] = cz[j] = NAN;
            if (i < nt) {
                cy[j] = y[c[j]];
                cz[j] = z[c[j]];
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (!isfinite(cz[j])) continue;
            const bool below = i0 + j * TPC_BLOCK < nd;
            const int k = below ? (c[j] < ra[1] ? 0 : 1) : (c[j] < rb[2] ? 2 : 3);
            const int first = below ? (c[j] < ra[1] ? d0 : ra[1]) : (c[j] < rb[2] ? ra[2] : rb[2]);
            const float sc = (k == 0 || k == 3) ? 2.0f : 1.0f;     // rows away
            window_hits<FILL>(L, nq, q0, q1, k, c[j] - first, cy[j], cz[j], sc * win_y, sc * win_z);
        }
    }
}

// Scores pairs of the listed queries [q0, q1), dealt out over the workgroup:
// those of (A, B) = (1, 2) and (2, 1) together (FOUR = false), or the
// (2, 2) of the queries without one (FOUR = true).  The operations are those
// of score_pair: the divisions by 1 or 2 are exact products.  rel: first id
// of each partner row relative to the down rows' and the up rows' first.
template <bool FOUR>
__device__ inline void deal_pairs(SegLds &L, int q0, int q1, const int rel[4], float cut_y, float cut_z) {
#pragma clang fp contract(off)
    const int tid = threadIdx.x;
    int P = 0;
    if (tid >= q0 && tid < q1) {
        const int32_t *c = L.cnt + 4 * tid;
        P = FOUR ? (L.best[tid] == ~0ull ? c[0] * c[3] : 0) : c[1] * c[3] + c[0] * c[2];
    }
    int total;
    const int ex = block_exclusive_scan(P, L.scan_sh, &total);
    L.pre[tid] = ex;
    __syncthreads();
    for (int t = tid; t < total; t += TPC_BLOCK) {
        int q = 0;                                     // the last query whose pairs start at or before t
#pragma unroll
        for (int s = SKIP_Q / 2; s > 0; s >>= 1) q += L.pre[q + s] <= t ? s : 0;
        int j = t - L.pre[q];
        const int32_t *c = L.cnt + 4 * q, *e = L.cur + 4 * q;   // (cursors stand at the lists' ends)
        int kd = 0, ku = 3;
        if (!FOUR) {
            const int n12 = c[1] * c[3];
            kd = j < n12 ? 1 : 0;
            ku = j < n12 ? 3 : 2;
            j -= j < n12 ? 0 : n12;
        }
        const int nd = c[kd];
        const int iu = (int)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)nd));   // j / nd: j < 2^20
        const int u = e[ku] - c[ku] + iu, d = e[kd] - nd + (j - iu * nd);
        const float hy = L.qy[q], hz = L.qz[q];
        const float sb = ku == 3 ? 0.5f : 1.0f, sa = kd == 0 ? 0.5f : 1.0f;
        const float g = FOUR ? 2.0f / 4.0f : 2.0f / 3.0f;
        const float2 pu = L.p[u], pd = L.p[d];
        const float ty = (pu.x - hy) * sb, tz = (pu.y - hz) * sb;
        const float sy = (hy - pd.x) * sa, sz = (hz - pd.y) * sa;
        const float ey = ty - sy, ez = tz - sz;
        const float dy = g * ey, dz = g * ez;
        const float qy = dy * dy, qz = dz * dz;
        const float qq = qy + qz;
        const unsigned long long key = ((unsigned long long)__float_as_uint(qq) << 32) |
                                       (uint32_t)(rel[ku] + L.pool[u]) << 16 | (uint32_t)(rel[kd] + L.pool[d]);
        if (fabsf(dy) <= cut_y && fabsf(dz) <= cut_z) atomicMin(&L.best[q], key);
    }
    __syncthreads();
}

// Bound by the chains of LDS reads of the window passes and, where a thread
// scored the pairs of a query alone, by the longest of those: 262 -> 145 us
// for an event of 10^4 tracks with one row in ten missing (the pool of 1024
// was also too small for its inner rows, whose queries then scanned whole
// rows).
__global__ void __launch_bounds__(TPC_BLOCK)
skip_seg(const int32_t *__restrict__ off, int32_t n_rows, const float *__restrict__ y,
         const float *__restrict__ z, float win_y, float win_z, float cut_y, float cut_z, int32_t *up,
         int32_t *dn, int32_t *count) {
#pragma clang fp contract(off)
    static_assert(4 * SKIP_ROW_MAX <= 65535 && SKIP_Q == TPC_BLOCK, "16-bit ids, a thread per query");
    __shared__ SegLds L;
    if (blockIdx.x == 0 && threadIdx.x == 0) *count = 0;       // of skip_prep
    // rows in ascending order over all sectors: the inner rows, which hold
    // the most clusters (loopers) and take longest, start first; blocks go
    // round-robin over the XCDs, so each gets a share of every row
    const int n_fs = gridDim.x / n_rows;
    const int r = blockIdx.x / n_fs;
    const int seg = (blockIdx.x % n_fs) * n_rows + r;
    if (r < 1 || r > n_rows - 2) return;
    const bool lo2 = r >= 2, hi2 = r <= n_rows - 3;
    if (!lo2 && !hi2) return;
    const int a = off[seg], b = off[seg + 1];
    if (a == b || skip_large(off, seg, n_rows)) return;
    int ra[4], rb[4];                         // rows r-2, r-1, r+1, r+2
    partner_row(off, seg, r, n_rows, -2, ra[0], rb[0]);
    partner_row(off, seg, r, n_rows, -1, ra[1], rb[1]);
    partner_row(off, seg, r, n_rows, 1, ra[2], rb[2]);
    partner_row(off, seg, r, n_rows, 2, ra[3], rb[3]);
    const int d0 = lo2 ? ra[0] : ra[1], u0 = ra[2];
    const int rel[4] = {0, ra[1] - d0, 0, hi2 ? ra[3] - u0 : 0};
    const int tid = threadIdx.x;
    for (int c0 = a; c0 < b; c0 += SKIP_Q) {
        const int h = c0 + tid;
        int uh = 0;
        float hy0 = 0.f, hz0 = 0.f;
        if (h < b) {
            uh = up[h];
            hy0 = y[h];
            hz0 = z[h];
        }
        // unlinked and finite (a non-finite cluster never links)
        const int unl = h < b && uh < 0 && isfinite(hy0) && isfinite(hz0);
        int nq;
        const int pos = block_exclusive_scan(unl, L.scan_sh, &nq);
        if (nq == 0) continue;                // uniform
        if (unl) {
            L.qh[pos] = h;
            L.qy[pos] = hy0;
            L.qz[pos] = hz0;
        }
        for (int k = tid; k < 4 * SKIP_Q; k += TPC_BLOCK) L.cnt[k] = 0;
        L.best[tid] = ~0ull;
        __syncthreads();
        // rank by z (ties by position): a permutation, as every z is finite
        if (tid < nq) {
            const float v = L.qz[tid];
            int rk = 0;
            for (int j = 0; j < nq; ++j) {
                const float w = L.qz[j];
                rk += (w < v) | ((w == v) & (j < tid));
            }
            L.rz[rk] = v;
            L.rq[rk] = tid;
        }
        __syncthreads();
        window_pass<false>(L, nq, 0, nq, ra, rb, lo2, hi2, y, z, win_y, win_z);
        __syncthreads();
        int c[4] = {0, 0, 0, 0}, total;
        if (tid < nq) {
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = L.cnt[4 * tid + k];
        }
        const int own = c[0] + c[1] + c[2] + c[3];
        const int before = block_exclusive_scan(own, L.scan_sh, &total);
        L.tot[tid] = before;
        if (tid == 0) L.tot[SKIP_Q] = total;
        __syncthreads();
        // as many queries at a time as the pool holds the candidates of
        for (int q0 = 0, q1; q0 < nq; q0 = q1) {
            q1 = q0;
            for (int s = SKIP_Q; s > 0; s >>= 1)
                if (q1 + s <= nq && L.tot[q1 + s] - L.tot[q0] <= SKIP_POOL) q1 += s;
            if (q1 == q0) {                   // not even one: by its thread alone
                q1 = q0 + 1;
                if (tid == q0) {
                    const float hy = L.qy[tid], hz = L.qz[tid];
                    tpc_nb::Best bt = {0.f, -1, -1}, c2 = {0.f, -1, -1};
                    if (hi2)
                        scan_rows<1, 2>(hy, hz, y, z, ra[1], rb[1], ra[3], rb[3], win_y, win_z, cut_y, cut_z, bt);
                    if (lo2)
                        scan_rows<2, 1>(hy, hz, y, z, ra[0], rb[0], ra[2], rb[2], win_y, win_z, cut_y, cut_z, c2);
                    if (c2.u >= 0 && tpc_nb::better(c2.q, c2.u, c2.d, bt)) bt = c2;
                    if (bt.u < 0 && lo2 && hi2)
                        scan_rows<2, 2>(hy, hz, y, z, ra[0], rb[0], ra[3], rb[3], win_y, win_z, cut_y, cut_z, bt);
                    if (bt.u >= 0) {
                        up[L.qh[tid]] = bt.u;
                        dn[L.qh[tid]] = bt.d;
                    }
                }
                continue;
            }
            __syncthreads();
            if (tid >= q0 && tid < q1) {
                int at = before - L.tot[q0];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    L.cur[4 * tid + k] = at;
                    at += c[k];
                }
            }
            __syncthreads();
            window_pass<true>(L, nq, q0, q1, ra, rb, lo2, hi2, y, z, win_y, win_z);
            __syncthreads();
            deal_pairs<false>(L, q0, q1, rel, cut_y, cut_z);
            if (lo2 && hi2) deal_pairs<true>(L, q0, q1, rel, cut_y, cut_z);
            if (tid >= q0 && tid < q1) {
                const unsigned long long best = L.best[tid];
                if (best != ~0ull) {
                    up[L.qh[tid]] = u0 + (int32_t)((uint32_t)best >> 16);
                    dn[L.qh[tid]] = d0 + (int32_t)(best & 0xFFFFu);
                }
            }
        }
        __syncthreads();
    }
}

}  // namespace

size_t skip_ws_layout(void *ws, int64_t N, int64_t NR, SkipWs *out) {
    const size_t nb = nb_ws_layout(ws, N, NR, out ? &out->nb : nullptr);
    WsCarver w(ws ? (void *)((char *)ws + nb) : nullptr);
    int2 *list = w.take<int2>(N > 0 ? N : 1);
    int32_t *count = w.take<int32_t>(1);
    if (out) {
        out->list = list;
        out->count = count;
    }
    return nb + ((w.off + 255) & ~size_t(255));
}

hipError_t launch_neighbours_skip(const tpc_context *ctx, const tpc_frames *fr, int32_t *up, int32_t *dn,
                                  const SkipWs &ws, hipStream_t st) {
    hipError_t e = launch_neighbours(ctx, fr, up, dn, ws.nb, st);
    if (e != hipSuccess) return e;
    const int NR = fr->n_frames * ctx->cfg.n_sectors * ctx->cfg.n_rows;
    const tpc_config &c = ctx->cfg;
    hipLaunchKernelGGL(skip_seg, dim3(NR), dim3(TPC_BLOCK), 0, st, fr->row_offsets, c.n_rows, fr->y, fr->z,
                       c.win_y, c.win_z, c.cut_y, c.cut_z, up, dn, ws.count);
    const bool sparse = (int64_t)fr->n_clusters < (int64_t)TPC_SPARSE_ROW * NR;
    const int gp = sparse && NR > TPC_SPARSE_GRID ? TPC_SPARSE_GRID : NR;
    hipLaunchKernelGGL(skip_prep, dim3(gp), dim3(TPC_BLOCK), 0, st, fr->row_offsets, NR, c.n_rows, fr->y, fr->z,
                       c.win_y, c.win_z, up, ws);
    int blocks = (int)(fr->n_clusters / (8 * TPC_BLOCK)) + 1;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(skip_query, dim3(blocks), dim3(TPC_BLOCK), 0, st, fr->row_offsets, c.n_rows, fr->y,
                       fr->z, c.win_y, c.win_z, c.cut_y, c.cut_z, ws, up, dn);
    return hipGetLastError();
}
