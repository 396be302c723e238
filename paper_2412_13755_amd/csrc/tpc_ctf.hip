// Track-model residual transform of a frame's clusters into flat integer
// arrays, the input of the entropy coder (gfx950).
//
//  ct_own_init     owner of every cluster := none
//  ct_own          workgroup per 64 tracks and 64 rows: 32-bit atomicMin of the
//                  kept tracks' indices on their clusters (lowest index owns)
//  ct_count        workgroup per 64 tracks: their own clusters, counted; the
//                  64's sums of kept tracks, row steps and second differences
//  ct_tapply       prefixes of those three over the tracks
//  ct_free         wavefront per segment: free clusters in id order (ballot
//                  prefixes), their split quantised values; the segment's
//                  count
//  ct_scan_segs    one workgroup: prefix of free clusters over segments (run
//                  between two ct_free passes: count, then emit)
//  ct_emit         wavefront per kept track: its own clusters compacted in row
//                  order into LDS, then each lane writes the row step and
//                  residuals of one cluster; the track record
#include "tpc_internal.hpp"

namespace {

struct CtArgs {
    const int32_t *row_offsets;
    const float *y, *z;
    int32_t N, NR, R, S;
    const int32_t *n_seeds;
    int32_t cap_seeds;
    const int32_t *frame, *sector, *rows, *status;
    float iy, iz;                 // 1 / quantisation step, single precision
    int32_t *own;                 // [N]
    int32_t *m;                   // [cap_seeds] own clusters of each kept track
    int32_t *kp, *dp, *rp;        // [cap_seeds + 1] prefixes: kept, row steps, residuals
    int32_t *fp;                  // [NR + 1] prefix of free clusters
    int32_t *bsum;                // [3 per 64 tracks] sums
    tpc_ctf_arrays out;
};

__device__ inline int32_t quant(float v, float inv) {
    const float s = v * inv;
    if (!(s > -1073741824.0f && s < 1073741824.0f)) return 0;
    return (int32_t)rintf(s);
}

__device__ inline int n_tracks(const CtArgs &A) {
    const int T = *A.n_seeds;
    return T < A.cap_seeds ? T : A.cap_seeds;
}

__global__ void __launch_bounds__(TPC_BLOCK) ct_own_init(CtArgs A) {
    for (int c = blockIdx.x * TPC_BLOCK + threadIdx.x; c < A.N; c += gridDim.x * TPC_BLOCK) A.own[c] = 0x7fffffff;
}

// An item is 64 consecutive tracks and CT_ROWS rows, read along the rows of
// the table (coalesced) into LDS and taken a row at a time along the tracks:
// consecutive tracks are of one sector, so the 64 clusters of a row lie in a
// few cache lines of `own`; along a track they lie in 64, and the memory
// side takes atomics line by line (45 -> 29 us for 2.6 10^4 tracks).
#define CT_TILE TPC_WAVE
#define CT_ROWS 64
__global__ void __launch_bounds__(TPC_BLOCK) ct_own(CtArgs A) {
    __shared__ int32_t tile[CT_TILE][CT_ROWS + 1];
    constexpr int W = TPC_BLOCK / TPC_WAVE;
    const int T = n_tracks(A);
    const int lane = threadIdx.x & (TPC_WAVE - 1), wid = threadIdx.x / TPC_WAVE;
    const int chunks = (A.R + CT_ROWS - 1) / CT_ROWS;
    for (int64_t i = blockIdx.x; i / chunks * CT_TILE < T; i += gridDim.x) {
        const int t0 = (int)(i / chunks) * CT_TILE, r0 = (int)(i % chunks) * CT_ROWS;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < CT_TILE / W; ++k) {
            const int t = t0 + wid + k * W, r = r0 + lane;
            int c = -1;
            if (t < T && r < A.R && A.status[t] == TPC_FIT_OK) c = A.rows[(size_t)t * A.R + r];
            tile[wid + k * W][lane] = c;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < CT_ROWS / W; ++k) {
            const int c = tile[lane][wid + k * W];
            if ((uint32_t)c < (uint32_t)A.N) atomicMin(&A.own[c], t0 + lane);
        }
    }
}

// Kept, row steps, residuals of a track with m own clusters.
__device__ inline void track_vals(bool kept, int m, int v[3]) {
    v[0] = kept ? 1 : 0;
    v[1] = kept && m > 1 ? m - 1 : 0;
    v[2] = kept && m > 2 ? m - 2 : 0;
}

// A workgroup counts CT_TILE tracks, a wavefront CT_TILE / 16 of them at once.
// Beyond CT_COUNT_ALL tracks the rows of those that are not kept are not read
// (most of them, where tracks are dense: 322 -> 133 us for 6.4 10^5); up to
// there waiting for the status first costs more (300 tracks: 2 us).
#define CT_COUNT_T 1024
#define CT_COUNT_ALL 65536
__global__ void __launch_bounds__(CT_COUNT_T) ct_count(CtArgs A) {
    constexpr int U = CT_TILE / (CT_COUNT_T / TPC_WAVE);
    __shared__ int cnt[CT_TILE];
    const int T = n_tracks(A);
    const int lane = threadIdx.x & (TPC_WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / TPC_WAVE);
    for (int t0 = blockIdx.x * CT_TILE; t0 < T; t0 += gridDim.x * CT_TILE) {
        int n[U] = {};
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + wid * U + u;
            ok[u] = t < T && (T <= CT_COUNT_ALL || A.status[t] == TPC_FIT_OK);
        }
        for (int r = lane; r - lane < A.R; r += TPC_WAVE) {
            int c[U];
            bool own[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                c[u] = ok[u] && r < A.R ? A.rows[(size_t)(t0 + wid * U + u) * A.R + r] : -1;
#pragma unroll
            for (int u = 0; u < U; ++u) own[u] = (uint32_t)c[u] < (uint32_t)A.N && A.own[c[u]] == t0 + wid * U + u;
#pragma unroll
            for (int u = 0; u < U; ++u) n[u] += __popcll(__ballot(own[u]));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (lane == 0) cnt[wid * U + u] = n[u];
        __syncthreads();
        if (wid == 0) {
            const int t = t0 + lane;
            const bool kept = t < T && A.status[t] == TPC_FIT_OK;
            const int m = kept ? cnt[lane] : 0;
            if (t < T) A.m[t] = m;
            int v[3];
            track_vals(kept, m, v);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int sum = __builtin_amdgcn_readlane(lane_scan(v[k]), TPC_WAVE - 1);
                if (lane == 0) A.bsum[t0 / CT_TILE * 3 + k] = sum;
            }
        }
        __syncthreads();
    }
}

// Exclusive scans of the three counts: every workgroup sums the 64s' sums
// before its tracks itself, and takes CT_SPAN 64s (with four, 2.5 10^6 tracks
// read 2.3 GB of sums); the last one has the totals.
#define CT_SPAN 16
__global__ void __launch_bounds__(TPC_BLOCK) ct_tapply(CtArgs A) {
    static_assert(CT_SPAN <= TPC_WAVE, "a lane per 64 tracks");
    constexpr int W = TPC_BLOCK / TPC_WAVE;
    __shared__ int sh[3][W];
    const int T = n_tracks(A);
    const int lane = threadIdx.x & (TPC_WAVE - 1), wid = threadIdx.x / TPC_WAVE;
    const int tiles = T > 0 ? (T + CT_TILE - 1) / CT_TILE : 0, b0 = blockIdx.x * CT_SPAN;
    if (b0 > 0 && b0 >= tiles) return;
    constexpr int Q = CT_SPAN / W;                   // 64s per wavefront
    int before[3] = {0, 0, 0}, mine[3], own[3], v[Q][3];
    for (int b = threadIdx.x; b < b0; b += TPC_BLOCK)
#pragma unroll
        for (int k = 0; k < 3; ++k) before[k] += A.bsum[b * 3 + k];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int t = (b0 + wid + q * W) * CT_TILE + lane;
        track_vals(t < T && A.status[t] == TPC_FIT_OK, t < T ? A.m[t] : 0, v[q]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        before[k] = __builtin_amdgcn_readlane(lane_scan(before[k]), TPC_WAVE - 1);
        if (lane == 0) sh[k][wid] = before[k];
        own[k] = lane < CT_SPAN && b0 + lane < tiles ? A.bsum[(b0 + lane) * 3 + k] : 0;
        mine[k] = lane_scan(own[k]);                 // lane: the sums up to its 64's end
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        before[k] = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) before[k] += sh[k][w];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int t = (b0 + wid + q * W) * CT_TILE + lane;
        int at[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            at[k] = before[k] + __shfl(mine[k] - own[k], wid + q * W, TPC_WAVE) + lane_scan(v[q][k]) - v[q][k];
        if (t < T) {
            A.kp[t] = at[0];
            A.dp[t] = at[1];
            A.rp[t] = at[2];
        }
    }
    if (threadIdx.x == TPC_WAVE - 1 && b0 + CT_SPAN >= tiles) {
        const int kept = before[0] + mine[0], steps = before[1] + mine[1], res = before[2] + mine[2];
        const int e = T > 0 ? T : 0;
        A.kp[e] = kept;
        A.dp[e] = steps;
        A.rp[e] = res;
        for (int k = 0; k < 9; ++k) A.out.counts[k] = kept;
        A.out.counts[9] = steps;
        A.out.counts[10] = res;
        A.out.counts[11] = res;
        A.out.counts[12] = A.NR;
    }
}

// EMIT == false: count the segment's free clusters into fp[s];
// EMIT == true: write them at fp[s] (the prefix by then) in id order.
template <bool EMIT>
__global__ void __launch_bounds__(TPC_BLOCK) ct_free(CtArgs A) {
    constexpr int U = 4;                                // wavefronts' worth of clusters in flight
    const int s = xcd_item(blockIdx.x, gridDim.x) * (TPC_BLOCK / TPC_WAVE) + threadIdx.x / TPC_WAVE;
    if (s >= A.NR) return;
    const int lane = threadIdx.x & (TPC_WAVE - 1);
    const int a = A.row_offsets[s], b = A.row_offsets[s + 1];
    const int first = EMIT ? A.fp[s] : 0;
    int base = first;
    for (int c0 = a + lane; c0 - lane < b; c0 += U * TPC_WAVE) {
        bool fr[U];
        float y[U], z[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int c = c0 + j * TPC_WAVE;
            fr[j] = c < b && A.own[c] == 0x7fffffff;
            if (EMIT) {
                y[j] = c < b ? A.y[c] : 0.f;
                z[j] = c < b ? A.z[c] : 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t m = __ballot(fr[j]);
            if (EMIT && fr[j]) {
                const int32_t qy = quant(y[j], A.iy), qz = quant(z[j], A.iz);
                const int o = base + lanes_below(m);
                A.out.free_yh[o] = qy >> 8;
                A.out.free_yl[o] = qy & 255;
                A.out.free_zh[o] = qz >> 8;
                A.out.free_zl[o] = qz & 255;
            }
            base += __popcll(m);
        }
    }
    if (lane == 0) (EMIT ? A.out.seg_nfree : A.fp)[s] = base - first;
}

// Prefix over the segments: a thread sums its run of them, and writes the
// run's prefixes from where the scan of the runs' sums puts it.
#define CT_SCAN_T 1024
__global__ void __launch_bounds__(CT_SCAN_T) ct_scan_segs(CtArgs A) {
    __shared__ int sh[CT_SCAN_T / TPC_WAVE];
    const int lane = threadIdx.x & (TPC_WAVE - 1), wid = threadIdx.x / TPC_WAVE;
    const int k = (A.NR + CT_SCAN_T - 1) / CT_SCAN_T;
    const int s0 = min((int)threadIdx.x * k, A.NR), s1 = min(s0 + k, A.NR);
    int sum = 0;
    for (int s = s0; s < s1; ++s) sum += A.fp[s];
    const int inc = lane_scan(sum);
    if (lane == TPC_WAVE - 1) sh[wid] = inc;
    __syncthreads();
    int run = inc - sum, total = 0;
#pragma unroll
    for (int w = 0; w < CT_SCAN_T / TPC_WAVE; ++w) {
        run += w < wid ? sh[w] : 0;
        total += sh[w];
    }
    for (int s = s0; s < s1; ++s) {
        const int v = A.fp[s];
        A.fp[s] = run;
        run += v;
    }
    if (threadIdx.x == 0) {
        A.fp[A.NR] = total;
        for (int j = 13; j < 17; ++j) A.out.counts[j] = total;
    }
}

// Wavefront per kept track: its own clusters compacted in row order into LDS,
// then lane k writes what cluster k contributes.  (A workgroup per track
// spent its time at its barriers: 49 -> 28 us for 2.6 10^4 tracks.)
__global__ void __launch_bounds__(TPC_BLOCK) ct_emit(CtArgs A) {
    constexpr int U = 4, W = TPC_BLOCK / TPC_WAVE;
    __shared__ int ly[W][TPC_MAX_ROWS], lz[W][TPC_MAX_ROWS], lr[W][TPC_MAX_ROWS];
    const int T = n_tracks(A);
    const int lane = threadIdx.x & (TPC_WAVE - 1), wid = threadIdx.x / TPC_WAVE;
    int *sy = ly[wid], *sz = lz[wid], *sr = lr[wid];
    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    for (int t = blockIdx.x * W + wid; t < T; t += gridDim.x * W) {
        const int32_t *rw = A.rows + (size_t)t * A.R;
        const int d = A.dp[t], g = A.rp[t], k0 = A.kp[t], seg = A.frame[t] * A.S + A.sector[t];
        if (A.status[t] != TPC_FIT_OK) continue;        // uniform over the wavefront
        int m = 0;
        for (int r0 = lane; r0 - lane < A.R; r0 += U * TPC_WAVE) {
            int c[U];
            bool mine[U];
            float y[U], z[U];
#pragma unroll
            for (int j = 0; j < U; ++j) c[j] = r0 + j * TPC_WAVE < A.R ? rw[r0 + j * TPC_WAVE] : -1;
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const bool in = (uint32_t)c[j] < (uint32_t)A.N;
                mine[j] = in && A.own[c[j]] == t;
                y[j] = in ? A.y[c[j]] : 0.f;
                z[j] = in ? A.z[c[j]] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint64_t b = __ballot(mine[j]);
                if (mine[j]) {
                    const int k = m + lanes_below(b);
                    sy[k] = quant(y[j], A.iy);
                    sz[k] = quant(z[j], A.iz);
                    sr[k] = r0 + j * TPC_WAVE;
                }
                m += __popcll(b);
            }
        }
        fence();
        for (int k = lane; k < m; k += TPC_WAVE) {
            if (k >= 1) A.out.hit_drow[d + k - 1] = sr[k] - sr[k - 1] - 1;
            if (k >= 2) {
                A.out.hit_ry[g + k - 2] = sy[k] - 2 * sy[k - 1] + sy[k - 2];
                A.out.hit_rz[g + k - 2] = sz[k] - 2 * sz[k - 1] + sz[k - 2];
            }
        }
        if (lane == 0) {
            const int qy0 = m ? sy[0] : 0, qz0 = m ? sz[0] : 0;
            A.out.trk_seg[k0] = seg;
            A.out.trk_n[k0] = m;
            A.out.trk_row0[k0] = m ? sr[0] : 0;
            A.out.trk_y0h[k0] = qy0 >> 8;
            A.out.trk_y0l[k0] = qy0 & 255;
            A.out.trk_z0h[k0] = qz0 >> 8;
            A.out.trk_z0l[k0] = qz0 & 255;
            A.out.trk_dy1[k0] = m >= 2 ? sy[1] - qy0 : 0;
            A.out.trk_dz1[k0] = m >= 2 ? sz[1] - qz0 : 0;
        }
        fence();
    }
}

int grid_for(int64_t items) {
    int64_t b = (items + TPC_BLOCK - 1) / TPC_BLOCK;
    if (b > 8192) b = 8192;
    return b < 1 ? 1 : (int)b;
}

}  // namespace

size_t ctf_ws_layout(void *ws, int64_t N, int64_t NR, int64_t cap_seeds, void *out) {
    WsCarver w(ws);
    int32_t *own = w.take<int32_t>(N > 0 ? N : 1);
    int32_t *m = w.take<int32_t>(cap_seeds > 0 ? cap_seeds : 1);
    int32_t *kp = w.take<int32_t>(cap_seeds + 1);
    int32_t *dp = w.take<int32_t>(cap_seeds + 1);
    int32_t *rp = w.take<int32_t>(cap_seeds + 1);
    int32_t *fp = w.take<int32_t>(NR + 1);
    int32_t *bs = w.take<int32_t>(3 * ((cap_seeds + CT_TILE - 1) / CT_TILE + 1));
    if (out) {
        int32_t **p = static_cast<int32_t **>(out);
        p[0] = own; p[1] = m; p[2] = kp; p[3] = dp; p[4] = rp; p[5] = fp; p[6] = bs;
    }
    return (w.off + 255) & ~size_t(255);
}

hipError_t launch_ctf_build(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd,
                            const int32_t *rows, const tpc_tracks *tr, float qy, float qz,
                            const tpc_ctf_arrays *out, void *ws, hipStream_t st) {
    const tpc_config &c = ctx->cfg;
    CtArgs A;
    A.row_offsets = fr->row_offsets;
    A.y = fr->y;
    A.z = fr->z;
    A.N = fr->n_clusters;
    A.NR = fr->n_frames * c.n_sectors * c.n_rows;
    A.R = c.n_rows;
    A.S = c.n_sectors;
    A.n_seeds = sd->n_seeds;
    A.cap_seeds = sd->cap_seeds;
    A.frame = sd->frame;
    A.sector = sd->sector;
    A.rows = rows;
    A.status = tr->status;
    A.iy = 1.0f / qy;
    A.iz = 1.0f / qz;
    int32_t *p[7];
    ctf_ws_layout(ws, A.N, A.NR, A.cap_seeds, p);
    A.own = p[0];
    A.m = p[1];
    A.kp = p[2];
    A.dp = p[3];
    A.rp = p[4];
    A.fp = p[5];
    A.bsum = p[6];
    A.out = *out;
    constexpr int W = TPC_BLOCK / TPC_WAVE;
    const int64_t tiles = ((int64_t)A.cap_seeds + CT_TILE - 1) / CT_TILE, chunks = (A.R + CT_ROWS - 1) / CT_ROWS;
    const int segs = A.NR > 0 ? (A.NR + W - 1) / W : 1;
    hipLaunchKernelGGL(ct_own_init, dim3(grid_for(A.N)), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(ct_own, dim3(grid_for(tiles * chunks * TPC_BLOCK)), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(ct_count, dim3(grid_for(tiles * TPC_BLOCK)), dim3(CT_COUNT_T), 0, st, A);
    hipLaunchKernelGGL(ct_tapply, dim3((unsigned)(tiles > 0 ? (tiles + CT_SPAN - 1) / CT_SPAN : 1)), dim3(TPC_BLOCK),
                       0, st, A);
    hipLaunchKernelGGL(ct_free<false>, dim3(segs), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(ct_scan_segs, dim3(1), dim3(CT_SCAN_T), 0, st, A);
    hipLaunchKernelGGL(ct_free<true>, dim3(segs), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(ct_emit, dim3(grid_for((int64_t)A.cap_seeds * TPC_WAVE)), dim3(TPC_BLOCK), 0, st, A);
    return hipGetLastError();
}
