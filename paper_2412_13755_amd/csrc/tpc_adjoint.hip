// Adjoint of the summed fit chi2 with respect to the per-(sector, row)
// cluster correction map (gfx950).
//
// L(M) = sum over successfully fitted seeds of chi2, with every cluster of
// (sector s, row r) corrected by -M[s][r]; dL/dM[s][r] = -(sum of dL/dm over
// the hits of (s, r)), scaled by the caller's upstream gradient dloss.
//
//  adj_tracks   one thread per seed, longest first, reverse mode by hand: for
//               each segment of ckpt_rows filter steps, from the innermost
//               backwards, restart from the forward checkpoint and recompute
//               the segment, keeping every fourth filter state in a
//               per-thread tape (global memory, laid out so a wavefront's
//               accesses are contiguous); then, from the last, recompute four
//               steps with their states in LDS and run the step adjoints over
//               them; finally the three-point start.  Writes dL/dm per seed
//               hit.
//  adj_partial  deterministic per-(frame, sector) sums per row: seeds of one
//               (frame, sector) are contiguous (seeds are ordered by their
//               first cluster id); each wavefront sums fixed chunks of them in
//               seed order
//  adj_final    fixed-order sum of the partials, times -dloss
#include "tpc_fit_common.hpp"

namespace {

struct AdjArgs {
    FitArgs F;
    const int32_t *status;
    const double *ckpt;
    float2 *g;          // [cap_hits] dL/d(my, mz) per seed hit
    double *tape;       // [threads / 64][adj_tape_states(K)][TPC_CKPT_WORDS][64]
    int32_t nthreads;
};

// Seed slot `gt` of pass `k` over the length order: passes run alternately
// up and down the threads, so that the wavefronts with the longest seeds of
// one pass take the shortest of the next.
__device__ inline int64_t snake(int64_t k, int gt, int nthreads) {
    return k * nthreads + ((k & 1) ? nthreads - 1 - gt : gt);
}

// Two wavefronts per SIMD (256 registers per lane, nothing spilled): one
// leaves the latency of its chain of operations exposed.  Seeds in descending length order (F.order): a
// wavefront runs as many steps as its longest seed, and seeds in their own
// order (12 hits on average, up to 151) left most lanes idle: one gradient
// of 645 000 seeds 3.15 -> 1.83 ms, and 1.06 since (735 us of it here).
__global__ void __launch_bounds__(TPC_BLOCK) __attribute__((amdgpu_waves_per_eu(2)))
adj_tracks(AdjArgs A) {
    // two states per thread: half of a CU's LDS, for half of its threads
    __shared__ double lt[(TPC_ADJ_SUB - 2) * TPC_CKPT_WORDS * TPC_BLOCK];
    const FitArgs &F = A.F;
    int T = *F.n_seeds;
    if (T > F.cap_seeds) T = F.cap_seeds;
    const int gt = blockIdx.x * TPC_BLOCK + threadIdx.x;
    const int K = adj_tape_states(F.ckpt_rows);
    // this wavefront's tape: word q of state s of lane l at
    // tp[(s * TPC_CKPT_WORDS + q) * 64 + l], so the 64 lanes touch one
    // contiguous 512-byte run
    const int wave = __builtin_amdgcn_readfirstlane(gt / TPC_WAVE);
    double *tp = A.tape + (size_t)wave * K * TPC_CKPT_WORDS * TPC_WAVE;
    if (F.order) T = *F.n_order < T ? *F.n_order : T;
    for (int64_t k = 0; k * A.nthreads < T; ++k) {
        const int64_t j = snake(k, gt, A.nthreads);
        if (j >= T) continue;
        const int i = F.order ? F.order[j] : (int)j;
        if ((uint32_t)i < (uint32_t)F.cap_seeds) 
            adj_one(F, A.status, A.ckpt, A.g, i, tp, threadIdx.x % TPC_WAVE, lt + threadIdx.x, TPC_BLOCK);
    }
}

// key of seed i: frame * n_sectors + sector (non-decreasing over seeds)
__device__ inline int seed_key(const int32_t *frame, const int32_t *sector, int n_sectors, int i) {
    return frame[i] * n_sectors + sector[i];
}

// First of the T seeds whose key is not below `key` (one whole wavefront, 64
// probes a step: four steps of dependent reads for 10^6 seeds, not twenty).
__device__ inline int lower_bound_key(const int32_t *frame, const int32_t *sector, int n_sectors,
                                      int T, int key) {
    const int lane = threadIdx.x & (TPC_WAVE - 1);
    int lo = 0, hi = T;
    while (hi > lo) {
        const int step = (hi - lo + TPC_WAVE - 1) / TPC_WAVE;
        const int64_t i = lo + (int64_t)lane * step;
        const int below = __popcll(__ballot(i < hi && seed_key(frame, sector, n_sectors, (int)i) < key));
        // the answer lies above probe below - 1, at most at probe below
        const int64_t top = lo + (int64_t)below * step;
        if (below > 0) lo += (below - 1) * step + 1;
        hi = top < hi ? (int)top : hi;
    }
    return lo;
}

// A wavefront takes 64 seeds at a time and adds their hits' gradients to its
// own row sums in LDS (read, add, write: LDS float atomics took three times as
// long), a seed per instruction, lane k its k-th hit: the reads are
// contiguous, TPC_ADJ_AHEAD seeds' are in flight, and a wavefront's adds
// happen in its order, so the sums are reproducible.  (A thread per row
// walking over the seeds that cross it read one value at a time: 285 -> 38 us
// for 645 000 seeds.)
#define TPC_ADJ_AHEAD 8
__global__ void __launch_bounds__(TPC_BLOCK)
adj_partial(const int32_t *__restrict__ n_seeds, int32_t cap_seeds, int32_t cap_hits,
            const int32_t *__restrict__ offsets, const int32_t *__restrict__ first_row,
            const int32_t *__restrict__ frame, const int32_t *__restrict__ sector,
            int32_t n_sectors, int32_t n_rows, const float2 *__restrict__ g,
            float2 *__restrict__ partial) {
    constexpr int W = TPC_BLOCK / TPC_WAVE;
    __shared__ float2 sum[W][TPC_MAX_ROWS];
    __shared__ int range[2];
    const int fs = blockIdx.x, gsub = blockIdx.y, G = gridDim.y;
    const int lane = threadIdx.x & (TPC_WAVE - 1), wid = threadIdx.x / TPC_WAVE;
    if (wid < 2) {
        int T = *n_seeds;
        if (T > cap_seeds) T = cap_seeds;
        const int at = lower_bound_key(frame, sector, n_sectors, T, fs + wid);
        if (lane == 0) range[wid] = at;
    }
    for (int r = lane; r < n_rows; r += TPC_WAVE) sum[wid][r] = make_float2(0.f, 0.f);
    // (a plain read, add and write: the wavefront is the only one, and its lanes
    // have different rows; an LDS atomic took longer.  The next seed's lanes
    // add to rows that others of this one's have written: the fence keeps the
    // compiler, as the hardware does, from taking them out of order.)
    auto add = [&](bool act, int r, const float2 &v) {
        if (act) {
            const float2 a = sum[wid][r];
            sum[wid][r] = make_float2(a.x + v.x, a.y + v.y);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    __syncthreads();
    const int hi = range[1];
    for (int64_t c0 = range[0] + (int64_t)(gsub * W + wid) * TPC_WAVE; c0 < hi; c0 += (int64_t)G * W * TPC_WAVE) {
        const int i = (int)c0 + lane;
        int so = 0, sn = 0, sr = 0;
        if (i < hi) {
            so = offsets[i];
            sn = offsets[i + 1] - so;
            sr = first_row[i];
            // seeds that fail the fit's sanity checks (seed_view) were never
            // written: those of a list that exceeded its hit capacity may
            // even end beyond g
            const bool sane = sn >= 3 && sr >= 0 && sr + sn <= n_rows && so >= 0 && so <= cap_hits - sn &&
                              (uint32_t)sector[i] < (uint32_t)n_sectors;
            if (!sane) sn = 0;
        }
        for (int q = 0; q < TPC_WAVE; q += TPC_ADJ_AHEAD) {
            float2 v[TPC_ADJ_AHEAD];
            int longest = 0;
#pragma unroll
            for (int u = 0; u < TPC_ADJ_AHEAD; ++u) {
                const int n = __builtin_amdgcn_readlane(sn, q + u), o = __builtin_amdgcn_readlane(so, q + u);
                v[u] = lane < n ? g[o + lane] : make_float2(0.f, 0.f);
                longest = max(longest, n);
            }
#pragma unroll
            for (int u = 0; u < TPC_ADJ_AHEAD; ++u) {
                const int n = __builtin_amdgcn_readlane(sn, q + u), r = __builtin_amdgcn_readlane(sr, q + u) + lane;
                add(lane < n, r, v[u]);
            }
            if (longest <= TPC_WAVE) continue;
            for (int k = lane + TPC_WAVE; k - lane < longest; k += TPC_WAVE) {
#pragma unroll
                for (int u = 0; u < TPC_ADJ_AHEAD; ++u) {
                    const int n = __builtin_amdgcn_readlane(sn, q + u), o = __builtin_amdgcn_readlane(so, q + u);
                    v[u] = k < n ? g[o + k] : make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int u = 0; u < TPC_ADJ_AHEAD; ++u) {
                    const int n = __builtin_amdgcn_readlane(sn, q + u), r = __builtin_amdgcn_readlane(sr, q + u) + k;
                    add(k < n, r, v[u]);
                }
            }
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < n_rows; r += TPC_BLOCK) {
        double ay = 0.0, az = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            ay += sum[w][r].x;
            az += sum[w][r].y;
        }
        partial[((size_t)fs * G + gsub) * n_rows + r] = make_float2((float)ay, (float)az);
    }
}

__global__ void __launch_bounds__(TPC_BLOCK)
adj_final(const float2 *__restrict__ partial, int32_t n_frames, int32_t n_sectors, int32_t n_rows,
          int32_t G, const float *__restrict__ dloss, float *__restrict__ grad) {
    const int idx = blockIdx.x * TPC_BLOCK + threadIdx.x;
    if (idx >= n_sectors * n_rows) return;
    const int s = idx / n_rows, r = idx % n_rows;
    double ay = 0.0, az = 0.0;
    for (int f = 0; f < n_frames; ++f)
#pragma unroll 8
        for (int q = 0; q < G; ++q) {
            const float2 v = partial[((size_t)(f * n_sectors + s) * G + q) * n_rows + r];
            ay += v.x;
            az += v.y;
        }
    const double d = dloss ? (double)*dloss : 1.0;
    grad[(size_t)idx * 2] = (float)(-d * ay);
    grad[(size_t)idx * 2 + 1] = (float)(-d * az);
}

}  // namespace

#define TPC_ADJ_MAX_BLOCKS 512     // persistent grid: 131072 threads, 8 waves per CU
// Workgroups per (frame, sector) in the row sums: enough for about 4096
// workgroups in all, at most 64 (each sums a fixed share of the seeds, so
// the result stays bit-reproducible).
static int adj_groups(int64_t n_fs) {
    int64_t g = n_fs > 0 ? 4096 / n_fs : 1;
    return (int)(g < 1 ? 1 : (g > 64 ? 64 : g));
}

static int adj_blocks(int32_t cap_seeds) {
    int b = (cap_seeds + TPC_BLOCK - 1) / TPC_BLOCK;
    if (b > TPC_ADJ_MAX_BLOCKS) b = TPC_ADJ_MAX_BLOCKS;
    return b < 1 ? 1 : b;
}

size_t adj_ws_layout(void *ws, int64_t cap_hits, int64_t cap_seeds, int64_t n_fs, int32_t n_rows,
                     int32_t K, float2 **g, double **tape, float2 **partial, float2 **hyz, FitOrderWs *ord) {
    WsCarver w(ws);
    float2 *pg = w.take<float2>(cap_hits > 0 ? cap_hits : 1);
    const int64_t nthreads = (int64_t)adj_blocks((int32_t)(cap_seeds < 0x7fffffff ? cap_seeds : 0x7fffffff)) * TPC_BLOCK;
    double *pt = w.take<double>(nthreads * adj_tape_states(K) * TPC_CKPT_WORDS);
    float2 *pp = w.take<float2>(n_fs * adj_groups(n_fs) * n_rows);
    float2 *ph = w.take<float2>(cap_hits > 0 ? cap_hits : 1);
    const FitOrderWs o = fit_order_carve(w, cap_seeds);
    if (ord) *ord = o;
    if (hyz) *hyz = ph;
    if (g) *g = pg;
    if (tape) *tape = pt;
    if (partial) *partial = pp;
    return (w.off + 255) & ~size_t(255);
}

hipError_t launch_adjoint(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd,
                          const float *map, const tpc_tracks *tr, const double *ckpt,
                          const float *dloss, float *grad_map, void *ws, hipStream_t st) {
    const tpc_config &c = ctx->cfg;
    const int64_t n_fs = (int64_t)fr->n_frames * c.n_sectors;
    AdjArgs A;
    A.F = make_fit_args(ctx, sd, map);
    A.status = tr->status;
    A.ckpt = ckpt;
    float2 *partial;
    float2 *hyz;
    FitOrderWs ord;
    adj_ws_layout(ws, sd->cap_hits, sd->cap_seeds, n_fs, c.n_rows, c.ckpt_rows, &A.g, &A.tape, &partial, &hyz, &ord);
    if (sd->hit_yz) {
        A.F.hyz = reinterpret_cast<const float2 *>(sd->hit_yz);
    } else {
        A.F.hyz = hyz;
        launch_gather(fr, sd, hyz, st);
    }
    if (sd->cap_seeds >= TPC_FIT_ORDER_MIN) launch_fit_order(A.F, ord, st);
    const int blocks = adj_blocks(sd->cap_seeds);
    A.nthreads = blocks * TPC_BLOCK;
    hipLaunchKernelGGL(adj_tracks, dim3(blocks), dim3(TPC_BLOCK), 0, st, A);
    const int groups = adj_groups(n_fs);
    hipLaunchKernelGGL(adj_partial, dim3((unsigned)n_fs, groups), dim3(TPC_BLOCK), 0, st,
                       sd->n_seeds, sd->cap_seeds, sd->cap_hits, sd->offsets, sd->first_row, sd->frame,
                       sd->sector, c.n_sectors, c.n_rows, A.g, partial);
    const int nout = c.n_sectors * c.n_rows;
    hipLaunchKernelGGL(adj_final, dim3((nout + TPC_BLOCK - 1) / TPC_BLOCK), dim3(TPC_BLOCK), 0, st,
                       partial, fr->n_frames, c.n_sectors, c.n_rows, groups, dloss, grad_map);
    return hipGetLastError();
}
