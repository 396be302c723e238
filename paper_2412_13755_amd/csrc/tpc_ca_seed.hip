// Seeding stage kernels; the work is in tpc_ca_device.hpp.
#include "tpc_ca_device.hpp"

namespace {

using namespace tpc_ca;

__global__ void __launch_bounds__(1024)
ca_block(int32_t N, int32_t n_rows, const int32_t *off, const int32_t *up, const int32_t *dn, CaWs ws) {
    __shared__ uint32_t W[TPC_CA_CAP];
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (ca_block_class(item, n_rows, off) == 1) return;
    ca_block_item(item, N, n_rows, off, up, dn, ws, W);
}

// Blocks too large for the LDS ranking with rows of at most
// TPC_CA_SWEEP_ROW clusters: ranked by a bottom-up row sweep.  A thread tests
// a block, so that a workgroup with few blocks to rank or none (the others
// it takes are ca_block's) does not wait for each one's row offsets.
__global__ void __launch_bounds__(1024)
ca_block_sweep(int32_t NB, int32_t N, int32_t n_rows, const int32_t *off, const int32_t *up, const int32_t *dn,
               CaWs ws) {
    __shared__ uint32_t P[2 * TPC_CA_SWEEP_ROW];
    const int tid = threadIdx.x;
    for (int64_t from = blockIdx.x; from < NB; from += (int64_t)gridDim.x * 1024) {
        const int64_t it = from + (int64_t)gridDim.x * tid;
        bool mine = it < NB && ca_block_class((int)it, n_rows, off) == 1;
        while (true) {                         // the blocks found, one after the other (P is all of the LDS)
            __syncthreads();
            if (tid == 0) P[0] = ~0u;
            __syncthreads();
            if (mine) atomicMin(&P[0], (uint32_t)tid);
            __syncthreads();
            const uint32_t w = P[0];
            __syncthreads();
            if (w == ~0u) break;
            if ((uint32_t)tid == w) mine = false;
            ca_sweep_item((int)(from + (int64_t)gridDim.x * w), N, n_rows, off, up, dn, ws, P);
        }
    }
}

__global__ void __launch_bounds__(TPC_BLOCK)
ca_tops(int32_t N, int32_t NR, const int32_t *up, const int32_t *dn, int32_t min_hits, int32_t n_rows, CaWs ws) {
    __shared__ CaTopsLds L;
    for (int64_t s = (int64_t)blockIdx.x * TPC_BLOCK + threadIdx.x; s < NR; s += (int64_t)gridDim.x * TPC_BLOCK) {
        ws.segcnt[s] = 0;                             // counted into by ca_firsts
        ws.seghits[s] = 0;
    }
    ca_tops_flat((int64_t)xcd_item(blockIdx.x, gridDim.x) * TPC_CA_FLAT, N, up, dn, min_hits, n_rows, ws, L);
}

// Wavefronts per segment: one where rows are small on average (there are
// then many, and launching a workgroup for each is what the time goes to:
// 64 uneven frames 577 -> 228 us), the four of a workgroup otherwise.
template <int PARTS>
__global__ void __launch_bounds__(TPC_BLOCK)
ca_firsts(int32_t N, int32_t NR, const int32_t *off, const int32_t *up, const int32_t *dn, int32_t min_hits,
          CaWs ws) {
    __shared__ int list[TPC_BLOCK / TPC_WAVE][2 * TPC_WAVE];
    constexpr int SEGS = TPC_BLOCK / TPC_WAVE / PARTS;
    const int wid = threadIdx.x / TPC_WAVE;
    const int seg = xcd_item(blockIdx.x, gridDim.x) * SEGS + wid / PARTS;
    if (seg < NR) ca_firsts_part(seg, wid % PARTS, PARTS, N, off, up, dn, min_hits, ws, list[wid]);
}

__device__ inline void put_totals(int seeds, int hits, int32_t *n_seeds, int32_t *n_hits, int32_t cap_seeds,
                                  int32_t cap_hits, int32_t *offsets, int32_t *dev_status) {
    *n_seeds = seeds;
    *n_hits = hits;
    const bool ok = seeds <= cap_seeds && hits <= cap_hits;
    *dev_status = ok ? TPC_OK : TPC_ERR_CAPACITY;
    if (seeds <= cap_seeds) offsets[seeds] = ok ? hits : 0;
}

// Single workgroup: exclusive scan of n (seed count, hit count) pairs into
// (pre_c, pre_h), totals into *n_seeds / *n_hits with the capacity check.
// Thread t owns the contiguous run [t k, (t+1) k), k = ceil(n / 1024): it
// sums its run, one workgroup scan turns run sums into run starts, and it
// writes the prefixes of its run.  Used on the segments directly when they
// are few, else on the chunk sums of ca_chunk_sums.
__global__ void __launch_bounds__(1024)
ca_scan(int32_t n, const int32_t *cnt, const int32_t *hits, int32_t *pre_c, int32_t *pre_h,
        int32_t *__restrict__ n_seeds,
        int32_t *__restrict__ n_hits, int32_t cap_seeds, int32_t cap_hits, int32_t *__restrict__ offsets,
        int32_t *__restrict__ dev_status) {
    __shared__ int shc[1024 / TPC_WAVE], shh[1024 / TPC_WAVE];
    const int tid = threadIdx.x, lane = tid & (TPC_WAVE - 1), wid = tid / TPC_WAVE;
    const int k = (n + 1023) / 1024;
    const int s0 = tid * k < n ? tid * k : n;
    const int s1 = s0 + k < n ? s0 + k : n;
    int vc = 0, vh = 0;
    for (int s = s0; s < s1; ++s) {
        vc += cnt[s];
        vh += hits[s];
    }
    const int ic = wave_inclusive_scan(vc), ih = wave_inclusive_scan(vh);
    if (lane == TPC_WAVE - 1) { shc[wid] = ic; shh[wid] = ih; }
    __syncthreads();
    int bc = 0, bh = 0, tc = 0, th = 0;
#pragma unroll
    for (int w = 0; w < 1024 / TPC_WAVE; ++w) {
        bc += w < wid ? shc[w] : 0;
        bh += w < wid ? shh[w] : 0;
        tc += shc[w];
        th += shh[w];
    }
    int pc = bc + ic - vc, ph = bh + ih - vh;
    for (int s = s0; s < s1; ++s) {              // in place allowed: read before write
        const int c = cnt[s], h = hits[s];
        pre_c[s] = pc;
        pre_h[s] = ph;
        pc += c;
        ph += h;
    }
    if (tid == 0) put_totals(tc, th, n_seeds, n_hits, cap_seeds, cap_hits, offsets, dev_status);
}

// Many segments: sums of chunks of TPC_SCAN_CHUNK segments (one workgroup
// per chunk) ...
__global__ void __launch_bounds__(TPC_BLOCK)
ca_chunk_sums(int32_t NR, CaWs ws) {
    __shared__ int sh[TPC_BLOCK / TPC_WAVE];
    const int ch = blockIdx.x, s0 = ch * TPC_SCAN_CHUNK;
    int vc = 0, vh = 0;
    for (int s = s0 + threadIdx.x; s < s0 + TPC_SCAN_CHUNK && s < NR; s += TPC_BLOCK) {
        vc += ws.segcnt[s];
        vh += ws.seghits[s];
    }
    int tc, th;
    block_exclusive_scan(vc, sh, &tc);
    block_exclusive_scan(vh, sh, &th);
    if (threadIdx.x == 0) { ws.chunk_c[ch] = tc; ws.chunk_h[ch] = th; }
}

// ... and, after ca_scan over the chunk sums, the segment prefixes within
// each chunk (thread t owns segments s0 + 4t .. 4t + 3).
__global__ void __launch_bounds__(TPC_BLOCK)
ca_chunk_prefix(int32_t NR, CaWs ws) {
    __shared__ int sh[TPC_BLOCK / TPC_WAVE];
    constexpr int PER = TPC_SCAN_CHUNK / TPC_BLOCK;
    const int ch = blockIdx.x, s0 = ch * TPC_SCAN_CHUNK + threadIdx.x * PER;
    int c[PER], h[PER], vc = 0, vh = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const bool in = s0 + j < NR;
        c[j] = in ? ws.segcnt[s0 + j] : 0;
        h[j] = in ? ws.seghits[s0 + j] : 0;
        vc += c[j];
        vh += h[j];
    }
    int tc, th;
    int pc = ws.chunk_c[ch] + block_exclusive_scan(vc, sh, &tc);
    int ph = ws.chunk_h[ch] + block_exclusive_scan(vh, sh, &th);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (s0 + j < NR) { ws.segbs[s0 + j] = pc; ws.segbh[s0 + j] = ph; }
        pc += c[j];
        ph += h[j];
    }
}

// SUM: every workgroup sums the counts of the segments before its own itself
// (they are in no scan), and the one with the last segment writes the totals.
template <int PARTS, bool SUM>
__global__ void __launch_bounds__(TPC_BLOCK)
ca_place(int32_t N, int32_t NR, const int32_t *off, const int32_t *up, const float *y, const float *z,
         int32_t n_sectors, int32_t n_rows, int32_t cap_seeds, int32_t cap_hits, tpc_seeds sd, int32_t *dev_status,
         CaWs ws) {
    constexpr int W = TPC_BLOCK / TPC_WAVE, SEGS = W / PARTS;
    __shared__ int list[W][2 * TPC_WAVE];
    __shared__ int2 count[W];
    const int wid = threadIdx.x / TPC_WAVE, part = wid % PARTS, lane = threadIdx.x % TPC_WAVE;
    const int s0 = xcd_item(blockIdx.x, gridDim.x) * SEGS, seg = s0 + wid / PARTS;
    int first_c = 0, first_h = 0;
    if constexpr (SUM) {
        static_assert(PARTS == 1 && SEGS % 4 == 0, "four counts at a time");
        const int4 *c4 = reinterpret_cast<const int4 *>(ws.segcnt), *h4 = reinterpret_cast<const int4 *>(ws.seghits);
        int c = 0, h = 0;
        for (int q = threadIdx.x; q < s0 / 4; q += TPC_BLOCK) {
            const int4 a = c4[q], b = h4[q];
            c += a.x + a.y + a.z + a.w;
            h += b.x + b.y + b.z + b.w;
        }
        c = __builtin_amdgcn_readlane(lane_scan(c), TPC_WAVE - 1);
        h = __builtin_amdgcn_readlane(lane_scan(h), TPC_WAVE - 1);
        if (lane == 0) count[wid] = make_int2(c, h);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) {
            first_c += count[w].x;
            first_h += count[w].y;
        }
        for (int s = s0; s < seg && s < NR; ++s) {
            first_c += ws.segcnt[s];
            first_h += ws.seghits[s];
        }
        if (seg == NR - 1 && lane == 0)
            put_totals(first_c + ws.segcnt[seg], first_h + ws.seghits[seg], sd.n_seeds, sd.n_hits, cap_seeds, cap_hits,
                       sd.offsets, dev_status);
    } else if (seg < NR) {
        first_c = ws.segbs[seg];
        first_h = ws.segbh[seg];
    }
    if constexpr (PARTS > 1) {                        // (then the whole workgroup has one segment)
        const int2 c = ca_place_count(seg, part, PARTS, off, ws, list[wid]);
        if (lane == 0) count[wid] = c;
        __syncthreads();
        for (int p = 0; p < part; ++p) {
            first_c += count[p].x;
            first_h += count[p].y;
        }
    }
    if (seg < NR)
        ca_place_part(seg, part, PARTS, first_c, first_h, N, off, up, y, z, n_sectors, n_rows, cap_seeds, cap_hits,
                      sd, ws, list[wid]);
}

__global__ void __launch_bounds__(TPC_BLOCK)
ca_members(int32_t N, const float *y, const float *z, int32_t cap_hits, tpc_seeds sd, CaWs ws) {
    ca_members_flat<4>((int64_t)xcd_item(blockIdx.x, gridDim.x) * 4 * TPC_BLOCK, N, y, z, cap_hits, sd, ws);
}

}  // namespace


hipError_t launch_ca_seed(const tpc_context *ctx, const tpc_frames *fr, const int32_t *up,
                          const int32_t *dn, const tpc_seeds *sd, int32_t *dev_status,
                          const CaWs &ws, hipStream_t st) {
    const tpc_config &c = ctx->cfg;
    const int NR = fr->n_frames * c.n_sectors * c.n_rows;
    const int32_t *off = fr->row_offsets;
    const int32_t N = fr->n_clusters;
    const int NB = fr->n_frames * c.n_sectors * ca_blocks_per_sector(c.n_rows);
    hipLaunchKernelGGL(ca_block, dim3(NB), dim3(1024), 0, st, N, c.n_rows, off, up, dn, ws);
    // no block is larger than the whole input; on frames of small rows one
    // workgroup per CU (its LDS admits one) looks for large blocks
    const bool sparse = (int64_t)N < (int64_t)TPC_SPARSE_ROW * fr->n_frames * c.n_sectors * c.n_rows;
    if (N > TPC_CA_CAP)
        hipLaunchKernelGGL(ca_block_sweep, dim3(sparse && NB > 256 ? 256 : NB), dim3(1024), 0, st, NB, N, c.n_rows,
                           off, up, dn, ws);
    const int flat = N > 0 ? (int)(((int64_t)N + TPC_CA_FLAT - 1) / TPC_CA_FLAT) : 1;
    static_assert(TPC_CA_FLAT == 4 * TPC_BLOCK, "ca_members takes four clusters per thread");
    constexpr int WB = TPC_BLOCK / TPC_WAVE;
    hipLaunchKernelGGL(ca_tops, dim3(flat), dim3(TPC_BLOCK), 0, st, N, NR, up, dn, c.min_hits, c.n_rows, ws);
    if (sparse)
        hipLaunchKernelGGL(ca_firsts<1>, dim3((NR + WB - 1) / WB), dim3(TPC_BLOCK), 0, st, N, NR, off, up, dn,
                           c.min_hits, ws);
    else
        hipLaunchKernelGGL(ca_firsts<WB>, dim3(NR), dim3(TPC_BLOCK), 0, st, N, NR, off, up, dn, c.min_hits, ws);
    // few segments: no scan of their own (a launch, 7 us, for the 5472 of an
    // event; their sums cost the placement about 3)
    const bool sum = sparse && NR <= TPC_SCAN_SUM;
    if (!sum && NR <= TPC_SCAN_DIRECT) {
        hipLaunchKernelGGL(ca_scan, dim3(1), dim3(1024), 0, st, NR, ws.segcnt, ws.seghits, ws.segbs,
                           ws.segbh, sd->n_seeds, sd->n_hits, sd->cap_seeds, sd->cap_hits, sd->offsets,
                           dev_status);
    } else if (!sum) {
        const int nch = (NR + TPC_SCAN_CHUNK - 1) / TPC_SCAN_CHUNK;
        hipLaunchKernelGGL(ca_chunk_sums, dim3(nch), dim3(TPC_BLOCK), 0, st, NR, ws);
        hipLaunchKernelGGL(ca_scan, dim3(1), dim3(1024), 0, st, nch, ws.chunk_c, ws.chunk_h, ws.chunk_c,
                           ws.chunk_h, sd->n_seeds, sd->n_hits, sd->cap_seeds, sd->cap_hits, sd->offsets,
                           dev_status);
        hipLaunchKernelGGL(ca_chunk_prefix, dim3(nch), dim3(TPC_BLOCK), 0, st, NR, ws);
    }
    auto place = [&](auto kernel, int blocks) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(TPC_BLOCK), 0, st, N, NR, off, up, fr->y, fr->z, c.n_sectors,
                           c.n_rows, sd->cap_seeds, sd->cap_hits, *sd, dev_status, ws);
    };
    if (sum) place(ca_place<1, true>, (NR + WB - 1) / WB);
    else if (sparse) place(ca_place<1, false>, (NR + WB - 1) / WB);
    else place(ca_place<WB, false>, NR);
    hipLaunchKernelGGL(ca_members, dim3(flat), dim3(TPC_BLOCK), 0, st, N, fr->y, fr->z, sd->cap_hits, *sd, ws);
    return hipGetLastError();
}

size_t ca_ws_layout(void *ws, int64_t N, int64_t NR, CaWs *out) {
    WsCarver w(ws);
    CaWs l;
    l.claim = w.take<unsigned long long>(N);
    l.pack = w.take<unsigned long long>(N);
    l.cc = w.take<int2>(N);
    l.cend = w.take<int32_t>(N);
    l.mrec = w.take<int2>(N);
    l.fbot = w.take<int32_t>(N);
    l.flen = w.take<int32_t>(N);
    l.segcnt = w.take<int32_t>(NR);
    l.seghits = w.take<int32_t>(NR);
    l.segbs = w.take<int32_t>(NR);
    l.segbh = w.take<int32_t>(NR);
    const int64_t nch = (NR + TPC_SCAN_CHUNK - 1) / TPC_SCAN_CHUNK;
    l.chunk_c = w.take<int32_t>(nch > 0 ? nch : 1);
    l.chunk_h = w.take<int32_t>(nch > 0 ? nch : 1);
    if (out) *out = l;
    return (w.off + 255) & ~size_t(255);
}
