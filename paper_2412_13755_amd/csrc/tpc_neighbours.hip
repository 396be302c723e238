// Neighbour search stage kernels: one workgroup per (frame, sector, row)
// segment; the per-segment work is in tpc_nb_device.hpp.  nb_bin only works
// on dense rows and their neighbouring rows (z-sorted copies), and
// nb_query_dense only on dense rows.
#include "tpc_nb_device.hpp"

// Dense h-rows of frames of dense rows are searched in TPC_NB_PARTS parts
// of about equal size, each by its own workgroup (two measured faster than
// whole rows, three or four parts).
#ifndef TPC_NB_PARTS
#define TPC_NB_PARTS 2
#endif

namespace {

__global__ void __launch_bounds__(TPC_BLOCK)
nb_bin(const int32_t *__restrict__ off, int32_t NR, int32_t n_rows, const float *__restrict__ y,
       const float *__restrict__ z, float win_y, float win_z, SegGrid *grid, int32_t *cstart, float *sy,
       float *sz, int32_t *sid) {
    __shared__ tpc_nb::BinLdsPerm L;
    // (taking the largest rows first, as the dense query does, made the
    // binning slower)
    tpc_nb::nb_bin_seg(xcd_item(blockIdx.x, NR), n_rows, off, y, z, win_y, win_z, grid, cstart, sy, sz, sid, L);
}

// Blocks from nb on, GROUP segments each: the segments whose neighbouring rows fit the mixed LDS
// form (24 KB per workgroup, six workgroups per CU), the very small ones by a
// wavefront, and the first and last rows.  Blocks below nb: the sorted copies that dense rows need, where the
// frames have few or none of them (a launch less than nb_bin's own; they
// come first because they run longest if there are any).
template <int GROUP>
__global__ void __launch_bounds__(TPC_BLOCK, 6)
nb_query_small(const int32_t *__restrict__ off, int32_t NR, int32_t nb, int32_t n_rows, const float *__restrict__ y,
               const float *__restrict__ z, float win_y, float win_z, float cut_y, float cut_z, SegGrid *grid,
               int32_t *cstart, float *sy, float *sz, int32_t *sid, int32_t *up, int32_t *dn) {
    __shared__ union {
        tpc_nb::MixLds mix;
        struct {
            tpc_nb::BinLds lds;
            int list[TPC_BLOCK], count;
        } bin;
    } U;
    if ((int)blockIdx.x < nb) {
        for (int from = 0; blockIdx.x + (int64_t)nb * from < NR; from += TPC_BLOCK) {
            const int m = tpc_nb::pick_items(from, blockIdx.x, nb, NR, [&](int s) { return tpc_nb::nb_bin_needed(off, s, n_rows); },
                                     U.bin.list, &U.bin.count);
            for (int k = 0; k < m; ++k)
                tpc_nb::nb_bin_seg(U.bin.list[k], n_rows, off, y, z, win_y, win_z, grid, cstart, sy, sz, sid,
                                   U.bin.lds);
        }
        return;
    }
    // One segment each: rows in ascending order over all sectors, so that the
    // inner rows, which take longest, start first and do not trail.
    const int b = blockIdx.x - nb, n_fs = NR / n_rows;
    const int s0 = GROUP > 1 ? GROUP * xcd_item(b, (NR + GROUP - 1) / GROUP) : b % n_fs * n_rows + b / n_fs;
    const int wid = threadIdx.x / TPC_WAVE;
    static_assert(GROUP <= TPC_BLOCK / TPC_WAVE, "a wavefront per segment");
    auto tiny = [&](int seg) {
        return tpc_nb::inner_row(seg, n_rows) && off[seg] < off[seg + 1] && tpc_nb::tiny_pair(off, seg);
    };
    if (wid < GROUP && s0 + wid < NR && tiny(s0 + wid))
        tpc_nb::tiny_query_wave(s0 + wid, off, y, z, win_y, win_z, cut_y, cut_z, up, dn);
#pragma unroll 1
    for (int seg = s0; seg < s0 + GROUP && seg < NR; ++seg) {
        if (off[seg] == off[seg + 1] || tpc_nb::edge_row(seg, off, n_rows, up, dn) || tpc_nb::tiny_pair(off, seg) ||
            !tpc_nb::small_pair(off, seg))
            continue;
        if (GROUP > 1) __syncthreads();              // LDS reuse
        tpc_nb::mix_query_seg(seg, off, y, z, win_y, win_z, cut_y, cut_z, up, dn, U.mix);
    }
}

// The segments that nb_query_small leaves, where the frames have few or none:
// rows of the large LDS form and dense rows.  (Both searches in one kernel
// need a few registers more than the 128 of four workgroups per CU.)
__global__ void __launch_bounds__(TPC_BLOCK, 3)
nb_query_rest(const int32_t *__restrict__ off, int32_t NR, int32_t n_rows, const float *__restrict__ y,
              const float *__restrict__ z, float win_y, float win_z, float cut_y, float cut_z, const SegGrid *grid,
              const int32_t *cstart, const float *sy, const float *sz, const int32_t *sid, int32_t *up,
              int32_t *dn) {
    __shared__ union {
        tpc_nb::MixLdsL mix;
        tpc_nb::DenseLds dense;
    } U;
    __shared__ int list[TPC_BLOCK], count;
    for (int from = 0; blockIdx.x + (int64_t)gridDim.x * from < NR; from += TPC_BLOCK) {
        const int m = tpc_nb::pick_items(from, blockIdx.x, gridDim.x, NR, [&](int s) { return tpc_nb::rest_hrow(off, s, n_rows); },
                                 list, &count);
        for (int k = 0; k < m; ++k) {
            const int seg = list[k];
            __syncthreads();             // LDS reuse
            if (tpc_nb::dense_hrow(off, seg, n_rows))
                tpc_nb::nb_dense_seg(seg, off, n_rows, win_y, win_z, cut_y, cut_z, grid, cstart, sy, sz, sid, up, dn,
                                     U.dense);
            else
                tpc_nb::mix_query_seg(seg, off, y, z, win_y, win_z, cut_y, cut_z, up, dn, U.mix);
        }
    }
}

// Rows whose neighbour rows fit the large mixed form only.
__global__ void __launch_bounds__(TPC_BLOCK)
nb_query(const int32_t *__restrict__ off, int32_t n_rows, const float *__restrict__ y,
         const float *__restrict__ z, float win_y, float win_z, float cut_y, float cut_z, int32_t *up, int32_t *dn) {
    __shared__ tpc_nb::MixLdsL L;
    const int seg = xcd_item(blockIdx.x, gridDim.x);
    if (tpc_nb::rest_hrow(off, seg, n_rows) && !tpc_nb::dense_hrow(off, seg, n_rows))
        tpc_nb::mix_query_seg(seg, off, y, z, win_y, win_z, cut_y, cut_z, up, dn, L);
}

// The order in which the dense query takes its work items, item
// TPC_NB_PARTS s + q being part q of dense h-row s: by descending size in
// steps of 128 clusters (the largest start first, so the last workgroups to
// finish are small ones), then the items with nothing to do.
__global__ void __launch_bounds__(TPC_BLOCK)
nb_dense_order(const int32_t *__restrict__ off, int32_t NR, int32_t n_rows, int32_t *__restrict__ order) {
    __shared__ int start[TPC_ORDER_BINS + 1];
    __shared__ int sh[TPC_BLOCK / TPC_WAVE];
    order_desc(TPC_NB_PARTS * NR, [&](int i) {
        const int s = i / TPC_NB_PARTS, q = i % TPC_NB_PARTS;
        if (!tpc_nb::dense_hrow(off, s, n_rows)) return 0;
        const int n = tpc_nb::seg_size(off, s);
        const int ps = tpc_nb::dense_split(n, q + 1, TPC_NB_PARTS) - tpc_nb::dense_split(n, q, TPC_NB_PARTS);
        const int b = ps >> 7;
        return ps == 0 ? 0 : 1 + (b < TPC_ORDER_BINS - 1 ? b : TPC_ORDER_BINS - 1);
    }, order, start, sh);
}

// Dense rows: slabs of the z-sorted rows, searched in LDS.  Four wavefronts
// per SIMD (the LDS allows four workgroups per CU): at most 128 VGPRs.
// order: the work items of nb_dense_order (row parts, largest first).
__global__ void __launch_bounds__(TPC_BLOCK, 4)
nb_query_dense(const int32_t *__restrict__ off, int32_t n_rows, float win_y, float win_z, float cut_y, float cut_z,
               const SegGrid *grid, const int32_t *cstart, const float *sy, const float *sz, const int32_t *sid,
               const int32_t *__restrict__ order, int32_t *up, int32_t *dn) {
    __shared__ tpc_nb::DenseLds L;
    const int item = order[blockIdx.x];
    tpc_nb::nb_dense_seg(item / TPC_NB_PARTS, off, n_rows, win_y, win_z, cut_y, cut_z, grid, cstart, sy, sz, sid, up,
                         dn, L, item % TPC_NB_PARTS, TPC_NB_PARTS);
}

}  // namespace


#define TPC_NB_GROUP_MIN 16384
hipError_t launch_neighbours(const tpc_context *ctx, const tpc_frames *fr, int32_t *up,
                             int32_t *dn, const NbWs &ws, hipStream_t st) {
    const int NR = fr->n_frames * ctx->cfg.n_sectors * ctx->cfg.n_rows;
    const tpc_config &c = ctx->cfg;
    // The binning, the large form and the dense query only work on segments
    // with large rows next to them.  Frames whose rows are small on average
    // have few such segments or none: two launches then, in which at most
    // TPC_SPARSE_GRID workgroups look for them.  Otherwise one workgroup per
    // segment, so that heavy segments run side by side; the dense query takes
    // parts of the dense h-rows, the largest first, so that the tail of a
    // grid of workgroups of very different lengths is made of short ones.
    // (Event of 10^4 tracks: 12 us in two more launches, 64 uneven frames:
    // 0.7 ms of workgroups walking over segments with nothing to do.)
    const bool sparse = (int64_t)fr->n_clusters < (int64_t)TPC_SPARSE_ROW * NR;
    const int gs = NR < TPC_SPARSE_GRID ? NR : TPC_SPARSE_GRID;
    const int nb = sparse ? (NR < TPC_SPARSE_GRID / 2 ? NR : TPC_SPARSE_GRID / 2) : 0;
    if (!sparse) {
        hipLaunchKernelGGL(nb_dense_order, dim3(1), dim3(TPC_BLOCK), 0, st, fr->row_offsets, NR, c.n_rows,
                           ws.order);
        hipLaunchKernelGGL(nb_bin, dim3(NR), dim3(TPC_BLOCK), 0, st, fr->row_offsets, NR, c.n_rows, fr->y,
                           fr->z, c.win_y, c.win_z, ws.grid, ws.cstart, ws.sy, ws.sz, ws.sid);
    }
    // Many segments (at ten times as many as run at a time, waiting for the
    // workgroup with the longest four does not matter): four per workgroup,
    // so that four very small ones run side by side and a quarter of the
    // workgroups are launched.
    auto small = [&](auto kernel, int group) {
        hipLaunchKernelGGL(kernel, dim3(nb + (NR + group - 1) / group), dim3(TPC_BLOCK), 0, st, fr->row_offsets, NR,
                           nb, c.n_rows, fr->y, fr->z, c.win_y, c.win_z, c.cut_y, c.cut_z, ws.grid, ws.cstart, ws.sy,
                           ws.sz, ws.sid, up, dn);
    };
    if (NR >= TPC_NB_GROUP_MIN)
        small(nb_query_small<4>, 4);
    else
        small(nb_query_small<1>, 1);
    if (sparse) {
        hipLaunchKernelGGL(nb_query_rest, dim3(gs), dim3(TPC_BLOCK), 0, st, fr->row_offsets, NR, c.n_rows, fr->y,
                           fr->z, c.win_y, c.win_z, c.cut_y, c.cut_z, ws.grid, ws.cstart, ws.sy, ws.sz, ws.sid, up,
                           dn);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(nb_query, dim3(NR), dim3(TPC_BLOCK), 0, st, fr->row_offsets, c.n_rows, fr->y,
                       fr->z, c.win_y, c.win_z, c.cut_y, c.cut_z, up, dn);
    hipLaunchKernelGGL(nb_query_dense, dim3(TPC_NB_PARTS * NR), dim3(TPC_BLOCK), 0, st, fr->row_offsets, c.n_rows,
                       c.win_y, c.win_z, c.cut_y, c.cut_z, ws.grid, ws.cstart, ws.sy, ws.sz, ws.sid, ws.order, up,
                       dn);
    return hipGetLastError();
}

size_t nb_ws_layout(void *ws, int64_t N, int64_t NR, NbWs *out) {
    WsCarver w(ws);
    NbWs l;
    l.grid = w.take<SegGrid>(NR);
    l.cstart = w.take<int32_t>(N + NR + 1);
    l.sy = w.take<float>(N);
    l.sz = w.take<float>(N);
    l.sid = w.take<int32_t>(N);
    l.order = w.take<int32_t>(TPC_NB_PARTS * NR);
    if (out) *out = l;
    return (w.off + 255) & ~size_t(255);
}
