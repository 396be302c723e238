// Per-seed access shared by the fit and its adjoint.
#pragma once

#include "tpc_fit_math.hpp"
#include "tpc_internal.hpp"

#define TPC_CKPT_WORDS 20      // doubles per checkpoint: p[5], covariance lower triangle[15]

struct FitArgs {
    const int32_t *offsets, *hits, *sector, *first_row, *n_seeds;
    int32_t cap_seeds, cap_hits;
    const float *row_x, *map;
    const float2 *hyz;     // (y, z) of every seed hit in seed-hit order (set by every launch of a fit)
    int32_t n_rows, n_sectors;
    float kbz, max_sin;
    double vy, vz, var_s, var_t, var_w;
    double *ckpt;
    int32_t ckpt_rows;
    tpc_tracks out;
    const int32_t *order;      // optional: fit seeds order[0 .. *n_order) instead of 0 .. T
    const int32_t *n_order;
};

struct SeedView {
    int32_t o0, n, row0, sec;
    bool sane;
    const int32_t *hh;     // hit ids of the seed
    const float *mp;       // map rows of the seed's sector, or null
};

// A seed from tpc_ca_seed always passes these checks; others are flagged
// instead of being read out of bounds.
__host__ __device__ inline SeedView seed_view(const FitArgs &A, int i) {
    SeedView v;
    v.o0 = A.offsets[i];
    v.n = A.offsets[i + 1] - v.o0;
    v.row0 = A.first_row[i];
    v.sec = A.sector[i];
    v.sane = v.n >= 3 && v.row0 >= 0 && v.row0 + v.n <= A.n_rows && v.sec >= 0 &&
             v.sec < A.n_sectors && v.o0 >= 0 && v.o0 <= A.cap_hits - v.n;
    v.hh = A.hits + v.o0;
    v.mp = (A.map && v.sane) ? A.map + (size_t)v.sec * A.n_rows * 2 : nullptr;
    return v;
}

// Corrected measurement of hit k in double precision (MAP: with a map).
template <bool MAP = true>
__host__ __device__ inline void hit_fix(const SeedView &v, int k, float2 raw, double &my, double &mz) {
    my = (double)raw.x;
    mz = (double)raw.y;
    if (MAP && v.mp) {
        my -= (double)v.mp[(v.row0 + k) * 2];
        mz -= (double)v.mp[(v.row0 + k) * 2 + 1];
    }
}

__host__ __device__ inline void hit_meas(const FitArgs &A, const SeedView &v, int k, double &my, double &mz) {
    hit_fix(v, k, A.hyz[v.o0 + k], my, mz);
}

__host__ __device__ inline bool start_state(const FitArgs &A, const SeedView &v, const float *xs, double p[5]) {
    const int ka = v.n - 1, kb = (v.n - 1) / 2;
    double ya, za, yb, zb, yc, zc;
    hit_meas(A, v, ka, ya, za);
    hit_meas(A, v, kb, yb, zb);
    hit_meas(A, v, 0, yc, zc);
    (void)zb;
    return helix_start<double>(xs[v.row0 + ka], ya, za, xs[v.row0 + kb], yb, xs[v.row0], yc, zc,
                               A.kbz, A.max_sin, p);
}

// Checkpoint slots: track i with hit offset o0 owns slots o0/K + i .. + ceil(n/K);
// slots of consecutive tracks never overlap.
__host__ __device__ inline int64_t ckpt_slot(int32_t o0, int32_t i, int32_t K) {
    return (int64_t)(o0 / K) + i;
}

__host__ __device__ inline void write_ckpt(double *ck, const double p[5], const SymT<double> &C) {
#pragma unroll
    for (int q = 0; q < 5; ++q) ck[q] = p[q];
    ck[5] = C.c00; ck[6] = C.c10; ck[7] = C.c11; ck[8] = C.c20; ck[9] = C.c21;
    ck[10] = C.c22; ck[11] = C.c30; ck[12] = C.c31; ck[13] = C.c32; ck[14] = C.c33;
    ck[15] = C.c40; ck[16] = C.c41; ck[17] = C.c42; ck[18] = C.c43; ck[19] = C.c44;
}

__host__ __device__ inline void read_ckpt(const double *ck, double p[5], SymT<double> &C) {
#pragma unroll
    for (int q = 0; q < 5; ++q) p[q] = ck[q];
    C.c00 = ck[5]; C.c10 = ck[6]; C.c11 = ck[7]; C.c20 = ck[8]; C.c21 = ck[9];
    C.c22 = ck[10]; C.c30 = ck[11]; C.c31 = ck[12]; C.c32 = ck[13]; C.c33 = ck[14];
    C.c40 = ck[15]; C.c41 = ck[16]; C.c42 = ck[17]; C.c43 = ck[18]; C.c44 = ck[19];
}

// Forward fit of seed i (one thread's work); xs = row table, readable one
// entry below its start.  CKPT: filter states to A.ckpt.
//
// Bound by instructions: a wavefront alone on its SIMD issues one about
// every five clocks whatever it is, so the loop carries no test that a
// template argument or the step before can decide, and ends by one
// condition (what the last step left is sorted out after it).
template <bool MAP, bool CKPT>
__host__ __device__ inline void fit_one(const FitArgs &A, int i, const float *xs) {
    SeedView sv = seed_view(A, i);
    double p[5] = {0, 0, 0, 0, 0};
    SymT<double> C = {};
    double chi2 = 0.0;
    int status = TPC_FIT_OK;
    float xcur = sv.sane ? xs[sv.row0 + sv.n - 1] : 0.0f;
    if (!sv.sane || !start_state(A, sv, xs, p)) status = TPC_FIT_INIT_FAIL;
    C.c00 = A.vy;
    C.c11 = A.vz;
    C.c22 = A.var_s;
    C.c33 = A.var_t;
    C.c44 = A.var_w;
    if (status == TPC_FIT_OK) {
        double *ck = CKPT ? A.ckpt + (size_t)ckpt_slot(sv.o0, i, A.ckpt_rows) * TPC_CKPT_WORDS : nullptr;
        int left = A.ckpt_rows;                       // updates until the next checkpoint
        if (CKPT) write_ckpt(ck, p, C);
        int k = sv.n - 2;
        // Each hit is read one step ahead, into the register its predecessor
        // has just been consumed from (no copy at the loop edge, so the load
        // is waited for only at its use a whole step later).
        const float2 *hp = A.hyz + sv.o0 + k;
        float2 raw = *hp;
        const float *xp = xs + sv.row0 + k;
        float xk = *xp, xl = xcur;                    // planes of hit k and of the hit before it
        // the covariance half of each update is applied at the next step,
        // beside its helix step (before the first update G leaves the start
        // covariance as it is)
        Gain<double> G = Gain<double>::none();
        bool stepped, good;
        do {
            double my, mz;
            hit_fix<MAP>(sv, k, raw, my, mz);
            hp -= k > 0;
            raw = *hp;
            kalman_cov(C, G, A.vy, A.vz);
            StepJac J;
            stepped = helix_step(p, xk - xl, A.kbz, A.max_sin, J);
            xcur = xl;
            xl = xk;
            xk = *--xp;                               // below the seed after its last hit, then unused
            sym_transport<double, false>(C, J);
            const double dchi = kalman_gain<double>(p, C, my, mz, A.vy, A.vz, G);
            chi2 += dchi;
            // evaluated to the end whatever happens: a failed track's final
            // state is not used
            const double chk = chi2 + p[0] + p[1] + p[2] + p[3] + p[4];
            good = (int)stepped & (int)(dchi >= 0.0) & (int)(chk - chk == 0.0);   // non-finite state too
            --k;
            // state after j updates opens segment j / ckpt_rows of the adjoint
            if (CKPT && --left == 0 && good && k >= 0) {
                left = A.ckpt_rows;
                ck += TPC_CKPT_WORDS;
                SymT<double> Cj = C;
                kalman_cov(Cj, G, A.vy, A.vz);
                write_ckpt(ck, p, Cj);
            }
        } while ((int)good & (int)(k >= 0));
        kalman_cov(C, G, A.vy, A.vz);                 // the last update's covariance half
        if (good) xcur = xl;
        else status = stepped ? TPC_FIT_NUM_FAIL : TPC_FIT_SIN_FAIL;
    }
    A.out.x[i] = xcur;
    float *po = A.out.par + (size_t)i * 5;
    for (int q = 0; q < 5; ++q) po[q] = (float)p[q];
    float *co = A.out.cov + (size_t)i * 15;
    const double cc[15] = {C.c00, C.c10, C.c11, C.c20, C.c21, C.c22, C.c30, C.c31,
                           C.c32, C.c33, C.c40, C.c41, C.c42, C.c43, C.c44};
    for (int q = 0; q < 15; ++q) co[q] = (float)cc[q];
    A.out.chi2[i] = (float)chi2;
    A.out.ndf[i] = 2 * sv.n - 5;
    A.out.status[i] = status;
}

// Tape of filter states before each step of one segment; word q of step s at
// tp[(s * TPC_CKPT_WORDS + q) * stride].
__device__ inline void tape_put(double *tp, int stride, int step, const double p[5],
                                         const SymT<double> &C) {
    double *b = tp + (size_t)step * TPC_CKPT_WORDS * stride;
    const double v[TPC_CKPT_WORDS] = {p[0], p[1], p[2], p[3], p[4], C.c00, C.c10, C.c11, C.c20, C.c21,
                                      C.c22, C.c30, C.c31, C.c32, C.c33, C.c40, C.c41, C.c42, C.c43, C.c44};
#pragma unroll
    for (int q = 0; q < TPC_CKPT_WORDS; ++q) b[q * stride] = v[q];
}

__device__ inline void tape_get(const double *tp, int stride, int step, double p[5],
                                         SymT<double> &C) {
    const double *b = tp + (size_t)step * TPC_CKPT_WORDS * stride;
    double v[TPC_CKPT_WORDS];
#pragma unroll
    for (int q = 0; q < TPC_CKPT_WORDS; ++q) v[q] = b[q * stride];
    p[0] = v[0]; p[1] = v[1]; p[2] = v[2]; p[3] = v[3]; p[4] = v[4];
    C.c00 = v[5]; C.c10 = v[6]; C.c11 = v[7]; C.c20 = v[8]; C.c21 = v[9]; C.c22 = v[10];
    C.c30 = v[11]; C.c31 = v[12]; C.c32 = v[13]; C.c33 = v[14]; C.c40 = v[15]; C.c41 = v[16];
    C.c42 = v[17]; C.c43 = v[18]; C.c44 = v[19];
}

// Steps of a sub-segment of the reverse pass.
#define TPC_ADJ_SUB 4
__host__ __device__ inline int adj_tape_states(int K) { return (K + TPC_ADJ_SUB - 1) / TPC_ADJ_SUB; }

// Reverse pass of seed i (one thread's work): writes dL/d(my, mz) for every
// hit of the seed into g[offsets[i] ..], zeros for a failed fit.
//
// A segment of K steps is run forward from its checkpoint, taping (tp, global
// memory) the state at every TPC_ADJ_SUB-th step only; each sub-segment, from
// the last, is then run forward again with its states in LDS (lt) and
// registers, and its steps reversed.  That is half a forward step more per
// step than with every state taped, and a third of the memory traffic, which
// was what the time went to (2.9 GB for 645 000 seeds; 1035 -> 735 us).
// (Everything is addressed by 32-bit indices from bases in scalar registers:
// the step adjoint needs nearly all of the vector ones.)
__device__ inline void adj_one(const FitArgs &F, const int32_t *status, const double *ckpt, float2 *gbuf, int i,
                               double *tp, int lane, double *lt, int lstride) {
    const int K = F.ckpt_rows;
    int n, row0, o0, m0;                                // hits, first row, hit offset, map entry of the first row
    {
        const SeedView sv = seed_view(F, i);
        if (!sv.sane) return;
        n = sv.n;
        row0 = sv.row0;
        o0 = sv.o0;
        m0 = sv.sec * F.n_rows + row0;
    }
    if (status[i] != TPC_FIT_OK) {
        for (int k = 0; k < n; ++k) gbuf[o0 + k] = make_float2(0.f, 0.f);
        return;
    }
    const int nsteps = n - 1;
    const int64_t slot = ckpt_slot(o0, i, K);
    double pbar[5] = {0, 0, 0, 0, 0};
    SymT<double> Cbar = {};
    auto meas = [&](int k, double &my, double &mz) {
        const float2 raw = F.hyz[o0 + k];
        my = (double)raw.x;
        mz = (double)raw.y;
        if (F.map) {
            const float *f = F.map + 2 * (size_t)(m0 + k);      // (4-byte aligned)
            my -= (double)f[0];
            mz -= (double)f[1];
        }
    };
    auto plane = [&](int k) { return F.row_x[row0 + k]; };
    for (int c = (nsteps + K - 1) / K - 1; c >= 0; --c) {
        double p[5];
        SymT<double> C;
        const int j0 = c * K;
        const int len = K < nsteps - j0 ? K : nsteps - j0;
        const int last = (len - 1) / TPC_ADJ_SUB;           // the last sub-segment
        auto forward = [&](int q) {                         // step q propagates from hit k + 1 to hit k
            const int k = n - 1 - (j0 + q);
            double my, mz;
            meas(k, my, mz);
            StepJac J;
            helix_step<double, float, 5>(p, plane(k) - plane(k + 1), F.kbz, 2.0f, J);
            sym_transport<double, false>(C, J);
            kalman_update<double>(p, C, my, mz, F.vy, F.vz);
        };
        auto open = [&](int u) {                            // the state that opens sub-segment u
            if (u > 0) tape_get(tp + lane, TPC_WAVE, u - 1, p, C);
            else read_ckpt(ckpt + (slot + c) * TPC_CKPT_WORDS, p, C);
        };
        open(0);
#pragma unroll 1
        for (int q = 1; q <= last * TPC_ADJ_SUB; ++q) {
            forward(q);
            if (q % TPC_ADJ_SUB == 0) tape_put(tp + lane, TPC_WAVE, q / TPC_ADJ_SUB - 1, p, C);
        }
        for (int u = last; u >= 0; --u) {
            const int s0 = u * TPC_ADJ_SUB;
            const int s1 = s0 + TPC_ADJ_SUB < len ? s0 + TPC_ADJ_SUB : len;
            if (u < last) open(u);
#pragma unroll 1
            for (int q = s0 + 1; q < s1; ++q) {
                forward(q);
                if (q < s1 - 1) tape_put(lt, lstride, q - s0 - 1, p, C);
            }
#pragma unroll 1
            for (int q = s1; q > s0; --q) {                 // (p, C): the state before step q
                if (q < s1) {
                    if (q > s0 + 1) tape_get(lt, lstride, q - s0 - 2, p, C);
                    else open(u);
                }
                const int k = n - 1 - (j0 + q);
                double my, mz;
                meas(k, my, mz);
                double mby, mbz;
                step_adjoint<double>(p, C, plane(k) - plane(k + 1), F.kbz, my, mz, F.vy, F.vz, 1.0, pbar, Cbar, mby,
                                     mbz);
                gbuf[o0 + k] = make_float2((float)mby, (float)mbz);
            }
        }
    }
    // three-point start: hits A = n-1, B = (n-1)/2, C = 0
    const int ka = n - 1, kb = (n - 1) / 2;
    double ya, za, yb, zb, yc, zc;
    meas(ka, ya, za);
    meas(kb, yb, zb);
    meas(0, yc, zc);
    (void)zb;
    double bya, bza, byb, byc, bzc;
    start_adjoint<double>(plane(ka), ya, za, plane(kb), yb, plane(0), yc, zc, F.kbz, pbar, bya, bza, byb, byc, bzc);
    float2 *g = gbuf + o0;
    g[ka] = make_float2((float)bya, (float)bza);
    const float2 gb = g[kb];
    g[kb] = make_float2(gb.x + (float)byb, gb.y);
    const float2 gc = g[0];
    g[0] = make_float2(gc.x + (float)byc, gc.y + (float)bzc);
}

FitArgs make_fit_args(const tpc_context *ctx, const tpc_seeds *sd, const float *map);
// The length order of the seeds into ord (workspace); sets A.order.
void launch_fit_order(FitArgs &A, const FitOrderWs &ord, hipStream_t st);
hipError_t launch_fit_args(const FitArgs &A, hipStream_t st, int block = 0, int spt = 0);
