// Kalman fit with material (gfx950): the seed fit with multiple scattering
// in the gas as process noise and rejection of outlying hits; the same
// kernel also fits seeds whose hits skip pad rows, with per-cluster errors.
//
//  fit_ms_tracks  thread per seed, double precision (plane distances and
//                 -c Bz too): three-point start at the outermost hit; for
//                 each inward step, the scattering of the segment about to
//                 be crossed enters the covariance (Highland, from the state
//                 at the plane the step leaves), then the helix step and
//                 transport (with energy loss, the loss of the segment
//                 is given back between the two, a map of q/pT whose
//                 Jacobian and straggling noise enter the covariance);
//                 the hit's predicted-residual chi2 decides
//                 whether it is used (update) or rejected (flagged).  The
//                 next hit's coordinates are loaded a step ahead.
//                 ROWS: the pad row of every hit is looked up in the
//                 cluster layout of the seed's (frame, sector) -- a binary
//                 search for the outermost hit, then a walk down from the
//                 row above for each next one (at most R + n reads of the
//                 row offsets per seed, all within the seed's R + 1, from
//                 LDS where the wavefront's seeds lie in two neighbouring
//                 (frame, sector)s) -- and a seed whose rows do not rise
//                 strictly, or with a hit outside its (frame, sector), is
//                 refused before the fit; the fit reads the rows found from
//                 a strip in LDS.
//                 ERRS: hit h is measured with variances err[h]^2.
//  smooth_tracks  thread per seed, after the fit over rows: the state at
//                 every hit's plane from all hits.  The reference starts
//                 at the outermost plane from the fit's final state (FP64,
//                 from the fit kernel) -- one helix step, or plane by plane
//                 with the energy loss taken away -- and runs inwards by the
//                 fit's own step; along it a Kalman filter of the deviation
//                 runs inwards (Jacobians, scattering and straggling noise
//                 taken on the reference, diffuse start, the hits the fit
//                 used; rows as the fit stored them), storing per hit the
//                 filtered deviation, its covariance, the reference and the
//                 step that leaves its plane inwards (Jacobian, noise,
//                 energy-loss factors; 38 doubles, 16-byte stores); then the
//                 Rauch-Tung-Striebel pass outwards reads them back (no
//                 step is taken again) and solves with P = F (C + Q) F^T
//                 by its L D L^T.
#include "tpc_fit_common.hpp"
#include "tpc_fit_ms.hpp"

namespace {

struct MsArgs {
    FitArgs F;
    double kbz;            // -c Bz in double precision
    double inv_x0, mass2, cut;
    bool scatter;          // x0 finite
    bool eloss;            // rho > 0
    double mass, rho, kza;         // energy loss: mass, density, K Z/A (K = 0.307075 MeV cm^2/mol),
    double inv_mass, inv_mass2, me_over_m, inv_exc2;   // 1/m, 1/m^2, m_e/m, 1/I^2
    uint8_t *rejected;     // [cap_hits] or null
    // fits over any rows
    const int32_t *row_offsets;   // cluster layout of the frames
    const int32_t *frame;         // frame of each seed
    int32_t n_frames;
    const float2 *err;            // (sigma_y, sigma_z) of every seed hit in seed-hit order, cm
    double *pfin;                 // [cap_seeds][5] final state in FP64, or null
    int16_t *rows_out;            // [cap_hits] row of every seed hit (ROWS), or null
};

// The segment of plane distance dx about to be crossed, seen from the
// state p at the plane the step leaves: path ds = |dx| sqrt(1+t^2) /
// sqrt(1-s^2), momentum P = sqrt(1+t^2)/|w|, energy E.  Inverses are kept
// instead of taken again (1/P^2 = w^2/(1+t^2), 1/beta^2 = E^2/P^2): no
// division is left below.  Meaningless for w = 0, which its users leave out.
struct Segment {
    double ds, t2, it2;        // path; 1 + t^2 and its inverse
    double P, P2, iP2, E, E2, iE;
};

__device__ inline Segment segment(const MsArgs &A, const double p[5], double dx) {
    const double s = p[2], t = p[3], w = p[4];
    Segment g;
    double ist, ics;
    g.t2 = fma(t, t, 1.0);
    const double st = sqrt_pos(g.t2, &ist);
    sqrt_pos(fma(-s, s, 1.0), &ics);
    g.ds = fabs(dx) * st * ics;
    g.it2 = ist * ist;
    g.P = st * recip_pos(fabs(w));
    g.P2 = g.P * g.P;
    g.iP2 = w * w * g.it2;
    g.E2 = g.P2 + A.mass2;
    g.E = sqrt_pos(g.E2, &g.iE);
    return g;
}

// Adds the scattering of the segment to C (Highland: theta0^2 =
// (0.0136 / (beta P))^2 ds/X0 (1 + 0.038 ln(ds/X0))^2; the logarithm, which
// only scales the noise, in single precision).
__device__ inline void add_scattering(const MsArgs &A, const double p[5], const Segment &g, SymT<double> &C) {
    const double s = p[2], t = p[3], w = p[4];
    if (!A.scatter || w == 0.0) return;
    const double xr = g.ds * A.inv_x0;
    const double f = 1.0 + 0.038 * (double)logf((float)xr);
    const double th2 = 0.0136 * 0.0136 * (g.E2 * g.iP2 * g.iP2) * xr * f * f;
    const double tt = th2 * g.t2, tw = th2 * t * w;
    C.c22 += tt * fma(-s, s, 1.0);
    C.c33 += tt * g.t2;
    C.c43 += tw * g.t2;
    C.c44 += tw * t * w;
}

// Energy-loss map of the segment (the particle moves outwards: dir = +1
// gives the mean loss back, a step inwards; -1 takes it away).  Mean loss
// ds rho <dE/dx> with the Bethe formula (unit charge, no density term; its
// logarithm in single precision, which changes the loss by ~1e-7 of
// itself), straggling variance of Bohr's relativistic form;
// P' = sqrt(E'^2 - m^2), w' = w P/P'.  With the loss held fixed, w' depends
// on t and w: j43 = dw'/dt, j44 = dw'/dw; vw is the straggling as variance
// of w at the start.  A segment that would change the momentum by more than
// 1 % is left alone (identity, no noise).  Returns true if the particle
// stops.
__device__ inline bool eloss_map(const MsArgs &A, const double p[5], const Segment &g, double dir, double &wo,
                                 double &j43, double &j44, double &vw) {
    const double t = p[3], w = p[4];
    wo = w;
    j43 = 0.0;
    j44 = 1.0;
    vw = 0.0;
    if (w == 0.0) return false;
    const double me = 0.51099895e-3;
    const double m = A.mass, r = A.me_over_m;
    const double mbg = 2.0 * me * A.inv_mass2 * g.P2;            // 2 m_e (beta gamma)^2
    const double W = mbg * recip_pos(1.0 + 2.0 * A.inv_mass * g.E * r + r * r);
    const double L = (double)logf((float)(mbg * W * A.inv_exc2));
    const double dedx = A.kza * (0.5 * L * g.E2 * g.iP2 - 1.0);
    const double E1 = g.E + dir * (g.ds * A.rho * dedx);
    if (!(E1 > m)) return true;
    double iP1;
    const double P1 = sqrt_pos(fma(E1, E1, -A.mass2), &iP1);
    if (fabs(P1 - g.P) > 0.01 * g.P) return false;
    const double q = g.P * iP1, e = E1 * g.iE;
    wo = w * q;
    j44 = q * q * q * e;
    j43 = wo * t * g.it2 * (1.0 - e * q * q);
    const double varE = A.kza * A.rho * g.ds * me * (1.0 - 0.5 * g.P2 * g.iE * g.iE) * (g.E2 * A.inv_mass2);
    const double dw = w * g.E * g.iP2;
    vw = varE * dw * dw;
    return false;
}

// C <- J C J^T for J the identity but for row 4 = (0, 0, 0, a, b).
__device__ inline void eloss_cov(SymT<double> &C, double a, double b) {
    const double c30 = C.c30, c31 = C.c31, c32 = C.c32, c33 = C.c33, c43 = C.c43, c44 = C.c44;
    C.c40 = a * c30 + b * C.c40;
    C.c41 = a * c31 + b * C.c41;
    C.c42 = a * c32 + b * C.c42;
    C.c43 = a * c33 + b * c43;
    C.c44 = a * a * c33 + 2.0 * a * b * c43 + b * b * c44;
}

// Fits over rows: the pad rows of the seeds of one wavefront, row of hit k of
// lane t at s[64 k + t] (four lanes share a bank: no conflicts), and the
// row starts of two neighbouring (frame, sector)s.  Seeds come ordered by
// (frame, sector), so those of a wavefront rarely need a third.
struct RowLds {
    uint8_t s[TPC_MAX_ROWS * TPC_WAVE];
    int32_t start[2][TPC_MAX_ROWS + 1];
};

// Rows of the hits of a seed into the strip, if every hit lies in the
// (frame, sector) whose R + 1 row starts are ro and the rows rise strictly:
// a binary search for the outermost hit, then a walk down for each next one
// (the first row below the last one's that starts at or before its id).
// The ids are read four hits ahead.
template <class RO>
__device__ inline bool seed_rows(RO ro, int R, const SeedView &sv, uint8_t *strip) {
    const int n = sv.n;
    if (n > R) return false;                      // (more hits than rows cannot rise strictly)
    const int32_t top = sv.hh[n - 1];
    int32_t id[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) id[j] = sv.hh[n - 2 - j > 0 ? n - 2 - j : 0];
    if (top < ro[0] || top >= ro[R]) return false;
    int lo = 0, hi = R - 1;                       // ro[lo] <= top < ro[hi + 1]
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ro[mid] <= top) lo = mid;
        else hi = mid - 1;
    }
    int r = lo;
    strip[(n - 1) * TPC_WAVE] = (uint8_t)r;
    for (int k0 = n - 2; k0 >= 0; k0 -= 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 - j;
            if (k < 0) break;
            const int32_t h = id[j];
            id[j] = sv.hh[k > 4 ? k - 4 : 0];
            --r;
            while (r >= 0 && ro[r] > h) --r;
            if (r < 0 || h >= ro[r + 1]) return false;
            strip[k * TPC_WAVE] = (uint8_t)r;
        }
    }
    return true;
}

// fs0: the (frame, sector) whose row starts L.start[0] holds (L.start[1] the
// next one's), -1 if some seed of the wavefront lies in neither.
template <bool ROWS, bool ERRS>
__device__ inline void fit_ms_one(const MsArgs &A, int i, const float *xs, RowLds *L, int fs0) {
    static_assert(ROWS || !ERRS, "per-cluster errors come with the row lookup");
    const FitArgs &F = A.F;
    SeedView sv = seed_view(F, i);
    uint8_t *strip = ROWS ? L->s + (threadIdx.x & (TPC_WAVE - 1)) : nullptr;
    int ra = 0, rb = 0, rc = 0;                   // rows of hits n-1, (n-1)/2, 0
    bool refused = false;
    if (ROWS) {
        // the layout gives the rows; first_row is not read
        const int32_t fi = A.frame[i];
        const bool inb = sv.n >= 3 && sv.o0 >= 0 && sv.o0 <= F.cap_hits - sv.n;
        if (inb && A.rejected)
            for (int k = 0; k < sv.n; ++k) A.rejected[sv.o0 + k] = 0;
        sv.sane = inb && sv.sec >= 0 && sv.sec < F.n_sectors && fi >= 0 && fi < A.n_frames;
        if (sv.sane) {
            const int fs = fi * F.n_sectors + sv.sec;
            if (fs0 >= 0) sv.sane = seed_rows(L->start[fs - fs0], F.n_rows, sv, strip);
            else sv.sane = seed_rows(A.row_offsets + (size_t)fs * F.n_rows, F.n_rows, sv, strip);
        }
        if (sv.sane) {
            ra = strip[(sv.n - 1) * TPC_WAVE];
            rb = strip[(sv.n - 1) / 2 * TPC_WAVE];
            rc = strip[0];
        }
        refused = !sv.sane;
    } else {
        if (sv.sane) {
            ra = sv.row0 + sv.n - 1;
            rb = sv.row0 + (sv.n - 1) / 2;
            rc = sv.row0;
        }
        if (sv.sane && A.rejected)
            for (int k = 0; k < sv.n; ++k) A.rejected[sv.o0 + k] = 0;
    }
    double p[5] = {0, 0, 0, 0, 0};
    SymT<double> C = {};
    double chi2 = 0.0;
    int status = TPC_FIT_OK, used = 1;
    double xcur = sv.sane ? (double)xs[ra] : 0.0;
    double vy = F.vy, vz = F.vz;
    if (ERRS && sv.sane) {
        const float2 e = A.err[sv.o0 + sv.n - 1];
        vy = (double)e.x * (double)e.x;
        vz = (double)e.y * (double)e.y;
    }
    if (!sv.sane) {
        status = TPC_FIT_INIT_FAIL;
    } else {
        const int ka = sv.n - 1, kb = (sv.n - 1) / 2;
        double ya, za, yb, zb, yc, zc;
        hit_meas(F, sv, ka, ya, za);
        hit_meas(F, sv, kb, yb, zb);
        hit_meas(F, sv, 0, yc, zc);
        (void)zb;
        if (!helix_start<double, double>((double)xs[ra], ya, za, (double)xs[rb], yb, (double)xs[rc], yc, zc,
                                         A.kbz, F.max_sin, p))
            status = TPC_FIT_INIT_FAIL;
    }
    if (!refused) {
        C.c00 = vy;
        C.c11 = vz;
        C.c22 = F.var_s;
        C.c33 = F.var_t;
        C.c44 = F.var_w;
    }
    if (status == TPC_FIT_OK) {
        // a hit's coordinates (and, with ERRS, its error), its row and its
        // plane are read a step ahead
        const float2 *hp = F.hyz + sv.o0 + sv.n - 2, *ep = ERRS ? A.err + sv.o0 + sv.n - 2 : nullptr;
        float2 raw = *hp, en = ERRS ? *ep : make_float2(0.f, 0.f);
        if (ROWS && A.rows_out) A.rows_out[sv.o0 + sv.n - 1] = (int16_t)ra;
        int rn = ROWS ? (int)strip[(sv.n - 2) * TPC_WAVE] : sv.row0 + sv.n - 2;
        float xn = xs[rn];
        for (int k = sv.n - 2; k >= 0; --k) {
            double my, mz;
            hit_fix<false>(sv, k, raw, my, mz);
            hp -= k > 0;
            raw = *hp;
            if (ROWS && A.rows_out) A.rows_out[sv.o0 + k] = (int16_t)rn;
            const double xk = (double)xn;
            if (k > 0) {
                rn = ROWS ? (int)strip[(k - 1) * TPC_WAVE] : rn - 1;
                xn = xs[rn];
            }
            if (ERRS) {
                vy = (double)en.x * (double)en.x;
                vz = (double)en.y * (double)en.y;
                ep -= k > 0;
                en = *ep;
            }
            const double dx = xk - xcur;
            if (A.scatter || A.eloss) {
                const Segment g = segment(A, p, dx);
                add_scattering(A, p, g, C);
                if (A.eloss) {
                    double w1, a, b, vw;
                    if (eloss_map(A, p, g, 1.0, w1, a, b, vw)) {
                        status = TPC_FIT_SIN_FAIL;
                        break;
                    }
                    C.c44 += vw;
                    eloss_cov(C, a, b);
                    p[4] = w1;
                }
            }
            StepJac J;
            if (!helix_step<double, double>(p, dx, A.kbz, F.max_sin, J)) {
                status = TPC_FIT_SIN_FAIL;
                break;
            }
            sym_transport<double, false>(C, J);
            xcur = xk;
            // the update, unless the predicted-residual chi2 rejects the hit
            // (a singular S is not a rejection: the update reports it, -1)
            double pn[5] = {p[0], p[1], p[2], p[3], p[4]};
            Gain<double> G;
            const double dchi = kalman_gain<double>(pn, C, my, mz, vy, vz, G);
            if (dchi > A.cut) {
                if (A.rejected) A.rejected[sv.o0 + k] = 1;
                continue;
            }
            kalman_cov(C, G, vy, vz);
            for (int q = 0; q < 5; ++q) p[q] = pn[q];
            chi2 += dchi;
            const double chk = chi2 + p[0] + p[1] + p[2] + p[3] + p[4];
            if (!((int)(dchi >= 0.0) & (int)(chk - chk == 0.0))) {
                status = TPC_FIT_NUM_FAIL;
                break;
            }
            ++used;
        }
    }
    if (A.pfin)
        for (int q = 0; q < 5; ++q) A.pfin[(size_t)i * 5 + q] = p[q];
    F.out.x[i] = (float)xcur;
    float *po = F.out.par + (size_t)i * 5;
    for (int q = 0; q < 5; ++q) po[q] = (float)p[q];
    float *co = F.out.cov + (size_t)i * 15;
    const double cc[15] = {C.c00, C.c10, C.c11, C.c20, C.c21, C.c22, C.c30, C.c31,
                           C.c32, C.c33, C.c40, C.c41, C.c42, C.c43, C.c44};
    for (int q = 0; q < 15; ++q) co[q] = (float)cc[q];
    F.out.chi2[i] = (float)chi2;
    F.out.ndf[i] = 2 * used - 5;
    F.out.status[i] = status;
}

// Workgroups of one wavefront: an event's seeds make fewer wavefronts than
// there are SIMDs, and single ones spread over all CUs.
#define MS_T TPC_WAVE
template <bool ROWS, bool ERRS>
__global__ void __launch_bounds__(MS_T) fit_ms_tracks(MsArgs A) {
    __shared__ float xs[TPC_MAX_ROWS];
    for (int r = threadIdx.x; r < A.F.n_rows; r += MS_T) xs[r] = A.F.row_x[r];
    __syncthreads();
    RowLds *L = nullptr;
    if constexpr (ROWS) {
        __shared__ RowLds rows;
        L = &rows;
    }
    int T = *A.F.n_seeds;
    if (T > A.F.cap_seeds) T = A.F.cap_seeds;
    for (int i0 = blockIdx.x * MS_T; i0 < T; i0 += gridDim.x * MS_T) {
        const int i = i0 + threadIdx.x;
        int fs0 = -1;
        if (ROWS) {
            // the row starts of the seeds' (frame, sector)s, if two in a row hold them all
            const int n_fs = A.n_frames * A.F.n_sectors;
            int fs = i < T ? A.frame[i] : -1;
            fs = (uint32_t)fs < (uint32_t)A.n_frames ? fs * A.F.n_sectors + A.F.sector[i] : -1;
            const bool in = (uint32_t)fs < (uint32_t)n_fs;
            int lo = in ? fs : INT32_MAX;
#pragma unroll
            for (int d = TPC_WAVE / 2; d > 0; d >>= 1) {
                const int o = __shfl_xor(lo, d, TPC_WAVE);
                lo = o < lo ? o : lo;
            }
            if (lo != INT32_MAX && __ballot(in && fs > lo + 1) == 0ull) fs0 = lo;
            __syncthreads();
            if (fs0 >= 0)
                for (int r = threadIdx.x; r <= A.F.n_rows; r += MS_T) {
                    L->start[0][r] = A.row_offsets[(size_t)fs0 * A.F.n_rows + r];
                    if (fs0 + 1 < n_fs) L->start[1][r] = A.row_offsets[(size_t)(fs0 + 1) * A.F.n_rows + r];
                }
            __syncthreads();
        }
        if (i < T) fit_ms_one<ROWS, ERRS>(A, i, xs, L, fs0);
    }
}

// Errors of every seed hit in seed-hit order, so that the fit reads them as
// it reads the coordinates (from the id that a step loads, the error's load
// was waited for in every step).  The whole capacity: a seed list that
// exceeded it, or has a malformed seed, holds good seeds whose hits neither
// the last offset nor the count bounds.  (Ids behind the last seed are
// whatever the buffer holds; their errors are not read.)
__global__ void __launch_bounds__(TPC_BLOCK)
gather_err(int32_t cap_hits, const int32_t *__restrict__ hits, const float2 *__restrict__ err, int32_t N,
           float2 *__restrict__ out) {
    for (int64_t j = blockIdx.x * TPC_BLOCK + threadIdx.x; j < cap_hits; j += gridDim.x * TPC_BLOCK) {
        const int32_t id = hits[j];
        out[j] = (uint32_t)id < (uint32_t)N ? err[id] : make_float2(0.f, 0.f);
    }
}

// Per seed hit the smoother keeps the filtered deviation (5), its
// covariance (15, packed), the reference state (5) and the step that leaves
// the hit's plane inwards (helix Jacobian (6), scattering and straggling
// noise (4), energy-loss factors (2)) in 38 doubles, 16-byte aligned.
constexpr int SM_REC = 38, SM_R = 20, SM_J = 26, SM_Q = 32, SM_E = 36;

__device__ inline void load_record(const double *rec, double w[SM_REC]) {
    const double2 *v = reinterpret_cast<const double2 *>(rec);
    for (int q = 0; q < SM_REC / 2; ++q) {
        const double2 x = v[q];
        w[2 * q] = x.x;
        w[2 * q + 1] = x.y;
    }
}

struct SmArgs {
    MsArgs M;
    SmWs w;
    const uint8_t *rej;
    float *hit_par, *hit_cov;
};

__device__ inline void sym_add(SymT<double> &C, const SymT<double> &Q) {
    C.c00 += Q.c00; C.c10 += Q.c10; C.c11 += Q.c11; C.c20 += Q.c20; C.c21 += Q.c21;
    C.c22 += Q.c22; C.c30 += Q.c30; C.c31 += Q.c31; C.c32 += Q.c32; C.c33 += Q.c33;
    C.c40 += Q.c40; C.c41 += Q.c41; C.c42 += Q.c42; C.c43 += Q.c43; C.c44 += Q.c44;
}

__device__ inline void sym_dense(const SymT<double> &C, double M[5][5]) {
    const double v[15] = {C.c00, C.c10, C.c11, C.c20, C.c21, C.c22, C.c30, C.c31,
                          C.c32, C.c33, C.c40, C.c41, C.c42, C.c43, C.c44};
    int q = 0;
    for (int r = 0; r < 5; ++r)
        for (int c = 0; c <= r; ++c, ++q) M[r][c] = M[c][r] = v[q];
}

// d <- F d for the step Jacobian (identity plus the six off-diagonal terms).
__device__ inline void jac_apply(const StepJac &J, const double d[5], double o[5]) {
    o[0] = d[0] + J.f02 * d[2] + J.f04 * d[4];
    o[1] = d[1] + J.f12 * d[2] + J.f13 * d[3] + J.f14 * d[4];
    o[2] = d[2] + J.f24 * d[4];
    o[3] = d[3];
    o[4] = d[4];
}

// A = F C (dense) for the step Jacobian.
__device__ inline void jac_times(const StepJac &J, const double C[5][5], double A[5][5]) {
    for (int c = 0; c < 5; ++c) {
        A[0][c] = C[0][c] + J.f02 * C[2][c] + J.f04 * C[4][c];
        A[1][c] = C[1][c] + J.f12 * C[2][c] + J.f13 * C[3][c] + J.f14 * C[4][c];
        A[2][c] = C[2][c] + J.f24 * C[4][c];
        A[3][c] = C[3][c];
        A[4][c] = C[4][c];
    }
}

// Solves P X = A (P symmetric positive definite, 5x5, lower triangle read)
// in place of A by P = L D L^T: five reciprocals and no square root; false
// if a pivot is not positive.
__device__ inline bool ldl_solve(double P[5][5], double A[5][5]) {
    double iD[5];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        double v[5], d = P[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) {
            v[k] = P[j][k];                          // L[j][k] D[k]
            P[j][k] = v[k] * iD[k];                  // L[j][k]
            d -= P[j][k] * v[k];
        }
        ok = ok && d > 0.0;
        iD[j] = recip_pos(d);
#pragma unroll
        for (int r = j + 1; r < 5; ++r)              // L[r][j] D[j]
#pragma unroll
            for (int k = 0; k < j; ++k) P[r][j] -= P[r][k] * P[j][k];
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) {
#pragma unroll
        for (int r = 1; r < 5; ++r)                  // L y = a
#pragma unroll
            for (int k = 0; k < r; ++k) A[r][c] -= P[r][k] * A[k][c];
#pragma unroll
        for (int r = 4; r >= 0; --r) {               // D L^T x = y
            A[r][c] *= iD[r];
#pragma unroll
            for (int k = r + 1; k < 5; ++k) A[r][c] -= P[k][r] * A[k][c];
        }
    }
    return ok;
}

template <bool ERRS>
__device__ inline void smooth_one(const SmArgs &S, int i, const float *xs) {
    const MsArgs &A = S.M;
    const FitArgs &F = A.F;
    const SeedView sv = seed_view(F, i);
    const int n = sv.n;
    if (!(n >= 3 && sv.o0 >= 0 && sv.o0 <= F.cap_hits - n)) return;
    float *hp = S.hit_par + (size_t)sv.o0 * 5;
    float *hc = S.hit_cov + (size_t)sv.o0 * 15;
    int status = F.out.status[i];
    if (status == TPC_FIT_OK) {
        // the fit accepted the seed and stored the row of every hit
        const double *pf = S.w.pfin + (size_t)i * 5;
        double *wd = S.w.wd + (size_t)sv.o0 * SM_REC;
        const int16_t *wr = S.w.wrow + sv.o0;
        const int ra = wr[n - 1], rc = wr[0];
        const uint8_t *rej = S.rej + sv.o0;
        // the reference at the outermost plane: one helix step from the fit's
        // final state, or, with energy loss, plane by plane taking the loss away
        double R[5];
        for (int q = 0; q < 5; ++q) R[q] = pf[q];
        StepJac J;
        if (A.eloss) {
            int row = wr[1], rlast = rc;
            for (int k = 1; k < n && status == TPC_FIT_OK; ++k) {
                const double dx = (double)xs[row] - (double)xs[rlast];
                rlast = row;
                row = wr[k + 1 < n ? k + 1 : k];
                double w1 = R[4], a, b, vw;
                if (!helix_step<double, double>(R, dx, A.kbz, F.max_sin, J) ||
                    eloss_map(A, R, segment(A, R, dx), -1.0, w1, a, b, vw))
                    status = TPC_FIT_SIN_FAIL;
                R[4] = w1;
            }
        } else if (!helix_step<double, double>(R, (double)xs[ra] - (double)xs[rc], A.kbz, F.max_sin, J)) {
            status = TPC_FIT_SIN_FAIL;
        }
        double vy = F.vy, vz = F.vz;
        if (ERRS) {
            const float2 e = A.err[sv.o0 + n - 1];
            vy = (double)e.x * (double)e.x;
            vz = (double)e.y * (double)e.y;
        }
        // inwards along the reference: Kalman filter of the deviation d;
        // the hit, its row and flag are read a step ahead
        double d[5] = {0, 0, 0, 0, 0};
        SymT<double> C = {};
        C.c00 = 1e4 * vy;
        C.c11 = 1e4 * vz;
        C.c22 = F.var_s;
        C.c33 = F.var_t;
        C.c44 = F.var_w;
        const float2 *hz = F.hyz + sv.o0;
        float2 raw = hz[n - 1];
        int rj = rej[n - 1];
        float xr = xs[ra], xl = xr;                   // x of planes k and k + 1
        int row = wr[n - 2];                          // row of plane k - 1
        for (int k = n - 1; k >= 0 && status == TPC_FIT_OK; --k) {
            const float2 hk = raw;
            const int rjk = rj, kn = k > 0 ? k - 1 : 0;
            const float xc = xr;
            raw = hz[kn];
            rj = rej[kn];
            xr = xs[row];
            row = wr[k > 1 ? k - 2 : 0];
            if (k < n - 1) {
                // the step from plane k + 1 to plane k, kept with plane k + 1
                SymT<double> Q = {};
                double ea = 0.0, eb = 1.0;
                const double dx = (double)xc - (double)xl;
                const Segment g = (A.scatter || A.eloss) ? segment(A, R, dx) : Segment{};
                add_scattering(A, R, g, Q);
                if (A.eloss) {
                    double w1, vw;
                    if (eloss_map(A, R, g, 1.0, w1, ea, eb, vw)) {
                        status = TPC_FIT_SIN_FAIL;
                        break;
                    }
                    Q.c44 += vw;
                    sym_add(C, Q);
                    eloss_cov(C, ea, eb);
                    d[4] = ea * d[3] + eb * d[4];
                    R[4] = w1;
                } else {
                    sym_add(C, Q);
                }
                if (!helix_step<double, double>(R, dx, A.kbz, F.max_sin, J)) {
                    status = TPC_FIT_SIN_FAIL;
                    break;
                }
                double2 *w = reinterpret_cast<double2 *>(wd + (size_t)(k + 1) * SM_REC + SM_J);
                w[0] = make_double2(J.f02, J.f04);
                w[1] = make_double2(J.f12, J.f13);
                w[2] = make_double2(J.f14, J.f24);
                w[3] = make_double2(Q.c22, Q.c33);
                w[4] = make_double2(Q.c43, Q.c44);
                w[5] = make_double2(ea, eb);
                double nd[5];
                jac_apply(J, d, nd);
                for (int q = 0; q < 5; ++q) d[q] = nd[q];
                sym_transport<double, false>(C, J);
                if (ERRS) {
                    const float2 e = A.err[sv.o0 + k];
                    vy = (double)e.x * (double)e.x;
                    vz = (double)e.y * (double)e.y;
                }
            }
            xl = xc;
            if (!rjk) {
                const double dchi =
                    kalman_update<double>(d, C, (double)hk.x - R[0], (double)hk.y - R[1], vy, vz);
                const double chk = dchi + d[0] + d[1] + d[2] + d[3] + d[4];
                if (!(chk - chk == 0.0)) {
                    status = TPC_FIT_NUM_FAIL;
                    break;
                }
            }
            double2 *w = reinterpret_cast<double2 *>(wd + (size_t)k * SM_REC);
            w[0] = make_double2(d[0], d[1]);
            w[1] = make_double2(d[2], d[3]);
            w[2] = make_double2(d[4], C.c00);
            w[3] = make_double2(C.c10, C.c11);
            w[4] = make_double2(C.c20, C.c21);
            w[5] = make_double2(C.c22, C.c30);
            w[6] = make_double2(C.c31, C.c32);
            w[7] = make_double2(C.c33, C.c40);
            w[8] = make_double2(C.c41, C.c42);
            w[9] = make_double2(C.c43, C.c44);
            w[10] = make_double2(R[0], R[1]);
            w[11] = make_double2(R[2], R[3]);
            w[12] = make_double2(R[4], 0.0);
        }
        // outwards: Rauch-Tung-Striebel, each record read a step ahead
        if (status == TPC_FIT_OK) {
            double ds[5] = {0, 0, 0, 0, 0}, Cs[5][5] = {};
            // smoothed state and covariance of plane k from its record and
            // those of plane k - 1 in (ds, Cs); false if P is singular
            auto rts = [&](int k, const double *w) {
                const SymT<double> Ck = {w[5],  w[6],  w[7],  w[8],  w[9],  w[10], w[11], w[12],
                                         w[13], w[14], w[15], w[16], w[17], w[18], w[19]};
                bool ok = true;
                if (k == 0) {
                    for (int q = 0; q < 5; ++q) ds[q] = w[q];
                    sym_dense(Ck, Cs);
                } else {
                    // the step inwards from plane k: F = Jh Je, noise Q
                    const StepJac Jk = {w[SM_J], w[SM_J + 1], w[SM_J + 2], w[SM_J + 3], w[SM_J + 4], w[SM_J + 5]};
                    const double ea = w[SM_E], eb = w[SM_E + 1];
                    SymT<double> Pq = Ck;
                    Pq.c22 += w[SM_Q];
                    Pq.c33 += w[SM_Q + 1];
                    Pq.c43 += w[SM_Q + 2];
                    Pq.c44 += w[SM_Q + 3];
                    double Cd[5][5], EC[5][5], X[5][5], ed[5] = {w[0], w[1], w[2], w[3], w[4]};
                    sym_dense(Ck, Cd);
                    sym_dense(Ck, EC);
                    if (A.eloss) {
                        eloss_cov(Pq, ea, eb);
                        ed[4] = ea * w[3] + eb * w[4];
                        for (int b = 0; b < 5; ++b) EC[4][b] = ea * Cd[3][b] + eb * Cd[4][b];
                    }
                    jac_times(Jk, EC, X);                        // F C_k
                    sym_transport<double, false>(Pq, Jk);       // P = F (C_k + Q) F^T
                    double P[5][5], D[5][5];
                    sym_dense(Pq, P);
                    for (int a = 0; a < 5; ++a)
                        for (int b = 0; b < 5; ++b) D[a][b] = Cs[a][b] - P[a][b];
                    ok = ldl_solve(P, X);                        // X = P^-1 F C_k = G^T
                    double pd[5], e[5];
                    jac_apply(Jk, ed, pd);
                    for (int q = 0; q < 5; ++q) e[q] = ds[q] - pd[q];
                    for (int a = 0; a < 5; ++a) {
                        double acc = w[a];
                        for (int b = 0; b < 5; ++b) acc += X[b][a] * e[b];
                        ds[a] = acc;
                    }
                    // Cs <- C_k + G (Cs - P) G^T
                    double T[5][5];
                    for (int a = 0; a < 5; ++a)
                        for (int b = 0; b < 5; ++b) {
                            double acc = 0.0;
                            for (int c = 0; c < 5; ++c) acc += X[c][a] * D[c][b];
                            T[a][b] = acc;
                        }
                    for (int a = 0; a < 5; ++a)
                        for (int b = 0; b <= a; ++b) {
                            double acc = Cd[a][b];
                            for (int c = 0; c < 5; ++c) acc += T[a][c] * X[c][b];
                            Cs[a][b] = Cs[b][a] = acc;
                        }
                }
                float *o = hp + (size_t)k * 5, *oc = hc + (size_t)k * 15;
                for (int q = 0; q < 5; ++q) o[q] = (float)(w[SM_R + q] + ds[q]);
                int q = 0;
                for (int a = 0; a < 5; ++a)
                    for (int b = 0; b <= a; ++b, ++q) oc[q] = (float)Cs[a][b];
                return ok;
            };
            double wa[SM_REC], wb[SM_REC];
            load_record(wd, wa);
            bool ok = true;
            for (int k = 0; k < n && ok; k += 2) {
                const int k1 = k + 1 < n ? k + 1 : n - 1, k2 = k + 2 < n ? k + 2 : n - 1;
                load_record(wd + (size_t)k1 * SM_REC, wb);
                ok = rts(k, wa);
                if (!ok || k + 1 >= n) break;
                load_record(wd + (size_t)k2 * SM_REC, wa);
                ok = rts(k + 1, wb);
            }
            if (!ok) status = TPC_FIT_NUM_FAIL;
        }
        if (status != TPC_FIT_OK) F.out.status[i] = status;
    }
    if (status != TPC_FIT_OK) {
        for (int k = 0; k < n; ++k) {
            for (int q = 0; q < 5; ++q) hp[(size_t)k * 5 + q] = 0.f;
            for (int q = 0; q < 15; ++q) hc[(size_t)k * 15 + q] = 0.f;
        }
    }
}

template <bool ERRS>
__global__ void __launch_bounds__(MS_T) smooth_tracks(SmArgs S) {
    __shared__ float xs[TPC_MAX_ROWS];
    for (int r = threadIdx.x; r < S.M.F.n_rows; r += MS_T) xs[r] = S.M.F.row_x[r];
    __syncthreads();
    int T = *S.M.F.n_seeds;
    if (T > S.M.F.cap_seeds) T = S.M.F.cap_seeds;
    for (int i = blockIdx.x * MS_T + threadIdx.x; i < T; i += gridDim.x * MS_T)
        smooth_one<ERRS>(S, i, xs);
}

MsArgs make_ms_args(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd, const float *err,
                    const tpc_material *mat, const tpc_tracks *tr, uint8_t *rejected, void *ws, hipStream_t st) {
    MsArgs A;
    A.F = make_fit_args(ctx, sd, nullptr);
    A.F.out = *tr;
    float2 *hyz, *herr;
    fit_ws_layout(ws, sd->cap_seeds, sd->cap_hits, nullptr, &hyz, nullptr, &herr);
    A.err = nullptr;
    if (err) {
        int64_t blocks = ((int64_t)sd->cap_hits + TPC_BLOCK - 1) / TPC_BLOCK;
        blocks = blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks);
        hipLaunchKernelGGL(gather_err, dim3((unsigned)blocks), dim3(TPC_BLOCK), 0, st, sd->cap_hits, sd->hits,
                           reinterpret_cast<const float2 *>(err), fr->n_clusters, herr);
        A.err = herr;
    }
    if (sd->hit_yz) {
        A.F.hyz = reinterpret_cast<const float2 *>(sd->hit_yz);
    } else {
        A.F.hyz = hyz;
        (void)launch_gather(fr, sd, hyz, st);    // a launch error surfaces at the fit's launch
    }
    A.kbz = -0.00299792458 * (double)ctx->cfg.bz;
    A.inv_x0 = mat ? 1.0 / (double)mat->x0 : 0.0;
    A.scatter = mat && mat->x0 < INFINITY;
    A.mass2 = mat ? (double)mat->mass * (double)mat->mass : 0.0;
    A.cut = mat ? (double)mat->chi2_cut : (double)INFINITY;
    A.eloss = mat && mat->rho > 0.f;
    A.mass = mat ? (double)mat->mass : 0.0;
    A.rho = mat ? (double)mat->rho : 0.0;
    A.kza = mat ? 0.307075e-3 * (double)mat->z_over_a : 0.0;
    A.inv_mass = A.eloss ? 1.0 / A.mass : 0.0;
    A.inv_mass2 = A.eloss ? 1.0 / A.mass2 : 0.0;
    A.me_over_m = A.eloss ? 0.51099895e-3 / A.mass : 0.0;
    A.inv_exc2 = A.eloss ? 1.0 / ((double)mat->mean_exc * (double)mat->mean_exc) : 0.0;
    A.rejected = rejected;
    A.row_offsets = fr->row_offsets;
    A.frame = sd->frame;
    A.n_frames = fr->n_frames;
    A.pfin = nullptr;
    A.rows_out = nullptr;
    return A;
}

int fit_blocks(const tpc_seeds *sd) {
    int blocks = (sd->cap_seeds + MS_T - 1) / MS_T;
    if (blocks > 32768) blocks = 32768;
    if (blocks < 1) blocks = 1;
    return blocks;
}

}  // namespace

hipError_t launch_fit_material(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd,
                               const tpc_material *mat, const tpc_tracks *tr, uint8_t *rejected,
                               void *ws, hipStream_t st) {
    const MsArgs A = make_ms_args(ctx, fr, sd, nullptr, mat, tr, rejected, ws, st);
    hipLaunchKernelGGL((fit_ms_tracks<false, false>), dim3(fit_blocks(sd)), dim3(MS_T), 0, st, A);
    return hipGetLastError();
}

hipError_t launch_fit_rows(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd, const float *err,
                           const tpc_material *mat, const tpc_tracks *tr, uint8_t *rejected, void *ws,
                           hipStream_t st) {
    const MsArgs A = make_ms_args(ctx, fr, sd, err, mat, tr, rejected, ws, st);
    if (err)
        hipLaunchKernelGGL((fit_ms_tracks<true, true>), dim3(fit_blocks(sd)), dim3(MS_T), 0, st, A);
    else
        hipLaunchKernelGGL((fit_ms_tracks<true, false>), dim3(fit_blocks(sd)), dim3(MS_T), 0, st, A);
    return hipGetLastError();
}

size_t smooth_ws_layout(void *ws, int64_t cap_seeds, int64_t cap_hits, SmWs *out) {
    const size_t fb = fit_ws_layout(nullptr, cap_seeds, cap_hits, nullptr, nullptr);
    WsCarver w(ws ? (void *)((char *)ws + fb) : nullptr);
    double *pfin = w.take<double>((size_t)(cap_seeds > 0 ? cap_seeds : 1) * 5);
    double *wd = w.take<double>((size_t)(cap_hits > 0 ? cap_hits : 1) * SM_REC);
    int16_t *wrow = w.take<int16_t>((size_t)(cap_hits > 0 ? cap_hits : 1));
    if (out) *out = SmWs{pfin, wd, wrow};
    return fb + ((w.off + 255) & ~size_t(255));
}

hipError_t launch_smooth(const tpc_context *ctx, const tpc_frames *fr, const tpc_seeds *sd, const float *err,
                         const tpc_material *mat, const tpc_tracks *tr, uint8_t *rejected, float *hit_par,
                         float *hit_cov, void *ws, hipStream_t st) {
    SmArgs S;
    S.M = make_ms_args(ctx, fr, sd, err, mat, tr, rejected, ws, st);
    smooth_ws_layout(ws, sd->cap_seeds, sd->cap_hits, &S.w);
    S.M.pfin = S.w.pfin;
    S.M.rows_out = S.w.wrow;
    S.rej = rejected;
    S.hit_par = hit_par;
    S.hit_cov = hit_cov;
    const int blocks = fit_blocks(sd);
    if (err) {
        hipLaunchKernelGGL((fit_ms_tracks<true, true>), dim3(blocks), dim3(MS_T), 0, st, S.M);
        hipLaunchKernelGGL((smooth_tracks<true>), dim3(blocks), dim3(MS_T), 0, st, S);
    } else {
        hipLaunchKernelGGL((fit_ms_tracks<true, false>), dim3(blocks), dim3(MS_T), 0, st, S.M);
        hipLaunchKernelGGL((smooth_tracks<false>), dim3(blocks), dim3(MS_T), 0, st, S);
    }
    return hipGetLastError();
}
