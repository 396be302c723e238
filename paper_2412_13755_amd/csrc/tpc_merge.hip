// Merging of fitted track segments across sector edges (gfx950).  A particle
// that crosses from one sector into the next on the same side leaves a
// fitted segment in each; carried to a common plane, their states agree
// within their covariances.
//
//  mg_best         lanes share a segment: over the segments of the two
//                  neighbouring sectors of its (frame, side) -- a contiguous
//                  seed range each, found by binary search, since seeds are
//                  ordered by first cluster and clusters by (frame, sector,
//                  row) -- its best outer partner (its innermost point at
//                  the smaller radius) and best inner partner: smallest chi2
//                  <= cut, smaller index on ties.  Pairs whose (tan(lambda),
//                  q/pT) difference alone has a chi2 above the cut are
//                  dropped first (both are unchanged by the transfer, so
//                  their covariance block is the sum of the two segments',
//                  and a sub-vector's chi2 never exceeds the full one: such a
//                  pair cannot pass); the survivors of each chunk of
//                  candidates go to the lane's own LDS column and only
//                  they are transferred.  FP64 throughout.
//  mg_link_next    next[a] = b when a's best outer partner b has a as its
//                  best inner partner (else -1, chi2 0); optionally the pair
//                  combined at b's plane (a's transferred state fused with
//                  b's: the joint fit of both for the linearised problem)
//  mg_link_prev    prev[b] = a when next[a] = b
//  lg_best, lg_link  optionally, the legs of loopers: per segment the
//                  best partner among the segments of its frame and side
//                  whose circle matches with curvature and tan(lambda)
//                  reversed, then mutual best
//
// The transfer: a state at plane x of the inner segment's frame is rotated
// into the outer segment's frame (turned by da: a point (x, y) ->
// (x cos da + y sin da, -x sin da + y cos da), phi -> phi - da, cos phi > 0
// kept) and carried along the helix to the outer segment's innermost plane;
// its Jacobian is the step's (at fixed distance) times the rotation's, plus
// the move of the start plane with y, which shortens the step.
#include "tpc_fit_math.hpp"
#include "tpc_merge.hpp"

namespace {

struct MgArgs {
    const float *x, *par, *cov;
    const int32_t *status, *frame, *sector, *n_seeds;
    int32_t cap, n_sectors;
    double kbz, cut;
    float max_sin;
    int32_t *next, *prev;
    float *chi2;
    float *mpar, *mcov;      // optional combined states of linked pairs
    int32_t *leg;            // optional pairing of the legs of loopers
    float *leg_chi2;
};

__device__ inline int mg_count(const MgArgs &A) {
    const int n = *A.n_seeds;
    return n < 0 ? 0 : (n < A.cap ? n : A.cap);
}

__device__ inline int64_t mg_key(const MgArgs &A, int i) {
    return (int64_t)A.frame[i] * A.n_sectors + A.sector[i];
}

// First seed index in [0, T) whose key is >= k.
__device__ inline int mg_lower(const MgArgs &A, int T, int64_t k) {
    int lo = 0, hi = T;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (mg_key(A, mid) < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ inline double sector_angle(int sec, int n_sectors) {
    const double pi = 3.14159265358979323846;
    return n_sectors == 1 ? 0.0 : (double)(sec % 18) * (pi / 9.0) + pi / 18.0;
}

// The angle that turns sector a's frame into sector b's, wrapped to (-pi, pi].
__device__ inline double turn_angle(int sa, int sb, int n_sectors) {
    const double pi = 3.14159265358979323846;
    double da = sector_angle(sb, n_sectors) - sector_angle(sa, n_sectors);
    if (da > pi) da -= 2.0 * pi;
    if (da < -pi) da += 2.0 * pi;
    return da;
}

#define TPC_MG_SLACK 1.000001   // far above the rounding of a chi2

// chi2 of carrying segment a onto segment b (INFINITY if it cannot be
// formed, or if it exceeds lim for certain); ca, sa: cos and sin of the turn
// from a's sector to b's.  With mp, mc non-null also the two combined at b's
// plane: a's transferred state (covariance P = J C_a J^T) and b's fused,
// x = p_a' + P S^-1 (p_b - p_a'), C = P S^-1 C_b (= P - P S^-1 P),
// S = P + C_b (packed, in float).
//
// chi2 = u^T D^-1 u with S = L D L^T, L u = d (L's diagonal is 1), grows
// with every component eliminated.  They are taken in the order (t, w, z, s,
// y): two candidates of similar direction and momentum lie anywhere along
// the beam, so z decides against nearly all of them after its own row of S,
// before the other rows are formed.
__device__ double pair_fuse(const MgArgs &A, int a, int b, double ca, double sa, double lim, float *mp, float *mc) {
    const float *pa = A.par + (size_t)a * 5, *pb = A.par + (size_t)b * 5;
    const double x = (double)A.x[a], y = (double)pa[0], s = (double)pa[2], t = (double)pa[3], w = (double)pa[4];
    if (!(fabs(s) < 1.0)) return INFINITY;
    double ic, ic2;
    const double c = sqrt_pos(fma(-s, s, 1.0), &ic);
    if (!(c * ca + s * sa > 0.0)) return INFINITY;
    const double x1 = x * ca + y * sa;
    double q[5] = {-x * sa + y * ca, (double)pa[1], s * ca - c * sa, t, w};
    StepJac F;
    if (!helix_step<double, double>(q, (double)A.x[b] - x1, A.kbz, A.max_sin, F)) return INFINITY;
    // J = F R - v e_0^T sin(da), R = diag(ca, 1, ca + (s/c) sa, 1, 1), v = (s2/c2, t/c2, kappa, 0, 0)
    const double r22 = ca + s * ic * sa;
    const double s2 = q[2], kap = A.kbz * w;
    sqrt_pos(fma(-s2, s2, 1.0), &ic2);
    double J[3][5];
    J[0][0] = ca - sa * s2 * ic2; J[0][1] = 0.0; J[0][2] = F.f02 * r22; J[0][3] = 0.0;   J[0][4] = F.f04;
    J[1][0] = -sa * t * ic2;      J[1][1] = 1.0; J[1][2] = F.f12 * r22; J[1][3] = F.f13; J[1][4] = F.f14;
    J[2][0] = -sa * kap;          J[2][1] = 0.0; J[2][2] = r22;         J[2][3] = 0.0;   J[2][4] = F.f24;
    double Ca[5][5], Cb[5][5];
    const float *ca_ = A.cov + (size_t)a * 15, *cb_ = A.cov + (size_t)b * 15;
#pragma unroll
    for (int i = 0, k = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j, ++k) {
            Ca[i][j] = Ca[j][i] = (double)ca_[k];
            Cb[i][j] = Cb[j][i] = (double)cb_[k];
        }
    // P = J Ca J^T in the order of elimination, rows 3 and 4 of J those of
    // the identity; L D in place of S's lower triangle
    constexpr int ord[5] = {3, 4, 1, 2, 0};
    double P[5][5], S[5][5], L[5][5], iD[5], u[5], d[5], chi = 0.0;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int ri = ord[i];
        double JC[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            double acc = ri < 3 ? 0.0 : Ca[ri][j];
            if (ri < 3)
#pragma unroll
                for (int k = 0; k < 5; ++k) acc += J[ri][k] * Ca[k][j];
            JC[j] = acc;
        }
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            const int rj = ord[j];
            double acc = rj < 3 ? 0.0 : JC[rj];
            if (rj < 3)
#pragma unroll
                for (int k = 0; k < 5; ++k) acc += JC[k] * J[rj][k];
            P[i][j] = P[j][i] = acc;
            S[i][j] = acc + Cb[ri][rj];
        }
        d[i] = q[ri] - (double)pb[ri];
        double acc = S[i][i], v = d[i];
#pragma unroll
        for (int j = 0; j < i; ++j) {
            double l = S[i][j];                       // L[i][j] D[j]
#pragma unroll
            for (int k = 0; k < j; ++k) l -= S[i][k] * L[j][k];
            S[i][j] = l;
            L[i][j] = l * iD[j];
            acc -= L[i][j] * l;
            v -= L[i][j] * u[j];
        }
        if (!(acc > 0.0)) return INFINITY;
        iD[i] = recip_pos(acc);
        u[i] = v;
        chi += v * v * iD[i];
        if (i == 2 && chi > lim * TPC_MG_SLACK) return INFINITY;
    }
    if (mp && mc) {
        // X = S^-1 P by the two triangular solves, column by column
        double X[5][5];
        for (int c = 0; c < 5; ++c) {
            double y[5];
            for (int i = 0; i < 5; ++i) {
                double acc = P[i][c];
                for (int k = 0; k < i; ++k) acc -= L[i][k] * y[k];
                y[i] = acc;
            }
            for (int i = 4; i >= 0; --i) {
                double acc = y[i] * iD[i];
                for (int k = i + 1; k < 5; ++k) acc -= L[k][i] * X[k][c];
                X[i][c] = acc;
            }
        }
        // d = p_a' - p_b: x = p_a' - P S^-1 d = p_a' - X^T d
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            double acc = q[ord[i]];
#pragma unroll
            for (int k = 0; k < 5; ++k) acc -= X[k][i] * d[k];
            mp[ord[i]] = (float)acc;
        }
        // C = P S^-1 C_b = X^T C_b, symmetrised (equal to P - P S^-1 P, with
        // no difference of large terms when one covariance dwarfs the other)
        constexpr int pos[5] = {4, 2, 3, 0, 1};       // of component i in the order
#pragma unroll
        for (int i = 0, k = 0; i < 5; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j, ++k) {
                double e = 0.0, f = 0.0;
#pragma unroll
                for (int m = 0; m < 5; ++m) {
                    e += X[m][pos[i]] * Cb[ord[m]][j];
                    f += X[m][pos[j]] * Cb[ord[m]][i];
                }
                mc[k] = (float)(0.5 * (e + f));
            }
    }
    return chi > 0.0 ? chi : INFINITY;
}

__device__ inline double pair_chi2(const MgArgs &A, int a, int b, double ca, double sa, double lim) {
    return pair_fuse(A, a, b, ca, sa, lim, nullptr, nullptr);
}

// SPLIT lanes of one wavefront share a segment and take every SPLIT-th
// candidate of each neighbouring sector (enough wavefronts for the chip);
// their best partners are reduced by shuffles at the end (smaller chi2, then
// smaller index: the serial order's choice).  Per chunk of MG_LANE_CHUNK
// candidates a lane, the ones that pass the tan(lambda) / q/pT test go to the
// lane's own LDS column, so that the transfer runs over short lists (a
// wavefront's iterations are the longest list of its lanes) instead of every
// candidate of every lane.  The test's bound is the best chi2 that any of the
// segment's lanes has found on the candidate's side (shared after each
// chunk), or the cut: a pair whose (t, w) chi2 alone is above it by more than
// rounding (TPC_MG_SLACK) can neither be nor tie the best.
// Sixteen lanes up to MG_MANY segments: four leave the SIMDs 1.1 wavefronts
// each on an event of 2.7 10^4 (515 us, 408 with sixteen; 1.3 10^5: 9.2, 8.9
// ms).  Beyond, four: fewer wavefronts share the bounds of more candidates
// (6.4 10^5: 279 ms with sixteen, 204 with four).
#define MG_MANY (1 << 18)
#define MG_LANE_CHUNK 16

// (chi, j) of another lane replaces this lane's best when smaller, or equal
// with a smaller index
__device__ inline void best_merge(double &chi, int &j, double oc, int oj) {
    if (oc < chi || (oc == chi && oj >= 0 && (j < 0 || oj < j))) {
        chi = oc;
        j = oj;
    }
}

template <int SPLIT>
__device__ __forceinline__ void best_partners(const MgArgs &A, int T, int (*cand)[TPC_BLOCK]) {
    constexpr int CHUNK = SPLIT * MG_LANE_CHUNK;
    const int sub = threadIdx.x % SPLIT;
    const int per_block = TPC_BLOCK / SPLIT;
    // whole workgroups step together: every lane reaches the shuffles
    for (int base = blockIdx.x * per_block; base < T; base += gridDim.x * per_block) {
        const int i = base + threadIdx.x / SPLIT;
        int bo = -1, bi = -1;
        double co = INFINITY, ci_ = INFINITY;         // this lane's best
        double lo = A.cut, li = A.cut;                // the segment's, at most the cut
        if (i < T && A.status[i] == 0 && A.n_sectors == 36) {
            const float *pi_ = A.par + (size_t)i * 5, *ci = A.cov + (size_t)i * 15;
            const double xi = (double)A.x[i], ri = hypot(xi, (double)pi_[0]);
            const double r2i = xi * xi + (double)pi_[0] * (double)pi_[0];
            const double ti = (double)pi_[3], wi = (double)pi_[4], vti = (double)ci[9], vwi = (double)ci[14];
            const double cti = (double)ci[13];
            const int sec = A.sector[i], side = sec / 18, s18 = sec % 18;
            for (int e = 0; e < 2; ++e) {
                const int sn = side * 18 + (e == 0 ? (s18 + 1) % 18 : (s18 + 17) % 18);
                const int64_t key = (int64_t)A.frame[i] * A.n_sectors + sn;
                const int j0 = mg_lower(A, T, key), j1 = mg_lower(A, T, key + 1);
                // the turn from this sector to the neighbour's (outer partners) and back
                const double da = turn_angle(sec, sn, A.n_sectors);
                const double cda = cos(da), sda = sin(da);
                const double dback = turn_angle(sn, sec, A.n_sectors);
                const double cdb = cos(dback), sdb = sin(dback);
                for (int c0 = j0; c0 < j1; c0 += CHUNK) {
                    const int c1 = c0 + CHUNK < j1 ? c0 + CHUNK : j1;
                    int n = 0;
                    for (int j = c0 + sub; j < c1; j += SPLIT) {
                        if (A.status[j] != 0) continue;
                        const float *pj = A.par + (size_t)j * 5, *cj = A.cov + (size_t)j * 15;
                        // the (t, w) block of the pair's covariance is the sum of the
                        // two (the transfer leaves t and w alone), and its chi2
                        // never exceeds the full one
                        const double dt = ti - (double)pj[3], dw = wi - (double)pj[4];
                        const double s33 = vti + (double)cj[9], s44 = vwi + (double)cj[14];
                        const double s43 = cti + (double)cj[13];
                        const double det = s33 * s44 - s43 * s43;
                        // j further out or in beyond rounding of its radius, or undecided
                        const double xj = (double)A.x[j], yj = (double)pj[0], r2j = xj * xj + yj * yj;
                        const double lim = r2j > r2i * (1.0 + 1e-9) ? lo : (r2j < r2i * (1.0 - 1e-9) ? li : fmax(lo, li));
                        if (det > 0.0 &&
                            (s44 * dt * dt - 2.0 * s43 * dt * dw + s33 * dw * dw) > lim * TPC_MG_SLACK * det)
                            continue;
                        cand[n++][threadIdx.x] = j;
                    }
                    for (int k = 0; k < n; ++k) {
                        const int j = cand[k][threadIdx.x];
                        const double rj = hypot((double)A.x[j], (double)A.par[(size_t)j * 5]);
                        if (ri < rj) {                        // j outside: an outer partner
                            const double chi = pair_chi2(A, i, j, cda, sda, fmin(lo, co));
                            if (chi <= A.cut && (chi < co || (chi == co && j < bo))) {
                                co = chi;
                                bo = j;
                            }
                        } else if (rj < ri) {                 // an inner partner
                            const double chi = pair_chi2(A, j, i, cdb, sdb, fmin(li, ci_));
                            if (chi <= A.cut && (chi < ci_ || (chi == ci_ && j < bi))) {
                                ci_ = chi;
                                bi = j;
                            }
                        }
                    }
                    // (the lanes of a segment walk the same chunks together)
                    lo = fmin(lo, co);
                    li = fmin(li, ci_);
#pragma unroll
                    for (int d = 1; d < SPLIT; d <<= 1) {
                        lo = fmin(lo, __shfl_xor(lo, d, TPC_WAVE));
                        li = fmin(li, __shfl_xor(li, d, TPC_WAVE));
                    }
                }
            }
        }
#pragma unroll
        for (int d = 1; d < SPLIT; d <<= 1) {
            best_merge(co, bo, __shfl_xor(co, d, TPC_WAVE), __shfl_xor(bo, d, TPC_WAVE));
            best_merge(ci_, bi, __shfl_xor(ci_, d, TPC_WAVE), __shfl_xor(bi, d, TPC_WAVE));
        }
        if (i < T && sub == 0) {
            A.next[i] = bo;
            A.chi2[i] = bo >= 0 ? (float)co : 0.f;
            A.prev[i] = bi;
        }
    }
}

__global__ void __launch_bounds__(TPC_BLOCK) mg_best(MgArgs A) {
    __shared__ int cand[MG_LANE_CHUNK][TPC_BLOCK];
    const int T = mg_count(A);
    if (T <= MG_MANY) best_partners<16>(A, T, cand);
    else best_partners<4>(A, T, cand);
}

__global__ void __launch_bounds__(TPC_BLOCK) mg_link_next(MgArgs A) {
    const int T = mg_count(A);
    for (int a = blockIdx.x * TPC_BLOCK + threadIdx.x; a < T; a += gridDim.x * TPC_BLOCK) {
        const int b = A.next[a];
        const bool linked = b >= 0 && b < T && A.prev[b] == a;
        if (!linked) {
            A.next[a] = -1;
            A.chi2[a] = 0.f;
        }
        if (A.mpar) {
            float *mp = A.mpar + (size_t)a * 5, *mc = A.mcov + (size_t)a * 15;
            for (int q = 0; q < 5; ++q) mp[q] = 0.f;
            for (int q = 0; q < 15; ++q) mc[q] = 0.f;
            if (linked) {
                const double da = turn_angle(A.sector[a], A.sector[b], A.n_sectors);
                pair_fuse(A, a, b, cos(da), sin(da), INFINITY, mp, mc);
            }
        }
    }
}

__global__ void __launch_bounds__(TPC_BLOCK) mg_link_prev(MgArgs A) {
    const int T = mg_count(A);
    for (int b = blockIdx.x * TPC_BLOCK + threadIdx.x; b < T; b += gridDim.x * TPC_BLOCK) {
        const int a = A.prev[b];
        if (!(a >= 0 && a < T && A.next[a] == b)) A.prev[b] = -1;
    }
}

// ---------------------------------------------------------------------------
// Legs of loopers.  A returning leg is fitted as a track running outwards
// along the same circle in the other sense: the same centre, curvature and
// tan(lambda) of opposite signs.  m = (X_c, Y_c, kappa, t) per segment in
// global coordinates, compared as m_A - D m_B, D = diag(1, 1, -1, -1), with
// chi2 = d^T (J_A C_A J_A^T + D J_B C_B J_B^T D)^-1 d (4 dof).  Candidates:
// fitted segments of one frame and side in any sectors, circle radius below
// 250 cm.

#define LEG_MAX_RADIUS 250.0

struct Circle {
    double m[4];
    double s00, s10, s11, s20, s21, s22, s30, s31, s32, s33;   // J C J^T, lower triangle
};

// The circle of segment i (false if too large or degenerate); ang: cosine
// and sine of the 18 sector angles of a side.
__device__ __forceinline__ bool leg_circle(const MgArgs &A, int i, const double (*ang)[2], Circle &o) {
    const float *p = A.par + (size_t)i * 5, *co = A.cov + (size_t)i * 15;
    const double y = (double)p[0], s = (double)p[2], t = (double)p[3], w = (double)p[4];
    const double k = A.kbz, kap = k * w;
    if (!(fabs(s) < 1.0) || !(fabs(kap) * LEG_MAX_RADIUS > 1.0)) return false;
    const int s18 = A.sector[i] % 18;
    const double *cs = ang[s18 < 0 ? s18 + 18 : s18];          // (a seed list may hold anything)
    double ic;
    const double c = sqrt_pos(fma(-s, s, 1.0), &ic), ca = cs[0], sa = cs[1];
    const double ik = copysign(recip_pos(fabs(kap)), kap);
    const double x = (double)A.x[i];
    const double xc = x - s * ik, yc = y + c * ik;
    o.m[0] = xc * ca - yc * sa;
    o.m[1] = xc * sa + yc * ca;
    o.m[2] = kap;
    o.m[3] = t;
    const double dxc[5] = {0.0, 0.0, -ik, 0.0, s * k * ik * ik};
    const double dyc[5] = {1.0, 0.0, -s * ic * ik, 0.0, -c * k * ik * ik};
    double J[4][5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        J[0][j] = dxc[j] * ca - dyc[j] * sa;
        J[1][j] = dxc[j] * sa + dyc[j] * ca;
        J[2][j] = j == 4 ? k : 0.0;
        J[3][j] = j == 3 ? 1.0 : 0.0;
    }
    double C[5][5];
#pragma unroll
    for (int a = 0, q = 0; a < 5; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b, ++q) C[a][b] = C[b][a] = (double)co[q];
    double JC[4][5];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 5; ++q) acc += J[a][q] * C[q][b];
            JC[a][b] = acc;
        }
    double S[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) {
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 5; ++q) acc += JC[a][q] * J[b][q];
            S[a][b] = acc;
        }
    o.s00 = S[0][0];
    o.s10 = S[1][0]; o.s11 = S[1][1];
    o.s20 = S[2][0]; o.s21 = S[2][1]; o.s22 = S[2][2];
    o.s30 = S[3][0]; o.s31 = S[3][1]; o.s32 = S[3][2]; o.s33 = S[3][3];
    return true;
}

// chi2 of legs a and b (m_a - D m_b against S_a + D S_b D, D = diag(1, 1,
// -1, -1): the (centre, kappa/t) cross terms of S_b change sign), by a 4x4
// L D L^T; INFINITY if the sum is not positive definite.
__device__ __forceinline__ double leg_chi2(const Circle &a, const Circle &b) {
    const double d0 = a.m[0] - b.m[0], d1 = a.m[1] - b.m[1], d2 = a.m[2] + b.m[2], d3 = a.m[3] + b.m[3];
    const double S00 = a.s00 + b.s00, S10 = a.s10 + b.s10, S11 = a.s11 + b.s11;
    const double S20 = a.s20 - b.s20, S21 = a.s21 - b.s21, S22 = a.s22 + b.s22;
    const double S30 = a.s30 - b.s30, S31 = a.s31 - b.s31, S32 = a.s32 + b.s32, S33 = a.s33 + b.s33;
    const double i0 = recip_pos(S00);
    const double l10 = S10 * i0, l20 = S20 * i0, l30 = S30 * i0;
    const double e1 = S11 - l10 * S10, i1 = recip_pos(e1);
    const double t21 = S21 - l20 * S10, t31 = S31 - l30 * S10, l21 = t21 * i1, l31 = t31 * i1;
    const double e2 = S22 - l20 * S20 - l21 * t21, i2 = recip_pos(e2);
    const double t32 = S32 - l30 * S20 - l31 * t21, l32 = t32 * i2;
    const double e3 = S33 - l30 * S30 - l31 * t31 - l32 * t32, i3 = recip_pos(e3);
    const double u1 = d1 - l10 * d0, u2 = d2 - l20 * d0 - l21 * u1, u3 = d3 - l30 * d0 - l31 * u1 - l32 * u2;
    const bool ok = (int)(S00 > 0.0) & (int)(e1 > 0.0) & (int)(e2 > 0.0) & (int)(e3 > 0.0);
    return ok ? d0 * d0 * i0 + u1 * u1 * i1 + u2 * u2 * i2 + u3 * u3 * i3 : INFINITY;
}

// Candidates are the segments of the segment's (frame, side): one
// contiguous seed range.  LG_SPLIT lanes of one wavefront share a segment
// and take every LG_SPLIT-th candidate, so that the chip holds enough
// wavefronts; their best candidates are reduced by shuffles at the end
// (smaller chi2, then smaller index: the serial order's choice).  The
// workgroup walks the union of its segments' ranges in tiles of TPC_BLOCK
// segments: each thread forms the circle of one tile segment into LDS, then
// the lanes test the tile from there.  Each circle is formed once per
// workgroup and tile instead of once per pair.  A lane first collects the
// tile's candidates whose (kappa, tan(lambda)) chi2 alone (exact rows of J:
// never above the full one) does not exceed the best full chi2 that any of
// the segment's lanes has found (shared after each tile; the cut before),
// with a slack far above rounding, then tests only those: the wavefront
// takes as many full tests as its longest list, not one whenever any lane
// has a candidate.
#define LG_SPLIT 8
#define LG_SEGS (TPC_BLOCK / LG_SPLIT)

struct LegTile {
    double m[4][TPC_BLOCK];
    double s[10][TPC_BLOCK];
    int ok[TPC_BLOCK];
    double ang[18][2];                           // cosine, sine of the sector angles
    uint8_t list[TPC_BLOCK / LG_SPLIT][TPC_BLOCK];   // each lane's candidates of the tile
};

__global__ void __launch_bounds__(TPC_BLOCK) lg_best(MgArgs A) {
    __shared__ LegTile tile;
    __shared__ int span[2];
    const int T = mg_count(A);
    const int sub = threadIdx.x % LG_SPLIT;
    if (threadIdx.x < 18) {
        const double al = sector_angle(threadIdx.x, A.n_sectors);
        tile.ang[threadIdx.x][0] = cos(al);
        tile.ang[threadIdx.x][1] = sin(al);
    }
    __syncthreads();
    // whole workgroups step together: every lane reaches the barriers and
    // the shuffles
    for (int base = blockIdx.x * LG_SEGS; base < T; base += gridDim.x * LG_SEGS) {
        const int i = base + threadIdx.x / LG_SPLIT;
        int best = -1;
        double bchi = INFINITY, lim = A.cut;          // this lane's best; the segment's, at most the cut
        Circle ci;
        const bool live = i < T && A.status[i] == 0 && A.n_sectors == 36 && leg_circle(A, i, tile.ang, ci);
        int j0 = T, j1 = 0;
        if (live) {
            const int64_t key = (int64_t)A.frame[i] * A.n_sectors + (A.sector[i] / 18) * 18;
            j0 = mg_lower(A, T, key);
            j1 = mg_lower(A, T, key + 18);
        }
        if (threadIdx.x == 0) {
            span[0] = T;
            span[1] = 0;
        }
        __syncthreads();
        if (live && sub == 0) {
            atomicMin(&span[0], j0);
            atomicMax(&span[1], j1);
        }
        __syncthreads();
        const int u0 = span[0], u1 = span[1];
        for (int c0 = u0; c0 < u1; c0 += TPC_BLOCK) {
            const int c = c0 + threadIdx.x;
            Circle cc;
            const bool okc = c < u1 && A.status[c] == 0 && leg_circle(A, c, tile.ang, cc);
            tile.ok[threadIdx.x] = okc;
            if (okc) {
#pragma unroll
                for (int q = 0; q < 4; ++q) tile.m[q][threadIdx.x] = cc.m[q];
                tile.s[0][threadIdx.x] = cc.s00; tile.s[1][threadIdx.x] = cc.s10; tile.s[2][threadIdx.x] = cc.s11;
                tile.s[3][threadIdx.x] = cc.s20; tile.s[4][threadIdx.x] = cc.s21; tile.s[5][threadIdx.x] = cc.s22;
                tile.s[6][threadIdx.x] = cc.s30; tile.s[7][threadIdx.x] = cc.s31; tile.s[8][threadIdx.x] = cc.s32;
                tile.s[9][threadIdx.x] = cc.s33;
            }
            __syncthreads();
            const int n = u1 - c0 < TPC_BLOCK ? u1 - c0 : TPC_BLOCK;
            if (live) {
                const int q0 = j0 > c0 ? j0 - c0 : 0;
                const int q1 = j1 - c0 < n ? j1 - c0 : n;
                // this lane's candidates: q = sub (mod LG_SPLIT) in [q0, q1)
                const double bound = lim * TPC_MG_SLACK;
                int cnt = 0;
#pragma unroll 4
                for (int q = q0 + ((sub - q0 % LG_SPLIT + LG_SPLIT) % LG_SPLIT); q < q1; q += LG_SPLIT) {
                    const double dk = ci.m[2] + tile.m[2][q], dt = ci.m[3] + tile.m[3][q];
                    const double S22 = ci.s22 + tile.s[5][q], S32 = ci.s32 + tile.s[8][q], S33 = ci.s33 + tile.s[9][q];
                    const double det = S22 * S33 - S32 * S32;
                    const bool far = S33 * dk * dk - 2.0 * S32 * dk * dt + S22 * dt * dt > bound * det;
                    if ((int)(tile.ok[q] != 0) & (int)(c0 + q != i) & (int)!((int)(det > 0.0) & (int)far))
                        tile.list[cnt++][threadIdx.x] = (uint8_t)q;
                }
                for (int k = 0; k < cnt; ++k) {
                    const int q = tile.list[k][threadIdx.x];
                    Circle cj;
                    cj.m[0] = tile.m[0][q]; cj.m[1] = tile.m[1][q]; cj.m[2] = tile.m[2][q]; cj.m[3] = tile.m[3][q];
                    cj.s00 = tile.s[0][q]; cj.s10 = tile.s[1][q]; cj.s11 = tile.s[2][q]; cj.s20 = tile.s[3][q];
                    cj.s21 = tile.s[4][q]; cj.s22 = tile.s[5][q]; cj.s30 = tile.s[6][q]; cj.s31 = tile.s[7][q];
                    cj.s32 = tile.s[8][q]; cj.s33 = tile.s[9][q];
                    const double chi = leg_chi2(ci, cj);
                    if (chi > 0.0 && chi <= A.cut && chi < bchi) {   // j ascends: ties keep the smaller
                        bchi = chi;
                        best = c0 + q;
                    }
                }
            }
            lim = fmin(lim, bchi);
#pragma unroll
            for (int d = 1; d < LG_SPLIT; d <<= 1) lim = fmin(lim, __shfl_xor(lim, d, TPC_WAVE));
            __syncthreads();
        }
#pragma unroll
        for (int d = 1; d < LG_SPLIT; d <<= 1) {
            best_merge(bchi, best, __shfl_xor(bchi, d, TPC_WAVE), __shfl_xor(best, d, TPC_WAVE));
        }
        if (i < T && sub == 0) {
            A.leg[i] = best;
            A.leg_chi2[i] = best >= 0 ? (float)bchi : 0.f;
        }
    }
}

// Mutual best, in place: a segment whose best does not choose it back is
// cleared; the value another thread reads can only change from "not me" to
// -1, and a mutual pair is never cleared.
__global__ void __launch_bounds__(TPC_BLOCK) lg_link(MgArgs A) {
    const int T = mg_count(A);
    for (int a = blockIdx.x * TPC_BLOCK + threadIdx.x; a < T; a += gridDim.x * TPC_BLOCK) {
        const int b = A.leg[a];
        if (!(b >= 0 && b < T && A.leg[b] == a)) {
            A.leg[a] = -1;
            A.leg_chi2[a] = 0.f;
        }
    }
}

}  // namespace

hipError_t launch_merge(const tpc_context *ctx, const tpc_seeds *sd, const tpc_tracks *tr, double cut,
                        int32_t *next, int32_t *prev, float *chi2, float *mpar, float *mcov, int32_t *leg,
                        float *leg_chi2, hipStream_t st) {
    MgArgs A;
    A.x = tr->x;
    A.par = tr->par;
    A.cov = tr->cov;
    A.status = tr->status;
    A.frame = sd->frame;
    A.sector = sd->sector;
    A.n_seeds = sd->n_seeds;
    A.cap = sd->cap_seeds;
    A.n_sectors = ctx->cfg.n_sectors;
    A.kbz = -0.00299792458 * (double)ctx->cfg.bz;
    A.cut = cut;
    A.max_sin = ctx->cfg.max_sin;
    A.next = next;
    A.prev = prev;
    A.chi2 = chi2;
    A.mpar = mpar;
    A.mcov = mcov;
    A.leg = leg;
    A.leg_chi2 = leg_chi2;
    int g = (sd->cap_seeds + TPC_BLOCK - 1) / TPC_BLOCK;
    g = g < 1 ? 1 : (g > 4096 ? 4096 : g);
    int gm = (int)(((int64_t)sd->cap_seeds * 16 + TPC_BLOCK - 1) / TPC_BLOCK);
    gm = gm < 1 ? 1 : (gm > 8192 ? 8192 : gm);
    hipLaunchKernelGGL(mg_best, dim3(gm), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(mg_link_next, dim3(g), dim3(TPC_BLOCK), 0, st, A);
    hipLaunchKernelGGL(mg_link_prev, dim3(g), dim3(TPC_BLOCK), 0, st, A);
    if (leg) {
        int gl = (int)(((int64_t)sd->cap_seeds * LG_SPLIT + TPC_BLOCK - 1) / TPC_BLOCK);
        gl = gl < 1 ? 1 : (gl > 8192 ? 8192 : gl);
        hipLaunchKernelGGL(lg_best, dim3(gl), dim3(TPC_BLOCK), 0, st, A);
        hipLaunchKernelGGL(lg_link, dim3(g), dim3(TPC_BLOCK), 0, st, A);
    }
    return hipGetLastError();
}
