// cvo_reduce.hip -- per-pair reduction of the pair-pass moments and the
// FP64 ascent step (Problem 1 solved by gradient ascent on SE(3), with the
// lengthscale annealed as in Sec. IV).
//
// From the per-query moments W_j = sum_i w_ij, D_j = sum_i w_ij d_ij and
// S_j = sum_i w_ij d_ij d_ij^T (d = x - z'), held as partial moments per
// piece of the query's candidate list, one O(M) pass gives
//   F        = sum_j W_j                                       (eq. (7))
//   omega    = ell^-2 sum_j z'_j x D_j,  v = ell^-2 sum_j D_j   (gradient)
//   H        = sum_j H_j, the 6x6 matrix with xi^T H xi equal to the second
//              derivative of F(Exp(tau xi) T) at tau = 0 for any xi:
//              with A = S/ell^4 - W I/ell^2 and Z = [z']_x,
//              H_ww = -Z A Z + (D z'^T + z' D^T)/(2 ell^2) - (D.z') I/ell^2
//              H_wv =  Z A - [D]_x /(2 ell^2),   H_vv = A
//   tr S / ell^3 = dF/dell (cutoff held fixed), |P| = sum n_j,
//   r_max = max_j |z'_j|,
// and, for the adaptive lengthscale (Sec. VI), over the targets with W_j > 0:
//   sum log W_j, sum r_j with r_j = tr S_j / W_j (the target's weighted mean
//   squared residual), and their number |Z+|.
// The curvature along a direction d is d^T H d.  Each block reduces a fixed
// slice of the queries in a fixed tree order; a second launch, one workgroup
// per pair, combines the block partials in a fixed order and, in step mode,
// takes the ascent step -- so results are bitwise reproducible.
#include "cvo_launch.hpp"

#include <algorithm>

namespace cvo {

// accumulator slots (R_LOGW .. R_ZP: the lengthscale objective's sums over
// the targets with W_j > 0, reduced only when asked for; 43 .. 47 unused)
enum {
    R_F = 0, R_OM = 1, R_V = 4, R_HWW = 7, R_HWV = 13, R_HVV = 22, R_TRS = 28, R_N = 29, R_RMAX = 30,
    R_ZS = 31, R_ZZ = 34, R_LOGW = 40, R_RSUM = 41, R_ZP = 42, R_END = 48
};

// Solve G d = g for the kinetic-energy metric of the moving cloud,
// G = [[(tr S + mu) I - S, C], [C^T, I]] with c = mean z', C = [c]_x,
// S = mean z' z'^T and mu = 1e-6 (tr S + 1e-12).  The lower right block is the
// identity, so eliminating v leaves a 3x3 system with M = (tr K + mu) I - K in
// the covariance K = S - c c^T, solved by cofactors: one division on the
// serial chain where a 6x6 Cholesky has six square roots and six divisions.
// False if G (equivalently M) is not positive definite.
__device__ __forceinline__ bool metric_solve(const double *tot, double im, const double g[6], double d[6])
{
    const double c0 = tot[R_ZS] * im, c1 = tot[R_ZS + 1] * im, c2 = tot[R_ZS + 2] * im;
    const double s00 = tot[R_ZZ + 0] * im, s11 = tot[R_ZZ + 3] * im, s22 = tot[R_ZZ + 5] * im;
    const double mu = 1e-6 * (s00 + s11 + s22 + 1e-12);
    const double k00 = s00 - c0 * c0, k11 = s11 - c1 * c1, k22 = s22 - c2 * c2;
    const double m00 = k11 + k22 + mu, m11 = k00 + k22 + mu, m22 = k00 + k11 + mu;
    const double m01 = c0 * c1 - tot[R_ZZ + 1] * im;
    const double m02 = c0 * c2 - tot[R_ZZ + 2] * im;
    const double m12 = c1 * c2 - tot[R_ZZ + 4] * im;
    const double a00 = m11 * m22 - m12 * m12, a01 = m02 * m12 - m01 * m22, a02 = m01 * m12 - m02 * m11;
    const double a11 = m00 * m22 - m02 * m02, a12 = m01 * m02 - m00 * m12, a22 = m00 * m11 - m01 * m01;
    const double det = m00 * a00 + m01 * a01 + m02 * a02;
    if (!(m00 > 0.0 && a22 > 0.0 && det > 0.0)) return false;
    // r = g_w - c x g_v;  d_w = M^-1 r;  d_v = g_v + c x d_w
    const double r0 = g[0] - (c1 * g[5] - c2 * g[4]);
    const double r1 = g[1] - (c2 * g[3] - c0 * g[5]);
    const double r2 = g[2] - (c0 * g[4] - c1 * g[3]);
    const double id = 1.0 / det;
    d[0] = (a00 * r0 + a01 * r1 + a02 * r2) * id;
    d[1] = (a01 * r0 + a11 * r1 + a12 * r2) * id;
    d[2] = (a02 * r0 + a12 * r1 + a22 * r2) * id;
    d[3] = g[3] + (c1 * d[2] - c2 * d[1]);
    d[4] = g[4] + (c2 * d[0] - c0 * d[2]);
    d[5] = g[5] + (c0 * d[1] - c1 * d[0]);
    return true;
}

// xi^T H xi for the reduced 6x6 curvature matrix
__device__ __forceinline__ double quad_form(const double *tot, const double xi[6])
{
    const double *w = tot + R_HWW, *x = tot + R_HWV, *v = tot + R_HVV;
    const double a = xi[0], b = xi[1], c = xi[2], p = xi[3], q = xi[4], r = xi[5];
    // rows of H_ww w + 2 H_wv v and of H_vv v
    const double h0 = w[0] * a + w[1] * b + w[2] * c + 2.0 * (x[0] * p + x[1] * q + x[2] * r);
    const double h1 = w[1] * a + w[3] * b + w[4] * c + 2.0 * (x[3] * p + x[4] * q + x[5] * r);
    const double h2 = w[2] * a + w[4] * b + w[5] * c + 2.0 * (x[6] * p + x[7] * q + x[8] * r);
    const double h3 = v[0] * p + v[1] * q + v[2] * r;
    const double h4 = v[1] * p + v[3] * q + v[4] * r;
    const double h5 = v[2] * p + v[4] * q + v[5] * r;
    return (a * h0 + b * h1 + c * h2) + (p * h3 + q * h4 + r * h5);
}

// SE(3) exponential of xi = (omega, v): R = I + a W + b W^2, V = I + b W + c W^2,
// p = V v with a = sin th / th, b = (1 - cos th) / th^2, c = (th - sin th) / th^3,
// th = |omega|; below th = 1e-2 the three coefficients are their Taylor
// series through th^6, above it b is written 2 sin^2(th/2) / th^2.
__device__ void exp_se3(const double xi[6], double E[12])
{
    const double w0 = xi[0], w1 = xi[1], w2 = xi[2];
    const double th2 = w0 * w0 + w1 * w1 + w2 * w2;
    double ca, cb, cc;
    if (th2 < 1e-4) {
        const double th4 = th2 * th2, th6 = th4 * th2;
        // (reciprocal factorials as constants: multiplications, not divisions)
        ca = 1.0 - th2 * (1.0 / 6.0) + th4 * (1.0 / 120.0) - th6 * (1.0 / 5040.0);
        cb = 0.5 - th2 * (1.0 / 24.0) + th4 * (1.0 / 720.0) - th6 * (1.0 / 40320.0);
        cc = 1.0 / 6.0 - th2 * (1.0 / 120.0) + th4 * (1.0 / 5040.0) - th6 * (1.0 / 362880.0);
    } else {
        const double th = sqrt(th2);
        const double sh = sin(0.5 * th);
        ca = sin(th) / th;
        cb = 2.0 * sh * sh / th2;
        cc = (th - sin(th)) / (th2 * th);
    }
    const double Wm[3][3] = {{0.0, -w2, w1}, {w2, 0.0, -w0}, {-w1, w0, 0.0}};
    double W2[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) W2[r][k] = Wm[r][0] * Wm[0][k] + Wm[r][1] * Wm[1][k] + Wm[r][2] * Wm[2][k];
    double V[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double I = (r == k) ? 1.0 : 0.0;
            E[4 * r + k] = I + ca * Wm[r][k] + cb * W2[r][k];
            V[r][k] = I + cb * Wm[r][k] + cc * W2[r][k];
        }
#pragma unroll
    for (int r = 0; r < 3; ++r) E[4 * r + 3] = V[r][0] * xi[3] + V[r][1] * xi[4] + V[r][2] * xi[5];
}

// The gradient of the reduced sums.
__device__ __forceinline__ void gradient(const double *tot, double il2, double g[6])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        g[k] = tot[R_OM + k] * il2;
        g[3 + k] = tot[R_V + k] * il2;
    }
}

// Publish an evaluation of one pair.
__device__ void publish_evaluation(PairState *st, PairState *host, const AlignConst &ac, const double *tot)
{
    const double ell = st->ell;
    const double il1 = 1.0 / ell;
    const double il2 = il1 * il1;
    double g[6];
    gradient(tot, il2, g);
    const double F = tot[R_F];
    const double ind = (ac.sqrt_nm > 0.0) ? F / ac.sqrt_nm : 0.0;
    const double curv = quad_form(tot, g);
    const double dl = tot[R_TRS] * il2 * il1;
    // lengthscale objective J = sum log W_j - 3 |Z+| log ell (all zero
    // unless its sums were reduced)
    const double mp = tot[R_ZP];
    const double J = mp > 0.0 ? tot[R_LOGW] - 3.0 * mp * log(ell) : 0.0;
    const double dJ = mp > 0.0 ? tot[R_RSUM] * il2 * il1 - 3.0 * mp * il1 : 0.0;
    const double ml = mp > 0.0 ? sqrt(tot[R_RSUM] / (3.0 * mp)) : 0.0;
    auto put = [&](PairState *o) {
        o->F = F;
        o->i_theta = ind;
        o->curv = curv;
        o->r_max = tot[R_RMAX];
        o->dF_dell = dl;
        o->n_pairs = tot[R_N];
#pragma unroll
        for (int k = 0; k < 6; ++k) o->grad[k] = g[k];
        o->J = J;
        o->dJ_dell = dJ;
        o->ell_ml = ml;
        o->zplus = mp;
    };
    put(st);
    if (host) put(host);  // (read after the stream has been waited for)
}

// What an ascent step reads of the pair's state.
struct StepIn {
    double T[12], ell, i_prev, total_pairs, rc_build;
    long long it;
    int cls_built;
};

// One ascent step of one pair (same decision sequence as the definition it
// follows): reads s, writes the fields of *st that later iterations and the
// host read, and returns 1 if the pair is done, 2 if it pauses, else 0.  One thread runs it, and its time is the number of instructions
// on that thread, so it computes nothing else: no evaluation fields, no
// inverse pose (only the backward uses one).
__device__ __forceinline__ int ascent_step(PairState *st, const StepIn &s, const AlignConst &ac, const double *tot,
                                            double *trace, long long trace_rows)
{
    const double ell = s.ell;
    const double il1 = 1.0 / ell;
    double g[6];
    gradient(tot, il1 * il1, g);
    const double F = tot[R_F];
    const double np = tot[R_N];
    const double ind = (ac.sqrt_nm > 0.0) ? F / ac.sqrt_nm : 0.0;
    st->F = F;
    st->i_theta = ind;
    st->n_pairs = np;
    const double gn2 = g[0] * g[0] + g[1] * g[1] + g[2] * g[2] + g[3] * g[3] + g[4] * g[4] + g[5] * g[5];
    if (np == 0.0) { st->status = ST_NO_OVERLAP; st->done = 1; return 1; }
    if (gn2 == 0.0) { st->status = ST_STATIONARY; st->done = 1; return 1; }
    // direction: the Riemannian gradient G^-1 g
    double d[6];
    if (ac.metric == 0) {
        if (!metric_solve(tot, ac.inv_m, g, d)) { st->status = ST_STATIONARY; st->done = 1; return 1; }
    } else {
#pragma unroll
        for (int k = 0; k < 6; ++k) d[k] = g[k];
    }
    const double slope = g[0] * d[0] + g[1] * d[1] + g[2] * d[2] + g[3] * d[3] + g[4] * d[4] + g[5] * d[5];
    const double curv_d = quad_form(tot, d);
    const double tauN = (curv_d < 0.0) ? slope / (-curv_d) : INFINITY;
    const double nw = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    const double nv = sqrt(d[3] * d[3] + d[4] * d[4] + d[5] * d[5]);
    const double tauC = ac.step_lambda * ell / (nw * tot[R_RMAX] + nv);
    const double tau = tauN < tauC ? tauN : tauC;
    double xi[6], E[12];
#pragma unroll
    for (int k = 0; k < 6; ++k) xi[k] = tau * d[k];
    exp_se3(xi, E);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            st->T[4 * r + k] = E[4 * r] * s.T[k] + E[4 * r + 1] * s.T[4 + k] + E[4 * r + 2] * s.T[8 + k];
        st->T[4 * r + 3] = E[4 * r] * s.T[3] + E[4 * r + 1] * s.T[7] + E[4 * r + 2] * s.T[11] + E[4 * r + 3];
    }
    const long long it = s.it;
    if (trace && it < trace_rows) {
        double *tr = trace + it * kTraceLen;
        tr[0] = (double)it;
        tr[1] = ell;
        tr[2] = F;
        tr[3] = sqrt(gn2);
        tr[4] = tau;
        tr[5] = ind;
        tr[6] = np;
        tr[7] = curv_d;
    }
    st->it = it + 1;
    st->total_pairs = s.total_pairs + np;
    double next = ell;  // lengthscale of the next iteration
    if (ac.ell_sched) {
        // replay of a given lengthscale sequence: no annealing or convergence decisions
        if (it + 1 >= ac.n_sched) {
            st->status = ST_MAX_ITER;
            st->done = 1;
            return 1;
        }
        next = ac.ell_sched[it + 1];
        st->ell = next;
    } else if (ac.ell_mode == 1 && !ac.fixed_iters) {
        // adaptive lengthscale: the objective's maximiser at this iteration's
        // (T, ell), clamped to [ell_min, ell_init] and to one factor `decay`
        const double mp = tot[R_ZP];
        const double ml = mp > 0.0 ? sqrt(tot[R_RSUM] / (3.0 * mp)) : 0.0;
        if (ml > 0.0) {
            double lo = ac.decay * ell, hi = ell / ac.decay;
            if (lo < ac.ell_min) lo = ac.ell_min;
            if (hi > ac.ell_init) hi = ac.ell_init;
            next = ml < lo ? lo : (ml > hi ? hi : ml);
        }
        const bool still = fabs(next - ell) <= ac.ind_rel_tol * ell;
        st->ell = next;
        if (still && tau * nw < ac.eps_rot && tau * nv < ac.eps_trans) {
            st->status = ST_CONVERGED;
            st->done = 1;
            return 1;
        }
    } else if (!ac.fixed_iters) {
        const double ip = s.i_prev;
        if (isfinite(ip) && fabs(ind - ip) <= ac.ind_rel_tol * fabs(ind) && ell > ac.ell_min) {
            const double e2 = ac.decay * ell;
            next = e2 > ac.ell_min ? e2 : ac.ell_min;
            st->ell = next;
            st->i_prev = NAN;
        } else {
            st->i_prev = ind;
        }
        if (next == ac.ell_min && tau * nw < ac.eps_rot && tau * nv < ac.eps_trans) {
            st->status = ST_CONVERGED;
            st->done = 1;
            return 1;
        }
    }
    if (it + 1 >= ac.max_iter) {
        st->status = ST_MAX_ITER;
        st->done = 1;
        return 1;
    }
    // the views no longer fit: the cutoff shrank past the rebuild ratio, or
    // the pair density fell to a lower class.  Decided from the iterates
    // alone, so where views change does not depend on how many iterations
    // are enqueued between host checks.
    // (An adaptive lengthscale may also grow: rebuild once the cutoff has
    // grown by the same ratio.)
    const bool cut = isfinite(ac.kappa);
    if ((cut && ac.kappa * next < ac.rebuild_ratio * s.rc_build) ||
        (cut && ac.rebuild_ratio < 1.0 && ac.kappa * next * ac.rebuild_ratio > s.rc_build) ||
        (ac.adaptive && s.cls_built >= 0 && density_class(np * ac.inv_m, ac.cls_t) < s.cls_built)) {
        st->pause = 1;
        return 2;
    }
    return 0;
}

static_assert(kRedThreads == 256 && R_END == 48 && R_END <= kRedVals, "reduction layout");

// ONE: every thread has at most one query (nblk * kRedThreads covers the
// largest cloud), so there is no loop over queries around the 48 sums.
template <bool ONE>
__global__ __launch_bounds__(kRedThreads) void reduce_kernel(const ReduceArgs a)
{
    const int b = blockIdx.y;
    const PairState *st = a.state + b;
    // the skip flags, the pose and the cloud range are loaded together (one
    // round trip) before the skip test
    const ClusterDesc cd = a.cdesc[b];
    double T[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) T[k] = st->T[k];
    const double ell = st->ell;
    if (st->done | st->pause) return;
    const double ascale = 1.4426950408889634 / (2.0 * ell * ell);
    const double isc = 1.0 / sqrt(ascale), ia = 1.0 / ascale;
    const double il2 = 1.0 / (ell * ell), il4 = il2 * il2;

    // every accumulator index below is a compile-time constant, so the 48
    // values stay in registers
    double acc[R_END];
#pragma unroll
    for (int k = 0; k < R_END; ++k) acc[k] = 0.0;
    const long long end = (long long)cd.pt_base + cd.n;
    auto add_query = [&](long long j) {
        const float4 zq = a.qpts[j];
        const int4 qm = a.map.qmap[j];  // (t, cluster size, pieces, first slot)
        const double z[3] = {T[0] * zq.x + T[1] * zq.y + T[2] * zq.z + T[3],
                             T[4] * zq.x + T[5] * zq.y + T[6] * zq.z + T[7],
                             T[8] * zq.x + T[9] * zq.y + T[10] * zq.z + T[11]};
        acc[R_RMAX] = fmax(acc[R_RMAX], sqrt(z[0] * z[0] + z[1] * z[1] + z[2] * z[2]));
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[R_ZS + k] += z[k];
        acc[R_ZZ + 0] += z[0] * z[0];
        acc[R_ZZ + 1] += z[0] * z[1];
        acc[R_ZZ + 2] += z[0] * z[2];
        acc[R_ZZ + 3] += z[1] * z[1];
        acc[R_ZZ + 4] += z[1] * z[2];
        acc[R_ZZ + 5] += z[2] * z[2];
        // the query's partial moments of its cluster's pieces, in piece
        // order: piece k's block starts at slot f0 + k n.  A query's thread
        // waits on memory most of its time (30,000 queries are 118 blocks),
        // so the next piece is requested before this one is added, in two
        // sets of registers: 30,000 queries of about 16 pieces 19.9 -> 15.2 us,
        // 4 pieces 8.8 -> 8.0 us.  Three or four in flight gain 1 us more in the
        // first case and lose as much in sparse ones (6.0 -> 7.0 us).
        long long nj = 0;  // (all pairs of a cluster's queries: up to 64 times the references)
        double Wt = 0.0, D0 = 0.0, D1 = 0.0, D2 = 0.0;
        double S0 = 0.0, S1 = 0.0, S2 = 0.0, S3 = 0.0, S4 = 0.0, S5 = 0.0;
        const int n = qm.y;
        const double *wd = a.WD + 4LL * (qm.w - qm.x) + qm.x;
        const float *sm = a.S + 6LL * (qm.w - qm.x) + qm.x;
        const int *ct = a.cnt + qm.w;
        struct Part {
            double w, dx, dy, dz;
            float s0, s1, s2, s3, s4, s5;
            int c;
        };
        auto load = [&]() {
            return Part{wd[0], wd[n], wd[2 * n], wd[3 * n], sm[0], sm[n], sm[2 * n], sm[3 * n], sm[4 * n], sm[5 * n], ct[0]};
        };
        auto add = [&](const Part &p) {
            nj += p.c;
            Wt += p.w;
            D0 += p.dx;
            D1 += p.dy;
            D2 += p.dz;
            S0 += (double)p.s0;
            S1 += (double)p.s1;
            S2 += (double)p.s2;
            S3 += (double)p.s3;
            S4 += (double)p.s4;
            S5 += (double)p.s5;
        };
        int left = qm.z;  // pieces not yet loaded
        auto step = [&]() {
            if (--left > 0) {
                wd += 4 * n;
                sm += 6 * n;
                ct += n;
            }
        };
        if (left > 0) {
            Part p0 = load(), p1;
            for (;;) {
                step();
                p1 = load();  // (past the end: the last piece again, not added)
                __builtin_amdgcn_sched_barrier(0);
                add(p0);
                if (left <= 0) break;
                step();
                p0 = load();
                __builtin_amdgcn_sched_barrier(0);
                add(p1);
                if (left <= 0) break;
            }
        }
        acc[R_N] += (double)nj;  // (a piece's pairs are all counted at its first query)
        if (Wt == 0.0 && D0 == 0.0 && D1 == 0.0 && D2 == 0.0 && S0 == 0.0 && S1 == 0.0 && S2 == 0.0 && S3 == 0.0 &&
            S4 == 0.0 && S5 == 0.0)
            return;
        const double Dt[3] = {D0 * isc, D1 * isc, D2 * isc};
        const double S6[6] = {S0 * ia, S1 * ia, S2 * ia, S3 * ia, S4 * ia, S5 * ia};
        acc[R_F] += Wt;
        acc[R_OM + 0] += z[1] * Dt[2] - z[2] * Dt[1];
        acc[R_OM + 1] += z[2] * Dt[0] - z[0] * Dt[2];
        acc[R_OM + 2] += z[0] * Dt[1] - z[1] * Dt[0];
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[R_V + k] += Dt[k];
        const double trs = S6[0] + S6[3] + S6[5];
        acc[R_TRS] += trs;
        if (a.ellobj && Wt > 0.0) {
            acc[R_LOGW] += log(Wt);
            acc[R_RSUM] += trs / Wt;
            acc[R_ZP] += 1.0;
        }
        // A = S/ell^4 - W I/ell^2
        const double A[3][3] = {{S6[0] * il4 - Wt * il2, S6[1] * il4, S6[2] * il4},
                                {S6[1] * il4, S6[3] * il4 - Wt * il2, S6[4] * il4},
                                {S6[2] * il4, S6[4] * il4, S6[5] * il4 - Wt * il2}};
        const double Zm[3][3] = {{0.0, -z[2], z[1]}, {z[2], 0.0, -z[0]}, {-z[1], z[0], 0.0}};
        double ZA[3][3];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) ZA[r][k] = Zm[r][0] * A[0][k] + Zm[r][1] * A[1][k] + Zm[r][2] * A[2][k];
        const double dz = Dt[0] * z[0] + Dt[1] * z[1] + Dt[2] * z[2];
        // upper triangle (r, k) of the symmetric 3x3 blocks, slot q
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int r = (q < 3) ? 0 : (q < 5 ? 1 : 2);
            const int k = (q < 3) ? q : (q < 5 ? q - 2 : 2);
            const double zaz = ZA[r][0] * Zm[0][k] + ZA[r][1] * Zm[1][k] + ZA[r][2] * Zm[2][k];
            const double m3 = 0.5 * (Dt[r] * z[k] + z[r] * Dt[k]) - (r == k ? dz : 0.0);
            acc[R_HWW + q] += -zaz + m3 * il2;
            acc[R_HVV + q] += A[r][k];
        }
        const double Dx[3][3] = {{0.0, -Dt[2], Dt[1]}, {Dt[2], 0.0, -Dt[0]}, {-Dt[1], Dt[0], 0.0}};
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[R_HWV + 3 * r + k] += ZA[r][k] - 0.5 * Dx[r][k] * il2;
    };
    const long long j0 = (long long)cd.pt_base + (long long)blockIdx.x * kRedThreads + threadIdx.x;
    if (ONE) {
        if (j0 < end) add_query(j0);
    } else {
        for (long long j = j0; j < end; j += (long long)a.nblk * kRedThreads) add_query(j);
    }


    // block reduction, 24 values at a time through LDS: every thread stores
    // its 24 values; thread (value kv = t / 8, stripe s = t % 8), t < 192,
    // adds the entries s, s + 8, ... of its value, and an 8-lane shuffle tree
    // finishes.  Fixed order throughout.
    constexpr int kChunk = 24, kStripes = 8;
    __shared__ double red[kChunk][kRedThreads + 8];  // (rows 64 bytes apart in the banks)
    const int tid = threadIdx.x;
    double *part = a.partials + (long long)b * a.nblk * kRedVals + blockIdx.x;  // value-major
    {
        const int kv = tid / kStripes, sl = tid % kStripes;
#pragma unroll
        for (int c = 0; c < R_END / kChunk; ++c) {
#pragma unroll
            for (int k = 0; k < kChunk; ++k) red[k][tid] = acc[kChunk * c + k];
            __syncthreads();
            if (kv < kChunk) {
                const bool mx = (kChunk * c + kv) == R_RMAX;
                double v = red[kv][sl];
#pragma unroll
                for (int m = 1; m < kRedThreads / kStripes; ++m) {
                    const double o = red[kv][sl + kStripes * m];
                    v = mx ? fmax(v, o) : v + o;
                }
#pragma unroll
                for (int off = kStripes / 2; off > 0; off >>= 1) {
                    const double o = __shfl_xor(v, off);
                    v = mx ? fmax(v, o) : v + o;
                }
                if (sl == 0) part[(long long)(kChunk * c + kv) * a.nblk] = v;
            }
            __syncthreads();
        }
    }
}

// Second stage, one workgroup per pair: thread (kv = t / 32, stripe sl =
// t % 32) adds blocks sl, sl + 32, ... of the values kv + 8 c (value-major
// partials: a wave's loads are two runs of 32 consecutive doubles), four
// stripes' loads in flight at once; a 32-lane shuffle tree finishes, and one thread
// finishes the pair.  Fixed order throughout.  A separate launch rather than
// a last-block ticket: the kernel boundary makes the partials visible to
// every XCD without a device-scope fence in each block of the first stage.
template <bool STEP>
__global__ __launch_bounds__(kRedThreads) void reduce_finish_kernel(const ReduceArgs a)
{
    const int b = blockIdx.x;
    __shared__ double tot[R_END];
    const int tid = threadIdx.x;
    // thread 0 holds the pair's state and constants in registers from the
    // start, so their loads overlap those of the partials; a skipped pair's
    // partials are read but not used.  (Vector loads: the addresses are made
    // opaque, as this many scalar loads go out in five dependent rounds.)
    PairState *st = a.state + b;
    const AlignConst *cp = a.ac + b;
    asm volatile("" : "+v"(st), "+v"(cp));
    int skip = 1;
    StepIn s;
    AlignConst ac;
    if (tid == 0) {
        skip = st->done | st->pause;
        ac = *cp;
        if (STEP) {
#pragma unroll
            for (int k = 0; k < 12; ++k) s.T[k] = st->T[k];
            s.ell = st->ell;
            s.i_prev = st->i_prev;
            s.total_pairs = st->total_pairs;
            s.rc_build = st->rc_build;
            s.it = st->it;
            s.cls_built = st->cls_built;
        }
    }
    const int kv = tid >> 5, sl = tid & 31;
    const double *pb = a.partials + (long long)b * a.nblk * kRedVals;
    double v[R_END / 8];
#pragma unroll
    for (int c = 0; c < R_END / 8; ++c) v[c] = 0.0;
    for (int q0 = sl; q0 < a.nblk; q0 += 4 * 32) {
        double p[4][R_END / 8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = q0 + 32 * u;
#pragma unroll
            for (int c = 0; c < R_END / 8; ++c) p[u][c] = (q < a.nblk) ? pb[(long long)(8 * c + kv) * a.nblk + q] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < R_END / 8; ++c)
                v[c] = ((8 * c + kv) == R_RMAX) ? fmax(v[c], p[u][c]) : v[c] + p[u][c];
    }
#pragma unroll
    for (int c = 0; c < R_END / 8; ++c) {
        const bool mx = (8 * c + kv) == R_RMAX;
        double x = v[c];
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) {
            const double o = __shfl_xor(x, off);
            x = mx ? fmax(x, o) : x + o;
        }
        if (sl == 0) tot[8 * c + kv] = x;
    }
    __syncthreads();
    if (skip) return;  // (threads other than 0, and pairs that are done or paused)
    if (STEP) {
        const int end =
            ascent_step(st, s, ac, tot, a.trace ? a.trace + (long long)b * a.trace_rows * kTraceLen : nullptr, a.trace_rows);
        if (a.mail)
            __hip_atomic_store(&a.mail->progress, (unsigned long long)(s.it + 1) << 2 | (unsigned long long)end,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        publish_evaluation(st, a.mail ? &a.mail->state[b] : nullptr, ac, tot);
    }
}

void launch_reduce(const ReduceArgs &a, int B, hipStream_t s)
{
    if (a.one_query)
        hipLaunchKernelGGL(reduce_kernel<true>, dim3(a.nblk, B), dim3(kRedThreads), 0, s, a);
    else
        hipLaunchKernelGGL(reduce_kernel<false>, dim3(a.nblk, B), dim3(kRedThreads), 0, s, a);
    if (a.mode)
        hipLaunchKernelGGL(reduce_finish_kernel<true>, dim3(B), dim3(kRedThreads), 0, s, a);
    else
        hipLaunchKernelGGL(reduce_finish_kernel<false>, dim3(B), dim3(kRedThreads), 0, s, a);
}

// ---------------------------------------------------------------- backward
// d(gF F)/d(query point) = gF * R_P^T D / ell^2, with R_P the rotation of
// the pose that mapped queries into the reference frame (T for Z, T^-1 for
// X), and feature gradients scaled back from pre-scaled columns.
// A block takes 64 queries: a wave adds one value's partials over the pieces
// of all 64 (neighbouring queries are neighbours in memory), the sums meet in
// LDS, and the rows are written with consecutive threads on consecutive
// columns.  Bound by reading the partials: 20,011 x 17,389 points of 24
// columns, both sides: 2 x 63 us with a thread per query and value-strided
// partials, 35 us for both now.
constexpr int kBackQ = 64;  // queries per block

__global__ __launch_bounds__(256) void backward_finish(const BackwardArgs a)
{
    extern __shared__ double s_v[];  // value v of query q at v * (kBackQ + 1) + q
    const BackwardSide &sd = a.side[blockIdx.y];
    const long long p0 = (long long)blockIdx.x * kBackQ;
    if (p0 >= sd.n) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int d4 = a.lay.d4, nv = 4 + d4;
    const bool in = p0 + lane < sd.n;
    const int4 qm = in ? sd.qmap[p0 + lane] : make_int4(0, 0, 0, 0);  // (t, cluster size, pieces, first slot)
    const long long f0 = qm.w - qm.x;
    for (int v = wv; v < nv; v += 4) {
        if (v < 3 ? !sd.dxyz : v == 3 ? !sd.lsum : !sd.dfeat) continue;
        double x = 0.0;
        const double *B = a.B + f0 * nv + (long long)v * qm.y + qm.x;
        for (int k = 0; k < qm.z; ++k) x += B[(long long)k * qm.y * nv];
        s_v[v * (kBackQ + 1) + lane] = x;
    }
    __syncthreads();
    const PairState *st = a.state;
    const double *P = sd.pose_is_inverse ? st->Tinv : st->T;
    const double ell = st->ell;
    const double ascale = 1.4426950408889634 / (2.0 * ell * ell);
    const double f = a.gF / (sqrt(ascale) * ell * ell);
    if (sd.lsum && wv == 0) {
        double l = in ? s_v[3 * (kBackQ + 1) + lane] : 0.0;
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
        if (lane == 0) sd.lsum[blockIdx.x] = l;
    }
    const int nq = (int)min((long long)kBackQ, sd.n - p0);
    if (sd.dxyz && threadIdx.x < 3 * nq) {
        const int q = threadIdx.x / 3, k = threadIdx.x % 3;
        const double d0 = s_v[q], d1 = s_v[kBackQ + 1 + q], d2 = s_v[2 * (kBackQ + 1) + q];
        sd.dxyz[3LL * sd.qperm[p0 + q] + k] = (float)(f * (P[k] * d0 + P[4 + k] * d1 + P[8 + k] * d2));
    }
    if (!sd.dfeat) return;
    const double *G = s_v + 4 * (kBackQ + 1);
    for (int i = threadIdx.x; i < nq * d4; i += 256) {
        const int q = i / d4, k = i - q * d4, col = a.lay.col[k];
        if (col >= 0)
            sd.dfeat[(long long)sd.qperm[p0 + q] * a.lay.src_dim + col] =
                (float)(a.gF * G[k * (kBackQ + 1) + q] * a.lay.gscale[k]);
    }
    if (a.lay.nlin > 0 && threadIdx.x < nq) {
        // folded LIN blocks: the gradient of a tensor-product column c
        // reaches u_b[digit_b(c)] times the other blocks' factors of c
        const int q = threadIdx.x;
        const long long o = sd.qperm[p0 + q];
        const float *u = sd.src_feat + o * a.lay.src_dim;
        double gl[64];
        for (int k = 0; k < 64; ++k) gl[k] = 0.0;
        for (int k = 0; k < d4; ++k) {
            if (a.lay.col[k] != -2) continue;
            const double gk = G[k * (kBackQ + 1) + q];
            int dig[8];
            int cc = k - a.lay.sed;
            for (int b = a.lay.nlin - 1; b >= 0; --b) {
                dig[b] = cc % a.lay.lin_dim[b];
                cc /= a.lay.lin_dim[b];
            }
            for (int b = 0; b < a.lay.nlin; ++b) {
                double other = 1.0;
                for (int b2 = 0; b2 < a.lay.nlin; ++b2)
                    if (b2 != b) other *= (double)u[a.lay.lin_src[b2] + dig[b2]];
                gl[a.lay.lin_src[b] + dig[b]] += gk * other;
            }
        }
        for (int b = 0; b < a.lay.nlin; ++b)
            for (int j = 0; j < a.lay.lin_dim[b]; ++j) {
                const int col = a.lay.lin_src[b] + j;
                sd.dfeat[o * a.lay.src_dim + col] = (float)(a.gF * gl[col]);
            }
    }
}

int backward_blocks(long long n) { return (int)((n + kBackQ - 1) / kBackQ); }

void launch_backward_finish(const BackwardArgs &a, hipStream_t s)
{
    int nb = 1;
    for (int k = 0; k < a.nsides; ++k) nb = std::max(nb, backward_blocks(a.side[k].n));
    const size_t lds = sizeof(double) * (4 + a.lay.d4) * (kBackQ + 1);
    hipLaunchKernelGGL(backward_finish, dim3(nb, a.nsides), dim3(256), lds, s, a);
}

__global__ __launch_bounds__(256) void sum_doubles(const double *in, long long n, double *out)
{
    double v = 0.0;
    for (long long i = threadIdx.x; i < n; i += 256) v += in[i];
    __shared__ double sh[256];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

void launch_sum_doubles(const double *in, long long n, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(sum_doubles, dim3(1), dim3(256), 0, s, in, n, out);
}

}  // namespace cvo
