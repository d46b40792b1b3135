// cvo_pairs.hip -- the pair pass: the truncated double sum of eq. (7) and its
// per-query moments, for one or many point-cloud pairs in one launch.
//
// Work decomposition (one 64-wide wavefront per piece: every np-th chunk of
// 64 candidates of one query cluster, np set per cluster at planning time):
//   * The cluster's n <= 64 query points are transformed into the reference
//     frame once (FP64), then re-expressed relative to the transformed
//     cluster centre c' and scaled by sqrt(a), a = log2(e) / (2 ell^2), in
//     FP32.  Relative coordinates are small, so FP32 keeps ~1e-7 of the
//     cutoff radius even at 40 m from the origin.
//   * Lanes are split into SUB = 64 / n' sub-streams (n' = n rounded up to a
//     power of two); lane (q, t) pairs query t with every SUB-th candidate, so
//     all 64 lanes stay busy for clusters of any size.
//   * Candidates are the reference points in the grid cells that the ball of
//     radius r_c + rho (rho: cluster radius) reaches.  Their
//     x-runs of cells are contiguous in the sorted reference array; up
//     to 64 runs are measured at once (one per lane), prefix-summed, and
//     their points loaded 64 at a time (each position finds its run by a
//     running max over the runs' first positions; both scans use DPP, not
//     the LDS, which the other waves' walks keep busy).  Points outside the
//     ball are culled; survivors (coordinates and feature rows) are compacted
//     with a ballot into a per-wave LDS queue.
//   * When the queue holds at least kQueueFlush entries every lane walks its
//     share: FP32 squared distance, cutoff test, one exp2 for the geometric
//     kernel and every SE feature block together, the LIN dot product; W =
//     sum w and D = sum w d are summed in FP32 over the flush and then added
//     in FP64, S = sum w d d^T is summed in FP32.
//     The backward, and an inner product of LIN columns alone, take their pairs in
//     FP64 throughout.
//   * Pairs whose FP32 squared distance lies within a proven error band of
//     the cutoff are decided again with the FP64 expression that defines the
//     pair set, so |P| is exact.
//   * The sub-streams are combined with lane shuffles (fixed order, so the
//     result is bitwise reproducible) and one lane per query writes its
//     moments.
#include "cvo_device.hpp"
#include "cvo_launch.hpp"

namespace cvo {

// Wave-uniform floating values kept in scalar registers.
__device__ __forceinline__ float uniform_f(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ double uniform_d(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The largest power of two that is at most v (v > 0, normal).
__device__ __forceinline__ double pow2_below(double v)
{
    return __longlong_as_double(__double_as_longlong(v) & 0x7ff0000000000000LL);
}

// 2^-e for e >= 0 (0 from about 1,075 on; NaN stays): e = n + f with n its nearest
// integer, 2^-f by the polynomial of degree 6 with the least maximum relative
// error on |f| <= 1/2 (a weighted least-squares fit, reweighted until its error
// peaks were level): 1.9e-9, where the FP32 exponential has about 1e-7.
__device__ __forceinline__ double exp2_neg(double e)
{
    constexpr double c[7] = {1.0000000005541698,   -0.6931472057372612,   0.24022646890619745, -0.055503287769749755,
                             0.009618488958667314, -0.0013399931216049354, 0.00015345811584973305};
    const double n = rint(e), f = e - n;
    double p = c[6];
#pragma unroll
    for (int k = 5; k >= 0; --k) p = fma(p, f, c[k]);
    return ldexp(p, -(int)n);
}

// Membership of (x, z) in the pair set, decided exactly as the set is defined:
// z'_r = ((R_r0 z0 + R_r1 z1) + R_r2 z2) + t_r, d = x - z',
// s = (dx dx + dy dy) + dz dz, member iff s <= rc2; every operation is a
// separately rounded IEEE double (contraction into FMA is switched off).
// One axis per loop trip, coordinates read from memory: this path is rare, and
// its registers (or a call's) would otherwise add to those of the loop around it.
__device__ __forceinline__ bool canonical_member(const double *T, const float4 *xp, const float4 *zp, double rc2)
{
#pragma clang fp contract(off)
    const float *x = reinterpret_cast<const float *>(xp);
    const float *z = reinterpret_cast<const float *>(zp);
    double s = 0.0;
#pragma unroll 1
    for (int r = 0; r < 3; ++r) {
        double t = T[4 * r + 0] * (double)z[0];
        const double q = T[4 * r + 1] * (double)z[1];
        t = t + q;
        const double u = T[4 * r + 2] * (double)z[2];
        t = t + u;
        t = t + T[4 * r + 3];
        const double d = (double)x[r] - t;
        const double dd = d * d;
        s = (r == 0) ? dd : s + dd;
    }
    return s <= rc2;
}

template <int SED, int LIND, int MODE> struct PassTraits {
    static constexpr int D = SED + LIND;
    static constexpr int D4 = (D + 3) & ~3;
    // waves per SIMD the register budget is sized for (no spills)
    static constexpr int kMinWaves = (MODE == 0 && D4 <= 24) ? 4 : 2;
};

template <int SED, int LIND, int MODE>
__global__ __launch_bounds__(kWave * kWavesPerBlock, (PassTraits<SED, LIND, MODE>::kMinWaves))
void pair_pass_kernel(const PairPassArgs a)
{
    constexpr int D = SED + LIND;
    constexpr int D4 = (D + 3) & ~3;
    constexpr int F4 = D4 / 4;
    constexpr int VF = D4 > 0 ? D4 : 1;
    // candidate queue, one entry of E4 float4s per candidate: the scaled
    // coordinates relative to the cluster centre and the source index's bits
    // (one float4; backward: FP64, two), then the feature row
    constexpr int C4 = MODE == 0 ? 1 : 2, E4 = C4 + F4;
    // (see launch_pair_pass for the modes)
    constexpr bool kGrad = MODE == 1;
    __shared__ float4 s_q[kWavesPerBlock][kQueueCap * E4];
    __shared__ int s_row[kWavesPerBlock][kWave];

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    const float sig2 = a.sig2;
    const bool cut = isfinite(a.kappa);

    // one piece per wave; pieces are ordered heaviest first, so the largest
    // pieces are dispatched first and the light ones fill in behind them
    {
        // The prologue's loads are requested in two dependent rounds: the
        // piece record (its index clamped, so the load stays in bounds before
        // the range check), then together the pair's flags, pose, lengthscale
        // and grid.  The query row follows the exit test of finished pairs, in
        // the round of the first cell-table reads.
        const int tk = wave_uniform(blockIdx.x * kWavesPerBlock + wv);
        const int npieces = a.npieces;
        const PieceRec rec = a.recs[min(tk, npieces - 1)];
        const int4 pc = rec.pc;
        const int b = wave_uniform(rec.b);
        const PairState *st = a.state + b;
        // (forward pieces always carry pose T)
        const int inverse = MODE == 1 ? wave_uniform(rec.inverse) : 0;
        const double *P = inverse ? st->Tinv : st->T;
        double Pm[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) Pm[k] = P[k];
        const double ell = st->ell;
        const int2 cl = make_int2(rec.first, rec.n);
        const Geo g = rec.geo;
        const GridDesc gd = a.grids[b];
        __builtin_amdgcn_sched_barrier(0);  // (the exit test below must not be scheduled between these loads)
        const int skip = st->done | st->pause;

#pragma unroll
        for (int k = 0; k < 12; ++k) in_sgpr(Pm[k]);
        in_sgpr(ell);
        in_sgpr(pc.y), in_sgpr(pc.z), in_sgpr(pc.w);
        in_sgpr(cl.x), in_sgpr(cl.y);
        in_sgpr(g.x), in_sgpr(g.y), in_sgpr(g.z), in_sgpr(g.w);
        in_sgpr(gd.ox), in_sgpr(gd.oy), in_sgpr(gd.oz), in_sgpr(gd.inv_h);
        in_sgpr(gd.nx), in_sgpr(gd.ny), in_sgpr(gd.nz), in_sgpr(gd.cell_base), in_sgpr(gd.n);
        in_sgpr(a.kappa);
        in_sgpr((long long)a.qpts), in_sgpr((long long)a.qfeat);
        if (tk >= npieces || skip) return;

        // query point owned by this lane; SUB sub-streams share the candidates
        const int n = cl.y;
        const int np2 = (n <= 1) ? 1 : (1 << (32 - __clz(n - 1)));
        const int lg = __ffs(np2) - 1;
        const int t = lane & (np2 - 1);
        const int qs = lane >> lg;
        const int SUB = kWave >> lg;
        const bool active = t < n;
        const int pq = cl.x + (active ? t : 0);
        const float4 zq = a.qpts[pq];  // (reloaded on the rare exact-recheck path)
        float vf[VF];
#pragma unroll
        for (int f = 0; f < VF / 4; ++f) vf[4 * f] = vf[4 * f + 1] = vf[4 * f + 2] = vf[4 * f + 3] = 0.0f;
#pragma unroll
        for (int f = 0; f < F4; ++f) {
            const float4 v4 = reinterpret_cast<const float4 *>(a.qfeat)[(long long)pq * F4 + f];
            vf[4 * f + 0] = v4.x;
            vf[4 * f + 1] = v4.y;
            vf[4 * f + 2] = v4.z;
            vf[4 * f + 3] = v4.w;
        }

        const double ascale = 1.4426950408889634 / (2.0 * ell * ell);  // log2(e) / (2 ell^2)
        const double sc = uniform_d(sqrt(ascale));
        const double rc = a.kappa * ell;
        const double rc2 = rc * rc;
        const Neighbourhood nb = neighbourhood(Pm, g, rc, cut, gd);
        // Coordinates are taken relative to the transformed centre rounded to
        // a grid of at most 1/256 of the cutoff (a power of two): the FP32
        // offsets of the reference points then stay what they are while the
        // pose moves by less than that, instead of being rounded anew each
        // iteration, and with the queries' rounding taken off D at the end
        // the gradient is smooth in the pose.  A cutoff of many lengthscales
        // (or one that overflows) counts as four: the pairs that weigh are
        // within that, and offsets from a centre off by more lose their digits.
        const double q0 = pow2_below(fmax(fmin(rc * (1.0 / 256.0), ell * (1.0 / 64.0)), 1e-240));
        const double q1 = 1.0 / q0;
        const double cx = uniform_d(rint(nb.cx * q1) * q0), cy = uniform_d(rint(nb.cy * q1) * q0),
                     cz = uniform_d(rint(nb.cz * q1) * q0);
        const double Rq = nb.Rm + q0;  // cull radius about that point

        // thresholds in scaled units: s' <= lo is certainly in P, s' > hi is
        // certainly out; between them the FP64 definition decides.  The band
        // is 8x the worst-case FP32 error 2^-24 (4 (1 + rho/rc) + 3) a rc^2
        // plus the rounding of the thresholds themselves.
        float hi = INFINITY, lo = INFINITY, cull2 = INFINITY;
        if (cut) {
            const double u = 5.9604644775390625e-8;
            const double G = u * (8.0 * (4.0 * (1.0 + (g.w + q0) / rc) + 3.0) + 4.0);
            const double r2s = rc2 * ascale;
            hi = uniform_f((float)(r2s * (1.0 + G)));
            lo = uniform_f((float)(r2s * (1.0 - G)));
            cull2 = uniform_f((float)(Rq * Rq * ascale));
        }
        if (!active) hi = -1.0f;  // (takes no pair)
        // (FP64 terms) the LIN columns of the query's features in FP64, where the
        // registers hold them beside the sums of all columns; else they are
        // converted for each pair
        constexpr bool kHoldV = MODE != 0 && LIND > 0 && (kGrad ? 2 * D4 : 0) + 2 * LIND + SED <= 150;
        double vl[kHoldV ? LIND : 1];
        vl[0] = 0.0;
#pragma unroll
        for (int k = 0; k < (kHoldV ? LIND : 0); ++k) vl[k] = (double)vf[SED + k];
        const double zpx = Pm[0] * zq.x + Pm[1] * zq.y + Pm[2] * zq.z + Pm[3];
        const double zpy = Pm[4] * zq.x + Pm[5] * zq.y + Pm[6] * zq.z + Pm[7];
        const double zpz = Pm[8] * zq.x + Pm[9] * zq.y + Pm[10] * zq.z + Pm[11];
        const double zsx = (zpx - cx) * sc, zsy = (zpy - cy) * sc, zsz = (zpz - cz) * sc;
        const float zrx = (float)zsx, zry = (float)zsy, zrz = (float)zsz;

        double W = 0.0, Dx = 0.0, Dy = 0.0, Dz = 0.0;
        float S00 = 0.f, S01 = 0.f, S02 = 0.f, S11 = 0.f, S12 = 0.f, S22 = 0.f;
        int cnt = 0;
        double Gf[MODE == 1 ? VF : 1];
        double Ls = 0.0;
        unsigned long long paired = 0;  // (backward) lanes that took a pair
#pragma unroll
        for (int k = 0; k < (MODE == 1 ? VF : 1); ++k) Gf[k] = 0.0;

        struct Coords {  // of a queue entry
            float4 a, b;
            __device__ explicit Coords(const float4 *e) : a(e[0]), b(e[C4 - 1]) {}
            static __device__ double join(float lo, float hi)
            {
                return __hiloint2double(__float_as_int(hi), __float_as_int(lo));
            }
            __device__ double dx() const { return join(a.x, a.y); }
            __device__ double dy() const { return join(a.z, a.w); }
            __device__ double dz() const { return join(b.x, b.y); }
        };
        // W and D are summed in FP32 over one queue flush (at most kQueueCap
        // terms per lane) and added to the FP64 accumulators after it.
        float w32 = 0.f, dx32 = 0.f, dy32 = 0.f, dz32 = 0.f;
        // One candidate entry (at `ent`; its offset d from the query and
        // squared distance s already taken) against this lane's query.  The
        // lanes that take it are held as a mask, so a comparison's result is
        // used as the wave writes it: the count is a scalar one, the rare
        // exact check a scalar branch.  (The FP32 VALU issues 90% of the time
        // in dense bands, so instructions are what counts: 38 -> 33 per pair
        // with five SE columns, with the loop below.  30,000 stereo points,
        // ell 0.95: 202 -> 188 us; 40,000 RGB-D, 0.1: 68 -> 64 us.)
        // `valid`: the lanes that have an entry (all but in the tail of a flush).
        auto members = [&](float s, const float4 *ent, unsigned long long valid) {
            unsigned long long take = __builtin_amdgcn_ballot_w64(s <= hi) & valid;
            const unsigned long long near = __builtin_amdgcn_ballot_w64(s > lo) & take;
            if (near) {
                bool in = true;
                if (__builtin_amdgcn_inverse_ballot_w64(near)) {
                    const float4 *rp = a.rpts + __float_as_int(ent[C4 - 1].w), *qp = a.qpts + pq;
                    in = canonical_member(st->T, inverse ? qp : rp, inverse ? rp : qp, rc2);
                }
                take &= __builtin_amdgcn_ballot_w64(in);
            }
            return take;
        };
        auto pair_term = [&](float dx, float dy, float dz, float s, const float4 *ent, unsigned long long valid) {
            const unsigned long long take = members(s, ent, valid);
            cnt += __popcll(take);
            if (__builtin_amdgcn_inverse_ballot_w64(take)) {
                float E = s;
                float lin = 0.0f, lin1 = 0.0f;  // even / odd LIN columns: two shorter FMA chains
#pragma unroll
                for (int f = 0; f < F4; ++f) {
                    const float4 u4 = ent[C4 + f];
                    const float uu[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int d = 4 * f + q;
                        if (d < SED) {
                            const float df = uu[q] - vf[d];
                            E = fmaf(df, df, E);
                        } else if (d < D) {
                            if ((d - SED) & 1) lin1 = fmaf(uu[q], vf[d], lin1);
                            else lin = fmaf(uu[q], vf[d], lin);
                        }
                    }
                }
                lin += lin1;
                // sigma^2 prod sigma_b^2 is applied once per query at the end
                const float wnl = __builtin_amdgcn_exp2f(-E);
                const float w = (LIND > 0) ? wnl * lin : wnl;
                w32 += w;
                const float wx = w * dx, wy = w * dy, wz = w * dz;
                dx32 += wx;
                dy32 += wy;
                dz32 += wz;
                S00 = fmaf(wx, dx, S00);
                S01 = fmaf(wx, dy, S01);
                S02 = fmaf(wx, dz, S02);
                S11 = fmaf(wy, dy, S11);
                S12 = fmaf(wy, dz, S12);
                S22 = fmaf(wz, dz, S22);
            }
        };
        // The pair of modes 1 and 2 is FP64 but for the sum over the SE columns: the
        // distance, the LIN dot, the weight and all sums.  With signed LIN weights
        // the terms of sum w s' cancel 10^3 to 10^4 times, and dF/dell keeps
        // what their rounding leaves: 10,000 points of 32 LIN columns, twelve
        // draws, relative error against 64 bits 3.0e-7 (geometric mean) and
        // 4.4e-6 (largest) with FP32 terms, 1.8e-8 and 4.8e-8 (its FP32 result's
        // own rounding) with these; dX 1.3e-7 -> 2.5e-8.  FP64 FMAs issue at the
        // rate of FP32's, so what it takes is conversions and the longer
        // exponential (both sides' pass): those 10,000 points 100 -> 137 us,
        // 20,011 x 17,389 of 5 SE + 19 LIN 197 -> 277 us, 40,000 RGB-D of 5 SE
        // 132 -> 204 us.
        auto exact_term = [&](const Coords &c, const float4 *ent, unsigned long long valid) {
            const double dx = c.dx() - zsx, dy = c.dy() - zsy, dz = c.dz() - zsz;
            const double s = fma(dz, dz, fma(dy, dy, dx * dx));
            const unsigned long long take = members((float)s, ent, valid);
            if (kGrad) paired |= take;
            else cnt += __popcll(take);
            if (__builtin_amdgcn_inverse_ballot_w64(take)) {
                float se = 0.0f, rest = 0.0f;
                double lin = 0.0;
#pragma unroll
                for (int f = 0; f < F4; ++f) {
                    const float4 u4 = ent[C4 + f];
                    const float uu[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int d = 4 * f + q;
                        if (d < SED) {
                            const float df = uu[q] - vf[d];
                            se = fmaf(df, df, se);
                        } else if (d < D) {
                            if (kHoldV) {
                                lin = fma((double)uu[q], vl[kHoldV ? d - SED : 0], lin);
                            } else {
                                const float pr = uu[q] * vf[d];
                                lin += (double)pr;
                                rest += fmaf(uu[q], vf[d], -pr);
                            }
                        }
                    }
                }
                double E = fmin(s, 2048.0);  // (2^-2048 is 0)
                if (SED > 0) E += (double)(se > 2048.0f ? 2048.0f : se);  // (NaN stays)
                const double wn = exp2_neg(E);
                const double w = (LIND > 0) ? wn * (kHoldV ? lin : lin + (double)rest) : wn;
                W += w;
                if (!kGrad) return;
                Dx = fma(w, dx, Dx);
                Dy = fma(w, dy, Dy);
                Dz = fma(w, dz, Dz);
                Ls = fma(w, s, Ls);
                // SE columns sum w u here and take v W off at the end: sum w (u - v).
                // A wide row is read and converted again, not held over the
                // exponential (20 columns more in registers spill).
                const float4 *row = ent + C4;
                if (LIND > 0 && D4 > 28) asm volatile("" : "+v"(row));
#pragma unroll
                for (int f = 0; f < F4; ++f) {
                    const float4 u4 = row[f];
                    const float uu[4] = {u4.x, u4.y, u4.z, u4.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int d = 4 * f + q;
                        if (MODE == 1 && d < D) Gf[d] = fma(d < SED ? w : wn, (double)uu[q], Gf[d]);
                    }
                }
            }
        };
        // Lane (q, t) walks entries q, q + SUB, ...: first the rows of SUB
        // entries that every sub-stream has, two per trip of a wave-uniform
        // loop (the next entry's coordinates read while this one is used, in
        // registers that take turns), then what is left, row by row.
        auto process = [&](int qn_) {
            w32 = 0.f, dx32 = 0.f, dy32 = 0.f, dz32 = 0.f;
            const int qn = wave_uniform(qn_);
            const int nfull = wave_uniform(qn >> (6 - lg));  // qn / SUB
            const float4 *ent = &s_q[wv][qs * E4];
            const int step = SUB * E4;
            auto one = [&](const Coords &c, const float4 *at, unsigned long long in) {
                if (MODE != 0) return exact_term(c, at, in);
                const float dx = c.a.x - zrx, dy = c.a.y - zry, dz = c.a.z - zrz;
                const float s = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                pair_term(dx, dy, dz, s, at, in);
            };
            // (the widest rows of the backward: one copy of the pair's code, as
            // three are not unrolled any more and put their sums in memory)
            constexpr bool kTwo = MODE == 0 || D4 <= 40;
            Coords e0(ent);
            for (int it = 0; kTwo && it < nfull - 1; it += 2) {
                const float4 *odd = ent + step;
                const Coords e1(odd);
                one(e0, ent, ~0ULL);
                ent = odd + ((it + 3 < nfull) ? step : 0);  // (the last pair re-reads its second row)
                e0 = Coords(ent);
                one(e1, odd, ~0ULL);
            }
            for (int k0 = kTwo ? wave_uniform((nfull & ~1) << (6 - lg)) : 0; k0 < qn; k0 += SUB) {
                const int kt = qs + k0;
                const bool in = kt < qn;
                const float4 *tl = &s_q[wv][(in ? kt : 0) * E4];
                one(Coords(tl), tl, __builtin_amdgcn_ballot_w64(in));
            }
            if (MODE == 0) {
                W += (double)w32;
                Dx += (double)dx32;
                Dy += (double)dy32;
                Dz += (double)dz32;
            }
        };

        // this piece takes chunks pidx, pidx + np, pidx + 2 np, ... of the
        // cluster's candidates (the neighbourhood rows concatenated; chunk k =
        // candidates [64 k, 64 k + 64)), so the np pieces of a cluster sample
        // its whole neighbourhood alike and together cover it at any pose
        const int pidx = pc.y, pstride = pc.z;
        int qn = 0;
        if (nb.any) {
            const int nyr = nb.iy1 - nb.iy0 + 1;
            const int nrows = nyr * (nb.iz1 - nb.iz0 + 1);
            const BallRows br = ball_rows(nb, gd, cut);
            int base = 0;  // candidates in earlier row batches
            // (the query's features have arrived: waited for here, not by the
            // pair loop, whose wait would take in the next chunk's points)
#pragma unroll
            for (int f = 0; f < VF; ++f) asm volatile("" : "+v"(vf[f]));
            for (int rb = 0; rb < nrows; rb += kWave) {
                const int r = rb + lane;
                int rs = 0, len = 0;
                if (r < nrows) {
                    const int iy = nb.iy0 + r % nyr, iz = nb.iz0 + r / nyr;
                    int i0, i1;
                    if (row_cells(nb, br, iy, iz, i0, i1)) {
                        const long long k0 =
                            (long long)gd.cell_base + (long long)gd.nx * (iy + (long long)gd.ny * iz);
                        rs = a.cell_start[k0 + i0];
                        len = a.cell_start[k0 + i1 + 1] - rs;
                    }
                }
                const int incl = wave_scan_add(len);
                const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
                // first chunk of this piece reaching into [base, base + total)
                int k = base / kWave;
                k += ((pidx - k) % pstride + pstride) % pstride;
                if (k * kWave < base + total) {
                    s_row[wv][lane] = 0;  // marks left by earlier chunks of this batch never exceed a later chunk's rows
                    wave_sync();
                    // The part of chunk k inside this batch of rows: its lanes, and
                    // their points on the way.  They are asked for before the
                    // queue is walked for the chunk before (40,000 RGB-D points,
                    // ell 0.1: 65 -> 63 us).  Holding the features of the chunk
                    // at hand over that request too costs 8 to 24 registers and
                    // the occupancy with them (71 us).
                    unsigned long long in_row = 0;
                    int src = 0;
                    float4 xp = make_float4(0.f, 0.f, 0.f, 0.f);
                    auto fetch = [&]() {
                        const int c0 = k * kWave - base, m = c0 + lane;
                        // the row (cell run) of each position of the chunk: every
                        // non-empty row reaching into the chunk marks its first
                        // position in it with its index, and a running max over
                        // the positions (on all lanes, before the branch below)
                        // fills in the rest
                        const int rx = incl - len;
                        if (len > 0 && rx < c0 + kWave && rx + len > c0) s_row[wv][max(rx - c0, 0)] = lane;
                        wave_sync();
                        const int row_ = wave_scan_max(s_row[wv][lane]);
                        const int first = __shfl(rs - rx, row_);  // its points start at first + (position)
                        in_row = __builtin_amdgcn_ballot_w64((unsigned)m < (unsigned)total);
                        if (__builtin_amdgcn_inverse_ballot_w64(in_row)) {
                            src = first + m;
                            xp = a.rpts[src];
                        }
                    };
                    fetch();
                    for (;;) {
                        const double xd[3] = {((double)xp.x - cx) * sc, ((double)xp.y - cy) * sc, ((double)xp.z - cz) * sc};
                        const float x0 = (float)xd[0], x1 = (float)xd[1], x2 = (float)xd[2];
                        const float r2 = fmaf(x2, x2, fmaf(x1, x1, x0 * x0));
                        const unsigned long long mask = __builtin_amdgcn_ballot_w64(r2 <= cull2) & in_row;
                        const int cur = src;
                        if (__builtin_amdgcn_inverse_ballot_w64(mask)) {
                            const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((unsigned)mask, qn));
                            float4 *q = &s_q[wv][__umul24(slot, E4)];
                            if (MODE == 0) {
                                q[0] = make_float4(x0, x1, x2, __int_as_float(cur));
                            } else {
                                auto half = [&](int k, bool hi) {
                                    return __int_as_float(hi ? __double2hiint(xd[k]) : __double2loint(xd[k]));
                                };
                                q[0] = make_float4(half(0, false), half(0, true), half(1, false), half(1, true));
                                q[C4 - 1] = make_float4(half(2, false), half(2, true), 0.f, __int_as_float(cur));
                            }
                            const float4 *fr = reinterpret_cast<const float4 *>(a.rfeat) + (long long)cur * F4;
#pragma unroll
                            for (int f = 0; f < F4; ++f) q[C4 + f] = fr[f];
                        }
                        k += pstride;
                        const bool more = k * kWave < base + total;
                        if (more) fetch();
                        qn += __popcll(mask);
                        wave_sync();
                        if (qn >= kQueueFlush) {
                            process(qn);
                            qn = 0;
                            wave_sync();
                        }
                        if (!more) break;
                    }
                    wave_sync();
                }
                base += total;
            }
        }
        process(qn);
        wave_sync();

        // (a lane without pairs takes nothing off: 0 times a feature that is not
        // finite is not 0)
        if (MODE == 1 && __builtin_amdgcn_inverse_ballot_w64(paired)) {
#pragma unroll
            for (int k = 0; k < SED; ++k) Gf[MODE == 1 ? k : 0] -= W * (double)vf[k];
        }
        float4 ze = make_float4(0.f, 0.f, 0.f, 0.f);
        if (MODE == 0) {  // the query's point again: it need not stay in registers over the walk
            int pe = pq;
            asm volatile("" : "+v"(pe));
            ze = a.qpts[pe];
        }
        // combine the sub-streams of each query (fixed shuffle order)
        for (int off = np2; off < kWave; off <<= 1) {
            W += __shfl_xor(W, off);
            Dx += __shfl_xor(Dx, off);
            Dy += __shfl_xor(Dy, off);
            Dz += __shfl_xor(Dz, off);
            if (MODE == 0) {
                S00 += __shfl_xor(S00, off);
                S01 += __shfl_xor(S01, off);
                S02 += __shfl_xor(S02, off);
                S11 += __shfl_xor(S11, off);
                S12 += __shfl_xor(S12, off);
                S22 += __shfl_xor(S22, off);
            } else if (kGrad) {
                Ls += __shfl_xor(Ls, off);
#pragma unroll
                for (int k = 0; k < (MODE == 1 ? VF : 1); ++k) Gf[k] += __shfl_xor(Gf[k], off);
            }
        }
        if (qs == 0 && active) {
            if (MODE == 0 && W != 0.0) {
                // the query's rounding (e: rounded less exact) taken off D to
                // first order: dD/dz = -(W I - 2 ln 2 sum w d d^T).  What is
                // left of the gradient's error is the reference points' rounding.
                const double ex = (double)zrx - (Pm[0] * ze.x + Pm[1] * ze.y + Pm[2] * ze.z + Pm[3] - cx) * sc;
                const double ey = (double)zry - (Pm[4] * ze.x + Pm[5] * ze.y + Pm[6] * ze.z + Pm[7] - cy) * sc;
                const double ez = (double)zrz - (Pm[8] * ze.x + Pm[9] * ze.y + Pm[10] * ze.z + Pm[11] - cz) * sc;
                const double l2 = 2.0 * 0.6931471805599453;
                Dx += W * ex - l2 * (S00 * ex + S01 * ey + S02 * ez);
                Dy += W * ey - l2 * (S01 * ex + S11 * ey + S12 * ez);
                Dz += W * ez - l2 * (S02 * ex + S12 * ey + S22 * ez);
            }
            // every output is linear in the kernel weights; written value by
            // value over the cluster's queries
            const double sg = (double)sig2;
            const long long f = pc.w;
            if (!kGrad) {  // (mode 2: D and S are zero)
                double *B = a.oWD + 4 * f + t;
                B[0] = sg * W;
                B[n] = sg * Dx;
                B[2 * n] = sg * Dy;
                B[3 * n] = sg * Dz;
                float *S = a.oS + 6 * f + t;
                S[0] = sig2 * S00;
                S[n] = sig2 * S01;
                S[2 * n] = sig2 * S02;
                S[3 * n] = sig2 * S11;
                S[4 * n] = sig2 * S12;
                S[5 * n] = sig2 * S22;
                a.oCnt[f + t] = t == 0 ? cnt : 0;  // counted for the wave
            } else {
                double *B = a.oB + f * (4 + D4) + t;
                B[0] = sg * Dx;
                B[n] = sg * Dy;
                B[2 * n] = sg * Dz;
                B[3 * n] = sg * Ls;
#pragma unroll
                for (int k = 0; k < (MODE == 1 ? D4 : 0); ++k) B[(4 + k) * n] = sg * Gf[k];
            }
        }
    }
}

// ---------------------------------------------------------------- dispatch
// Compiled feature layouts (SE columns, LIN columns); other layouts are
// padded with zero columns up to the nearest compiled one.
#define CVO_LAYOUTS(X)                                                                                     \
    X(0, 0) X(0, 4) X(0, 19) X(0, 32) X(0, 64) X(5, 0) X(5, 4) X(5, 19) X(5, 32) X(8, 0) X(8, 4) X(8, 19)    \
        X(8, 32) X(16, 0) X(16, 19) X(16, 32) X(32, 0) X(32, 19) X(32, 32)

bool pair_layout_supported(int sed, int lind)
{
#define CVO_CHECK(S, L) if (sed == S && lind == L) return true;
    CVO_LAYOUTS(CVO_CHECK)
#undef CVO_CHECK
    return false;
}

// Layouts whose inner product takes FP64 terms: LIN columns, whose signed weights may
// cancel (10,000 points of 32, twelve draws, F's largest relative error against 64 bits
// 1.1e-6 -> 4.9e-8, the FP32 result's own rounding; pass 36 -> 50 us), without SE
// columns beside them, whose rounding to FP32 when they are scaled leaves as much
// (5 SE + 19 LIN, 20,011 points, would take 103 instead of 61 us).
constexpr bool pair_exact(int sed, int lind) { return sed == 0 && lind > 0; }

template <int S, int L, int MODE>
static void launch_one(const PairPassArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((pair_pass_kernel<S, L, MODE>), dim3((a.npieces + kWavesPerBlock - 1) / kWavesPerBlock),
                       dim3(kWave * kWavesPerBlock), 0, s, a);
}

bool launch_pair_pass(const PairPassArgs &a, const FeatLayout &lay, int mode, hipStream_t s)
{
    if (a.npieces <= 0) return true;
#define CVO_LAUNCH(S, L)                                          \
    if (lay.sed == S && lay.lind == L) {                          \
        if (mode == 1) launch_one<S, L, 1>(a, s);                 \
        else if (mode == 2 && pair_exact(S, L)) launch_one<S, L, pair_exact(S, L) ? 2 : 0>(a, s); \
        else launch_one<S, L, 0>(a, s);                           \
        return true;                                              \
    }
    CVO_LAYOUTS(CVO_LAUNCH)
#undef CVO_LAUNCH
    return false;
}

}  // namespace cvo

