// The bottom of the hierarchy in one launch: the level of 8^3 (or 6^3) points
// and the coarsest level below it, by one workgroup with both levels in LDS.
// As launches of their own these two levels took seven dependent launches of
// 2.5-6.5 us per V-cycle (29 us) for 0.3 us of arithmetic; here a half-sweep
// costs one LDS round trip, the point solve's chain and a barrier (1370
// cycles), the whole launch 16-19 us (6^3: 13; the adjoint's 14; about 210 where
// the coarsest inverse is formed).  It is bound by those chains: the loads
// 5000 cycles, eight half-sweeps 11000-14000, the coarsest solve 3500-6000 per
// iteration.  One thread per point and half-sweep (four waves at 8^3): two
// points per thread in two waves measured 24 us.  Every value is computed by the
// functions the per-level kernels use, in their order, so results are theirs bit
// for bit.
#pragma once

#include "coarse.h"
#include "smooth.h"

namespace pfc {

// N: points per axis of the upper level (8 or 6).  A thread owns the x-pair of
// points (2I + a, 2J + b, 2K + zz), one of each colour; the four threads of a
// coarse cell are a quad of lanes.
// PH: the scheme's cycle, or the adjoint's linear one (f = b, phk = D; the
// iterate starts at zero and the coarse correction is the coarse iterate).
template <typename T, int PH, bool DELTA, bool MOB, int N, int TH = (N * N * N / 2 + 63) / 64 * 64>
struct Tail {
    static constexpr bool ADJ = PH == BP_ADJ;
    static constexpr int HN = N / 2, HC = N * N * HN, NC = HN, PC = NC * NC * NC;
    static constexpr int kActive = 4 * PC, kThreads = TH;
    static_assert(kActive <= TH && TH % 64 == 0, "a thread per x-pair, whole waves");
    static constexpr int NF = MOB ? 4 : 3;
    struct Shared {
        T u[NF][2][HC];                 // upper level, colour-split
        T cu[3][PC], cf[3][PC], cb[3][PC];  // coarsest: iterate, right-hand side, I u
        CoarseShared cs;
        unsigned long long wm[kThreads / 64];
    };

    const TailArgs<T> &a;
    Shared &sm;
    int I, J, K, zz, b;
    bool act;
    double own[2];  // phi of the thread's points while a smoothing run lasts
    T f[2][3], ak[2], bb[2];  // of the thread's point of each colour

    __device__ __forceinline__ Tail(const TailArgs<T> &a_, Shared &s_) : a(a_), sm(s_) {
        const int t = threadIdx.x;
        act = kActive == TH || t < kActive;
        const int cell = act ? t >> 2 : 0;
        zz = t >> 1 & 1;
        b = t & 1;
        I = cell % NC;
        J = cell / NC % NC;
        K = cell / (NC * NC);
    }

    // LDS positions of the thread's point of colour c and its neighbours
    struct Pt {
        int x, y, z, q, nb[6];  // xp, xm, yp, ym, zp, zm (other colour)
    };
    __device__ __forceinline__ Pt pt(int c) const {
        Pt p;
        p.y = 2 * J + b;
        p.z = 2 * K + zz;
        const int s = (b + zz + c) & 1;  // x parity
        p.x = 2 * I + s;
        const int row = (p.z * N + p.y) * HN;
        p.q = row + I;
        p.nb[0] = row + (s ? (I == HN - 1 ? 0 : I + 1) : I);
        p.nb[1] = row + (s ? I : (I == 0 ? HN - 1 : I - 1));
        p.nb[2] = (p.z * N + wrap_p(p.y, N)) * HN + I;
        p.nb[3] = (p.z * N + wrap_m(p.y, N)) * HN + I;
        p.nb[4] = (wrap_p(p.z, N) * N + p.y) * HN + I;
        p.nb[5] = (wrap_m(p.z, N) * N + p.y) * HN + I;
        return p;
    }
    __device__ __forceinline__ double sum(int fl, int c, const Pt &p) const {
        const T *o = &sm.u[fl][c ^ 1][0];
        return ((double)o[p.nb[0]] + (double)o[p.nb[1]]) + ((double)o[p.nb[2]] + (double)o[p.nb[3]]) +
               ((double)o[p.nb[4]] + (double)o[p.nb[5]]);
    }
    __device__ __forceinline__ void laps(int c, const Pt &p, double (&ls)[3], double (&w)[3]) const {
        const double h2inv = a.op.h2inv;
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) {
            w[fl] = (double)sm.u[fl][c][p.q];
            ls[fl] = (sum(fl, c, p) - 6.0 * w[fl]) * h2inv;
        }
        if constexpr (MOB) {
            const double pc = (double)sm.u[3][c][p.q];
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e)
                s += face_mob(a.op.mob, pc, (double)sm.u[3][c ^ 1][p.nb[e]]) *
                     ((double)sm.u[1][c ^ 1][p.nb[e]] - w[1]);
            ls[1] = s * h2inv;
        }
    }
    // point_solve in two parts, its operations in its order: what the own old value
    // gives is formed while the neighbours' loads are under way (with every neighbour's
    // load ahead of the sums, own values in registers and the coarsest product's loads
    // ahead of its sums: cycle of 32^3 60.1 -> 59.3 us, 64^3 106.3 -> 105.4, 96^3 F
    // 353.2 -> 351.5).  Here and not in point_solve: split there, the compiler lays the
    // two-sweep launch out otherwise, 128^3 252 -> 258 us per cycle.
    __device__ __forceinline__ void point_cubic(const PointCoef &q, double phin, double k, double base,
                                                double &c, double &cubic) const {
        if (!DELTA && a.picard) {
            const double qq = q.fo ? phin * phin : 0.25 * (phin * phin + k * k);
            c = qq + q.lin_c;
            cubic = q.fo ? 0.0 : qq * k;
        } else {
            const double gp = dg_of<DELTA>(q.fo, phin, k, base);
            c = gp + q.lin_c;
            cubic = g_of<DELTA>(q.fo, phin, k, base) - gp * phin;
        }
    }
    // s3: the neighbours' sums of phi, mu, omega
    __device__ __forceinline__ void point_rest(const PointCoef &q, double c, double cubic, double f1,
                                               double f2, double f3, const double (&s3)[3], double &phi,
                                               double &mu, double &om) const {
        const double r2 = f2 + s3[2] * q.h2inv + cubic;
        const double r1 = f1 + q.tau * s3[1] * q.h2inv;
        const double r3 = f3 + q.w3 * s3[0] * q.h2inv;
        phi = (r1 - q.A * r2 + q.AB * r3) / (1.0 + q.A * (c + q.BD));
        om = r3 - q.Dd * phi;
        mu = r2 + c * phi - q.B * om;
    }
    __device__ __forceinline__ void half_sweep(int c) {
        if (act) {
            const Pt p = pt(c);
            const double phin = own[c], k = (double)ak[c];
            const double f0 = (double)f[c][0], f1 = (double)f[c][1], f2 = (double)f[c][2];
            double phi, mu, om;
            if constexpr (ADJ) {
                const double s3[3] = {sum(0, c, p), sum(1, c, p), sum(2, c, p)};
                double l[3];
                adj_point_solve(a.op, k, f0, f1, f2, s3, l);
                phi = l[0];
                mu = l[1];
                om = l[2];
            } else if constexpr (MOB) {
                const double pc = (double)sm.u[3][c][p.q];
                double msum = 0.0, smm = 0.0;
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    const double mf = face_mob(a.op.mob, pc, (double)sm.u[3][c ^ 1][p.nb[e]]);
                    msum += mf;
                    smm += mf * (double)sm.u[1][c ^ 1][p.nb[e]];
                }
                point_solve_mob(a.op, a.picard, phin, k, f0, f1, f2, msum, smm, sum(2, c, p),
                                sum(0, c, p), phi, mu, om);
            } else {
                double nb[3][6], co, cubic, s3[3];
#pragma unroll
                for (int fl = 0; fl < 3; ++fl)
#pragma unroll
                    for (int e = 0; e < 6; ++e) nb[fl][e] = (double)sm.u[fl][c ^ 1][p.nb[e]];
                const PointCoef q(a.op);
                point_cubic(q, phin, k, (double)bb[c], co, cubic);
#pragma unroll
                for (int fl = 0; fl < 3; ++fl)
                    s3[fl] = (nb[fl][0] + nb[fl][1]) + (nb[fl][2] + nb[fl][3]) + (nb[fl][4] + nb[fl][5]);
                point_rest(q, co, cubic, f0, f1, f2, s3, phi, mu, om);
            }
            own[c] = (double)(T)phi;
            sm.u[0][c][p.q] = (T)phi;
            sm.u[1][c][p.q] = (T)mu;
            sm.u[2][c][p.q] = (T)om;
        }
        __syncthreads();
    }

    // The visits of the level: one cycle, or an F-cycle and then a V-cycle.  On
    // the first the iterate starts at I u and f takes the tau correction.  The
    // loops stay loops (the code is fetched by this one workgroup alone).
    __device__ __forceinline__ void cycles(bool cached) {
        if (act && !ADJ)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                double ls[3], w[3], nv[3];
                laps(c, pt(c), ls, w);
                n_of_point<DELTA>(a.op, ls, w[0], w[1], w[2], (double)ak[c], (double)bb[c], nv);
#pragma unroll
                for (int fl = 0; fl < 3; ++fl) f[c][fl] = (T)((double)f[c][fl] + nv[fl]);
            }
        __syncthreads();
#pragma unroll 1
        for (int visit = 0; visit <= a.fcycle; ++visit) {
#pragma unroll 1
            for (int side = 0; side < 2; ++side) {  // before and after the coarsest solve
                if (side == 1) {
                    restrict_();
                    __syncthreads();
                    // an F-cycle solves twice on its way down
                    if (threadIdx.x < 64) coarsest(a.fcycle && visit == 0 ? 2 : 1, cached);
                    cached = true;
                    __syncthreads();
                    prolong();
                    __syncthreads();
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) own[c] = act ? (double)sm.u[0][c][pt(c).q] : 0.0;
#pragma unroll 1
                for (int s = 0; s < (side ? a.nu2 : a.nu1); ++s) {
                    half_sweep(0);
                    half_sweep(1);
                }
            }
        }
    }

    // the coarsest level's tau correction (starting its iterate at I u) and solves
    __device__ __forceinline__ void coarsest(int solves, bool cached) {
        const Tri<T> cu{sm.cu[0], sm.cu[1], sm.cu[2]}, cf{sm.cf[0], sm.cf[1], sm.cf[2]};
        if constexpr (ADJ) {  // linear: a second solve would repeat the first
            adj_coarse_body(a.opc, cu, cst(cf), a.phkc, a.lap1, a.lap3, a.minv, cached, a.valid, sm.cs);
            wave_sync();
            return;
        }
        const Tri<const T> cb{sm.cb[0], sm.cb[1], sm.cb[2]};
        tau_body<T, DELTA, MOB>(a.opc, cb, cf, cu, a.phkc, a.basec, threadIdx.x);
        wave_sync();
#pragma unroll 1
        for (int q = 0; q < solves; ++q) {
            coarse_body<T, DELTA, MOB>(a.opc, cu, cst(cf), a.phkc, a.basec, a.lap1, a.lap3, a.minv,
                                       cached || q > 0, a.valid, a.iters, sm.cs, a.lap2);
            wave_sync();
        }
    }

    // residual and iterate to the coarsest level, the cell's children added in
    // the order 000, 100, 010, 110, 001, ... (its quad's lanes in turn)
    __device__ __forceinline__ void restrict_() {
        double r[2][3], w[2][3];  // [colour]
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            double ls[3];
            laps(c, pt(c), ls, w[c]);
            if constexpr (ADJ)
                adj_resid_from_lap(a.op, ls, w[c], (double)f[c][0], (double)f[c][1], (double)f[c][2],
                                   (double)ak[c], r[c]);
            else
                resid_from_lap<DELTA>(a.op, ls, w[c][0], w[c][1], w[c][2], (double)f[c][0],
                                      (double)f[c][1], (double)f[c][2], (double)ak[c], (double)bb[c],
                                      r[c]);
        }
        const int o = (K * NC + J) * NC + I;
        const bool c1 = ((b + zz) & 1) != 0;  // the pair's even-x point is colour 1
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) {
            const double r0 = c1 ? r[1][fl] : r[0][fl], r1 = c1 ? r[0][fl] : r[1][fl];
            const double u0 = c1 ? w[1][fl] : w[0][fl], u1 = c1 ? w[0][fl] : w[1][fl];
            double sr = 0.0, su = 0.0;
            sr += quad_bcast<0>(r0);
            sr += quad_bcast<0>(r1);
            sr += quad_bcast<1>(r0);
            sr += quad_bcast<1>(r1);
            sr += quad_bcast<2>(r0);
            sr += quad_bcast<2>(r1);
            sr += quad_bcast<3>(r0);
            sr += quad_bcast<3>(r1);
            su += quad_bcast<0>(u0);
            su += quad_bcast<0>(u1);
            su += quad_bcast<1>(u0);
            su += quad_bcast<1>(u1);
            su += quad_bcast<2>(u0);
            su += quad_bcast<2>(u1);
            su += quad_bcast<3>(u0);
            su += quad_bcast<3>(u1);
            if (act && zz == 0 && b == 0) {
                sm.cf[fl][o] = (T)(0.125 * sr);
                sm.cb[fl][o] = (T)(0.125 * su);
            }
        }
    }

    __device__ __forceinline__ void prolong() {
        if (!act) return;
        const int Im[2] = {wrap_m(I, NC), wrap_p(I, NC)};
        const int J1 = b ? wrap_p(J, NC) : wrap_m(J, NC), K1 = zz ? wrap_p(K, NC) : wrap_m(K, NC);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) {
            auto e = [&](int x, int y, int z) {
                const int o = (z * NC + y) * NC + x;
                return ADJ ? (double)sm.cu[fl][o] : (double)(T)((double)sm.cu[fl][o] - (double)sm.cb[fl][o]);
            };
            auto wt = [&](int x) {
                return 0.75 * (0.75 * e(x, J, K) + 0.25 * e(x, J1, K)) +
                       0.25 * (0.75 * e(x, J, K1) + 0.25 * e(x, J1, K1));
            };
            const double w1 = wt(I);
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int c = (x + b + zz) & 1, q = ((2 * K + zz) * N + 2 * J + b) * HN + I;
                sm.u[fl][c][q] = (T)((double)sm.u[fl][c][q] + (0.75 * w1 + 0.25 * wt(Im[x])));
            }
        }
    }

    __device__ __forceinline__ void run() {
        const bool cached = coarse_load_inverse<kThreads>(a.minv, a.valid, sm.cs);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const Pt p = pt(c);
            const unsigned g = (unsigned)(c * HC + p.q);  // the level's colour-split storage
            T ub[3] = {(T)0, (T)0, (T)0};
            if constexpr (!ADJ) {
                ub[0] = a.ub.a[g];
                ub[1] = a.ub.b[g];
                ub[2] = a.ub.c[g];
            }
            f[c][0] = a.f.a[g];
            f[c][1] = a.f.b[g];
            f[c][2] = a.f.c[g];
            ak[c] = a.phk[g];
            bb[c] = DELTA ? a.base[g] : (T)0;
            if (act) {
#pragma unroll
                for (int fl = 0; fl < 3; ++fl) sm.u[fl][c][p.q] = ub[fl];
                if constexpr (MOB) sm.u[3][c][p.q] = (T)a.op.mob.phs[g];
            }
        }
        const bool test = a.stop.partial != nullptr;
        int counted = 0;
        if (test) {
            counted = *a.stop.st.cycles;
            const unsigned long long m = wave_umax(stop_test_max<kThreads>(a.stop));
            if ((threadIdx.x & 63) == 0) sm.wm[threadIdx.x >> 6] = m;
        }
        __syncthreads();
        if (test) {
            unsigned long long m = sm.wm[0];
            for (int w = 1; w < kThreads / 64; ++w) m = umax(m, sm.wm[w]);
            if (!stop_test_decide(a.stop, m, counted)) return;
        }
        cycles(cached);
        if (act)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const Pt p = pt(c);
                const unsigned g = (unsigned)(c * HC + p.q);
                a.u.a[g] = sm.u[0][c][p.q];
                a.u.b[g] = sm.u[1][c][p.q];
                a.u.c[g] = sm.u[2][c][p.q];
            }
    }
};

}  // namespace pfc
