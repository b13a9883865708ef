// The coarsest level's exact solve and the tau correction of one point, shared
// by the per-level launches, the small-level tail and the batched form.
#pragma once

#include "device_common.h"

namespace pfc {

// ------------------------------------------------------- tau correction
//
// Coarse right-hand side of the FAS: f_c = N_c(I u) + I r (f holds I r on
// entry); also starts the coarse iterate at I u, unless u.a is null.
template <typename T, bool DELTA, bool MOB = false>
__device__ __forceinline__ void tau_body(const OpParams &op, Tri<const T> ubar, Tri<T> f, Tri<T> u,
                                         const T *__restrict__ phk, const T *__restrict__ base,
                                         unsigned t) {
    const Lay &L = op.lay;
    if (t >= (unsigned)npts(L)) return;
    int i, j, k;
    decode(L, t, i, j, k);
    const Off q = offs(L, i, j, k);
    const double phi = ubar.a[t], mu = ubar.b[t], om = ubar.c[t];
    double lmu;
    if constexpr (MOB) {
        const double *ps = op.mob.phs;
        const double pc = ps[q.c];
        const unsigned nb6[6] = {q.xp, q.xm, q.yp, q.ym, q.zp, q.zm};
        double sm = 0.0;
#pragma unroll
        for (int e = 0; e < 6; ++e)
            sm += face_mob(op.mob, pc, ps[nb6[e]]) * ((double)ubar.b[nb6[e]] - mu);
        lmu = sm * op.h2inv;
    } else {
        lmu = (nsum(ubar.b, q) - 6.0 * mu) * op.h2inv;
    }
    const double ls[3] = {(nsum(ubar.a, q) - 6.0 * phi) * op.h2inv, lmu,
                          (nsum(ubar.c, q) - 6.0 * om) * op.h2inv};
    // every load ahead of the first store (which may alias them as far as the
    // compiler knows); I u's own values are copied from phi, mu, om (exact)
    const double f0 = f.a[t], f1 = f.b[t], f2 = f.c[t];
    double nv[3];
    n_of_point<DELTA>(op, ls, phi, mu, om, (double)phk[t], DELTA ? (double)base[t] : 0.0, nv);
    f.a[t] = (T)(f0 + nv[0]);
    f.b[t] = (T)(f1 + nv[1]);
    f.c[t] = (T)(f2 + nv[2]);
    if (u.a) {
        u.a[t] = (T)phi;
        u.b[t] = (T)mu;
        u.c[t] = (T)om;
    }
}

// ------------------------------------------------------ coarsest solve

// LDS of the coarsest solve.  A: the Newton inverse (column-major,
// A[col * P + row]), also the workspace it is rebuilt in.
struct CoarseShared {
    double A[64 * 64];
    double vec[64], dvec[64];
    int perm[64];
};

// The cached inverse into LDS, by the workgroup's TH threads; returns
// whether there is one.  The caller's next barrier makes it visible.
template <int TH>
__device__ __forceinline__ bool coarse_load_inverse(const double *minv, const int *valid,
                                                    CoarseShared &sm) {
    // minv is 64 x 64 doubles whatever P is: the loads of TH threads in one block
    constexpr int kPer = 64 * 64 / TH;
    double r[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) r[i] = minv[threadIdx.x + i * TH];
    const int ok = *valid;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sm.A[threadIdx.x + i * TH] = r[i];
    return ok != 0;
}

// Exact solve of N_c(u) = f on the coarsest level (natural layout, n = 3 or
// 4, P = n^3 <= 64 points), one 64-lane wavefront, lane p owning point p (the
// first wavefront of its workgroup; the others wait at the caller's barrier).
// omega and mu enter linearly and are eliminated exactly:
//   F(phi) = phi - tau Lap(g(phi) + (1-eps)/2 phi) - tau/2 Lap^3 phi - b = 0,
//   b = f1 + tau Lap(f2 + Lap f3),
//   F'(phi) = I - tau Lap diag(g'(phi) + (1-eps)/2) - tau/2 Lap^3,
// then omega = f3 + Lap phi / 2 and mu = f2 + g(phi) + (1-eps)/2 phi + Lap omega.
// Iteration: phi <- phi - Minv F(phi) with Minv = F'(phi_0)^{-1} kept across
// calls (chord method; the caller copies it to sm.A, where the iterations read
// it, with coarse_load_inverse, whose return value is `cached`); when an iteration contracts by less than 4x, Minv is
// rebuilt at the current iterate (which makes that step a Newton step).  The
// inverse comes from Gauss-Jordan elimination with partial pivoting in LDS.
// Stops when max|update| <= 1e-14 max(1, max|phi|) (or after 60 iterations).
// First-order scheme (op.fo): g(phi) = phi^3, (1-eps) phi, the Lap^3 term with
// tau instead of tau/2 and omega = f3 + Lap phi.
// MOB (variable mobility): the outer Lap of the first equation becomes the
// flux operator L_M = d(M D), so F(phi) = phi - tau L_M(g(phi) + (1-eps)/2 phi)
// - tau/2 L_M Lap^2 phi - b with b = f1 + tau L_M(f2 + Lap f3); its Jacobian
// uses the dense Lap^2 (lap2) for the L_M Lap^2 block.
template <typename T, bool DELTA, bool MOB = false>
__device__ __forceinline__ void coarse_body(const OpParams &op, Tri<T> u, Tri<const T> f,
                                            const T *__restrict__ phk, const T *__restrict__ base,
                                            const double *__restrict__ lap1,
                                            const double *__restrict__ lap3, double *minv,
                                            bool cached, int *valid, int *iters, CoarseShared &sm,
                                            const double *__restrict__ lap2 = nullptr) {
    double *A = sm.A, *vec = sm.vec, *dvec = sm.dvec;
    const int n = op.lay.n, P = n * n * n;
    const int p = threadIdx.x;
    const bool act = p < P;
    const double h2inv = op.h2inv, tau = op.tau, lc = lin_of(op), w3 = w3_of(op);

    int nb[6] = {0, 0, 0, 0, 0, 0};
    if (act) {
        const int i = p % n, j = (p / n) % n, k = p / (n * n);
        nb[0] = (k * n + j) * n + wrap_p(i, n);
        nb[1] = (k * n + j) * n + wrap_m(i, n);
        nb[2] = (k * n + wrap_p(j, n)) * n + i;
        nb[3] = (k * n + wrap_m(j, n)) * n + i;
        nb[4] = (wrap_p(k, n) * n + j) * n + i;
        nb[5] = (wrap_m(k, n) * n + j) * n + i;
    }
    // Lap of the field held in v[] at point p (call between barriers)
    auto lap_lds = [&](const double *v, double own) -> double {
        return ((v[nb[0]] + v[nb[1]]) + (v[nb[2]] + v[nb[3]]) + (v[nb[4]] + v[nb[5]]) - 6.0 * own) *
               h2inv;
    };
    // face mobilities of point p (MOB), and L_M of the field held in vec[]
    double mf[6] = {1.0, 1.0, 1.0, 1.0, 1.0, 1.0}, msum = 6.0;
    if constexpr (MOB) {
        if (act) {
            msum = 0.0;
            for (int e = 0; e < 6; ++e) {
                mf[e] = face_mob(op.mob, op.mob.phs[p], op.mob.phs[nb[e]]);
                msum += mf[e];
            }
        }
    }
    auto lapo_lds = [&](const double *v, double own) -> double {  // the first equation's outer operator
        if constexpr (MOB) {
            double s6 = 0.0;
            for (int e = 0; e < 6; ++e) s6 += mf[e] * (v[nb[e]] - own);
            return s6 * h2inv;
        } else {
            return lap_lds(v, own);
        }
    };
    const double a = act ? (double)phk[p] : 0.0;
    const double bs = (DELTA && act) ? (double)base[p] : 0.0;
    const double F1 = act ? (double)f.a[p] : 0.0;
    const double F2 = act ? (double)f.b[p] : 0.0;
    const double F3 = act ? (double)f.c[p] : 0.0;
    double x = act ? (double)u.a[p] : 0.0;

    vec[p] = F3;
    wave_sync();
    const double t3 = act ? lap_lds(vec, F3) : 0.0;
    wave_sync();
    vec[p] = F2 + t3;
    wave_sync();
    const double bp = F1 + tau * (act ? lapo_lds(vec, F2 + t3) : 0.0);
    wave_sync();

    // Builds Minv = F'(x)^{-1} into global memory.
    auto rebuild = [&]() {
        dvec[p] = dg_of<DELTA>(op.fo, x, a, bs) + lc;
        wave_sync();
        if (act && !MOB) {
            // row p of F'(x); the dense Lap and Lap^3 come from global memory,
            // so their loads are issued 16 at a time ahead of the stores
            for (int q0 = 0; q0 < P; q0 += 16) {
                double l1v[16], l3v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int q = q0 + i;
                    l1v[i] = q < P ? lap1[q * P + p] : 0.0;
                    l3v[i] = q < P ? lap3[q * P + p] : 0.0;
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int q = q0 + i;
                    if (q < P)
                        A[q * P + p] =
                            (q == p ? 1.0 : 0.0) - tau * l1v[i] * dvec[q] - w3 * tau * l3v[i];
                }
            }
        }
        if constexpr (MOB) {
            if (act)
                for (int q = 0; q < P; ++q) {
                    // row p of L_M and of L_M Lap^2 (lap2 column-major: [col * P + row])
                    double lm = q == p ? -msum : 0.0, lmd2 = -msum * lap2[q * P + p];
                    for (int e = 0; e < 6; ++e) {
                        if (nb[e] == q) lm += mf[e];
                        lmd2 += mf[e] * lap2[q * P + nb[e]];
                    }
                    A[q * P + p] = (q == p ? 1.0 : 0.0) - tau * (lm * h2inv) * dvec[q] -
                                   0.5 * tau * (lmd2 * h2inv);
                }
        }
        wave_sync();
        gj_invert(A, P, sm.perm);
        if (act)
            for (int q = 0; q < P; ++q) minv[q * P + p] = A[q * P + p];
        wave_sync();
    };

    bool need = !cached, fresh = need;  // rebuild before the next iteration; just rebuilt
    double dprev = 0.0;
    int it;
#pragma unroll 1
    for (it = 1; it <= 60; ++it) {
        if (need) {
            rebuild();
            need = false;
        }
        const double w = g_of<DELTA>(op.fo, x, a, bs) + lc * x;
        vec[p] = w;
        dvec[p] = x;
        wave_sync();
        const double lw = act ? lapo_lds(vec, w) : 0.0;
        const double l1 = act ? lap_lds(dvec, x) : 0.0;
        wave_sync();
        vec[p] = l1;
        wave_sync();
        const double l2 = act ? lap_lds(vec, l1) : 0.0;
        wave_sync();
        vec[p] = l2;
        wave_sync();
        const double l3 = act ? lapo_lds(vec, l2) : 0.0;
        dvec[p] = act ? (x - tau * lw - w3 * tau * l3 - bp) : 0.0;
        wave_sync();
        double d = 0.0;
        // 8 columns' loads in one block, ahead of the sums over the 8 before; past P: 0
        // times 0
        double ma[8], va[8], mb[8], vb[8];
        auto load = [&](double (&m)[8], double (&v)[8], int q0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                m[i] = A[(q0 + i) * P + p];
                v[i] = dvec[q0 + i];
            }
        };
        auto add = [&](const double (&m)[8], const double (&v)[8], int q0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) d -= (act && q0 + i < P ? m[i] : 0.0) * v[i];
        };
        load(ma, va, 0);
#pragma unroll 1
        for (int q0 = 0; q0 < P; q0 += 16) {
            load(mb, vb, q0 + 8);
            add(ma, va, q0);
            load(ma, va, q0 + 16 < P ? q0 + 16 : 0);
            add(mb, vb, q0 + 8);
        }
        x += d;
        const double dm = wave_max(fabs(d));
        const double xm = wave_max(fabs(x));
        wave_sync();
        if (!(dm == dm)) break;
        if (dm <= 1e-14 * fmax(1.0, xm)) break;
        need = fresh = !fresh && it > 1 && dm > 0.25 * dprev;
        dprev = dm;
    }
    if (it > 60) it = 60;
    vec[p] = x;
    wave_sync();
    const double lx = act ? lap_lds(vec, x) : 0.0;
    wave_sync();
    const double om = F3 + w3 * lx;
    vec[p] = om;
    wave_sync();
    const double lom = act ? lap_lds(vec, om) : 0.0;
    const double mu = F2 + g_of<DELTA>(op.fo, x, a, bs) + lc * x + lom;
    if (act) {
        u.a[p] = (T)x;
        u.b[p] = (T)mu;
        u.c[p] = (T)om;
    }
    if (p == 0) {
        *valid = 1;
        if (iters) *iters = it;
    }
}

// The adjoint's exact solve on the coarsest level (as coarse_body: one
// wavefront, lane p owning point p): with lambda2 = b2 + tau Lap lambda1 and
// lambda3 = b3 + Lap lambda2 eliminated,
//   (I - tau D Lap - tau/2 Lap^3) lambda1 = b1 + D b2 + 1/2 Lap(b3 + Lap b2).
// minv keeps the inverse of that matrix while *valid is set; it is in sm.A when
// `cached`.
__device__ __forceinline__ void adj_coarse_body(const OpParams &op, Tri<double> lam,
                                                Tri<const double> b, const double *__restrict__ D,
                                                const double *__restrict__ lap1,
                                                const double *__restrict__ lap3, double *minv,
                                                bool cached, int *valid, CoarseShared &sm) {
    double *A = sm.A, *vec = sm.vec;
    const int n = op.lay.n, P = n * n * n;
    const int p = threadIdx.x;
    const bool act = p < P;
    int nb[6] = {0, 0, 0, 0, 0, 0};
    if (act) {
        const int i = p % n, j = (p / n) % n, k = p / (n * n);
        nb[0] = (k * n + j) * n + wrap_p(i, n);
        nb[1] = (k * n + j) * n + wrap_m(i, n);
        nb[2] = (k * n + wrap_p(j, n)) * n + i;
        nb[3] = (k * n + wrap_m(j, n)) * n + i;
        nb[4] = (wrap_p(k, n) * n + j) * n + i;
        nb[5] = (wrap_m(k, n) * n + j) * n + i;
    }
    auto lap_lds = [&](double own) -> double {  // of vec[]
        return ((vec[nb[0]] + vec[nb[1]]) + (vec[nb[2]] + vec[nb[3]]) + (vec[nb[4]] + vec[nb[5]]) -
                6.0 * own) * op.h2inv;
    };
    const double d = act ? D[p] : 0.0;
    const double b1 = act ? b.a[p] : 0.0, b2 = act ? b.b[p] : 0.0, b3 = act ? b.c[p] : 0.0;
    if (!cached) {
        if (act)
            for (int q = 0; q < P; ++q) {
                const int o = q * P + p;
                A[o] = (q == p ? 1.0 : 0.0) - op.tau * d * lap1[o] - 0.5 * op.tau * lap3[o];
            }
        wave_sync();
        gj_invert(A, P, sm.perm);
        if (act)
            for (int q = 0; q < P; ++q) minv[q * P + p] = A[q * P + p];
        wave_sync();
    }
    vec[p] = b2;
    wave_sync();
    const double lb2 = act ? lap_lds(b2) : 0.0;
    wave_sync();
    vec[p] = b3 + lb2;
    wave_sync();
    const double rhs = b1 + d * b2 + 0.5 * (act ? lap_lds(b3 + lb2) : 0.0);
    wave_sync();
    vec[p] = rhs;
    wave_sync();
    double l1 = 0.0;
    if (act)
        for (int q = 0; q < P; ++q) l1 += A[q * P + p] * vec[q];
    wave_sync();
    vec[p] = l1;
    wave_sync();
    const double l2 = b2 + op.tau * (act ? lap_lds(l1) : 0.0);
    wave_sync();
    vec[p] = l2;
    wave_sync();
    const double l3 = b3 + (act ? lap_lds(l2) : 0.0);
    if (act) {
        lam.a[p] = l1;
        lam.b[p] = l2;
        lam.c[p] = l3;
    }
    if (p == 0) *valid = 1;
}

}  // namespace pfc
