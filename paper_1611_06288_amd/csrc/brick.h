// Brick kernels: everything a V-cycle does on one level before it descends
// (pre: tau correction, pre-sweeps, residual, restriction; on the finest level
// also the stop test's norm of the input) or after it comes back (post:
// interpolation, post-sweeps) in ONE launch, for levels too small to keep the
// device busy with a launch per half-sweep.
//
// A workgroup owns a box of points.  It loads the box and the halo that the
// whole chain of half-sweeps can reach (BrickGeo) into LDS, runs every stage
// there on a region that shrinks by one face step per stage, and writes the
// box.  Halo values are recomputed by each workgroup that needs them, from the
// same inputs with the same arithmetic (the functions the half-sweep, tau,
// residual and interpolation kernels use), so results equal those kernels' bit
// for bit.  The iterate is read from one buffer and written to another: other
// workgroups read this one's points as their halo.
//
// Why: on the levels of 12^3 to 96^3 a launch takes 3.3-10 us whatever it
// does, and a level of a V(2,2) cycle took 11 dependent launches.  A launch
// here is bound by one chain of latencies: two dependent loads (the point list,
// then every field at once: 5000-7000 cycles), the stages of 1100-1700 cycles
// each between barriers, and on 64^3 and 96^3 the halo's arithmetic as well.
// Up to 32^3 that chain is what counts: 4^3 boxes, both sweeps of a side in one
// launch; 8 x 4 x 4 at 32^3, where 4^3 boxes are two per CU and share its cycles
// (a 32^3 cycle 69 -> 62.5 us, 64^3 117 -> 110).  From 48^3 on the halo of two
// sweeps costs more than a launch (8^3 boxes with both sweeps: 57 us per cycle at
// 64^3, one sweep per launch 45).  The cycle gate is tested behind the loads, not
// ahead of them (0.3-0.5 us per launch; 64^3 cycle 108.6 -> 105.3 us, 96^3 F-cycle
// 363.5 -> 353.5).
// Measured per V(2,2) cycle, kernel time (half-sweeps -> now): 64^3 finest with its
// stop-test norm 60 -> 44 us in 11 -> 4 launches, 32^3 43 -> 18, 16^3 39 -> 15; a
// 64^3 long-run cycle in all 178 -> 104 us.  From 128^3 on, where bandwidth counts,
// the z-marching kernels take over.
#pragma once

#include "brick_geo.h"
#include "device_common.h"
#include "smooth.h"

namespace pfc {

// One point's six neighbours in a brick's LDS arrays (other colour).
template <typename G>
struct BrickNbr {
    int q, qp;  // own position in its colour, the same plus the x parity
    template <typename T>
    __device__ __forceinline__ double sum(const T *o) const {
        return ((double)o[qp] + (double)o[qp - 1]) + ((double)o[q + G::HX] + (double)o[q - G::HX]) +
               ((double)o[q + G::HX * G::EY] + (double)o[q - G::HX * G::EY]);
    }
    __device__ __forceinline__ int at(int e) const {  // xp, xm, yp, ym, zp, zm
        return e == 0 ? qp : e == 1 ? qp - 1 : e == 2 ? q + G::HX : e == 3 ? q - G::HX
             : e == 4 ? q + G::HX * G::EY : q - G::HX * G::EY;
    }
};

// Threads of a workgroup: one per point of the larger colour's first stage.
constexpr int brick_threads(int n0, int n1) {
    const int n = n0 > n1 ? n0 : n1;
    return (n + 63) / 64 * 64;
}

// Waves per SIMD to compile for: as many as the LDS admits, up to 6 (80 VGPRs).
constexpr int brick_waves(int threads, size_t lds) {
    const int w = ((int)(163840 / lds) * threads + 255) / 256;
    return w < 1 ? 1 : w > 6 ? 6 : w;
}

// Point update (the smoother's 3x3 solve) from the neighbour sums.
template <int PH, bool DELTA, bool MOB>
__device__ __forceinline__ void brick_solve(const OpParams &op, int picard, double phin, double ak,
                                            double bb, const double (&f)[3], const double (&s)[3],
                                            double msum, double smm, double (&o)[3]) {
    if constexpr (PH == BP_ADJ) {
        adj_point_solve(op, ak, f[0], f[1], f[2], s, o);
    } else if constexpr (MOB) {
        point_solve_mob(op, picard, phin, ak, f[0], f[1], f[2], msum, smm, s[2], s[0], o[0], o[1],
                        o[2]);
    } else {
        point_solve<DELTA>(op, picard, phin, ak, bb, f[0], f[1], f[2], s[1], s[2], s[0], o[0], o[1],
                           o[2]);
    }
}

// Kernel body shared by both directions: LDS fields, item geometry.
template <typename T, int PH, bool DELTA, bool MOB, typename G_, int BX, int BY, int BZ, int H>
struct BrickBody {
    using G = G_;
    static constexpr int NF = MOB ? 4 : 3;
    using Field = T[NF][2][G::HC];

    const BrickArgs<T> &a;
    Field &u;
    int n, hn, x0, y0, z0;
    unsigned Hn;

    __device__ __forceinline__ BrickBody(const BrickArgs<T> &a_, Field &u_, int b) : a(a_), u(u_) {
        n = a.op.lay.n;
        hn = n >> 1;
        Hn = (unsigned)n * (unsigned)n * (unsigned)hn;
        const int nbx = n / BX, nby = n / BY;
        x0 = (b % nbx) * BX;
        y0 = (b / nbx) % nby * BY;
        z0 = b / (nbx * nby) * BZ;
    }
    __device__ __forceinline__ int wrap(int v) const { return v < 0 ? v + n : (v >= n ? v - n : v); }

    struct Item {
        BrickNbr<G> nb;
        unsigned g;  // storage offset in the level
        int x, y, z, d;  // d: face steps to the box (beyond every stage past the list's end)
    };
    // item idx of the list of colour C up to distance D; past its end, the
    // last one again (loaded, never used)
    template <int C, int D>
    __device__ __forceinline__ Item item(int idx) const {
        constexpr int c = C;
        const unsigned e = kBrickRows<G, C, D>.p[min(idx, G::cnt(C, D) - 1)];
        Item t;
        t.x = (int)(e & 255u);
        t.y = (int)(e >> 8 & 255u);
        t.z = (int)(e >> 16 & 255u);
        t.d = idx < G::cnt(C, D) ? (int)(e >> 24) : 255;
        t.nb.q = (t.z * G::EY + t.y) * G::HX + (t.x >> 1);
        t.nb.qp = t.nb.q + (t.x & 1);
        const int gx = wrap(x0 - H + t.x), gy = wrap(y0 - H + t.y), gz = wrap(z0 - H + t.z);
        t.g = (unsigned)c * Hn + ((unsigned)gz * (unsigned)n + (unsigned)gy) * (unsigned)hn +
              (unsigned)(gx >> 1);
        return t;
    }
    // sums of the three fields over the neighbours of an item of colour c
    __device__ __forceinline__ void sums(int c, const BrickNbr<G> &nb, double (&s)[3]) const {
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) s[fl] = nb.sum(&u[fl][c ^ 1][0]);
    }
    // flux sum of mu (MOB) around an item of colour c, own value m0
    __device__ __forceinline__ double flux(int c, const BrickNbr<G> &nb, double m0) const {
        const double pc = (double)u[NF - 1][c][nb.q];
        double sm = 0.0;
#pragma unroll
        for (int e = 0; e < 6; ++e)
            sm += face_mob(a.op.mob, pc, (double)u[NF - 1][c ^ 1][nb.at(e)]) *
                  ((double)u[1][c ^ 1][nb.at(e)] - m0);
        return sm;
    }
    // Laplacians (mu: flux form when MOB) and own values of an item
    __device__ __forceinline__ void laps(int c, const BrickNbr<G> &nb, double (&ls)[3],
                                         double (&w)[3]) const {
        double s[3];
        sums(c, nb, s);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) w[fl] = (double)u[fl][c][nb.q];
        const double h2inv = a.op.h2inv;
        ls[0] = (s[0] - 6.0 * w[0]) * h2inv;
        ls[2] = (s[2] - 6.0 * w[2]) * h2inv;
        if constexpr (MOB)
            ls[1] = flux(c, nb, w[1]) * h2inv;
        else
            ls[1] = (s[1] - 6.0 * w[1]) * h2inv;
    }
    __device__ __forceinline__ void resid(int c, const BrickNbr<G> &nb, const T (&f)[3], T ak, T bb,
                                          double (&r)[3]) const {
        double ls[3], w[3];
        laps(c, nb, ls, w);
        if constexpr (PH == BP_ADJ)
            adj_resid_from_lap(a.op, ls, w, (double)f[0], (double)f[1], (double)f[2], (double)ak, r);
        else
            resid_from_lap<DELTA>(a.op, ls, w[0], w[1], w[2], (double)f[0], (double)f[1],
                                  (double)f[2], (double)ak, (double)bb, r);
    }
    // Work on one item of each colour.  Small boxes leave most lanes idle and
    // run both as one chain of latencies; large ones have waves to hide it in,
    // and no registers to spare.
    template <typename F0, typename F1>
    __device__ static __forceinline__ void both(bool c0, bool c1, F0 w0, F1 w1) {
        if constexpr (BX * BY * BZ < 512) {
            if (c0 || c1) {
                w0();
                w1();
            }
        } else {
            if (c0) w0();
            if (c1) w1();
        }
    }
    // old values of the point stored at g (mu, omega only where `all`)
    template <bool ZERO>
    __device__ __forceinline__ void load_u(unsigned g, T (&v)[NF], bool all) const {
        v[0] = v[1] = v[2] = (T)0;
        if constexpr (!ZERO) {
            v[0] = a.u.a[g];
            if (all) {
                v[1] = a.u.b[g];
                v[2] = a.u.c[g];
            }
        }
        if constexpr (MOB) v[3] = (T)a.op.mob.phs[g];
    }
    __device__ __forceinline__ void load_f(unsigned g, T (&f)[3], T &ak, T &bb) const {
        ak = a.phk[g];
        f[0] = a.f.a[g];
        f[1] = a.f.b[g];
        f[2] = a.f.c[g];
        bb = DELTA ? a.base[g] : (T)0;
    }
    // max |S - N(u)| over the box's points into part[b]; every thread calls it
    // (its barrier frees the old colour-0 values to change)
    __device__ __forceinline__ void norm(const Item &i0, const T (&f0)[3], T a0, T b0, const Item &i1,
                                         const T (&f1)[3], T a1, T b1, unsigned long long *wm,
                                         unsigned long long *part, int b) const {
        double r0[3] = {0.0, 0.0, 0.0}, r1[3] = {0.0, 0.0, 0.0};
        both(i0.d == 0, i1.d == 0, [&]() { resid(0, i0.nb, f0, a0, b0, r0); },
             [&]() { resid(1, i1.nb, f1, a1, b1, r1); });
        const unsigned long long m0 = umax(abs_bits(r0[0]), umax(abs_bits(r0[1]), abs_bits(r0[2])));
        const unsigned long long m1 = umax(abs_bits(r1[0]), umax(abs_bits(r1[1]), abs_bits(r1[2])));
        unsigned long long m = umax(i0.d == 0 ? m0 : 0, i1.d == 0 ? m1 : 0);
        m = block_max_u64_waves(m, wm);
        if (threadIdx.x == 0) part[b] = m;
    }
    // the item's right-hand side takes the tau correction
    __device__ __forceinline__ void tau(int c, const Item &it, T (&f)[3], T ak, T bb) const {
        double ls[3], w[3], nv[3];
        laps(c, it.nb, ls, w);
        n_of_point<DELTA>(a.op, ls, w[0], w[1], w[2], (double)ak, (double)bb, nv);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) f[fl] = (T)((double)f[fl] + nv[fl]);
    }
    __device__ __forceinline__ void store_f(const Item &it, const T (&f)[3]) const {
        if (it.d == 0) {
            a.fo.a[it.g] = f[0];
            a.fo.b[it.g] = f[1];
            a.fo.c[it.g] = f[2];
        }
    }
    // one point of a half-sweep, in place
    __device__ __forceinline__ void relax(int c, const BrickNbr<G> &nb, const T (&f)[3], T ak,
                                          T bb) {
        double s[3], o[3], msum = 0.0, smm = 0.0;
        sums(c, nb, s);
        const double phin = PH == BP_ADJ ? 0.0 : (double)u[0][c][nb.q];
        if constexpr (MOB) {
            const double pc = (double)u[NF - 1][c][nb.q];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const double mf = face_mob(a.op.mob, pc, (double)u[NF - 1][c ^ 1][nb.at(e)]);
                msum += mf;
                smm += mf * (double)u[1][c ^ 1][nb.at(e)];
            }
        }
        const double ff[3] = {(double)f[0], (double)f[1], (double)f[2]};
        brick_solve<PH, DELTA, MOB>(a.op, a.picard, phin, (double)ak, (double)bb, ff, s, msum, smm, o);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl) u[fl][c][nb.q] = (T)o[fl];
    }
};

// Before the descent: [norm of the input], [tau correction], S sweeps,
// residual and iterate restricted to the coarse level, the box's iterate
// written (mu and omega of colour-0 points left out: the post kernel's first
// half-sweep overwrites them unread).  Every colour's items are dealt to the
// TH threads in list order; a stage works on those within its distance.
template <typename T, int PH, bool DELTA, bool MOB, int BX, int BY, int BZ, int S, bool TAU, bool NRM,
          bool ZERO>
struct BrickPre {
    static constexpr int H = 2 * S + 1;
    using G = BrickGeo<BX, BY, BZ, H>;
    using Body = BrickBody<T, PH, DELTA, MOB, G, BX, BY, BZ, H>;
    static constexpr int NB = BX * BY * BZ;
    static constexpr int D0 = 2 * S, DF = 2 * S - 1, DU = 2 * S + 1;  // colour 0; colour 1: f, u
    static constexpr int TH = brick_threads(G::cnt(0, D0), G::cnt(1, DF));
    struct Shared {
        typename Body::Field u;
        double r[3][NB];
        unsigned long long wm[TH / 64];
    };
    static constexpr int WAVES = brick_waves(TH, sizeof(Shared));
    static constexpr int slots(int cnt) { return (cnt + TH - 1) / TH; }
    static constexpr int N0 = slots(G::cnt(0, D0)), F1 = slots(G::cnt(1, DF)), N1 = slots(G::cnt(1, DU));
    static_assert(G::template box_end<0, D0>() <= TH && G::template box_end<1, DF>() <= TH,
                  "the box's items are slot 0");

    __device__ static __forceinline__ void run(const BrickArgs<T> &a, int b, Shared &sm,
                                               unsigned long long *part) {
        Body B(a, sm.u, b);
        const int tid = threadIdx.x;
        typename Body::Item i0[N0], i1[F1], iu[N1];
        T f0[N0][3], a0[N0], b0[N0], f1[F1][3], a1[F1], b1[F1];
        T v0[N0][Body::NF], v1[N1][Body::NF];
#pragma unroll
        for (int i = 0; i < N1; ++i) iu[i] = B.template item<1, DU>(tid + i * TH);
#pragma unroll
        for (int i = 0; i < N0; ++i) i0[i] = B.template item<0, D0>(tid + i * TH);
#pragma unroll
        for (int i = 0; i < F1; ++i) i1[i] = B.template item<1, DF>(tid + i * TH);
        // every load of the kernel in one block; old mu, omega of colour 0 are
        // read by the norm and the tau correction only
#pragma unroll
        for (int i = 0; i < N1; ++i) B.template load_u<ZERO>(iu[i].g, v1[i], true);
#pragma unroll
        for (int i = 0; i < N0; ++i) B.template load_u<ZERO>(i0[i].g, v0[i], TAU || NRM);
#pragma unroll
        for (int i = 0; i < N0; ++i) B.load_f(i0[i].g, f0[i], a0[i], b0[i]);
#pragma unroll
        for (int i = 0; i < F1; ++i) B.load_f(i1[i].g, f1[i], a1[i], b1[i]);
        if (gate_closed(a.op.gate)) return;  // its load runs beside the others
#pragma unroll
        for (int i = 0; i < N1; ++i)
            if (iu[i].d <= DU) {
#pragma unroll
                for (int fl = 0; fl < Body::NF; ++fl) sm.u[fl][1][iu[i].nb.q] = v1[i][fl];
            }
#pragma unroll
        for (int i = 0; i < N0; ++i)
            if (i0[i].d <= D0) {
#pragma unroll
                for (int fl = 0; fl < Body::NF; ++fl) sm.u[fl][0][i0[i].nb.q] = v0[i][fl];
            }
        __syncthreads();
        if constexpr (NRM) B.norm(i0[0], f0[0], a0[0], b0[0], i1[0], f1[0], a1[0], b1[0], sm.wm, part, b);
        if constexpr (TAU) {
            B.both(i0[0].d <= D0, i1[0].d <= DF, [&]() { B.tau(0, i0[0], f0[0], a0[0], b0[0]); },
                   [&]() { B.tau(1, i1[0], f1[0], a1[0], b1[0]); });
#pragma unroll
            for (int i = 1; i < N0; ++i)
                if (i0[i].d <= D0) B.tau(0, i0[i], f0[i], a0[i], b0[i]);
#pragma unroll
            for (int i = 1; i < F1; ++i)
                if (i1[i].d <= DF) B.tau(1, i1[i], f1[i], a1[i], b1[i]);
            B.store_f(i0[0], f0[0]);
            B.store_f(i1[0], f1[0]);
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < 2 * S; ++s) {
            const int left = 2 * S - s;  // face steps the rest of the chain reaches
            if ((s & 1) == 0) {
#pragma unroll
                for (int i = 0; i < N0; ++i)
                    if (i0[i].d <= left) B.relax(0, i0[i].nb, f0[i], a0[i], b0[i]);
            } else {
#pragma unroll
                for (int i = 0; i < F1; ++i)
                    if (i1[i].d <= left) B.relax(1, i1[i].nb, f1[i], a1[i], b1[i]);
            }
            __syncthreads();
        }
        auto out = [&](int c, const typename Body::Item &it, const double (&r)[3]) {
            const int o = ((it.z - H) * BY + (it.y - H)) * BX + (it.x - H);
#pragma unroll
            for (int fl = 0; fl < 3; ++fl) sm.r[fl][o] = r[fl];
            a.uo.a[it.g] = sm.u[0][c][it.nb.q];
            if (c) {
                a.uo.b[it.g] = sm.u[1][c][it.nb.q];
                a.uo.c[it.g] = sm.u[2][c][it.nb.q];
            }
        };
        if constexpr (NB < 512) {
            if (i0[0].d == 0 || i1[0].d == 0) {
                double r0[3], r1[3];
                B.resid(0, i0[0].nb, f0[0], a0[0], b0[0], r0);
                B.resid(1, i1[0].nb, f1[0], a1[0], b1[0], r1);
                if (i0[0].d == 0) out(0, i0[0], r0);
                if (i1[0].d == 0) out(1, i1[0], r1);
            }
        } else {
            double r[3];
            if (i0[0].d == 0) {
                B.resid(0, i0[0].nb, f0[0], a0[0], b0[0], r);
                out(0, i0[0], r);
            }
            if (i1[0].d == 0) {
                B.resid(1, i1[0].nb, f1[0], a1[0], b1[0], r);
                out(1, i1[0], r);
            }
        }
        __syncthreads();
        // 8-child means, children in the order 000, 100, 010, 110, 001, ...
        constexpr int NC = NB / 8;
        for (int t = tid; t < 6 * NC; t += TH) {
            const int cmp = t / NC, cell = t - cmp * NC;
            const int I = cell % (BX / 2), J = cell / (BX / 2) % (BY / 2), K = cell / (BX / 2 * (BY / 2));
            double s = 0.0;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const int x = 2 * I + (ch & 1), y = 2 * J + (ch >> 1 & 1), z = 2 * K + (ch >> 2);
                if (cmp < 3)
                    s += sm.r[cmp][(z * BY + y) * BX + x];
                else
                    s += (double)sm.u[cmp - 3][(x + y + z) & 1]
                                     [((z + H) * G::EY + y + H) * G::HX + ((x + H) >> 1)];
            }
            const unsigned g = sidx32(a.LC, B.x0 / 2 + I, B.y0 / 2 + J, B.z0 / 2 + K);
            T *o = cmp == 0 ? a.cr.a : cmp == 1 ? a.cr.b : cmp == 2 ? a.cr.c
                 : cmp == 3 ? a.cu.a : cmp == 4 ? a.cu.b : a.cu.c;
            if (PH != BP_ADJ || cmp < 3) o[g] = (T)(0.125 * s);
        }
    }
};

// S sweeps, the box's iterate written.  PROL (the first sweeps after the
// descent): on u + P(v - I u); old values are corrected where the first
// half-sweep reads them, all fields of colour 1 and phi of colour 0.
// Otherwise with the norm of the input, the tau correction or a zero start as
// the pre kernel.  a.skip0: another sweep follows, so mu and omega of colour-0
// points are left out.
template <typename T, int PH, bool DELTA, bool MOB, int BX, int BY, int BZ, int S, bool PROL, bool TAU,
          bool NRM, bool ZERO>
struct BrickSweep {
    static constexpr int H = 2 * S;
    using G = BrickGeo<BX, BY, BZ, H>;
    using Body = BrickBody<T, PH, DELTA, MOB, G, BX, BY, BZ, H>;
    static constexpr int D0 = 2 * S - 1, DF = 2 * S - 2, DU = 2 * S;  // colour 0; colour 1: f, u
    static constexpr int TH = brick_threads(G::cnt(0, D0), G::cnt(1, DF));
    static constexpr int CX = BX / 2 + H + 2, CY = BY / 2 + H + 2, CZ = BZ / 2 + H + 2;
    static constexpr int NCE = CX * CY * CZ;
    struct Shared {
        typename Body::Field u;
        T e[3][PROL ? CZ : 1][CY][CX];  // coarse error v - I u
        unsigned long long wm[TH / 64];
    };
    static constexpr int WAVES = brick_waves(TH, sizeof(Shared));
    static constexpr int slots(int cnt) { return (cnt + TH - 1) / TH; }
    static constexpr int N0 = slots(G::cnt(0, D0)), F1 = slots(G::cnt(1, DF)), N1 = slots(G::cnt(1, DU)),
                         NE = slots(NCE);
    static_assert(G::template box_end<0, D0>() <= TH && G::template box_end<1, DF>() <= TH,
                  "the box's items are slot 0");

    __device__ static __forceinline__ void run(const BrickArgs<T> &a, int b, Shared &sm,
                                               unsigned long long *part) {
        Body B(a, sm.u, b);
        const int tid = threadIdx.x;
        typename Body::Item i0[N0], i1[F1], iu[N1];
        T f0[N0][3], a0[N0], b0[N0], f1[F1][3], a1[F1], b1[F1];
        T v0[N0][Body::NF], v1[N1][Body::NF], ce[NE][3];
#pragma unroll
        for (int i = 0; i < N1; ++i) iu[i] = B.template item<1, DU>(tid + i * TH);
#pragma unroll
        for (int i = 0; i < N0; ++i) i0[i] = B.template item<0, D0>(tid + i * TH);
#pragma unroll
        for (int i = 0; i < F1; ++i) i1[i] = B.template item<1, DF>(tid + i * TH);
        if constexpr (PROL) {
            const int nc = a.LC.n;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int c = min(tid + i * TH, NCE - 1);
                auto wc = [nc](int v) { return v < 0 ? v + nc : (v >= nc ? v - nc : v); };
                const unsigned g = sidx32(a.LC, wc(B.x0 / 2 - H / 2 - 1 + c % CX),
                                          wc(B.y0 / 2 - H / 2 - 1 + c / CX % CY),
                                          wc(B.z0 / 2 - H / 2 - 1 + c / (CX * CY)));
                if (PH != BP_ADJ) {
                    ce[i][0] = (T)((double)a.v.a[g] - (double)a.ub.a[g]);
                    ce[i][1] = (T)((double)a.v.b[g] - (double)a.ub.b[g]);
                    ce[i][2] = (T)((double)a.v.c[g] - (double)a.ub.c[g]);
                } else {
                    ce[i][0] = a.v.a[g];
                    ce[i][1] = a.v.b[g];
                    ce[i][2] = a.v.c[g];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < N1; ++i) B.template load_u<ZERO>(iu[i].g, v1[i], true);
#pragma unroll
        for (int i = 0; i < N0; ++i) B.template load_u<ZERO>(i0[i].g, v0[i], TAU || NRM);
#pragma unroll
        for (int i = 0; i < N0; ++i) B.load_f(i0[i].g, f0[i], a0[i], b0[i]);
#pragma unroll
        for (int i = 0; i < F1; ++i) B.load_f(i1[i].g, f1[i], a1[i], b1[i]);
        if (gate_closed(a.op.gate)) return;  // its load runs beside the others
        if constexpr (PROL) {
            T *e = &sm.e[0][0][0][0];
#pragma unroll
            for (int i = 0; i < NE; ++i)
                if (tid + i * TH < NCE) {
#pragma unroll
                    for (int fl = 0; fl < 3; ++fl) e[fl * NCE + tid + i * TH] = ce[i][fl];
                }
            __syncthreads();
            // trilinear, in the order of the interpolation kernels
            auto interp = [&](int fl, const typename Body::Item &it) {
                const int X = (it.x >> 1) + 1, Y = (it.y >> 1) + 1, Z = (it.z >> 1) + 1;
                const int X1 = X + ((it.x & 1) ? 1 : -1), Y1 = Y + ((it.y & 1) ? 1 : -1),
                          Z1 = Z + ((it.z & 1) ? 1 : -1);
                auto w = [&](int xx) {
                    return 0.75 * (0.75 * (double)sm.e[fl][Z][Y][xx] + 0.25 * (double)sm.e[fl][Z][Y1][xx]) +
                           0.25 * (0.75 * (double)sm.e[fl][Z1][Y][xx] + 0.25 * (double)sm.e[fl][Z1][Y1][xx]);
                };
                return 0.75 * w(X) + 0.25 * w(X1);
            };
#pragma unroll
            for (int i = 0; i < N1; ++i)
                if (iu[i].d <= DU) {
#pragma unroll
                    for (int fl = 0; fl < 3; ++fl) v1[i][fl] = (T)((double)v1[i][fl] + interp(fl, iu[i]));
                }
#pragma unroll
            for (int i = 0; i < N0; ++i)
                if (PH != BP_ADJ && i0[i].d <= D0) v0[i][0] = (T)((double)v0[i][0] + interp(0, i0[i]));
        }
#pragma unroll
        for (int i = 0; i < N1; ++i)
            if (iu[i].d <= DU) {
#pragma unroll
                for (int fl = 0; fl < Body::NF; ++fl) sm.u[fl][1][iu[i].nb.q] = v1[i][fl];
            }
#pragma unroll
        for (int i = 0; i < N0; ++i)
            if (i0[i].d <= D0) {
#pragma unroll
                for (int fl = 0; fl < Body::NF; ++fl) sm.u[fl][0][i0[i].nb.q] = v0[i][fl];
            }
        __syncthreads();
        if constexpr (NRM) B.norm(i0[0], f0[0], a0[0], b0[0], i1[0], f1[0], a1[0], b1[0], sm.wm, part, b);
        if constexpr (TAU) {
            B.both(i0[0].d <= D0, i1[0].d <= DF, [&]() { B.tau(0, i0[0], f0[0], a0[0], b0[0]); },
                   [&]() { B.tau(1, i1[0], f1[0], a1[0], b1[0]); });
#pragma unroll
            for (int i = 1; i < N0; ++i)
                if (i0[i].d <= D0) B.tau(0, i0[i], f0[i], a0[i], b0[i]);
#pragma unroll
            for (int i = 1; i < F1; ++i)
                if (i1[i].d <= DF) B.tau(1, i1[i], f1[i], a1[i], b1[i]);
            B.store_f(i0[0], f0[0]);
            B.store_f(i1[0], f1[0]);
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < 2 * S; ++s) {
            const int left = 2 * S - 1 - s;
            if ((s & 1) == 0) {
#pragma unroll
                for (int i = 0; i < N0; ++i)
                    if (i0[i].d <= left) B.relax(0, i0[i].nb, f0[i], a0[i], b0[i]);
            } else {
#pragma unroll
                for (int i = 0; i < F1; ++i)
                    if (i1[i].d <= left) B.relax(1, i1[i].nb, f1[i], a1[i], b1[i]);
            }
            if (s + 1 < 2 * S) __syncthreads();
        }
        // each thread wrote its box items itself
        auto out = [&](int c, const typename Body::Item &it) {
            a.uo.a[it.g] = sm.u[0][c][it.nb.q];
            if (c || !a.skip0) {
                a.uo.b[it.g] = sm.u[1][c][it.nb.q];
                a.uo.c[it.g] = sm.u[2][c][it.nb.q];
            }
        };
        if (i0[0].d == 0) out(0, i0[0]);
        if (i1[0].d == 0) out(1, i1[0]);
    }
};

template <typename T, int PH, bool DELTA, bool MOB, int BX, int BY, int BZ, int S, bool TAU, bool NRM,
          bool ZERO>
__global__ __launch_bounds__((BrickPre<T, PH, DELTA, MOB, BX, BY, BZ, S, TAU, NRM, ZERO>::TH),
                             (BrickPre<T, PH, DELTA, MOB, BX, BY, BZ, S, TAU, NRM, ZERO>::WAVES)) void
k_brick_pre(BrickArgs<T> a) {
    using K = BrickPre<T, PH, DELTA, MOB, BX, BY, BZ, S, TAU, NRM, ZERO>;
    __shared__ typename K::Shared sm;
    K::run(a, (int)xcd_block(), sm, a.part);
}

template <typename T, int PH, bool DELTA, bool MOB, int BX, int BY, int BZ, int S, bool PROL, bool TAU,
          bool NRM, bool ZERO>
__global__ __launch_bounds__((BrickSweep<T, PH, DELTA, MOB, BX, BY, BZ, S, PROL, TAU, NRM, ZERO>::TH),
                             (BrickSweep<T, PH, DELTA, MOB, BX, BY, BZ, S, PROL, TAU, NRM, ZERO>::WAVES)) void
k_brick_sweep(BrickArgs<T> a) {
    using K = BrickSweep<T, PH, DELTA, MOB, BX, BY, BZ, S, PROL, TAU, NRM, ZERO>;
    __shared__ typename K::Shared sm;
    K::run(a, (int)xcd_block(), sm, a.part);
}

// Launch of one kernel's form: plain, the first of a coarse level, with the norm.
template <typename Box, bool PRE, typename T, int PH, bool DELTA, bool MOB, int S, bool TAU, bool NRM, bool ZERO>
static void brick_go(hipStream_t s, const BrickArgs<T> &a) {
    const dim3 grid(Box::blocks(a.op.lay.n));
    if constexpr (PRE) {
        using K = BrickPre<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, TAU, NRM, ZERO>;
        hipLaunchKernelGGL((k_brick_pre<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, TAU, NRM, ZERO>), grid,
                           dim3(K::TH), 0, s, a);
    } else {
        using K = BrickSweep<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, false, TAU, NRM, ZERO>;
        hipLaunchKernelGGL((k_brick_sweep<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, false, TAU, NRM, ZERO>),
                           grid, dim3(K::TH), 0, s, a);
    }
}

template <typename Box, bool PRE, typename T, int PH, bool DELTA, bool MOB, int S>
static void brick_form(hipStream_t s, const BrickArgs<T> &a, int form) {
    if (form == BRICK_FIRST)
        return brick_go<Box, PRE, T, PH, DELTA, MOB, S, PH != BP_ADJ, false, PH == BP_ADJ>(s, a);
    if constexpr (!DELTA) {
        if (form == BRICK_NORM) return brick_go<Box, PRE, T, PH, DELTA, MOB, S, false, true, false>(s, a);
    }
    brick_go<Box, PRE, T, PH, DELTA, MOB, S, false, false, false>(s, a);
}

template <typename Box, typename T, int PH, bool DELTA, bool MOB, int S>
static void brick_post(hipStream_t s, const BrickArgs<T> &a) {
    using K = BrickSweep<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, true, false, false, false>;
    hipLaunchKernelGGL((k_brick_sweep<T, PH, DELTA, MOB, Box::X, Box::Y, Box::Z, S, true, false, false, false>),
                       dim3(Box::blocks(a.op.lay.n)), dim3(K::TH), 0, s, a);
}

// The launches of one operator with boxes that take up to two sweeps per launch ...
template <typename Box, typename T, int PH, bool DELTA, bool MOB>
static void brick_two(hipStream_t s, const BrickArgs<T> &a, int kind, int sweeps, int form) {
    if (kind == BRICK_POST)
        sweeps == 1 ? brick_post<Box, T, PH, DELTA, MOB, 1>(s, a) : brick_post<Box, T, PH, DELTA, MOB, 2>(s, a);
    else
        sweeps == 1 ? brick_form<Box, true, T, PH, DELTA, MOB, 1>(s, a, form)
                    : brick_form<Box, true, T, PH, DELTA, MOB, 2>(s, a, form);
}

// ... and with boxes that take one.
template <typename Box, typename T, int PH, bool DELTA, bool MOB>
static void brick_one(hipStream_t s, const BrickArgs<T> &a, int kind, int form) {
    if (kind == BRICK_POST)
        brick_post<Box, T, PH, DELTA, MOB, 1>(s, a);
    else if (kind == BRICK_SWEEP)
        brick_form<Box, false, T, PH, DELTA, MOB, 1>(s, a, form);
    else
        brick_form<Box, true, T, PH, DELTA, MOB, 1>(s, a, form);
}

template <typename T, int PH, bool DELTA, bool MOB>
static void brick_launch(hipStream_t s, const BrickArgs<T> &a, int kind, int sweeps, int form) {
    const int n = a.op.lay.n;
    if (!brick_small(n))
        brick_one<BrickBox<8, 8, 8>, T, PH, DELTA, MOB>(s, a, kind, form);
    else if (brick_wide(n))
        brick_two<BrickBox<8, 4, 4>, T, PH, DELTA, MOB>(s, a, kind, sweeps, form);
    else
        brick_two<BrickBox<4, 4, 4>, T, PH, DELTA, MOB>(s, a, kind, sweeps, form);
}

}  // namespace pfc
