// Two full red-black sweeps of a large level in one pass over memory, from
// u_in to u_out (two buffers; colour-split storage).
//
// A workgroup owns an x-y column of PX x PY points and a range of planes and
// walks it in z; a thread owns one x-pair of points, one of each colour, of
// the box or of its halo of four points.  At step p, when the old colour-1
// values of plane p have arrived, the four half-sweeps run as a pipeline:
//     colour 0 (first sweep)  on plane p-1, from old colour 1,
//     colour 1 (first sweep)  on plane p-2, from the first colour 0,
//     colour 0 (second sweep) on plane p-3,
//     colour 1 (second sweep) on plane p-4.
// A point's z-neighbours are its own thread's: the plane above is the value the
// thread formed just before in the same step, the plane below its own LDS slot.
// Only x and y neighbours come from other threads, from the plane those formed
// a step earlier.  So a half-sweep's values live in two LDS planes, a step has
// one barrier, and nothing else is kept: the slot a value is written to is the
// one whose old value the same thread has just taken as its lower neighbour.
// A point at face-step distance d from the box (in x, y and z) takes part in
// the half-sweeps that the box can see at that distance, 3, 2, 1, 0 in turn.
// Values are formed by the half-sweeps' functions in their order, so results
// are those of four half-sweep launches bit for bit.
//
// Why: a sweep is bound by memory (64 B per point against 65 operations), and
// two in one pass move 64 B per point once.  What is left above that are the
// halo's second reads, which the L2 catches in part: the box is as large as the
// LDS admits (141 of 160 KB; 32 x 16 boxes, two workgroups per CU, take 350 us at
// 256^3 for the 301 of 64 x 16; the ensembles' levels need them), a workgroup runs fourteen waves, and
// the inputs stay in registers between the sweeps (122-128 VGPRs; without the
// coefficients in scalar registers they spill).  Two sweeps, two fused sweeps ->
// this: 512^3 3.9 -> 2.4 ms, 256^3 479 -> 297 us, 192^3 195 -> 138, 128^3 54 -> 50
// (halo planes: half of the steps); FP32 at 256^3 327 (half-sweeps) -> 252.  The
// FP32 pair is bound by its FP64 arithmetic (VALU 68% busy), so its LDS planes hold
// the rounded values as FP64, converted once by their writer and not by each
// reader (259 -> 252 us; the LDS has the room).
//
// Variable mobility: phi* rides along as a fourth field (read only) and the mu sum
// becomes the face-mobility sum of the flux form.  Four fields of the wide box do
// not fit the LDS, so its box is 32 x 16 (103 KB, one workgroup of eight waves per
// CU, 144-160 VGPRs).  Two fused sweeps -> this: 256^3 654 -> 484 us, 192^3 367 ->
// 242, 128^3 84 -> 76.
#pragma once

#include "device_common.h"
#include "smooth.h"

namespace pfc {

constexpr int kPH = 4;  // halo

template <int PX, int PY, int TH>
struct PairGeo {
    static constexpr int kX = PX, kY = PY, kThreads = TH;  // box, threads
    static constexpr int kW = PX / 2 + kPH;                // x-pairs with the halo
    static constexpr int kR = PY + 2 * kPH;                // rows with the halo

    // distance of a local coordinate to the box's extent b
    __host__ __device__ static constexpr int excess(int v, int b) {
        return v < kPH ? kPH - v : (v >= kPH + b ? v - (kPH + b - 1) : 0);
    }
    // The x-pairs by the distance of their nearer point to the box, the box
    // first, so that a half-sweep's idle lanes fill whole waves.
    // Entry: pair | row << 8.
    struct List {
        unsigned short e[TH];
        int n;
    };
    static constexpr List list() {
        List l{};
        for (int d = 0; d <= kPH; ++d)
            for (int r = 0; r < kR; ++r)
                for (int m = 0; m < kW; ++m) {
                    const int a = excess(2 * m, PX), b = excess(2 * m + 1, PX);
                    if (excess(r, PY) + (a < b ? a : b) == d) l.e[l.n++] = (unsigned short)(m | r << 8);
                }
        for (int i = l.n; i < TH; ++i) l.e[i] = 0xffff;
        return l;
    }
    // LDS planes of the values a half-sweep reads: old colour 1, colour 0 and
    // colour 1 of the first sweep, colour 0 of the second.  Buffer B holds the
    // points up to distance 4 - B.
    template <int B>
    struct Buf {
        static constexpr int X = B / 2, Y = B;  // first pair, first row
        static constexpr int W = kW - 2 * X, R = kR - 2 * Y;
        static constexpr int N = W * R;  // of one field and plane
    };
    static constexpr int lds(int fields) {  // doubles
        return 2 * fields * (Buf<0>::N + Buf<1>::N + Buf<2>::N + Buf<3>::N);
    }
};
using PairWide = PairGeo<64, 16, 896>;   // one workgroup per CU
using PairSmall = PairGeo<32, 16, 512>;  // two

template <typename G>
__device__ constexpr typename G::List kPairList = G::list();

// One buffer as a thread sees it: its own slot and its neighbours'.
template <typename P, int NF>
struct PairSlot {
    double *q;  // own x-pair, field 0, plane slot 0
    __device__ __forceinline__ double *at(int slot) const { return q + slot * NF * P::N; }
    __device__ __forceinline__ void put(int slot, const double (&v)[NF]) const {
        double *w = at(slot);
#pragma unroll
        for (int fl = 0; fl < NF; ++fl) w[fl * P::N] = v[fl];
    }
    __device__ __forceinline__ void get(int slot, double (&v)[NF]) const {
        const double *w = at(slot);
#pragma unroll
        for (int fl = 0; fl < NF; ++fl) v[fl] = w[fl * P::N];
    }
    // neighbour sums of the three fields: x and y from the plane in `slot`, z
    // given; s: x parity of the point
    __device__ __forceinline__ void sums(int slot, int s, const double (&zp)[NF], const double (&zm)[NF],
                                         double (&out)[3]) const {
        const double *w = at(slot);
        const double *wx = w + (s ? 1 : -1);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl)
            out[fl] = (w[fl * P::N] + wx[fl * P::N]) +
                      (w[fl * P::N + P::W] + w[fl * P::N - P::W]) +
                      (zp[fl] + zm[fl]);
    }
    // mobilities of the point's faces xp, xm, yp, ym, zp, zm (phi*: field 3; own
    // value pc) and mu beyond them
    __device__ __forceinline__ void faces(int slot, int s, const double (&zp)[NF], const double (&zm)[NF],
                                          const Mobility &mob, double pc, double (&mf)[6],
                                          double (&mu)[6]) const {
        const double *w = at(slot) + P::N;  // mu
        const double *xp = w + (s ? 1 : 0), *xm = w + (s ? 0 : -1);
        constexpr int ph = (NF - 2) * P::N;  // from mu to phi*
        const double p[6] = {xp[ph], xm[ph], w[ph + P::W], w[ph - P::W], zp[NF - 1], zm[NF - 1]};
        mu[0] = xp[0];
        mu[1] = xm[0];
        mu[2] = w[P::W];
        mu[3] = w[-P::W];
        mu[4] = zp[1];
        mu[5] = zm[1];
#pragma unroll
        for (int e = 0; e < 6; ++e) mf[e] = face_mob(mob, pc, p[e]);
    }
};

// NRM: as the fused sweep's, half of the stop-test norm: 1 over the colour-0 points of the input (formed with the
// first half-sweep's neighbour sums), 2 over the colour-1 points of the output
// (with the last one's).  PK1: f.a is phi^k itself, loaded once.
// One workgroup's column: the box at (x0, y0), px points wide (the whole box or
// its left part), planes [z0, z1).  Returns the thread's share of the norm.
template <typename G, typename T, bool DELTA, bool MOB, int NRM, bool PK1>
__device__ __forceinline__ unsigned long long pair_column(const PairArgs<T> &a, int x0, int y0, int px,
                                                          int z0, int z1, double *lds) {
    static_assert(!(MOB && DELTA), "M = 1 in the FP32 cycle");
    constexpr int NF = MOB ? 4 : 3;  // phi, mu, omega (, phi*: rides along unchanged)
    constexpr int NI = (PK1 ? 3 : 4) + (DELTA ? 1 : 0);  // phi^k, f2, f3 (, f1) (, base)
    const int n = a.op.lay.n, hn = n >> 1;
    const unsigned un = (unsigned)n, uhn = (unsigned)hn, plane = un * uhn, H = un * plane;
    const unsigned e = kPairList<G>.e[threadIdx.x];
    const bool act = e != 0xffffu;
    const int mx = act ? (int)(e & 255u) : kPH, row = act ? (int)(e >> 8) : kPH;
    auto wn = [n](int v) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    const int y = y0 - kPH + row;
    const int m = x0 / 2 - kPH / 2 + mx;
    const unsigned g0 = (unsigned)wn(y) * uhn + (unsigned)(m < 0 ? m + hn : (m >= hn ? m - hn : m));
    // distance to the box in x and y of the pair's two points
    const int d0 = act ? G::excess(row, G::kY) + G::excess(2 * mx, px) : 64;
    const int d1 = act ? G::excess(row, G::kY) + G::excess(2 * mx + 1, px) : 64;
    auto parity = [y](int c, int q) { return (c + y + q) & 1; };
    // steps of the chain left at the point of colour c of plane q
    auto dist = [&](int c, int q) {
        const int dz = q < z0 ? z0 - q : (q >= z1 ? q - z1 + 1 : 0);
        return (parity(c, q) ? d1 : d0) + dz;
    };
    auto gidx = [&](int c, int q) { return (c ? H : 0u) + (unsigned)wn(q) * plane + g0; };

    using B0 = typename G::template Buf<0>;
    using B1 = typename G::template Buf<1>;
    using B2 = typename G::template Buf<2>;
    using B3 = typename G::template Buf<3>;
    double *const l0 = lds, *const l1 = l0 + 2 * NF * B0::N, *const l2 = l1 + 2 * NF * B1::N,
            *const l3 = l2 + 2 * NF * B2::N;
    // A thread whose pair lies outside a buffer never touches it: clamp its slot
    auto own = [&](auto buf, double *l) {
        using P = decltype(buf);
        const int r = min(max(row - P::Y, 0), P::R - 1), c = min(max(mx - P::X, 0), P::W - 1);
        return l + r * P::W + c;
    };
    const PairSlot<B0, NF> o1{own(B0{}, l0)};  // old colour 1
    const PairSlot<B1, NF> a0{own(B1{}, l1)};  // first sweep
    const PairSlot<B2, NF> a1{own(B2{}, l2)};
    const PairSlot<B3, NF> b0{own(B3{}, l3)};  // second sweep, colour 0

    PointCoef co(a.op);
    co.to_scalar();
    T c1n[NF];             // old colour 1 of the next plane
    T phin[NF];            // old phi (NRM = 1: mu, omega; phi*) of the next colour-0 point
    T in0[4][NI], in1[4][NI];  // inputs of colour 0 at planes p, p-1 .. p-3, of colour 1 a plane lower
    auto load_in = [&](int c, int q, T (&v)[NI]) {
        const unsigned g = gidx(c, q);
        v[0] = a.phk[g];
        v[1] = a.f.b[g];
        v[2] = a.f.c[g];
        if constexpr (!PK1) v[3] = a.f.a[g];
        if constexpr (DELTA) v[NI - 1] = a.base[g];
    };
    auto load_c1 = [&](int q) {
        if (dist(1, q) <= 4) {
            const unsigned g = gidx(1, q);
            c1n[0] = a.u.a[g];
            c1n[1] = a.u.b[g];
            c1n[2] = a.u.c[g];
            if constexpr (MOB) c1n[3] = a.op.mob.phs[g];
        }
    };
    auto load_points = [&](int p) {  // what step p + 1 relaxes first: colour 0 of p, colour 1 of p - 1
        const int d = dist(0, p);
        if (d <= 3) {
            const unsigned g = gidx(0, p);
            phin[0] = a.u.a[g];
            if constexpr (MOB) phin[3] = a.op.mob.phs[g];
            if (NRM == 1 && d == 0) {
                phin[1] = a.u.b[g];
                phin[2] = a.u.c[g];
            }
            load_in(0, p, in0[0]);
        }
        if (dist(1, p - 1) <= 2) load_in(1, p - 1, in1[0]);
    };
    // one point of a half-sweep: old phi ph, inputs v, neighbours in the plane `slot`
    // of buf and zp, zm, own phi* pc; before and after see the sums and faces
    auto relax = [&](const auto &buf, int slot, int s, const double (&zp)[NF], const double (&zm)[NF],
                     double ph, double pc, const T (&v)[NI], double (&o)[NF], auto &&before, auto &&after) {
        double sm[3], mf[6], mu[6], x, y2, w;
        buf.sums(slot, s, zp, zm, sm);
        if constexpr (MOB) buf.faces(slot, s, zp, zm, a.op.mob, pc, mf, mu);
        before(sm, mf, mu);
        if constexpr (MOB) {
            double msum = 0.0, smm = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                msum += mf[e];
                smm += mf[e] * mu[e];
            }
            point_solve_mob(a.op, a.picard, ph, (double)v[0], (double)(PK1 ? v[0] : v[3]), (double)v[1],
                            (double)v[2], msum, smm, sm[2], sm[0], x, y2, w);
            o[NF - 1] = pc;
        } else {
            point_solve<DELTA>(co, a.picard, ph, (double)v[0], DELTA ? (double)v[NI - 1] : 0.0,
                               (double)(PK1 ? v[0] : v[3]), (double)v[1], (double)v[2], sm[1], sm[2],
                               sm[0], x, y2, w);
        }
        o[0] = (T)x;  // rounded to the level's type
        o[1] = (T)y2;
        o[2] = (T)w;
        after(sm, mf, mu);
    };
    auto none = [](const double (&)[3], const double (&)[6], const double (&)[6]) {};
    unsigned long long nrm = 0;
    auto norm = [&](const double (&w)[NF], const T (&v)[NI], const double (&s)[3], const double (&mf)[6],
                    const double (&mu)[6]) {
        const double h2inv = a.op.h2inv;
        double ls[3] = {(s[0] - 6.0 * w[0]) * h2inv, (s[1] - 6.0 * w[1]) * h2inv, (s[2] - 6.0 * w[2]) * h2inv};
        if constexpr (MOB) {  // flux form
            double f6 = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e) f6 += mf[e] * (mu[e] - w[1]);
            ls[1] = f6 * h2inv;
        }
        double r[3];
        resid_from_lap<false>(a.op, ls, w[0], w[1], w[2],
                              (double)(PK1 ? v[0] : v[3]), (double)v[1], (double)v[2], (double)v[0], 0.0, r);
        nrm = umax(nrm, umax(abs_bits(r[0]), umax(abs_bits(r[1]), abs_bits(r[2]))));
    };
    auto store = [&](int c, int q, const double (&v)[NF], bool all) {
        const unsigned g = gidx(c, q);
        if (a.stream) {
            __builtin_nontemporal_store((T)v[0], &a.o.a[g]);
            if (all) {
                __builtin_nontemporal_store((T)v[1], &a.o.b[g]);
                __builtin_nontemporal_store((T)v[2], &a.o.c[g]);
            }
        } else {
            a.o.a[g] = (T)v[0];
            if (all) {
                a.o.b[g] = (T)v[1];
                a.o.c[g] = (T)v[2];
            }
        }
    };

    load_c1(z0 - 4);
    for (int p = z0 - 4; p <= z1 + 3; ++p) {
        const int k = p & 1;  // LDS slot of planes p, p-2, p-4
        // a value's lower z-neighbour is taken from the slot it replaces
        double c1[NF], lo[NF], v[NF], w[NF], w0[NF];
#pragma unroll
        for (int fl = 0; fl < NF; ++fl) w0[fl] = phin[fl];
        o1.get(k, lo);  // old colour 1, plane p-2
        if (dist(1, p) <= 4) {
#pragma unroll
            for (int fl = 0; fl < NF; ++fl) c1[fl] = c1n[fl];
            o1.put(k, c1);
        }
#pragma unroll
        for (int i = 3; i > 0; --i)
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                in0[i][t] = in0[i - 1][t];
                in1[i][t] = in1[i - 1][t];
            }
        load_c1(p + 1);
        load_points(p);
        const int da = dist(0, p - 1), db = dist(1, p - 2), dc = dist(0, p - 3), dd = dist(1, p - 4);
        double old = lo[0], own = lo[NF - 1];  // old phi (MOB: phi*) of the next half-sweep's point
        if (da <= 3)
            relax(o1, k ^ 1, parity(0, p - 1), c1, lo, w0[0], w0[NF - 1], in0[1], v,
                  [&](const double (&s)[3], const double (&mf)[6], const double (&mu)[6]) {
                      if constexpr (NRM == 1)
                          if (da == 0) norm(w0, in0[1], s, mf, mu);
                  }, none);
        a0.get(k ^ 1, lo);  // colour 0, plane p-3
        if (da <= 3) a0.put(k ^ 1, v);
        if (db <= 2) relax(a0, k, parity(1, p - 2), v, lo, old, own, in1[1], w, none, none);
        old = lo[0];
        own = lo[NF - 1];
        a1.get(k, lo);  // colour 1, plane p-4
        if (db <= 2) a1.put(k, w);
        if (dc <= 1) {
            relax(a1, k ^ 1, parity(0, p - 3), w, lo, old, own, in0[3], v, none, none);
            if (dc == 0) store(0, p - 3, v, !a.skip0);
        }
        old = lo[0];
        own = lo[NF - 1];
        b0.get(k ^ 1, lo);  // second colour 0, plane p-5
        if (dc <= 1) b0.put(k ^ 1, v);
        if (dd <= 0) {
            relax(b0, k, parity(1, p - 4), v, lo, old, own, in1[3], w, none,
                  [&](const double (&s)[3], const double (&mf)[6], const double (&mu)[6]) {
                      if constexpr (NRM == 2) norm(w, in1[3], s, mf, mu);
                  });
            store(1, p - 4, w, true);
        }
        __syncthreads();
    }
    return nrm;
}

}  // namespace pfc
