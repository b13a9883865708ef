// Two red-black sweeps per launch on large levels (sweep_pair.h).
#include "sweep_pair.h"

#include <algorithm>

namespace pfc {

__device__ constexpr PairList kPairList = pair_list();

// NRM: as the fused sweep's, half of the stop-test norm as per-workgroup maxima
// in part[blockIdx.x]: 1 over the colour-0 points of the input (formed with the
// first half-sweep's neighbour sums), 2 over the colour-1 points of the output
// (with the last one's).  PK1: f.a is phi^k itself, loaded once.
template <typename T, bool DELTA, int NRM, bool PK1>
__global__ __launch_bounds__(kPT, 4) void k_sweep_pair(PairArgs<T> a) {
    __shared__ double lds[kPairLds];
    __shared__ unsigned long long wmax[kPT / 64];
    if (gate_closed(a.op.gate)) return;
    constexpr int NI = (PK1 ? 3 : 4) + (DELTA ? 1 : 0);  // phi^k, f2, f3 (, f1) (, base)
    const int n = a.op.lay.n, hn = n >> 1;
    const unsigned un = (unsigned)n, uhn = (unsigned)hn, plane = un * uhn, H = un * plane;
    const int nbx = n / kPX, nby = n / kPY;
    const int b = (int)xcd_block();
    const int x0 = b % nbx * kPX, y0 = b / nbx % nby * kPY, bz = b / (nbx * nby);
    const int z0 = bz * n / a.nz, z1 = (bz + 1) * n / a.nz;
    const unsigned e = kPairList.e[threadIdx.x];
    const bool act = e != 0xffffu;
    const int mx = act ? (int)(e & 255u) : kPH, row = act ? (int)(e >> 8) : kPH;
    auto wn = [n](int v) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    const int y = y0 - kPH + row;
    const int m = x0 / 2 - kPH / 2 + mx;
    const unsigned g0 = (unsigned)wn(y) * uhn + (unsigned)(m < 0 ? m + hn : (m >= hn ? m - hn : m));
    // distance to the box in x and y of the pair's two points
    const int d0 = act ? pair_dy(row) + pair_dx(2 * mx) : 64;
    const int d1 = act ? pair_dy(row) + pair_dx(2 * mx + 1) : 64;
    auto parity = [y](int c, int q) { return (c + y + q) & 1; };
    // steps of the chain left at the point of colour c of plane q
    auto dist = [&](int c, int q) {
        const int dz = q < z0 ? z0 - q : (q >= z1 ? q - z1 + 1 : 0);
        return (parity(c, q) ? d1 : d0) + dz;
    };
    auto gidx = [&](int c, int q) { return (c ? H : 0u) + (unsigned)wn(q) * plane + g0; };

    double *const l0 = lds, *const l1 = l0 + 6 * PairBuf<0>::N, *const l2 = l1 + 6 * PairBuf<1>::N,
            *const l3 = l2 + 6 * PairBuf<2>::N;
    // A thread whose pair lies outside a buffer never touches it: clamp its slot
    auto own = [&](auto buf, double *l) {
        using P = decltype(buf);
        const int r = min(max(row - P::Y, 0), P::R - 1), c = min(max(mx - P::X, 0), P::W - 1);
        return l + r * P::W + c;
    };
    const PairSlot<0> o1{own(PairBuf<0>{}, l0)};  // old colour 1
    const PairSlot<1> a0{own(PairBuf<1>{}, l1)};  // first sweep
    const PairSlot<2> a1{own(PairBuf<2>{}, l2)};
    const PairSlot<3> b0{own(PairBuf<3>{}, l3)};  // second sweep, colour 0

    PointCoef co(a.op);
    co.to_scalar();
    T c1n[3];              // old colour 1 of the next plane
    T phin[3];             // old phi (NRM = 1: mu, omega) of the next colour-0 point
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
        }
    };
    auto load_points = [&](int p) {  // what step p + 1 relaxes first: colour 0 of p, colour 1 of p - 1
        const int d = dist(0, p);
        if (d <= 3) {
            const unsigned g = gidx(0, p);
            phin[0] = a.u.a[g];
            if (NRM == 1 && d == 0) {
                phin[1] = a.u.b[g];
                phin[2] = a.u.c[g];
            }
            load_in(0, p, in0[0]);
        }
        if (dist(1, p - 1) <= 2) load_in(1, p - 1, in1[0]);
    };
    auto solve = [&](double ph, const T (&v)[NI], const double (&s)[3], double (&o)[3]) {
        double x, y2, w;
        point_solve<DELTA>(co, a.picard, ph, (double)v[0], DELTA ? (double)v[NI - 1] : 0.0,
                           (double)(PK1 ? v[0] : v[3]), (double)v[1], (double)v[2], s[1], s[2], s[0], x,
                           y2, w);
        o[0] = (T)x;  // rounded to the level's type
        o[1] = (T)y2;
        o[2] = (T)w;
    };
    unsigned long long nrm = 0;
    auto norm = [&](const double (&w)[3], const T (&v)[NI], const double (&s)[3]) {
        const double h2inv = a.op.h2inv;
        const double ls[3] = {(s[0] - 6.0 * w[0]) * h2inv, (s[1] - 6.0 * w[1]) * h2inv,
                              (s[2] - 6.0 * w[2]) * h2inv};
        double r[3];
        resid_from_lap<false>(a.op, ls, w[0], w[1], w[2],
                              (double)(PK1 ? v[0] : v[3]), (double)v[1], (double)v[2], (double)v[0], 0.0, r);
        nrm = umax(nrm, umax(abs_bits(r[0]), umax(abs_bits(r[1]), abs_bits(r[2]))));
    };
    auto store = [&](int c, int q, const double (&v)[3], bool all) {
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
        double c1[3], lo[3], v[3], w[3], w0[3] = {phin[0], phin[1], phin[2]};
        o1.get(k, lo);  // old colour 1, plane p-2
        if (dist(1, p) <= 4) {
            c1[0] = c1n[0];
            c1[1] = c1n[1];
            c1[2] = c1n[2];
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
        const double oldb = lo[0];  // old phi of plane p-2
        if (da <= 3) {
            double s[3];
            o1.sums(k ^ 1, parity(0, p - 1), c1, lo, s);
            if constexpr (NRM == 1)
                if (da == 0) norm(w0, in0[1], s);
            solve(w0[0], in0[1], s, v);
        }
        a0.get(k ^ 1, lo);  // colour 0, plane p-3
        if (da <= 3) a0.put(k ^ 1, v);
        const double oldc = lo[0];
        if (db <= 2) {
            double s[3];
            a0.sums(k, parity(1, p - 2), v, lo, s);
            solve(oldb, in1[1], s, w);
        }
        a1.get(k, lo);  // colour 1, plane p-4
        if (db <= 2) a1.put(k, w);
        const double oldd = lo[0];
        if (dc <= 1) {
            double s[3];
            a1.sums(k ^ 1, parity(0, p - 3), w, lo, s);
            solve(oldc, in0[3], s, v);
            if (dc == 0) store(0, p - 3, v, !a.skip0);
        }
        b0.get(k ^ 1, lo);  // second colour 0, plane p-5
        if (dc <= 1) b0.put(k ^ 1, v);
        if (dd <= 0) {
            double s[3];
            b0.sums(k, parity(1, p - 4), v, lo, s);
            solve(oldd, in1[3], s, w);
            if constexpr (NRM == 2) norm(w, in1[3], s);
            store(1, p - 4, w, true);
        }
        __syncthreads();
    }
    if constexpr (NRM != 0) {
        nrm = block_max_u64_waves(nrm, wmax);
        if (threadIdx.x == 0) a.part[blockIdx.x] = nrm;
    }
}

bool pair_fits(int n, bool fp32) {
    return n >= (fp32 ? kPairMinN32 : kPairMinN) && n % kPX == 0 && n % kPY == 0;
}

// The level's u, f and phi^k do not stay in the 256 MB last-level cache from one
// launch to the next, so the stores leave the caches to the halo's second reads:
// 256^3 pair 300 -> 295 us, 192^3 139.5 -> 138.  At 128^3 they do (plain stores:
// the next launch reads them there; 50 against 54 us with the norm half).
template <typename T>
static int pair_stream(int n) {
    return 9.0 * sizeof(T) * n * n * n > 256e6;
}

int pair_slots(int device, bool fp32) {
    int occ = 0, cus = 0;
    const void *fn = fp32 ? (const void *)k_sweep_pair<float, true, 0, false>
                          : (const void *)k_sweep_pair<double, false, 0, true>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, kPT, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return 0;
    return occ * cus;
}

// Plane ranges per column: the fewest waves of resident workgroups times the
// steps of one, a range's eight halo planes counted as five (the points in them
// thin out).
int pair_nz(int n, int slots) {
    const int cols = (n / kPX) * (n / kPY);
    int best = 1;
    long cost = -1;
    for (int nz = 1; nz <= n / 4; ++nz) {
        const int waves = slots > 0 ? (cols * nz + slots - 1) / slots : 1;
        const long c = (long)waves * ((n + nz - 1) / nz + 5);
        if (cost < 0 || c < cost) {
            cost = c;
            best = nz;
        }
    }
    return best;
}

int pair_blocks(int n, int nz) { return (n / kPX) * (n / kPY) * nz; }


void launch_sweep_pair64(hipStream_t s, const OpParams &op, int picard, int nz, Tri<const double> uin,
                         Tri<double> uout, Tri<const double> f, const double *phk, int nrm,
                         unsigned long long *part, bool skip0) {
    PairArgs<double> a{op, picard, nz, skip0 ? 1 : 0, pair_stream<double>(op.lay.n), uin, f, uout, phk, nullptr, part};
    const dim3 grid((unsigned)pair_blocks(op.lay.n, nz));
    // the norm halves belong to a time step's finest level, whose f.a is phk
    if (f.a != phk)
        hipLaunchKernelGGL((k_sweep_pair<double, false, 0, false>), grid, dim3(kPT), 0, s, a);
    else if (nrm == 1)
        hipLaunchKernelGGL((k_sweep_pair<double, false, 1, true>), grid, dim3(kPT), 0, s, a);
    else if (nrm == 2)
        hipLaunchKernelGGL((k_sweep_pair<double, false, 2, true>), grid, dim3(kPT), 0, s, a);
    else
        hipLaunchKernelGGL((k_sweep_pair<double, false, 0, true>), grid, dim3(kPT), 0, s, a);
}

void launch_sweep_pair32(hipStream_t s, const OpParams &op, int nz, Tri<const float> ein, Tri<float> eout,
                         Tri<const float> f, const float *phk, const float *base, bool skip0) {
    PairArgs<float> a{op, 0, nz, skip0 ? 1 : 0, pair_stream<float>(op.lay.n), ein, f, eout, phk, base, nullptr};
    hipLaunchKernelGGL((k_sweep_pair<float, true, 0, false>), dim3((unsigned)pair_blocks(op.lay.n, nz)),
                       dim3(kPT), 0, s, a);
}

}  // namespace pfc
