// Two red-black sweeps per launch on large levels (sweep_pair.h).
#include "sweep_pair.h"

#include <algorithm>
#include <type_traits>

namespace pfc {

template <typename G, typename T, bool DELTA, bool MOB, int NRM, bool PK1>
__global__ __launch_bounds__(G::kThreads, MOB ? 2 : 4) void k_sweep_pair(PairArgs<T> a) {
    __shared__ double lds[G::lds(MOB ? 4 : 3)];
    __shared__ unsigned long long wmax[G::kThreads / 64];
    if (gate_closed(a.op.gate)) return;
    const int n = a.op.lay.n, nbx = n / G::kX, nby = n / G::kY;
    const int b = (int)xcd_block(), bz = b / (nbx * nby);
    unsigned long long nrm = pair_column<G, T, DELTA, MOB, NRM, PK1>(
        a, b % nbx * G::kX, b / nbx % nby * G::kY, G::kX, bz * n / a.nz, (bz + 1) * n / a.nz, lds);
    if constexpr (NRM != 0) {
        nrm = block_max_u64_waves(nrm, wmax);
        if (threadIdx.x == 0) a.part[blockIdx.x] = nrm;
    }
}

bool pair_fits(int n, bool fp32) {
    return n >= (fp32 ? kPairMinN32 : kPairMinN) && n % PairWide::kX == 0 && n % PairWide::kY == 0;
}

// The level's u, f and phi^k do not stay in the 256 MB last-level cache from one
// launch to the next, so the stores leave the caches to the halo's second reads:
// 256^3 pair 300 -> 295 us, 192^3 139.5 -> 138.  At 128^3 they do (plain stores:
// the next launch reads them there; 50 against 54 us with the norm half).
template <typename T>
static int pair_stream(int n) {
    return 9.0 * sizeof(T) * n * n * n > 256e6;
}

int pair_slots(int device, int form) {
    int occ = 0, cus = 0;
    const void *fn = form == PAIR_FP32 ? (const void *)k_sweep_pair<PairWide, float, true, false, 0, false>
                     : form == PAIR_MOB
                         ? (const void *)k_sweep_pair<PairSmall, double, false, true, 0, true>
                         : (const void *)k_sweep_pair<PairWide, double, false, false, 0, true>;
    const int th = form == PAIR_MOB ? PairSmall::kThreads : PairWide::kThreads;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, th, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return 0;
    return occ * cus;
}

static int pair_cols(int n, int form) {
    return form == PAIR_MOB ? (n / PairSmall::kX) * (n / PairSmall::kY) : (n / PairWide::kX) * (n / PairWide::kY);
}

// Plane ranges per column: the fewest waves of resident workgroups times the
// steps of one, a range's eight halo planes counted as five (the points in them
// thin out).
int pair_nz(int n, int slots, int form) {
    const int cols = pair_cols(n, form);
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

int pair_blocks(int n, int nz, int form) { return pair_cols(n, form) * nz; }


void launch_sweep_pair64(hipStream_t s, const OpParams &op, int picard, int nz, Tri<const double> uin,
                         Tri<double> uout, Tri<const double> f, const double *phk, int nrm,
                         unsigned long long *part, bool skip0) {
    PairArgs<double> a{op, picard, nz, skip0 ? 1 : 0, pair_stream<double>(op.lay.n), uin, f, uout, phk, nullptr, part};
    const bool mob = op.mob.phs != nullptr;
    const dim3 grid((unsigned)pair_blocks(op.lay.n, nz, mob ? PAIR_MOB : PAIR_FP64));
    auto go = [&](auto kernel, int threads) { hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, a); };
    auto forms = [&](auto geo, auto m) {
        using G = decltype(geo);
        constexpr bool M = decltype(m)::value;
        // the norm halves belong to a time step's finest level, whose f.a is phk
        if (f.a != phk)
            go(k_sweep_pair<G, double, false, M, 0, false>, G::kThreads);
        else if (nrm == 1)
            go(k_sweep_pair<G, double, false, M, 1, true>, G::kThreads);
        else if (nrm == 2)
            go(k_sweep_pair<G, double, false, M, 2, true>, G::kThreads);
        else
            go(k_sweep_pair<G, double, false, M, 0, true>, G::kThreads);
    };
    if (mob)
        forms(PairSmall{}, std::true_type{});
    else
        forms(PairWide{}, std::false_type{});
}

void launch_sweep_pair32(hipStream_t s, const OpParams &op, int nz, Tri<const float> ein, Tri<float> eout,
                         Tri<const float> f, const float *phk, const float *base, bool skip0) {
    PairArgs<float> a{op, 0, nz, skip0 ? 1 : 0, pair_stream<float>(op.lay.n), ein, f, eout, phk, base, nullptr};
    hipLaunchKernelGGL((k_sweep_pair<PairWide, float, true, false, 0, false>),
                       dim3((unsigned)pair_blocks(op.lay.n, nz, PAIR_FP32)),
                       dim3(PairWide::kThreads), 0, s, a);
}

// ---------------------------------------------------------- batched form

template <int NRM>
__global__ __launch_bounds__(PairSmall::kThreads, 4) void kb_sweep_pair(
    const PairArgs<double> *__restrict__ segs, const PairTile *__restrict__ tiles,
    unsigned long long *__restrict__ part) {
    using G = PairSmall;
    __shared__ double lds[G::lds(3)];
    __shared__ unsigned long long wmax[G::kThreads / 64];
    const PairTile t = tiles[blockIdx.x];
    const PairArgs<double> a = segs[t.seg];
    if (gate_closed(a.op.gate)) return;
    unsigned long long nrm = pair_column<G, double, false, false, NRM, true>(a, t.x0, t.y0, t.px, t.z0, t.z1, lds);
    nrm = block_max_u64_waves(nrm, wmax);
    if (threadIdx.x == 0) part[t.slot] = nrm;
}

bool batch_pair_fits(int n) { return n >= PairSmall::kX && n % PairSmall::kY == 0; }

int batch_pair_slots(int device) {
    int occ = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void *)kb_sweep_pair<1>,
                                                     PairSmall::kThreads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return 0;
    return occ * cus;
}

std::vector<PairTile> batch_pair_tiles(int n, int zmax) {
    using G = PairSmall;
    const int nz = (n + zmax - 1) / zmax;
    std::vector<PairTile> v;
    for (int z = 0; z < nz; ++z)
        for (int y0 = 0; y0 < n; y0 += G::kY)
            for (int x0 = 0; x0 < n; x0 += G::kX)
                v.push_back(PairTile{0, x0, y0, std::min(G::kX, n - x0), z * n / nz, (z + 1) * n / nz, 0, 0});
    return v;
}

void launch_batch_pair(hipStream_t s, int nrm, const PairArgs<double> *segs, const PairTile *tiles,
                       int ntiles, unsigned long long *part) {
    if (nrm == 1)
        hipLaunchKernelGGL(kb_sweep_pair<1>, dim3(ntiles), dim3(PairSmall::kThreads), 0, s, segs, tiles, part);
    else
        hipLaunchKernelGGL(kb_sweep_pair<2>, dim3(ntiles), dim3(PairSmall::kThreads), 0, s, segs, tiles, part);
}

}  // namespace pfc
