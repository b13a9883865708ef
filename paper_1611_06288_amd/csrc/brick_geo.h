// Geometry of the brick kernels (brick.hip): a workgroup owns a BX x BY x BZ
// box of grid points and works on it plus a halo of H points.  A value that
// is D half-sweeps (or stencil applications) away from the box can be reached
// from it only through points at most D face steps away, so the halo's points
// are listed by their face-step distance d to the box and each stage works on
// a prefix of the list: 3472 of the 18^3 = 5832 points for an 8^3 box and H = 5.
#pragma once

#include <hip/hip_runtime.h>

namespace pfc {

template <int BX, int BY, int BZ, int H>
struct BrickGeo {
    static constexpr int EX = BX + 2 * H, EY = BY + 2 * H, EZ = BZ + 2 * H;
    static constexpr int HX = EX / 2;       // points of one colour per row
    static constexpr int HC = HX * EY * EZ;  // storage of one colour of one field
    static_assert(EX % 2 == 0 && BX % 2 == 0 && BY % 2 == 0 && BZ % 2 == 0, "whole pairs");

    static constexpr int excess(int v, int b) { return v < H ? H - v : (v >= H + b ? v - (H + b - 1) : 0); }
    static constexpr int dist(int x, int y, int z) {
        return excess(x, BX) + excess(y, BY) + excess(z, BZ);
    }
    // colour of a local point: boxes start at even coordinates
    static constexpr int colour(int x, int y, int z) { return (x + y + z + H) & 1; }

    struct Count {
        int n[2][H + 1];  // points of colour c with distance <= d
    };
    static constexpr Count count() {
        Count r{};
        for (int z = 0; z < EZ; ++z)
            for (int y = 0; y < EY; ++y)
                for (int x = 0; x < EX; ++x) {
                    const int d = dist(x, y, z);
                    if (d <= H) ++r.n[colour(x, y, z)][d];
                }
        for (int c = 0; c < 2; ++c)
            for (int d = 1; d <= H; ++d) r.n[c][d] += r.n[c][d - 1];
        return r;
    }
    static constexpr Count kCount = count();
    static constexpr int cnt(int c, int d) { return kCount.n[c][d]; }

    // The points of colour C with distance <= D as x | y << 8 | z << 16 | d << 24,
    // whole rows in y and x of one plane after the other, from the box's planes
    // outwards: a wave's lanes then load row segments, the box's points come
    // first, and the waves that a later stage does not need are the last ones.
    // (Sorted by distance instead, a row's ends land in other waves than its
    // middle: 38.5 against 33.3 us for a 64^3 level in 8^3 boxes with H = 5.)
    template <int C, int D>
    struct Rows {
        unsigned p[cnt(C, D)];
    };
    template <int C, int D>
    static constexpr Rows<C, D> rows() {
        Rows<C, D> r{};
        int at = 0;
        for (int k = 0; k < EZ; ++k) {
            // planes H .. H + BZ - 1, then H - 1, H + BZ, H - 2, ...
            const int z = k < BZ ? H + k : ((k - BZ) & 1) ? H + BZ + (k - BZ) / 2 : H - 1 - (k - BZ) / 2;
            for (int y = 0; y < EY; ++y)
                for (int x = 0; x < EX; ++x) {
                    const int d = dist(x, y, z);
                    if (d <= D && colour(x, y, z) == C)
                        r.p[at++] = (unsigned)(x | y << 8 | z << 16 | d << 24);
                }
        }
        return r;
    }
    // position of the last box point in Rows<C, D>, plus one
    template <int C, int D>
    static constexpr int box_end() {
        const Rows<C, D> r = rows<C, D>();
        int e = 0;
        for (int i = 0; i < cnt(C, D); ++i)
            if ((r.p[i] >> 24) == 0) e = i + 1;
        return e;
    }
};

template <typename G, int C, int D>
__device__ constexpr typename G::template Rows<C, D> kBrickRows = G::template rows<C, D>();

}  // namespace pfc
