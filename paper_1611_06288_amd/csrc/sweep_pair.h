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
// LDS admits (141 of 160 KB in FP64; 32 x 16 boxes, two workgroups per CU, take
// 350 us at 256^3 for the 301 of 64 x 16), a workgroup runs fourteen waves, and
// the inputs stay in registers between the sweeps (122-128 VGPRs; without the
// coefficients in scalar registers they spill).  Two sweeps, two fused sweeps ->
// this: 512^3 3.9 -> 2.4 ms, 256^3 479 -> 297 us, 192^3 195 -> 138, 128^3 54 -> 50
// (halo planes: half of the steps); FP32 at 256^3 327 (half-sweeps) -> 252.  The
// FP32 pair is bound by its FP64 arithmetic (VALU 68% busy), so its LDS planes hold
// the rounded values as FP64, converted once by their writer and not by each
// reader (259 -> 252 us; the LDS has the room).
#pragma once

#include "device_common.h"
#include "smooth.h"

namespace pfc {

constexpr int kPX = 64, kPY = 16;               // box
constexpr int kPH = 4;                          // halo
constexpr int kPW = kPX / 2 + kPH;              // x-pairs with the halo
constexpr int kPR = kPY + 2 * kPH;              // rows with the halo
constexpr int kPT = 896;                        // threads

// The x-pairs by the distance of their nearer point to the box, the box first,
// so that a half-sweep's idle lanes fill whole waves.  Entry: pair | row << 8.
struct PairList {
    unsigned short e[kPT];
    int n;
};
constexpr int pair_dx(int x) { return x < kPH ? kPH - x : (x >= kPH + kPX ? x - (kPH + kPX - 1) : 0); }
constexpr int pair_dy(int r) { return r < kPH ? kPH - r : (r >= kPH + kPY ? r - (kPH + kPY - 1) : 0); }
constexpr PairList pair_list() {
    PairList l{};
    for (int d = 0; d <= kPH; ++d)
        for (int r = 0; r < kPR; ++r)
            for (int m = 0; m < kPW; ++m) {
                const int a = pair_dx(2 * m), b = pair_dx(2 * m + 1);
                if (pair_dy(r) + (a < b ? a : b) == d) l.e[l.n++] = (unsigned short)(m | r << 8);
            }
    for (int i = l.n; i < kPT; ++i) l.e[i] = 0xffff;
    return l;
}
static_assert(pair_list().n <= kPT, "one thread per x-pair");

// LDS planes of the values a half-sweep reads: old colour 1, colour 0 and
// colour 1 of the first sweep, colour 0 of the second.  Buffer B holds the
// points up to distance 4 - B.
template <int B>
struct PairBuf {
    static constexpr int X = B / 2;               // first pair, first row
    static constexpr int Y = B;
    static constexpr int W = kPW - 2 * X, R = kPR - 2 * Y;
    static constexpr int N = W * R;               // of one field and plane
};
constexpr int kPairLds = 6 * (PairBuf<0>::N + PairBuf<1>::N + PairBuf<2>::N + PairBuf<3>::N);

template <typename T>
struct PairArgs {
    OpParams op;
    int picard = 0, nz = 1, skip0 = 0;
    int stream = 0;  // stores past the caches
    Tri<const T> u, f;
    Tri<T> o;
    const T *phk = nullptr, *base = nullptr;
    unsigned long long *part = nullptr;
};

// One buffer as a thread sees it: its own slot and its neighbours'.
template <int B>
struct PairSlot {
    using P = PairBuf<B>;
    double *q;  // own x-pair, field 0, plane slot 0
    __device__ __forceinline__ double *at(int slot) const { return q + slot * 3 * P::N; }
    __device__ __forceinline__ void put(int slot, const double (&v)[3]) const {
        double *w = at(slot);
        w[0] = v[0];
        w[P::N] = v[1];
        w[2 * P::N] = v[2];
    }
    __device__ __forceinline__ void get(int slot, double (&v)[3]) const {
        const double *w = at(slot);
        v[0] = w[0];
        v[1] = w[P::N];
        v[2] = w[2 * P::N];
    }
    // neighbour sums of the three fields: x and y from the plane in `slot`, z
    // given; s: x parity of the point
    __device__ __forceinline__ void sums(int slot, int s, const double (&zp)[3], const double (&zm)[3],
                                         double (&out)[3]) const {
        const double *w = at(slot);
        const double *wx = w + (s ? 1 : -1);
#pragma unroll
        for (int fl = 0; fl < 3; ++fl)
            out[fl] = (w[fl * P::N] + wx[fl * P::N]) +
                      (w[fl * P::N + P::W] + w[fl * P::N - P::W]) +
                      (zp[fl] + zm[fl]);
    }
};

}  // namespace pfc
