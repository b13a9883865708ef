// Internal interface between the HIP kernels (kernels.hip) and the host
// runtime.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace pfc {

// Three grid functions (phi, mu, omega) of one level.
template <typename T>
struct Tri {
    T *a;  // phi (or its correction)
    T *b;  // mu
    T *c;  // omega
};

template <typename T>
__host__ __device__ inline Tri<const T> cst(Tri<T> t) { return Tri<const T>{t.a, t.b, t.c}; }

// Division by n = 2^s or 3*2^s without integer divide instructions (by no other n:
// it would divide by a smaller number of that form).
struct Div {
    unsigned shift;  // s
    unsigned three;  // 1 if n = 3*2^s
    __host__ __device__ unsigned q(unsigned x) const {
        x >>= shift;
        return three ? (unsigned)(((unsigned long long)x * 0xAAAAAAABull) >> 33) : x;
    }
};

Div make_div(int d);  // host

// Storage of one level's fields.  Natural: C order [k][j][i].  Colour-split
// (n even): the points of colour c = (i+j+k) mod 2 are stored in block c of
// size n^3/2, row (k, j) by row, a point at position i >> 1 of its row.
struct Lay {
    int n;
    int split;
    Div dn;   // division by n
    Div dh;   // division by n/2 (split only)
};

Lay make_lay(int n, bool split);

inline size_t npts_host(const Lay &L) { return (size_t)L.n * L.n * L.n; }

// Variable mobility M(v) = max(mmin, m0 + m1 v + m2 v^2) of the first
// equation's flux form, evaluated on each face at the face average of phi*
// (phi* in the level's layout; null: M = 1).
struct Mobility {
    const double *phs = nullptr;
    double m0 = 1.0, m1 = 0.0, m2 = 0.0, mmin = 0.0;
};

// Scalar parameters of one level's operator.
struct OpParams {
    Lay lay;
    double h2inv;  // 1 / h_l^2
    double tau;    // time step
    double eps;    // epsilon
    // 1: the first-order convex-splitting scheme (N2 with phi^3 and (1-eps)
    // phi, N3 = omega - Lap phi); 0: the second-order scheme of Section 5
    int fo = 0;
    Mobility mob{};
    // Cycle gate (time loop replayed as a graph): when set and *gate == 0 the
    // cycle's kernels return at once, so cycles after convergence do nothing.
    const int *gate = nullptr;
};

constexpr int kBlock = 256;
constexpr int kMaxReduceBlocks = 16384;
constexpr int kMaxN = 1024;

// ---- building blocks; T = double or float, DELTA selects the correction
// form g(base + e) - g(base) of the cubic term ----
template <typename T, bool DELTA>
void launch_smooth(hipStream_t s, const OpParams &op, int colour, int picard, Tri<T> u,
                   Tri<const T> f, const T *phk, const T *base);

// The first half-sweep of colour `colour` on a coarse level whose iterate
// starts at I u (ubar), forming the tau correction f += N(I u) at that
// colour's points as it smooths (f holds I r on entry, I u is not copied into
// u); two calls (colour 0, then 1) equal launch_tau followed by two
// launch_smooth calls bit for bit.
template <typename T, bool DELTA>
void launch_smooth_tau(hipStream_t s, const OpParams &op, int colour, int picard, Tri<T> u,
                       Tri<T> f, Tri<const T> ubar, const T *phk, const T *base);

// One full red-black sweep in place on a level of at most kSmallSweepN^3
// points, by a single workgroup (colour 0, barrier, colour 1).  Measured:
// 3.8 us against two 2.3 us launches at 8^3, but 14 us against two 3.3 us
// launches at 16^3 (one CU then carries too much latency-bound work).
constexpr int kSmallSweepN = 8;
template <typename T, bool DELTA>
void launch_sweep_small(hipStream_t s, const OpParams &op, int picard, Tri<T> u, Tri<const T> f,
                        const T *phk, const T *base);
// The same as the first sweep of a coarse level, forming the tau correction
// (as launch_smooth_tau).
template <typename T, bool DELTA>
void launch_sweep_small_tau(hipStream_t s, const OpParams &op, int picard, Tri<T> u, Tri<T> f,
                            Tri<const T> ubar, const T *phk, const T *base);

// One full red-black sweep (colour 0 then colour 1) from uin into uout
// (distinct buffers, colour-split storage), bitwise equal to two launch_smooth
// calls; the level is cut into nz plane ranges (see fused_nz).  Instantiated
// for double only.  nrm (M = 1 only) adds half of the stop-test norm as
// per-workgroup maxima of |S - N(u)| bits in part[0 .. fused_blocks(n, nz)):
// 1 over the colour-0 points of uin, 2 over the colour-1 points of uout.
// skip0: mu and omega of colour-0 points are not written to uout (only when
// the next operation on uout is another fused sweep, which does not read them).
template <typename T, bool DELTA>
void launch_sweep_fused(hipStream_t s, const OpParams &op, int picard, int nz, Tri<const T> uin,
                        Tri<T> uout, Tri<const T> f, const T *phk, const T *base, int nrm = 0,
                        unsigned long long *part = nullptr, bool skip0 = false);
int fused_blocks(int n, int nz);  // workgroups of one fused-sweep launch
bool fused_fits(int n);           // n admits the fused sweep's column tiling
int fused_slots(int device, bool mob = false);      // resident fused-sweep workgroups on the device (0 on error)
int fused_nz(int n, int slots);   // plane ranges per column for a level of size n
constexpr int kFusedMinN = 128;  // smaller levels use the half-sweeps

// One level's two sweeps in one pass (sweep_pair.h).
template <typename T>
struct PairArgs {
    OpParams op;
    int picard = 0, nz = 1, skip0 = 0;
    int stream = 0;  // stores past the caches
    Tri<const T> u{nullptr, nullptr, nullptr}, f{nullptr, nullptr, nullptr};
    Tri<T> o{nullptr, nullptr, nullptr};
    const T *phk = nullptr, *base = nullptr;
    unsigned long long *part = nullptr;
};

// Two full red-black sweeps in one pass (sweep_pair.h), bitwise two fused sweeps;
// arguments as launch_sweep_fused.  The level is cut into pair_nz
// plane ranges.
void launch_sweep_pair64(hipStream_t s, const OpParams &op, int picard, int nz, Tri<const double> uin,
                         Tri<double> uout, Tri<const double> f, const double *phk, int nrm = 0,
                         unsigned long long *part = nullptr, bool skip0 = false);
void launch_sweep_pair32(hipStream_t s, const OpParams &op, int nz, Tri<const float> ein, Tri<float> eout,
                         Tri<const float> f, const float *phk, const float *base, bool skip0 = false);
bool pair_fits(int n, bool fp32);
enum { PAIR_FP64 = 0, PAIR_FP32 = 1, PAIR_MOB = 2 };  // forms
int pair_slots(int device, int form);  // resident workgroups on the device (0 on error)
int pair_nz(int n, int slots, int form);
int pair_blocks(int n, int nz, int form);  // workgroups of one launch
// Smallest levels: FP64 at 128^3 two fused sweeps 54-57 us, the pair 50; an FP32
// step of 24 cycles at 128^3 in half-sweeps 5.63 ms, in pairs 5.93, at 192^3 13.8 and
// 14.1 (its operands sit in the last-level cache), at 256^3 29.9 and 26.0.
constexpr int kPairMinN = 128, kPairMinN32 = 256;

// ---- brick launches (brick.h): one level's part of a cycle on either side of
// the descent, for levels of 12^3 to 96^3 ----
enum { BP_FAS = 0, BP_ADJ = 1 };  // the scheme's operator; its adjoint J^T
enum { BRICK_PRE = 0, BRICK_SWEEP = 1, BRICK_POST = 2 };  // kinds
enum { BRICK_PLAIN = 0, BRICK_FIRST = 1, BRICK_NORM = 2 };  // forms of the first two
template <typename T>
struct BrickArgs {
    OpParams op;
    int picard = 0;
    int skip0 = 0;                               // BRICK_SWEEP, BRICK_POST: another sweep follows
    Tri<const T> u{nullptr, nullptr, nullptr};   // iterate (BRICK_FIRST: I u) read
    Tri<T> uo{nullptr, nullptr, nullptr};        // iterate written, another buffer
    Tri<const T> f{nullptr, nullptr, nullptr};   // right-hand side (BRICK_FIRST: I r)
    Tri<T> fo{nullptr, nullptr, nullptr};        // BRICK_FIRST: f + N(I u), another buffer
    const T *phk = nullptr, *base = nullptr;
    Lay LC{};                                    // the next coarser level
    Tri<T> cu{nullptr, nullptr, nullptr}, cr{nullptr, nullptr, nullptr};  // pre: its I u and I r
    Tri<const T> v{nullptr, nullptr, nullptr}, ub{nullptr, nullptr, nullptr};  // post: its iterate, I u
    unsigned long long *part = nullptr;          // BRICK_NORM: per-workgroup max |S - N(u)|
};
// 4^3 boxes with both sweeps of a side in one launch up to 32^3, where a launch
// has CUs to spare; from 48^3 on 8^3 boxes and one sweep per launch, whose
// halos cost less than the launch they would save.
inline bool brick_small(int n) { return n <= 32; }
inline bool batch_brick(int n) { return n <= 16; }  // those of a batch (launch_batch_brick)
inline bool brick_size(int n) { return n >= 12 && n <= 96 && n % (brick_small(n) ? 4 : 8) == 0; }
constexpr int kBrickMaxSweeps = 2;  // sweeps per side of the descent
template <int BX, int BY, int BZ>
struct BrickBox {
    static constexpr int X = BX, Y = BY, Z = BZ;
    static int blocks(int n) { return (n / BX) * (n / BY) * (n / BZ); }
};
// 8 x 4 x 4 boxes where the 4^3 ones are more than the device's CUs, of which then
// some run two and share their cycles (of the levels up to 32^3 that one: 512).
constexpr int kCUs = 256;
inline bool brick_wide(int n) { return n % 8 == 0 && BrickBox<4, 4, 4>::blocks(n) > kCUs; }
inline int brick_blocks(int n) {
    return !brick_small(n) ? BrickBox<8, 8, 8>::blocks(n)
           : brick_wide(n) ? BrickBox<8, 4, 4>::blocks(n)
                           : BrickBox<4, 4, 4>::blocks(n);
}
// sweeps of the launch: 1 or, with small boxes, 2
void launch_brick64(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form);
void launch_brick64_mob(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form);
void launch_brick32(hipStream_t s, const BrickArgs<float> &a, int kind, int sweeps, int form);
void launch_brick_adj(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form);

// The launches of one level with their buffers: u is the iterate between
// cycles, x and y two more.  Before the descent u -> x (-> y), after it back
// to u, so the iterate is never overwritten before the cycle's last launch.
// a: everything but u, uo and skip0; go(args, kind, sweeps, form).
template <typename T>
inline Tri<T> brick_mid(int n, int nu1, Tri<T> x, Tri<T> y) {
    return nu1 == 1 || brick_small(n) ? x : y;
}
template <typename T, typename Go>
inline void brick_run_pre(BrickArgs<T> a, int nu1, Tri<const T> u, Tri<T> x, Tri<T> y, int form, Go go) {
    a.u = u;
    a.uo = x;
    if (nu1 == 1 || brick_small(a.op.lay.n)) return go(a, BRICK_PRE, nu1, form);
    a.skip0 = 1;
    go(a, BRICK_SWEEP, 1, form);
    a.u = cst(x);
    a.uo = y;
    if (form == BRICK_FIRST) a.f = cst(a.fo);
    go(a, BRICK_PRE, 1, BRICK_PLAIN);
}
template <typename T, typename Go>
inline void brick_run_post(BrickArgs<T> a, int nu1, int nu2, Tri<T> u, Tri<T> x, Tri<T> y, Go go) {
    const Tri<T> mid = brick_mid(a.op.lay.n, nu1, x, y);
    a.u = cst(mid);
    a.uo = u;
    if (nu2 == 1 || brick_small(a.op.lay.n)) return go(a, BRICK_POST, nu2, BRICK_PLAIN);
    const Tri<T> other = mid.a == x.a ? y : x;
    a.uo = other;
    a.skip0 = 1;
    go(a, BRICK_POST, 1, BRICK_PLAIN);
    a.u = cst(other);
    a.uo = u;
    a.skip0 = 0;
    go(a, BRICK_SWEEP, 1, BRICK_PLAIN);
}

// Device-side stop test of the time loop: the cycle loop's decision on the
// residual max-norm before a cycle, reduced from the per-workgroup maxima
// partial[0 .. count) (IEEE bit patterns) by the same one-block launch, made
// on the GPU so that a
// replayed graph of cycles needs no host round trip.  active: cycles still
// wanted (the gate of the cycle kernels); cycles: cycles started; status: a
// pfc_status; res0/res: first and latest norm.
// host (may be null): pinned memory that takes the state when a test of an
// active step has decided.
struct RunHost {
    int active, cycles, status, unused;
    double res0, res;
};
struct RunState {
    int *active = nullptr;
    int *cycles = nullptr;
    int *status = nullptr;
    double *res0 = nullptr;
    double *res = nullptr;
    RunHost *host = nullptr;
};
struct StopTest {
    const unsigned long long *partial = nullptr;  // null: no test
    int count = 0, max_cycles = 0;
    double tol = 0.0;
    RunState st{};
};

// ---- the 8^3 (6^3) level and the coarsest below it in one launch (tail.h) ----
template <typename T>
struct TailArgs {
    OpParams op, opc;  // the level, the coarsest level
    int picard = 0, nu1 = 0, nu2 = 0;
    int fcycle = 0;    // an F-cycle followed by a V-cycle, as the cycle above visits the level
    Tri<T> u{nullptr, nullptr, nullptr};         // iterate (written)
    Tri<const T> f{nullptr, nullptr, nullptr}, ub{nullptr, nullptr, nullptr};  // I r, I u
    const T *phk = nullptr, *base = nullptr, *phkc = nullptr, *basec = nullptr;
    const double *lap1 = nullptr, *lap2 = nullptr, *lap3 = nullptr;
    double *minv = nullptr;
    int *valid = nullptr, *iters = nullptr;
    StopTest stop{};  // also takes the loop's decision (everything before it is scratch)
};
inline bool tail_size(int n) { return n == 8 || n == 6; }
void launch_tail64(hipStream_t s, const TailArgs<double> &a);
void launch_tail32(hipStream_t s, const TailArgs<float> &a);
// The adjoint's: f is b, phk and phkc the diagonal D, the iterate starts at zero
// (ub unused).
void launch_tail_adj(hipStream_t s, const TailArgs<double> &a);

// Residual of a large level by z-marching column tiles (residual.hip), with
// one of five epilogues.
enum { RT_NORM = 0, RT_RESTRICT = 1, RT_CAST = 2, RT_CAST_CORR = 3, RT_RESTRICT32 = 4, RT_MODES = 5 };
struct ResidTileArgs {
    // FP64 operator: RT_NORM, RT_RESTRICT, RT_CAST, RT_CAST_CORR
    Tri<const double> u{nullptr, nullptr, nullptr}, f{nullptr, nullptr, nullptr};
    const double *phk = nullptr;
    Tri<double> ubar{nullptr, nullptr, nullptr};  // RT_RESTRICT: I u
    Tri<double> rr{nullptr, nullptr, nullptr};    // RT_RESTRICT: I r
    Tri<float> r32{nullptr, nullptr, nullptr};    // RT_CAST*: r in FP32
    float *base32 = nullptr;                      // RT_CAST*: phi in FP32
    Tri<const float> e{nullptr, nullptr, nullptr};  // RT_CAST_CORR: correction added to u
    Tri<double> uout{nullptr, nullptr, nullptr};    // RT_CAST_CORR: u + e (distinct from u)
    // FP32 correction operator: RT_RESTRICT32
    Tri<const float> e32{nullptr, nullptr, nullptr}, f32{nullptr, nullptr, nullptr};
    const float *phk32 = nullptr, *b32 = nullptr;
    Tri<float> ebar32{nullptr, nullptr, nullptr}, rr32{nullptr, nullptr, nullptr};
    Lay LC{};                               // restrictions: the coarse level
    unsigned long long *partial = nullptr;  // RT_NORM, RT_CAST*: per-workgroup max |r|
};
bool resid_tile_fits(const Lay &L);
// The stop-test norm takes the column tiles from this size on; on a 64^3
// level each column holds a few planes and the thread-per-point norm is
// faster (7 against 11 us), while the restriction keeps the tiles there.
constexpr int kTileNormMinN = 128;
int resid_tile_slots(int device, int mode, bool mob = false);   // resident workgroups (0 on error)
int resid_tile_nz(int n, int slots, int mode);
int launch_resid_tile(hipStream_t s, int mode, const OpParams &op, int nz,
                      const ResidTileArgs &a);  // returns the workgroup count

template <typename T, bool DELTA>
void launch_resid_restrict(hipStream_t s, const OpParams &op, const Lay &coarse, Tri<const T> u,
                           Tri<const T> f, const T *phk, const T *base, Tri<T> ubar_c, Tri<T> rr_c);

template <typename T>
void launch_restrict(hipStream_t s, const Lay &fine, const Lay &coarse, const T *fine_v, T *coarse_v);

template <typename T, bool DELTA>
void launch_tau(hipStream_t s, const OpParams &opc, Tri<const T> ubar, Tri<T> f, Tri<T> u,
                const T *phk, const T *base);

// fine += P (v - ubar); ubar.a may be null; fine.b null: one field only.
// phi0: a smoothing sweep follows, so mu and omega at colour-0 points may be
// left uncorrected (they are dead until the sweep overwrites them); the tiled
// levels skip them, the others correct everything.
template <typename T>
void launch_prolong(hipStream_t s, const Lay &coarse, const Lay &fine, Tri<const T> v,
                    Tri<const T> ubar, Tri<T> fine_u, const int *gate = nullptr,
                    bool phi0 = false, int nzr = 0);
int prolong_tile_slots(int device, bool fp32);  // resident workgroups (0 on error)
int prolong_tile_nzr(int slots, int nc, int nf);  // coarse-plane ranges per column

// Residual r = f - N(u) (r.a may be null) and per-block maxima of |r| as
// IEEE bit patterns; returns the number of partials written.
template <typename T, bool DELTA>
int launch_resid_max(hipStream_t s, const OpParams &op, Tri<const T> u, Tri<const T> f,
                     const T *phk, const T *base, Tri<T> r, unsigned long long *partial);

void launch_max_final(hipStream_t s, const unsigned long long *partial, int count, double *out,
                      const int *gate = nullptr);
// dst[0] = max of partial[0 .. count), dst[1 .. dcount) = 0 (bit patterns).
void launch_norm_seed(hipStream_t s, const unsigned long long *partial, int count,
                      unsigned long long *dst, int dcount);

void launch_run_reset(hipStream_t s, RunState st);
void launch_stop_test(hipStream_t s, const StopTest &t);

// Coarsest level (natural layout, n = 3 or 4).  lu/piv: cached factorisation
// of the Newton matrix (device scratch of 64*64 doubles and 64 ints), reused
// across calls while *lu_valid is set.  With ubar.a set the launch first
// applies the level's tau correction (f holds I r; fw is f writable) and
// starts u at I u = ubar, as launch_tau does.
template <typename T, bool DELTA>
void launch_coarse(hipStream_t s, const OpParams &op, Tri<T> u, Tri<const T> f, const T *phk,
                   const T *base, const double *lap1, const double *lap3, double *lu, int *piv,
                   int *lu_valid, int *iters, const double *lap2 = nullptr,
                   Tri<const T> ubar = Tri<const T>{nullptr, nullptr, nullptr},
                   Tri<T> fw = Tri<T>{nullptr, nullptr, nullptr});

// phi* = 3/2 phi^k - 1/2 phi^{k-1} from natural-layout inputs into layout L.
void launch_phistar(hipStream_t s, const Lay &L, const double *phk, const double *phkm1,
                    double *out);

// Finest-level source from natural-layout phi^k, phi^{k-1} into layout `op.lay`.
void launch_source(hipStream_t s, const OpParams &op, const double *phk, const double *phkm1,
                   Tri<double> f);
void launch_init_guess(hipStream_t s, const OpParams &nat, const double *phi0, double *mu,
                       double *om);

// A time step's set-up on a colour-split finest level (setup.hip): source, starting
// iterate and phi^k from the natural-layout fields; and its iterate back to them.
void launch_step_begin(hipStream_t s, const OpParams &op, const double *cur, const double *prev,
                       const double *mu, const double *om, Tri<double> f, Tri<double> u, double *phk);
void launch_step_end(hipStream_t s, const Lay &L, Tri<double> u, double *phi, double *mu, double *om);

// Layout conversion of `count` consecutive fields between natural and `lay`
// (with a type cast).
template <typename S, typename D>
void launch_to_lay(hipStream_t s, const Lay &lay, const S *src, D *dst, int count);
template <typename S, typename D>
void launch_from_lay(hipStream_t s, const Lay &lay, const S *src, D *dst, int count);

// Energy on natural-layout fields: per-block sums (partial: 6 energy_blocks(n) + 6
// doubles), then fixed-order final sums of phi^4, phi^2, |D phi|^2, (Lap phi)^2,
// |D(phi - phi_prev)|^2 and phi, to device or pinned memory; launch_energy goes on
// to out3 (energy, modified energy, mass) on the device.
int energy_blocks(int n);
__host__ __device__ inline void energy_out(const double *sums, double h, double eps, double *out) {
    const double h3 = h * h * h;
    const double F = h3 * (0.25 * sums[0] + 0.5 * (1.0 - eps) * sums[1] - sums[2] + 0.5 * sums[3]);
    out[0] = F;
    out[1] = F + 0.5 * h3 * sums[4];
    out[2] = h3 * sums[5];
}
void launch_energy_sums(hipStream_t s, const Lay &nat, double h, const double *phi,
                        const double *phi_prev, double *partial, double *sums6);
void launch_energy(hipStream_t s, const Lay &nat, double h, double eps, const double *phi,
                   const double *phi_prev, double *partial, double *out3);

// ---- mixed-precision helpers (FP64 finest level, FP32 correction) ----
// u64 += e32 on three fields (same layout, n points each).
void launch_add_correction(hipStream_t s, size_t P, Tri<double> u, Tri<const float> e);
// r = f - N(u) in FP64, per-block max-norm partials, and FP32 copies of r and
// of u.a (the base of the correction cycle).
int launch_resid_cast(hipStream_t s, const OpParams &op, Tri<const double> u, Tri<const double> f,
                      const double *phk, Tri<float> r32, float *base32,
                      unsigned long long *partial);
// Fills `count` floats with zero.
void launch_zero(hipStream_t s, float *p, size_t count);


// ---- batched form ----
enum { BK_SMOOTH = 0, BK_RR = 1, BK_TAU = 2, BK_PROLONG = 3, BK_ERR = 4, BK_NORM = 5, BK_KINDS = 6 };
// Batched tile shapes: a tile covers W consecutive work items of a plane
// (W = kTileMin << (shape % kWOpts): 64 .. 1024) in Z consecutive planes
// (Z = 1 << (shape / kWOpts): 1 .. 8), walked plane by plane; the stop
// test's norm uses shape kNormShape (W = 256, Z = 4).
constexpr int kTileMin = 64, kWOpts = 5, kZOpts = 4, kShapes = kWOpts * kZOpts;
constexpr int kNormShape = 2 + kWOpts * 2;

// One instance on one level, as seen by a batched launch.
struct BSeg {
    OpParams op;                 // this level
    Lay lay_c;                   // next coarser level (restriction, interpolation)
    Tri<double> u, f, ubar;      // this level
    Tri<double> uc, fc, ubarc;   // next coarser level
    double *phk;                 // phi^k on this level
    const double *lap1, *lap3;   // coarsest-level matrices of this instance
    double *minv;                // cached coarsest inverse
    int *valid, *iters;
    const int *active;           // the instance's convergence flag
    int inst;
    // first tile of this segment in the work-list of a launch over its list,
    // per phase kind and tile shape: segments are padded to whole tiles, so
    // a workgroup finds a tile's segment by binary search
    unsigned first[BK_KINDS][kShapes];
    // the same for the column-tiled interpolation, per coarse planes per
    // tile (1 << zi); every tile of a segment is a whole column
    unsigned ptf[kZOpts];
};

// Per-instance state of the batched stop test (device arrays).
struct BState {
    int *active, *cycles, *status;
    double *res0, *res;
    const unsigned *norm_first, *norm_blocks;  // per finest-level segment
};

// One launch of a batched phase over `ntiles` tiles of shape `shape`,
// `threads` per workgroup: one tile per workgroup (slots = 0) or
// persistent, at most `slots` workgroups walking the tiles.  arg0,
// arg1: the half-sweep's colour and picard flag (BK_SMOOTH); for BK_PROLONG
// arg0 = 1 when a smoothing sweep follows (colour-0 mu, omega left
// unwritten).
void launch_batch(hipStream_t s, int kind, const BSeg *segs, int nseg, unsigned ntiles, int shape,
                  int threads, unsigned slots, int arg0, int arg1);
// Work items of one segment as planes: Q items per plane, NPL planes (the
// item index is plane * Q + position), for the tile shapes.
void bseg_planes_host(const BSeg &g, int kind, unsigned &Q, unsigned &NPL);
// Resident workgroups of a phase kind's kernel at `threads` per workgroup.
int batch_phase_slots(int kind, int threads, int device);
void launch_batch_coarse(hipStream_t s, const BSeg *segs, int nseg, int tau);
void launch_batch_norm(hipStream_t s, const BSeg *segs, int nseg, unsigned ntiles,
                       unsigned long long *partial, BState st, double tol, int max_cycles);
// The same test on the two halves that the batched pairs leave, part[b] and
// second[b] for the blocks b of an instance (st.norm_first, st.norm_blocks).
void launch_batch_update(hipStream_t s, const BSeg *segs, int nseg, const unsigned long long *part,
                         const unsigned long long *second, BState st, double tol, int max_cycles);
// The whole-level norm of every instance (partial as launch_batch_norm's, the
// blocks by st) into the first of its blocks in second (by pst), zeros in the others.
void launch_batch_seed(hipStream_t s, const BSeg *segs, int nseg, unsigned ntiles,
                       unsigned long long *partial, BState st, BState pst, unsigned long long *second);
// Two sweeps of every instance's finest level in one launch: a column of planes
// [z0, z1) per workgroup, the box at (x0, y0) px points wide, the norm half (1, 2
// as launch_sweep_pair64) to part[slot].  The gate in a seg's op is its instance's
// active flag.
struct PairTile {
    int seg, x0, y0, px, z0, z1;
    unsigned slot;
    int unused;
};
bool batch_pair_fits(int n);
int batch_pair_slots(int device);
// Tiles of one level at most zmax planes long (seg and slots to be filled in).
std::vector<PairTile> batch_pair_tiles(int n, int zmax);
void launch_batch_pair(hipStream_t s, int nrm, const PairArgs<double> *segs, const PairTile *tiles,
                       int ntiles, unsigned long long *part);
void launch_batch_reset(hipStream_t s, BState st, int count, int **valid);
// Set-up and end of a step of every instance (setup.hip).  p: an instance's three
// phi buffers, of which ip, ic, in are the previous, the current and the next; a
// workgroup takes block blk of instance or segment seg.
struct BatchIO {
    OpParams op;
    double *p[3];
    double *mu, *om;
    Tri<double> f, u;
    double *phk;
};
struct BlockRef {
    int seg;
    unsigned blk;
};
struct RestrictSeg {
    Lay fine, coarse;
    const double *from;
    double *to;
};
// Brick launches (4^3 boxes, levels of 12^3 and 16^3) and two-level tails of many
// instances; the gate in a segment's op is its instance's active flag.
void launch_batch_brick(hipStream_t s, int kind, int sweeps, bool first, const BrickArgs<double> *segs,
                        const BlockRef *blocks, unsigned count);
void launch_batch_tail(hipStream_t s, const TailArgs<double> *segs, int nseg, int fcycle);
void launch_batch_begin(hipStream_t s, const BatchIO *io, const BlockRef *blocks, unsigned count, int ip,
                        int ic);
void launch_batch_end(hipStream_t s, const BatchIO *io, const BlockRef *blocks, unsigned count, int in);
void launch_batch_restrict(hipStream_t s, const RestrictSeg *segs, const BlockRef *blocks, unsigned count);
// Column-tiled interpolation of the batched form (fine levels whose size is a
// multiple of kBPX): a kBPX x 8 fine column and 1 << zi coarse planes of one
// instance per workgroup, the coarse error formed while staged (no
// coarse-error pass before it).  Same results as the coarse-error pass
// followed by the interpolation phase.
constexpr int kBPX = 16;
bool batch_ptile_fits(const BSeg &g);
unsigned batch_ptile_count(const BSeg &g, int zi);
void launch_batch_ptile(hipStream_t s, const BSeg *segs, int nseg, unsigned ntiles, int zi,
                        int phi0);

}  // namespace pfc
