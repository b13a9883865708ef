// Handle layout shared by the host-side translation units of the runtime.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <string>
#include <vector>

#include "pfc.h"

#include "pfc_internal.h"

namespace pfc {

constexpr int kMaxLevels = 24;

// One level of the FP64 multigrid hierarchy.  Smoothed levels are stored
// colour-split, the coarsest level in natural order.
struct Level {
    int n = 0;
    double h = 0, h2inv = 0;
    size_t P = 0;
    Lay lay{};
    Tri<double> u{nullptr, nullptr, nullptr};     // iterate
    Tri<double> f{nullptr, nullptr, nullptr};     // right-hand side
    Tri<double> ubar{nullptr, nullptr, nullptr};  // restricted fine iterate I u (scratch on level 0)
    Tri<double> u2{nullptr, nullptr, nullptr};    // second iterate buffer (fused sweeps, fused correction, bricks)
    // third iterate buffer (bricks that run the two sweeps of a side apart): fr, which
    // a cycle reads in its first launch only, on level 0 the scratch ubar
    Tri<double> u3{nullptr, nullptr, nullptr};
    Tri<double> fr{nullptr, nullptr, nullptr};    // I r of a coarse brick level (its f is f + N(I u))
    double *phk = nullptr;                        // phi^kappa on this level
    double *phs = nullptr;                        // phi* of the variable mobility (else null)
    bool phs_set = false;                         // phs holds a field
    bool fused = false;                           // smoothed by the fused red-black sweep
    int nz = 1;                                   // its plane ranges per column
    bool pair = false;                            // two sweeps in a row take one launch (sweep_pair.h)
    int pnz = 1;                                  // its plane ranges per column
    bool brick = false;                           // one brick launch on either side of the descent
    bool tail = false;                            // this level and the coarsest in one launch
    bool rt = false;                              // residuals by column tiles
    int rt_nz[RT_MODES] = {1, 1, 1, 1, 1};        // their plane ranges, per epilogue
    int pz[2] = {0, 0};  // plane ranges of the tiled interpolation onto this level (FP64, FP32)
};

// One level of the FP32 correction cycle of the mixed-precision form.
struct Level32 {
    Tri<float> e{nullptr, nullptr, nullptr};     // correction iterate
    Tri<float> f{nullptr, nullptr, nullptr};     // right-hand side
    Tri<float> ebar{nullptr, nullptr, nullptr};  // restricted fine correction (unused on level 0)
    Tri<float> e2{nullptr, nullptr, nullptr}, e3{nullptr, nullptr, nullptr};  // more iterate buffers (bricks, pairs), as u2, u3
    Tri<float> fr{nullptr, nullptr, nullptr};    // I r of a coarse brick level
    bool pair = false;                           // two sweeps in a row take one launch (sweep_pair.h)
    int pnz = 1;                                 // its plane ranges per column
    float *phk = nullptr;                        // phi^kappa
    float *base = nullptr;                       // FP64 iterate's phi, rounded and restricted
};

// One timed launch: n of the launches that `kind` counts (a launch that runs
// several sweeps counts as that many; its time and bytes are shared evenly).
struct TimedLaunch {
    int kind;
    hipEvent_t a, b;
    double bytes;  // the launch's algorithmic HBM bytes
    int n = 1;
    bool ahead = false;  // launched before the loop's decision (see retract_ahead)
    int kind2 = -1;      // the launch's second sweep counts there; half its time and bytes
};

bool level_sizes(int n, std::vector<int> &out);
std::string validate_config(const pfc_config *c);
void coarse_matrices(int n, double h, std::vector<double> &l1, std::vector<double> &l2,
                     std::vector<double> &l3);

}  // namespace pfc

struct pfc_handle {
    pfc_config cfg{};
    hipStream_t stream = nullptr;
    int device = 0;
    int nlev = 0;
    pfc::Level lev[pfc::kMaxLevels];
    pfc::Level32 lev32[pfc::kMaxLevels];
    std::vector<void *> allocs;
    // the block of the requests smaller than kOwnBlock: counted in a first pass over
    // the requests (planning), then allocated once and dealt out in a second
    bool planning = false;
    char *arena = nullptr;
    size_t arena_left = 0;
    unsigned long long *partial = nullptr;
    int *d_iters = nullptr;
    double *h_pin = nullptr;
    double *lap1 = nullptr, *lap2 = nullptr, *lap3 = nullptr;
    double *minv64 = nullptr, *minv32 = nullptr;  // cached coarsest Newton inverses
    int *valid64 = nullptr, *valid32 = nullptr;
    double *minv_adj = nullptr;  // cached coarsest inverse of the adjoint solve
    int *valid_adj = nullptr;
    double *energy_part = nullptr;
    // stop test split over the finest level's fused sweeps (FP64): the
    // last post-sweep of a cycle leaves the colour-1 half of the norm in
    // partial[split_pre .. split_pre + split_post), the next cycle's first
    // pre-sweep (with the second, where two take one launch), run ahead of
    // the decision, the colour-0 half in partial[0 .. split_pre)
    bool split_norm = false;
    // Set by a time step's set-up: the finest level's f.a holds phi^k, a copy
    // of phk (the first component of S is phi^k itself), so the finest-level
    // kernels read phk in its place (see frhs).  Cleared by the entry points
    // that load a caller's right-hand side into the finest level.
    bool f1_phk = false;
    int split_pre = 0, split_post = 0;
    // graph-driven time loop (pfc_run)
    const int *gate = nullptr;            // cycle gate, set only while its graph is recorded
    pfc::StopTest stop{};                 // the loop's decision, for the cycle's first tail launch to take
    hipStream_t run_stream = nullptr;     // the loop's own stream (capturable)
    hipEvent_t run_ev = nullptr;
    hipEvent_t norm_ev = nullptr;         // the mixed form's norm copied to the host
    hipEvent_t unit_ev[2] = {nullptr, nullptr};  // units of a host-driven loop (run_units)
    int *d_run = nullptr;                 // active, cycles, status of the current step
    double *d_runres = nullptr;           // res0, res of the current step
    hipGraph_t run_graph = nullptr;       // norm, stop test, one gated cycle
    hipGraphExec_t run_exec = nullptr;
    const void *run_key[pfc::kMaxLevels] = {};  // level iterates the graph was recorded with
    double *spare = nullptr;              // third phi buffer of the loop
    int last_cycles = 0;                  // cycles of the previous step (launch count guess)
    hipGraph_t mix_graph = nullptr;       // one FP32 correction cycle (mixed form)
    hipGraphExec_t mix_exec = nullptr;
    std::string err;
    // instrumentation
    bool timing = false;
    int cur_event = -1;
    std::vector<pfc::TimedLaunch> pending;
    std::vector<hipEvent_t> pool;
    int64_t t_count[PFC_KERNEL_COUNT] = {};
    double t_ms[PFC_KERNEL_COUNT] = {};
    double t_bytes[PFC_KERNEL_COUNT] = {};

    // bytes < 0: the kind's algorithmic bytes per finest-level launch
    void begin_timed(int kind, int level, double bytes = -1.0, int n = 1, bool ahead = false,
                     int kind2 = -1);
    void end_timed();
    void collect_timings();
    // The step stopped: the sweeps of the last launch ahead of the decision,
    // whose output is dropped, are taken out of the counts again.
    void retract_ahead();
    int ahead_kind = -1, ahead_n = 0;
    double ahead_ms = 0, ahead_bytes = 0;
    ~pfc_handle();
};

namespace pfc {
OpParams op_of(const pfc_handle *H, int l);
// flags of cycle64 (the first two at the finest level)
constexpr unsigned kCyclePreDone = 1;   // its first pre-sweeps have already run (ahead64;
                                        // a brick level: the whole part before the descent)
constexpr unsigned kCyclePostNorm = 2;  // its last post-sweep leaves the colour-1 norm half
constexpr unsigned kCycleTauSweep = 8;  // (coarse level) f holds I r and the
                                        // iterate is still in ubar: the first pre-sweep (the
                                        // coarsest: its solve) forms the tau correction and
                                        // reads the old values there
void cycle64(pfc_handle *H, int l, bool fcycle, unsigned flags = 0);
// The part of a cycle before the descent on brick level l:
// BRICK_PLAIN, BRICK_FIRST (a coarse level's first visit: f holds nothing yet,
// I r is in fr and the iterate in ubar) or BRICK_NORM (finest level: also the
// norm of the iterate, as the returned number of maxima in H->partial).  The
// iterate stays in u, the smoothed one goes to another buffer, from where the
// part after the descent takes it: dropping the launch's output costs nothing.
int brick_pre64(pfc_handle *H, int l, int form);
// The two-level tail's launch on level l (but fcycle and the stop test).
TailArgs<double> tail_args64(const pfc_handle *H, int l);
// Level l's right-hand side as its kernels read it.  In a time step the
// first component of the finest level's S is phi^k itself (scheme-PFC-s1),
// held bitwise in both f.a and phk; reading it from phk spares the kernels a
// second 8-byte stream per point (the fused sweep, the residual passes and
// the FP64 defect pass).
inline Tri<const double> frhs(const pfc_handle *H, int l) {
    const Level &A = H->lev[l];
    if (l == 0 && H->f1_phk) return Tri<const double>{A.phk, A.f.b, A.f.c};
    return Tri<const double>{A.f.a, A.f.b, A.f.c};
}

// One smoothing sweep of level l; nrm as in launch_sweep_fused (split_norm
// only); then_sweep: the next operation on the iterate is another sweep of
// this level (a fused sweep then leaves the dead colour-0 mu, omega
// unwritten); tau: a coarse level's first sweep forming the tau correction
// (launch_smooth_tau; on a fused level into the second buffer, which then
// becomes the iterate).
void sweep64(pfc_handle *H, int l, int nrm = 0, bool then_sweep = false,
             bool tau = false);
// Sweeps from .. count - 1 of one side of the descent, in pairs where the level
// takes two per launch.  norm: the last one leaves the colour-1 half of the norm of
// its output; tau: sweep 0 forms the tau correction.
void sweeps64(pfc_handle *H, int l, int from, int count, bool norm = false, bool tau = false);
// The pre-sweeps that run ahead of the loop's decision (split_norm): the first,
// or the first two where they take one launch.  One exchange of the iterate
// buffers, so exchanging them back drops the launch.
inline int sweep_launches(const pfc_handle *H, int l) {  // a cycle's, both sides of the descent
    const int c = H->lev[l].pair ? 1 : 0;
    return ((H->cfg.nu1 + c) >> c) + ((H->cfg.nu2 + c) >> c);
}
inline int ahead_sweeps(const pfc_handle *H) { return H->lev[0].pair && H->cfg.nu1 >= 2 ? 2 : 1; }
void ahead64(pfc_handle *H);
void restrict_phk(pfc_handle *H);
pfc_status resid_norm64(pfc_handle *H, Tri<double> r, double *out);
int enqueue_norm64(pfc_handle *H, unsigned long long *dst = nullptr);
pfc_status read_norm(pfc_handle *H, int partials, double *out);
void mixed_plan(pfc_handle *H);   // the FP32 levels' forms
bool mixed_alloc(pfc_handle *H);  // their memory
// pfc_create.  A batch launches its instances' cycles itself and needs fewer buffers:
// bricks on its small levels only, a second iterate on level 0 for paired sweeps.
enum HandleUse { USE_SINGLE, USE_BATCH, USE_BATCH_PAIRS };
pfc_status create_handle(const pfc_config *cfg, void *stream, HandleUse use, pfc_handle **out);
pfc_status step64(pfc_handle *h, const double *phi_prev, const double *phi_cur, double *phi_next,
                  double *mu, double *omega, pfc_step_info *info);
// The device state of a cycle loop; its decisions reach h_pin through slot 0 or 1.
inline RunHost *run_host(const pfc_handle *H, int slot) {
    return reinterpret_cast<RunHost *>(H->h_pin + 16 + 8 * slot);
}
inline RunState run_state(pfc_handle *H, int slot = 0) {
    return RunState{H->d_run,        H->d_run + 1,    H->d_run + 2, H->d_runres,
                    H->d_runres + 1, run_host(H, slot)};
}
// A cycle loop driven by the host, the decisions on the device.  Unit i is
// head(i, ride), the launches up to and with the stop test (into run_state(H, i & 1);
// ride: the test may ride in a launch of the body), and body(i), the rest of a cycle,
// every launch gated on the test.  While the norms so far say that the loop goes on,
// units are enqueued whole, one ahead of the host, so that the device does not wait
// between cycles (a 32^3 step waited 12-25 us of every 78 us cycle).  Where they say
// that a test will stop it, or say nothing yet, its body waits for the decision:
// behind a stop it would do nothing, but takes 4 us a launch (a step that starts
// converged, all units whole: 64^3 V(2,2) 178 us instead of 105, 96^3 F(4,4), 150
// launches a cycle, 1411 instead of 120).  Without brick and tail launches (more than
// two sweeps per side) a cycle is 50 to 150 launches, and one queued for nothing costs
// more than the waits that ten saved: there a test has to be expected to fail by a
// factor of ten (96^3 F(4,4), stopping after the first cycle 1540 -> 1170 us, after
// the eighth 10.4 -> 9.1 ms).
// first: the norm at the first test where the host has it, else NaN.  tol: the
// test's.  out: the last decision.
template <typename Head, typename Body>
pfc_status run_units(pfc_handle *H, double tol, double first, Head head, Body body, RunHost *out);
pfc_status unit_events(pfc_handle *H);
// The unit of a time step's loop (pfc_step after its first, and recorded as pfc_run's
// graph), what pfc_run needs before the first one, and whether the level iterates are
// back in their buffers after one, so that units can follow each other unseen.
void step_head(pfc_handle *H, int slot, bool ride);
void step_body(pfc_handle *H);
// The unit's decision on `count` maxima in H->partial.  scratch: whatever the unit
// launches from here to the 8^3 (6^3) level writes neither the iterate nor the
// cached inverse; the test then rides in that level's launch instead of taking
// 4.4 us of its own (cycle of 16^3 46.5 -> 44.8 us, 32^3 63 -> 61.4, 64^3 110.9 ->
// 109.6), up to 64^3: beyond, the maxima are more than that workgroup reads in
// passing (96^3 207 -> 209) and the descent of the unit that stops, now run for
// nothing, costs as much.
constexpr int kTailTestMaxN = 64;
void unit_stop_test(pfc_handle *H, int slot, int count, double tol, bool scratch);
void step_unit_seed(pfc_handle *H);
bool units_usable(const pfc_handle *H);
// The handle's own non-blocking stream (created on first use): recorded
// graphs need a capturable stream.  own_stream_enter makes it follow the
// caller's stream and returns that stream; own_stream_leave makes the caller's
// stream follow it again.
pfc_status own_stream_enter(pfc_handle *H, hipStream_t *user);
pfc_status own_stream_leave(pfc_handle *H, hipStream_t user);
pfc_status mixed_step(pfc_handle *H, const double *phi_prev, const double *phi_cur,
                      double *phi_next, double *mu, double *omega, pfc_step_info *info);
double algorithmic_bytes(const pfc_handle *H, int kernel);
// Finest-level set-up of one time step (source, layout conversion of the
// guess and of phi^k, phi^k hierarchy) and the conversion back.
void step_begin(pfc_handle *H, const double *phi_prev, const double *phi_cur, const double *mu,
                const double *omega);
void step_end(pfc_handle *H, double *phi_next, double *mu, double *omega);
void invalidate_coarse(pfc_handle *H);
// Device memory of a handle, given back with it.  The small ones of its some 40
// requests share one block of exactly their size (96^3: 870 us to create with a call
// for each, 240 in one block).
constexpr size_t kOwnBlock = (size_t)64 << 20;
bool dalloc_bytes(pfc_handle *H, void **p, size_t bytes);
template <typename T>
bool dalloc(pfc_handle *H, T **p, size_t count) {
    void *q = nullptr;
    if (!dalloc_bytes(H, &q, count * sizeof(T))) return false;
    *p = (T *)q;
    return true;
}
template <typename T>
bool dalloc(pfc_handle *H, Tri<T> *t, size_t P) {
    T *q;
    if (!dalloc(H, &q, 3 * P)) return false;
    *t = q ? Tri<T>{q, q + P, q + 2 * P} : Tri<T>{nullptr, nullptr, nullptr};
    return true;
}
pfc_status fail(pfc_handle *H, pfc_status st, const std::string &msg);
pfc_status hip_fail(pfc_handle *H, hipError_t e, const char *what);
}  // namespace pfc

#define HIP_TRY(H, expr)                                                  \
    do {                                                                  \
        hipError_t e_ = (expr);                                           \
        if (e_ != hipSuccess) return pfc::hip_fail((H), e_, #expr);       \
    } while (0)

namespace pfc {
template <typename Head, typename Body>
pfc_status run_units(pfc_handle *H, double tol, double first, Head head, Body body, RunHost *out) {
    const pfc_status st = unit_events(H);
    if (st != PFC_OK) return st;
    struct Gate {  // set while the units are enqueued
        pfc_handle *H;
        explicit Gate(pfc_handle *h) : H(h) { H->gate = H->d_run; }
        ~Gate() { H->gate = nullptr; }
    } gate(H);
    launch_run_reset(H->stream, run_state(H));
    auto enqueue = [&](int i, bool whole) -> pfc_status {
        head(i, whole);
        if (whole) body(i);
        HIP_TRY(H, hipGetLastError());
        HIP_TRY(H, hipEventRecord(H->unit_ev[i & 1], H->stream));
        return PFC_OK;
    };
    const bool few = H->nlev >= 2 && H->lev[H->nlev - 2].tail;  // launches a cycle
    // test i's norm; its ratio to the one before (until two are known a good cycle's); the last known
    double expect = first, rate = few ? 0.1 : 0.0, res = first;
    const double above = few ? tol : 10.0 * tol;
    auto goes_on = [&](int i, double norm) { return norm > above && i < H->cfg.max_cycles; };
    bool whole = goes_on(0, expect);
    pfc_status e = enqueue(0, whole);
    if (e != PFC_OK) return e;
    for (int i = 0;; ++i) {
        bool next = whole && goes_on(i + 1, expect * rate);
        if (whole && (e = enqueue(i + 1, next)) != PFC_OK) return e;
        HIP_TRY(H, hipEventSynchronize(H->unit_ev[i & 1]));
        const RunHost r = *run_host(H, i & 1);
        if (!r.active) {
            *out = r;
            return PFC_OK;
        }
        if (i - 2 > H->cfg.max_cycles)  // (max_cycles may be INT_MAX)
            return fail(H, PFC_ERR_HIP, "cycle loop: the device stop test did not end it");
        if (i > 0) rate = r.res / res;
        res = r.res;
        expect = res * rate;
        if (!whole) {
            body(i);
            next = goes_on(i + 1, expect);
            if ((e = enqueue(i + 1, next)) != PFC_OK) return e;
        }
        whole = next;
    }
}
}  // namespace pfc
