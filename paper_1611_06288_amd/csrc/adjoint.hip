// Adjoint of one time step of scheme (1.10) (M = 1), for gradients of a
// loss of phi^{k+1} with respect to phi^k, phi^{k-1} and eps.
//
// The step solution u = (phi^{k+1}, mu, omega) satisfies G = N(u) - S = 0
// (scheme-PFC-o1..o3 and scheme-PFC-s1..s3).  By the implicit-function
// theorem, with J = dN/du at u,
//     J^T lambda = (gbar_next, 0, 0),
//     gbar_cur  += -(dG/dphi^k)^T lambda
//                = lambda1 + (g_a(phi^{k+1}; phi^k) + (1-eps)/2) lambda2
//                  + 3 Lap lambda2 + Lap lambda3 / 2,
//     gbar_prev += -(dG/dphi^{k-1})^T lambda = -Lap lambda2,
//     geps      += -(dG/deps)^T lambda = -1/2 sum lambda2 (phi^{k+1} + phi^k),
// where J = [[I, -tau Lap, 0], [-D, I, -Lap], [-Lap/2, 0, I]],
// D = diag(g_phi(phi^{k+1}; phi^k) + (1-eps)/2), g_a = dg/dphi^k.
//
// J^T lambda = b is solved by linear multigrid (correction scheme) on the
// same hierarchy: red-black block Gauss-Seidel on the 3x3 point blocks of
// J^T, 8-child restriction of the residual and of D, trilinear
// interpolation of the correction, and an exact solve on the coarsest level
// after eliminating lambda2 = b2 + tau Lap lambda1 and
// lambda3 = b3 + Lap lambda2:
//     (I - tau D Lap - tau/2 Lap^3) lambda1 = b1 + D b2 + 1/2 Lap(b3 + Lap b2).
#include <cmath>

#include "coarse.h"
#include "runtime_internal.h"

namespace pfc {

// D = g_phi(phi^{k+1}; phi^k) + (1-eps)/2 from natural-layout fields into `lay`.
__global__ __launch_bounds__(kBlock) void k_adj_D(Lay lay, double eps, const double *__restrict__ phin,
                                                  const double *__restrict__ phk,
                                                  double *__restrict__ D) {
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t >= (unsigned)npts(lay)) return;
    int i, j, k;
    decode_nat(lay, t, i, j, k);
    D[sidx32(lay, i, j, k)] = Cubic<false>::dg(phin[t], phk[t], 0.0) + 0.5 * (1.0 - eps);
}

// Red-black block Gauss-Seidel on J^T, one colour (adj_point_solve).
__global__ __launch_bounds__(kBlock) void k_adj_smooth(OpParams op, int colour, Tri<double> lam,
                                                       Tri<const double> b,
                                                       const double *__restrict__ D) {
    if (gate_closed(op.gate)) return;
    const Lay &L = op.lay;
    const int n = L.n, hn = n >> 1;
    const unsigned H = (unsigned)((size_t)n * n * n / 2);
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t >= H) return;
    const unsigned row = L.dh.q(t);
    const int m = (int)(t - row * (unsigned)hn);
    const int k = (int)L.dn.q(row);
    const int j = (int)(row - (unsigned)k * (unsigned)n);
    const int i = 2 * m + ((colour + j + k) & 1);
    const Off q = offs(L, i, j, k);
    const double s[3] = {nsum(lam.a, q), nsum(lam.b, q), nsum(lam.c, q)};
    double l[3];
    adj_point_solve(op, D[q.c], b.a[q.c], b.b[q.c], b.c[q.c], s, l);
    lam.a[q.c] = l[0];
    lam.b[q.c] = l[1];
    lam.c[q.c] = l[2];
}

// r = b - J^T lambda at one point.
__device__ __forceinline__ void adj_resid_at(const OpParams &op, const Tri<const double> &lam,
                                             const Tri<const double> &b, const double *D,
                                             const Off &q, double &r1, double &r2, double &r3) {
    const double w[3] = {lam.a[q.c], lam.b[q.c], lam.c[q.c]};
    const double ls[3] = {(nsum(lam.a, q) - 6.0 * w[0]) * op.h2inv,
                          (nsum(lam.b, q) - 6.0 * w[1]) * op.h2inv,
                          (nsum(lam.c, q) - 6.0 * w[2]) * op.h2inv};
    double r[3];
    adj_resid_from_lap(op, ls, w, b.a[q.c], b.b[q.c], b.c[q.c], D[q.c], r);
    r1 = r[0];
    r2 = r[1];
    r3 = r[2];
}

__global__ __launch_bounds__(kBlock) void k_adj_resid_max(OpParams op, Tri<const double> lam,
                                                          Tri<const double> b,
                                                          const double *__restrict__ D,
                                                          unsigned long long *partial) {
    if (gate_closed(op.gate)) return;
    const Lay &L = op.lay;
    const unsigned total = (unsigned)npts(L);
    unsigned long long mx = 0;
    for (unsigned t = xcd_block() * kBlock + threadIdx.x; t < total; t += gridDim.x * kBlock) {
        int i, j, k;
        decode(L, t, i, j, k);
        const Off q = offs(L, i, j, k);
        double r1, r2, r3;
        adj_resid_at(op, lam, b, D, q, r1, r2, r3);
        mx = umax(mx, umax(abs_bits(r1), umax(abs_bits(r2), abs_bits(r3))));
    }
    mx = block_max_u64(mx);
    if (threadIdx.x == 0) partial[blockIdx.x] = mx;
}

// Coarse right-hand side b_c = I (b - J^T lambda), eight threads per coarse
// cell (one per child, child ch = (ch & 1, (ch >> 1) & 1, ch >> 2) in x, y, z),
// so each thread waits on one child's loads; the cell's eight lanes add
// their residuals in the order ch = 0..7 and the first stores b_c and clears
// the coarse iterate lam_c (the coarse problem starts from zero).
__global__ __launch_bounds__(kBlock) void k_adj_resid_restrict(OpParams op, Lay LC,
                                                               Tri<const double> lam,
                                                               Tri<const double> b,
                                                               const double *__restrict__ D,
                                                               Tri<double> bc, Tri<double> lamc) {
    if (gate_closed(op.gate)) return;
    const unsigned g = xcd_block() * kBlock + threadIdx.x;
    const unsigned tn = g >> 3;
    const int ch = (int)(g & 7u);
    const bool act = tn < (unsigned)npts(LC);
    double r[3] = {0.0, 0.0, 0.0};
    unsigned t = 0;
    if (act) {
        int I, J, K;
        decode_nat(LC, tn, I, J, K);
        t = sidx32(LC, I, J, K);
        const Off q = offs(op.lay, 2 * I + (ch & 1), 2 * J + ((ch >> 1) & 1), 2 * K + (ch >> 2));
        adj_resid_at(op, lam, b, D, q, r[0], r[1], r[2]);
    }
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int e = 0; e < 3; ++e) s[e] += __shfl(r[e], c, 8);
    if (act && ch == 0) {
        bc.a[t] = 0.125 * s[0];
        bc.b[t] = 0.125 * s[1];
        bc.c[t] = 0.125 * s[2];
        lamc.a[t] = 0.0;
        lamc.b[t] = 0.0;
        lamc.c[t] = 0.0;
    }
}

__global__ __launch_bounds__(64) void k_adj_coarse(OpParams op, Tri<double> lam,
                                                   Tri<const double> b,
                                                   const double *__restrict__ D,
                                                   const double *__restrict__ lap1,
                                                   const double *__restrict__ lap3, double *minv,
                                                   int *valid) {
    __shared__ CoarseShared sm;
    if (gate_closed(op.gate)) return;
    const bool cached = coarse_load_inverse<64>(minv, valid, sm);
    wave_sync();
    adj_coarse_body(op, lam, b, D, lap1, lap3, minv, cached, valid, sm);
}

__global__ __launch_bounds__(kBlock) void k_fill(double *p, size_t count, double v) {
    const size_t t = (size_t)xcd_block() * kBlock + threadIdx.x;
    if (t < count) p[t] = v;
}

// gbar_cur += lambda1 + (g_a + (1-eps)/2) lambda2 + 3 Lap lambda2 + Lap lambda3 / 2
// (natural layout; lam holds lambda in natural order).
__global__ __launch_bounds__(kBlock) void k_adj_accum_cur(OpParams nat, Tri<const double> lam,
                                                          const double *__restrict__ phin,
                                                          const double *__restrict__ phk,
                                                          double *__restrict__ gcur) {
    const Lay &L = nat.lay;
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t >= (unsigned)npts(L)) return;
    int i, j, k;
    decode(L, t, i, j, k);
    const Off q = offs(L, i, j, k);
    const double l2 = lam.b[t], l3 = lam.c[t];
    const double L2 = (nsum(lam.b, q) - 6.0 * l2) * nat.h2inv;
    const double L3 = (nsum(lam.c, q) - 6.0 * l3) * nat.h2inv;
    const double x = phin[t], a = phk[t];
    const double ga = 0.25 * (x * x + 2.0 * x * a + 3.0 * a * a);
    gcur[t] += lam.a[t] + (ga + 0.5 * (1.0 - nat.eps)) * l2 + 3.0 * L2 + 0.5 * L3;
}

// gbar_prev -= Lap lambda2 (natural layout).
__global__ __launch_bounds__(kBlock) void k_adj_accum_prev(OpParams nat, const double *__restrict__ l2v,
                                                           double *__restrict__ gprev) {
    const Lay &L = nat.lay;
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t >= (unsigned)npts(L)) return;
    int i, j, k;
    decode(L, t, i, j, k);
    const Off q = offs(L, i, j, k);
    gprev[t] -= (nsum(l2v, q) - 6.0 * l2v[t]) * nat.h2inv;
}

// Per-block sums of lambda2 (phi^{k+1} + phi^k); the final pass adds
// -1/2 of their fixed-order total into geps[0].
__global__ __launch_bounds__(kBlock) void k_adj_eps_part(size_t P, const double *__restrict__ l2v,
                                                         const double *__restrict__ phin,
                                                         const double *__restrict__ phk,
                                                         double *__restrict__ part) {
    __shared__ double red[kBlock];
    double s = 0.0;
    for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < P; t += (size_t)gridDim.x * kBlock)
        s += l2v[t] * (phin[t] + phk[t]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kBlock) void k_adj_eps_final(const double *__restrict__ part, int count,
                                                          double *geps) {
    __shared__ double red[kBlock];
    double s = 0.0;
    for (int b = threadIdx.x; b < count; b += kBlock) s += part[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) geps[0] += -0.5 * red[0];
}

// ------------------------------------------------------------- driver

static void fill(hipStream_t s, double *p, size_t count, double v) {
    hipLaunchKernelGGL(k_fill, dim3(blocks_for(count)), dim3(kBlock), 0, s, p, count, v);
}

static void adj_sweep(pfc_handle *H, int l) {
    Level &A = H->lev[l];
    const OpParams op = op_of(H, l);
    for (int colour = 0; colour < 2; ++colour)
        hipLaunchKernelGGL(k_adj_smooth, dim3(blocks_for(A.P / 2)), dim3(kBlock), 0, H->stream, op,
                           colour, A.u, cst(A.f), (const double *)A.phk);
}

// The part of a cycle before the descent on brick level l (as brick_pre64).
// BRICK_FIRST: a coarse level's first visit, from zero.
static int adj_brick_pre(pfc_handle *H, int l, int form) {
    Level &A = H->lev[l];
    BrickArgs<double> a;
    a.op = op_of(H, l);
    a.f = cst(A.f);
    a.phk = A.phk;
    a.LC = H->lev[l + 1].lay;
    a.fo = A.f;  // the right-hand side stays what it is
    a.cr = H->lev[l + 1].f;
    a.part = H->partial;
    brick_run_pre<double>(a, H->cfg.nu1, cst(A.u), A.u2, A.u3, form,
                          [&](const BrickArgs<double> &b, int kind, int sweeps, int fm) {
                              launch_brick_adj(H->stream, b, kind, sweeps, fm);
                          });
    return brick_blocks(A.n);
}

static void adj_brick_post(pfc_handle *H, int l) {
    Level &A = H->lev[l];
    BrickArgs<double> a;
    a.op = op_of(H, l);
    a.f = cst(A.f);
    a.phk = A.phk;
    a.LC = H->lev[l + 1].lay;
    a.v = cst(H->lev[l + 1].u);
    brick_run_post<double>(a, H->cfg.nu1, H->cfg.nu2, A.u, A.u2, A.u3,
                           [&](const BrickArgs<double> &b, int kind, int sweeps, int fm) {
                               launch_brick_adj(H->stream, b, kind, sweeps, fm);
                           });
}

static void adj_tail(pfc_handle *H, int l, bool fcycle) {
    Level &A = H->lev[l];
    TailArgs<double> a;
    a.op = op_of(H, l);
    a.opc = op_of(H, l + 1);
    a.nu1 = H->cfg.nu1;
    a.nu2 = H->cfg.nu2;
    a.fcycle = fcycle ? 1 : 0;
    a.u = A.u;
    a.f = cst(A.f);
    a.phk = A.phk;
    a.phkc = H->lev[l + 1].phk;
    a.lap1 = H->lap1;
    a.lap3 = H->lap3;
    a.minv = H->minv_adj;
    a.valid = H->valid_adj;
    a.stop = H->stop;
    H->stop = StopTest{};
    launch_tail_adj(H->stream, a);
}

// first: a coarse level's first visit, its right-hand side new and its iterate
// to start from zero (clear already on a level without bricks); done: the part
// before the descent has already run.
static void adj_cycle(pfc_handle *H, int l, bool fcycle, bool first, bool done = false) {
    Level &A = H->lev[l];
    if (A.tail) return adj_tail(H, l, fcycle);
    if (A.brick) {
        if (!done) adj_brick_pre(H, l, first ? BRICK_FIRST : BRICK_PLAIN);
        adj_cycle(H, l + 1, fcycle, true);
        if (fcycle && !H->lev[l + 1].tail) adj_cycle(H, l + 1, false, false);
        return adj_brick_post(H, l);
    }
    if (l == H->nlev - 1) {
        hipLaunchKernelGGL(k_adj_coarse, dim3(1), dim3(64), 0, H->stream, op_of(H, l), A.u, cst(A.f),
                           (const double *)A.phk, (const double *)H->lap1,
                           (const double *)H->lap3, H->minv_adj, H->valid_adj);
        return;
    }
    Level &B = H->lev[l + 1];
    for (int s = 0; s < H->cfg.nu1; ++s) adj_sweep(H, l);
    hipLaunchKernelGGL(k_adj_resid_restrict, dim3(blocks_for(8 * B.P)), dim3(kBlock), 0, H->stream,
                       op_of(H, l), B.lay, cst(A.u), cst(A.f), (const double *)A.phk, B.f, B.u);
    adj_cycle(H, l + 1, fcycle, true);
    if (fcycle && !B.tail) adj_cycle(H, l + 1, false, false);
    launch_prolong<double>(H->stream, B.lay, A.lay, cst(B.u),
                           Tri<const double>{nullptr, nullptr, nullptr}, A.u, H->gate, false,
                           A.pz[0]);
    for (int s = 0; s < H->cfg.nu2; ++s) adj_sweep(H, l);
}

// The norm of the residual; on a brick level by the next cycle's launches before
// the descent, ahead of the loop's decision (they leave the iterate alone).
// Returns the number of maxima in H->partial.
static int adj_norm(pfc_handle *H) {
    Level &A = H->lev[0];
    if (A.brick) return adj_brick_pre(H, 0, BRICK_NORM);
    const unsigned blocks = reduce_blocks(A.P);
    hipLaunchKernelGGL(k_adj_resid_max, dim3(blocks), dim3(kBlock), 0, H->stream, op_of(H, 0),
                       cst(A.u), cst(A.f), (const double *)A.phk, H->partial);
    return (int)blocks;
}

pfc_status adjoint_step(pfc_handle *H, const double *phi_prev, const double *phi_cur,
                        const double *phi_next, const double *gbar_next, double *gbar_cur,
                        double *gbar_prev, double *geps, double adj_tol, int32_t *cycles) {
    (void)phi_prev;  // the step's Jacobian does not depend on phi^{k-1}
    Level &A = H->lev[0];
    const size_t P = A.P;
    const Lay nat = make_lay(A.n, false);
    // D on every level (stored in the phi^k slots of the hierarchy)
    hipLaunchKernelGGL(k_adj_D, dim3(blocks_for(P)), dim3(kBlock), 0, H->stream, A.lay, H->cfg.eps,
                       phi_next, phi_cur, A.phk);
    restrict_phk(H);
    // b = (gbar_next, 0, 0), lambda = 0
    launch_to_lay<double, double>(H->stream, A.lay, gbar_next, A.f.a, 1);
    fill(H->stream, A.f.b, 2 * P, 0.0);
    fill(H->stream, A.u.a, 3 * P, 0.0);
    (void)hipMemsetAsync(H->valid_adj, 0, sizeof(int), H->stream);
    HIP_TRY(H, hipGetLastError());
    double bnorm = 0.0;
    int parts = adj_norm(H);
    pfc_status st = read_norm(H, parts, &bnorm);
    if (st != PFC_OK) return st;
    if (!std::isfinite(bnorm)) return fail(H, PFC_ERR_NONFINITE, "gbar_next is not finite");
    int c = 0;
    pfc_status status = PFC_OK;
    const double tol = adj_tol * bnorm;
    if (H->nlev == 1) {  // solved in one cycle: the host decides (4^3 285 us in units, here 251)
        for (double rho = bnorm; rho > tol; ++c) {
            if (c == H->cfg.max_cycles) {
                status = PFC_ERR_NOT_CONVERGED;
                break;
            }
            adj_cycle(H, 0, H->cfg.cycle == PFC_CYCLE_F, false);
            st = read_norm(H, adj_norm(H), &rho);
            if (st != PFC_OK) return st;
            if (!std::isfinite(rho)) {
                status = PFC_ERR_NONFINITE;
                ++c;
                break;
            }
        }
    } else if (bnorm > 0.0) {  // the first unit tests |b| itself
        RunHost r{};
        st = run_units(
            H, tol, bnorm,
            [&](int i, bool ride) { unit_stop_test(H, i & 1, parts, tol, A.brick && ride); },
            [&](int) {
                adj_cycle(H, 0, H->cfg.cycle == PFC_CYCLE_F, false, A.brick);
                parts = adj_norm(H);
            },
            &r);
        if (st != PFC_OK) return st;
        c = r.cycles;
        status = r.status;
    }
    if (status == PFC_OK || status == PFC_ERR_NOT_CONVERGED) {
        // lambda back to natural order (level-0 scratch), then accumulate
        launch_from_lay<double, double>(H->stream, A.lay, A.u.a, A.ubar.a, 3);
        OpParams op = op_of(H, 0);
        op.lay = nat;
        const Tri<const double> lam{A.ubar.a, A.ubar.b, A.ubar.c};
        hipLaunchKernelGGL(k_adj_accum_cur, dim3(blocks_for(P)), dim3(kBlock), 0, H->stream, op, lam,
                           phi_next, phi_cur, gbar_cur);
        hipLaunchKernelGGL(k_adj_accum_prev, dim3(blocks_for(P)), dim3(kBlock), 0, H->stream, op,
                           (const double *)A.ubar.b, gbar_prev);
        const unsigned eb = reduce_blocks(P);
        hipLaunchKernelGGL(k_adj_eps_part, dim3(eb), dim3(kBlock), 0, H->stream, P,
                           (const double *)A.ubar.b, phi_next, phi_cur, H->energy_part);
        hipLaunchKernelGGL(k_adj_eps_final, dim3(1), dim3(kBlock), 0, H->stream,
                           (const double *)H->energy_part, (int)eb, geps);
    }
    HIP_TRY(H, hipGetLastError());
    HIP_TRY(H, hipStreamSynchronize(H->stream));
    if (cycles) *cycles = c;
    if (status != PFC_OK) return fail(H, status, pfc_status_string(status));
    return PFC_OK;
}

}  // namespace pfc

extern "C" pfc_status pfc_adjoint_step(pfc_handle *h, const double *phi_prev, const double *phi_cur,
                                       const double *phi_next, const double *gbar_next,
                                       double *gbar_cur, double *gbar_prev, double *geps,
                                       double adj_tol, int32_t *cycles) {
    if (!h) return PFC_ERR_INVALID_ARG;
    if (!phi_prev || !phi_cur || !phi_next || !gbar_next || !gbar_cur || !gbar_prev || !geps)
        return pfc::fail(h, PFC_ERR_INVALID_ARG, "NULL pointer");
    if (!(adj_tol > 0.0) || !std::isfinite(adj_tol))
        return pfc::fail(h, PFC_ERR_INVALID_ARG, "adj_tol must be > 0");
    if (h->cfg.mobility != PFC_MOBILITY_ONE)
        return pfc::fail(h, PFC_ERR_INVALID_ARG, "the adjoint is derived for constant mobility");
    if (h->cfg.scheme != PFC_SCHEME_CS2)
        return pfc::fail(h, PFC_ERR_INVALID_ARG, "the adjoint is derived for scheme (1.10)");
    if (gbar_next == gbar_cur || gbar_next == gbar_prev)
        return pfc::fail(h, PFC_ERR_INVALID_ARG, "gbar_next aliases an output");
    return pfc::adjoint_step(h, phi_prev, phi_cur, phi_next, gbar_next, gbar_cur, gbar_prev, geps,
                             adj_tol, cycles);
}
