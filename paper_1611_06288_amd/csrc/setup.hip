// Set-up and end of a time step on the finest level, one launch each, and the
// same for all instances of a batch.
//
// Begin: from the caller's natural-order phi^k, phi^{k-1}, mu and omega the
// source S (scheme-PFC-s1..s3), the starting iterate (phi^k, mu, omega) and phi^k
// in the level's colour-split storage.  End: the iterate back to natural order.
// Bound by memory (88 and 48 B per point) on large levels and by launches on
// small ones: as a source launch and four conversions (begin) and three (end)
// these were 8 launches of 4.4 us and more per step, 512 for a batch of 64.
// A thread owns an x-pair of points, one of each colour, as the conversions do.
// 256^3: begin 487 -> 321 us, end 255 -> 134; ensemble of 64, one step with its
// states in and out, 66.9 -> 65.2 ms.
#include "device_common.h"

namespace pfc {

namespace {

struct XP {
    double v[2];
};

__device__ __forceinline__ XP ldp(const double *p) { return *reinterpret_cast<const XP *>(p); }

// Position t of an x-pair in either colour's block: its row, storage offsets of
// the even and the odd point, natural offset of the even one.
struct Where {
    unsigned j, k, i, q0, q1, nat;
    __device__ __forceinline__ Where(const Lay &L, unsigned t) {
        const unsigned n = (unsigned)L.n, hn = n >> 1, H = n * n * hn;
        const unsigned row = L.dh.q(t);
        k = L.dn.q(row);
        j = row - k * n;
        i = 2 * (t - row * hn);
        const unsigned odd = (j + k) & 1u;  // colour of the even point
        q0 = odd * H + t;
        q1 = (odd ^ 1u) * H + t;
        nat = row * n + i;
    }
};

// Laplacians of v at the pair's points, own values in c (neighbours in nsum's order).
__device__ __forceinline__ void pair_lap(const double *__restrict__ v, const Where &w, int n, double h2inv,
                                         XP &c, double (&l)[2]) {
    const unsigned un = (unsigned)n;
    const unsigned base = w.nat - w.i;
    const unsigned yp = (w.k * un + (unsigned)wrap_p((int)w.j, n)) * un + w.i;
    const unsigned ym = (w.k * un + (unsigned)wrap_m((int)w.j, n)) * un + w.i;
    const unsigned zp = ((unsigned)wrap_p((int)w.k, n) * un + w.j) * un + w.i;
    const unsigned zm = ((unsigned)wrap_m((int)w.k, n) * un + w.j) * un + w.i;
    c = ldp(v + w.nat);
    const double xm = v[base + (unsigned)wrap_m((int)w.i, n)];
    const double xp = v[base + (unsigned)wrap_p((int)w.i + 1, n)];
    const XP a = ldp(v + yp), b = ldp(v + ym), d = ldp(v + zp), e = ldp(v + zm);
    l[0] = ((c.v[1] + xm) + (a.v[0] + b.v[0]) + (d.v[0] + e.v[0]) - 6.0 * c.v[0]) * h2inv;
    l[1] = ((xp + c.v[0]) + (a.v[1] + b.v[1]) + (d.v[1] + e.v[1]) - 6.0 * c.v[1]) * h2inv;
}

__device__ __forceinline__ void begin_pair(const OpParams &op, unsigned t, const double *__restrict__ cur,
                                           const double *__restrict__ prev, const double *__restrict__ mu,
                                           const double *__restrict__ om, const Tri<double> &f,
                                           const Tri<double> &u, double *phk) {
    const Where w(op.lay, t);
    XP a, b;
    double lk[2], lp[2];
    pair_lap(cur, w, op.lay.n, op.h2inv, a, lk);
    pair_lap(prev, w, op.lay.n, op.h2inv, b, lp);
    const XP m = ldp(mu + w.nat), o = ldp(om + w.nat);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const unsigned q = e ? w.q1 : w.q0;
        const double v = a.v[e];
        f.a[q] = v;
        if (op.fo) {  // first-order scheme: (phi^k, 2 Lap phi^k, 0)
            f.b[q] = 2.0 * lk[e];
            f.c[q] = 0.0;
        } else {
            f.b[q] = 0.5 * (1.0 - op.eps) * v + 3.0 * lk[e] - lp[e];
            f.c[q] = 0.5 * lk[e];
        }
        u.a[q] = v;
        u.b[q] = m.v[e];
        u.c[q] = o.v[e];
        phk[q] = v;
    }
}

__device__ __forceinline__ void end_pair(const Lay &L, unsigned t, const Tri<double> &u, double *phi,
                                         double *mu, double *om) {
    const Where w(L, t);
    *reinterpret_cast<XP *>(phi + w.nat) = XP{{u.a[w.q0], u.a[w.q1]}};
    *reinterpret_cast<XP *>(mu + w.nat) = XP{{u.b[w.q0], u.b[w.q1]}};
    *reinterpret_cast<XP *>(om + w.nat) = XP{{u.c[w.q0], u.c[w.q1]}};
}

__device__ __forceinline__ unsigned half_points(const Lay &L) {
    return (unsigned)L.n * (unsigned)L.n * ((unsigned)L.n >> 1);
}

}  // namespace

__global__ __launch_bounds__(kBlock) void k_step_begin(OpParams op, const double *cur, const double *prev,
                                                       const double *mu, const double *om, Tri<double> f,
                                                       Tri<double> u, double *phk) {
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t < half_points(op.lay)) begin_pair(op, t, cur, prev, mu, om, f, u, phk);
}

__global__ __launch_bounds__(kBlock) void k_step_end(Lay L, Tri<double> u, double *phi, double *mu,
                                                     double *om) {
    const unsigned t = xcd_block() * kBlock + threadIdx.x;
    if (t < half_points(L)) end_pair(L, t, u, phi, mu, om);
}

void launch_step_begin(hipStream_t s, const OpParams &op, const double *cur, const double *prev,
                       const double *mu, const double *om, Tri<double> f, Tri<double> u, double *phk) {
    hipLaunchKernelGGL(k_step_begin, dim3(blocks_for(npts_host(op.lay) / 2)), dim3(kBlock), 0, s, op, cur,
                       prev, mu, om, f, u, phk);
}

void launch_step_end(hipStream_t s, const Lay &L, Tri<double> u, double *phi, double *mu, double *om) {
    hipLaunchKernelGGL(k_step_end, dim3(blocks_for(npts_host(L) / 2)), dim3(kBlock), 0, s, L, u, phi, mu, om);
}

// ---------------------------------------------------------- batched form

__global__ __launch_bounds__(kBlock) void kb_step_begin(const BatchIO *__restrict__ io,
                                                        const BlockRef *__restrict__ blocks, int ip, int ic) {
    const BlockRef b = blocks[xcd_block()];
    const BatchIO &q = io[b.seg];
    const unsigned t = b.blk * kBlock + threadIdx.x;
    if (t < half_points(q.op.lay)) begin_pair(q.op, t, q.p[ic], q.p[ip], q.mu, q.om, q.f, q.u, q.phk);
}

__global__ __launch_bounds__(kBlock) void kb_step_end(const BatchIO *__restrict__ io,
                                                      const BlockRef *__restrict__ blocks, int in) {
    const BlockRef b = blocks[xcd_block()];
    const BatchIO &q = io[b.seg];
    const unsigned t = b.blk * kBlock + threadIdx.x;
    if (t < half_points(q.op.lay)) end_pair(q.op.lay, t, q.u, q.p[in], q.mu, q.om);
}

// 8-child means of one depth's phi^k, the children added as k_restrict does.
__global__ __launch_bounds__(kBlock) void kb_restrict(const RestrictSeg *__restrict__ segs,
                                                      const BlockRef *__restrict__ blocks) {
    const BlockRef b = blocks[xcd_block()];
    const RestrictSeg &g = segs[b.seg];
    const unsigned tn = b.blk * kBlock + threadIdx.x;
    if (tn >= (unsigned)npts(g.coarse)) return;
    int I, J, K;
    decode_nat(g.coarse, tn, I, J, K);
    double s = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c)
        s += g.from[sidx32(g.fine, 2 * I + (c & 1), 2 * J + (c >> 1 & 1), 2 * K + (c >> 2))];
    g.to[sidx32(g.coarse, I, J, K)] = 0.125 * s;
}

void launch_batch_begin(hipStream_t s, const BatchIO *io, const BlockRef *blocks, unsigned count, int ip,
                        int ic) {
    hipLaunchKernelGGL(kb_step_begin, dim3(count), dim3(kBlock), 0, s, io, blocks, ip, ic);
}

void launch_batch_end(hipStream_t s, const BatchIO *io, const BlockRef *blocks, unsigned count, int in) {
    hipLaunchKernelGGL(kb_step_end, dim3(count), dim3(kBlock), 0, s, io, blocks, in);
}

void launch_batch_restrict(hipStream_t s, const RestrictSeg *segs, const BlockRef *blocks, unsigned count) {
    hipLaunchKernelGGL(kb_restrict, dim3(count), dim3(kBlock), 0, s, segs, blocks);
}

}  // namespace pfc
