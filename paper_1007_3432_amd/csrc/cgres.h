// FP64 conjugate gradient on Q = M^T M (Sec. 4.1), plain and preconditioned
// (Sec. 4.2), with the whole solve resident on the chip: lattices too large
// for one workgroup and small enough that the vectors and links fit the
// registers of one block per CU (restile.h).
//
// Plain CG with one grid sum an iteration, over x, r and p:
//   1. q = Q p; its rim goes to the neighbours and the block's r.r, p.q, r.q
//      and q.q to the grid sum (gridsum.h);
//   2. alpha = r.r / p.q; |r - alpha q|^2 = r.r - 2 alpha r.q + alpha^2 q.q over r.r
//      gives beta before the new r exists (after Saad 1985 and Meurant 1987); x +=
//      alpha p, r -= alpha q, p = r + beta p.
//      On the halo, where q has come from the neighbours, r and p follow the
//      same recurrences: the block keeps the values that their owners have.
// Only beta rests on the expanded square: alpha and the convergence test take
// the r.r that is summed anew, and Q p is formed anew, in every iteration.  So
// the iterations are those of Hestenes and Stiefel's arrangement also where the
// coupling is strong.  (With Q p and p.Qp by recurrence, after Chronopoulos and
// Gear, which is as fast, d = 1 64 x 128 at U = -6 took up to 22% more iterations
// to 1e-12, and after a residual had been replaced the p.Qp of one of the next
// steps came out negative: in 22 of 110 solves between U = -2 and -7 emulated on
// the host, all of which converge now.)
// The kernel ends when r.r meets tol, after a number of iterations, or when
// it cannot go on; the state is in memory then.  Convergence is decided
// between launches as in the other solvers: the true residual phi - Q x
// replaces r, and if it does not meet tol the iteration starts again from it, p
// = r.  (Keeping p, as the multi-kernel solver does, took as many iterations in
// most of those solves, and one then went on replacing without an end.)
//
// What bounds an iteration is the grid sum (1.8 to 2.5 us), the halo read after
// it and the LDS traffic of the stencils, where it was three kernels and 80
// bytes a site of memory traffic.  Before and now, us an iteration: d = 1
// 256 x 128 9.4 and 3.0, 4096 x 128 15.2 and 4.2, 2048 x 512 20.5 and 4.8; d = 2
// 33 x 60 11.9 and 3.4; d = 3 8^3 x 80 12.1 and 3.3, 16^3 x 128 17.2 and 5.8.
// (Hestenes and Stiefel's arrangement, with two grid sums an iteration, took
// 4.5, 5.7, 7.0, 5.3, 4.8 and 11.0.)
#pragma once

#include <utility>

#include "restile.h"

namespace hub {

template <int D, bool WHOLE, int KO, int KY, int KH>
__global__ __launch_bounds__(kResBlock) void k_cg_resident(ResArgs a) {
    extern __shared__ __align__(16) double res_lds[];
    ResTile<D, WHOLE, KO, KY, KH> T;
    T.init(a, res_lds);
    GridSum<4> gs{a.slots, res_lds, a.limit, 0};
    auto give_up = [&]() {
        if (threadIdx.x == 0)
            __hip_atomic_store(&a.st->given_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    double x[KO], r[KO], p[KO];
    double rh[KH], ph[KH];
    ResState c{};
    if (a.mode != kResFirst) c = *a.st;
    const double* r0 = a.mode == kResFirst ? a.phi : a.R;
    const double* p0 = a.mode == kResOn ? a.P : r0;
#pragma unroll
    for (int k = 0; k < KO; ++k) {
        r[k] = T.ook[k] ? *at(r0, T.ogi[k]) : 0.0;
        p[k] = T.ook[k] ? *at(p0, T.ogi[k]) : 0.0;
        x[k] = T.ook[k] && a.mode != kResFirst ? *at(a.x, T.ogi[k]) : 0.0;
    }
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        rh[k] = *at(r0, T.hgi[k]);
        ph[k] = *at(p0, T.hgi[k]);
    }

    for (int n = 0;; ++n) {
        double q[KO];
        T.apply_q(p, ph, q);
        T.publish(q);
        double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            part[0] += r[k] * r[k];
            part[1] += p[k] * q[k];
            part[2] += r[k] * q[k];
            part[3] += q[k] * q[k];
        }
        gs.deposit(part);
        double sum[4];
        if (!gs.wait(sum)) return give_up();
        double qh[KH];
        T.fetch(qh);
        const double rr = sum[0], pq = sum[1];
        const bool first = n == 0 && a.mode != kResOn;
        if (first && a.mode == kResFirst) c.phi2 = rr;
        // (A residual just replaced has not met tol by the sum that decides.)
        if (!isfinite(rr)) c.done = kDoneBreakdown;
        else if (rr <= a.tol2 * c.phi2 && !(first && a.mode == kResReplaced))
            c.done = kDoneIterConverged;
        else if (c.iter >= a.max_iter) c.done = kDoneMaxIter;
        else if (n < a.iters && (!(pq > 0.0) || !isfinite(pq))) c.done = kDoneBreakdown;
        if (c.done != kRunning || n == a.iters) break;
        const double inv = 1.0 / pq, alpha = rr * inv;
        const double beta = fmax(1.0 + (alpha * sum[3] - 2.0 * sum[2]) * inv, 0.0);
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            x[k] = x[k] + alpha * p[k];
            r[k] = r[k] - alpha * q[k];
            p[k] = r[k] + beta * p[k];
        }
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            rh[k] = rh[k] - alpha * qh[k];
            ph[k] = rh[k] + beta * ph[k];
        }
        ++c.iter;
    }
#pragma unroll
    for (int k = 0; k < KO; ++k)
        if (T.ook[k]) {
            const int i = fresh(T.ogi[k]);
            *at_w(a.x, i) = x[k];
            *at_w(a.R, i) = r[k];
            *at_w(a.P, i) = p[k];
        }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // Not given_up, which another block may write.
        a.st->phi2 = c.phi2;
        a.st->iter = c.iter;
        a.st->done = c.done;
    }
}

// Preconditioned CG, z = P(Q) r by n quadratic factors (cheb.h), two products
// with Q each, every product's input rim going to the neighbours before it.
// The sums are those of the standard method (rho = r.z, p.Qp), and r.r, which
// decides convergence, travels while the first product is formed.  An
// iteration is 2n + 1 products; what bounds it is the exchange before each of
// them (about 2 us), the halo read and their LDS traffic, where each product
// was a sweep over memory: us a product, before and now, 16^3 x 128 (n = 16)
// 6.9 and 4.7, 4096 x 128 (16) 5.0 and 3.2, 2048 x 512 (32) 6.2 and 3.3, 64^2
// x 60 (8) 7.6 and 3.3, 8^3 x 80 (8) 5.6 and 2.7, 32 x 64 (8) 3.3 and 2.0.  x
// is in memory: it is touched once in 2n + 1 products.
template <int D, bool WHOLE, int KO, int KY, int KH>
__global__ __launch_bounds__(kResBlock) void k_pcg_resident(ResArgs a) {
    extern __shared__ __align__(16) double res_lds[];
    ResTile<D, WHOLE, KO, KY, KH> T;
    T.init(a, res_lds);
    GridSum<1> gs{a.slots, res_lds, a.limit, 0};
    auto give_up = [&]() {
        if (threadIdx.x == 0)
            __hip_atomic_store(&a.st->given_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    double r[KO], p[KO];
    ResState c{};
    if (a.mode == kResFirst) {
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            r[k] = T.ook[k] ? *at(a.phi, T.ogi[k]) : 0.0;
            p[k] = 0.0;
            if (T.ook[k]) *at_w(a.x, T.ogi[k]) = 0.0;
        }
    } else {
        c = *a.st;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            r[k] = T.ook[k] ? *at(a.R, T.ogi[k]) : 0.0;
            p[k] = T.ook[k] ? *at(a.P, T.ogi[k]) : 0.0;
        }
    }
    int mode = a.mode, n = 0;
    for (;;) {
        double v[KO], t[KO], vh[KH];
        double part[1] = {0.0}, sum[1];
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            v[k] = r[k];
            part[0] += r[k] * r[k];
        }
        T.publish(v);
        gs.deposit(part);
        if (!T.exchange()) return give_up();
        T.fetch(vh);
        T.apply_q(v, vh, t);
        if (!gs.wait(sum)) return give_up();
        const double rr = sum[0];
        if (mode == kResFirst) c.phi2 = rr;
        // (A residual just replaced has not met tol by the sum that decides.)
        if (!isfinite(rr)) c.done = kDoneBreakdown;
        else if (rr <= a.tol2 * c.phi2 && mode != kResReplaced) c.done = kDoneIterConverged;
        else if (c.iter >= a.max_iter) c.done = kDoneMaxIter;
        if (c.done != kRunning || n == a.iters) break;
        for (int j = 0;;) {
            double z[KO];
            T.publish(t);
            if (!T.exchange()) return give_up();
            T.fetch(vh);
            T.apply_q(t, vh, z);
            const double c2 = a.f[3 * j], c1 = a.f[3 * j + 1], c0 = a.f[3 * j + 2];
#pragma unroll
            for (int k = 0; k < KO; ++k) v[k] = c2 * z[k] + c1 * t[k] + c0 * v[k];
            if (++j == a.nf) break;
            T.publish(v);
            if (!T.exchange()) return give_up();
            T.fetch(vh);
            T.apply_q(v, vh, t);
        }
        part[0] = 0.0;
#pragma unroll
        for (int k = 0; k < KO; ++k) part[0] += r[k] * v[k];
        gs.deposit(part);
        if (!gs.wait(sum)) return give_up();
        const double rz = sum[0];
        if (!(rz > 0.0) || !isfinite(rz)) {
            c.done = kDoneBreakdown;
            break;
        }
        const double beta = mode == kResOn ? rz / c.rho : 0.0;
        c.rho = rz;
        mode = kResOn;
        part[0] = 0.0;
#pragma unroll
        for (int k = 0; k < KO; ++k) p[k] = v[k] + beta * p[k];
        T.publish(p);
        if (!T.exchange()) return give_up();
        T.fetch(vh);
        T.apply_q(p, vh, t);
#pragma unroll
        for (int k = 0; k < KO; ++k) part[0] += p[k] * t[k];
        gs.deposit(part);
        if (!gs.wait(sum)) return give_up();
        const double pq = sum[0];
        if (!(pq > 0.0) || !isfinite(pq)) {
            c.done = kDoneBreakdown;
            break;
        }
        const double alpha = rz / pq;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            if (T.ook[k]) {
                double* xk = at_w(a.x, fresh(T.ogi[k]));
                *xk = *xk + alpha * p[k];
            }
            r[k] = r[k] - alpha * t[k];
        }
        ++c.iter;
        ++n;
    }
#pragma unroll
    for (int k = 0; k < KO; ++k)
        if (T.ook[k]) {
            const int i = fresh(T.ogi[k]);
            *at_w(a.R, i) = r[k];
            *at_w(a.P, i) = p[k];
        }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // Not given_up, which another block may write.
        a.st->rho = c.rho;
        a.st->phi2 = c.phi2;
        a.st->iter = c.iter;
        a.st->done = c.done;
    }
}

// The kernel of a dimension, level and cut (cgres_d1.hip, _d2, _d3).
using ResKernel = void (*)(ResArgs);
template <int D, int L>
ResKernel res_kernel_l(bool whole, bool pcg) {
    constexpr ResLevel K = kResLevels[L];
    if constexpr (K.whole)
        if (whole)
            return pcg ? &k_pcg_resident<D, true, K.own, K.rim, K.halo>
                       : &k_cg_resident<D, true, K.own, K.rim, K.halo>;
    return pcg ? &k_pcg_resident<D, false, K.own, K.rim, K.halo>
               : &k_cg_resident<D, false, K.own, K.rim, K.halo>;
}
template <int D, int... L>
ResKernel res_kernel_of(int level, bool whole, bool pcg, std::integer_sequence<int, L...>) {
    ResKernel k = nullptr;
    (void)((level == L ? (k = res_kernel_l<D, L>(whole, pcg), true) : false) || ...);
    return k;
}
template <int D>
ResKernel res_kernel_d(int level, bool whole, bool pcg) {
    return res_kernel_of<D>(level, whole, pcg, std::make_integer_sequence<int, kResLevelCount>());
}
ResKernel res_kernel_d1(int level, bool whole, bool pcg);
ResKernel res_kernel_d2(int level, bool whole, bool pcg);
ResKernel res_kernel_d3(int level, bool whole, bool pcg);

}  // namespace hub
