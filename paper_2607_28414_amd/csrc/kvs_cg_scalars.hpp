// The scalar steps of the projection's CG (Sec. 3.2.3) on the device control
// block, and their place: either one-block kernels between the sweeps, or
// ("folded") the start of the sweep that needs them.  In the folded form every
// block of a sweep sums the partials that the sweep before it left, in the
// same fixed order, and forms the same scalars in LDS; block 0 also writes the
// new control block, into the other of two copies, so no block reads what
// another one is writing.  That takes a launch (3 to 5 us with its gap) out of
// each half iteration; every block re-reads the partials, so it is used up to
// kFoldMax of them.  us per iteration, kernels between the sweeps and folded
// (blocks): FP32 48^3 (92) 12.9, 11.9; 128^3 (252) 21.6, 20.4; 256^3 (504) 95.2, 93.3;
// FP64 48^3 (138) 16.5, 14.0; 128^3 (256) 39.8, 36.4; 256^3 (512) 205, 201; beyond
// the line, FP32 320 x 256 x 256 (1512) 156.3, 157.7.
#pragma once

#include "kvs_internal.hpp"

namespace {

// Partials up to which the scalars are folded into the sweeps.
constexpr int kFoldMax = 1024;

// The stop test after an iteration that left r.r in s.rr.
__device__ __forceinline__ void cg_stop_test(CgState& s) {
    if (s.fixed_iters > 0) {
        if (s.iters >= s.fixed_iters) s.done = 1;
    } else if (sqrt(s.rr / s.bb) < sqrt(s.tol2)) {
        s.done = 1;
    } else if (s.iters >= s.max_iter) {
        s.status = KVS_ENOTCONV;
        s.done = 1;
    }
}

// alpha = r.z / p.Ap with the breakdown guard
__device__ __forceinline__ void cg_apply_alpha(CgState& s, double pap) {
    s.pAp = pap;
    if (!(pap > 0.0) || !isfinite(pap)) {
        s.status = KVS_EBREAKDOWN;
        s.done = 1;
    } else {
        s.alpha = s.rz / pap;
    }
}

// plain CG / Jacobi-PCG: beta, r.r, the count and the stop test
__device__ __forceinline__ void cg_apply_beta(CgState& s, double rr, double rz) {
    s.iters += 1;
    if (!isfinite(rr) || rr < 0.0 || !isfinite(rz)) {
        s.status = KVS_EBREAKDOWN;
        s.done = 1;
        return;
    }
    const double rz_new = s.jacobi ? rz : rr;
    s.beta = rz_new / s.rz;
    s.rz = rz_new;
    s.rr = rr;
    cg_stop_test(s);
}

// Smallest r1.r1 / r.r a pair's second iteration is formed from.  r1.r1 and
// p1.A p1 are differences of sums the size of r.r and p.q, with about 1e-15 of
// those in rounding error: below 1e-15 / kPairFall they would have no digits.
// On a grid of a few unknowns one iteration takes the residual to 0, and the
// second one went along a direction of noise with a step of any size (3 x 3 x 3
// nodes with Jacobi: phi off by half, KVS_ENOTCONV).  On ordinary grids r1.r1 /
// r.r stays above 0.1 (20^3 to 60^3 nodes, 100 to 300 iterations).
constexpr double kPairFall = 1e-6;

// Two iterations at once (kvs_cg_pair.hip): the coefficients of the pair from
// p.q, r.q, q.q, r.Ar, q.Ar, q.Aq; one iteration alone where it ends the solve,
// the residual falls by more than kPairFall or the second has no positive p.Ap.
__device__ __forceinline__ void cg_apply_pair(CgState& s, double pq, double rq, double qq, double rar, double qar,
                                              double qaq) {
    s.pAp = pq;
    if (!(pq > 0.0) || !isfinite(pq)) {
        s.status = KVS_EBREAKDOWN;
        s.done = 1;
        return;
    }
    const double zs = s.jacobi ? s.dinv : 1.0;
    const double a0 = s.rz / pq;
    const double r11 = s.rr - 2.0 * a0 * rq + a0 * a0 * qq;
    const double b0 = r11 / s.rr;
    const double pap1 = zs * zs * (rar - 2.0 * a0 * qar + a0 * a0 * qaq) + 2.0 * zs * b0 * (rq - a0 * qq) + b0 * b0 * pq;
    const long long last = s.fixed_iters > 0 ? s.fixed_iters : s.max_iter;
    const bool met = s.fixed_iters <= 0 && !(sqrt(r11 / s.bb) >= sqrt(s.tol2));
    const bool two = !met && s.iters + 1 < last && r11 > kPairFall * s.rr && isfinite(r11) && pap1 > 0.0 && isfinite(pap1);
    s.alpha = a0;
    s.pair_a0 = a0;
    s.pair_b0 = two ? b0 : 0.0;
    s.pair_a1 = two ? zs * r11 / pap1 : 0.0;
    s.pair_r11 = r11;
    s.pair_m = two ? 2 : 1;
}

// After the pair's update: r.r of the residual as stored.
__device__ __forceinline__ void cg_apply_pair_end(CgState& s, double rr) {
    s.iters += s.pair_m;
    if (!isfinite(rr) || rr < 0.0) {
        s.status = KVS_EBREAKDOWN;
        s.done = 1;
        return;
    }
    s.beta = rr / (s.pair_m == 2 ? s.pair_r11 : s.rr);
    s.rr = rr;
    s.rz = s.jacobi ? s.dinv * rr : rr;
    cg_stop_test(s);
}

// A value that is the same in every lane, held in scalar registers (read from
// a control block in LDS it would take two vector registers).
__device__ __forceinline__ double cg_uniform(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

enum CgScalars { CG_ALPHA = 0, CG_BETA = 1, CG_PAIR = 2, CG_PAIR_END = 3 };
template <int MODE>
constexpr int cg_sums() {
    return MODE == CG_PAIR ? 6 : MODE == CG_BETA ? 2 : 1;
}

// Fixed-order sums of NS partial arrays by a block of NT >= 256 threads: 256
// strided running sums, then a tree; sum s is left in sh[s][0].
template <int NS, int NT>
__device__ __forceinline__ void cg_sum_partials(const double* part, int count, int stride, int tid, double (&sh)[NS][256]) {
    constexpr int G = NT / 256;  // groups of 256 threads, one sum each at a time
    const int g = tid >> 8, t = tid & 255;
    if (g < G)
        for (int s = g; s < NS; s += G) {
            double acc = 0.0;
            for (int q = t; q < count; q += 256) acc += part[s * stride + q];
            sh[s][t] = acc;
        }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (g < G && t < o)
            for (int s = g; s < NS; s += G) sh[s][t] += sh[s][t + o];
        __syncthreads();
    }
}

template <int MODE>
__device__ __forceinline__ void cg_apply(CgState& s, const double (*sh)[256]) {
    if constexpr (MODE == CG_ALPHA) {
        cg_apply_alpha(s, sh[0][0]);
    } else if constexpr (MODE == CG_BETA) {
        cg_apply_beta(s, sh[0][0], sh[1][0]);
    } else if constexpr (MODE == CG_PAIR) {
        cg_apply_pair(s, sh[0][0], sh[1][0], sh[2][0], sh[3][0], sh[4][0], sh[5][0]);
    } else {
        cg_apply_pair_end(s, sh[0][0]);
    }
}

// Folded scalars of a sweep: `in` the control block before them, `out` the
// copy that block 0 fills (null: not folded, `in` is current), the partials of
// the sweep before.
struct CgFold {
    const CgState* in;
    CgState* out;
    const double* part;
    int count, stride;
};

// The control block a sweep works with.  MODE is what its scalars step is: the
// end of an iteration (CG_BETA, CG_PAIR_END: only when an update's sums are
// `pending`) or its middle (CG_ALPHA, CG_PAIR: the update that follows will
// leave its sums pending).  Contains block barriers: every thread calls it.
template <int MODE, int NT>
__device__ __forceinline__ const CgState* cg_fold(const CgFold& f, int tid) {
    if (!f.out) return f.in;
    constexpr bool END = MODE == CG_BETA || MODE == CG_PAIR_END;
    constexpr int NS = cg_sums<MODE>();
    __shared__ CgState s;
    __shared__ double sh[NS][256];
    const bool need = !f.in->done && (!END || f.in->pending);
    if (tid == 0) s = *f.in;
    if (need) cg_sum_partials<NS, NT>(f.part, f.count, f.stride, tid, sh);
    if (tid == 0) {
        if (need) {
            cg_apply<MODE>(s, sh);
            s.pending = !END && !s.done;
        }
        if (blockIdx.x == 0) *f.out = s;
    }
    __syncthreads();
    return &s;
}

// The same step as a kernel of one block, in place.  Folded solves launch it
// for the end of an iteration before the host reads the control block.
template <int MODE>
__global__ __launch_bounds__(256) void cg_scalars_kernel(const double* part, int count, int stride, int pending_only,
                                                         CgState* st) {
    constexpr int NS = cg_sums<MODE>();
    __shared__ double sh[NS][256];
    if (st->done || (pending_only && !st->pending)) return;
    cg_sum_partials<NS, 256>(part, count, stride, threadIdx.x, sh);
    if (threadIdx.x == 0) {
        cg_apply<MODE>(*st, sh);
        st->pending = 0;
    }
}

}  // namespace
