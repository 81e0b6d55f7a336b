// Device-resident scalar state of the multishift CG and the two scalar stages
// of an iteration: alpha after the first stencil's norms, beta after the
// second's.  A stage runs either in a kernel of its own (one block per RHS) or
// inside a stencil launch: then every block of the launch forms the one value
// its sites need (alpha or beta) from the previous launch's partial sums, and
// one extra block per RHS runs the whole stage beside them.
#pragma once

#include "../../include/ovl.h"
#include "device.h"

namespace ovl {

constexpr int NR = OVL_MAX_RHS;
constexpr int NS = OVL_MAX_SHIFTS;
constexpr int MB = OVL_MAX_BLOCK;   // longest block of the blocked shift update

// Coefficients of the blocked shift update.  Over a block of iterations
// k0..k0+T-1 the shift recurrences x_j += a_j p_j, p_j = z_j' r + b_j p_j are
// linear in the block-start p_j and the stored residuals r^{k0+1..k0+T}:
//   p_j^{k0+t} = P p_j^{k0} + sum_{i<=t} C_i r^{k0+i},
//   x_j^{k0+T} = x_j^{k0} + XP p_j^{k0} + sum_i X_i r^{k0+i}.
struct Blk {
    double P[NR][NS], XP[NR][NS];
    double C[NR][NS][MB + 1], X[NR][NS][MB + 1];
    int inblk[NR][NS];   // shift active when the block started
    int t[NR];           // iterations done in the current block
};
// Scalar state of a multishift CG on (Q^2 + s_j) x_j = b, one system per RHS,
// kept in device memory so the iteration runs without host round trips.
struct MState {
    double rr[NR], bb[NR], alpha[NR], alpha_old[NR], beta[NR];
    double zeta[NR][NS], zeta_old[NR][NS], zeta_new[NR][NS], aj[NR][NS], bj[NR][NS];
    double delta[NS];      // s_j - s0 (shift offsets from the base shift)
    double s0r[NR];        // base shift of each RHS system
    double tol2r[NR];      // squared relative tolerance of each RHS system
    int act[NR][NS];       // shift still iterating
    int act_cur[NR][NS];   // shifts updated in the current iteration
    int frozen_at[NR][NS];
    double frozen_rr[NR][NS];   // zeta^2 |r|^2 of a shift at the iteration it froze
    int iter[NR];
    int skip[NR];          // RHS finished (every shift frozen) or failed (set by K_b alone during a solve)
    int nonfinite[NR];
    int nrhs, nshift;
    int jlive;             // an RHS is finished once systems jlive.. are frozen (1: system 0 is a base
                           // that only carries the others)
    // reliable-update bookkeeping (mixed solver)
    double rr_ref[NR];     // |r|^2 at the last residual replacement
    int want_update[NR];
    // hand-over to another precision: an RHS whose base residual reached the
    // hand-over level stops (skip set, paused set) until the solve that
    // continues its recurrences clears both
    int paused[NR];
    int run_c[NR];         // the RHS takes part in this iteration: its p0 (or t) update is due (set and
                           // cleared by K_a alone)
    double one[NR];        // 1 per RHS: the alpha of a residual replacement's update stencil
    double rr_iter[NR];    // |r|^2 at the start of this iteration (set by K_a): what beta divides by
                           // in the blocks that run beside the beta stage, which replaces rr
};

enum { PRO_NONE = 0, PRO_ALPHA = 1, PRO_BETA = 2, PRO_LANCZOS = 3 };

// A scalar stage carried by a kernel: its partial sums (row stride pstride, of
// which the first pcnt slots count) and the state it updates.
struct ProArgs {
    int kind;
    int pcnt, pstride;
    int nrhs;
    int shifted;   // PRO_ALPHA: some RHS's base shift is not 0 (|p|^2 enters)
    const double *pin;
    MState *st;
    Blk *bk;       // block coefficients (null: none kept)
    double sw2;    // PRO_BETA: pause an RHS with |r|^2 <= sw2 |b|^2 (0: never)
    int reset;     // PRO_ALPHA: a block's first iteration, which starts its coefficients
    double *tab;   // PRO_LANCZOS: the step's coefficients (LzTab) and, bout, where |u| goes
    double *bout;
};

// Sum of n slots, valid in every thread of a block of NT threads.  The order
// does not depend on NT: 256 strided sums, a butterfly over each 64 of them,
// then those four in pairs; so a stage gives the same bits in its own kernel
// and in any stencil that carries it.  slot_part is a thread's share (loads
// only; a block of one wave holds four of the strided sums per thread),
// slot_fold the rest.
template <int NT>
struct SlotPart {
    static constexpr int N = NT == 64 ? 4 : 1;
    double v[N] = {};
};
template <int NT>
__device__ __forceinline__ SlotPart<NT> slot_part(const double *p, int n)
{
    SlotPart<NT> s;
    if (threadIdx.x < 256)
#pragma unroll
        for (int w = 0; w < SlotPart<NT>::N; w++)
            for (int k = threadIdx.x + 64 * w; k < n; k += 256) s.v[w] += p[k];
    return s;
}
template <int NT>
__device__ __forceinline__ double slot_fold(SlotPart<NT> s, double *lds /* >= 4 */)
{
    static_assert(NT == 64 || NT == 256 || NT == 512, "slot_fold: block size");
#pragma unroll
    for (int w = 0; w < SlotPart<NT>::N; w++)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s.v[w] += __shfl_xor(s.v[w], off, 64);
    if constexpr (NT == 64) return (s.v[0] + s.v[1]) + (s.v[2] + s.v[3]);
    if (threadIdx.x < 256 && (threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s.v[0];
    __syncthreads();
    const double t = (lds[0] + lds[1]) + (lds[2] + lds[3]);
    __syncthreads();
    return t;
}

// A thread's shares of the sums a stage starts from: |r|^2 for beta; |t|^2
// and, with a shifted base, |p|^2 for alpha (an unshifted base needs no |p|^2:
// its t stencil writes only the first set of partials).
// rr: the |r|^2 that goes with them.
template <int NT>
struct ProSums {
    SlotPart<NT> a, b;
    double rr = 0.0;
};
template <int NT>
__device__ __forceinline__ ProSums<NT> pro_sums(const ProArgs &p, int r)
{
    ProSums<NT> s;
    s.rr = p.kind == PRO_ALPHA ? p.st->rr[r] : p.kind == PRO_BETA ? p.st->rr_iter[r] : 0.0;
    s.a = slot_part<NT>(p.pin + (size_t)r * p.pstride, p.pcnt);
    if (p.shifted) s.b = slot_part<NT>(p.pin + (size_t)(p.nrhs + r) * p.pstride, p.pcnt);
    return s;
}

// |t|^2 + s0 |p|^2, alpha's denominator
template <int NT>
__device__ __forceinline__ double alpha_den(const ProArgs &p, int r, const ProSums<NT> &s, double *lds)
{
    const double tt = slot_fold<NT>(s.a, lds);
    return p.shifted ? fma(p.st->s0r[r], slot_fold<NT>(s.b, lds), tt) : tt;
}

// alpha for RHS r in a block whose sites need it; false if it is not finite
// (the stage's own block then ends the RHS)
template <int NT>
__device__ __forceinline__ bool pro_alpha(const ProArgs &p, int r, const ProSums<NT> &s, double *lds, double *alpha)
{
    const double pq = alpha_den<NT>(p, r, s, lds);
    *alpha = s.rr / pq;
    return isfinite(*alpha) && pq > 0.0;
}

// beta for RHS r in a block whose sites need it
template <int NT>
__device__ __forceinline__ double pro_beta(const ProArgs &p, int r, const ProSums<NT> &s, double *lds)
{
    return slot_fold<NT>(s.a, lds) / s.rr;
}

// Whether RHS r's sites stand still in a launch that carries stage p (kind 0:
// none; skip: the launch's flags, may be null).  The stage's block runs beside
// the site blocks, and every wave of a block must come to the same answer (the
// sums that follow have barriers), so the answer comes from a flag that the
// stage does not write: alpha writes run_c and leaves skip alone, beta writes
// skip and leaves run_c alone.
__device__ __forceinline__ bool sits_out(const ProArgs &p, const int *skip, int r)
{
    return p.kind == PRO_BETA ? !p.st->run_c[r] : skip && skip[r];
}

// K_a: alpha and the shifted zeta_j', alpha_j of RHS r; shift j is thread j
// (NS <= 64: all in wave 0).  An RHS without a finite alpha is marked and left
// out of the iteration; K_b then ends it.
template <int NT>
__device__ __forceinline__ void alpha_stage(const ProArgs &a, int r, double *lds)
{
    MState *st = a.st;
    const int j = threadIdx.x;
    if (a.reset && j < NS) {
        Blk *bk = a.bk;
        bk->P[r][j] = 1.0;
        bk->XP[r][j] = 0.0;
        bk->inblk[r][j] = j < st->nshift ? st->act[r][j] : 0;
        if (j == 0) bk->t[r] = 0;
    }
    if (st->skip[r]) {
        if (j == 0) st->run_c[r] = 0;
        if (j < NS) st->act_cur[r][j] = 0;
        return;
    }
    const double pq = alpha_den<NT>(a, r, pro_sums<NT>(a, r), lds);
    const double rr = st->rr[r];
    const double alpha = rr / pq;
    if (!isfinite(alpha) || !(pq > 0.0)) {
        if (j < st->nshift) st->act_cur[r][j] = 0;
        if (j == 0) {
            st->run_c[r] = 0;
            st->nonfinite[r] = 1;
        }
        return;
    }
    if (j == 0) {
        st->run_c[r] = 1;
        st->alpha[r] = alpha;
        st->rr_iter[r] = rr;
    }
    if (j < st->nshift) {
        const int on = st->act[r][j];
        st->act_cur[r][j] = on;
        if (on) {
            const double ao = st->alpha_old[r], be = st->beta[r];
            const double z = st->zeta[r][j], zo = st->zeta_old[r][j];
            const double zn = z * zo * ao / (alpha * be * (zo - z) + zo * ao * (1.0 + alpha * st->delta[j]));
            st->zeta_new[r][j] = zn;
            st->aj[r][j] = alpha * zn / z;
        }
    }
}

// K_b: beta, beta_j, freezing of shifts and (bk) the block coefficients of RHS
// r; shift j is thread j.  sw2 > 0: an RHS with |r|^2 <= sw2 |b|^2 pauses
// (hand-over).
template <int NT>
__device__ __forceinline__ void beta_stage(const ProArgs &a, int r, double *lds)
{
    MState *st = a.st;
    Blk *bk = a.bk;
    const int j = threadIdx.x;
    if (!st->run_c[r]) {   // finished before, or without a finite alpha
        if (j == 0 && st->nonfinite[r]) st->skip[r] = 1;
        return;
    }
    const double rr_new = slot_fold<NT>(slot_part<NT>(a.pin + (size_t)r * a.pstride, a.pcnt), lds);
    const int it = st->iter[r] + 1;
    if (!isfinite(rr_new)) {
        if (j == 0) {
            st->iter[r] = it;
            st->nonfinite[r] = 1;
            st->skip[r] = 1;
        }
        return;
    }
    const double beta = rr_new / st->rr_iter[r];
    const double thr = st->tol2r[r] * st->bb[r];
    const int t = bk ? bk->t[r] : 0;
    int live = 0;
    __shared__ double sa[NS], sb[NS];   // aj, bj of the shifts that run (son)
    __shared__ int son[NS];
    const int on = j < st->nshift && st->act_cur[r][j];
    if (j < NS) son[j] = on;
    if (on) {
        const double z = st->zeta[r][j], zn = st->zeta_new[r][j];
        const double q = zn / z;
        const double bj = beta * q * q;
        if (bk) {
            const double aj = st->aj[r][j];
            // x += a p^{(t)};  p^{(t+1)} = zn r^{(t+1)} + bj p^{(t)}
            const double P = bk->P[r][j];
            bk->XP[r][j] += aj * P;
            bk->P[r][j] = bj * P;
            sa[j] = aj;
            sb[j] = bj;
            bk->C[r][j][t + 1] = zn;
            bk->X[r][j][t + 1] = 0.0;
        }
        st->bj[r][j] = bj;
        st->zeta_old[r][j] = z;
        st->zeta[r][j] = zn;
        if (zn * zn * rr_new <= thr) {
            st->act[r][j] = 0;
            st->frozen_at[r][j] = it;
            st->frozen_rr[r][j] = zn * zn * rr_new;
        } else {
            live = j >= st->jlive;
        }
    } else if (bk && j < st->nshift) {
        bk->C[r][j][t + 1] = bk->X[r][j][t + 1] = 0.0;   // frozen: no part of this residual
    }
    // also the barrier between every thread's reads of rr, iter and t and
    // thread 0's writes below
    const int left = __syncthreads_count(live);
    // the block's earlier coefficients, a thread each (a thread for all of a
    // shift's is a chain of t loads and stores: 9.6 -> 7.2 us at up to 32 residuals)
    for (int k = j; k < st->nshift * t; k += NT) {
        const int q = k / t, i = 1 + k % t;
        if (!son[q]) continue;
        const double c = bk->C[r][q][i];
        bk->X[r][q][i] += sa[q] * c;
        bk->C[r][q][i] = sb[q] * c;
    }
    if (j == 0) {
        st->iter[r] = it;
        st->beta[r] = beta;
        if (bk) bk->t[r] = t + 1;
        st->rr[r] = rr_new;
        st->alpha_old[r] = st->alpha[r];
        if (!left) {
            st->skip[r] = 1;
        } else if (a.sw2 > 0.0 && rr_new <= a.sw2 * st->bb[r]) {
            st->paused[r] = 1;
            st->skip[r] = 1;
        }
    }
}

// Coefficients of one step of the two-pass Lanczos recurrence on unnormalised
// vectors u_k = |u_k| v_k (lanczos_sign.hip), four per RHS:
//   u_{k+1} = (c0 Q u_k - c1 u_{k-1}) - c2 u_k,   y += cy u_k,
// c0 = 1/|u_k|, c1 = |u_k| / |u_{k-1}|, c2 = <v_k, Q v_k> c0.
constexpr int kLzTab = 4 * NR;   // doubles per step, [rhs][c0, c1, c2, cy]

// c0 and c1 from |u_k|^2 and the previous step's c0 (an invariant subspace
// ends in u_k = 0, which stays 0)
__device__ __forceinline__ void lz_scale(double n2, double c0_prev, double *norm, double *c0, double *c1)
{
    const double b = sqrt(fmax(n2, 0.0));
    *norm = b;
    *c0 = b > 0.0 ? 1.0 / b : 0.0;
    *c1 = b * c0_prev;
}

template <int NT>
__device__ __forceinline__ void lanczos_stage(const ProArgs &a, int r, double *lds)
{
    const double n2 = slot_fold<NT>(slot_part<NT>(a.pin + (size_t)r * a.pstride, a.pcnt), lds);
    if (threadIdx.x == 0) {
        double *t = a.tab + 4 * r;
        lz_scale(n2, t[-kLzTab], &a.bout[r], &t[0], &t[1]);
    }
}

// The stage's own block inside a launch that carries it.
template <int NT>
__device__ __forceinline__ void pro_stage(const ProArgs &a, int r, double *lds)
{
    if (a.kind == PRO_ALPHA) alpha_stage<NT>(a, r, lds);
    else if (a.kind == PRO_BETA) beta_stage<NT>(a, r, lds);
    else lanczos_stage<NT>(a, r, lds);
}

}  // namespace ovl
