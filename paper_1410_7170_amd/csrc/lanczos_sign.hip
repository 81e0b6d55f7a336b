// sign(Q) b by a Krylov subspace method instead of a rational function: the
// Lanczos approximation |b| V_k sign(T_k) e_1 on the Krylov space of the
// Hermitian Q = Gamma_5 D_W (the paper's "sign function iteration" approximates
// sign(Gamma_5 D_W) chi by a Krylov method, Section 5; it restarts with thick
// restarts to bound memory).  Here memory is bounded by two passes instead:
//   pass 1: Lanczos on Q from v_1 = b/|b|, keeping only the coefficients
//           alpha_k, beta_k (on the device); every kCheck steps the host forms
//           c_k = |b| sign(T_k) e_1 from an eigen-decomposition of T_k and an
//           RHS stops once |c_k - c_{k-kCheck}| <= tol |b|;
//   pass 2: the same recurrence regenerates v_1..v_m from the stored
//           coefficients, accumulating y = sum_k c_k v_k (every other step,
//           two vectors at a time), all in the stencil's epilogue.
// The vectors are kept unnormalised (u_k = |u_k| v_k) and the division goes
// into the recurrence's coefficients, so that no kernel waits for a norm only
// to scale a field.  Two FP64 work fields per RHS, twice the stencils of one pass.
// Each RHS of a batch has its own coefficients; the passes run in step for all
// of them.  At 16^3x32, 320 steps: 8 launches a step (both passes) -> 3 (4 where the
// stencil streams), 45.3 -> 35.6 ms, and 30.2 with the checks' host work beside
// the device's next steps; at 32^3x64, 707 -> 463 ms.
#include <cmath>
#include <cstddef>
#include <cstring>
#include <vector>

#include "mscg.h"
#include "tridiag.h"

namespace ovl {

constexpr int kLzMax = 4096;   // longest Lanczos sequence
constexpr int kCheck = 32;     // steps between convergence checks

// per-RHS Lanczos coefficients on the device: a[k][r] = <v_k, Q v_k>,
// b[k][r] = the norm of the unnormalised next vector, and the recurrence's
// coefficients of every step (kLzTab doubles each, after a step of zeros)
struct LzCoef {
    double a[kLzMax][NR], b[kLzMax][NR];
    double tab[kLzMax + 1][kLzTab];
};

// The rest of a step of pass 1: u_{k+1} = t - c2 u_k over t (t = c0 Q u_k - c1
// u_{k-1} from the stencil), partial |u_{k+1}|^2 per RHS.  Every block forms
// c2 from the stencil's partial sums of <u_k, Q u_k>; the first of each RHS
// records it and a_k.  Bound by its three fields; with the division by |u| in
// the coefficients and the dot in the stencil, a step of pass 1 moves 8 fields
// and the links where a stencil, a dot, an update and a scaling moved 12.
__global__ __launch_bounds__(kBlock) void k_lz_axpy(Geom g, int nb, const double2 *u, double2 *t, LzCoef *cf, int k,
                                                     const double *pin, int pstride, int pcnt, double *partials)
{
    __shared__ double lds[4];
    const int r = blockIdx.y, bl = blockIdx.x;
    const int p = bl / nb, i = (bl % nb) * kBlock + threadIdx.x;
    const SlotPart<kBlock> part = slot_part<kBlock>(pin + (size_t)r * pstride, pcnt);
    cplx<double> tv[4][3], uv[4][3];
    const auto TF = spinor_ref<P_F64>(t, nullptr, g.S, r);
    if (i < g.Vh) {
        TF.load(p, i, tv);
        spinor_ref<P_F64>(u, nullptr, g.S, r).load(p, i, uv);
    }
    double *tab = cf->tab[k + 1] + 4 * r;
    const double c0 = tab[0];
    const double a = slot_fold<kBlock>(part, lds) * c0 * c0, c2 = a * c0;
    if (bl == 0 && threadIdx.x == 0) {
        cf->a[k][r] = a;
        tab[2] = c2;
    }
    double n2 = 0.0;
    if (i < g.Vh) {
#pragma unroll
        for (int q = 0; q < 12; q++) {
            cplx<double> &w = tv[q / 3][q % 3];
            w = fmac(w, -c2, uv[q / 3][q % 3]);
            n2 += norm2(w);
        }
        TF.store(p, i, tv);
    }
    const double s = block_sum(n2, lds);
    if (threadIdx.x == 0) partials[(size_t)r * gridDim.x + bl] = s;
}

// |u_k| and the step's c0, c1 in a kernel of their own (one block per RHS)
__global__ __launch_bounds__(kBlock) void k_lz_scale(ProArgs a)
{
    __shared__ double lds[4];
    lanczos_stage<kBlock>(a, blockIdx.x, lds);
}

// the first step's coefficients from |b| per RHS (c1 = 0: no vector before it)
struct LzFirst {
    double c0[NR];
};
__global__ void k_lz_first(LzCoef *cf, LzFirst f)
{
    const int j = threadIdx.x;
    if (j < kLzTab) {
        cf->tab[0][j] = 0.0;
        cf->tab[1][j] = (j & 3) == 0 ? f.c0[j >> 2] : 0.0;
    }
}

// the weights of pass 2: cy of step k is c_k / |u_k|
__global__ __launch_bounds__(kBlock) void k_lz_weights(LzCoef *cf, const double *c, int n)
{
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j < n * NR) {
        double *t = cf->tab[j / NR + 1] + 4 * (j % NR);
        t[3] = c[j] * t[0];
    }
}

size_t lanczos_sign_ws_bytes(const Lat &L, int nrhs)
{
    WsCarve c{nullptr, 0, 0};
    const size_t F = field_bytes(P_F64, L.V);
    c.take(2 * F * nrhs);                                  // u_{k-1}, u_k
    c.take(sizeof(LzCoef));
    c.take(sizeof(double) * (size_t)kLzMax * NR);          // pass-2 weights
    c.take(sizeof(double) * 2 * NR * part_stride(L));      // of the stencil, of the update
    c.take(sizeof(double) * 4 * NR);
    return c.off + 256;
}

// y = sign(Q) b for the nrhs fields of b (FP64); iters[q] the Lanczos steps
// of RHS q.  tol: relative change of the coefficient vector between checks.
int lanczos_sign(const Lat &L, const void *U64, double m0, Fld b, Fld y, double tol, int maxiter, int *iters,
                 char *ws, size_t ws_bytes, hipStream_t st)
{
    const int R = b.nrhs;
    if (ws_bytes < lanczos_sign_ws_bytes(L, R)) return OVL_ERR_WORKSPACE;
    const int kmax = std::min(maxiter, kLzMax - 1);
    WsCarve c{ws, 0, ws_bytes};
    const size_t F = field_bytes(P_F64, L.V);
    char *f2 = (char *)c.take(2 * F * R);
    Fld va{f2, nullptr, P_F64, R}, vb{f2 + F * R, nullptr, P_F64, R};
    LzCoef *cf = (LzCoef *)c.take(sizeof(LzCoef));
    double *cw = (double *)c.take(sizeof(double) * (size_t)kLzMax * NR);
    const int pstr = part_stride(L), nblk = site_blocks(L);
    double *partials = (double *)c.take(sizeof(double) * 2 * NR * pstr);
    double *partials2 = partials + (size_t)NR * pstr;
    double *red = (double *)c.take(sizeof(double) * 4 * NR);
    dim3 grid(nblk, R);
    auto tab = [&](int k) { return (double *)((char *)cf + offsetof(LzCoef, tab)) + (size_t)(k + 1) * kLzTab; };
    auto bnorm = [&](int k) { return (double *)((char *)cf + offsetof(LzCoef, b)) + (size_t)k * NR; };
    // |b| per RHS
    std::vector<double> bn(R);
    {
        OVL_HIP(launch_norm2(L, b, partials, st));
        OVL_HIP(launch_reduce(partials, 1, R, nblk, red, st));
        OVL_HIP(hipMemcpyAsync(bn.data(), red, sizeof(double) * R, hipMemcpyDeviceToHost, st));
        OVL_HIP(hipStreamSynchronize(st));
        for (int q = 0; q < R; q++) {
            if (!std::isfinite(bn[q])) return OVL_ERR_NONFINITE;
            bn[q] = std::sqrt(bn[q]);
        }
    }
    WArgs A{};
    A.U = U64;
    A.diag = m0 + 4.0;
    A.nrhs = R;
    // start: u_{-1} = 0, u_0 = b (an all-zero b gives y = 0)
    LzFirst lf{};
    for (int q = 0; q < R; q++) lf.c0[q] = bn[q] > 0 ? 1.0 / bn[q] : 0.0;
    auto start = [&]() -> int {
        OVL_HIP(launch_zero(L, va, st));
        OVL_HIP(hipMemcpyAsync(vb.d, b.d, F * R, hipMemcpyDeviceToDevice, st));
        return OVL_OK;
    };
    // the two fields swap roles every step: u_{k+1} goes over u_{k-1}
    Fld vprev = va, vk = vb;
    std::vector<int> mq(R, 0);          // steps of each RHS (0: not converged yet)
    std::vector<std::vector<double>> cprev(R), cbest(R);
    std::vector<double> ha((size_t)(kmax + 1) * NR), hb((size_t)(kmax + 1) * NR);
    k_lz_first<<<1, kLzTab, 0, st>>>(cf, lf);
    OVL_HIP(hipGetLastError());
    int rc = start();
    if (rc) return rc;
    // |u_k| and the step's coefficients ride in its stencil where that can
    // carry them (see carries_scalars)
    const bool carry = stencil_shape(L, P_F64, R).ts == 0 && nblk <= 1024;
    const int npart = stencil_partials(L, P_F64, R);
    ProArgs pro{PRO_LANCZOS, nblk, nblk, R, 0, partials2, nullptr, nullptr, 0.0, 0, nullptr, nullptr};
    int k = 0, checked = 0;   // steps launched, and those of the last check
    bool all = false;
    for (int q = 0; q < R; q++)
        if (!(bn[q] > 0)) mq[q] = -1;   // nothing to do
    auto step = [&]() -> int {
        // (after a check |u_k| and the coefficients are there already)
        const bool scaled = k % kCheck == 0;
        if (!scaled) {
            pro.tab = tab(k);
            pro.bout = bnorm(k - 1);
            if (!carry) k_lz_scale<<<R, kBlock, 0, st>>>(pro);
        }
        A.in = vk.d;
        A.p = vprev.d;
        A.out = vprev.d;
        A.alpha = tab(k);
        A.partials = partials;
        OVL_HIP(launch_wilson(L, P_F64, W_LZ1, true, A, st, nullptr, nullptr, carry && !scaled ? &pro : nullptr));
        k_lz_axpy<<<grid, kBlock, 0, st>>>(L.g, L.nb, (const double2 *)vk.d, (double2 *)vprev.d, cf, k, partials,
                                           pstr, npart, partials2);
        OVL_HIP(hipGetLastError());
        std::swap(vprev, vk);
        k++;
        return OVL_OK;
    };
    // The steps run ahead of the checks (below), never past the next one; the
    // last check is at kmax, also where the steps have come that far already.
    while (!all && checked < kmax) {
        const int kc = std::min(kmax, (checked / kCheck + 1) * kCheck);
        while (k < kc)
            if ((rc = step())) return rc;
        checked = kc;
        pro.tab = tab(k);
        pro.bout = bnorm(k - 1);
        k_lz_scale<<<R, kBlock, 0, st>>>(pro);
        OVL_HIP(hipGetLastError());
        // device addresses of the coefficient arrays (no host access to cf)
        const double *da = (const double *)((const char *)cf + offsetof(LzCoef, a));
        const double *db = (const double *)((const char *)cf + offsetof(LzCoef, b));
        OVL_HIP(hipMemcpyAsync(ha.data(), da, sizeof(double) * NR * k, hipMemcpyDeviceToHost, st));
        OVL_HIP(hipMemcpyAsync(hb.data(), db, sizeof(double) * NR * k, hipMemcpyDeviceToHost, st));
        OVL_HIP(hipStreamSynchronize(st));
        // Each open RHS's T_k, cut where its Krylov space closes; coefficients
        // that are not finite end the call while nothing is in flight.
        int open = 0;
        std::vector<double> a[NR], bt[NR];
        bool brk[NR] = {};
        for (int q = 0; q < R; q++) {
            if (mq[q] != 0) continue;
            open++;
            for (int j = 0; j < kc && !brk[q]; j++) {
                a[q].push_back(ha[(size_t)j * NR + q]);
                bt[q].push_back(hb[(size_t)j * NR + q]);
                if (!std::isfinite(a[q][j]) || !std::isfinite(bt[q][j])) return OVL_ERR_NONFINITE;
                brk[q] = bt[q][j] <= 1e-14 * std::fabs(a[q][j]) + 1e-300;   // invariant subspace: exact
            }
        }
        // The device goes on while the host decomposes T_k, by no more steps
        // than that takes (at least 15 ns per row squared of each RHS; a step: its
        // 8 fields and links at 5 TB/s, or 15 us), so that none delays pass 2
        // where this check is the last.
        const double host = 15e-9 * k * k * open;
        const double gpu = std::max(15e-6, 2.5e3 * (double)L.V * R / 5e12);
        const int ahead = std::min(std::min(kCheck - 1, kmax - k), (int)(host / gpu));
        for (int j = 0; j < ahead; j++)
            if ((rc = step())) return rc;
        all = true;
        for (int q = 0; q < R; q++) {
            if (mq[q] != 0) continue;
            const int kk = (int)a[q].size();
            std::vector<double> cq;
            if (!tridiag_sign_e1(kk, a[q].data(), bt[q].data(), bn[q], cq)) {
                OVL_HIP(hipStreamSynchronize(st));   // the steps ahead use the caller's memory
                return OVL_ERR_NONFINITE;
            }
            double diff = 0.0;
            for (int j = 0; j < kk; j++) {
                const double o = j < (int)cprev[q].size() ? cprev[q][j] : 0.0;
                diff += (cq[j] - o) * (cq[j] - o);
            }
            if (brk[q] || std::sqrt(diff) <= tol * bn[q]) {
                mq[q] = kk;
                cbest[q] = cq;
            } else {
                all = false;
                cprev[q] = cq;
            }
        }
    }
    int status = OVL_OK;
    int kmx = 0;
    for (int q = 0; q < R; q++) {
        if (mq[q] == 0) {   // maxiter: use the last coefficients
            status = OVL_NOT_CONVERGED;
            mq[q] = (int)cprev[q].size();
            cbest[q] = cprev[q];
        }
        if (mq[q] < 0) mq[q] = 0;
        kmx = std::max(kmx, mq[q]);
        if (iters) iters[q] = mq[q];
    }
    // pass 2: the weights c_k per RHS (0 beyond its own steps), then the same
    // recurrence from the stored coefficients with y += c_k v_k
    std::vector<double> hc((size_t)std::max(kmx, 1) * NR, 0.0);
    for (int q = 0; q < R; q++)
        for (int j = 0; j < mq[q]; j++) hc[(size_t)j * NR + q] = cbest[q][j];
    OVL_HIP(hipMemcpyAsync(cw, hc.data(), sizeof(double) * hc.size(), hipMemcpyHostToDevice, st));
    k_lz_weights<<<(std::max(kmx, 1) * NR + kBlock - 1) / kBlock, kBlock, 0, st>>>(cf, cw, kmx);
    OVL_HIP(hipGetLastError());
    OVL_HIP(launch_zero(L, y, st));
    rc = start();
    if (rc) return rc;
    vprev = va;
    vk = vb;
    for (int j = 0; j < kmx; j++) {
        // y takes two steps at a time: at odd j, and at the last
        A.in = vk.d;
        A.p = vprev.d;
        A.out = vprev.d;
        A.alpha = tab(j);
        A.rin = y.d;
        A.rin_first = j & 1;
        OVL_HIP(launch_wilson(L, P_F64, (j & 1) || j + 1 == kmx ? W_LZ3 : W_LZ2, true, A, st));
        std::swap(vprev, vk);
    }
    OVL_HIP(hipStreamSynchronize(st));
    return status;
}

}  // namespace ovl
