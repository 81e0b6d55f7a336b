// Layout conversion and BLAS-1 kernels on packed even-odd fields.
//
// All kernels here are site parallel: block b of a launch covers parity
// b / nb, checkerboard sites (b % nb)*256 .. +255, and blockIdx.y selects the
// RHS.  Per-block partial sums go to partials[rhs][block] and are combined by
// k_reduce in a fixed order, so every reduction is bitwise reproducible.
#include "internal.h"

namespace ovl {

Lat make_lat(const ovl_lattice *lat)
{
    Lat L;
    for (int m = 0; m < 4; m++) {
        L.g.L[m] = lat->dims[m];
        L.g.bc[m] = lat->bc[m];
    }
    L.V = (int64_t)lat->dims[0] * lat->dims[1] * lat->dims[2] * lat->dims[3];
    L.Vh = (int)(L.V / 2);
    L.g.Vh = L.Vh;
    L.g.S = padded_stride(L.Vh);
    L.g.T = lat->tile_t;
    L.g.Ts = lat->stream_t;
    L.g.Ts64 = lat->stream_t64;
    L.g.Kr = lat->rhs_tile >= 8 ? 3 : lat->rhs_tile >= 4 ? 2 : lat->rhs_tile >= 2 ? 1 : 0;
    L.g.Mfma = lat->mfma;
    L.nb = (L.Vh + kBlock - 1) / kBlock;
    L.tile = pick_tile(L.g.L, L.V);
    return L;
}

static thread_local int g_last_hip = 0;
int hip_fail(hipError_t e)
{
    g_last_hip = (int)e;
    return OVL_ERR_HIP;
}
int last_hip_error() { return g_last_hip; }

int site_blocks(const Lat &L) { return 2 * L.nb; }

// ---------------------------------------------------------------- pack
template <int PREC>
__global__ __launch_bounds__(kBlock) void k_pack_spinor(Geom g, int64_t V, const double2 *canon, void *d, float *sc)
{
    using T = typename Real<PREC>::T;
    int64_t lex = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int r = blockIdx.y;
    if (lex >= V) return;
    int x3 = (int)(lex % g.L[3]);
    int64_t t = lex / g.L[3];
    int x2 = (int)(t % g.L[2]);
    t /= g.L[2];
    int x1 = (int)(t % g.L[1]);
    int x0 = (int)(t / g.L[1]);
    int p = (x0 + x1 + x2 + x3) & 1;
    int i = (int)(lex >> 1);
    const double2 *src = canon + ((size_t)r * V + lex) * 12;
    cplx<T> s[4][3];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        double2 v = src[k];
        s[k / 3][k % 3] = {(T)v.x, (T)v.y};
    }
    spinor_ref<PREC>(d, sc, g.S, r).store(p, i, s);
}

// Bound by its reads and writes.  A thread's 12 components go through LDS (rows
// of 13: no bank conflicts) so that a wave writes whole lines of the canonical
// field: written 16 bytes a lane at a stride of 192, FP64 at 32^3x64 took
// 215 us, now 155 (5.2 TB/s).
template <int PREC>
__global__ __launch_bounds__(kBlock) void k_unpack_spinor(Geom g, int64_t V, const void *d, const float *sc, double2 *canon)
{
    using T = typename Real<PREC>::T;
    __shared__ double2 lds[kBlock * 13];
    const int64_t first = (int64_t)blockIdx.x * kBlock, lex = first + threadIdx.x;
    const int r = blockIdx.y;
    if (lex < V) {
        int x3 = (int)(lex % g.L[3]);
        int64_t t = lex / g.L[3];
        int x2 = (int)(t % g.L[2]);
        t /= g.L[2];
        int x1 = (int)(t % g.L[1]);
        int x0 = (int)(t / g.L[1]);
        int p = (x0 + x1 + x2 + x3) & 1;
        int i = (int)(lex >> 1);
        cplx<T> s[4][3];
        spinor_ref<PREC>(d, sc, g.S, r).load(p, i, s);
#pragma unroll
        for (int k = 0; k < 12; k++)
            lds[threadIdx.x * 13 + k] = make_double2((double)s[k / 3][k % 3].x, (double)s[k / 3][k % 3].y);
    }
    __syncthreads();
    double2 *dst = canon + ((size_t)r * V + first) * 12;
    const int n = 12 * (int)(V - first < kBlock ? V - first : kBlock);
    for (int j = threadIdx.x; j < n; j += kBlock) dst[j] = lds[j / 12 * 13 + j % 12];
}

// Rows 0 and 1 of the links of kPackSites sites, read once for every packed
// copy that is asked for (null: not asked for).  Bound by its reads and writes.
// The links pass through LDS: read in order of the canonical field, written 32
// sites of one parity, direction and component at a time.  A pass per copy,
// eight sites a run, took 1326 us at 32^3x64 for FP64, FP32 and FP16 (3.6 GB
// read, 1.4 written); one pass takes 541 us (4.8 TB/s).
constexpr int kPackSites = 64;   // 8 runs (parity, direction) of 32 pairs of x3 neighbours: 256 threads

__global__ __launch_bounds__(kBlock) void k_pack_gauge(Geom g, int64_t V, const double2 *canon, double2 *o64,
                                                        float4 *o32, uint2 *o16)
{
    __shared__ double2 lds[24][kPackSites + 1];
    const int64_t first = (int64_t)blockIdx.x * kPackSites;
    const int n = (int)(V - first < kPackSites ? V - first : kPackSites);
    const double2 *src = canon + (size_t)first * 36;
    for (int j = threadIdx.x; j < n * 36; j += kBlock) {
        const int l = j / 9, c = j % 9;
        if (c < 6) {
            const nt_d2 v = __builtin_nontemporal_load((const nt_d2 *)&src[j]);
            lds[(l & 3) * 6 + c][l >> 2] = make_double2(v.x, v.y);
        }
    }
    __syncthreads();
    const int k = threadIdx.x & 31, pm = threadIdx.x >> 5, p = pm >> 2, mu = pm & 3;
    if (2 * k >= n) return;
    const int64_t lex = first + 2 * k;   // the pair's first site
    int x3 = (int)(lex % g.L[3]);
    int64_t t = lex / g.L[3];
    int x2 = (int)(t % g.L[2]);
    t /= g.L[2];
    int x1 = (int)(t % g.L[1]);
    int x0 = (int)(t / g.L[1]);
    const int site = 2 * k + (((x0 + x1 + x2 + x3) & 1) ^ p);
    const size_t i = (size_t)(lex >> 1);
    const size_t Vh = (size_t)g.S;   // component stride
    double2 u[6];
#pragma unroll
    for (int e = 0; e < 6; e++) u[e] = lds[mu * 6 + e][site];
    if (o64) {
        double2 *o = o64 + (size_t)pm * 6 * Vh + i;
#pragma unroll
        for (int e = 0; e < 6; e++) o[e * Vh] = u[e];
    }
    if (o32) {
        float4 *o = o32 + (size_t)pm * 3 * Vh + i;
#pragma unroll
        for (int e = 0; e < 3; e++)
            o[e * Vh] = make_float4((float)u[2 * e].x, (float)u[2 * e].y, (float)u[2 * e + 1].x, (float)u[2 * e + 1].y);
    }
    if (o16) {
        uint2 *o = o16 + (size_t)pm * 3 * Vh + i;
#pragma unroll
        for (int e = 0; e < 3; e++) {
            unsigned a = (unsigned)f2h((float)u[2 * e].x) | ((unsigned)f2h((float)u[2 * e].y) << 16);
            unsigned b = (unsigned)f2h((float)u[2 * e + 1].x) | ((unsigned)f2h((float)u[2 * e + 1].y) << 16);
            o[e * Vh] = make_uint2(a, b);
        }
    }
}

hipError_t launch_pack_spinor(const Lat &L, const void *canon, Fld out, hipStream_t st)
{
    dim3 grid((unsigned)((L.V + kBlock - 1) / kBlock), out.nrhs);
    if (out.prec == P_F64)
        k_pack_spinor<P_F64><<<grid, kBlock, 0, st>>>(L.g, L.V, (const double2 *)canon, out.d, out.sc);
    else if (out.prec == P_F48)
        k_pack_spinor<P_F48><<<grid, kBlock, 0, st>>>(L.g, L.V, (const double2 *)canon, out.d, out.sc);
    else if (out.prec == P_F32)
        k_pack_spinor<P_F32><<<grid, kBlock, 0, st>>>(L.g, L.V, (const double2 *)canon, out.d, out.sc);
    else
        k_pack_spinor<P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.V, (const double2 *)canon, out.d, out.sc);
    return hipGetLastError();
}

hipError_t launch_unpack_spinor(const Lat &L, Fld in, void *canon, hipStream_t st)
{
    dim3 grid((unsigned)((L.V + kBlock - 1) / kBlock), in.nrhs);
    if (in.prec == P_F64)
        k_unpack_spinor<P_F64><<<grid, kBlock, 0, st>>>(L.g, L.V, in.d, in.sc, (double2 *)canon);
    else if (in.prec == P_F48)
        k_unpack_spinor<P_F48><<<grid, kBlock, 0, st>>>(L.g, L.V, in.d, in.sc, (double2 *)canon);
    else if (in.prec == P_F32)
        k_unpack_spinor<P_F32><<<grid, kBlock, 0, st>>>(L.g, L.V, in.d, in.sc, (double2 *)canon);
    else
        k_unpack_spinor<P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.V, in.d, in.sc, (double2 *)canon);
    return hipGetLastError();
}

hipError_t launch_pack_gauge(const Lat &L, const void *canon, void *f64, void *f32, void *f16, hipStream_t st)
{
    dim3 grid((unsigned)((L.V + kPackSites - 1) / kPackSites));
    k_pack_gauge<<<grid, kBlock, 0, st>>>(L.g, L.V, (const double2 *)canon, (double2 *)f64, (float4 *)f32,
                                          (uint2 *)f16);
    return hipGetLastError();
}

// ---------------------------------------------------------------- BLAS-1
template <int PREC>
__global__ __launch_bounds__(kBlock) void k_norm2(Geom g, int nb, const void *d, const float *sc, double *partials)
{
    using T = typename Real<PREC>::T;
    __shared__ double lds[4];
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    double v = 0.0;
    if (i < g.Vh) {
        cplx<T> s[4][3];
        spinor_ref<PREC>(d, sc, g.S, r).load(p, i, s);
        T a = 0;
#pragma unroll
        for (int k = 0; k < 12; k++) a += norm2(s[k / 3][k % 3]);
        v = (double)a;
    }
    double t = block_sum(v, lds);
    if (threadIdx.x == 0) partials[(size_t)r * gridDim.x + b] = t;
}

// |a - b|^2 with both fields widened to double
template <int PA, int PB>
__global__ __launch_bounds__(kBlock) void k_diff_norm2(Geom g, int nb, const void *da, const float *sa,
                                                       const void *db, const float *sb, double *partials)
{
    using TA = typename Real<PA>::T;
    using TB = typename Real<PB>::T;
    __shared__ double lds[4];
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    double v = 0.0;
    if (i < g.Vh) {
        cplx<TA> s[4][3];
        cplx<TB> t[4][3];
        spinor_ref<PA>(da, sa, g.S, r).load(p, i, s);
        spinor_ref<PB>(db, sb, g.S, r).load(p, i, t);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            double dx = (double)s[k / 3][k % 3].x - (double)t[k / 3][k % 3].x;
            double dy = (double)s[k / 3][k % 3].y - (double)t[k / 3][k % 3].y;
            v += dx * dx + dy * dy;
        }
    }
    double t = block_sum(v, lds);
    if (threadIdx.x == 0) partials[(size_t)r * gridDim.x + b] = t;
}

// Re and Im of <a, b> (partials [2][nrhs][nblk])
__global__ __launch_bounds__(kBlock) void k_dot_f64(Geom g, int nb, int nrhs, const void *da, const void *db, double *partials)
{
    __shared__ double lds[8];
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    double re = 0.0, im = 0.0;
    if (i < g.Vh) {
        cplx<double> s[4][3], t[4][3];
        spinor_ref<P_F64>(da, nullptr, g.S, r).load(p, i, s);
        spinor_ref<P_F64>(db, nullptr, g.S, r).load(p, i, t);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            cplx<double> c = cmc(s[k / 3][k % 3], t[k / 3][k % 3]);
            re += c.x;
            im += c.y;
        }
    }
    double t0 = block_sum(re, lds);
    double t1 = block_sum(im, lds + 4);
    if (threadIdx.x == 0) {
        partials[(size_t)r * gridDim.x + b] = t0;
        partials[(size_t)(nrhs + r) * gridDim.x + b] = t1;
    }
}

__global__ __launch_bounds__(kBlock) void k_reduce(const double *partials, int nblk, int cnt, double *out)
{
    __shared__ double lds[4];
    const double *src = partials + (size_t)blockIdx.x * nblk;
    double v = 0.0;
    for (int k = threadIdx.x; k < cnt; k += kBlock) v += src[k];
    double t = block_sum(v, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

template <int PS, int PD>
__global__ __launch_bounds__(kBlock) void k_convert(Geom g, int nb, const void *ds, const float *ss, void *dd, float *sd)
{
    using TS = typename Real<PS>::T;
    using TD = typename Real<PD>::T;
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    if (i >= g.Vh) return;
    cplx<TS> s[4][3];
    cplx<TD> t[4][3];
    spinor_ref<PS>(ds, ss, g.S, r).load(p, i, s);
#pragma unroll
    for (int k = 0; k < 12; k++) t[k / 3][k % 3] = {(TD)s[k / 3][k % 3].x, (TD)s[k / 3][k % 3].y};
    spinor_ref<PD>(dd, sd, g.S, r).store(p, i, t);
}

// y = a x + b y computed in the precision of y's arithmetic type
template <int PX, int PY>
__global__ __launch_bounds__(kBlock) void k_axpby(Geom g, int nb, double a, const void *dx, const float *sx, double bcoef,
                                                  void *dy, float *sy)
{
    using TX = typename Real<PX>::T;
    using TY = typename Real<PY>::T;
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    if (i >= g.Vh) return;
    cplx<TX> s[4][3];
    cplx<TY> t[4][3];
    spinor_ref<PX>(dx, sx, g.S, r).load(p, i, s);
    auto yr = spinor_ref<PY>(dy, sy, g.S, r);
    if (bcoef != 0.0) {
        yr.load(p, i, t);
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) t[k / 3][k % 3] = {(TY)0, (TY)0};
    }
    const TY A = (TY)a, B = (TY)bcoef;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        cplx<TY> &v = t[k / 3][k % 3];
        v = {fma(A, (TY)s[k / 3][k % 3].x, B * v.x), fma(A, (TY)s[k / 3][k % 3].y, B * v.y)};
    }
    yr.store(p, i, t);
}

template <int PREC>
__global__ __launch_bounds__(kBlock) void k_zero(Geom g, int nb, void *d, float *sc)
{
    using T = typename Real<PREC>::T;
    int r = blockIdx.y, b = blockIdx.x;
    int p = b / nb, i = (b % nb) * kBlock + threadIdx.x;
    if (i >= g.Vh) return;
    cplx<T> t[4][3];
#pragma unroll
    for (int k = 0; k < 12; k++) t[k / 3][k % 3] = {(T)0, (T)0};
    spinor_ref<PREC>(d, sc, g.S, r).store(p, i, t);
}

#define DISPATCH1(prec, KERNEL, ...)                                  \
    do {                                                              \
        if ((prec) == P_F64) KERNEL<P_F64><<<__VA_ARGS__>>>;          \
    } while (0)

hipError_t launch_norm2(const Lat &L, Fld f, double *partials, hipStream_t st)
{
    dim3 grid(2 * L.nb, f.nrhs);
    if (f.prec == P_F64) k_norm2<P_F64><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc, partials);
    else if (f.prec == P_F48) k_norm2<P_F48><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc, partials);
    else if (f.prec == P_F32) k_norm2<P_F32><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc, partials);
    else k_norm2<P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc, partials);
    return hipGetLastError();
}

hipError_t launch_diff_norm2(const Lat &L, Fld a, Fld b, double *partials, hipStream_t st)
{
    dim3 grid(2 * L.nb, a.nrhs);
    if (a.prec != P_F64 || b.prec == P_F48) return hipErrorInvalidValue;
    if (b.prec == P_F64) k_diff_norm2<P_F64, P_F64><<<grid, kBlock, 0, st>>>(L.g, L.nb, a.d, a.sc, b.d, b.sc, partials);
    else if (b.prec == P_F32) k_diff_norm2<P_F64, P_F32><<<grid, kBlock, 0, st>>>(L.g, L.nb, a.d, a.sc, b.d, b.sc, partials);
    else k_diff_norm2<P_F64, P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.nb, a.d, a.sc, b.d, b.sc, partials);
    return hipGetLastError();
}

hipError_t launch_dot(const Lat &L, Fld a, Fld b, double *partials, hipStream_t st)
{
    if (a.prec != P_F64 || b.prec != P_F64) return hipErrorInvalidValue;
    dim3 grid(2 * L.nb, a.nrhs);
    k_dot_f64<<<grid, kBlock, 0, st>>>(L.g, L.nb, a.nrhs, a.d, b.d, partials);
    return hipGetLastError();
}

hipError_t launch_reduce(const double *partials, int nq, int nrhs, int nblk, double *out, hipStream_t st, int cnt)
{
    k_reduce<<<nq * nrhs, kBlock, 0, st>>>(partials, nblk, cnt < 0 ? nblk : cnt, out);
    return hipGetLastError();
}

template <int PS>
static hipError_t convert_to(const Lat &L, Fld s, Fld d, hipStream_t st)
{
    dim3 grid(2 * L.nb, s.nrhs);
    if (d.prec == P_F64) k_convert<PS, P_F64><<<grid, kBlock, 0, st>>>(L.g, L.nb, s.d, s.sc, d.d, d.sc);
    else if (d.prec == P_F48) k_convert<PS, P_F48><<<grid, kBlock, 0, st>>>(L.g, L.nb, s.d, s.sc, d.d, d.sc);
    else if (d.prec == P_F32) k_convert<PS, P_F32><<<grid, kBlock, 0, st>>>(L.g, L.nb, s.d, s.sc, d.d, d.sc);
    else k_convert<PS, P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.nb, s.d, s.sc, d.d, d.sc);
    return hipGetLastError();
}

hipError_t launch_convert(const Lat &L, Fld s, Fld d, hipStream_t st)
{
    if (s.prec == P_F64) return convert_to<P_F64>(L, s, d, st);
    if (s.prec == P_F48) return convert_to<P_F48>(L, s, d, st);
    if (s.prec == P_F32) return convert_to<P_F32>(L, s, d, st);
    return convert_to<P_F16S>(L, s, d, st);
}

template <int PX>
static hipError_t axpby_to(const Lat &L, double a, Fld x, double b, Fld y, hipStream_t st)
{
    dim3 grid(2 * L.nb, x.nrhs);
    if (y.prec == P_F64) k_axpby<PX, P_F64><<<grid, kBlock, 0, st>>>(L.g, L.nb, a, x.d, x.sc, b, y.d, y.sc);
    else if (y.prec == P_F32) k_axpby<PX, P_F32><<<grid, kBlock, 0, st>>>(L.g, L.nb, a, x.d, x.sc, b, y.d, y.sc);
    else k_axpby<PX, P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.nb, a, x.d, x.sc, b, y.d, y.sc);
    return hipGetLastError();
}

hipError_t launch_axpby(const Lat &L, double a, Fld x, double b, Fld y, hipStream_t st)
{
    if (x.prec == P_F48 || y.prec == P_F48) return hipErrorInvalidValue;   // not needed on 48-bit fields
    if (x.prec == P_F64) return axpby_to<P_F64>(L, a, x, b, y, st);
    if (x.prec == P_F32) return axpby_to<P_F32>(L, a, x, b, y, st);
    return axpby_to<P_F16S>(L, a, x, b, y, st);
}

hipError_t launch_zero(const Lat &L, Fld f, hipStream_t st)
{
    dim3 grid(2 * L.nb, f.nrhs);
    if (f.prec == P_F64) k_zero<P_F64><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc);
    else if (f.prec == P_F48) k_zero<P_F48><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc);
    else if (f.prec == P_F32) k_zero<P_F32><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc);
    else k_zero<P_F16S><<<grid, kBlock, 0, st>>>(L.g, L.nb, f.d, f.sc);
    return hipGetLastError();
}

}  // namespace ovl
