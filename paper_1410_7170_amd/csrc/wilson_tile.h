// Tile form of the FP64 Wilson stencil (wilson.h), for lattices whose time
// streams would leave the chip idle.
//
// A block owns the sites of one four-dimensional tile, one thread a site, and
// keeps their spinors in LDS as stored (FP64 or 48 bits), so that only the
// hops that leave the tile read a spinor from memory: at 16^3x32 with tiles
// of 4x4x2x16, two per site instead of the one-site form's eight.  What
// bounds that form there is the fetch of neighbours that its 4 MB of L2 per
// die no longer hold (a die's share of one field and its links is 9 MB).
// Links are loaded one hop ahead of their use.  Measured at 16^3x32, one
// field: FP64 D_W 35-41 -> 23 us, the 48-bit solver stencils 34-36 -> 25 us
// (107 MB at least).  FP32 and FP16 keep the one-site form, which is no slower
// there (15.8 against 15.8 and 11 against 12 us): their share of a die fits its
// L2.
#pragma once

#include "wilson.h"

namespace ovl {

// A site's spinor staged as stored.
template <int PREC, int NT>
struct Stage;
template <int NT>
struct Stage<P_F64, NT> {
    double2 d[12][NT];
    __device__ void fill(int l, const SpinorRef<P_F64> &f, int p, int i)
    {
        const double2 *b = f.d + (size_t)p * 12 * f.Vh + i;
        double2 v[12];
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = b[(size_t)k * f.Vh];
#pragma unroll
        for (int k = 0; k < 12; k++) d[k][l] = v[k];
    }
    __device__ void load(int l, cplx<double> s[4][3]) const
    {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double2 v = d[k][l];
            s[k / 3][k % 3] = {v.x, v.y};
        }
    }
};
template <int NT>
struct Stage<P_F48, NT> {
    uint4 d[9][NT];
    __device__ void fill(int l, const SpinorRef<P_F48> &f, int p, int i)
    {
        F48Code c;
        f.load_raw(p, i, c);
#pragma unroll
        for (int k = 0; k < 6; k++) d[k][l] = c.h[k];
#pragma unroll
        for (int k = 0; k < 3; k++) d[6 + k][l] = c.l[k];
    }
    __device__ void load(int l, cplx<double> s[4][3]) const
    {
        F48Code c;
#pragma unroll
        for (int k = 0; k < 6; k++) c.h[k] = d[k][l];
#pragma unroll
        for (int k = 0; k < 3; k++) c.l[k] = d[6 + k][l];
        f48_decode(c, s);
    }
};
// An FP64 link as stored: loaded ahead of its use, its third row rebuilt there.
struct RawLink {
    double2 e[6];
    __device__ __forceinline__ void load(const GaugeRef<P_F64> &U, int p, int mu, int i)
    {
        const double2 *b = U.d + (size_t)(p * 4 + mu) * 6 * U.Vh + i;
#pragma unroll
        for (int k = 0; k < 6; k++) e[k] = b[(size_t)k * U.Vh];
    }
    __device__ __forceinline__ void get(cplx<double> u[3][3]) const
    {
#pragma unroll
        for (int k = 0; k < 6; k++) u[k / 3][k % 3] = {e[k].x, e[k].y};
        rebuild_row2(u);
    }
};

// Keeps values where they are.  Without it on the sums the compiler sinks the
// products of all eight hops below the last branch and spills their operands.
__device__ __forceinline__ void pin(cplx<double> a[4][3])
{
#pragma unroll
    for (int s = 0; s < 4; s++)
        asm volatile("" : "+v"(a[s][0].x), "+v"(a[s][0].y), "+v"(a[s][1].x), "+v"(a[s][1].y), "+v"(a[s][2].x),
                     "+v"(a[s][2].y));
}

// One site's place in its tile and in the lattice, per direction.
struct TileSite {
    int l, i, p;
    int c[4], x[4];       // coordinates in the tile and in the lattice
    int ls[4], gs[4];     // strides of the tile's and of the lattice's sites
    int lex;
};

// lexicographic index of the neighbour in direction MU
template <int MU, bool FWD>
__device__ __forceinline__ int nb_lex(const Geom &g, const TileSite &s)
{
    const int L = g.L[MU], wrap = (L - 1) * s.gs[MU];
    return FWD ? (s.x[MU] == L - 1 ? s.lex - wrap : s.lex + s.gs[MU])
               : (s.x[MU] == 0 ? s.lex + wrap : s.lex - s.gs[MU]);
}

template <int MU, bool FWD>
__device__ __forceinline__ void link_tile(const Geom &g, const GaugeRef<P_F64> &U, const TileSite &s, RawLink &r)
{
    r.load(U, FWD ? s.p : 1 - s.p, MU, FWD ? s.i : nb_lex<MU, FWD>(g, s) >> 1);
}

template <int PREC, int MU, bool FWD, int NT>
__device__ __forceinline__ void hop_tile(const Geom &g, const Tile &tl, const SpinorRef<PREC> &in,
                                         const Stage<PREC, NT> &st, const TileSite &t, const RawLink &r,
                                         cplx<double> acc[4][3])
{
    cplx<double> s[4][3], u[3][3];
    const int Tm = tl.T[MU], lw = (Tm - 1) * t.ls[MU];
    const bool edge = t.c[MU] == (FWD ? Tm - 1 : 0);
    const bool whole = Tm == g.L[MU];   // the tile spans the direction: its neighbours wrap inside
    const int step = FWD ? t.ls[MU] : -t.ls[MU], back = FWD ? -lw : lw;
    const double bc = g.bc[MU];
    if (edge & !whole) {
        in.load(1 - t.p, nb_lex<MU, FWD>(g, t) >> 1, s);
        pin(s);   // in this branch alone: else the two may be merged into one flat load
    } else {
        st.load(t.l + (edge ? back : step), s);
    }
    r.get(u);
    const bool wrap = t.x[MU] == (FWD ? g.L[MU] - 1 : 0);
    hop<double, MU, FWD>(acc, s, u, wrap ? bc : 1.0);
    pin(acc);
}

// Modes, arguments and block order (tile, RHS fastest) as in k_wilson.  Threads
// beyond the tile's sites (its volume need not be NT) only take part in the
// sums.
template <int PREC, int MODE, bool G5, int NT>
__global__ __launch_bounds__(NT, 2) void k_wilson_tile(WArgs a, Tile tl, ProArgs pro)
{
    __shared__ Stage<PREC, NT> stage;
    __shared__ double lds[2 * NT / 64 < 4 ? 4 : 2 * NT / 64];
    const Geom &g = a.g;
    const int first = kPro<MODE> && pro.kind ? a.nrhs : 0;
    if (kPro<MODE> && (int)blockIdx.x < first) {
        pro_stage<NT>(pro, blockIdx.x, lds);
        return;
    }
    const int lbr = xcd_remap(blockIdx.x - first, gridDim.x - first);
    const int r = lbr % a.nrhs;
    const int lb = lbr / a.nrhs;
    if (kPro<MODE> ? sits_out(pro, a.skip, r) : a.skip && a.skip[r]) return;
    const double rin_s = MODE == W_RESNORM && a.rin_scale ? a.rin_scale[r] : 1.0;
    TileSite t;
    t.l = threadIdx.x;
    {
        unsigned q = ((unsigned)t.l * tl.m3) >> 20;
        t.c[3] = t.l - (int)q * tl.T[3];
        unsigned q2 = (q * tl.m2) >> 20;
        t.c[2] = (int)q - (int)q2 * tl.T[2];
        q = (q2 * tl.m1) >> 20;
        t.c[1] = (int)q2 - (int)q * tl.T[1];
        t.c[0] = (int)q;
        int b = lb;
        t.x[3] = b % tl.N[3] * tl.T[3] + t.c[3];
        b /= tl.N[3];
        t.x[2] = b % tl.N[2] * tl.T[2] + t.c[2];
        b /= tl.N[2];
        t.x[1] = b % tl.N[1] * tl.T[1] + t.c[1];
        t.x[0] = b / tl.N[1] * tl.T[0] + t.c[0];
    }
    const bool valid = t.c[0] < tl.T[0];
    const int p = (t.x[0] + t.x[1] + t.x[2] + t.x[3]) & 1;
    t.p = p;
    t.gs[3] = 1;
    t.gs[2] = g.L[3];
    t.gs[1] = g.L[2] * t.gs[2];
    t.gs[0] = g.L[1] * t.gs[1];
    t.ls[3] = 1;
    t.ls[2] = tl.T[3];
    t.ls[1] = tl.T[2] * t.ls[2];
    t.ls[0] = tl.T[1] * t.ls[1];
    t.lex = t.x[0] * t.gs[0] + t.x[1] * t.gs[1] + t.x[2] * t.gs[2] + t.x[3];
    const int i = t.lex >> 1;
    t.i = i;
    const SpinorRef<PREC> in = spinor_ref<PREC>(a.in, a.in_sc, g.S, r);
    const GaugeRef<P_F64> U = gauge_ref<P_F64>(a.U, g.S);
    RawLink u0, u1;
    if (valid) {
        stage.fill(t.l, in, p, i);
        link_tile<0, true>(g, U, t, u0);
    }
    double shift_r, alpha_r;
    if (!site_scalars<MODE, NT>(a, pro, r, lds, &shift_r, &alpha_r)) return;
    __syncthreads();
    double q0 = 0.0, q1 = 0.0;
    if (valid) {
        cplx<double> acc[4][3];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) acc[s][k] = {0.0, 0.0};
        link_tile<0, false>(g, U, t, u1);
        hop_tile<PREC, 0, true, NT>(g, tl, in, stage, t, u0, acc);
        link_tile<1, true>(g, U, t, u0);
        hop_tile<PREC, 0, false, NT>(g, tl, in, stage, t, u1, acc);
        link_tile<1, false>(g, U, t, u1);
        hop_tile<PREC, 1, true, NT>(g, tl, in, stage, t, u0, acc);
        link_tile<2, true>(g, U, t, u0);
        hop_tile<PREC, 1, false, NT>(g, tl, in, stage, t, u1, acc);
        link_tile<2, false>(g, U, t, u1);
        hop_tile<PREC, 2, true, NT>(g, tl, in, stage, t, u0, acc);
        link_tile<3, true>(g, U, t, u0);
        hop_tile<PREC, 2, false, NT>(g, tl, in, stage, t, u1, acc);
        link_tile<3, false>(g, U, t, u1);
        hop_tile<PREC, 3, true, NT>(g, tl, in, stage, t, u0, acc);
        hop_tile<PREC, 3, false, NT>(g, tl, in, stage, t, u1, acc);
        cplx<double> d[4][3];
        stage.load(t.l, d);
        const double dn2 = diag_minus_half(acc, d, a.diag);
        site_out<PREC, MODE, G5>(a, r, r, 0, p, i, shift_r, rin_s, alpha_r, acc, dn2, q0, q1);
    }
    if (kSums<MODE>) {
        const double t0 = block_sum_w<NT / 64>(q0, lds);
        if (threadIdx.x == 0) a.partials[(size_t)r * a.nblk + lb] = t0;
        if (MODE == W_NORM) {
            const double t1 = block_sum_w<NT / 64>(q1, lds + NT / 64);
            if (threadIdx.x == 0) a.partials[(size_t)(a.nrhs + r) * a.nblk + lb] = t1;
        }
    }
}

}  // namespace ovl
