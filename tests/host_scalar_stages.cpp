// Host check of the multishift CG's scalar stages (csrc/scalars.h): the stages
// are compiled for the CPU as one lane of a one-wave block, with one shift and
// one partial sum.  A launch that carries a stage runs it beside its site
// blocks, whose waves read the RHS's "sits out" flag at any time: the answer
// before the stage must be the answer after it, whatever the stage decides.
// Built and run by tests/test_scalar_stages.py with g++ against a device.h of
// its own; exit status 0 and a final "ok" line mean every check passed.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <limits>

#include "csrc/scalars.h"

using namespace ovl;

static int failures = 0;

static void check(bool ok, const char *what)
{
    if (!ok) {
        std::printf("FAIL %s\n", what);
        failures++;
    }
}

// one RHS with |r|^2 = |b|^2 = 1, tolerance 1e-3, one open shift
static void fresh(MState &st)
{
    std::memset(&st, 0, sizeof st);
    st.nrhs = st.nshift = 1;
    st.rr[0] = st.bb[0] = st.alpha[0] = st.alpha_old[0] = 1.0;
    st.zeta[0][0] = st.zeta_old[0][0] = st.zeta_new[0][0] = 1.0;
    st.tol2r[0] = 1e-6;
    st.act[0][0] = 1;
    st.frozen_at[0][0] = -1;
}

int main()
{
    static MState st;
    static Blk bk;
    double lds[4], sum = 0.0;
    const double nan = std::numeric_limits<double>::quiet_NaN();
    const ProArgs pa{PRO_ALPHA, 1, 1, 1, 0, &sum, &st, &bk, 0.0, 1};
    ProArgs pb{PRO_BETA, 1, 1, 1, 0, &sum, &st, &bk, 0.0, 0};

    // alpha from |t|^2: in order, zero, not finite, negative
    for (double tt : {0.5, 0.0, nan, -1.0}) {
        fresh(st);
        sum = tt;
        const bool before = sits_out(pa, st.skip, 0);
        alpha_stage<64>(pa, 0, lds);
        check(!before && sits_out(pa, st.skip, 0) == before, "alpha stage: sites see one answer");
        const bool good = tt == 0.5;
        check(st.run_c[0] == good && st.nonfinite[0] == !good && st.alpha[0] == (good ? 2.0 : 1.0),
              "alpha stage: state");
        // the next launch carries beta: its sites take part only after a good alpha
        sum = 0.25;
        const bool beta_before = sits_out(pb, st.skip, 0);
        check(beta_before == !good, "beta stage: sites follow alpha");
        beta_stage<64>(pb, 0, lds);
        check(sits_out(pb, st.skip, 0) == beta_before, "beta stage: sites see one answer");
        check(st.skip[0] == !good && st.iter[0] == good, "beta stage: a failed RHS has ended");
    }
    // beta from |r|^2: goes on, finishes, pauses, not finite
    struct { double rr, sw2; int skip, paused, nonfinite; } ends[] = {
        {0.25, 0.0, 0, 0, 0}, {1e-8, 0.0, 1, 0, 0}, {1e-4, 1e-3, 1, 1, 0}, {nan, 0.0, 1, 0, 1}};
    for (const auto &e : ends) {
        fresh(st);
        sum = 0.5;
        alpha_stage<64>(pa, 0, lds);
        sum = e.rr;
        pb.sw2 = e.sw2;
        const bool before = sits_out(pb, st.skip, 0);
        beta_stage<64>(pb, 0, lds);
        check(!before && sits_out(pb, st.skip, 0) == before, "beta stage: sites see one answer");
        check(st.skip[0] == e.skip && st.paused[0] == e.paused && st.nonfinite[0] == e.nonfinite, "beta stage: state");
        // the iteration after: an ended RHS takes no part in either launch
        const bool off = sits_out(pa, st.skip, 0);
        alpha_stage<64>(pa, 0, lds);
        check(off == (e.skip != 0) && sits_out(pa, st.skip, 0) == off, "alpha stage: an ended RHS stands still");
        check(sits_out(pb, st.skip, 0) == off, "beta stage: an ended RHS stands still");
    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
