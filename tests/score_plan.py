"""The library's plan of the score passes (csrc/score_plan.h), built for the host: what a call's rows, keys and workspace are cut into."""
import ctypes
from collections import namedtuple

from tests.host_plan import host_library

SOURCE = r"""
#include <initializer_list>
#include "score_plan.h"
using namespace metok;
// the plan of a call, and the one that it would have with whole rows
extern "C" int plans(int batch, int64_t S, int Hq, int Hkv, int dh, int Tq, int vis_start, int n_vis, int dtype, int mode, int64_t* out) {
    ScoreGeom whole, g;
    ScorePlan pw, p;
    if (!make_geom(S, Hq, Hkv, dh, Tq, vis_start, n_vis, dtype, mode, &whole)) return 1;
    g = whole;
    plan_grid(whole, n_vis, chunk_count(dh, dtype), batch, select_bytes(n_vis), &pw);
    plan_score(&g, n_vis, dtype, batch, &p);
    auto put = [&](const ScoreGeom& a, const ScorePlan& b) {
        for (int64_t v : {int64_t(a.rs), int64_t(a.rbw), int64_t(b.nx1), int64_t(b.per1), int64_t(b.nx2), int64_t(b.per2), int64_t(b.off_qfrag), int64_t(b.off_pstat),
                          int64_t(b.off_norm), int64_t(b.off_colpart), int64_t(b.off_sel), int64_t(b.off_inplace), int64_t(b.total), int64_t(partial_bytes(a, b))})
            *out++ = v;
    };
    put(g, p);
    put(whole, pw);
    *out++ = g.rb_total; *out++ = select_general_bytes(n_vis); *out++ = sizeof(FastSel); *out++ = inplace_bytes(S);
    return 0;
}
"""
Plan = namedtuple("Plan", "rs rbw nx1 per1 nx2 per2 qfrag pstat norm colpart sel inplace total partials")
Plans = namedtuple("Plans", "plan whole rb_total general_bytes fast_bytes inplace_bytes split")


def score_plans(S, n_vis, Hq, Hkv, dh, Tq, dtype="bf16", batch=1, vis_start=0, mode=0):
    out = (ctypes.c_int64 * 32)()
    i, q = ctypes.c_int, ctypes.c_int64
    assert host_library(SOURCE).plans(i(batch), q(S), i(Hq), i(Hkv), i(dh), i(Tq), i(vis_start), i(n_vis), i(1 if dtype == "bf16" else 0), i(mode), out) == 0
    plan, whole = Plan(*out[:14]), Plan(*out[14:28])
    return Plans(plan, whole, *out[28:32], plan.rs != whole.rs)
