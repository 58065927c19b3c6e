// Which kernels the planner sends a convolution pass to, for tests that have to reach one of them (built by
// conftest.py as a shared library; host code only).
#include "../paper_1312_5853_amd/csrc/plan.h"

using namespace convnet;

// ws_bytes: what the call brings, or -1: as much as it wants.  out: 0 fp32 kernels, 1 three-part kernels, 2 vector units, 3
// bf16 with the input window in LDS; fold; splits of the reduction; rows, columns of a tile; workspace; of the window kernel
// channel blocks per step and chunks; whether the columns of a bf16 backward-filter run in one launch; whether a three-part pass
// looks for operands that two parts hold; whether it runs on the four-wave tiles
extern "C" int plan_query(int op, int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int groups, int dtype,
                          long long ws_bytes, long long *out)
{
    Problem pb;
    const int rc = make_problem(pb, N, C / groups, H, W, K / groups, R, S, stride, pad, 0, 0, dtype);
    if (rc != kStatusOk) return rc;
    if (groups > 1) {
        pb.groups = groups;
        pb.x_bs = (int64_t)C * H * W; pb.y_bs = (int64_t)K * pb.P * pb.Q;
        pb.x_gs = pb.x_bs / groups; pb.y_gs = pb.y_bs / groups; pb.w_gs = (int64_t)(K / groups) * (C / groups) * R * S;
    }
    const Plan pl = ws_bytes < 0 ? make_plan(op, pb) : plan_for_workspace(op, pb, (size_t)ws_bytes);
    out[0] = pl.direct ? 2 : pl.sp || pl.rows_split ? 1 : pl.win ? 3 : 0;
    out[1] = pl.sp ? (pl.sp_fold > 1 ? pl.sp_fold : 1) : 1;
    out[2] = pl.nsplit;
    out[3] = pl.sp ? pl.sp_bm : pl.win ? pl.win_bm : pl.tile.bm();
    out[4] = pl.sp ? pl.sp_bn : pl.win ? pl.win_tn * 32 * (pl.win_bm == 64 ? 4 : 2) : pl.tile.bn();
    out[5] = (long long)pl.total;
    out[6] = pl.win ? pl.win_ncb : 0;
    out[7] = pl.win ? pl.win_cb / pl.win_ncb : 0;
    out[8] = pl.lin && pl.fused_groups && !pl.direct;
    out[9] = pl.sp_two;
    out[10] = pl.sp_pair;
    return kStatusOk;
}

// Walks a split forward / stride-1 backward-data pass from step to step as its kernel does, by split_steps: how many
// steps read from elsewhere than the place that their channel block and tap have in the re-laid copy, or from outside it.  -1: the
// pass runs on other kernels.
extern "C" long long split_walk(int op, int N, int C, int H, int W, int K, int R, int pad)
{
    Problem pb;
    if (make_problem(pb, N, C, H, W, K, R, R, 1, pad, 0, 0, kDtypeF32) != kStatusOk) return -1;
    const Plan pl = make_plan(op, pb);
    if (!pl.sp || op == kOpBwdFilter) return -1;
    const int sign = op == kOpFwd ? 1 : -1;
    const int64_t plane = (int64_t)pl.sp_hp * pl.sp_wp * 32, copy = pl.sp_cb * 3 * plane;
    const ClassGrid h = class_grid(op == kOpFwd, H, R, 1, pad, 0), w = class_grid(op == kOpFwd, W, R, 1, pad, 0);
    const int ty = h.first + pl.sp_ph, tx = w.first + pl.sp_pw;
    const SplitSteps d = split_steps((unsigned)plane, pl.sp_wp, R, R, sign);
    long long wrong = 0;
    int64_t at = sign > 0 ? 0 : ((int64_t)ty * pl.sp_wp + tx) * 32;
    for (int cb = 0; cb < pl.sp_cb; ++cb)
        for (int r = 0; r < R; ++r)
            for (int s = 0; s < R; ++s) {
                const int64_t place = cb * 3 * plane + ((int64_t)(sign > 0 ? r : ty - r) * pl.sp_wp + (sign > 0 ? s : tx - s)) * 32;
                wrong += at != place || at < 0 || at >= copy;
                at += s + 1 < R ? d.s : r + 1 < R ? d.r : d.c;
            }
    return wrong;
}
