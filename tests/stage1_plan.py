"""The library's plan of stage 1 (csrc/stage1_plan.h), built for the host."""
from tests.host_plan import host_library

SOURCE = r"""
#include "stage1_plan.h"
using namespace metok;
extern "C" int workgroups(int frames, int grid_h, int grid_w, int d, int dtype, int s1, int s2, int pool_edge) {
    return pool_workgroups(frames, grid_h, grid_w, d, dtype, s1, s2, pool_edge);
}
extern "C" int small(int T, int grid_h, int grid_w, int d, int dtype, int s1, int s2, int pool_edge, int one_pass) {
    return small_video(T, grid_h * grid_w, d, dtype, worst_case_rows(T, grid_h, grid_w, s1, s2, pool_edge), one_pass);
}
"""


def pool_workgroups(frames, grid_h, grid_w, d, dtype, s1, s2, edge=0):
    return host_library(SOURCE).workgroups(frames, grid_h, grid_w, d, 1 if dtype == "bf16" else 0, s1, s2, edge)


def small_video(T, grid, d, dtype, s1, s2, edge=0, one_pass=False):
    """Whether a video's call is one launch; one_pass: in the form where every stride is 2."""
    return bool(host_library(SOURCE).small(T, grid[0], grid[1], d, 1 if dtype == "bf16" else 0, s1, s2, edge, int(one_pass)))
