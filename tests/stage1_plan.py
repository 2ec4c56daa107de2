"""The library's plan of stage 1 (csrc/stage1_plan.h), built for the host."""
from tests.host_plan import host_library

SOURCE = r"""
#include "stage1_plan.h"
using namespace metok;
extern "C" int workgroups(int grid_h, int grid_w, int d, int dtype, int s1, int s2, int pool_edge) {
    return pool_workgroups(grid_h, grid_w, d, dtype, s1, s2, pool_edge);
}
"""


def pool_workgroups(grid_h, grid_w, d, dtype, s1, s2, edge=0):
    return host_library(SOURCE).workgroups(grid_h, grid_w, d, 1 if dtype == "bf16" else 0, s1, s2, edge)
