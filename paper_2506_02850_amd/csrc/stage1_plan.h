// How stage 1 lies on the chip: host arithmetic in plain C++, without HIP, so that it can be built and checked on its own.
#pragma once

#include <stdint.h>

#include "metok.h"

namespace metok {

constexpr int kPoolThreads = 256;

// Pooled rows when every frame takes the smaller of the two strides (s / alpha >= s, so no frame yields more).
inline int64_t worst_case_rows(int T, int grid_h, int grid_w, int s1, int s2, int pool_edge) {
    const int gmax = grid_h > grid_w ? grid_h : grid_w;
    int s_min = s1 < s2 ? s1 : s2;
    s_min = s_min < 1 ? 1 : (s_min > gmax ? gmax : s_min);
    auto side = [&](int g) { return pool_edge == METOK_POOL_FLOOR ? (g / s_min > 1 ? g / s_min : 1) : (g + s_min - 1) / s_min; };
    return static_cast<int64_t>(T) * side(grid_h) * side(grid_w);
}

// Workgroups of the pooling pass per frame: one for every kPoolThreads chunks of a frame at its smallest stride (782 frames of 24 x 24 x
// 136: 55 us with 36 workgroups, 26 so), made odd, and at most 47 (64 and more are up to a quarter slower).
// Odd: consecutive workgroups go to the chip's eight dies in turn, and in a frame of a larger stride only the first ones have work; with an even
// number those of all frames of the launch meet on some of the dies.  Whole calls by graph replay, us: 64 frames of 16 x 16 x 1024, 32 workgroups 29.8,
// 33 26.3; 200 of 16 x 16 x 768, 24 46.4, 25 40.6; 8 videos of 12 frames of 16 x 16 x 1024, 32 38.1, 33 33.8; 8 x 36 of 16 x 16 x 256 in fp32, 16 46.5, 17 38.2; 4
// x 212 of 16 x 14 x 1152, 32 221, 33 153.  Turning the shares of a frame's workgroups from frame to frame instead, with any number of them, is as
// good or 1 % slower.
// 47: 8 x 64 frames of 27 x 27 x 1152, 36 301, 47 291; 12 of 24 x 24 x 1024, 36 25.0, 47 23.5 (16 of them 24.7, 25.4); in fp32 37 of 16 x 16 x 1024,
// 36 29.2, 35 30.6, 47 29.7, 5 of 24 x 24 x 768 at strides 1 and 2 36 33.7, 47 30.3.  bf16 frames that may stay as they are (stride 1) take
// fewer in large launches: 4 x 316 of 15 x 15 x 464, 35 157, 47 172; 4 x 116 of 24 x 16 x 1024 167, 171; 2 x 64 of 24 x 24 x 1024 84.7, 83.6.
inline int pool_workgroups(int grid_h, int grid_w, int d, int dtype, int s1, int s2, int pool_edge) {
    const int most = (s1 == 1 || s2 == 1) && dtype == METOK_BF16 ? 35 : 47;
    const int64_t items = worst_case_rows(1, grid_h, grid_w, s1, s2, pool_edge) * (d / (dtype == METOK_BF16 ? 8 : 4));
    const int64_t odd = (items + kPoolThreads - 1) / kPoolThreads | 1;
    return odd < most ? static_cast<int>(odd) : most;
}

}  // namespace metok
