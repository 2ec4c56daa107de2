// How stage 1 lies on the chip: host arithmetic in plain C++, without HIP, so that it can be built and checked on its own.
#pragma once

#include <stdint.h>

#include "metok.h"

namespace metok {

constexpr int kSegThreads = 1024;
constexpr int kPoolThreads = 256;

// Up to here one workgroup adds up the partials too, two frames per wave, and nothing is handed over; but not where the frames
// beyond one per wave bring more than kOneReducePartials partial sums, which a second workgroup would read in the meantime.  Whole
// calls of T frames x C partials, us, one workgroup / several: 32 x 256 17.8 / 18.3 and 16.1 / 16.7, 32 x 576 22.4 / 21.6 and 29.3 / 28.3,
// 32 x 4096 67.3 / 60.4; 24 x 1024 25.0 / 25.3, 24 x 1600 30.5 / 30.0; 17 x 4096 43.0 / 43.1.
constexpr int kOneReduceFrames = 32, kOneReducePartials = 8192;

// Pooled rows when every frame takes the smaller of the two strides (s / alpha >= s, so no frame yields more).
inline int64_t worst_case_rows(int T, int grid_h, int grid_w, int s1, int s2, int pool_edge) {
    const int gmax = grid_h > grid_w ? grid_h : grid_w;
    int s_min = s1 < s2 ? s1 : s2;
    s_min = s_min < 1 ? 1 : (s_min > gmax ? gmax : s_min);
    auto side = [&](int g) { return pool_edge == METOK_POOL_FLOOR ? (g / s_min > 1 ? g / s_min : 1) : (g + s_min - 1) / s_min; };
    return static_cast<int64_t>(T) * side(grid_h) * side(grid_w);
}

// Workgroups of the pooling pass per frame, for a launch of `frames` frames (of all its videos): one for every kPoolThreads chunks of a
// frame at its smallest stride (782 frames of 24 x 24 x 136: 55 us with 36 workgroups, 26 so), at most 36 to 47 (64 and more are up
// to a quarter slower), and below that no multiple of four.
// No multiple of four: consecutive workgroups go to the chip's eight dies in turn, and in a frame of a larger stride only the first ones
// have work; with a multiple of 8 (4) those of all frames meet on one (two) of the dies.  Whole calls by graph replay, us: 64 frames of
// 16 x 16 x 1024, 32 workgroups 29.8, 33 26.3; 200 of 16 x 16 x 768, 24 46.4, 25 40.6; 8 videos of 12 frames of 16 x 16 x 1024, 32 38.1, 33
// 33.8; 8 x 36 of 16 x 16 x 256 in fp32, 16 46.5, 17 38.2; 4 x 212 of 16 x 14 x 1152, 32 221, 33 153.  Counts that are even otherwise are as
// good as the next odd one (4 x 241 of 12 x 12 x 1024, 18 115.9, 19 116.1; 2 x 144 of 14 x 14 x 224, 6 and 7 31.1).  Turning the shares of
// a frame's workgroups from frame to frame instead, with any number of them, is as good or 1 % slower.
// At most 47 in bf16: 8 x 64 frames of 27 x 27 x 1152, 36 301, 47 291; frames that may stay as they are (stride 1) take fewer in large
// launches: 4 x 316 of 15 x 15 x 464, 35 157, 47 172; 4 x 116 of 24 x 16 x 1024 167, 171; 2 x 64 of 24 x 24 x 1024 84.7, 83.6.  At most 36
// in fp32, where limits from 35 to 49 differ by 1 % in the mean over 39 shapes: 37 of 16 x 16 x 1024 36 29.5, 35 30.6, 47 30.0; 24 of the same
// 30.9, 31.6, 32.5; 83 of 24 x 24 x 728 at strides 1 and 2 78.7, 78.3, 76.0.
// Fewer than 16 frames have nothing to spread and take up to 36: 10 of 24 x 24 x 1024 at strides 1 and 2, 36 29.7, 35 32.3; 7 of 27 x 27 x
// 184, 18 26.0, 19 26.8; 12 of 27 x 27 x 768 in fp32, 36 27.2, 47 27.9 (12 of 24 x 24 x 1024 25.0, 23.5).
inline int pool_workgroups(int64_t frames, int grid_h, int grid_w, int d, int dtype, int s1, int s2, int pool_edge) {
    const bool few = frames < 16;
    const int most = few || dtype != METOK_BF16 ? 36 : (s1 == 1 || s2 == 1 ? 35 : 47);
    const int64_t items = worst_case_rows(1, grid_h, grid_w, s1, s2, pool_edge) * (d / (dtype == METOK_BF16 ? 8 : 4));
    const int64_t n = (items + kPoolThreads - 1) / kPoolThreads;
    if (n >= most) return most;
    return static_cast<int>(n < 1 ? 1 : (!few && n % 4 == 0 ? n + 1 : n));
}

constexpr int kSmallRun = 4;                        // frames of a token that sixteen lanes take together
constexpr int kSmallTokens = 512;                   // of all frames of the video
constexpr int64_t kSmallBytes = 128 * 1024;

// Whether small_video_kernel takes the call: the rounds of loads that its statistics and its pooling take one after the other, and what
// it reads at one compute unit's rate.  Whole calls by graph replay, us, three launches / this one: 8 frames of 4 x 4 x 64 fp32 (32 KB)
// 12.7 / 8.3, 4 of 5 x 5 x 64 12.9 / 8.4, 4 of 4 x 4 x 1024 (128 KB) 13.8 / 10.8, 8 of 8 x 8 x 128 (128 KB) 14.3 / 12.7, 32 of 4 x 4 x
// 128 (128 KB) 15.0 / 13.5; beyond the lines, 2 of 16 x 16 x 64 (4 rounds of the statistics with half the frames missing) 11.7 / 14.3, 4
// of 2 x 2 x 4096 (16 rounds) 13.6 / 15.6, 32 of 4 x 4 x 128 at stride 1 (8 rounds of the pooling) 14.7 / 19.8.  Where the one-pass
// kernel makes it two launches: 8 of 4 x 4 x 64 fp32 10.1 / 7.9, 32 of 4 x 4 x 128 12.1 / 14.4.
inline bool small_video(int T, int N, int d, int dtype, int64_t worst_rows, bool one_pass) {
    const int64_t chunks = d / (dtype == METOK_BF16 ? 8 : 4), units = static_cast<int64_t>((T + kSmallRun - 1) / kSmallRun) * N;
    if (T > kOneReduceFrames || units * kSmallRun > kSmallTokens || T * N * chunks * 16 > kSmallBytes) return false;
    const int64_t stats = (units + kSegThreads / 16 - 1) / (kSegThreads / 16) * ((chunks + 31) / 32), pool = (worst_rows * chunks + kSegThreads - 1) / kSegThreads;
    return one_pass ? stats <= 1 && pool <= 1 : stats <= 4 && pool <= 2;
}

}  // namespace metok
