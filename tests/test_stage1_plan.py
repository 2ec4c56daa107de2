"""The plan of stage 1's kernels, on the host."""
import random

from tests.stage1_plan import pool_workgroups


def test_pooling_workgroups():
    rng = random.Random(3)
    for _ in range(3000):
        frames, gh, gw, d = rng.choice([rng.randint(1, 20), rng.randint(1, 5000)]), rng.randint(1, 40), rng.randint(1, 40), 8 * rng.randint(1, 300)
        dtype, s1, s2, edge = rng.choice(["bf16", "f32"]), rng.randint(1, 6), rng.randint(1, 6), rng.choice([0, 1])
        n = pool_workgroups(frames, gh, gw, d, dtype, s1, s2, edge)
        s = min(s1, s2, max(gh, gw))
        side = (lambda g: max(1, g // s)) if edge == 0 else (lambda g: -(-g // s))
        chunks = side(gh) * side(gw) * d // (8 if dtype == "bf16" else 4)
        wanted, a = -(-chunks // 256), (frames, gh, gw, d, dtype, s1, s2, edge, n)
        assert 1 <= n <= 47 and (n in (wanted, wanted + 1) or 35 <= n < wanted), a
        if frames >= 16:
            assert n % 4 or n == 36 and dtype == "f32", a


def test_a_batch_of_short_videos_is_spread_over_the_dies():
    # 8 videos of 12 frames are 96 frames of one launch: 33.8 us with 33 workgroups a frame, 38.1 with 32
    assert pool_workgroups(12, 16, 16, 1024, "bf16", 2, 3) == 32 and pool_workgroups(96, 16, 16, 1024, "bf16", 2, 3) == 33
