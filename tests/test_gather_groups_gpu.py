"""Window gather with one, two and four groups of threads per object tile, against the
oracle (gradients 1e-4 relative L2): hit counts that leave groups with unequal runs or none,
several chunks of positions, several slices, tile rows that do not divide by eight, and
windows that are dropped."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import compare, custom_problem, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu

CASES = [
    # N, S, H, K: windows per 16 x 16 tile, tiles
    (32, 1, 77, 3),     # 1 per tile: one group
    (32, 1, 77, 47),    # 18 per tile, 25 tiles: four groups, fewer than four runs
    (32, 1, 49, 1100),  # above 1000 per tile: two chunks of positions
    (64, 2, 99, 60),    # slices: 98 tiles, 39 per tile
    (64, 1, 530, 720),  # 1156 tiles, 16 per tile: two groups
]


@pytest.mark.parametrize("N,S,H,K", CASES)
def test_gather_groups(N, S, H, K):
    torch_cuda()
    from paper_2510_20929_amd import Plan
    p, I = custom_problem(500 + N + H + K, N, 1, 1, S, H, K, lz=40.0 if S > 1 else 0.0)
    pos = p.positions.copy()
    pos[0] = (0.0, 0.0)
    pos[1] = (H - N - 1, H - N - 1)
    p = replace(p, positions=pos)
    grads = ("obj", "probe")
    plan = Plan.for_problem(p)
    got = run_gpu(plan, p, I, grads)
    compare(got, run_oracle(p, I, grads), grads, tag=f"N{N} S{S} H{H} K{K}")
    again = run_gpu(plan, p, I, grads)
    assert np.array_equal(got["g_obj"], again["g_obj"])
