"""64^2 (and smaller) frames: the object window that goes through LDS and the row-wise
window pass at their edges (integer and sub-pixel fractions in either direction, the last
windows that fit, whose row or column N lies outside the object), the probe accumulator
that the first position writes without reading it (workgroups with none, one and several
positions), and calls without an accumulator, against the oracle (forward 1e-5, gradients
1e-4 relative L2)."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import compare, custom_problem, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu


def _edges(p, want_pos):
    pos = p.positions.copy()
    hi = np.float32(p.H - p.N)  # an integer position needs no row N
    pos[0] = np.floor(pos[0])
    pos[1, 0] = np.floor(pos[1, 0])
    pos[2, 1] = np.floor(pos[2, 1])
    pos[3] = (0.0, 0.0)
    if not want_pos:  # the position gradient needs a full window
        pos[4] = (hi, hi)
        pos[5] = (hi, 0.5)
        pos[6] = (1.25, hi)
    return replace(p, positions=pos)


@pytest.mark.parametrize("N,M,E,grads,tune", [
    (64, 1, 1, ("obj", "probe"), None),
    (64, 2, 1, ("obj", "probe", "pos"), {"grid": 5}),
    (64, 1, 1, ("obj", "probe"), {"variant": 1, "grid": 20}),
    (64, 2, 3, ("obj", "probe", "pos", "weights"), {"variant": 2, "grid": 4}),
    (64, 3, 1, ("obj",), {"variant": 3, "recompute": 1}),
    (64, 2, 1, ("obj", "probe"), {"variant": 4, "probe_stage": 1}),
    (32, 2, 2, ("obj", "probe", "weights"), {"grid": 3}),
    (128, 2, 1, ("obj", "probe", "pos"), {"variant": 0, "grid": 2}),
    (128, 1, 1, ("obj", "probe"), {"variant": 3, "grid": 2}),
])
def test_edges(N, M, E, grads, tune):
    torch_cuda()
    from paper_2510_20929_amd import Plan
    p, I = custom_problem(700 + N + M + E, N, M, E, 1, N + 23, 11, weights="opr" if E > 1 else None)
    p = _edges(p, "pos" in grads)
    plan = Plan.for_problem(p, tune=tune)
    first = run_gpu(plan, p, I, grads)
    compare(first, run_oracle(p, I, grads), grads, tag=f"N{N} M{M} E{E} {tune}")
    again = run_gpu(plan, p, I, grads)
    for g in grads:
        assert np.array_equal(first["g_" + g], again["g_" + g]), g
