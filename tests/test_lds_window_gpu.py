"""128^2 frames on the LDS-resident kernels: the row-wise window pass at its edges (integer
and sub-pixel fractions in either direction, positions at the object's border, an object
wider than high) and the far fields that the mode-split form hands from its forward to
its adjoint pass (groups of unequal size, weights, a forward call in between), against
the oracle (forward 1e-5, gradients 1e-4 relative L2)."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import compare, custom_problem, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu


def _plan(p, tune):
    torch_cuda()
    from paper_2510_20929_amd import Plan
    return Plan.for_problem(p, tune=tune)


def _edges(p):
    """Fractions 0 and not in y and x, and the first and last windows that fit."""
    pos = p.positions.copy()
    hi = np.float32(p.H - p.N - 1)
    pos[0] = np.floor(pos[0])
    pos[1, 0] = np.floor(pos[1, 0])
    pos[2, 1] = np.floor(pos[2, 1])
    pos[3] = (0.0, 0.0)
    pos[4] = (hi, hi)
    pos[5] = (0.5, hi - np.float32(0.25))
    return replace(p, positions=pos)


@pytest.mark.parametrize("S,M,E,tune", [
    (1, 1, 1, {"variant": 6, "recompute": 1}),
    (1, 3, 1, {"variant": 5, "recompute": 1, "grid": 4}),
    (1, 2, 3, {"variant": 6, "recompute": 1}),
    (1, 3, 1, {"variant": 5, "mode_groups": 2}),
    (1, 5, 2, {"variant": 5, "mode_groups": 2, "grid": 5}),
    (1, 5, 2, {"variant": 4, "mode_groups": 2, "grid": 5}),
    (3, 1, 1, {"variant": 5}),
    (2, 3, 1, {"variant": 5, "recompute": 1, "grid": 3}),
])
def test_edges(S, M, E, tune):
    p, I = custom_problem(400 + 10 * S + M + E, 128, M, E, S, 150, 9, weights="opr" if E > 1 else None,
                          lz=40.0 if S > 1 else 0.0)
    p = _edges(p)
    grads = ("obj", "probe", "pos") + (("weights",) if E > 1 else ())
    plan = _plan(p, tune)
    first = run_gpu(plan, p, I, grads)
    compare(first, run_oracle(p, I, grads), grads, tag=f"S{S} M{M} E{E} {tune}")
    # the same plan again, after a forward call on it, gives the same bits
    run_gpu(plan, p, I, ())
    again = run_gpu(plan, p, I, grads)
    for key in ("g_obj", "g_probe", "g_pos"):
        assert np.array_equal(first[key], again[key]), key
