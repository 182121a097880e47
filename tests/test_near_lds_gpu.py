"""Near field of 128^2 frames on the LDS-resident kernel at the edges of its dispatch, against
the oracle (forward 1e-5, gradients 1e-4 relative L2): one mode (nothing parked between
modes), several with weights and staged or accumulated probe gradients, each subset of
gradients, more workgroups than positions and fewer, a dropped position, and the forward
call alone."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import compare, custom_problem, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu


def _plan(p, tune):
    torch_cuda()
    from paper_2510_20929_amd import Plan
    return Plan.for_problem(p, tune=tune)


@pytest.mark.parametrize("M,E,loss,weights,grads,tune", [
    (1, 1, "amplitude", None, ("obj", "probe", "pos", "lambda_z"), None),
    (1, 1, "poisson", None, ("obj",), {"grid": 3}),
    (3, 1, "amplitude", "amp", ("probe", "weights", "lambda_z"), {"grid": 2, "variant": 1}),
    (2, 3, "amplitude", "opr", ("obj", "probe", "pos", "weights", "lambda_z"), {"grid": 4}),
    (2, 1, "poisson", None, ("probe", "pos"), {"probe_stage": 1, "grid": 20}),
])
def test_near_lds(M, E, loss, weights, grads, tune):
    p, I = custom_problem(600 + 10 * M + E, 128, M, E, 1, 157, 7, loss=loss, weights=weights, det_lambda_z=45.0)
    pos = p.positions.copy()
    pos[0] = np.floor(pos[0])
    pos[1, 0] = np.floor(pos[1, 0])
    p = replace(p, positions=pos)
    plan = _plan(p, tune)
    first = run_gpu(plan, p, I, grads)
    compare(first, run_oracle(p, I, grads), grads, tag=f"near M{M} E{E} {tune}")
    fwd = run_gpu(plan, p, I, ())
    assert fwd["loss"] == first["loss"]
    again = run_gpu(plan, p, I, grads)
    for g in grads:
        assert np.array_equal(first["g_" + g], again["g_" + g]), g


def test_dropped_position():
    """A position whose window leaves the object adds nothing, also where it is the only one
    of its workgroup."""
    p, I = custom_problem(640, 128, 2, 1, 1, 160, 4, det_lambda_z=45.0)
    grads = ("obj", "probe", "lambda_z")
    bad = p.positions.copy()
    bad[2] = (140.0, 3.5)
    keep = [0, 1, 3]
    got = run_gpu(_plan(p, None), replace(p, positions=bad), I, grads, want_ipred=False)
    assert got["flags"] != 0
    compare(got, run_oracle(p.subset(keep), I[keep], grads, norm_count=4), grads, tag="near dropped")
