"""The LDS-resident 128^2 bodies add intensities, patch gradients and probe gradients one rounded
term at a time, as the register-resident ones do."""
import numpy as np
import pytest

from gpu_util import custom_problem, dev, run_gpu, torch_cuda

pytestmark = pytest.mark.gpu


def _plan(p, **tune):
    torch_cuda()
    from paper_2510_20929_amd import Plan
    return Plan.for_problem(p, tune=tune)


@pytest.mark.parametrize("weights,tunes", [
    (None, [{"variant": 1}, {"variant": 5}, {"variant": 6}]),
    ("amp", [{"variant": 1}, {"variant": 5}, {"variant": 6}]),
    (None, [{"variant": 4, "mode_groups": 2}, {"variant": 5, "mode_groups": 2}]),
])
def test_intensities(weights, tunes):
    """The forward transform rounds alike in both layouts, so the intensities are the same bits."""
    p, I = custom_problem(81, 128, 5, 1, 1, 160, 5, weights=weights)
    res = [run_gpu(_plan(p, **t), p, I, ("obj",))["I_pred"] for t in tunes]
    for r in res[1:]:
        assert np.array_equal(r, res[0])


@pytest.mark.parametrize("variant", [1, 5, 6])
@pytest.mark.parametrize("weighted", [False, True])
def test_opposite_terms_cancel(variant, weighted):
    """Two modes (positions) with the same probe (patch) and opposite far fields: rounded terms
    cancel to 0 in the patch (probe) gradient; a term whose products meet the sum unrounded
    leaves a remainder."""
    for M, K in ((2, 1), (1, 2)):
        p, _ = custom_problem(91, 128, M, 1, 1, 160, K)
        probe = np.repeat(p.probe[:, :1], M, 1)
        pos = np.repeat(p.positions[:1], K, 0)
        rng = np.random.default_rng(17)
        y = (rng.normal(size=(128, 128)) + 1j * rng.normal(size=(128, 128))).astype(np.complex64)
        Y = np.stack([y, -y]).reshape(K, M, 128, 128)
        w = dev(np.ones((K, 1), np.float32)) if weighted else None
        g_obj, g_probe = _plan(p, variant=variant, grid=1).apply_AH(dev(Y), dev(p.obj), dev(probe), dev(pos), weights=w)
        assert not (g_obj if M == 2 else g_probe).cpu().numpy().any(), (M, K)
        assert (g_probe if M == 2 else dev(np.ones(1))).cpu().numpy().any()
