"""Weight gradients of the four-step frames: the terms of eight pixels, or eight products, at most
are summed in FP32 before FP64, whether the fused kernel sums them or the contraction of the
staged frames."""
import numpy as np
import pytest

from gpu_util import W, dev, torch_cuda

pytestmark = pytest.mark.gpu


def _constant_problem(N, E, K, seed):
    """Constant frames: every weight-gradient term of a position is the same."""
    rng = np.random.default_rng(seed)
    probe = (1 + 1j) * np.ones((E, 1, N, N)) * rng.uniform(0.5, 2.0, (E, 1, 1, 1))
    w = rng.uniform(0.5, 2.0, (K, E))
    return W.Problem("constant", np.ones((1, N, N), np.complex64), probe.astype(np.complex64),
                     np.zeros((K, 2), np.float32), w.astype(np.float32), "amplitude")


def _weights(plan, p, plain=False):
    I = dev(np.zeros((p.K, p.N, p.N), np.float32))
    out = plan.forward_adjoint(dev(p.obj), dev(p.probe), dev(p.positions), I, weights=dev(p.weights),
                               grads=("weights",), plain=plain)
    return out["g_weights"].cpu().numpy().astype(float)


@pytest.mark.parametrize("N,tune", [(256, {}), (256, {"variant": 1}), (512, {})])
def test_contraction(N, tune):
    """g_w[k][e] is the same multiple of U_e for all e, up to the rounding of the sums: 5.4e-8
    rms over the mantissas for eight equal products (1.1e-7 for 16, 4.6e-7 for 64) and the
    result's own 2.4e-8, 6e-8 together; 9e-8 is allowed."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    p = _constant_problem(N, 16, 40, 5)
    r = _weights(Plan.for_problem(p, tune=tune), p) / p.probe[:, 0, 0, 0].real.astype(float)
    e = float(np.sqrt(np.mean((r / r.mean(1, keepdims=True) - 1.0) ** 2)))
    print(f"N={N} {tune}: {e:.2e}", flush=True)
    assert e <= 9e-8


@pytest.mark.parametrize("N,variant", [(256, 0), (256, 1), (512, 0), (512, 1)])
def test_one_eigenprobe(N, variant):
    """The fused kernel's own sums beside the per-step form's, which are FP64 throughout: the
    rounding of sums of eight equal terms, at most 5.4e-8 rms, and two results' own 2.4e-8;
    9e-8 is allowed."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    p = _constant_problem(N, 1, 64, 7)
    plan = Plan.for_problem(p, tune={"variant": variant})
    a, b = _weights(plan, p), _weights(plan, p, plain=True)
    e = float(np.sqrt(np.mean((a / b - 1.0) ** 2)))
    print(f"N={N} variant={variant}: {e:.2e}", flush=True)
    assert e <= 9e-8


@pytest.mark.parametrize("K", [1, 2, 16, 17, 32, 33, 257])
@pytest.mark.parametrize("N,E", [(256, 2), (256, 16), (512, 3)])
def test_few_positions(N, E, K):
    """Edges of the contraction's two row blocks of 16 positions and of its splits, beside the
    per-step form: every product, eight sums of one sign at most and the two results are rounded
    to 2^-24 each, so 16 * 2^-24 = 9.5e-7 bounds the difference of any weight."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    p = _constant_problem(N, E, K, 100 + K)
    plan = Plan.for_problem(p)
    e = float(np.max(np.abs(_weights(plan, p) / _weights(plan, p, plain=True) - 1.0)))
    print(f"N={N} E={E} K={K}: {e:.2e}", flush=True)
    assert e <= 16 * 2.0 ** -24
