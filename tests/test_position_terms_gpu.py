"""Position gradients: no rounding beside that of the terms themselves. The fused bodies sum
few terms in FP32 before FP64 and take differences of the patch gradient before they
interpolate it."""

import numpy as np
import pytest

from gpu_util import W, custom_problem, rel_l2, run_gpu, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,variant,M,K", [(64, 0, 2, 60), (64, 1, 1, 60), (128, 0, 2, 40), (128, 1, 2, 40),
                                           (128, 6, 4, 40)])
def test_as_accurate_as_the_per_step_form(N, variant, M, K):
    """Error against the FP64 oracle over three problems beside the per-step form's on the
    same inputs, whose terms are summed in FP64 as they come. Each figure is the rms of
    at least 240 values (4.6 % of it, one sigma), so that equal ones agree within 26 % at
    four sigma of their ratio."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    sq = np.zeros(2)
    for seed in range(3):
        p, I = custom_problem(7100 + 10 * seed + variant, N, M, 1, 1, 190 if N == 128 else 110, K)
        plan = Plan.for_problem(p, tune={"variant": variant})
        ref = run_oracle(p, I, ("obj", "pos"))["g_pos"]
        for i, plain in enumerate((False, True)):
            sq[i] += rel_l2(run_gpu(plan, p, I, ("obj", "pos"), plain=plain)["g_pos"], ref) ** 2
    fused, plain = np.sqrt(sq / 3)
    print(f"N={N} variant={variant}: fused {fused:.2e}, per-step {plain:.2e}", flush=True)
    assert fused <= 1.26 * plain


@pytest.mark.parametrize("N,variant", [(256, 0), (256, 1), (512, 0), (512, 1)])
def test_long_sums_of_equal_terms(N, variant):
    """Constant frames, nothing measured, and an object that steps by 1 just below the frame: the
    last row's N terms are equal, all others 0. An FP32 sum of n equal values one after the
    other is off by 1.1e-7 (n = 16) or 2.3e-7 (32) rms over their mantissas, exact up to n = 4;
    the terms themselves carry six roundings (weight, exit wave, 2 dl/dI, conjugate
    products; 2.4e-8 rms each, 6e-8 together). 32 position weights: 1e-7 is allowed."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    rng = np.random.default_rng(31)
    K, u = 32, np.float32(1.37)
    obj = np.ones((1, N + 4, N + 4), np.complex64)
    obj[:, N:] = 2.0
    p = W.Problem("step", obj, np.full((1, 1, N, N), u, np.complex64), np.zeros((K, 2), np.float32),
                  rng.uniform(0.5, 2.0, (K, 1)).astype(np.float32), "amplitude")
    I = np.zeros((K, N, N), np.float32)
    got = run_gpu(Plan.for_problem(p, tune={"variant": variant}), p, I, ("obj", "pos"))["g_pos"][:, 0].astype(float)
    ref = 2.0 / (K * N * N) * p.weights[:, 0].astype(float) ** 2 * float(u) ** 2 * N
    e = float(np.sqrt(np.mean((got / ref - 1.0) ** 2)))
    print(f"N={N} variant={variant}: {e:.2e}", flush=True)
    assert e <= 1e-7
