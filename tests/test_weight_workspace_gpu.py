"""Weight gradients of staged 512^2 frames in calls of several chunks: the split partial sums
take room for one chunk, whatever the call's size, and every chunk's results land at its own
positions, in the mode-split form and in the fused one."""
import numpy as np
import pytest

from gpu_util import custom_problem, dev, torch_cuda

pytestmark = pytest.mark.gpu


def test_workspace_per_position():
    """Beyond a chunk, a position costs its partial sums (loss, two position terms a group, E
    weights) and nothing that grows with the splits: 8 (1 + 2 15 + 3) = 272 bytes."""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    size = []
    for K in (4000, 12000):
        plan = Plan(512, n_modes=15, n_eig=3, obj_h=600, obj_w=600, max_positions=K,
                    tune={"mode_groups": 15, "plain_chunk": 1})
        size.append(plan.info()["workspace_bytes"])
        plan.close()
    assert size[1] - size[0] <= 512 * 8000


@pytest.mark.parametrize("tune", [{"plain_chunk": 1}, {"mode_groups": 15, "plain_chunk": 1}])
def test_chunks(tune):
    """One call of 75 positions (chunks of 68 at most) against calls of 25 with the same
    normaliser: weight gradients agree to the rounding of FP64 sums taken in other splits,
    i.e. to FP32's last digit."""
    torch = torch_cuda()
    from paper_2510_20929_amd import Plan
    p, _ = custom_problem(57, 512, 15, 3, 1, 560, 1, weights="opr")
    rng = np.random.default_rng(5)
    K = 75
    pos = dev(rng.uniform(0, 46, (K, 2)).astype(np.float32))
    w = dev((rng.normal(size=(K, 3)) * [0.1, 0.05, 0.05] + [1, 0, 0]).astype(np.float32))
    I = torch.rand((K, 512, 512), device="cuda") * 0.2

    def run(n):
        plan = Plan(512, n_modes=15, n_eig=3, obj_h=560, obj_w=560, max_positions=n, norm_count=K, tune=tune)
        out = []
        for k in range(0, K, n):
            s = slice(k, k + n)
            out.append(plan.forward_adjoint(dev(p.obj), dev(p.probe), pos[s].contiguous(), I[s].contiguous(),
                                            weights=w[s].contiguous(), grads=("weights",))["g_weights"].cpu().numpy())
        assert plan.get_error() == 0
        plan.close()
        return np.concatenate(out)

    whole, parts = run(K), run(25)
    scale = np.abs(parts).max(1, keepdims=True)
    assert scale.min() > 0
    assert (np.abs(whole - parts) <= 2.4e-7 * scale).all()
