"""The batched window gather with two groups of threads a tile, which runs where every dataset of a
frame-size class meets at least 16 windows a tile: against the oracle and one call per dataset, with
odd object sizes, a dropped position, and both tile sides in one launch; and one group beside a
dataset without positions."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import compare, custom_problem, dev, rel_l2, run_oracle, torch_cuda

pytestmark = pytest.mark.gpu
GRADS = ("obj", "probe", "pos")


def _hits(p):
    """Windows that a tile meets on average, and whether the tiles have the larger side."""
    big = -(-p.W // 32) * -(-p.H // 32) >= 8192
    ts = 32 if big else 16
    return p.K * (p.N + ts) ** 2 / (p.H * p.W), big


def _run(probs, meas, per_call=False):
    torch = torch_cuda()
    from paper_2510_20929_amd import Batch
    b = Batch(probs)
    outs = [b.bind(i, dev(p.obj), dev(p.probe), dev(p.positions), I if torch.is_tensor(I) else dev(I))
            for i, (p, I) in enumerate(zip(probs, meas))]
    b.launch(GRADS, per_call=per_call)
    torch.cuda.synchronize()
    res = [{k: (float(v[0]) if k == "loss" else v.cpu().numpy()) for k, v in o.items()} for o in outs]
    flags = b.get_error()
    b.close()
    return res, flags


def _compare(probs, meas, drop=None, tag=""):
    got, flags = _run(probs, meas)
    pc, _ = _run(probs, meas, per_call=True)
    assert (flags != 0) == (drop is not None)
    for i, (p, I) in enumerate(zip(probs, meas)):
        for k in ("g_obj", "g_probe", "g_pos"):
            assert rel_l2(got[i][k], pc[i][k]) <= 1e-6 or not got[i][k].any(), (i, k)
        if p.K == 0:
            assert not got[i]["g_obj"].any() and got[i]["loss"] == 0.0
            continue
        keep = [k for k in range(p.K) if drop != (i, k)]
        ref = run_oracle(p.subset(keep), I[keep], GRADS, norm_count=p.K)
        got[i]["g_pos"] = got[i]["g_pos"][keep]
        compare(got[i], ref, GRADS, tag=f"{tag} {i}")


@pytest.mark.parametrize("N,shapes", [
    (64, [(101, 60), (97, 45), (118, 70)]),
    (128, [(180, 28), (163, 24)]),
])
def test_dense_datasets(N, shapes):
    cases = [custom_problem(300 + N + i, N, 1 + i % 2, 1, 1, H, K) for i, (H, K) in enumerate(shapes)]
    probs, meas = [c[0] for c in cases], [c[1] for c in cases]
    bad = probs[1].positions.copy()
    bad[3] = (shapes[1][0] - N + 7.0, 1.5)
    probs[1] = replace(probs[1], positions=bad)
    assert all(_hits(p)[0] >= 16 for p in probs)
    _compare(probs, meas, drop=(1, 3), tag=f"dense {N}")


def test_a_dataset_without_positions():
    (p, I), (q, J) = custom_problem(311, 64, 1, 1, 1, 101, 50), custom_problem(312, 64, 1, 1, 1, 93, 4)
    q = q.subset(np.arange(0))
    _compare([p, q], [I, J[:0]], tag="empty beside dense")


def test_both_tile_sides():
    """A large and a small dense object in one launch: the tiles of 32^2 and 16^2 hold separate
    state. Against one call per dataset (the large one has 5400 positions)."""
    torch = torch_cuda()
    p, I = custom_problem(321, 128, 1, 1, 1, 180, 28)
    rng = np.random.default_rng(3)
    H, K = 2917, 5400
    y, x = np.meshgrid(np.arange(H), np.arange(H), indexing="ij")
    obj = np.exp(0.3j * np.sin(y / 37.0) * np.cos(x / 23.0)).astype(np.complex64)[None]
    big = replace(p, obj=obj, positions=rng.uniform(0, H - 129, (K, 2)).astype(np.float32))
    assert _hits(big)[0] >= 16 and _hits(big)[1] and not _hits(p)[1]
    J = torch.rand((K, 128, 128), device="cuda")
    got, flags = _run([big, p], [J, I])
    pc, _ = _run([big, p], [J, I], per_call=True)
    assert flags == 0
    for a, c in zip(got, pc):
        for k in ("g_obj", "g_probe", "g_pos"):
            assert rel_l2(a[k], c[k]) <= 1e-6, k
    compare(got[1], run_oracle(p, I, GRADS), GRADS, tag="small beside large")
