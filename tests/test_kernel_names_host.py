"""The kernel instances that the bench line reports exist in the built library under those names, and
the record of their traffic is tied to every source that they are compiled from (no GPU)."""
import os
import re
import shutil
import subprocess
import types

import pytest

import bench
from paper_2510_20929_amd import build

# frame, modes, slices, loss, detector distance, tune, threads
PLANS = [
    (64, 1, 1, "amplitude", None, None, 512),
    (64, 1, 1, "amplitude", None, {"variant": 4}, 256),
    (128, 4, 1, "poisson", None, {"variant": 4}, 1024),
    (128, 4, 1, "poisson", None, {"variant": 5}, 1024),
    (128, 4, 1, "poisson", None, {"variant": 6}, 1024),
    (128, 2, 8, "amplitude", None, {"variant": 5}, 1024),
    (128, 2, 8, "amplitude", None, {"variant": 1}, 1024),
    (128, 2, 1, "amplitude", 45.0, None, 1024),
    (64, 2, 1, "amplitude", 45.0, None, 512),
    (256, 1, 1, "amplitude", None, {"variant": 0}, 1024),
    (512, 1, 1, "poisson", None, {"variant": 0}, 512),
    (512, 1, 1, "amplitude", None, {"variant": 1}, 256),
]


@pytest.fixture(scope="module")
def symbols():
    nm = shutil.which("nm") or "/opt/rocm/llvm/bin/llvm-nm"
    out = subprocess.run([nm, "-C", build.LIB], capture_output=True, text=True, check=True).stdout
    return set(re.findall(r"ptyhip::(\w+_kernel<[^>]*>)", out))


@pytest.mark.parametrize("N,M,S,loss,det,tune,threads", PLANS)
def test_reported_instance_exists(symbols, N, M, S, loss, det, tune, threads):
    plan = types.SimpleNamespace(info=lambda: {"threads": threads})
    prob = types.SimpleNamespace(N=N, M=M, S=S, loss=loss, det_lambda_z=det)
    assert bench.kernel_instance(plan, prob, tune) in symbols


def test_hash_covers_the_headline_kernel():
    """The unit of the LDS-resident kernels and every header it includes, but for launch.hpp's
    declarations of other units."""
    root = os.path.dirname(os.path.abspath(bench.__file__))
    todo, seen = ["paper_2510_20929_amd/csrc/kernels/fused_lds.hip"], set()
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        with open(os.path.join(root, f)) as fh:
            for inc in re.findall(r'#include "([^"]+)"', fh.read()):
                todo.append(os.path.normpath(os.path.join(os.path.dirname(f), inc)))
    missing = seen - set(bench.KERNEL_SOURCES)
    assert missing <= {"paper_2510_20929_amd/csrc/kernels/launch.hpp"}, missing
