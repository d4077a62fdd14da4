"""The benchmark's account of launches that passes share, on the CPU."""
import os
import re

import pytest

import bench
from paper_1912_12607_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_shared_launch_has_its_work():
    names = re.findall(r'"([a-z0-9_]+trio_kernel)"', open(os.path.join(ROOT, "paper_1912_12607_amd", "csrc", "profile.hip")).read())
    assert set(names) == set(bench.SHARED_KERNELS)


@pytest.mark.parametrize("kernel", bench.SHARED_KERNELS)
def test_passes_of_a_shared_launch(kernel):
    L = inputs.CONFIGS[1][0]
    alg = bench.pass_algorithmic(L, 32)
    others = [kernel, "quantize_batch_kernel", "dsgc_sweep_kernel"]

    def passes(*names):
        return [sum(alg[p][0] for p in names), sum(alg[p][1] for p in names), "mfma", 1]
    assert bench.shared_work(kernel, L, 32, others, False) == passes("fwd", "bwd_data", "bwd_weight")
    assert bench.shared_work(kernel, L, 32, others, True) == passes("bwd_data", "bwd_weight")
    # the forward pass ran ahead, in a launch of its own
    assert bench.shared_work(kernel, L, 32, others + ["band_kernel"], False) == passes("bwd_data", "bwd_weight")
