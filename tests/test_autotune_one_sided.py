"""The launch-shape tuner times only workloads that the shapes decide: the one-sided kernel's clusters, below
4096 and above 2^20 particles."""
import inspect
import os
import re

import numpy as np
import pytest

from paper_1003_3896_amd import autotune, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bounds_are_those_of_the_kernels():
    src = open(os.path.join(ROOT, "paper_1003_3896_amd", "csrc", "nb_internal.h")).read()
    m = re.search(r"constexpr int kSymMin = (\d+), kSymMax = 1 << (\d+);", src)
    assert (autotune.SYM_MIN, autotune.SYM_MAX) == (int(m.group(1)), 1 << int(m.group(2)))


def test_tuned_workloads_run_the_one_sided_kernel_alone():
    for ncl in inspect.signature(autotune.tune_all).parameters["classes"].default:
        b = autotune.representative(ncl)
        sizes = autotune.one_sided(b.offsets)
        assert len(sizes) == b.B
        assert {autotune.size_class(int(n)) for n in (sizes.min(), sizes.max())} == {ncl}


@pytest.mark.parametrize("sizes", [(4096,), (1 << 20,), (5000, 65536)])
def test_sweep_refuses_what_the_shapes_do_not_decide(sizes):
    b = inputs.concat([inputs.single(np.zeros((n, 3)), np.zeros((n, 3)), np.ones(n), 1e-3, False) for n in sizes])
    with pytest.raises(ValueError, match="launch shapes"):
        autotune.sweep(b, "fp32c")
