"""The flops that the benchmark's roofline counts for a spin-1 fine step as
executed, on both sides of the change from squarings to the closed form."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("exponentials", [1, 2])
def test_executed_flops_per_fine_step(exponentials):
    product = 2 * 9 * 8  # two columns of three entries, three complex multiply-adds each
    for tau in (0, 8, 15):
        assert (bench.spin_one_executed_flops_per_fine_step(tau, exponentials)
                == exponentials * (96 * tau + product))
    for tau in (16, 20, 24, 28):
        assert (bench.spin_one_executed_flops_per_fine_step(tau, exponentials)
                == exponentials * (20 + 22 + 71 + product))
