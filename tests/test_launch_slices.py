"""Lane-slices of a single simulation at shapes where they decide: SIMDs just
filled by one or two waves of one lane per interval (256 CUs of 4 SIMDs).  The
slices listed are within 9 % of the fastest measured, and the ones left
out are further behind.  No GPU is needed: 256 CUs are assumed without one."""
import pytest

from paper_2204_05586_amd import native, workloads as W


@pytest.mark.parametrize("spin, K, L, good", [
    (1, 100_000, 20, (2, 4)),     # 1, 2, 4, 8 slices: 37, 33, 31, 38 us
    (1, 128_000, 100, (2, 4)),    # 1, 2, 4: 106, 93, 89 us
    (2, 128_000, 100, (2, 4)),    # 1, 2, 4: 214, 194, 185 us
    (2, 50_021, 20, (2,)),        # 1, 2: 34, 28 us
    (2, 200_000, 10, (2,)),
    (2, 1_000_000, 10, (1,)),     # 1, 2: 159, 172 us
    (1, 300_001, 20, (1, 2)),
])
def test_planned_slices(spin, K, L, good):
    prob = W.spin_half_rabi(K, L) if spin == 1 else W.spin_one_sensing(K, L)
    assert native.plan_launch(prob)[0] in good
