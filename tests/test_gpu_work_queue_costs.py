"""The persistent integrator's queue with items of unlike cost: the costly
items of one simulation among many cheap ones go to as many waves as there
are, whichever place they have in the queue, and every operator is still
bitwise that of the plain integrator."""
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

WAVE = 64        # intervals of an item at one lane per interval
RESIDENT = 2048  # waves of the default grid
COSTLY = W.spin_one_sensing(WAVE * 96 - 5, 3000)     # 96 items, some 5 ms each
CHEAP = W.spin_one_sensing(WAVE * 6 * RESIDENT, 2)   # 12,288 items, some 5 us each


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    native.lib()
    return torch


def _plan(problems):
    from paper_2204_05586_amd import native
    plan = native.BatchPlan(problems, slices_spin_one=1)
    bufs = plan.allocate(store_u=True)
    bufs["U"].fill_(float("nan"))
    return plan, bufs


def _milliseconds(dev, plan, bufs):
    times = []
    for _ in range(3):
        a, b = (dev.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        plan.integrate(bufs)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("place", [0, 1, 2, 4])
def test_costly_items_spread_over_the_waves(dev, place):
    from paper_2204_05586_amd import native
    print(f"[gpu] costly items at place {place}", flush=True)
    plan, bufs = _plan([COSTLY])
    alone = _milliseconds(dev, plan, bufs)
    plan.close()
    plan, bufs = _plan([CHEAP] * 4)
    cheap = _milliseconds(dev, plan, bufs)
    plan.close()
    problems = [CHEAP] * 4
    problems.insert(place, COSTLY)
    plan, bufs = _plan(problems)
    took = _milliseconds(dev, plan, bufs)
    # a wave holds at most two items at a time near them, one of which it may
    # reach after a costly one: under twice a costly item's time and the rest,
    # where four in a row are four times it
    print(f"[gpu] alone {alone:.2f} cheap {cheap:.2f} together {took:.2f} ms", flush=True)
    assert took <= 2.0 * alone + cheap
    off = 0
    for p in problems:
        n = p.n_samples * 9
        if p is COSTLY:
            ref = dev.empty((p.n_samples, 3, 3), dtype=dev.complex128, device="cuda")
            native.integrate(p, native.device_params(p), ref, launch=(1, 256))
            got = bufs["U"][off:off + n]
            assert dev.equal(dev.view_as_real(got), dev.view_as_real(ref.view(-1)))
        off += n
    assert not bool(dev.isnan(dev.view_as_real(bufs["U"])).any())
    plan.close()
