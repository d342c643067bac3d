"""The persistent integrator's queue: waves begin with the item of their own
number, take four, two or one items at a time by what is left, and waves
beyond the resident ones begin from the counter.  On both sides of each line
every operator is bitwise that of the plain integrator at the same slicing,
whose queue-free grid has a wave for every item."""
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

WAVE = 64       # intervals of an item at one lane per interval
RESIDENT = 2048  # waves of the default grid


@pytest.mark.parametrize("waves_per_simd", [0, 1, 4])
@pytest.mark.parametrize("items", [1, 2047, 2048, 2049, 4 * 2048 + 1, 8 * 2048, 8 * 2048 + 3,
                                   20 * 2048 + 5])
def test_every_item_is_taken_once(items, waves_per_simd):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    print(f"[gpu] work queue items={items} waves_per_simd={waves_per_simd}", flush=True)
    # two simulations, spin-1/2 and spin-1, that share the items unevenly; the
    # last item of each is partly filled
    first = max(1, items // 3)
    rest = max(1, items - first)
    probs = [W.spin_half_rabi(WAVE * first - 5, 2), W.spin_one_sensing(WAVE * rest - 7, 2)]
    plan = native.BatchPlan(probs, slices_spin_half=1, slices_spin_one=1,
                            waves_per_simd=waves_per_simd)
    bufs = plan.allocate(store_u=True)
    bufs["U"].fill_(float("nan"))
    for _ in range(2):
        plan.integrate(bufs)
    torch.cuda.synchronize()
    off = 0
    for p in probs:
        n = p.n_samples * p.dim * p.dim
        ref = torch.empty((p.n_samples, p.dim, p.dim), dtype=torch.complex128, device="cuda")
        native.integrate(p, native.device_params(p), ref, launch=(1, 256))
        assert torch.equal(torch.view_as_real(bufs["U"].view(-1).view(torch.complex128)[off:off + n]),
                           torch.view_as_real(ref.view(-1)))
        off += n
    plan.close()
