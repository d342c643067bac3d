"""evaluate() with a stream of its own: the memory it takes may be that of a
tensor just dropped, which work queued on the current stream still reads, and
the scratch it drops may go to the next evaluation while its own stream still
uses it."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

K, N = 30000, 3
TERMS = [W.Term(W.COS, W.X, a_slot=1, f_slot=0), W.Term(W.CONST, W.Z, a_slot=0)]


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd.simulator import Simulator
    sim = Simulator(TERMS, spin=1)

    def evaluate(call, stream=None, **kw):
        params, psi0 = call
        return sim.evaluate(psi0, 0.0, K * 5e-7, 5e-8, 5e-7, params=params, stream=stream, **kw)

    rng = np.random.default_rng(11)
    calls = [(rng.uniform([690e3, 500.0], [710e3, 2000.0]), W.random_state(N, rng))
             for _ in range(24)]
    return torch, evaluate, calls


@pytest.mark.parametrize("want_spin", [False, True])
def test_queued_readers_of_a_dropped_tensor_see_it_whole(dev, want_spin):
    torch, evaluate, calls = dev
    side = torch.cuda.Stream()
    print(f"[gpu] dropped tensors, evaluate on a side stream, spin={want_spin}", flush=True)
    # blocks of the sizes evaluate() takes (states, operators, spin projections)
    shapes = [((K, N), torch.complex128), ((K, N, N), torch.complex128), ((K, 3), torch.float64)]
    ones = [torch.ones(s, dtype=d, device="cuda") for s, d in shapes]
    for call in calls[:6]:
        work = [o * 2.0 for o in ones]
        torch.cuda.synchronize()
        # some milliseconds of queued work before the reads
        busy = torch.ones(1 << 26, device="cuda")
        for _ in range(60):
            busy.mul_(1.0)
        copies = [w.clone() for w in work]
        del work
        r = evaluate(call, side, keep_operators=True, want_spin=want_spin)
        torch.cuda.synchronize()
        for c in copies:
            assert torch.equal(c, torch.full_like(c, 2.0))
        alone = evaluate(call, keep_operators=True, want_spin=want_spin)
        assert torch.equal(r.state, alone.state) and torch.equal(r.state_final, alone.state_final)


@pytest.mark.parametrize("want_spin", [False, True])
def test_evaluations_on_two_streams_share_no_scratch(dev, want_spin):
    torch, evaluate, calls = dev
    sides = [torch.cuda.Stream(), torch.cuda.Stream()]
    print(f"[gpu] alternating side streams, spin={want_spin}", flush=True)
    queued = [evaluate(c, sides[i % 2], keep_operators=False, want_spin=want_spin)
              for i, c in enumerate(calls)]
    torch.cuda.synchronize()
    for r, c in zip(queued, calls):
        alone = evaluate(c, keep_operators=False, want_spin=want_spin)
        assert torch.equal(r.state, alone.state) and torch.equal(r.state_final, alone.state_final)
        if want_spin:
            assert torch.equal(r.spin, alone.spin)


def test_a_stream_known_by_its_handle(dev):
    """A stream object needs only its handle (``cuda_stream``)."""
    torch, evaluate, calls = dev

    class Handle:
        def __init__(self, stream):
            self.cuda_stream = stream.cuda_stream

    side = torch.cuda.Stream()
    r = evaluate(calls[0], Handle(side), keep_operators=False)
    side.synchronize()
    alone = evaluate(calls[0], keep_operators=False)
    assert torch.equal(r.state, alone.state) and torch.equal(r.state_final, alone.state_final)
