"""Evaluations queued one behind another without waiting, on the current and
on another stream: every one keeps the parameters and initial state it was
called with (they go to the device by an asynchronous copy)."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side_stream", [False, True])
@pytest.mark.parametrize("spin, specialize", [(0.5, False), (1, True)])
def test_queued_evaluations_keep_their_inputs(side_stream, spin, specialize):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd.simulator import Simulator
    terms = [W.Term(W.COS, W.X, a_slot=1, f_slot=0), W.Term(W.CONST, W.Z, a_slot=0)]
    sim = Simulator(terms, spin=spin, specialize=specialize)
    rng = np.random.default_rng(4)
    calls = [(rng.uniform([500.0, 100.0], [2000.0, 400.0]),
              W.random_state(2 if spin == 0.5 else 3, rng)) for _ in range(40)]
    stream = torch.cuda.Stream() if side_stream else None

    def evaluate(params, psi0):
        # long enough that the queue runs ahead of the device
        return sim.evaluate(psi0, 0.0, 3e-1, 1e-6, 1e-5, params=params, keep_operators=False,
                            stream=stream)

    print(f"[gpu] queued evaluations spin={spin} side_stream={side_stream}", flush=True)
    queued = [evaluate(p, v) for p, v in calls]
    torch.cuda.synchronize()
    for r, (p, v) in zip(queued, calls):
        alone = evaluate(p, v)
        torch.cuda.synchronize()
        assert torch.equal(r.state, alone.state) and torch.equal(r.state_final, alone.state_final)
        assert np.array_equal(r.state[0].cpu().numpy(), v)
