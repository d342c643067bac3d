"""solve() and evaluate() upload their inputs from the host, so they are
refused under stream capture, and leave the capture usable."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want_spin", [False, True])
@pytest.mark.parametrize("params", [[], [7e5, 1e3]])
def test_evaluate_is_refused_under_capture(params, want_spin):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd.simulator import Simulator
    print(f"[gpu] evaluate under capture params={len(params)} spin={want_spin}", flush=True)
    terms = ([W.Term(W.COS, W.X, a_slot=1, f_slot=0), W.Term(W.CONST, W.Z, a_slot=0)] if params
             else W.neural_pulse_terms())
    sim = Simulator(terms, spin=1)
    psi0 = np.array([1, 0, 0], dtype=complex)

    def evaluate():
        return sim.evaluate(psi0, 0.0, 5e-4, 5e-8, 5e-7, params=params, keep_operators=False,
                            want_spin=want_spin)

    before = evaluate().state.clone()
    x = torch.zeros(256, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        with pytest.raises(RuntimeError):
            evaluate()
    for n in range(1, 4):
        graph.replay()
        assert torch.equal(evaluate().state, before)
        torch.cuda.synchronize()
        assert torch.equal(x, torch.full_like(x, float(n)))
