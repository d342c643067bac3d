"""The adjoint's closed-form exponential derivatives on both sides of every
change of form (short series, long series, tangent squarings) and its
shared phases (a cosine and sine of one phase, and pairs that differ in one
respect only) against the oracle's adjoint."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

K, L = 67, 3


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    native.lib()
    return torch


def _terms(pair, span):
    """Four parameterised terms: a pair on x and y and another beside it.
    pair says how the second of each differs from the first, if at all."""
    T = W.Term
    if pair == "segments":
        a = dict(f=1.1, n_seg=5, seg_t0=0.1 * span, seg_len=0.21 * span, seg_a_slot=0,
                 seg_phi_slot=5)
        return [T(W.PWC_COS, W.X, **a), T(W.PWC_SIN, W.Y, **a),
                T(W.PWC_SIN, W.X, **{**a, "seg_len": 0.2 * span}),
                T(W.PWC, W.Y, n_seg=5, seg_t0=0.0, seg_len=0.2 * span, seg_a_slot=10)]
    a = dict(a_slot=0, f_slot=1, phi_slot=2, t_on=0.2 * span, t_off=0.9 * span)
    b = {"same": {}, "window": {"t_off": 0.7 * span}, "phase": {"phi_slot": 3},
         "frequency": {"f_slot": 4}}[pair]
    return [T(W.COS, W.X, **a), T(W.SIN, W.Y, **{**a, **b}), T(W.SIN, W.X, **{**a, "a_slot": 5}),
            T(W.CONST, W.Y, a_slot=6)]


# Angles of a fine step: below 2^-6, between it and 1, above 1 (where the
# squarings run, as they do at tau = 6 from 1e-6 on).  A gradient entry sums
# some 2 K L = 400 products of order 1, each rounded a few dozen times.
@pytest.mark.parametrize("pair", ["same", "window", "phase", "frequency", "segments"])
@pytest.mark.parametrize("tau", [6, 24, 28])
def test_gradients_match_the_oracle(dev, oracle, pair, tau):
    from paper_2204_05586_amd import native
    probs = []
    for spin in (1, 2):
        for j, angle in enumerate((0.008, 0.05, 0.5, 2.5)):
            rng = np.random.default_rng(1000 * spin + 10 * tau + j)
            dt = 2 * angle * L / (2 * np.pi)   # fields of order 1 Hz, two exponentials a step
            params = rng.uniform(0.3, 1.0, 15)
            terms = _terms(pair, K * dt) + [W.Term(W.CONST, W.Z, a=0.3)]
            if spin == 2:
                terms.append(W.Term(W.CONST, W.Q, a=0.4))
            probs.append(W.Problem(spin, terms, 0.0, dt, K, L, tau if spin == 2 else 0,
                                   bool(j % 2), params=params,
                                   psi0=W.random_state(spin + 1, rng)))
    plan = native.AdjointPlan(probs, 1)
    bufs = plan.allocate()
    print(f"[gpu] adjoint series tau={tau} pair={pair}", flush=True)
    plan.run(bufs)
    dev.cuda.synchronize()
    for i, p in enumerate(probs):
        loss, grad = oracle.adjoint_population(p, 1)
        got = plan.grad_of(bufs, i).cpu().numpy()
        assert abs(float(bufs["loss"][i]) - loss) <= 1e-12, i
        assert np.max(np.abs(got - grad)) <= 1e-11 * max(np.max(np.abs(grad)), 1.0), i
    plan.close()


# A few short simulations leave the device idle, so the backward pass gives an
# interval as many lanes as it has fine steps for, up to 16: one step a lane,
# uneven shares, and interval counts that do not fill a wave.  The mixed list
# takes the lanes of its shortest.
@pytest.mark.parametrize("fine", [(1,), (2,), (3,), (5,), (16,), (17,), (33, 70)])
@pytest.mark.parametrize("samples", [1, 3, 16, 67])
def test_interval_split_over_lanes(dev, oracle, fine, samples):
    from paper_2204_05586_amd import native
    probs = []
    for spin in (1, 2):
        for j, L in enumerate(fine):
            rng = np.random.default_rng(100 * spin + 10 * samples + j)
            dt = 0.01 * L
            terms = _terms("segments", samples * dt) + [W.Term(W.CONST, W.Z, a=1.2)]
            probs.append(W.Problem(spin, terms, 0.0, dt, samples, L, 28 if spin == 2 else 0,
                                   bool((j + samples) % 2), params=rng.uniform(0.3, 1.0, 15),
                                   psi0=W.random_state(spin + 1, rng)))
    plan = native.AdjointPlan(probs, 1)
    bufs = plan.allocate()
    print(f"[gpu] adjoint lanes L={fine} K={samples}", flush=True)
    plan.run(bufs)
    dev.cuda.synchronize()
    for i, p in enumerate(probs):
        loss, grad = oracle.adjoint_population(p, 1)
        assert abs(float(bufs["loss"][i]) - loss) <= 1e-12, i
        got = plan.grad_of(bufs, i).cpu().numpy()
        assert np.max(np.abs(got - grad)) <= 1e-11 * max(np.max(np.abs(grad)), 1.0), i
    plan.close()
