"""The integrator's exponentials on both sides of every change of form
(short series, long series, tau residual squarings) against the oracle,
which squares always: one exponential per interval, the generator of every
interval drawn on its own."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

# Sizes of the angle vector around the series' bounds (eigenvalues 2^-6 and 1)
# and beyond both; K covers a whole wave and a remainder.
SIZES = [0.0, 1e-9, 3e-4, 0.0135, 0.0155, 0.0175, 0.2, 0.8, 0.95, 1.2, 3.0]
K = 67


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    native.lib()
    return torch


def _problem(spin, comps, size, tau, seed):
    """K intervals of one midpoint step of length 1, each with its own
    constant field over the given components: angles of norm `size`, every
    third without the transverse components, every fifth without the rest."""
    rng = np.random.default_rng(seed)
    a = rng.normal(size=(len(comps), K))
    transverse = np.array([c in (W.X, W.Y) for c in comps])
    a[np.ix_(transverse, np.arange(0, K, 3))] = 0.0
    a[np.ix_(~transverse, np.arange(1, K, 5))] = 0.0
    norm = np.linalg.norm(a, axis=0)  # 0 where both were taken out: no field
    a *= size / (2 * np.pi) / np.where(norm > 0.0, norm, 1.0)
    terms = [W.Term(W.PWC, c, n_seg=K, seg_t0=0.0, seg_len=1.0, seg_a_slot=i * K)
             for i, c in enumerate(comps)]
    return W.Problem(spin, terms, 0.0, 1.0, K, 1, tau, False, params=a.ravel(),
                     method=W.MIDPOINT)


# Both sides exponentiate to a few roundings of the angles: the squarings
# within 10 tau of them (11e-15 |theta| at tau = 50) and the series within 20.
# Where the series stands for tau squarings the splitting differs from it by
# at most 2^-54 |theta|.  The series' operators are also unitary to rounding.
@pytest.mark.parametrize("tau", [0, 1, 5, 20, 24, 28, 50])
@pytest.mark.parametrize("basis", ["half", "one", "full"])
def test_exponentials_match_the_oracle(dev, oracle, basis, tau):
    import torch
    from paper_2204_05586_amd import native
    spin = 1 if basis == "half" else 2
    comps = {"half": [W.X, W.Y, W.Z], "one": [W.X, W.Y, W.Z, W.Q],
             "full": [W.X, W.Y, W.Z, W.Q, W.U1, W.U2, W.V1, W.V2]}[basis]
    for j, size in enumerate(SIZES):
        prob = _problem(spin, comps, size, tau if spin == 2 else 0, seed=100 * tau + j)
        print(f"[gpu] exponential {basis} tau={tau} size={size}", flush=True)
        U = torch.empty((K, prob.dim, prob.dim), dtype=torch.complex128, device="cuda")
        native.integrate(prob, native.device_params(prob), U)
        torch.cuda.synchronize()
        got, ref = U.cpu().numpy(), oracle.operators(prob)
        off = np.max(np.abs(got - ref))
        assert off <= 1e-15 + 2e-14 * size, (basis, tau, size, off)
