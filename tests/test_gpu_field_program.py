"""The interpreter's walk over a field program, both nodes of a fine step at
once and constant components apart, against the same program compiled into
the integrator (bit for bit) and the oracle."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

T = W.Term
K, DT = 41, 1e-5

# Lists on each side of the split: only constant components, none, constants
# of one component around its varying terms, a constant that a window makes
# varying, and no term at all.  Windows end between the two nodes of a step
# (node offsets 0.211 and 0.789 of the step) and on an output time.
LISTS = {
    "empty": [],
    "constant": [T(W.CONST, W.Z, a=2e3), T(W.CONST, W.Q, a=30.0), T(W.CONST, W.Z, a_slot=0),
                 T(W.CONST, W.X, a=100.0)],
    "varying": [T(W.COS, W.X, a=150.0, f=2e3), T(W.SIN, W.Y, a_slot=0, f=1e3, phi=0.3),
                T(W.COS, W.Z, a=500.0, f_slot=1)],
    "around": [T(W.CONST, W.X, a=20.0), T(W.CONST, W.Z, a=2e3), T(W.COS, W.X, a=90.0, f=2e3),
               T(W.CONST, W.X, a_slot=0), T(W.CONST, W.Z, a=-40.0), T(W.SIN, W.X, a=7.0, f=9e3)],
    "window": [T(W.CONST, W.Z, a=1e3), T(W.CONST, W.Z, a=3e2, t_on=7.5 * DT, t_off=20.5 * DT),
               T(W.COS, W.X, a=200.0, f=1e3, t_on=3 * DT, t_off=30.25 * DT),
               T(W.CONST, W.Y, a=50.0, t_off=15.5 * DT),
               T(W.PWC, W.Y, n_seg=5, seg_t0=-DT, seg_len=8.5 * DT, seg_a_slot=2)],
}


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    native.lib()
    return torch


@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("terms", sorted(LISTS))
def test_interpreter_is_the_compiled_program(dev, oracle, terms, spin):
    from paper_2204_05586_amd import native
    program = [t for t in LISTS[terms] if spin == 2 or t.comp != W.Q]
    sampler = native.Sampler.for_terms(program)
    for method in (W.CF4, W.MIDPOINT, W.HEUN):
        for fine in (1, 3):
            prob = W.Problem(spin, program, 0.0, DT, K, fine, 28 if spin == 2 else 0, True,
                             params=np.array([120.0, 800.0, 5.0, -60.0, 80.0, 0.0, 33.0]),
                             method=method)
            print(f"[gpu] field program {terms} L={fine} method={method} spin={spin}", flush=True)
            params = native.device_params(prob)
            shape = (K, prob.dim, prob.dim)
            U = dev.empty(shape, dtype=dev.complex128, device="cuda")
            V = dev.empty(shape, dtype=dev.complex128, device="cuda")
            native.integrate(prob, params, U)
            sampler.integrate(prob.replace(terms=[]), params, V)
            dev.cuda.synchronize()
            assert dev.equal(U, V)
            # angles up to 0.1 a step and 6 steps' roundings, phases below 1e2
            assert np.max(np.abs(U.cpu().numpy() - oracle.operators(prob))) <= 2e-14
    sampler.close()


# Phases 2 pi f t + phi around 2^30, where the sines change their reduction:
# below, across it within a fine step (f = 2e9 Hz, 25 rad between nodes), and
# beyond; and at the 1.5e6 rad of a 0.35 s sensing run.
@pytest.mark.parametrize("t_start, f", [(0.35, 7e5), (0.08, 2e9), (0.0854459, 2e9), (0.09, 2e9),
                                        (1e3, 7e5)])
def test_sines_of_large_phases(dev, oracle, t_start, f):
    from paper_2204_05586_amd import native
    for spin in (1, 2):
        program = [T(W.COS, W.X, a=3e3, f=f), T(W.SIN, W.Y, a=1e3, f=f, phi=1.0),
                   T(W.CONST, W.Z, a=2e3)]
        prob = W.Problem(spin, program, t_start, 2e-7, K, 3, 28 if spin == 2 else 0, True)
        U = dev.empty((K, prob.dim, prob.dim), dtype=dev.complex128, device="cuda")
        print(f"[gpu] phases from {2 * np.pi * f * t_start:.4g} spin={spin}", flush=True)
        native.integrate(prob, None, U)
        dev.cuda.synchronize()
        # the phases round alike on both sides; angles of 1e-3 a step
        assert np.max(np.abs(U.cpu().numpy() - oracle.operators(prob))) <= 5e-15
