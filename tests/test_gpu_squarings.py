"""Spin-1 exponentials by the squarings, where the closed form is not the
scheme's exponential to rounding: small tau and large angles, compiled fields
(which below tau = 16 have the squarings in the integrator's loop, from there
on as a call) against the interpreter bit for bit and against the oracle."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

T = W.Term
K = 67  # a second, partly filled wave


@pytest.fixture(scope="module")
def dev():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    native.lib()
    return torch


@pytest.mark.parametrize("method", [W.CF4, W.MIDPOINT, W.HEUN])
@pytest.mark.parametrize("tau", [0, 1, 8, 15, 16, 17, 28])
def test_squarings_of_compiled_fields(dev, oracle, tau, method):
    from paper_2204_05586_amd import native
    # a drive whose angles pass through zero, so that closed forms and
    # squarings meet within a wave; angles up to 0.4 and 3 a fine step
    program = [T(W.COS, W.X, a_slot=0, f=3e3), T(W.SIN, W.Y, a=40.0, f=1e3, phi=0.2),
               T(W.CONST, W.Z, a=3e3), T(W.CONST, W.Q, a=25.0)]
    sampler = native.Sampler.for_terms(program)
    for dt_out, fine in ((2e-5, 4), (2e-3, 2)):
        prob = W.Problem(2, program, 0.0, dt_out, K, fine, tau, True, params=np.array([400.0]),
                         method=method)
        print(f"[gpu] squarings tau={tau} method={method} dt={dt_out}", flush=True)
        params = native.device_params(prob)
        U = dev.empty((K, 3, 3), dtype=dev.complex128, device="cuda")
        V = dev.empty_like(U)
        native.integrate(prob, params, U)
        sampler.integrate(prob.replace(terms=[]), params, V)
        dev.cuda.synchronize()
        assert dev.equal(U, V)
        # at most 8 exponentials of angles up to 6 rad with 30 roundings each,
        # phases below 1e4 rad: 8 (30 + 6) 2^-53 and the phases' 1e4 2^-53 a step
        assert np.max(np.abs(U.cpu().numpy() - oracle.operators(prob))) <= 1e-11
    sampler.close()
