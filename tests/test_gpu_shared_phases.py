"""Generated field programs in which a term takes the window, segments, sines
and cosines of the term before it: pairs of one phase, windowed and in
segments, runs of three, and pairs that differ in one respect only, bit for
bit against the interpreter (which shares nothing) and against the oracle."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu

T = W.Term
K, DT = 41, 1e-5
# windows that open and close between the nodes of a fine step (offsets 0.211
# and 0.789 of it) for 1 and 3 steps, before the first and after the last
# interval, and the empty one
WINDOW = dict(t_on=3.5 * DT, t_off=30.5 * DT)
WAVE = dict(a_slot=0, f_slot=1, phi_slot=2)
SEGMENTS = dict(f=900.0, n_seg=5, seg_t0=-DT, seg_len=8.5 * DT, seg_a_slot=3, seg_phi_slot=8)
NEVER = dict(t_on=5 * DT, t_off=5 * DT)


def _pair(first, **differs):
    return [T(W.COS, W.X, **first), T(W.SIN, W.Y, **{**first, **differs})]


PROGRAMS = {
    "pair": _pair(WAVE),
    "windowed": _pair({**WAVE, **WINDOW}),
    "early": _pair({**WAVE, "t_off": 2.5 * DT}),
    "late": _pair({**WAVE, "t_on": 38.5 * DT}),
    "other window": _pair({**WAVE, **WINDOW}, t_off=20.5 * DT),
    "one windowed": _pair(WAVE, **WINDOW),
    "other phase": _pair(WAVE, phi_slot=-1, phi=0.4),
    "other frequency": _pair(WAVE, f_slot=-1, f=800.0),
    "literals": _pair(dict(a=90.0, f=1e3, phi=0.3, **WINDOW)),
    "three": [T(W.COS, W.X, **WAVE, **WINDOW), T(W.COS, W.Y, **WAVE, **WINDOW),
              T(W.SIN, W.X, **{**WAVE, "a_slot": 2}, **WINDOW)],
    "between": [T(W.COS, W.X, **WAVE), T(W.CONST, W.Y, a=40.0, **WINDOW), T(W.SIN, W.Y, **WAVE)],
    "never between": [T(W.COS, W.X, **WAVE, **WINDOW), T(W.SIN, W.X, **WAVE, **NEVER),
                      T(W.SIN, W.Y, **WAVE, **WINDOW)],
    "segments": [T(W.PWC_COS, W.X, **SEGMENTS), T(W.PWC_SIN, W.Y, **SEGMENTS)],
    "segments, other amplitude": [T(W.PWC_COS, W.X, **SEGMENTS, **WINDOW),
                                  T(W.PWC_SIN, W.Y, **{**SEGMENTS, "seg_a_slot": 8}, **WINDOW)],
    "other segments": [T(W.PWC_COS, W.X, **SEGMENTS),
                       T(W.PWC_SIN, W.Y, **{**SEGMENTS, "seg_len": 7 * DT}),
                       T(W.PWC, W.X, n_seg=5, seg_t0=0.0, seg_len=9 * DT, seg_a_slot=3)],
}
PARAMS = np.array([120.0, 950.0, 0.7, 30.0, -60.0, 80.0, 0.0, 33.0, 0.1, 2.0, -1.0, 0.5, 3.0])


@pytest.mark.parametrize("spin", [1, 2])
@pytest.mark.parametrize("name", sorted(PROGRAMS))
def test_shared_phases(oracle, name, spin):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    program = PROGRAMS[name] + [T(W.CONST, W.Z, a=1e3)]
    sampler = native.Sampler.for_terms(program)
    for method in (W.CF4, W.MIDPOINT, W.HEUN):
        for fine in (1, 3):
            prob = W.Problem(spin, program, 0.0, DT, K, fine, 28 if spin == 2 else 0, True,
                             params=PARAMS, method=method)
            print(f"[gpu] shared phases {name} L={fine} method={method} spin={spin}", flush=True)
            params = native.device_params(prob)
            U = torch.empty((K, prob.dim, prob.dim), dtype=torch.complex128, device="cuda")
            V = torch.empty_like(U)
            native.integrate(prob, params, U)
            sampler.integrate(prob.replace(terms=[]), params, V)
            torch.cuda.synchronize()
            assert torch.equal(U, V)
            # angles up to 0.1 a step and 6 steps' roundings, phases below 1e2
            assert np.max(np.abs(U.cpu().numpy() - oracle.operators(prob))) <= 2e-14
    sampler.close()
