"""Short single-sequence scans: up to four tiles of 256 operators are scanned
in one workgroup, more of them by two launches.  Both sides of every tile
edge give bitwise the states of the batch plan's segmented scan and, within
rounding, those of the oracle's sequential product; one captured launch
replays them."""
import numpy as np
import pytest

from paper_2204_05586_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [256, 257, 300, 511, 512, 513, 768, 769, 1023, 1024, 1025])
@pytest.mark.parametrize("N", [2, 3])
def test_short_scan_equals_batch_scan_and_oracle(oracle, N, K):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_05586_amd import native
    print(f"[gpu] short scan N={N} K={K}", flush=True)
    prob = (W.spin_half_rabi if N == 2 else W.spin_one_sensing)(K, 10)
    U = torch.empty((K, N, N), dtype=torch.complex128, device="cuda")
    native.integrate(prob, None, U)
    ws = native.alloc_workspace(native.propagate_workspace_size(N - 1, K))
    start = native.device_state(prob.psi0)
    psi = torch.empty((K, N), dtype=torch.complex128, device="cuda")
    fin = torch.empty((N,), dtype=torch.complex128, device="cuda")
    native.propagate(N - 1, U, start, psi, fin, ws)
    plan = native.BatchPlan([prob])
    bufs = plan.allocate(store_u=True)
    bufs["U"].copy_(U.view(-1))
    plan.propagate(bufs)
    torch.cuda.synchronize()
    assert torch.equal(psi.view(-1), bufs["psi"])
    assert torch.equal(fin, bufs["psi_final"])
    plan.close()
    ref_psi, ref_fin = oracle.states(U.cpu().numpy(), prob.psi0)
    d = max(np.max(np.abs(psi.cpu().numpy() - ref_psi)), np.max(np.abs(fin.cpu().numpy() - ref_fin)))
    # at most 4 N rounding errors of 2^-53 per product on either side
    assert d < 2 * K * 4 * N * 2.0 ** -53

    g = torch.cuda.CUDAGraph()
    out = torch.empty_like(psi)
    with torch.cuda.graph(g):
        native.propagate(N - 1, U, start, out, None, ws)
    for _ in range(3):
        out.zero_()
        g.replay()
        native.propagate(N - 1, U, start, psi, fin, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, psi)
