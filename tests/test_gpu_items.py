"""Per-item kernels (a thread per bus, branch or slot) at the batch sizes where
their work is laid out differently: every case against the same case alone;
the Jacobian's zero padding; the mismatch with and without room in LDS for
every bus's voltage."""
import numpy as np
import pytest

import gridgen
from gpu_helpers import Staged, dev, grid, log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# 8, 63: whole cases per XCD (63 leaves one turn empty); 9: spread over them
@pytest.mark.parametrize("Bn", [1, 8, 9, 63])
@pytest.mark.parametrize("n", [2, 70, 301])
def test_cases_match_alone(n, Bn):
    from paper_1811_02512_amd import binding as B

    g = grid(n, 5)
    s = Staged(g)
    info = s.info
    log(f"[items] n={n} B={Bn}")
    rng = np.random.default_rng(1)
    r, x, b = (dev(v * rng.uniform(0.9, 1.1, (Bn, g.m))) for v in (g.r, g.x, g.b))
    Vm, Va = dev(rng.uniform(0.9, 1.1, (Bn, n))), dev(rng.uniform(-0.5, 0.5, (Bn, n)))
    new = lambda k, w: torch.full((k, w), float("nan"), dtype=torch.float64, device="cuda")

    def run(c0, k):
        rr, xx, bb, vm, va = (t[c0:c0 + k].contiguous() for t in (r, x, b, Vm, Va))
        y = s.sym.build_ybus(rr, xx, bb)
        mat = new(k, info.fd_mat_doubles)
        B.pf_fdpf_matrices(s.sym.h, k, rr, xx, bb, g.m, s.type, 0, mat, info.fd_mat_doubles)
        vals = new(k, info.vals_doubles)
        B.pf_jacobian(s.sym.h, k, y, y.shape[1], s.type, 0, vm, va, n, vals, info.vals_doubles, 1)
        flows = torch.stack(s.sym.branch_flows(rr, xx, bb, vm, va), 1)
        M = info.fd_mat_doubles // 2
        used = (info.nn + 7) // 8 * 8 + 2 * info.nnz_l
        return y, mat.view(k, 2, M)[:, :, :used], vals, flows

    whole = run(0, Bn)
    assert not any(torch.isnan(t).any() for t in whole)
    assert (whole[2][:, 4 * info.nn:info.lu_offset] == 0).all()
    for c in sorted({0, Bn // 2, Bn - 1}):
        for got, want in zip(whole, run(c, 1)):  # the same operations: the same bits
            assert torch.equal(got[c], want[0])


# voltages of 10,176 buses fit in LDS; 257, 600: two and three per thread
@pytest.mark.parametrize("n", [2, 257, 600, 10176, 10177])
def test_mismatch_matches_numpy(n):
    from paper_1811_02512_amd import binding as B

    g = grid(n, 7)
    s = Staged(g)
    log(f"[items] mismatch n={n}")
    rng = np.random.default_rng(2)
    vm, va = rng.uniform(0.9, 1.1, n), rng.uniform(-0.5, 0.5, n)
    nn = s.info.nn
    rhs = torch.empty(1, 2 * nn, dtype=torch.float64, device="cuda")
    norm = torch.empty(1, dtype=torch.float64, device="cuda")
    PQ = torch.empty(1, 2 * n, dtype=torch.float64, device="cuda")
    B.pf_mismatch(s.sym.h, 1, s.yval, 0, s.type, 0, s.Psp, s.Qsp, 0, dev(vm), dev(va), n, rhs,
                  2 * nn, norm, PQ)
    y = 1.0 / (g.r + 1j * g.x)
    V = vm * np.exp(1j * va)
    f, t = g.f, g.t
    I = np.zeros(n, complex)
    np.add.at(I, f, (y + 0.5j * g.b) * V[f] - y * V[t])
    np.add.at(I, t, (y + 0.5j * g.b) * V[t] - y * V[f])
    S = V * np.conj(I)
    mag = np.zeros(n)
    np.add.at(mag, f, 2 * np.abs(y))
    np.add.at(mag, t, 2 * np.abs(y))
    # a row's terms are at most 1.21 * 2 |y| each way; fewer than 64 roundings
    tol = 64 * np.finfo(float).eps * 1.21 * (mag.max() + 1.0)
    got = PQ.cpu().numpy().reshape(n, 2)
    np.testing.assert_allclose(got[:, 0], S.real, rtol=0, atol=tol)
    np.testing.assert_allclose(got[:, 1], S.imag, rtol=0, atol=tol)
    dP, dQ = S.real - g.Psp, np.where(g.bus_type == gridgen.BUS_PV, 0.0, S.imag - g.Qsp)
    F = np.delete(np.stack([dP, dQ], 1), 0, 0)
    assert abs(norm.item() - np.abs(F).max()) <= tol
    perm = s.sym.export()["perm"]
    np.testing.assert_allclose(rhs.cpu().numpy().reshape(nn, 2), F[perm - 1], rtol=0, atol=tol)
