"""The fast decoupled kernel's four LDS layouts, each reached by the batch and
the LDS budget that call for it, and top cliques on both sides of the 64 nodes
that a wavefront's registers hold; against the CPU oracle."""
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


def _O():
    from oracle import oracle as O

    return O


# 1,200 buses, 64 threads: up to 16 workgroups per compute unit.  One case:
# everything apart.  1,290 cases (6 per unit of 256): apart leaves room for
# fewer of them; no tail: (e, f) in the workspace; a budget of exactly the
# (e, f) copy: x under it; 64 KB: the tail leaves x no room there.
@pytest.mark.parametrize("Bn,budget", [(1, 65536), (1290, 0), (1290, 16 * 1200), (1290, 65536)])
def test_layouts_match_oracle(Bn, budget):
    O = _O()
    g = grid(1200, 6)
    s = Staged(g)
    s.sym.set_launch(64, budget, 1)
    s.sym.upload()
    log(f"[fdpf layouts] B={Bn} budget={budget}: {s.sym.info.tail_nodes} tail nodes")
    P, Q = gridgen.scenario_injections(g, 3, seed=4)
    mat, st = s.sym.fdpf_factors(s.r, s.x, s.b, s.type)
    assert st.item() == 0
    pick = np.arange(Bn) % 3
    Vm = s.Vm0.repeat(Bn, 1).contiguous()
    Va = s.Va0.repeat(Bn, 1).contiguous()
    it, _, status, _ = s.sym.fdpf(s.yval[0], s.type, dev(P[pick]), dev(Q[pick]), Vm, Va, mat)
    assert status.abs().sum().item() == 0
    Vm0, Va0 = g.flat_start()
    osym, Y = O.Sym(g.n, g.f, g.t), O.grid_ybus(g)
    for c in range(min(3, Bn)):
        ref = osym.fdpf(Y, g, P[c], Q[c], Vm0, Va0)
        assert ref.status == 0 and it[c].item() == ref.iters
        np.testing.assert_allclose(Vm[c].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
        np.testing.assert_allclose(Va[c].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
        # the cases with the same inputs: the same operations in the same order
        assert torch.equal(Vm[c::3], Vm[c].expand_as(Vm[c::3]))
        assert torch.equal(Va[c::3], Va[c].expand_as(Va[c::3]))


def complete(n):
    """Every bus joined to every other: the filled graph is one clique."""
    f, t = np.triu_indices(n, 1)
    rng = np.random.default_rng(n)
    m = f.size
    kind = np.zeros(n, np.int8) + gridgen.BUS_PQ
    kind[0] = gridgen.BUS_SLACK
    kind[1:n // 3] = gridgen.BUS_PV
    return gridgen.Grid(
        n=n, f=f.astype(np.int32), t=t.astype(np.int32), r=rng.uniform(0.01, 0.03, m),
        x=rng.uniform(0.1, 0.3, m), b=rng.uniform(0.0, 0.02, m), bus_type=kind,
        vset=np.where(kind == gridgen.BUS_PQ, 1.0, 1.02), Pd=rng.uniform(0.5, 1.5, n),
        Qd=rng.uniform(0.1, 0.5, n), Pg=rng.uniform(0.0, 1.0, n), pts=np.zeros((n, 2)))


@pytest.mark.parametrize("n", [4, 64, 65, 66, 70, 90])
def test_cliques_match_oracle(n):
    O = _O()
    g = complete(n)
    s = Staged(g)
    s.sym.set_launch(512, 161792, 1)
    s.sym.upload()
    log(f"[fdpf layouts] complete graph n={n}: {s.sym.info.tail_nodes} tail nodes")
    ref = O.solve_grid(g)
    Vm, Va, it, _, status, _ = s.newton()
    assert ref.status == 0 and status.item() == 0 and it.item() == ref.iters
    np.testing.assert_allclose(Vm[0].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
    np.testing.assert_allclose(Va[0].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
    mat, st = s.sym.fdpf_factors(s.r, s.x, s.b, s.type)
    Vm = s.Vm0.repeat(1, 1).contiguous()
    Va = s.Va0.repeat(1, 1).contiguous()
    it, _, status, _ = s.sym.fdpf(s.yval[0], s.type, s.Psp, s.Qsp, Vm, Va, mat)
    ref = O.solve_grid_fdpf(g)
    assert ref.status == 0 and st.item() == 0 and status.item() == 0
    assert it.item() == ref.iters
    np.testing.assert_allclose(Vm[0].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
    np.testing.assert_allclose(Va[0].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
