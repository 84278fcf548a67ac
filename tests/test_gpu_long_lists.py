"""Tail destinations with many operations on one level: buses with leaves, and two
buses that share them (a long slot as well as two long diagonals), at the counts
where a wavefront takes over and where its lanes go round again; on the smallest
and the largest workgroup, against the CPU oracle."""
import numpy as np
import pytest

from gpu_helpers import Staged, log
from topologies import grid_of

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# 8 one after the other; 16 quads (64 lanes in the fast decoupled sweep) share
# the rest: 24 and 72 fill them once
@pytest.mark.parametrize("threads", [64, 512])
@pytest.mark.parametrize("leaves", [7, 8, 9, 24, 25, 72, 73, 300])
@pytest.mark.parametrize("hubs", [1, 2])
def test_matches_oracle(hubs, leaves, threads):
    from oracle import oracle as O

    # the slack joins the first hub, the hubs each other, each leaf all hubs
    edges = [(0, 1)] + [(h, h + 1) for h in range(1, hubs)]
    edges += [(h, hubs + 1 + i) for i in range(leaves) for h in range(1, hubs + 1)]
    g = grid_of(1 + hubs + leaves, edges)
    s = Staged(g)
    s.sym.set_launch(threads, 161792, 1)
    log(f"[long lists] {hubs} hubs, {leaves} leaves, {threads} threads")
    assert s.sym.info.tail_nodes == g.n - 1
    ref = O.solve_grid(g)
    Vm, Va, it, _, st, _ = s.newton()
    assert ref.status == st.item() == 0 and it.item() == ref.iters
    np.testing.assert_allclose(Vm[0].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
    np.testing.assert_allclose(Va[0].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
    ref = O.solve_grid_fdpf(g)
    mat, st = s.sym.fdpf_factors(s.r, s.x, s.b, s.type)
    assert st.item() == 0
    Vm, Va = s.Vm0.repeat(1, 1).contiguous(), s.Va0.repeat(1, 1).contiguous()
    it, _, st, _ = s.sym.fdpf(s.yval[0], s.type, s.Psp, s.Qsp, Vm, Va, mat)
    assert ref.status == st.item() == 0 and it.item() == ref.iters
    np.testing.assert_allclose(Vm[0].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
    np.testing.assert_allclose(Va[0].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
