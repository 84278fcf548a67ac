"""The workgroup's size splits the work and changes no operation or order: the
same bits from 64 to 512 threads (among them the two sizes that batches up to
512 cases and larger ones get), for the grids' sparse patterns and for tails of
long rows and of a bus with many neighbours."""
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


def _case(name):
    """Branch ends, ordering."""
    if name == "hub":  # 118 leaves on bus 1
        return 120, [(0, 1)] + [(1, i) for i in range(2, 120)]
    if name == "band":
        return 60, [(i, i + d) for i in range(60) for d in range(1, 31) if i + d < 60]
    g = grid(int(name), 3)
    return g.n, list(zip(g.f.tolist(), g.t.tolist()))


@pytest.mark.parametrize("budget", [16384, 161792])
@pytest.mark.parametrize("name", ["hub", "band", "200", "487", "2000"])
def test_factors_and_solutions(name, budget):
    from paper_1811_02512_amd import api, binding as B

    n, edges = _case(name)
    f, t = (np.array(v, np.int32) for v in zip(*edges))
    rng = np.random.default_rng(5)
    sym = api.Symbolic(n, f, t, 0, B.PF_ORDER_NATURAL if name == "band" else B.PF_ORDER_MINDEG)
    info, first = sym.info, None
    a = rng.uniform(-1, 1, info.vals_doubles)
    D = a[:4 * info.nn].reshape(-1, 2, 2)
    D += (4.0 + 2.0 * np.sqrt(info.nnz_l)) * np.eye(2)
    rhs = rng.uniform(-1, 1, 2 * info.nn)
    for threads in (64, 128, 256, 512):
        sym.set_launch(threads, budget, 1)
        sym.upload()
        log(f"[workgroup] {name} budget {budget}: {sym.info.tail_nodes} tail nodes, {threads}")
        v, x = dev(a).reshape(1, -1), dev(rhs).reshape(1, -1)
        st = torch.empty(1, dtype=torch.int32, device="cuda")
        B.pf_factor(sym.h, 1, v, info.vals_doubles, st)
        B.pf_solve(sym.h, 1, v, info.vals_doubles, x, 2 * info.nn)
        assert st.item() == 0
        first = first or (v, x)
        assert torch.equal(v, first[0]) and torch.equal(x, first[1]), threads


@pytest.mark.parametrize("n", [200, 487, 2000])
def test_newton_and_fast_decoupled(n):
    g = grid(n, 3)
    s = Staged(g)
    P, Q = (dev(a) for a in gridgen.scenario_injections(g, 3, seed=2))
    first = None
    for threads in (64, 128, 256, 512):
        s.sym.set_launch(threads, 65536, 1)
        s.sym.upload()
        log(f"[workgroup] grid {n}, {threads} threads")
        nr = s.newton(3, P, Q)
        assert (nr[4] == 0).all()
        mat, _ = s.sym.fdpf_factors(s.r, s.x, s.b, s.type)
        Vm, Va = s.Vm0.repeat(3, 1).contiguous(), s.Va0.repeat(3, 1).contiguous()
        it, _, st, _ = s.sym.fdpf(s.yval[0], s.type, P, Q, Vm, Va, mat)
        assert (st == 0).all()
        got = [*nr[:4], Vm, Va, it]
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), threads
