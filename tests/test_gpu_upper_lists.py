"""The levels below the tail of a spread launch: on grids with much fill, with
their lists whole and cut short, with far more destinations on a level than the
launch has threads, and with destinations of a hundred terms and more; each
against the CPU oracle."""
import numpy as np
import pytest

from gpu_helpers import Staged, log
from topologies import complete, grid_of, mesh

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def check(s, ref, keep=False):
    Vm, Va, it, _, st, ws = s.newton(keep=keep)
    assert st.item() == ref.status == 0 and it.item() == ref.iters
    # the tolerance and iteration counts of the parity tests
    np.testing.assert_allclose(Vm[0].cpu().numpy(), ref.Vm, rtol=0, atol=1e-9)
    np.testing.assert_allclose(Va[0].cpu().numpy(), ref.Va, rtol=0, atol=1e-9)
    return ws


def same_factors(sym, ws, other):
    """The factors kept for the gradients, to rounding (without the padding of
    the diagonal section, which nothing writes)."""
    i = sym.info
    for k in (slice(0, 4 * i.nn), slice(i.lu_offset, i.vals_doubles)):
        a, b = ws.reshape(-1)[k], other.reshape(-1)[k]
        assert (a - b).abs().max().item() <= 1e-9 * a.abs().max().item()


@pytest.mark.parametrize("budget", [0, 65536])
@pytest.mark.parametrize("name", ["mesh", "complete"])
def test_whole_and_cut_short(name, budget):
    from oracle import oracle as O
    from paper_1811_02512_amd import binding as B

    g = grid_of(900, mesh(30, 30)) if name == "mesh" else grid_of(120, complete(120))
    ref = O.solve_grid(g)
    s = Staged(g)
    s.sym.set_launch(256, budget, 1)
    short = s.sym.info.dev_bytes
    B.pf_symbolic_set_spread(s.sym.h, 8)  # after the upload: the lists there stay
    log(f"[upper lists] {name} budget {budget}: {short} bytes cut short")
    ws = check(s, ref, keep=True)
    w = Staged(g)
    w.sym.set_launch(256, budget, 1)
    w.sym.set_spread(8)  # uploads again
    assert w.sym.info.dev_bytes > 1.3 * short and len(w.sym.kept) == 1
    wh = check(w, ref, keep=True)
    same_factors(s.sym, ws, wh)
    # a member of a plan keeps its device copy, and the plan its validity
    p = Staged(g)
    from paper_1811_02512_amd import api

    plan = api.MultiPlan([p.sym])
    p.sym.set_spread(8)
    assert not p.sym.kept
    check(p, ref)
    del plan


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("name", ["band", "hub"])
def test_more_destinations_than_threads(name, keep):
    """128 threads in all; the band's levels have 700 destinations, the hub's
    one level a diagonal of 198 terms."""
    from oracle import oracle as O
    from paper_1811_02512_amd import binding as B

    if name == "band":
        n, edges = 90, [(i, i + d) for i in range(90) for d in range(1, 38) if i + d < 90]
    else:
        n, edges = 200, [(0, 1)] + [(1, i) for i in range(2, 200)]
    g = grid_of(n, edges)
    ref = O.solve_grid(g)
    s = Staged(g, B.PF_ORDER_NATURAL if name == "band" else B.PF_ORDER_MINDEG)
    s.sym.set_launch(64, 0, 1)
    s.sym.set_spread(2)
    ex = s.sym.export()
    deg = np.diff(ex["Lp"])
    log(f"[upper lists] {name}: up to {int((deg * (deg + 1) // 2).max())} operations a node")
    spread = check(s, ref, keep)
    s.sym.set_spread(0)
    one = check(s, ref, keep)
    if keep:
        same_factors(s.sym, one, spread)
