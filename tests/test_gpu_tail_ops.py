"""The LDS tail's operation lists at their edges: one destination with a term
from every leaf of a hub, more levels than one wavefront holds table entries
for (a path), more operations on a level than the workgroup has threads (a
band with long rows), on the smallest and the largest workgroup.  Factors and
both solves against a dense LAPACK solve of the assembled matrix."""
import numpy as np
import pytest

from gpu_helpers import dev, log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _topology(name):
    if name == "hub":  # 198 leaves on bus 1
        return 200, [(0, 1)] + [(1, i) for i in range(2, 200)]
    if name == "path":  # 149 one-node levels
        return 150, [(i, i + 1) for i in range(149)]
    return 60, [(i, i + d) for i in range(60) for d in range(1, 38) if i + d < 60]


@pytest.mark.parametrize("threads", [64, 512])
@pytest.mark.parametrize("name", ["hub", "path", "band"])
def test_tail_lists_match_dense(name, threads):
    from paper_1811_02512_amd import api, binding as B

    n, edges = _topology(name)
    f, t = (np.array(v, np.int32) for v in zip(*edges))
    rng = np.random.default_rng(3)
    # natural order keeps the band's rows long and the path one node a level
    sym = api.Symbolic(n, f, t, 0, B.PF_ORDER_MINDEG if name == "hub" else B.PF_ORDER_NATURAL)
    sym.set_launch(threads, 161792, 1)
    sym.upload()
    info, ex = sym.info, sym.export()
    assert info.tail_nodes == info.nn, "the whole grid sits in the tail"
    log(f"[tail] {name}: {info.nlevels} levels, {info.nnz_l} slots, {threads} threads")
    nn, lp, li = info.nn, ex["Lp"], ex["Li"]
    A = np.zeros((2 * nn, 2 * nn))
    vals = np.zeros(info.vals_doubles)
    for p in range(nn):
        D = rng.uniform(-1, 1, (2, 2)) + (4.0 + 2 * (lp[p + 1] - lp[p])) * np.eye(2)
        if name == "hub" and p == nn - 1:
            D += 400.0 * np.eye(2)
        vals[4 * p:4 * p + 4] = D.ravel()
        A[2 * p:2 * p + 2, 2 * p:2 * p + 2] = D
        for s in range(lp[p], lp[p + 1]):
            k = li[s]
            lo, up = rng.uniform(-1, 1, (2, 2, 2))
            o = info.lu_offset + 8 * s
            vals[o:o + 4], vals[o + 4:o + 8] = lo.ravel(), up.ravel()
            A[2 * k:2 * k + 2, 2 * p:2 * p + 2] = lo
            A[2 * p:2 * p + 2, 2 * k:2 * k + 2] = up
    # values at rounding of products of these sizes: 1e-10 of the largest
    # entry, the tolerance of the factor and solve tests
    b = rng.uniform(-1, 1, 2 * nn)
    v = dev(vals).reshape(1, -1)
    st = torch.empty(1, dtype=torch.int32, device="cuda")
    B.pf_factor(sym.h, 1, v, info.vals_doubles, st)
    for transpose in (0, 1):
        x = dev(b).reshape(1, -1)
        B.pf_solve(sym.h, 1, v, info.vals_doubles, x, 2 * nn, transpose=transpose)
        want = np.linalg.solve(A.T if transpose else A, b)
        got = x[0].cpu().numpy()
        assert st.item() == 0
        assert np.abs(got - want).max() <= 1e-10 * np.abs(want).max(), (name, transpose)
