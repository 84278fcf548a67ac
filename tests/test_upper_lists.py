"""The lists that a spread launch reads: a grid with much fill carries them whole
only where a spread was set, and buffers of either size are taken."""
import numpy as np
import pytest

from paper_1811_02512_amd import binding as B
from stub_runtime import run
from topologies import complete, mesh


@pytest.mark.parametrize("n,edges", [(900, mesh(30, 30)), (4000, mesh(80, 50)),
                                     (300, complete(300))])
def test_size_without_a_spread(n, edges):
    f, t = (np.ascontiguousarray(v, np.int32) for v in zip(*edges))
    h = B.pf_analyze(n, f, t)
    for budget in (65536, 161792):
        B.pf_symbolic_set_launch(h, 0, budget, 4)
        i = B.pf_symbolic_info(h)
        # update pairs (8 bytes), again where the tail pulls them; per slot its
        # record, neighbours and the tail's and the bounded lists' entries (at
        # most 4 of 20 or 8 bytes); per node and admittance entry the rest
        most = 16 * i.n_upd + 220 * i.nnz_l + 300 * n + 24 * i.nnz_y + 50 * 256
        assert i.dev_bytes <= most, (budget, i.dev_bytes, most)
    B.pf_symbolic_destroy(h)


def test_a_spread_set_before_or_after_the_upload():
    run("""
        from tests.topologies import complete, grid_of, mesh
        s = Sym(grid_of(200, complete(200)))
        small = s.info.dev_bytes
        assert lib.pf_symbolic_set_spread(s.h, 16) == 0
        large = s.info.dev_bytes
        assert large > 2 * small
        assert mismatch(s) == 0  # what is on the device still serves
        assert s.upload(small - 1) != 0
        assert s.upload(small) == 0 and s.info.dev_bytes == small
        assert lib.pf_symbolic_set_spread(s.h, 16) == 0 and s.upload(large) == 0
        # a new budget keeps them; so does a launch on one workgroup
        assert lib.pf_symbolic_set_spread(s.h, 0) == 0
        assert lib.pf_symbolic_set_launch(s.h, 0, I64(32768), 1) == 0
        assert s.info.dev_bytes > 2 * small
        # a batch that shares its largest grids out
        m = Sym(grid_of(1600, mesh(40, 40)))
        small = m.info.dev_bytes
        plan, arr = C.c_void_p(), (C.c_void_p * 1)(m.h)
        assert lib.pf_multi_create(1, arr, C.byref(plan)) == 0
        assert lib.pf_multi_set_spread(plan, 1) == 0 and m.info.dev_bytes == small
        assert lib.pf_multi_set_spread(plan, 4) == 0 and m.info.dev_bytes > 1.5 * small
    """)
