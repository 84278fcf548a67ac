"""The fast decoupled launch's LDS over the tests' HIP runtime (256 compute units
of 160 KB): a budget below the default holds for all of it, and the batches and
budgets of the GPU test of the four layouts reach one each."""
import test_gpu_fdpf_layouts as layouts
from stub_runtime import run


def test_a_lowered_budget_holds():
    run("""
        import gridgen
        for n in (200, 1200, 3001):
            g = gridgen.make_grid(n, 6)
            mask = 2 * (n // 64 + 2) * 8
            for budget in (0, 4096, 16 * n, 32768, 65535):
                if budget >= 65536:
                    continue
                s = Sym(g, 0, budget)
                for B in (1, 300, 2000):
                    assert fdpf(s, B) == 0, lib.pf_last_error()
                    assert latest()[3] <= budget + mask, (n, budget, B, latest())
    """)

def test_each_layout_is_reached():
    # (batch, budget) of the GPU test, 1,200 buses on 64 threads
    at = [m for m in layouts.test_layouts_match_oracle.pytestmark
          if m.name == "parametrize"][0].args[1]
    run(f"""
        import gridgen
        g = gridgen.make_grid(1200, 6)
        names = []
        for B, budget in {at!r}:
            s = Sym(g, 64, budget)
            assert fdpf(s, B) == 0, lib.pf_last_error()
            names.append(latest()[0])
        # FD_APART, FD_NONE, FD_OVER_X, FD_OVER
        assert [n.split("ILi")[1][0] for n in names] == ["3", "0", "2", "1"], names
    """)
