"""The fast decoupled launch's LDS over the tests' HIP runtime (256 compute units
of 160 KB): a budget below the default holds for all of it."""
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
