"""Launch shape of a per-item kernel over the tests' HIP runtime: one dimension,
whole turns of eight, from eight cases and three quarters of the turns on."""
from stub_runtime import run


def test_shape_by_batch():
    run("""
        import gridgen
        s = Sym(gridgen.make_grid(1000, 1))
        nb = -(-4 * 1000 // 256)  # four threads a row
        for B in range(1, 70):
            rc = lib.pf_build_ybus(s.h, B, PTR, PTR, PTR, I64(0), None, I64(0), PTR,
                                   I64(2 * s.info.nnz_y), None)
            assert rc == 0, lib.pf_last_error()
            full = -(-B // 8) * 8
            assert latest()[1] == (nb * full if B >= 8 and 3 * full <= 4 * B else nb), (B, latest())
    """)
