"""Dynamic LDS that the entry points ask a device for, over the tests' HIP
runtime: a launch that needs more than the default limit is made only where the
limit has been raised, on each device and from each thread, and has a way
without it."""
from stub_runtime import run


def test_mismatch_where_the_limit_cannot_be_raised():
    run("""
        import gridgen
        stub.stub_refuse_attributes(1)
        s = Sym(gridgen.make_grid(6000, 1))  # 96,000 bytes of voltages
        assert mismatch(s) == 0, lib.pf_last_error()
        assert latest()[3] == 0  # the voltages from their polar values
        stub.stub_refuse_attributes(0)
        small = Sym(gridgen.make_grid(600, 1))
        assert mismatch(small) == 0 and latest()[3] == 9600
    """)


def test_every_device_of_a_process():
    run("""
        import gridgen
        s = Sym(gridgen.make_grid(6000, 1))
        for dev in (0, 3):
            stub.hipSetDevice(dev)
            assert mismatch(s) == 0, (dev, lib.pf_last_error())
            assert latest()[3] == 96000
            assert fdpf(s) == 0, (dev, lib.pf_last_error())
            rhs = lambda tr: lib.pf_solve(s.h, 1, PTR, I64(s.info.vals_doubles), 1, PTR, I64(0),
                                          tr, None)
            assert rhs(0) == 0 and rhs(1) == 0, (dev, lib.pf_last_error())
            assert latest()[3] == 16 * s.info.nn
    """)


def test_first_calls_from_several_threads():
    run("""
        import threading
        import gridgen
        s = Sym(gridgen.make_grid(6000, 1))
        stub.stub_slow_attributes(20000)
        got, go = {}, threading.Barrier(4)

        def call(k):
            go.wait()
            got[k] = (mismatch(s), latest()[3])

        ts = [threading.Thread(target=call, args=(k,)) for k in range(4)]
        [t.start() for t in ts]
        [t.join() for t in ts]
        assert set(got.values()) == {(0, 96000)}, got
    """)
