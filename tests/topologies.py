"""Branch lists of grids with much fill, for the tests of the analysis' sizes and
of the launches that share such a grid's levels."""
import numpy as np

import gridgen


def mesh(a, b):
    """a x b lattice."""
    at = np.arange(a * b).reshape(a, b)
    return [*zip(at[:-1].ravel(), at[1:].ravel()), *zip(at[:, :-1].ravel(), at[:, 1:].ravel())]


def complete(n):
    return list(zip(*np.triu_indices(n, 1)))


def grid_of(n, edges, seed=1):
    """A lightly loaded grid on these branches, the slack at bus 0."""
    f, t = (np.array(v, np.int32) for v in zip(*edges))
    rng = np.random.default_rng(seed)
    m = f.size
    kind = np.full(n, gridgen.BUS_PQ, np.int8)
    kind[0] = gridgen.BUS_SLACK
    kind[1:n // 4] = gridgen.BUS_PV
    return gridgen.Grid(
        n=n, f=f, t=t, r=rng.uniform(0.001, 0.003, m), x=rng.uniform(0.01, 0.03, m),
        b=rng.uniform(0.0, 0.005, m), bus_type=kind,
        vset=np.where(kind == gridgen.BUS_PQ, 1.0, 1.02),
        Pd=rng.uniform(0.0, 0.05, n), Qd=rng.uniform(0.0, 0.02, n),
        Pg=np.where(kind == gridgen.BUS_PV, 0.1, 0.0), pts=np.zeros((n, 2)))
