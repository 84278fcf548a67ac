"""The operation lists of the LDS tail and of the upper levels, walked on the CPU
as the kernels walk them (check_lists.cpp), also beyond the LDS budgets that the
library accepts, where a level's offsets would no longer fit their field."""
import os
import subprocess

import pytest

import gridgen
from topologies import complete, mesh

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1811_02512_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lists") / "check_lists")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(HERE, "check_lists.cpp"), os.path.join(CSRC, "analyze.cpp"),
                    "-o", exe], check=True)
    return exe


def topology(name):
    kind, _, arg = name.partition(" ")
    k = [int(v) for v in arg.split()]
    if kind == "grid":
        g = gridgen.make_grid(k[0], 1)
        return g.n, list(zip(g.f.tolist(), g.t.tolist()))
    if kind == "mesh":
        return k[0] * k[1], mesh(*k)
    if kind == "complete":
        return k[0], complete(k[0])
    if kind == "path":
        return k[0], [(i, i + 1) for i in range(k[0] - 1)]
    if kind == "band":
        return k[0], [(i, i + d) for i in range(k[0]) for d in range(1, k[1]) if i + d < k[0]]
    # rows of k[0] slots under one clique of k[0]: hubs and their leaves
    n = 1 + k[0] + k[1]
    hubs, leaves = range(1, k[0] + 1), range(k[0] + 1, n)
    return n, ([(0, 1)] + [(a, b) for a in hubs for b in hubs if a < b] +
               [(a, b) for a in hubs for b in leaves])


@pytest.mark.parametrize("name,ordering,budget", [
    ("grid 2", 0, 65536), ("grid 200", 0, 65536), ("grid 2000", 0, 0), ("grid 2000", 0, 65536),
    ("grid 5003", 0, 161792), ("mesh 20 20", 0, 65536), ("mesh 20 20", 0, 0),
    ("complete 70", 0, 161792), ("path 300", 1, 65536), ("band 90 38", 1, 65536),
    ("leaves 1 198", 0, 161792), ("leaves 2 300", 0, 161792), ("leaves 40 40", 0, 161792),
    # 72,928 operations on the leaves' level
    ("leaves 52 53", 0, 400000), ("leaves 45 60", 0, 400000)])
def test_every_update_comes_once(checker, name, ordering, budget):
    n, edges = topology(name)
    text = f"{n} {len(edges)} {ordering} {budget}\n" + "".join(f"{a} {b}\n" for a, b in edges)
    r = subprocess.run([checker], input=text, text=True, stdout=subprocess.PIPE, timeout=120)
    assert r.returncode == 0, r.stdout
    print(r.stdout)
