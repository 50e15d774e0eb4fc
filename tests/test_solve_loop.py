"""The host side of a solve against a HIP runtime without a device (fake_hip.cpp, loaded
ahead of the library): which launches a call makes and what it makes of the stopping rule's
reports.  Each case runs in a process of its own."""
import os
import shutil
import subprocess
import sys

import pytest

from conftest import ROOT
from paper_2008_03885_amd import mg

PRELUDE = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library: its HIP calls go here
from paper_2008_03885_amd import mg, rbc
F, U = 0x1000, 0x2000  # never dereferenced: kernels do nothing
def counts():
    k, g = ctypes.c_int(), ctypes.c_int()
    fake.fake_counts(ctypes.byref(k), ctypes.byref(g))
    return k.value, g.value
def raises(call, *args):
    try:
        call(*args)
    except mg.MGError as e:
        return e.status
    return mg.MG_OK
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if not os.path.exists(mg.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run([gxx, "-shared", "-fPIC", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)
    return so


def _run(fake, body, **env):
    keep = {k: v for k, v in os.environ.items() if not k.startswith("MG_")}
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake], env=dict(keep, PYTHONPATH=ROOT, **env), cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    if r.returncode != 0:
        pytest.fail(r.stdout + r.stderr, pytrace=False)


@pytest.mark.parametrize("call,graph,nth", [("mg.mg_solve", "0", 6), ("mg.mg_solve_async", "0", 6),
                                            ("mg.mg_solve_async", "1", 5)])
def test_solve_after_a_failed_one(fake, call, graph, nth):
    """A solve that a launch's error ended leaves checks on the stream.  They report before
    the next solve begins, which then counts its own checks only."""
    _run(fake, r"""
h = mg.mg_setup(mg.make_config(dim=2, n=257, max_cycles=20))
fake.fake_stop_at(1)
fake.fake_fail_launch(%d)  # the first check is in
assert raises(%s, h, F, U) == mg.MG_EDEVICE
fake.fake_fail_launch(0)
fake.fake_stop_at(6)
st, res = mg.mg_solve(h, F, U)
assert st == mg.MG_OK and res.cycles == 5, (st, res.cycles)
mg.mg_destroy(h)
""" % (nth, call), MG_GRAPH=graph)


def test_red_black_coarsening_solve_after_a_failed_one(fake):
    """The same for mg_rbc_solve."""
    _run(fake, r"""
h = rbc.setup(rbc.make_config(n=257, levels=9, max_cycles=20))
fake.fake_stop_at(1)
counts()
fake.fake_fail_launch(4)  # start, first pass and check are in
assert raises(rbc.solve, h, F, U, 20) == mg.MG_EDEVICE
fake.fake_fail_launch(0)
fake.fake_stop_at(6)
st, k, hist = rbc.solve(h, F, U, 20)
assert k == 5, (st, k)
rbc.destroy(h)
""")


@pytest.mark.parametrize("n,sync_graph,async_graph", [(65, 0, 0), (129, 0, 0), (257, 0, 1), (4097, 0, 1)])
def test_graphs_by_launches_of_a_step(fake, n, sync_graph, async_graph):
    """A step of about 4, 6, 8 or 16 launches: mg_solve launches its kernels, and
    mg_solve_async, which enqueues every step before it returns, replays a graph above 6."""
    _run(fake, r"""
n, sync_graph, async_graph = %d, %d, %d
h = mg.mg_setup(mg.make_config(dim=2, n=n, max_cycles=20))
fake.fake_stop_at(6)
counts()
st, res = mg.mg_solve(h, F, U)
kernels, graphs = counts()
assert st == mg.MG_OK and res.cycles == 5 and graphs == 6 * sync_graph, (st, res.cycles, graphs)
mg.mg_solve_async(h, F, U)
kernels, graphs = counts()
assert graphs == 21 * async_graph and (kernels < 6) == bool(async_graph), (kernels, graphs)
st, res = mg.mg_query(h)
assert st == mg.MG_OK and res.cycles == 5, (st, res.cycles)
st, res = mg.mg_solve(h, F, U)
assert st == mg.MG_OK and res.cycles == 5, (st, res.cycles)
mg.mg_destroy(h)
""" % (n, sync_graph, async_graph))
