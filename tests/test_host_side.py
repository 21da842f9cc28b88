"""The library's host side without a GPU: a stand-in for the HIP runtime
(native/fake_hip.cpp: device memory is the host's, kernels do not run) takes
the real one's place in a process of its own, and is told what to refuse.
"""
import subprocess
import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]

PRELUDE = """
import ctypes, os, sys, types
sys.modules["torch"] = types.ModuleType("torch")  # (the binding loads it for its HIP runtime)
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("live", "peak", "allocs", "launches", "streams"):
    getattr(hip, "fake_" + f).restype = ctypes.c_int64
hip.fake_limit.argtypes = [ctypes.c_int64, ctypes.c_int64]
hip.fake_waits.argtypes, hip.fake_waits.restype = [ctypes.c_void_p], ctypes.c_int64
import numpy as np
import gridgen
from paper_2201_00241_amd import rh

def geo(n, seed=1):
    return gridgen.geometric(n, int(1.35 * n), max(3, n // 10), seed=seed, alpha=0.1, kappa=0.0085)

def solved_on_device(net):
    # kernels do not run, so the factors come back as zeros: every status but
    # the device's is as good as any
    try:
        net.solve_device()
    except rh.RhError as e:
        if e.status == rh.RH_EDEVICE:
            raise
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = tmp_path_factory.mktemp("native") / "libfake_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I/opt/rocm/include",
                    str(ROOT / "tests/native/fake_hip.cpp"), "-o", str(out)], check=True)

    def run(code):
        res = subprocess.run([sys.executable, "-c", PRELUDE + code, str(out)], cwd=ROOT, capture_output=True, text=True,
                             timeout=100)
        assert res.returncode == 0, res.stdout + res.stderr
        return res.stdout

    return run


def test_a_small_networks_fronts_leave_a_large_ones_bound(fake):
    """The dynamic LDS that a kernel may use is the kernel's, not a network's:
    a network built later, with smaller fronts, must not lower it."""
    fake("""
ctx = rh.Context(0)
large, small = rh.Network(ctx, geo(3000)), rh.Network(ctx, gridgen.ring9())
solved_on_device(large)
solved_on_device(small)
solved_on_device(large)
""")


@pytest.mark.parametrize("call,after", [("hipFuncSetAttribute", 0), ("hipMemcpy", 20), ("hipMalloc", 20)])
def test_an_error_of_the_device_is_not_taken_for_a_lack_of_memory(fake, call, after):
    """Only fronts that there is no memory for give way to the row-by-row
    factorisation; any other error ends the call."""
    fake(f"""
net = rh.Network(rh.Context(0), geo(1000))
before = hip.fake_live()
hip.fake_refuse(b"{call}", {after})  # the fronts' arrays are among the first of the device Newton
try:
    net.solve_device()
    assert False, "the refused call went unnoticed"
except rh.RhError as e:
    assert e.status == rh.RH_EDEVICE, e
assert hip.fake_live() == before
""")


def test_no_memory_for_the_fronts(fake):
    fake("""
net = rh.Network(rh.Context(0), geo(1000))
hip.fake_limit(-1, 8 << 20)  # the fronts of 1,000 buses take 14 MB, no other array more than 2
solved_on_device(net)
""")


@pytest.mark.parametrize("prec", ["RH_FP64", "RH_FP32_REFINED"])
def test_scratch_per_direction_holds_for_every_call(fake, prec):
    """A call's launch scratch is at most rh_network_device_bytes' figure for
    each of its directions, counted in whole chunks, on both paths, also
    beside a larger network (a batch's work list is extra); and the server's
    footprint holds it."""
    fake(f"prec = rh.{prec}" + """
grids = [geo(1000), geo(8600), geo(12000)]  # states: 1,899; 16,339; 22,799 (the tree path's from 16,000 on)
W = np.zeros(1)
whole = lambda k: -(-k // rh.RH_CHUNK_DIRS) * rh.RH_CHUNK_DIRS
for k in (1, 3, 15, 16, 17, 40):
    for g in grids[:2]:
        net = rh.Network(rh.Context(0), g)
        net.solve()
        per, before = net.device_bytes(prec)[1], hip.fake_live()
        figures = 32 * 64 if prec else 0  # the refined mode's report
        rh.rh_hvp_device(net.h, k, W.ctypes.data, net.n_p, W.ctypes.data, net.n_p, prec)
        assert 0 < hip.fake_live() - before - figures <= whole(k) * per, (k, net.n_x)
ctx = rh.Context(0)
nets = [rh.Network(ctx, g) for g in grids[1:]]
for net in nets:
    net.solve()
per = [net.device_bytes(prec)[1] for net in nets]
ptr = [W.ctypes.data] * 2
for ks in ((1, 1), (40, 2), (200, 1)):
    before = hip.fake_live()
    b = rh.rh_batch_create(ctx.h, [n.h for n in nets], ks, ptr, [n.n_p for n in nets], ptr, [n.n_p for n in nets], prec=prec)
    assert hip.fake_live() - before <= sum(whole(k) * p for k, p in zip(ks, per)) + 8192, ks
    rh.rh_batch_destroy(b)
from paper_2201_00241_amd.serving import Request, Server
server = Server.__new__(Server)
server.nets, server.dirs_per_launch, server.block = {"a": nets[1]}, 4096, 100
for k, dirs in ((1, 16), (16, 16), (17, 32), (100, 112), (101, 128)):
    W = 2 * k * nets[1].n_p * 8
    assert server.footprint_bytes(Request(0, "a", k, prec=prec)) == W + dirs * per[1]
""")


@pytest.mark.parametrize("prec", ["RH_FP64", "RH_FP32_REFINED"])
def test_rounds_shorten_where_memory_is_short(fake, prec):
    """A call whose directions' scratch is not to be had runs in shorter
    rounds, eager and recorded, down to a chunk."""
    fake(f"prec = rh.{prec}" + """
ctx = rh.Context(0)
net = rh.Network(ctx, geo(8600))
net.solve()
W = np.zeros(1)
per = net.device_bytes(prec)[1]
args = [ctx.h, [net.h], [1024], [W.ctypes.data], [net.n_p], [W.ctypes.data], [net.n_p]]
def call():
    before = hip.fake_launches()
    rh.rh_hvp_device(net.h, 1024, W.ctypes.data, net.n_p, W.ctypes.data, net.n_p, prec)
    rounds = hip.fake_launches() - before
    before = hip.fake_launches()
    rh.rh_batch_destroy(rh.rh_batch_create(*args, prec=prec))
    assert hip.fake_launches() - before == rounds
    return rounds
hip.fake_limit(-1, 17 * per)  # a chunk
one = call() // 64
hip.fake_limit(-1, 16 * 20 * per)  # 64 chunks, halved to 16
assert call() == 4 * one
hip.fake_limit(-1, -1)
assert call() == one
net2 = rh.Network(rh.Context(0), geo(8600))
net2.solve()
hip.fake_limit(-1, 15 * per)
try:
    rh.rh_hvp_device(net2.h, 16, W.ctypes.data, net.n_p, W.ctypes.data, net.n_p, prec)
    assert False, "no chunk fits"
except rh.RhError as e:
    assert e.status == rh.RH_ENOMEM, e
""")


def test_no_memory_for_the_nodes_matrices(fake):
    """The one-workgroup path takes a network whose nodes' matrices find no
    memory, and gives it back with the next solve that finds it; an error of the
    device is none of this."""
    fake("""
net = rh.Network(rh.Context(0), geo(8600))
W = np.zeros(1)
def launches():
    before = hip.fake_launches()
    rh.rh_hvp_device(net.h, 16, W.ctypes.data, net.n_p, W.ctypes.data, net.n_p)
    return hip.fake_launches() - before
hip.fake_refuse(b"memory", 10)
net.solve()
assert launches() == 1
net.solve()
assert launches() > 10
hip.fake_refuse(b"hipMalloc", 10)
net = rh.Network(rh.Context(0), geo(8600))
try:
    net.solve()
    assert False, "the refused call went unnoticed"
except rh.RhError as e:
    assert e.status == rh.RH_EDEVICE, e
""")


@pytest.mark.parametrize("force", ["RH_NO_LDS", "RH_DIRS_PER_GROUP"])
@pytest.mark.parametrize("n_bus", [1000, 8600])
def test_the_allocation_free_call_never_allocates(fake, n_bus, force):
    """Not for a launch shape forced after the solve either, whose arrays a
    network of the tree path does not hold."""
    fake(f"""
net = rh.Network(rh.Context(0), geo({n_bus}))
net.solve()
os.environ["{force}"] = "1"
W = np.zeros(1)
before = hip.fake_allocs(), hip.fake_launches()
for prec in (rh.RH_FP64, rh.RH_FP32_REFINED):
    for k in (1, 300):
        rh.rh_hvp_device_noalloc(net.h, k, W.ctypes.data, net.n_p, W.ctypes.data, net.n_p, prec)
assert hip.fake_allocs() == before[0] and hip.fake_launches() >= before[1] + 4
""")


MIXED = """
ctx = rh.Context(0)
nets = [rh.Network(ctx, g) for g in (geo(60), geo(8600), geo(100), geo(8700, 2))]
for net in nets:
    net.solve()
W = np.zeros(1)
ptr = [W.ctypes.data] * 4
def batch(stream, prec=rh.RH_FP64):
    n_p = [n.n_p for n in nets]
    rh.rh_hvp_batch_device(ctx.h, [n.h for n in nets], [5, 17, 1, 3], ptr, n_p, ptr, n_p, None, prec, stream)
"""


def test_the_first_batch_of_both_paths_sets_up_little(fake):
    """Its scratch is one allocation, as that of other batches."""
    fake(MIXED + """
allocs = hip.fake_allocs()
batch(0x100)
assert hip.fake_allocs() == allocs + 3  # the scratch and the two work lists
batch(0x100)
assert hip.fake_allocs() == allocs + 3
""")


def test_contexts_take_turns_with_the_side_streams(fake):
    """A stream takes from a tenth of a millisecond to several to create: a new
    context's batches use one that is there, calls under way on other streams
    keep theirs, and there are never more than four."""
    fake(MIXED + """
streams = hip.fake_streams()
batch(0x100)
batch(0x200, rh.RH_FP32_REFINED)
assert hip.fake_streams() == streams + 1
ctx = rh.Context(0)
nets = [rh.Network(ctx, g) for g in (geo(60), geo(8600), geo(100), geo(8700, 2))]
for net in nets:
    net.solve()
batch(0x100)
assert hip.fake_streams() == streams + 1
hip.fake_busy(1)
for n in (2, 3, 4, 4, 4):
    batch(0x100)
    assert hip.fake_streams() == streams + n
hip.fake_busy(0)
batch(0x300)
assert hip.fake_streams() == streams + 4
""")


@pytest.mark.parametrize("list_of", [0, 1])
def test_the_callers_stream_waits_for_what_is_under_way(fake, list_of):
    """An exception between the two kinds of launches of a batch leaves none
    of them running beside the caller's stream."""
    fake(MIXED + f"""
batch(0x100)
before = hip.fake_waits(0x100)
hip.fake_refuse(b"hipMemcpyAsync", {list_of})
try:
    batch(0x100)
    assert False, "the exception went unnoticed"
except rh.RhError as e:
    assert e.status == rh.RH_ENOMEM, e
assert hip.fake_waits(0x100) == before + 1
""")


@pytest.mark.parametrize("n,nrhs,launches", [(1, 1, 3), (30, 65, 3), (64, 64, 3), (65, 1, 5)])
def test_launches_of_a_dense_solve(fake, n, nrhs, launches):
    """Panels, a block of the solution each, and the solution's way out, also
    with more than 64 right-hand sides.  (From eight enqueued operations on a
    call takes 40 us longer to return.)"""
    fake(f"""
A = np.zeros(1)
rh.rh_cholesky_solve_device(rh.Context(0).h, {n}, A.ctypes.data, {n}, A.ctypes.data, {n}, {nrhs})
assert hip.fake_launches() == {launches}, hip.fake_launches()
""")


def test_the_leaves_matrices_are_kept_once(fake):
    """The refined mode reads the leaves' matrices, four fifths of all, in FP64
    as well: with a copy of them in FP32 this network held 62.5 MB."""
    fake("""
net = rh.Network(rh.Context(0), geo(8600))
net.solve()
assert net.device_bytes()[0] < 52e6, net.device_bytes()
""")


@pytest.mark.parametrize("n_bus", [60, 1000, 8600])
def test_resident_bytes_are_all_that_is_held(fake, n_bus):
    """Also the device solve's fronts, the largest part at 1,000 buses."""
    fake(f"""
net = rh.Network(rh.Context(0), geo({n_bus}))
before = hip.fake_live()
net.solve()
assert net.device_bytes()[0] == hip.fake_live() - before
net.solve_device()
assert net.device_bytes()[0] == hip.fake_live() - before
net.solve()
assert net.device_bytes()[0] == hip.fake_live() - before
""")


def test_the_tuner_tries_a_whole_call_of_the_tree_path(fake, tmp_path):
    """A full Hessian with k_block = 0 must not be slower than with any other:
    calls of up to 4,096 directions are among the candidates, and a shape
    cached before they were is not taken."""
    fake(f"""
os.environ["RH_TUNE_CACHE"] = "{tmp_path}/tiles.txt"
""" + """
net = rh.Network(rh.Context(0), geo(12000))
net.solve()
hip.fake_peak_reset()
before = hip.fake_live()
t = net.autotune()
assert t["source"] == 1
assert hip.fake_peak() - before >= net.n_p * net.n_p * 8, (net.n_p, hip.fake_peak() - before)
path = os.environ["RH_TUNE_CACHE"]
line = open(path).read().split()
key = next(i for i, w in enumerate(line) if "-tree" in w)
old = line[:key] + ["fp64-tree", "128"] + line[key + 2:]
open(path, "w").write(" ".join(old) + "\\n")
net = rh.Network(rh.Context(0), geo(12000))
net.solve()
assert net.autotune()["source"] == 1
assert net.autotune()["source"] == 2
""")


def test_a_dense_solve_names_the_error_of_its_workspace(fake):
    fake("""
A = np.zeros(1)
ctx = rh.Context(0)
for call, says in ((b"memory", "out of memory"), (b"hipMalloc", "refused")):
    hip.fake_refuse(call, 0)
    try:
        rh.rh_cholesky_solve_device(ctx.h, 9, A.ctypes.data, 9, A.ctypes.data, 9, 1)
        assert False, "the refused call went unnoticed"
    except rh.RhError as e:
        assert e.status == rh.RH_ENOMEM and says in str(e), e
# and none is left for the next call to find
rh.rh_cholesky_solve_device(ctx.h, 9, A.ctypes.data, 9, A.ctypes.data, 9, 1)
""")
