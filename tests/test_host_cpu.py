"""What the host side enqueues, without a GPU: libbtdf runs in a child process
over a stand-in for the HIP runtime (host_hip.c) whose kernels do nothing and
which looks over every launch of the one-launch step where it would run. Each
such launch has to step every tile of the lattice exactly once."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes
import numpy as np
import btdf_workloads as W
from paper_1806_09403_amd import _lib, api
hip = ctypes.CDLL(None)

def handle(nx, ny, bodies, precision=8, kind=W.COS4):
    h = api.btdf_create(nx, ny, 0.8, kind, 2.6, W.FULLY_PERIODIC, precision=precision)
    for b in bodies:
        api.btdf_add_body(h, b.xy, None, b.cx, b.cy, b.ds)
    return h

def steps_found():
    p = ctypes.POINTER(ctypes.c_int)()
    n = hip.host_hip_steps(ctypes.byref(p))
    return np.ctypeslib.as_array(p, (n, 4)).copy() if n else np.zeros((0, 4), int)
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "libhost_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", os.path.join(ROOT, "tests", "host_hip.c"), "-o", out,
                    "-ldl"], check=True)
    return out


def child(stand_in, code):
    env = dict(os.environ)
    env["LD_PRELOAD"] = " ".join([stand_in] + env.get("LD_PRELOAD", "").split())
    r = subprocess.run([sys.executable, "-c", PRELUDE + code], cwd=ROOT, env=env, capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


@pytest.mark.parametrize("velocity", [(0.02, 0.01, 0.0), (0.0, 0.02, 0.0), (-0.015, 0.0, 0.001)])
def test_every_step_of_moving_bodies_covers_every_tile(stand_in, velocity):
    """The work list of a step changes its length as bodies move from tile to
    tile; steps enqueued singly and steps replayed from a graph both take the
    whole list of the moment."""
    child(stand_in, """
tiles = 10 * 25
for chunk in (0, 8, 5, 50):
    before = len(steps_found())
    h = handle(300, 200, [W.cylinder_body(90.0, 100.0, 12.0, 38)])
    api.btdf_set_option(h, _lib.OPT_GRAPH_CHUNK, chunk)
    api.btdf_set_body_motion(h, 0, *%r)
    forced = set()
    for k in range(60):
        api.btdf_step(h, 17)
        forced.add(api.btdf_get_option(h, _lib.OPT_FORCED_TILES))
    f = steps_found()[before:]
    assert len(forced) > 1, forced                       # (the case keeps its purpose)
    assert len(f) == 60 * 17, len(f)
    bad = np.flatnonzero((f[:, 2] != tiles) | (f[:, 3] != 0))
    assert bad.size == 0, (chunk, bad[:5], f[bad[:5]])
    assert np.all(f[:, 1] > f[:, 0])
    api.btdf_destroy(h)
""" % (velocity,))


def test_forces_without_pinned_memory(stand_in):
    """Forces and histories are read by plain copies where no pinned host memory
    is to be had."""
    child(stand_in, """
hip.host_hip_fail_pinned(1)
h = handle(64, 48, [W.cylinder_body(30.0, 20.0, 8.0, 25)])
for k in range(5):
    api.btdf_step(h, 1)
    assert api.btdf_forces(h).shape == (1, 3)
api.btdf_step(h, 300)
assert api.btdf_force_history(h, 400).shape == (305, 1, 3)
assert hip.host_hip_pinned_calls() == 1          # (not asked for in every read)
hip.host_hip_fail_pinned(0)
for k in range(80):
    api.btdf_forces(h)
assert hip.host_hip_pinned_calls() == 2 and hip.host_hip_pinned_live() == 1   # (nor given up for good)
api.btdf_destroy(h)
""")


def test_pinned_memory_is_made_once_and_given_back(stand_in):
    """Reads of any length, by any number of handles and threads at once, share
    one allocation, which goes with the last handle."""
    child(stand_in, """
import threading
for turn in range(2):
    calls = hip.host_hip_pinned_calls()
    hs = [handle(48, 40, [W.cylinder_body(20.0, 20.0, 8.0, 25)] * (1 + k % 3)) for k in range(12)]

    def read(h, nb):
        for n in (1, 2, 30, 90, 400, 1100, 2000, 3):
            api.btdf_step(h, n)
            assert api.btdf_forces(h).shape == (nb, 3)
            assert api.btdf_force_history(h, n).shape == (n, nb, 3)

    def every(some):
        for h in some:
            read(h, api.btdf_forces(h).shape[0])

    threads = [threading.Thread(target=every, args=(hs[k::6],)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert hip.host_hip_pinned_calls() == calls + 1, hip.host_hip_pinned_calls() - calls
    for h in hs:
        assert hip.host_hip_pinned_live() == 1
        api.btdf_destroy(h)
    assert hip.host_hip_pinned_live() == 0
h = handle(48, 40, [W.cylinder_body(20.0, 20.0, 8.0, 25)])
api.btdf_step(h, 5)
calls = hip.host_hip_pinned_calls()
api.btdf_force_history(h, 5)
assert hip.host_hip_pinned_calls() == calls   # (a single read does not pay for it)
api.btdf_destroy(h)
""")


@pytest.mark.parametrize("n,bodies,passes,whole", [
    (64, 1, 2, True), (65, 1, 2, False), (80, 1, 3, True), (128, 1, 3, False), (128, 1, 6, True), (129, 1, 8, False),
    (256, 1, 8, False), (256, 4, 3, False), (80, 1, 1, True), (81, 1, 1, False), (200, 1, 1, False),
    (100, 60, 2, True), (100, 60, 1, True), (200, 160, 2, True)])
def test_bodies_are_formed_whole_where_that_is_faster(stand_in, n, bodies, passes, whole):
    """One workgroup per body for small bodies, and for many; launches over all
    markers for few large bodies. (passes = 1: the implicit method.)"""
    child(stand_in, """
n, bodies, passes, whole = %r
g = int(1.2 * n / np.pi) + 20
k = int(np.ceil(bodies ** 0.5))
h = handle(k * g, k * g, [W.cylinder_body((i %% k + 0.5) * g, (i // k + 0.5) * g, 1.2 * n / np.pi, n)
                          for i in range(bodies)], kind=W.ROMA3)
api.btdf_set_option(h, *((_lib.OPT_FORCING_METHOD, 1) if passes == 1 else (_lib.OPT_FORCING_PASSES, passes)))
api.btdf_set_option(h, _lib.OPT_TEMPORAL_BLOCKING, 0)
api.btdf_step(h, 3)
ran = [hip.host_hip_launched(b) for b in (b"body_kernel", b"9ib_kernel", b"ib_pass_kernel", b"idf_kernel")]
want = [3, 0, 0, 0] if whole else [0, 3, 3 * (passes - 1), 3 * (passes == 1)]
assert ran == want, (ran, want)
""" % ((n, bodies, passes, whole),))


@pytest.mark.parametrize("n,one", [(63, True), (700, True), (800, False), (4000, False)])
def test_steps_of_tiles_with_very_many_markers_take_two_launches(stand_in, n, one):
    """(700 markers on D = 20: 264 in a tile; 800: 302.)"""
    child(stand_in, """
n, one = %r
h = handle(200, 120, [W.cylinder_body(70.3, 60.2, 20.0, n)])
api.btdf_step(h, 4)
ran = [hip.host_hip_launched(b) for b in (b"11step_kernel", b"9ib_kernel", b"10lbm_kernel")]
assert ran == ([4, 0, 0] if one else [0, 4, 4]), ran
""" % ((n, one),))


@pytest.mark.parametrize("nx,ny,bodies", [(300, 200, 1), (64, 48, 1), (420, 400, 9)])
def test_consecutive_tiles_of_a_step_share_an_xcd(stand_in, nx, ny, bodies):
    """Workgroup b runs on XCD b % 8: with BTDF_OPT_XCD_REMAP (the default)
    those of an XCD take a run of consecutive tiles, among the tiles with markers
    (which come first) and among the others; without it workgroups take the
    tiles in order. The option takes effect at any time, and moves no tile
    twice or none."""
    child(stand_in, """
nx, ny, bodies = %r
h = handle(nx, ny, [W.cylinder_body(20.0 + 40 * (i %% 3), 20.0 + 40 * (i // 3), 12.0, 38) for i in range(bodies)])
ntx = (nx + 31) // 32

def items():
    p = ctypes.POINTER(ctypes.c_int)()
    n = hip.host_hip_last_step(ctypes.byref(p))
    return np.ctypeslib.as_array(p, (n, 4)).copy()

def tiles(part):   # in the order of the lattice
    return [(t >> 16) * ntx + (t & 65535) for it in part for t in it[:2] if t >= 0]

plain = None
for remap in (None, 0, 1, 0):
    if remap is not None:
        api.btdf_set_option(h, _lib.OPT_XCD_REMAP, remap)
    api.btdf_step(h, 2)
    it = items()
    nf = int(np.sum(it[:, 3] > it[:, 2]))
    assert nf > 0 and np.all(it[:nf, 3] > it[:nf, 2])
    whole = []
    for first, last in ((0, nf), (nf, len(it))):
        if remap == 0:
            runs = [it[first:last]]
        else:
            runs = [it[[b for b in range(first, last) if b %% 8 == x]] for x in range(8)]
        order = [t for r in runs for t in tiles(r)]
        assert order == sorted(order), (remap, order)
        whole.append(order)
        assert remap == 0 or max(map(len, runs)) - min(map(len, runs)) <= 1
    plain = plain or whole
    assert whole == plain
assert np.all(steps_found()[:, 2] == ntx * ((ny + 7) // 8)) and not np.any(steps_found()[:, 3])
""" % ((nx, ny, bodies),))


@pytest.mark.parametrize("g,bodies,n,precision,records", [(106, 3, 200, 8, True), (106, 4, 200, 8, False),
                                                          (176, 2, 384, 8, False), (106, 5, 200, 8, True),
                                                          (54, 9, 64, 8, True), (106, 3, 200, 4, True)])
def test_matrices_that_fill_the_l2_keep_the_lattice_kernel(stand_in, g, bodies, n, precision, records):
    """(Bodies per row of a square of them.)"""
    child(stand_in, """
g, k, n, precision, records = %r
h = handle(k * g, k * g, [W.cylinder_body((i %% k + 0.5) * g, (i // k + 0.5) * g, 1.2 * n / np.pi, n)
                          for i in range(k * k)], precision, W.ROMA3)
api.btdf_set_option(h, _lib.OPT_FORCING_METHOD, 1)
api.btdf_step(h, 2)
ran = [hip.host_hip_launched(b) for b in (b"11step_kernel", b"10lbm_kernel")]
assert ran == ([2, 0] if records else [0, 2]), ran
""" % ((g, bodies, n, precision, records),))


@pytest.mark.parametrize("n,passes,whole", [(64, 2, True), (65, 2, False), (96, 3, True), (97, 3, False), (128, 4, True),
                                            (129, 9, False), (96, 1, True), (97, 1, False)])
def test_bodies_are_formed_whole_beside_a_blocked_pass(stand_in, n, passes, whole):
    """There a launch more costs more. (passes = 1: the implicit method.)"""
    child(stand_in, """
n, passes, whole = %r
h = handle(1100, 1000, [W.cylinder_body(500.0, 500.0, 1.2 * n / np.pi, n)], 4, W.ROMA3)
api.btdf_set_option(h, *((_lib.OPT_FORCING_METHOD, 1) if passes == 1 else (_lib.OPT_FORCING_PASSES, passes)))
assert api.btdf_get_option(h, _lib.OPT_STEPS_PER_PASS) == 5
api.btdf_step(h, 10)
ran = [hip.host_hip_launched(b) for b in (b"body_kernel", b"9ib_kernel")]
assert ran == ([10, 0] if whole else [0, 10]), ran
api.btdf_set_option(h, _lib.OPT_TEMPORAL_BLOCKING, 0)   # (and not without it)
api.btdf_step(h, 1)
ran = [hip.host_hip_launched(b) - k for b, k in zip((b"body_kernel", b"9ib_kernel"), ran)]
assert ran == ([1, 0] if n <= min(128, 80 if passes == 1 else 16 * passes + 32) else [0, 1]), ran
""" % ((n, passes, whole),))


@pytest.mark.parametrize("bodies,one", [(25, True), (121, False)])
def test_near_steps_of_many_tiles_take_two_launches(stand_in, bodies, one):
    """(25 bodies: some 190 tiles with markers, 121: some 900.)"""
    child(stand_in, """
bodies, one = %r
k = int(bodies ** 0.5)
g = 1600 / k
h = handle(1600, 1600, [W.cylinder_body((i %% k + 0.5) * g, (i // k + 0.5) * g, 24.0, 75) for i in range(bodies)], 4,
           W.ROMA3)
assert api.btdf_get_option(h, _lib.OPT_STEPS_PER_PASS) == 5
assert (api.btdf_get_option(h, _lib.OPT_FORCED_TILES) <= 600) == one
api.btdf_step(h, 10)
ran = [hip.host_hip_launched(b) for b in (b"11step_kernel", b"9ib_kernel")]
assert ran == ([10, 0] if one else [10, 10]), ran
""" % ((bodies, one),))


def test_forces_before_any_step_do_not_read_an_unwritten_workspace(stand_in):
    """A workspace is the caller's memory, whatever it holds: before the state
    is made there are no forces and no instability."""
    child(stand_in, """
h = handle(64, 48, [W.cylinder_body(30.0, 20.0, 8.0, 25)])
n = api.btdf_workspace_bytes(h)
ws = np.full(n + 256, 0xff, np.uint8)
at = -(-ws.ctypes.data // 256) * 256
api.btdf_bind_workspace(h, at, n)
assert not np.any(api.btdf_forces(h))
assert api.btdf_force_history(h, 0).shape[0] == 0
assert api.btdf_force_history(h, 10).shape[0] == 0
api.btdf_step(h, 3)
assert api.btdf_force_history(h, 10).shape == (3, 1, 3)
api.btdf_destroy(h)
""")
