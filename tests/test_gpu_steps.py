"""The launches a step, a pass, a reversed step and a copy of the state are
made of, at the sizes where each can go wrong: lattices smaller than a tile
and its surroundings, one node past a tile, odd numbers of tiles; more markers
in a tile than one LDS chunk holds (64) and bodies around the size of a wave
and of a workgroup's share (256 markers); rows of odd width.

Against the oracle the bounds are those of the per-step parity tests (a few
ulps of values of order one over a handful of steps: 1e-14 for populations and
marker moments, 1e-12 relative for forces summed over markers; 1e-13 and 1e-10
where a matrix inverse enters; 1e-11 relative for gradients). Against another
route of the same library the results are the same bits.
"""
import numpy as np
import pytest

import btdf_workloads as W
from oracle.oracle import OracleSim

pytestmark = pytest.mark.gpu

WALLS_Y = (W.PERIODIC, W.PERIODIC, W.BOUNCEBACK_WALL, W.BOUNCEBACK_WALL)
INLET = (W.VELOCITY_INLET, W.ZERO_GRADIENT_OUTLET, W.BOUNCEBACK_WALL, W.BOUNCEBACK_WALL)


def log(msg):
    print(msg, flush=True)


def case(seed, nx, ny, kind, bc, bodies):
    """A lattice with bodies (centre as fractions of it, diameter, markers)."""
    c = W.random_case(seed, nx=nx, ny=ny, kind=kind, bc=bc, n_bodies=0)
    rng = np.random.default_rng(seed)
    for fx, fy, D, n in bodies:
        c.bodies.append(W.cylinder_body(fx * nx, fy * ny, D, n, rng.uniform(-0.02, 0.02, (n, 2))))
    return c


def oracle_of(c, nf=1, method=0):
    s = OracleSim(c.nx, c.ny, c.bc, c.tau, c.kind, c.thickening, c.G, c.inflow, c.init)
    for b in c.bodies:
        s.add_body(b.xy, b.uv, b.cx, b.cy, b.ds)
    ux, uy = c.init_fields()
    s.init_equilibrium(ux, uy, np.full((c.ny, c.nx), c.init[0]))
    if nf > 1:
        s.set_forcing_passes(nf)
    if method:
        s.set_forcing_method(method)
    return s


def gpu_of(c, precision=8, **options):
    from paper_1806_09403_amd import Sim, _lib
    s = Sim.from_case(c, precision=precision)
    for k, v in options.items():
        s.set_option(getattr(_lib, "OPT_" + k), v)
    return s


def agree(o, g, step, pop=1e-14, force=1e-12):
    assert o.unstable == 0, step
    assert np.max(np.abs(g.populations() - o.populations())) < pop, step
    mo, mg = o.marker_data(), g.marker_data()
    scale = max(1e-300, np.max(np.abs(mo["Fx"])) + np.max(np.abs(mo["Fy"])))
    for k in ("Fx", "Fy"):
        assert np.max(np.abs(mg[k] - mo[k])) < force * scale, (step, k)
    Fo, Fg = o.forces(), g.forces()
    assert np.max(np.abs(Fg - Fo)) < force * max(1e-300, np.max(np.abs(Fo))), step


def results(s, steps):
    """Everything a run leaves behind (the history once: a read consumes it)."""
    return dict(s.marker_data(), populations=s.populations(), history=s.force_history(steps))


def same(a, b):
    assert a.keys() == b.keys()
    for k in a:
        assert np.array_equal(a[k], b[k]), k


# (seed, nx, ny, kind, bc, bodies): one tile is 32 x 8 nodes
STEP_CASES = [
    (1, 8, 8, W.ROMA3, W.FULLY_PERIODIC, [(0.5, 0.5, 3.0, 9)]),          # a stencil meets a tile across both edges
    (2, 13, 11, W.COS4, W.FULLY_PERIODIC, [(0.1, 0.9, 4.0, 70)]),        # one marker more than a chunk and some
    (3, 33, 9, W.PESKIN4, W.FULLY_PERIODIC, [(0.99, 0.5, 3.0, 64)]),     # a tile of one column; a full chunk
    (4, 41, 25, W.COS4, W.FULLY_PERIODIC, [(0.5, 0.5, 8.0, 200)]),       # several chunks in a tile
    (5, 64, 24, W.LINEAR2, WALLS_Y, [(0.5, 0.5, 7.0, 30), (0.02, 0.4, 5.0, 20)]),
    (6, 65, 31, W.ROMA3, INLET, [(0.4, 0.5, 8.0, 65)]),                  # the outlet's columns in two tiles
    (7, 66, 40, W.COS4, W.FAR_FIELD, [(0.5, 0.5, 9.0, 40)]),
    (8, 97, 40, W.ROMA3, W.FAR_FIELD, [(0.5, 0.5, 9.0, 129)]),           # the ghost column alone in a tile
]


@pytest.mark.parametrize("seed,nx,ny,kind,bc,bodies", STEP_CASES)
def test_steps_match_the_oracle(seed, nx, ny, kind, bc, bodies):
    log("step launches %dx%d kind=%d" % (nx, ny, kind))
    c = case(seed, nx, ny, kind, bc, bodies)
    o, g = oracle_of(c), gpu_of(c)
    for step in range(5):
        o.step(1)
        g.step(1)
        agree(o, g, step)
    g.close()


@pytest.mark.parametrize("precision", [4, 8])
@pytest.mark.parametrize("seed,nx,ny,kind,bc,bodies", STEP_CASES)
def test_one_launch_and_two_launch_steps_are_the_same_bits(seed, nx, ny, kind, bc, bodies, precision):
    """Launch shape 6 takes a step in one launch, shape 0 in two; NF > 1 hands
    the tiles marker records; graphs chain the steps' force sums."""
    c = case(seed, nx, ny, kind, bc, bodies)
    for nf in (1, 3):
        ref = gpu_of(c, precision, LBM_VARIANT=0, FORCING_PASSES=nf)
        ref.step(11)
        want = results(ref, 11)
        ref.close()
        for chunk in (0, 4):
            g = gpu_of(c, precision, LBM_VARIANT=6, FORCING_PASSES=nf, GRAPH_CHUNK=chunk)
            g.step(1)
            g.step(10)
            same(results(g, 11), want)
            g.close()


@pytest.mark.parametrize("n", [63, 64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("nf,method", [(3, 0), (1, 1)])
def test_bodies_of_every_size_match_the_oracle(n, nf, method):
    """Forcing passes and the implicit method body by body: one workgroup per
    body up to 256 markers, the general launches beyond."""
    D = 1.2 * n / np.pi
    nx, ny = int(D) + 25, int(D) + 18
    log("bodies of %d markers nf=%d method=%d on %dx%d" % (n, nf, method, nx, ny))
    c = case(20 + n, nx, ny, W.ROMA3, W.FULLY_PERIODIC, [(0.55, 0.45, D, n)])
    o = oracle_of(c, nf, method)
    g = gpu_of(c, 8, FORCING_PASSES=nf, FORCING_METHOD=method)
    for step in range(3):
        o.step(1)
        g.step(1)
        agree(o, g, step, *((1e-13, 1e-10) if method else (1e-14, 1e-12)))
    g.close()


@pytest.mark.parametrize("gap", [1.0, 3.0, 9.0])
def test_passes_of_bodies_near_each_other_match_the_oracle(gap):
    """Bodies whose stencils meet take their passes together."""
    D = 10.0
    c = case(31, 70, 41, W.COS4, W.FULLY_PERIODIC, [(0.3, 0.5, D, 32), (0.3 + (D + gap) / 70, 0.5, D, 32)])
    o, g = oracle_of(c, 4), gpu_of(c, 8, FORCING_PASSES=4)
    for step in range(4):
        o.step(1)
        g.step(1)
        agree(o, g, step)
    g.close()


@pytest.mark.parametrize("precision", [4, 8])
@pytest.mark.parametrize("bc", [W.FULLY_PERIODIC, WALLS_Y])
def test_moving_bodies_in_one_and_two_launches_are_the_same_bits(bc, precision):
    """A one-launch step leaves the next step's places in the second of two
    sets: odd and even runs, past a rebuild of the tile lists, beside a body at
    rest whose velocities change between runs, in graphs and timed."""
    c = case(35, 90, 61, W.COS4, bc, [(0.3, 0.5, 12.0, 40), (0.7, 0.45, 9.0, 300), (0.55, 0.7, 5.0, 16)])
    uv = np.random.default_rng(7).uniform(-0.01, 0.01, (300, 2))

    def run(timed=False, **options):
        s = gpu_of(c, precision, **options)
        s.set_body_motion(0, 0.02, 0.011, 0.004)
        s.set_body_motion(2, -0.013, 0.004, -0.006)
        for k, n in enumerate((1, 2, 1, 7, 60)):
            s.step_timed(n) if timed else s.step(n)
            if k == 2:
                s.set_marker_velocity(1, uv)
        r = dict(results(s, 71), xy=s.marker_positions(), states=np.array([s.body_state(b) for b in range(3)]))
        s.close()
        return r

    want = run(LBM_VARIANT=0)
    for chunk in (0, 4, 5):
        same(run(LBM_VARIANT=6, GRAPH_CHUNK=chunk), want)
    same(run(timed=True, LBM_VARIANT=6), want)


@pytest.mark.parametrize("precision,depth", [(4, 5), (4, 4), (8, 3)])
@pytest.mark.parametrize("bc", [W.FULLY_PERIODIC, W.FAR_FIELD, INLET])
def test_passes_beside_the_near_tiles_are_the_same_bits(bc, precision, depth):
    """Large groups beside the steps of the tiles near bodies and edges, with
    every remainder of steps, in and out of graphs."""
    c = case(41, 420, 300, W.COS4, bc, [(0.3, 0.5, 21.0, 66), (0.6, 0.3, 12.0, 100)])
    steps = 3 * depth + 2
    ref = gpu_of(c, precision, TEMPORAL_BLOCKING=0)
    ref.step(steps)
    want = results(ref, steps)
    ref.close()
    for chunk in (0, depth, 2 * depth):
        g = gpu_of(c, precision, TEMPORAL_BLOCKING=depth, EDGE_TILES=0, GRAPH_CHUNK=chunk)
        g.step(1)
        g.step(steps - 1)
        same(results(g, steps), want)
        g.close()


@pytest.mark.parametrize("precision", [4, 8])
@pytest.mark.parametrize("nx,ny,align", [(8, 9, 0), (31, 10, 0), (32, 8, 128), (33, 11, 128), (129, 12, 256)])
def test_populations_in_and_out(nx, ny, align, precision):
    """Every value lands where it belongs, through the host and through device
    memory at any 8-byte offset; the stored deviations are exact to the type."""
    import torch
    from paper_1806_09403_amd import Sim, _lib
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
    f = w[:, None, None] * (1.0 + np.random.default_rng(nx).uniform(-0.05, 0.05, (9, ny, nx)))
    # deviations up to 0.05 * 4/9 < 2^-5, rounded to 24 bits; values below 1/2 to 53 bits, twice
    bound = 2.0 ** -53 + (2.0 ** -5 * 2.0 ** -24 if precision == 4 else 2.0 ** -53)
    s = Sim(nx, ny, 0.8, W.ROMA3, 1.9, W.FULLY_PERIODIC, precision=precision)
    s.set_option(_lib.OPT_ROW_ALIGN, align)
    s.set_populations(f)
    got = s.populations()
    assert np.max(np.abs(got - f)) <= bound
    for shift in (0, 1):
        buf = torch.full((9 * ny * nx + 2,), -7.0, dtype=torch.float64, device="cuda")
        out = buf[shift:shift + 9 * ny * nx].view(9, ny, nx)
        s.populations_to(out)
        assert np.array_equal(out.cpu().numpy(), got)
        rest = buf.cpu().numpy()
        assert np.all(rest[:shift] == -7.0) and np.all(rest[shift + 9 * ny * nx:] == -7.0)
        t = Sim(nx, ny, 0.8, W.ROMA3, 1.9, W.FULLY_PERIODIC, precision=precision)
        t.set_populations_from(out)
        assert np.max(np.abs(t.populations() - got)) <= bound
        t.close()
    s.close()


@pytest.mark.parametrize("n", [3, 127, 128, 129, 300])
def test_marker_velocities_take_effect_at_the_next_step(n):
    """Small sets travel with a launch, larger ones by a copy. Replaced before
    any step: the same bits as a body that had the last set from the start.
    Replaced between steps, back to back: the oracle's steps (but for three
    markers 14.7 nodes apart, whose force overshoots fifteenfold every step
    and the last bit with it)."""
    rng = np.random.default_rng(n)
    uv = [rng.uniform(-0.02, 0.02, (n, 2)) for _ in range(3)]
    c = case(50, 61, 47, W.COS4, W.FULLY_PERIODIC, [(0.4, 0.5, 14.0, n)])
    c.bodies[0].uv = uv[0]
    g, o = gpu_of(c), oracle_of(c)
    for k in range(3):
        if k:
            g.set_marker_velocity(0, uv[k - 1])  # (replaced before any step)
            g.set_marker_velocity(0, uv[k])
            o.set_marker_velocity(0, uv[k])
        if n > 3:
            g.step(1)
            o.step(1)
            agree(o, g, k)
    g.close()
    g = gpu_of(c)
    g.set_marker_velocity(0, uv[1])
    g.set_marker_velocity(0, uv[2])
    c.bodies[0].uv = uv[2]
    ref = gpu_of(c)
    for s in (g, ref):
        s.step(1)
    same(results(g, 1), results(ref, 1))
    g.close()
    ref.close()


@pytest.mark.parametrize("before", [0, 4000, 4090])
def test_force_history_of_every_length(before):
    """Rows come back in order whatever the lengths of the calls that made
    them and of those that read them, also where the ring of 4096 rows wraps."""
    c = case(60, 48, 40, W.ROMA3, W.FULLY_PERIODIC, [(0.3, 0.5, 8.0, 25), (0.7, 0.5, 8.0, 25)])
    ref, g = gpu_of(c), gpu_of(c, GRAPH_CHUNK=8)
    for s in (ref, g):
        if before:
            s.step(before)
            assert s.force_history(before).shape == (before, 2, 3)
    ref.step(100)
    want = ref.force_history(100)
    assert want.shape == (100, 2, 3)
    done = 0
    for k in (1, 2, 7, 30, 60):
        g.step(k)
        assert np.array_equal(g.forces(), want[done + k - 1])
        got = [g.force_history(m) for m in (1, k // 2 + 1, k)]  # (the last what is left)
        assert np.array_equal(np.concatenate(got), want[done:done + k])
        done += k
    g.close()
    ref.close()


# (one adjoint tile is 64 x 4 nodes)
@pytest.mark.parametrize("seed,nx,ny,kind,bc,bodies,n", [
    (71, 12, 9, W.ROMA3, W.FULLY_PERIODIC, [(0.5, 0.5, 3.0, 9)], 4),                       # every tile is touched
    (72, 65, 21, W.COS4, W.FULLY_PERIODIC, [(0.01, 0.5, 6.0, 100)], 5),                    # over 64 markers in a tile
    (73, 66, 24, W.PESKIN4, WALLS_Y, [(0.5, 0.5, 6.0, 16), (0.1, 0.5, 5.0, 17)], 4),       # 33 markers: a last group of one
    (74, 130, 30, W.COS4, INLET, [(0.4, 0.5, 8.0, 48)], 5),
    (75, 40, 18, W.LINEAR2, W.FULLY_PERIODIC, [], 3),                                      # no markers at all
])
def test_reversed_steps_match_the_oracle(seed, nx, ny, kind, bc, bodies, n):
    log("reversed steps %dx%d kind=%d" % (nx, ny, kind))
    c = case(seed, nx, ny, kind, bc, bodies)
    hbar = np.random.default_rng(seed).standard_normal((n, len(bodies), 3))
    go = oracle_of(c).adjoint(n, hbar)
    s = gpu_of(c)
    gg, _ = s.adjoint(n, hbar)
    for gk, ok in (("populations", "populations"), ("inflow", "inflow"), ("body_force", "body_force"),
                   ("marker_xy", "xy"), ("marker_uv", "uv"), ("centres", "centres")):
        ref, got = go[ok], gg[gk]
        assert got.shape == ref.shape, gk
        scale = np.max(np.abs(ref), initial=0.0)
        assert np.max(np.abs(got - ref), initial=0.0) <= 1e-11 * scale + 1e-300, gk
    s.close()


@pytest.mark.parametrize("precision", [4, 8])
def test_reversed_steps_of_a_lattice_of_many_tiles(precision):
    """Above 28 000 tiles those no stencil touches have launches of their own.
    A strip of 64 x 112 400 nodes (28 100 tiles) at rest but for a body: within
    its reach the gradients are those of a strip of 64 x 64, beyond it zero."""
    from paper_1806_09403_amd import Sim
    n = 3
    rng = np.random.default_rng(81)
    uv, hbar = rng.uniform(-0.02, 0.02, (25, 2)), rng.standard_normal((n, 1, 3))
    b = W.cylinder_body(30.3, 31.7, 8.0, 25)
    grads = []
    for ny in (64, 112400):
        s = Sim(64, ny, 0.8, W.COS4, 2.6, W.FULLY_PERIODIC, init=(1.0, 0.02, 0.01), precision=precision)
        s.add_body(b.xy, uv, b.cx, b.cy, b.ds)
        g, _ = s.adjoint(n, hbar)
        s.close()
        grads.append(g)
    small, large = grads
    assert np.any(small["populations"])
    assert np.array_equal(large["populations"][:, :64], small["populations"])
    assert not np.any(large["populations"][:, 64:])
    for k in ("body_force", "marker_xy", "marker_uv", "centres"):
        assert np.array_equal(large[k], small[k]), k
