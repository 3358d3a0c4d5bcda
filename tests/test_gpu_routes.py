"""Rules that send the same work to one kernel or another: on both sides of
each the results are the same bits."""
import numpy as np
import pytest

import btdf_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [4, 8])
@pytest.mark.parametrize("n,far,passes", [(31, (64, 65), 2), (64, (96, 97), 4), (100, (128, 129), 6), (17, (80, 81), 1),
                                          (50, (63, 100), 1)])
def test_bodies_formed_whole_or_by_launches_over_all_markers(n, far, passes, precision):
    """A far body of one marker more changes the kernels that form the forces
    of a first one (passes = 1: the implicit method), whose first steps, before
    the far one's flow reaches it, do not change by a bit."""
    from paper_1806_09403_amd import Sim, _lib
    out = []
    for m in far:
        s = Sim(260, 90, 0.8, W.ROMA3, 1.9, W.FULLY_PERIODIC, init=(1.0, 0.02, 0.01), precision=precision)
        for x, k in ((50.3, n), (190.6, m)):
            b = W.cylinder_body(x, 45.2, 1.2 * k / np.pi, k, np.random.default_rng(k).uniform(-0.01, 0.01, (k, 2)))
            s.add_body(b.xy, b.uv, b.cx, b.cy, b.ds)
        s.set_option(*((_lib.OPT_FORCING_METHOD, 1) if passes == 1 else (_lib.OPT_FORCING_PASSES, passes)))
        s.step(7)
        d = s.marker_data()
        out.append([s.populations()[:, :, :100], s.force_history(7)[:, 0]] + [v[:n] for v in d.values()])
        s.close()
    assert np.any(out[0][1])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision,depth", [(4, 5), (4, 4), (8, 3)])
def test_passes_beside_the_near_tiles_with_every_remainder(precision, depth):
    """Runs of depth .. 2 depth - 1 steps (one pass and each number of steps left
    over, of two and three in passes of their own) and timed runs, which take
    the same groups in turn, against single steps."""
    from paper_1806_09403_amd import Sim, _lib

    def run(blocking, go):
        s = Sim(420, 300, 0.8, W.COS4, 2.6, W.FAR_FIELD, inflow=(0.03, 0.0), init=(1.0, 0.02, 0.0), precision=precision)
        s.set_option(_lib.OPT_TEMPORAL_BLOCKING, blocking)
        s.set_option(_lib.OPT_EDGE_TILES, 0)
        for x, y, D, n in ((126.3, 150.2, 21.0, 66), (250.7, 90.4, 12.0, 100)):
            b = W.cylinder_body(x, y, D, n)
            s.add_body(b.xy, None, b.cx, b.cy, b.ds)
        out = []
        for n in range(depth, 2 * depth):
            getattr(s, go)(n)
            out += [s.populations(), s.force_history(n), *s.marker_data().values()]
        s.close()
        return out

    want = run(0, "step")
    for go in ("step", "step_timed_pass", "step_timed_split"):
        for a, b in zip(run(depth, go), want):
            assert np.array_equal(a, b), go


@pytest.mark.parametrize("precision,bodies", [(4, 49), (4, 121), (8, 121)])
def test_near_steps_in_one_and_two_launches_beside_a_pass(precision, bodies):
    """Few tiles with markers take a near step in one launch, more than 600 in
    two: both as single steps without a pass, in and out of graphs."""
    from paper_1806_09403_amd import Sim, _lib
    k = int(bodies ** 0.5)

    def run(blocking, chunk):
        s = Sim(1210, 1100, 0.8, W.ROMA3, 1.9, W.FULLY_PERIODIC, init=(1.0, 0.02, 0.01), precision=precision)
        s.set_option(_lib.OPT_TEMPORAL_BLOCKING, blocking)
        s.set_option(_lib.OPT_GRAPH_CHUNK, chunk)
        for i in range(bodies):
            b = W.cylinder_body((i % k + 0.5) * 1210 / k, (i // k + 0.5) * 1100 / k, 24.0, 75,
                                np.random.default_rng(i).uniform(-0.01, 0.01, (75, 2)))
            s.add_body(b.xy, b.uv, b.cx, b.cy, b.ds)
        assert (s.get_option(_lib.OPT_FORCED_TILES) > 600) == (bodies > 100)
        s.step(32)
        r = (s.populations(), s.force_history(32), *s.marker_data().values())
        s.close()
        return r

    want = run(0, 0)
    for chunk in (0, 15):
        for a, b in zip(run(1, chunk), want):
            assert np.array_equal(a, b), chunk


@pytest.mark.parametrize("nx,ny,precision", [(1400, 1200, 4), (1500, 1300, 4), (1000, 800, 8), (1100, 900, 8)])
def test_gradients_recomputed_in_one_and_two_launches(nx, ny, precision):
    """Up to 128 MB of populations a segment is recomputed in one launch a step,
    beyond in two: both give the gradients of the run that keeps every state."""
    from paper_1806_09403_amd import Sim
    n, grads = 7, []
    for every in (3, n):
        s = Sim(nx, ny, 0.8, W.ROMA3, 1.9, W.CHANNEL, inflow=(0.03, 0.0), init=(1.0, 0.03, 0.0), precision=precision)
        b = W.cylinder_body(0.3 * nx + 0.2, 0.5 * ny, 30.0, 94)
        s.add_body(b.xy, np.random.default_rng(5).uniform(-0.01, 0.01, (94, 2)), b.cx, b.cy, b.ds)
        grads.append(s.adjoint(n, np.random.default_rng(6).standard_normal((n, 1, 3)), every)[0])
        s.close()
    assert np.any(grads[0]["marker_uv"])
    for k in grads[0]:
        assert np.array_equal(grads[0][k], grads[1][k]), k
