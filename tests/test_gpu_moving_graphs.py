"""Moving bodies under graph replay where rebuilding the tile lists changes how
many tiles a stencil touches, and so the length of a step's work list: the
results are the bits of two launches per step without graphs."""
import numpy as np
import pytest

import btdf_workloads as W

pytestmark = pytest.mark.gpu


def tiles_touched(x, y, D, n, nx, ny):
    """Tiles of 32 x 8 nodes that the 4-point stencils grown by the lists'
    margin of 3 nodes touch."""
    t = 2.0 * np.pi * np.arange(n) / n
    X, Y = x + 0.5 * D * np.cos(t), y + 0.5 * D * np.sin(t)
    hit = set()
    for a, b in zip(np.floor(X).astype(int), np.floor(Y).astype(int)):
        for i in range(a - 1 - 3, a + 3 + 3):
            for j in range(b - 1 - 3, b + 3 + 3):
                hit.add(((i % nx) // 32, (j % ny) // 8))
    return len(hit)


@pytest.mark.parametrize("precision", [4, 8])
@pytest.mark.parametrize("v", [(0.02, 0.01), (0.0, 0.02)])
def test_graphs_follow_work_lists_of_changing_length(v, precision):
    from paper_1806_09403_amd import Sim, _lib
    nx, ny, D, n = 300, 200, 12.0, 38
    counts = [tiles_touched(90.0 + v[0] * s, 100.0 + v[1] * s, D, n, nx, ny) for s in range(0, 400, 50)]
    print("tiles touched", counts, flush=True)
    assert max(counts) - min(counts) >= 2

    def run(**options):
        s = Sim(nx, ny, 0.75, W.COS4, 2.6, W.FULLY_PERIODIC, init=(1.0, 0.02, 0.0), precision=precision)
        for k, val in options.items():
            s.set_option(getattr(_lib, "OPT_" + k), val)
        b = W.cylinder_body(90.0, 100.0, D, n)
        s.add_body(b.xy, None, b.cx, b.cy, b.ds)
        s.set_body_motion(0, v[0], v[1], 0.003)
        for k in (37, 163, 200):
            s.step(k)
        r = (s.populations(), s.force_history(400), s.marker_positions(), *s.marker_data().values())
        s.close()
        return r

    want = run(LBM_VARIANT=0)
    for chunk in (0, 5, 8):
        for a, b in zip(run(LBM_VARIANT=6, GRAPH_CHUNK=chunk), want):
            assert np.array_equal(a, b), chunk
