"""GPU: the near-field grid where its cells hold many faces each, as on a surface that has shrunk since its
first mesh (the near radius stays): E and dE against FP64 pair terms, the same from call to call, and the
time of a grid of one cell."""
import time

import numpy as np
import pytest

from paper_2107_01664_amd import meshgen as mg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01664_amd import tpsurf
    tpsurf.lib()
    return tpsurf


@pytest.mark.parametrize("scale", [0.02, 0.08, 0.25, 0.5])
@pytest.mark.parametrize("nu,nv", [(13, 11), (62, 41)])
def test_shrunk(tp, nu, nv, scale):
    """286 and 5,084 faces, cells of all of them down to a few, runs on both sides of those that a lane takes
    by itself."""
    m = mg.add_noise(mg.torus(nu, nv, 1.0, 0.3), 1e-3, 3)
    V, F = torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()
    print(f"[near dense] faces {m.nF} scale {scale}", flush=True)
    with tp.Problem(V, F) as P, tp.Problem(scale * V, F, tp.default_params(precision=2)) as Q:
        P.set_vertices(scale * V)
        E, g = P.gradient()
        Ee = P.energy()
        P.set_vertices(scale * V)
        E2, g2 = P.gradient()
        assert E == E2 and torch.equal(g, g2) and P.energy() == Ee
        E0, g0 = Q.gradient()
    assert abs(E - E0) <= 1e-5 * E0 and abs(Ee - E0) <= 1e-5 * E0
    assert (g - g0).norm() <= 1e-5 * g0.norm()


def best(f):
    out = np.inf
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        out = min(out, time.perf_counter() - t)
    return out


def test_one_cell(tp):
    """32,000 faces in one cell: all pairs are near ones, and the grid is not what takes the time.
    Against row by row FP64, the kernel of near pairs alone is 2.6 times as long; with faces ordered and
    counted one by one the whole was 4.3 times, with parts of waves 2.7."""
    m = mg.torus(160, 100, 1.0, 0.3)
    V, F = torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()
    small = 0.02 * V
    with tp.Problem(V, F) as P, tp.Problem(V, F, tp.default_params(precision=2, sym_pairs=0)) as Q:
        def near():
            P.set_vertices(small)
            P.gradient()

        def direct():
            Q.set_vertices(small)
            Q.gradient()

        a, b = best(near), best(direct)
    print(f"[near dense] one cell {1e3 * a:.2f} ms, row by row FP64 {1e3 * b:.2f}", flush=True)
    assert a <= 3.3 * b
