"""GPU: E + dE in FP64 with every unordered pair once, where its blocks have edges: a part of one
block, a whole one, one face more, several with a remainder; general exponents; the sizes on both
sides of where it begins."""
import numpy as np
import pytest

import oracle as O
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


def grad(tp, m, **kw):
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), tp.default_params(precision=2, **kw)) as P:
        E, g = P.gradient()
        E2, g2 = P.gradient()
    assert E == E2 and torch.equal(g, g2)
    return E, g.cpu().numpy()


# 2^-53 times the terms' condition (powers of a difference of positions, under 1e3) and a sum's length
TOL = 1e-11


@pytest.mark.parametrize("ab", [(6.0, 12.0), (4.5, 10.0)])
@pytest.mark.parametrize("nu,nv", [(3, 3), (16, 8), (43, 3), (19, 17), (40, 21)])
def test_symmetric_fp64(tp, nu, nv, ab):
    """18, 256, 258, 646 and 1,680 faces against the oracle."""
    m = mg.add_noise(mg.torus(nu, nv, 1.0, 0.3), 1e-3, nu)
    print(f"[grad64] faces {m.nF} exponents {ab}", flush=True)
    E, g = grad(tp, m, sym_pairs=1, alpha=ab[0], beta=ab[1])
    E0, g0 = O.gradient(m.V, m.F, alpha=ab[0], beta=ab[1])
    assert abs(E - E0) <= TOL * E0
    assert np.linalg.norm(g - g0) <= TOL * np.linalg.norm(g0)


@pytest.mark.parametrize("nu,nv", [(73, 70), (74, 70), (128, 65)])
def test_both_sides_of_the_rule(tp, nu, nv):
    """10,220 faces (row by row), 10,360 and 16,640: the default against row by row."""
    m = mg.add_noise(mg.torus(nu, nv, 1.0, 0.3), 1e-4, nu)
    print(f"[grad64] faces {m.nF}", flush=True)
    E, g = grad(tp, m)
    E0, g0 = grad(tp, m, sym_pairs=0)
    assert abs(E - E0) <= TOL * E0
    assert np.linalg.norm(g - g0) <= TOL * np.linalg.norm(g0)
