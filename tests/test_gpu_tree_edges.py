"""GPU: the tree's build and walk at their edges, against the oracle's tree: a root that is a leaf,
leaves of one face, leaves and waves that end early, as many leaves as one workgroup of the build
takes, one more, several levels above the subtrees, exponents that are not 6 and 12."""
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


@pytest.mark.parametrize("prec", [2, 3])
@pytest.mark.parametrize("n,leaf,ab", [
    (0, 64, (6.0, 12.0)),      # 20 faces, one leaf
    (2, 1, (6.0, 12.0)),       # 320 leaves of one face: two subtrees
    (2, 3, (6.0, 12.0)),       # 107 leaves, the last of two faces
    (3, 5, (4.5, 10.0)),       # 1,280 faces, 256 leaves
    (3, 4, (6.0, 12.0)),       # 320 leaves
    (4, 1, (6.0, 12.0)),       # 5,120 leaves: 32 subtrees
    (4, 33, (4.5, 10.0)),      # 156 leaves
])
def test_tree_edges(tp, n, leaf, ab, prec):
    m = mg.add_noise(mg.icosphere(n), 0.02 / 2 ** n, n + 1)
    print(f"[tree] faces {m.nF} leaf {leaf} exponents {ab} precision {prec}", flush=True)
    E0, g0, terms = O.bh_gradient(m.V, m.F, 0.5, leaf=leaf, alpha=ab[0], beta=ab[1])
    p = tp.default_params(precision=prec, theta=0.5, leaf_size=leaf, alpha=ab[0], beta=ab[1])
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), p) as P:
        E, g = P.gradient()
        assert tuple(P.bh_stats()) == tuple(terms)
        assert P.energy() == E
    # rounding of the terms: 2^-52 and 2^-24 times the condition of a term (the powers of a
    # difference of positions: under 1e2 here) and of the sum
    tE, tG = (1e-12, 1e-10) if prec == 2 else (1e-5, 1e-5)
    assert abs(E - E0) <= tE * E0
    assert np.linalg.norm(g.cpu().numpy() - g0) <= tG * np.linalg.norm(g0)


@pytest.mark.parametrize("prec,tol", [(2, 1e-12), (3, 1e-5)])
@pytest.mark.parametrize("leaf,k", [(1, 1), (1, 9), (2, 5), (3, 3)])
def test_long_exact_lists(tp, leaf, k, prec, tol):
    """Nothing is admissible: every leaf's exact list holds all leaves, 1,280 (three parts), 640 (two)
    and 427 (one) of them, and the hierarchical product is the direct one."""
    m = mg.add_noise(mg.icosphere(3), 0.002, 2)
    u = mg.random_columns(m.nV, k, 3)
    print(f"[lists] leaf {leaf} columns {k} precision {prec}", flush=True)
    ref = O.fractional_apply(m.V, m.F, u)
    p = tp.default_params(precision=prec, chi=1e-9, leaf_size=leaf)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), p) as P:
        y = P.fractional_apply(torch.from_numpy(u).cuda()).cpu().numpy()
        assert P.bct_stats() == (0, (-(-m.nF // leaf)) ** 2)
    assert np.linalg.norm(y - ref) <= tol * np.linalg.norm(ref)
