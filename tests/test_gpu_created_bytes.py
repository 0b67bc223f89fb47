"""GPU: a problem without theta and chi holds no tree: what creation allocates is its mesh, its face data
and what sorts the faces."""
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


def test_no_tree_unasked(tp):
    """Per face of 40,000: mesh 24, face data 112 (and padding of 1 %), keys and order 28, sort space of at
    most 32.  The tree takes 250 more (nodes of eight faces: 240 bytes for every four)."""
    m = mg.torus(200, 100, 1.0, 0.3)
    V, F = torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()
    with tp.Problem(V, F) as P, tp.Problem(V, F, tp.default_params(theta=0.5)) as Q:
        held = P.device_bytes()
        assert held <= 200 * m.nF, held / m.nF
        assert Q.device_bytes() - held >= 250 * m.nF
        E, E0 = Q.energy(), P.energy()
        assert abs(E - E0) <= 0.05 * E0
