"""GPU: the energy of more faces than the pairs of blocks that fit one dimension of a launch: its pairs
taken once against every ordered pair, for a mesh and for the same faces given by their quantities."""
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


@pytest.mark.parametrize("nu,nv", [(725, 512), (1250, 600)])
def test_energy(tp, nu, nv):
    """742,400 faces (4,206,450 pairs of blocks: more than the first dimension takes, a ragged rest) and
    1,500,000.  Both sums have FP32 pair terms, of 1e-5 at most each."""
    m = mg.torus(nu, nv, 1.0, 0.3)
    V, F = torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()
    E = []
    for kw in ({}, {"sym_pairs": 0}):
        print(f"[energy large] faces {m.nF} {kw}", flush=True)
        with tp.Problem(V, F, tp.default_params(**kw)) as P:
            E.append(P.energy())
    assert abs(E[0] - E[1]) <= 1e-5 * E[1]


def test_energy_faces(tp):
    m = mg.torus(1250, 600, 1.0, 0.3)
    c = torch.from_numpy(m.V).cuda()[torch.from_numpy(m.F).cuda().long()]
    N = torch.linalg.cross(c[:, 1] - c[:, 0], c[:, 2] - c[:, 0])
    X, a = c.mean(1), 0.5 * N.norm(dim=1)
    N = N / (2.0 * a[:, None])
    print(f"[energy large] given faces {m.nF}", flush=True)
    E, E0 = (tp.tp_energy_faces(X, N, a, tp.default_params(sym_pairs=q, precision=1)) for q in (-1, 0))
    assert abs(E - E0) <= 1e-5 * E0
