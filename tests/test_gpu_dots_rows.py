"""GPU: the sum over splits of the row by row energy with the FP64 near field as its last slice, at the
edges of its chunks: chunks of faces that are empty, hold one face, or more than a wave takes at once.
(By default the energy of a mesh takes every pair once, at any size, and so another sum.)"""
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


@pytest.mark.parametrize("nu,nv", [(8, 8), (16, 8), (17, 8), (129, 64), (130, 127)])
def test_row_by_row_with_near_field(tp, nu, nv):
    """128, 256, 272, 16,512 and 33,020 faces: E against the oracle (FP32 far pairs: 1e-5) and the same
    from call to call; E + dE row by row agrees with it."""
    m = mg.add_noise(mg.torus(nu, nv, 1.0, 0.3), 1e-4, nu)
    print(f"[dots rows] faces {m.nF}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(),
                    tp.default_params(precision=3, sym_pairs=0)) as P:
        E = P.energy()
        Eg, _ = P.gradient()
        assert P.energy() == E
    E0 = O.energy(m.V, m.F)
    assert abs(E - E0) <= 1e-5 * E0 and abs(Eg - E0) <= 1e-5 * E0
