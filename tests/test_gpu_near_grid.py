"""GPU: the near-field grid's build where it has edges: one cell, runs of very different lengths,
more problems in a batch than one launch takes."""
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


def dented():
    """A sphere whose northern cap is drawn together: hundreds of its faces share a cell."""
    m = mg.geodesic_sphere(18)
    s = np.where(m.V[:, 2] > 0.5, 0.15 + 0.85 * (1.0 - m.V[:, 2]) / 0.5, 1.0)
    m.V[:, :2] *= s[:, None]
    return mg.add_noise(m, 1e-4, 5)


MESHES = {
    "one_cell": lambda: mg.add_noise(mg.icosahedron(), 0.02, 3),
    "ragged": lambda: mg.add_noise(mg.torus(41, 19, 1.0, 0.3), 0.002, 6),
    "dense_cap": dented,
}


@pytest.mark.parametrize("name", list(MESHES))
def test_near_field(tp, name):
    """E and dE with the FP64 near field against the oracle, at the tolerance of FP32 pair terms."""
    m = MESHES[name]()
    print(f"[near grid] {name} faces {m.nF}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as P:
        E, dE = P.gradient()
        E1 = P.energy()
        E2, dE2 = P.gradient()
    assert E == E2 and torch.equal(dE, dE2)
    E0, dE0 = O.gradient(m.V, m.F)
    assert abs(E - E0) <= 1e-5 * E0 and abs(E1 - E0) <= 1e-5 * E0
    assert np.linalg.norm(dE.cpu().numpy() - dE0) <= 1e-5 * np.linalg.norm(dE0)


def test_seventeen_grids_in_a_batch(tp):
    """Seventeen problems take two launches per phase of the build; each steps as it does alone."""
    meshes = [mg.add_noise(mg.geodesic_sphere(3 + q % 4), 0.01, q) for q in range(17)]
    out = []
    for together in (True, False):
        probs = [tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) for m in meshes]
        if together:
            sts, _ = tp.batch_step(probs)
            assert sts == [0] * 17
        else:
            for P in probs:
                P.step()
        out.append([P.vertices().cpu().numpy() for P in probs])
        for P in probs:
            P.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
