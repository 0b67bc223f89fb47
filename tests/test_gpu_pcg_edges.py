"""GPU: the persistent preconditioned Poisson solve where its layout has edges: a block alone,
ragged blocks, rows longer than the entries kept on chip whose neighbours do not all fit the
block's halo, blocks that touch so many aggregates that the coarse values of nine columns no
longer fit one batch, several components, every number of columns a thread can own."""
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


def bipyramid(n):
    """Two apices of degree n over a wavy rim."""
    a = np.arange(n) * 2.0 * np.pi / n
    V = np.concatenate([np.stack([np.cos(a), np.sin(a), 0.1 * np.sin(3.0 * a)], 1), [[0, 0, 1.0], [0, 0, -1.0]]])
    i = np.arange(n)
    F = np.concatenate([np.stack([i, (i + 1) % n, np.full(n, n)], 1), np.stack([(i + 1) % n, i, np.full(n, n + 1)], 1)])
    return mg.Mesh(V, F.astype(np.int32))


MESHES = {
    "one_block": lambda: mg.add_noise(mg.icosahedron(), 0.02, 3),
    "ragged_sphere": lambda: mg.add_noise(mg.geodesic_sphere(16), 0.002, 4),      # 21 blocks of 122
    "components": lambda: mg.linked_tori(40, 23, 1.0, 0.25, 1.0),
    "degree_40": lambda: bipyramid(40),
    "degree_600": lambda: bipyramid(600),                                          # halo beyond its capacity
}


@pytest.mark.parametrize("k", [1, 4, 5, 8, 9])
@pytest.mark.parametrize("name", list(MESHES))
def test_poisson_edges(tp, name, k):
    """The true relative residual, recomputed with the oracle's matrix, meets the solver's 1e-10 up
    to the rounding of the recomputation (eps |C||x| / |b|), and the solution is the oracle's
    within the residual times the norm of the inverse."""
    m = MESHES[name]()
    b = mg.random_columns(m.nV, k, 10 + k)
    print(f"[pcg edges] {name} k={k} vertices {m.nV}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as P:
        x, rep = P.poisson_solve(torch.from_numpy(b).cuda())
    x = x.cpu().numpy()
    C = O.cotan_laplacian(m.V, m.F)
    _, labels = O.components(m.F, m.nV)
    Pb = O.project_mean_zero(b, labels)
    nb = np.linalg.norm(Pb, axis=0)
    lam = np.linalg.eigvalsh(C.toarray())
    lmin, lmax = lam[lam > 1e-9 * lam[-1]][0], lam[-1]
    r = np.linalg.norm(Pb - C @ x, axis=0)
    rounding = 64 * np.finfo(float).eps * lmax * np.linalg.norm(x, axis=0)
    assert (r <= 1.0001e-10 * nb + rounding).all(), (r / nb, rounding / nb)
    x0 = O.poisson_solve(C, b, labels)
    err = np.linalg.norm(x - x0, axis=0)
    assert (err <= (1.0001e-10 * nb + 2 * rounding) / lmin).all(), (err, nb / lmin)
    assert rep.cg_iters[0] <= 400
