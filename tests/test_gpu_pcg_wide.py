"""GPU: the Poisson solve of more blocks than workgroups that are resident at once, where its layout
changes: two and four blocks per workgroup, a last workgroup that is not full, column groups that are
not full, rows longer than the entries kept on chip, more blocks than the persistent form takes."""
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


def globe(nu, nv):
    """A sphere of nv rings of nu vertices between two poles of degree nu."""
    th = np.pi * (np.arange(nv) + 1.0) / (nv + 1.0)
    ph = 2.0 * np.pi * np.arange(nu) / nu
    V = np.stack([np.outer(np.sin(th), np.cos(ph)), np.outer(np.sin(th), np.sin(ph)),
                  np.repeat(np.cos(th)[:, None], nu, 1)], 2).reshape(-1, 3)
    V = np.concatenate([V, [[0, 0, 1.0], [0, 0, -1.0]]])
    i, j = np.meshgrid(np.arange(nu), np.arange(nv - 1))
    a, b = (j * nu + i).ravel(), (j * nu + (i + 1) % nu).ravel()
    k = np.arange(nu)
    F = np.concatenate([np.stack([a, a + nu, b], 1), np.stack([b, a + nu, b + nu], 1),
                        np.stack([k, (k + 1) % nu, np.full(nu, nu * nv)], 1),
                        np.stack([(nv - 1) * nu + (k + 1) % nu, (nv - 1) * nu + k, np.full(nu, nu * nv + 1)], 1)])
    return mg.Mesh(V, F.astype(np.int32))


@pytest.mark.parametrize("name,make,k", [
    ("globe", lambda: globe(190, 190), 2),                       # 36,102 vertices, 283 blocks, rows of 191
    ("sphere_64", lambda: mg.geodesic_sphere(64), 4),            # 40,962: 321 blocks, columns 3 + 1
    ("sphere_82", lambda: mg.geodesic_sphere(82), 1),            # 67,242: 526 blocks
    ("sphere_82", lambda: mg.geodesic_sphere(82), 5),            # columns 3 + 2
    ("sphere_115", lambda: mg.geodesic_sphere(115), 3),          # 132,252: 1,034 blocks, launch by launch
])
def test_poisson_many_blocks(tp, name, make, k):
    """The true relative residual, recomputed with the oracle's matrix, meets the solver's 1e-10 up
    to the rounding of the recomputation (eps |C||x| / |b|, eight terms a row), and the solution is
    mean-zero."""
    m = make()
    b = mg.random_columns(m.nV, k, 20 + k)
    print(f"[pcg wide] {name} k={k} vertices {m.nV}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as P:
        x, rep = P.poisson_solve(torch.from_numpy(b).cuda())
        x2, _ = P.poisson_solve(torch.from_numpy(b).cuda())
    assert torch.equal(x, x2)
    x = x.cpu().numpy()
    C = O.cotan_laplacian(m.V, m.F)
    _, labels = O.components(m.F, m.nV)
    Pb = O.project_mean_zero(b, labels)
    nb = np.linalg.norm(Pb, axis=0)
    r = np.linalg.norm(Pb - C @ x, axis=0)
    noise = 8 * 2.0 ** -52 * np.linalg.norm(abs(C) @ abs(x), axis=0)
    assert np.all(r <= 1e-10 * nb * (1 + 1e-6) + noise), (r / nb, noise / nb)
    assert np.abs(O.project_mean_zero(x, labels) - x).max() <= 1e-12 * np.abs(x).max()
