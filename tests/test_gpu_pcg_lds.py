"""GPU: the persistent Poisson solve where its on-chip memory is full: nearly as many blocks as it
takes, around a pole whose block has more neighbouring rows than fit beside them, alone and in a batch
with a small mesh of a wide halo."""
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


def bipyramid(n):
    """Two apices of degree n over a wavy rim."""
    a = np.arange(n) * 2.0 * np.pi / n
    V = np.concatenate([np.stack([np.cos(a), np.sin(a), 0.1 * np.sin(3.0 * a)], 1), [[0, 0, 1.0], [0, 0, -1.0]]])
    i = np.arange(n)
    F = np.concatenate([np.stack([i, (i + 1) % n, np.full(n, n)], 1), np.stack([(i + 1) % n, i, np.full(n, n + 1)], 1)])
    return mg.Mesh(V, F.astype(np.int32))


@pytest.mark.parametrize("nu,nv,k", [(181, 180, 9), (190, 172, 9), (190, 172, 8), (256, 126, 7)])
def test_blocks_and_halo(tp, nu, nv, k):
    """253 to 256 blocks and a halo of 256 rows and more: the true relative residual, recomputed with
    the oracle's matrix, meets the solver's 1e-10 up to the rounding of the recomputation (eps |C||x| / |b|
    for every term of a row)."""
    m = globe(nu, nv)
    b = mg.random_columns(m.nV, k, 30 + k)
    print(f"[pcg lds] globe {nu} x {nv} k={k} vertices {m.nV}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as P:
        x, _ = P.poisson_solve(torch.from_numpy(b).cuda())
    x = x.cpu().numpy()
    C = O.cotan_laplacian(m.V, m.F)
    _, labels = O.components(m.F, m.nV)
    Pb = O.project_mean_zero(b, labels)
    nb = np.linalg.norm(Pb, axis=0)
    r = np.linalg.norm(Pb - C @ x, axis=0)
    terms = np.diff(C.tocsr().indptr)[:, None] + 1
    noise = 2.0 ** -52 * np.linalg.norm(terms * (abs(C) @ abs(x)), axis=0)
    assert np.all(r <= 1e-10 * nb * (1 + 1e-6) + noise), (r / nb, noise / nb)


def test_batch_of_both(tp):
    """A torus of 250 blocks and a small bipyramid whose blocks have 256 rows of halo: a step of both
    together gives each the bits of its own."""
    meshes = [mg.add_noise(mg.torus(250, 128, 1.0, 0.3), 1e-5, 3), bipyramid(600)]
    print("[pcg lds] batch", [m.nV for m in meshes], flush=True)
    probs = [tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) for m in meshes]
    sts, reps = tp.batch_step(probs, tp.step_opts(tau0=1e-6, line_search=0))
    assert sts == [0, 0]
    for m, r, P in zip(meshes, reps, probs):
        with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as Q:
            a = Q.step(tp.step_opts(tau0=1e-6, line_search=0))
            assert (a.E, a.slope, a.E_new) == (r.E, r.slope, r.E_new)
            assert torch.equal(Q.vertices(), P.vertices())
        P.close()
