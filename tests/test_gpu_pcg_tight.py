"""GPU: the Poisson solve of more blocks than workgroups that are resident at once, at tolerances
close to the rounding of FP64: it converges there in about the iterations that the rate of the
solve asks for, two and four blocks per workgroup."""
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


@pytest.mark.parametrize("freq,k,rtol", [(64, 4, 3e-14), (82, 1, 1e-13), (100, 3, 1e-13)])
def test_tight(tp, freq, k, rtol):
    """321, 526 and 782 blocks.  The solve's own residual meets rtol, the recomputed one up to the
    rounding of the recomputation (eps |C||x| / |b| for every term of a row), and the iterations are
    at most 1.5 log(rtol) / log(1e-6) times those of 1e-6."""
    m = mg.geodesic_sphere(freq)
    b = mg.random_columns(m.nV, k, 60 + k)
    print(f"[pcg tight] sphere {freq} k={k} rtol {rtol} vertices {m.nV}", flush=True)
    V, F, bd = torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), torch.from_numpy(b).cuda()
    its = []
    for r in (1e-6, rtol):
        with tp.Problem(V, F, tp.default_params(cg_rtol=r, cg_maxiter=2000)) as P:
            x, rep = P.poisson_solve(bd)
        assert rep.cg_relres[0] <= r
        its.append(rep.cg_iters[0])
    assert its[1] <= 1.5 * np.log(rtol) / np.log(1e-6) * its[0], its
    x = x.cpu().numpy()
    C = O.cotan_laplacian(m.V, m.F).tocsr()
    _, labels = O.components(m.F, m.nV)
    Pb = O.project_mean_zero(b, labels)
    nb = np.linalg.norm(Pb, axis=0)
    r = np.linalg.norm(Pb - C @ x, axis=0)
    noise = 2.0 ** -52 * np.linalg.norm((np.diff(C.indptr)[:, None] + 1) * (abs(C) @ abs(x)), axis=0)
    assert np.all(r <= rtol * nb * (1 + 1e-6) + noise), (r / nb, noise / nb)
