"""GPU: the hierarchical product of a vector with one infinite value: rows that it does not touch are
-inf (their kernel weights are positive), not NaN, and the other columns are as without it."""
import numpy as np
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


@pytest.mark.parametrize("prec,k", [(3, 1), (2, 1), (3, 6), (3, 9)])
def test_one_infinite_value(tp, prec, k):
    m = mg.geodesic_sphere(24)
    u = mg.random_columns(m.nV, k, 3)
    print(f"[tree inf] precision {prec} k={k}", flush=True)
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), tp.default_params(precision=prec, chi=0.5)) as P:
        y0 = P.fractional_apply(torch.from_numpy(u).cuda()).cpu().numpy()
        for v in range(0, m.nV, 397):
            w = u.copy()
            w[v, 0] = np.inf
            y = P.fractional_apply(torch.from_numpy(w).cuda()).cpu().numpy()
            far = np.ones(m.nV, bool)
            far[m.F[(m.F == v).any(1)]] = False
            assert np.all(y[far, 0] == -np.inf), (v, int(np.isnan(y[far, 0]).sum()))
            assert np.array_equal(y[:, 1:], y0[:, 1:])
