"""GPU: the one-launch sums at the edges of their chunks, through the entry points that use them:
E and dE where chunks of faces are empty, hold one face, or hold more than a wave takes at once, on
both sides of the size where the pair kernels change, and more problems than one launch takes."""
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
@pytest.mark.parametrize("nu,nv", [(8, 8), (16, 8), (17, 8), (129, 64), (130, 127)])
def test_energy_sums(tp, nu, nv, prec):
    """128, 256, 272 faces (chunks of one and two), 16,512 (the symmetric energy's sum over pairs of
    blocks and faces) and 33,020: E against the oracle, the same from E alone, E + dE and a step."""
    m = mg.add_noise(mg.torus(nu, nv, 1.0, 0.3), 1e-4, nu)
    print(f"[dots] faces {m.nF} precision {prec}", flush=True)
    tol = 1e-11 if prec == 2 else 1e-5
    with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda(), tp.default_params(precision=prec)) as P:
        E = P.energy()
        Eg, _ = P.gradient()
        assert P.energy() == E
        rep = P.step(tp.step_opts(tau0=1e-9, line_search=0)) if nu <= 17 else None
    E0 = O.energy(m.V, m.F)
    assert abs(E - E0) <= tol * E0 and abs(Eg - E0) <= tol * E0
    if rep is not None:
        assert abs(rep.E - E0) <= tol * E0
        A, V6 = O.total_area(m.V, m.F), O.total_volume(m.V, m.F)
        # phi_before: the constraints at the first positions, whose targets are these sums
        assert abs(rep.phi_before[0]) <= 1e-13 * A and abs(rep.phi_before[1]) <= 1e-13 * abs(V6)


def test_many_jobs(tp):
    """Nine problems with both constraints need more sums per launch than one takes."""
    meshes = [mg.add_noise(mg.geodesic_sphere(4), 0.01, q) for q in range(9)]
    probs = [tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) for m in meshes]
    sts, reps = tp.batch_step(probs)
    assert sts == [0] * 9
    for m, r, P in zip(meshes, reps, probs):
        with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as Q:
            a = Q.step()
            assert (a.E, a.slope, a.tau, a.E_new) == (r.E, r.slope, r.tau, r.E_new)
            assert torch.equal(Q.vertices(), P.vertices())
        P.close()


def test_more_problems_than_a_launch(tp):
    """Seventeen problems of unequal sizes, some of two components: one more than the vertex and
    face passes take in a launch.  Each gives the bits of its own step."""
    meshes = [mg.linked_tori(8 + q, 8, 1.0, 0.25, 1.0) if q % 3 == 0 else mg.add_noise(mg.torus(10 + q, 9, 1.0, 0.3), 1e-3, q)
              for q in range(17)]
    probs = [tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) for m in meshes]
    sts, reps = tp.batch_step(probs)
    assert sts == [0] * 17
    for q, (m, r, P) in enumerate(zip(meshes, reps, probs)):
        print(f"[batch] problem {q} faces {m.nF}", flush=True)
        with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as Q:
            a = Q.step()
            assert (a.E, a.slope, a.tau, a.E_new) == (r.E, r.slope, r.tau, r.E_new)
            assert torch.equal(Q.vertices(), P.vertices())
        P.close()
