"""GPU: a batch that fails because the near-field grid of its second problem cannot be allocated leaves
the first problem without a grid, not with one that was never built."""
import ctypes

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


def cells(nF):
    """Bytes of the cell table: 8 per cell, cbrt(8 nF) cells per axis, rounded down."""
    return 8 * int((8.0 * nF) ** (1.0 / 3.0)) ** 3


def test_second_allocation_fails(tp):
    meshes = [mg.add_noise(mg.torus(20, 12, 1.0, 0.3), 1e-3, 1), mg.add_noise(mg.torus(31, 17, 1.0, 0.3), 1e-3, 2)]
    refused = cells(meshes[1].nF)
    armed = [False, 0]

    def alloc(nbytes, stream, user):
        if armed[0] and nbytes == refused:
            armed[1] += 1
            return None
        return torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(), int(stream or 0))

    cbs = (tp._ALLOC_FN(alloc), tp._FREE_FN(lambda ptr, nbytes, stream, user: torch.cuda.caching_allocator_delete(ptr)))
    L = tp.lib()
    assert L.tp_set_allocator(ctypes.cast(cbs[0], ctypes.c_void_p), ctypes.cast(cbs[1], ctypes.c_void_p), None) == 0
    try:
        probs = [tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) for m in meshes]
        armed[0] = True
        opts = tp.step_opts(tau0=1e-6, line_search=0)
        try:
            sts, _ = tp.batch_step(probs, opts)
        except tp.TpError as e:
            sts = [e.status] * 2
        armed[0] = False
        assert armed[1] >= 1 and all(s != 0 for s in sts), (armed, sts)
        got = [P.gradient() for P in probs]
        for P in probs:
            P.close()
        for m, (E, g) in zip(meshes, got):
            with tp.Problem(torch.from_numpy(m.V).cuda(), torch.from_numpy(m.F).cuda()) as Q:
                E0, g0 = Q.gradient()
            assert E == E0 and torch.equal(g, g0)
    finally:
        assert L.tp_set_allocator(None, None, None) == 0
