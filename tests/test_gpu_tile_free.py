"""The plane kernels take no vector tile: the autotuner times them once and keeps
the same tile every time, and meshes of one class with different tiles still
share their launches."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2512_08571_amd import fehx, inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def _mesh(N, p, dq=0, seed=78):
    A = np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]])
    s = inputs.make_custom(A, N, p, p + 1 + dq, kpoint=(0, 0, 0), nvec=1, seed=seed, gga=True)
    m = fehx.Mesh(A, N, p, p + 1 + dq, (0, 0, 0), device=0)
    pts = m.quad_points()
    m.set_potential(inputs.eval_vloc(s, pts), inputs.eval_vgga(s, pts))
    return m


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_autotune_times_one_kernel_once(prec):
    m = _mesh((4, 4, 4), 4)
    best, ms = m.autotune(prec, 16, reps=2)
    assert len({t for t in ms.values() if t >= 0}) == 1
    for _ in range(3):
        assert m.autotune(prec, 16, reps=2)[0] == best
    # n_q > n_p: the tile is the staged kernel's, and each is timed
    assert len({t for t in _mesh((4, 4, 4), 3, dq=2).autotune(prec, 16, reps=2)[1].values() if t >= 0}) > 1


def _nodes(f):
    """Nodes of the graph that f(stream) captures."""
    hip = fehx.lib()
    s = torch.cuda.Stream()
    g, n = ctypes.c_void_p(), ctypes.c_size_t()
    p = ctypes.c_void_p(s.cuda_stream)
    assert hip.hipStreamBeginCapture(p, 1) == 0      # thread-local
    try:
        f(s)
    finally:
        assert hip.hipStreamEndCapture(p, ctypes.byref(g)) == 0
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(g) == 0
    return n.value


@pytest.mark.parametrize("dq,tiles", [(0, (4, 16)), (2, (4, 8))])
def test_batch_of_differently_tuned_meshes(dq, tiles):
    ms = [_mesh((4, 3, 4), 4, dq, seed=i) for i in range(2)]
    X = [torch.rand(m.ndofs, 9, dtype=torch.float64, device="cuda") for m in ms]
    Y = [torch.empty_like(x) for x in X]
    count = []
    for t in ((tiles[0], tiles[0]), tiles):
        for m, vt in zip(ms, t):
            m.set_tile("f64", vt)
        fehx.batch_apply(ms, X, Y)
        want = [y.clone() for y in Y]
        for m, x, w in zip(ms, X, want):
            y = torch.empty_like(x)
            m.apply(x, y)
            assert torch.equal(y, w)
        torch.cuda.synchronize()
        count.append(_nodes(lambda s: fehx.batch_apply(ms, X, Y, stream=s)))
    assert count[1] == count[0] if dq == 0 else count[1] > count[0]
