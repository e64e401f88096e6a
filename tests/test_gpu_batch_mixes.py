"""A system's result does not depend on what shares its launch: batches and
server steps that mix blocks of even and odd lane counts, blocks off their
alignment, diagonal and general metrics and systems of very different size
equal separate applications bit for bit.

The two routes from the plane kernels to the staged one (complex FP32 / BF16
blocks that start between pairs of lanes, a z plane of nodes past 2 GiB) are
compared with the plane kernels: the same operator, relative to the largest
entry 1e-12 in FP64 and 2e-5 in FP32 (a few hundred roundings of 2^-24), and
2e-2 in BF16 (up to five partial stores rounding by 2^-9).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2512_08571_amd import fehx, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
TOL = {"f64": 1e-12, "f32": 2e-5, "bf16": 2e-2}


def _mesh(N, p, k=(0, 0, 0), shear=0.0, dq=0, seed=76):
    A = np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]])
    A[1, 0] = shear
    s = inputs.make_custom(A, N, p, p + 1 + dq, kpoint=k, nvec=1, seed=seed, gga=True)
    m = fehx.Mesh(A, N, p, p + 1 + dq, k, device=0)
    pts = m.quad_points()
    m.set_potential(inputs.eval_vloc(s, pts), inputs.eval_vgga(s, pts))
    return m


def _lanes(m, prec, lanes, off=0, ld=None, seed=0):
    """[ndofs, ld] real lanes of which `lanes` are the block, `off` elements into their storage."""
    ld = ld or lanes
    x = torch.zeros(off + m.ndofs * ld, dtype=DT[prec], device="cuda")
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = x[off:].view(m.ndofs, ld)
    v[:, :lanes] = torch.rand(m.ndofs, lanes, device="cuda", generator=g).mul_(2).sub_(1).to(DT[prec])
    return v


def _apply(m, X, Y, lanes, prec):
    """Through the C-ABI, on real lanes (torch has no complex view of an odd storage offset)."""
    C = 2 if m.is_complex else 1
    st = fehx.lib().fe_apply_H(m._h, X.data_ptr(), X.stride(0) // C, Y.data_ptr(), Y.stride(0) // C, lanes // C,
                               fehx.PREC[prec], torch.cuda.current_stream().cuda_stream)
    assert st == 0


def _batch(ms, Xs, Ys, lanes, prec):
    n = len(ms)
    C = [2 if m.is_complex else 1 for m in ms]
    ptr = lambda ts: (fehx.c_p * n)(*[t.data_ptr() for t in ts])  # noqa: E731
    ld = lambda ts: (fehx.i64 * n)(*[t.stride(0) // c for t, c in zip(ts, C)])  # noqa: E731
    st = fehx.lib().fe_batch_apply(n, (fehx.c_p * n)(*[m._h for m in ms]), ptr(Xs), ld(Xs), ptr(Ys), ld(Ys),
                                   (fehx.i64 * n)(*[a // c for a, c in zip(lanes, C)]), fehx.PREC[prec],
                                   torch.cuda.current_stream().cuda_stream)
    assert st == 0


def _batch_equals_separate(ms, blocks, lanes, prec):
    Ya, Yb = [torch.zeros_like(x) for x in blocks], [torch.zeros_like(x) for x in blocks]
    for m, x, y, n in zip(ms, blocks, Ya, lanes):
        _apply(m, x, y, n, prec)
    _batch(ms, blocks, Yb, lanes, prec)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(Ya, Yb)):
        assert torch.equal(a, b), i


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_large_even_and_small_odd(prec):
    ms = [_mesh((16, 16, 16), 6), _mesh((4, 4, 6), 6), _mesh((12, 12, 12), 6)]
    lanes = [256, 33, 48]
    _batch_equals_separate(ms, [_lanes(m, prec, n, seed=i) for i, (m, n) in enumerate(zip(ms, lanes))], lanes, prec)


@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_complex_block_off_its_alignment(prec):
    ms = [_mesh((4, 3, 5), 4, (0.2, 0.1, 0.3), seed=s) for s in (1, 2)]
    lanes = [14, 10]
    blocks = [_lanes(ms[0], prec, 14), _lanes(ms[1], prec, 10, off=1)]
    assert blocks[1].data_ptr() % (2 * blocks[1].element_size())
    _batch_equals_separate(ms, blocks, lanes, prec)
    # the staged kernel there, against the plane kernel on an aligned copy
    Y, Z = torch.empty_like(blocks[1]), torch.zeros(1 + blocks[1].numel(), dtype=DT[prec], device="cuda")
    Z = Z[1:].view_as(Y)
    _apply(ms[1], blocks[1].clone(), Y, 10, prec)
    _apply(ms[1], blocks[1], Z, 10, prec)
    assert float((Y.double() - Z.double()).abs().max()) < TOL[prec] * float(Y.double().abs().max())


def test_metrics_in_one_batch():
    ms = [_mesh((4, 3, 5), 4, seed=1), _mesh((4, 3, 5), 4, shear=0.4, seed=2), _mesh((3, 3, 4), 4, seed=3)]
    for prec in ("f64", "f32"):
        _batch_equals_separate(ms, [_lanes(m, prec, 9, seed=i) for i, m in enumerate(ms)], [9] * 3, prec)


@pytest.mark.parametrize("prec", ["f64", "bf16"])
def test_z_plane_past_two_gib(prec):
    """The same few vectors as a window of rows so long that a z plane spans more
    than the plane kernels' offsets reach."""
    m = _mesh((16, 16, 2), 2)
    es = torch.empty((), dtype=DT[prec]).element_size()
    ld = (2 << 30) // (32 * 32 * es) + 8
    X = _lanes(m, prec, 5)
    Y = torch.empty_like(X)
    W = torch.zeros(m.ndofs, ld, dtype=DT[prec], device="cuda")
    V = torch.empty_like(X)
    M = torch.empty_like(X)
    m.apply(X, Y, prec)
    m.apply(X, W, prec, nvec=5)
    assert float((Y.double() - W[:, :5].double()).abs().max()) < TOL[prec] * float(Y.double().abs().max())
    assert not W[:, 5:16].any()
    V.copy_(W[:, :5])
    fehx.batch_apply([m, _mesh((8, 8, 2), 2)], [X, X[:16 * 16 * 4].contiguous()], [W, M[:16 * 16 * 4]], prec, nvecs=[5, 5])
    assert torch.equal(V, W[:, :5])
    m.apply_mass(X, M, prec)
    m.apply_mass(X, W, prec, nvec=5)
    assert float((M.double() - W[:, :5].double()).abs().max()) < TOL[prec] * float(M.double().abs().max())


def test_server_mix():
    """A request's FP32 result is the one it has alone, whatever else is in flight."""
    shapes = [((8, 8, 8), 64, 0), ((4, 4, 6), 33, 0), ((6, 5, 7), 18, 2), ((5, 5, 5), 7, 0)]
    ms = [_mesh(N, 4, dq=dq, seed=i) for i, (N, _, dq) in enumerate(shapes)]
    X = [_lanes(m, "f32", n, seed=i) for i, (m, (_, n, _)) in enumerate(zip(ms, shapes))]
    lam = [torch.linspace(-1.0, 1.0, n, dtype=torch.float64, device="cuda") for _, n, _ in shapes]

    def run(together, kind):
        srv = fehx.Server(hbm_budget=16 << 30, max_active=8)
        out = [x.double() if kind == "filter" else torch.zeros_like(x) for x in X]
        for i, m in enumerate(ms):
            if kind == "filter":
                srv.submit_filter(m, out[i], lam[i], 6, -2.0, 2.0, 60.0, inner="f32")
            else:
                srv.submit_apply(m, X[i], out[i], "f32")
            if not together:
                srv.drain()
        srv.drain()
        torch.cuda.synchronize()
        srv.close()
        return out

    for kind in ("apply", "filter"):
        for a, b in zip(run(False, kind), run(True, kind)):
            assert torch.equal(a, b)
