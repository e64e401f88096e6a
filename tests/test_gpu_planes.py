"""The plane kernels of the local operator against the assembled oracle: every
degree, lane counts at the edges of a wave's tile, columns cut into segments
and whole, Dirichlet ends on the segmented axis, two streams on one mesh, and a
user's own capture.

Tolerance 1e-12 relative to the largest entry (FP64): sums of the same few
hundred terms in another order.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from oracle import operator as op  # noqa: E402
from oracle.mesh import Mesh as OMesh  # noqa: E402
from paper_2512_08571_amd import fehx, inputs  # noqa: E402

from gpu_common import lib_side, oracle_side, rel, to_dev  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _tile(p):
    """Lanes of one wave in FP64 (k_local_planes.h): an even number of threads per plane."""
    return 64 // (p + 1) & ~1


def _system(p, k, N, nvec, gga=True, seed=71):
    return inputs.make_custom(np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]]), N, p, p + 1, kpoint=k, nvec=nvec,
                              seed=seed, gga=gga)


@pytest.mark.parametrize("k", [(0, 0, 0), (0.3, -0.2, 0.1)], ids=["real", "complex"])
@pytest.mark.parametrize("p", range(2, 9))
def test_segmented_columns_and_tile_edges(p, k):
    N = (3, 2, 5) if p < 7 else (2, 3, 4)
    t = _tile(p)
    nv_max = t + 1
    s = _system(p, k, N, nv_max, gga=p % 3 != 0)
    om, vl, vg, _, _ = oracle_side(s)
    H = op.assemble_H(om, vl, vg)
    m = lib_side(s, vl, vg)
    X = inputs.make_vectors(s)
    want = op.apply_sparse(H, X)
    for nv in sorted({1, t // 2, t - 1, t, t + 1}):
        Xd = to_dev(X[:, :nv])
        wide = torch.full((s.ndofs, nv + 2), float("nan"), dtype=Xd.dtype, device="cuda")
        m.apply(Xd, wide, nvec=nv)
        assert rel(wide[:, :nv].cpu().numpy(), want[:, :nv]) < TOL, (p, nv)
        assert torch.isnan(wide[:, nv:].real).all()


@pytest.mark.parametrize("p,k", [(2, (0, 0, 0)), (3, (0.2, 0.1, 0.3)), (6, (0, 0, 0)), (7, (0.1, 0.2, 0.0))])
def test_whole_columns(p, k):
    """Enough tiles (2048 waves) that a column is one segment."""
    N = (2, 2, 3)
    cplx = any(k)
    nv = 2048 * _tile(p) // (2 if cplx else 1)
    s = _system(p, k, N, 5)
    om, vl, vg, _, _ = oracle_side(s)
    H = op.assemble_H(om, vl, vg)
    m = lib_side(s, vl, vg)
    X = inputs.make_vectors(s)
    want = op.apply_sparse(H, X)
    Xd = to_dev(X).repeat(1, nv // 5 + 1)[:, :nv].contiguous()
    Yd = torch.empty_like(Xd)
    m.apply(Xd, Yd)
    ref = to_dev(want)
    for j in range(5):
        d = (Yd[:, j::5] - ref[:, j:j + 1]).abs().max()
        assert float(d) < TOL * np.abs(want).max()


@pytest.mark.parametrize("open_axes", [(False, True, True), (True, False, True), (True, True, False)])
def test_dirichlet_ends_of_segments(open_axes):
    s = _system(5, (0, 0, 0), (3, 3, 4), 11)
    om = OMesh(s.lattice, s.ncell, s.degree, s.nq, s.kpoint, periodic=open_axes)
    idx = om.dirichlet_dofs()
    pts = om.quad_points()
    vl, vg = inputs.eval_vloc(s, pts), inputs.eval_vgga(s, pts)
    m = fehx.Mesh(s.lattice, s.ncell, s.degree, s.nq, s.kpoint, device=0, periodic=open_axes)
    m.set_potential(vl, vg)
    X = inputs.make_vectors(s, ndofs=len(idx))
    want = op.apply_sparse(op.assemble_H(om, vl, vg)[idx][:, idx], X)
    Xd = to_dev(X)
    Yd = torch.full_like(Xd, float("nan"))
    m.apply(Xd, Yd)
    assert rel(Yd.cpu().numpy(), want) < TOL


def test_two_streams_share_one_mesh():
    """Applications of one mesh on two streams share its segment planes: each result equals the one alone."""
    s = _system(4, (0, 0, 0), (4, 4, 6), 24)
    om, vl, vg, _, _ = oracle_side(s)
    m = lib_side(s, vl, vg)
    X = [to_dev(inputs.make_vectors(s, seed_offset=i)) for i in range(2)]
    alone = []
    for x in X:
        y = torch.empty_like(x)
        m.apply(x, y)
        alone.append(y)
    torch.cuda.synchronize()
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    Y = [torch.empty_like(x) for x in X]
    for _ in range(6):
        for i in range(2):
            Y[i].fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(3):
            for i in range(2):
                m.apply(X[i], Y[i], stream=st[i])
        torch.cuda.synchronize()
        for i in range(2):
            assert torch.equal(Y[i], alone[i])


def test_users_own_capture_without_a_call_before():
    """The first application of a mesh may be inside a capture: nothing is allocated there."""
    s = _system(4, (0.2, 0.0, 0.1), (3, 4, 6), 9)
    om, vl, vg, _, _ = oracle_side(s)
    m = lib_side(s, vl, vg)
    X = to_dev(inputs.make_vectors(s))
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.apply(X, Y, stream=torch.cuda.current_stream())
    for i in range(4):
        Y.fill_(float("nan"))
        X.mul_(1.25)
        g.replay()
        m.apply(X, Z)
        torch.cuda.synchronize()
        assert rel(Y.cpu().numpy(), Z.cpu().numpy()) < TOL
