"""The projector reduction and update at the lane counts where their row groups,
tiles and tails change, against the assembled oracle.

The reduction moves a block row with 8, 16, 32 or 64 threads of four lanes;
the counts below sit at the edges of those forms (real lanes; a complex vector
is two), with full and ragged last groups, four and nine projectors per atom.
Tolerances relative to the largest entry: FP64 sums of at most a few thousand
terms in another order, 1e-12; FP32 the same sums at 2^-24 each, 2e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from oracle import operator as op  # noqa: E402
from paper_2512_08571_amd import inputs  # noqa: E402

from gpu_common import lib_side, oracle_side, rel, to_dev  # noqa: E402

pytestmark = pytest.mark.gpu
NV_MAX = 260


@pytest.fixture(scope="module", params=[((0, 0, 0), "sp"), ((0.3, -0.2, 0.1), "spd")], ids=["real-sp", "complex-spd"])
def system(request):
    k, pset = request.param
    s = inputs.make_custom(np.diag([7.5, 8.0, 7.3]), (3, 4, 3), 5, 6, kpoint=k, nvec=NV_MAX, seed=23, natoms=3,
                           pset=pset, rc=3.2)
    om, vl, vg, P, h = oracle_side(s)
    X = inputs.make_vectors(s)
    return s, lib_side(s, vl, vg), X, op.apply_sparse(op.assemble_H(om, vl, vg), X, P, h)


@pytest.mark.parametrize("nvec", [1, 2, 7, 8, 9, 16, 17, 32, 33, 64, 65, 127, 128, 129, 257])
def test_projector_terms_at_group_edges(system, nvec):
    s, m, X, want = system
    Xd = to_dev(X[:, :nvec])
    Yd = torch.full_like(Xd, float("nan"))
    m.apply(Xd, Yd)
    assert rel(Yd.cpu().numpy(), want[:, :nvec]) < 1e-12
    # the same columns as a window of a wider block: nothing past them is touched
    wide = torch.full((s.ndofs, nvec + 3), float("nan"), dtype=Xd.dtype, device="cuda")
    m.apply(Xd, wide, nvec=nvec)
    assert torch.equal(wide[:, :nvec], Yd) and torch.isnan(wide[:, nvec:].real).all()
    X32 = Xd.to(torch.complex64 if s.is_complex else torch.float32)
    Y32 = torch.empty_like(X32)
    m.apply(X32, Y32, "f32")
    assert rel(Y32.cpu().numpy(), want[:, :nvec]) < 2e-5
