"""The separable mass operator of affine cells (M X) against the assembled M:
every degree, both quadrature rules, sheared boxes, Dirichlet axes, lane counts
at the edges of a wave's tile, and all precisions.

Tolerances relative to the largest entry: FP64 1e-12, FP32 2e-5, BF16 2e-2 on
input already in BF16 (up to five partial stores, each rounding by 2^-9).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from oracle import operator as op  # noqa: E402
from oracle.mesh import Mesh as OMesh  # noqa: E402
from paper_2512_08571_amd import fehx  # noqa: E402

from gpu_common import rel  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 2e-5, "bf16": 2e-2}
DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("p", range(2, 9))
def test_mass_planes(p, prec):
    N = (3, 2, 5) if p < 6 else (2, 3, 4)
    dq = (0, 2, 0)[p % 3]
    A = np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]])
    if p % 2:
        A[1, 0] = 0.4                       # a sheared box: the Jacobian is still constant
    per = (True, True, True) if p % 4 else (True, False, False)
    om = OMesh(A, N, p, p + 1 + dq, (0, 0, 0), periodic=per)
    idx = np.arange(om.m) if all(per) else om.dirichlet_dofs()
    M = op.assemble_M(om)[idx][:, idx]
    m = fehx.Mesh(A, N, p, p + 1 + dq, (0, 0, 0), device=0, periodic=per)
    t = 64 // (p + 1) & ~1
    X = torch.from_numpy(np.random.default_rng(p).uniform(-1, 1, (len(idx), 2 * t + 2))).to(DT[prec])
    want = M @ X.double().numpy()
    for nv in (1, t, t + 1, 2 * t, 2 * t + 2):
        Xd = X[:, :nv].contiguous().cuda()
        Y = torch.full((len(idx), nv + 1), float("nan"), dtype=DT[prec], device="cuda")
        m.apply_mass(Xd, Y, prec, nvec=nv)
        assert rel(Y[:, :nv].double().cpu().numpy(), want[:, :nv]) < TOL[prec], (p, nv)
        assert torch.isnan(Y[:, nv:]).all()
