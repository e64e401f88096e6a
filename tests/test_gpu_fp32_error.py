"""The FP32 operator is no less exact with its weights folded into the 1D tables
than with the weights applied at the points: relative 2-norm error against FP64
below what one cell of that form has in FP32 arithmetic (emulated step by step,
cubic cells of 1.25 bohr, uniform input: 1.64e-7, 2.31e-7, 1.79e-7 and 2.11e-7
at 5 to 8 points; the folded tables as they come have 1.71e-7, 1.89e-7, 2.00e-7
and 2.14e-7)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2512_08571_amd import fehx, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
POINTWISE = {4: 1.64e-7, 5: 2.31e-7, 6: 1.79e-7, 7: 2.11e-7}


@pytest.mark.parametrize("gga", [True, False])
@pytest.mark.parametrize("p", sorted(POINTWISE))
def test_error_of_the_folded_tables(p, gga):
    N = (6, 5, 6)
    A = np.diag([1.25 * n for n in N])
    s = inputs.make_custom(A, N, p, p + 1, kpoint=(0, 0, 0), nvec=1, seed=79, gga=gga)
    m = fehx.Mesh(A, N, p, p + 1, (0, 0, 0), device=0)
    pts = m.quad_points()
    m.set_potential(inputs.eval_vloc(s, pts), inputs.eval_vgga(s, pts))
    X = torch.rand(m.ndofs, 64, device="cuda").mul_(2).sub_(1)
    Y, Z = torch.empty_like(X), torch.empty(X.shape, dtype=torch.float64, device="cuda")
    m.apply(X, Y, "f32")
    m.apply(X.double(), Z)
    err = float((Y.double() - Z).norm() / Z.norm())
    print(f"p {p} gga {gga}: {err:.3e}")
    assert err < POINTWISE[p]
