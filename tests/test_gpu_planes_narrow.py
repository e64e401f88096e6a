"""FP32 and BF16 plane kernels of the local operator against the assembled
oracle: blocks that threads of two lanes take (even, pair-aligned rows), blocks
that only threads of one can (odd counts, odd leading dimensions, rows that
start between pairs), and a complex block off its pair alignment.

Tolerances relative to the largest entry: FP32 2e-5 as for the other kernels
(a few hundred roundings of 2^-24).  BF16, on input already in BF16: each of a
node's up to five partial stores rounds by 2^-9 of a partial sum no larger than
about twice the result: 2e-2.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from oracle import operator as op  # noqa: E402
from paper_2512_08571_amd import inputs  # noqa: E402

from gpu_common import lib_side, oracle_side, rel  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {"f32": 2e-5, "bf16": 2e-2}
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _lanes(X):
    """[ndofs, real lanes] in float64."""
    if np.iscomplexobj(X):
        return np.stack([X.real, X.imag], -1).reshape(X.shape[0], -1)
    return X


def _block(m, prec, lanes, ld, off):
    """An uninitialised block of `lanes` real lanes, leading dimension ld, `off` lanes into its storage."""
    flat = torch.full((m.ndofs * ld + off,), float("nan"), dtype=DT[prec], device="cuda")
    v = flat[off:].view(m.ndofs, ld)[:, :lanes]
    if not m.is_complex:
        return v
    v = v.unflatten(1, (lanes // 2, 2))
    return torch.view_as_complex(v) if prec == "f32" else v


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("k", [(0, 0, 0), (0.3, -0.2, 0.1)], ids=["real", "complex"])
@pytest.mark.parametrize("p", range(2, 9))
def test_lane_pairs_and_single_lanes(p, k, prec):
    N = (3, 2, 5) if p < 7 else (2, 3, 4)
    t = 64 // (p + 1) & ~1
    cplx = any(k)
    s = inputs.make_custom(np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]]), N, p, p + 1, kpoint=k, nvec=2 * t + 2,
                           seed=72, gga=p % 3 != 0)
    om, vl, vg, _, _ = oracle_side(s)
    H = op.assemble_H(om, vl, vg)
    m = lib_side(s, vl, vg)
    X = inputs.make_vectors(s)
    X = torch.from_numpy(_lanes(X).copy()).to(DT[prec])
    full = X.double().numpy()
    if cplx:
        want = _lanes(op.apply_sparse(H, full[:, ::2] + 1j * full[:, 1::2]))
    else:
        want = op.apply_sparse(H, full)
    C = 2 if cplx else 1
    # (lanes, extra leading dimension, offset of the storage)
    forms = [(C, C, 0), (2 * t, 0, 0), (2 * t + 2, 2, 0)]
    if not cplx:
        forms += [(t - 1, 0, 0), (t + 1, 2, 0), (2 * t, 1, 0), (2 * t, 2, 1)]
    for lanes, pad, off in forms:
        ld = lanes + pad
        xb, yb = _block(m, prec, lanes, ld, off), _block(m, prec, lanes, ld, off)
        src = X[:, :lanes].cuda()
        if cplx:
            src = src.unflatten(1, (lanes // 2, 2))
            src = torch.view_as_complex(src.contiguous()) if prec == "f32" else src
        xb.copy_(src)
        m.apply(xb, yb, prec, nvec=lanes // C)
        got = torch.view_as_real(yb) if cplx and prec == "f32" else yb
        got = got.float().cpu().double().numpy().reshape(m.ndofs, lanes)
        assert rel(got, want[:, :lanes]) < TOL[prec], (p, lanes, pad, off)
        if pad:   # the columns past the block stay untouched
            rest = yb._base.flatten() if yb._base is not None else yb.flatten()
            rest = torch.view_as_real(rest).flatten() if rest.is_complex() else rest
            assert int(torch.isnan(rest).sum()) >= m.ndofs * pad


@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_few_and_many_waves(prec):
    """Narrow threads on a small device load, pairs on a full one: the same operator."""
    N = (3, 3, 4)
    s = inputs.make_custom(np.diag([1.3 * N[0], 1.2 * N[1], 1.4 * N[2]]), N, 4, 5, kpoint=(0, 0, 0), nvec=4, seed=73)
    om, vl, vg, _, _ = oracle_side(s)
    H = op.assemble_H(om, vl, vg)
    m = lib_side(s, vl, vg)
    X = torch.from_numpy(inputs.make_vectors(s).copy()).to(DT[prec])
    want = op.apply_sparse(H, X.double().numpy())
    for reps in (1, 2048):
        Xd = X.cuda().repeat(1, reps).contiguous()
        Yd = torch.full_like(Xd, float("nan"))
        m.apply(Xd, Yd, prec)
        ref = torch.from_numpy(want).cuda()
        for j in range(4):
            d = (Yd[:, j::4].double() - ref[:, j:j + 1]).abs().max()
            assert float(d) < TOL[prec] * np.abs(want).max(), (reps, j)
