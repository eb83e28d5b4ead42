"""The row-owned kernel's unclamped Hessians and products are as exact as the same elements' through the atomic
scatter, whose derivatives are taken in the caller's axes: springs, squared lengths and length residuals, each edge on
vertices of its own but for the triangle's other two."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_00406_amd import mad

from . import parity as PR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind,okind,prm", [(mad.SPRING, O.SPRING, (7.0, 0.5)), (mad.RES_EDGE, O.RES_EDGE, (3.0,)),
                                            (mad.EDGE_SQLEN, O.EDGE_SQLEN, ())])
def test_as_exact_as_atomic(kind, okind, prm, precision):
    """The rms error in units of the contributing elements' largest entries over 4,000 loose triangles, whose off-diagonal
    blocks (24,000, 216,000 entries) are one edge's each: its scatter is below one part in a hundred, so a tenth more is a
    different arithmetic."""
    import torch
    print("[case] rows' error", kind, precision, flush=True)
    n = 4000
    r = np.random.default_rng(41)
    tris = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    one = np.array([[0.0, 0, 0], [1.0, 0, 0], [0.2, 0.9, 0]])
    rest = one[None] + r.normal(0, 0.1, (n, 3, 3))
    q, _ = np.linalg.qr(r.normal(size=(n, 3, 3)))
    x = np.ascontiguousarray(np.einsum("nij,nvj->nvi", q, rest + r.normal(0, 0.1, (n, 3, 3))).reshape(-1, 3))
    rest = rest.reshape(-1, 3)
    P = O.Problem(tris, rest, 3 * n, 3)
    P.add_term(okind, prm)
    P.build_pattern()
    ref = P.eval(x.ravel(), 1 | 2 | 4)
    v = r.normal(size=x.size)
    yr, ys = P.hvp(x.ravel(), v)
    rms = {}
    for scatter in (mad.SCATTER_ATOMIC, mad.SCATTER_PATCH):
        prob = mad.Problem(mad.Mesh(tris, 3 * n), 3, precision, scatter=scatter)
        prob.add_term(kind, prm, rest if kind in mad.NEEDS_REST else None)
        prob.finalize()
        xt = torch.from_numpy(x.ravel()).cuda()
        out = prob.eval(xt, 1 | 2 | 4)
        y = prob.hvp(xt, torch.from_numpy(v).cuda())[0]
        errs = []
        for got, want, scale in ((out[1], ref.grad, ref.gscale), (out[2], ref.hess, ref.hscale), (y, yr, ys)):
            w, s = np.asarray(want).ravel(), np.asarray(scale).ravel()
            e = (got.cpu().numpy().astype(np.float64).ravel() - w) / s
            assert np.abs(e).max() <= PR.RTOL[precision]
            errs.append(float(np.sqrt(np.mean(e**2))))
        rms[scatter] = errs
    print("rms error, atomic and rows:", rms[mad.SCATTER_ATOMIC], rms[mad.SCATTER_PATCH], flush=True)
    for a, b in zip(rms[mad.SCATTER_ATOMIC], rms[mad.SCATTER_PATCH]):
        assert b <= 1.1 * a
