"""A few patches over the LDS budget among many that fit are halved and the others stay as large as asked for: a grid
beside loose triangles, whose patches hold twice the vertices and blocks; against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
SHELL = [(4, (1.0, 1.0)), (5, (1.0, 1.0))]
ALL = 1 | 2 | 4


def parts(faces, target, coarse=8192):
    """patches of a component before any is halved: cut in powers of two to at most `coarse` faces, then evenly"""
    n = 1
    while n * coarse < faces:
        n *= 2
    sizes = [faces]
    while len(sizes) < n:
        sizes = [q for s in sizes for q in (s // 2, s - s // 2)]
    return sum(-(-s // target) for s in sizes)


@pytest.mark.parametrize("precision,target", [(1, 256), (0, 160)])
def test_few_over_the_budget(precision, target):
    import torch
    print("[case] halved patches", precision, target, flush=True)
    r = np.random.default_rng(9)
    gt, gp = meshgen.grid(120)
    k = 300
    one = np.array([[0.0, 0, 0], [1.0, 0, 0], [0.2, 0.9, 0]])
    loose = (one[None] + r.normal(0, 0.1, (k, 3, 3))).reshape(-1, 3) * 0.02 + [2.0, 0, 0]
    tris = np.concatenate([gt, np.arange(3 * k).reshape(k, 3) + len(gp)]).astype(np.int32)
    rest = np.concatenate([gp, loose])
    x = 1.1 * rest + r.normal(0, 1e-4, rest.shape)
    _, prob = PR.build_gpu(tris, rest, len(rest), 3, SHELL, precision, patch_faces=target)
    lay = prob.layout()
    # the target stood, so the grid's patches did not shrink; more patches than it asks for were made by halving
    whole = parts(len(tris), target)
    assert lay["patch_faces"] == target
    assert whole < lay["n_patches"] <= whole + whole // 32
    P = PR.build_oracle(tris, rest, len(rest), 3, SHELL)
    xt = torch.from_numpy(np.ascontiguousarray(x).ravel()).cuda()
    for mode in (ALL, ALL | 8):
        ref = P.eval(np.ascontiguousarray(x).ravel(), mode)
        e, g, h = (t.cpu().numpy() for t in prob.eval(xt, mode))
        rtol = PR.RTOL[precision]
        assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
        PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
        PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
