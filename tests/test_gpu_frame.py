"""The clamp in the element's own axes (membrane 4 x 4 + 2 x 2, hinge 8 x 8 after its null direction) against the
oracle's dense 9 x 9 / 12 x 12 clamp: randomly placed hinges with any fold and any orientation, triangles without a
plane, a positive eigenvalue floor (which the null direction and the translations then take too)."""
from __future__ import annotations

import numpy as np
import pytest

from . import parity as PR

ALL_SPD = 1 | 2 | 4 | 8


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch


def hinges(n, seed, scale):
    """n disjoint pairs of triangles: rest flat and well shaped, current positions drawn at random."""
    r = np.random.default_rng(seed)
    base = np.arange(n, dtype=np.int32)[:, None] * 4
    tris = np.concatenate([base + [0, 1, 2], base + [1, 0, 3]], axis=1).reshape(-1, 3).astype(np.int32)
    quad = np.array([[0, 0, 0], [1, 0, 0], [0.4, 0.8, 0], [0.6, -0.7, 0]])
    rest = (quad[None] + r.normal(0, 0.1, (n, 4, 3))).reshape(-1, 3) * scale
    x = r.normal(0, 1.0, (4 * n, 3)) * scale
    return tris, rest, x


def check(torch, tris, rest, x, terms, precision, eps):
    nv = rest.shape[0]
    _, prob = PR.build_gpu(tris, rest, nv, 3, terms, precision, patch_faces=40, spd_eps=eps)
    P = PR.build_oracle(tris, rest, nv, 3, terms)
    ref = P.eval(x.ravel(), ALL_SPD, spd_eps=eps)
    xt = torch.from_numpy(x.ravel()).cuda()
    e, g, h = (t.cpu().numpy() for t in prob.eval(xt, ALL_SPD))
    rtol = PR.RTOL[precision]
    assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
    PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
    PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
    nonfinite, _ = prob.status()
    assert not nonfinite


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("eps", [0.0, 0.05])
@pytest.mark.parametrize("terms", [[(5, (1.0, 1.0))], [(4, (1.0, 0.7))], [(2, ())]])
def test_random_elements(torch_cuda, precision, eps, terms):
    print("frame clamp, random elements", precision, eps, terms, flush=True)
    tris, rest, x = hinges(150, 11, 1.0)
    check(torch_cuda, tris, rest, x, terms, precision, eps)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_hinge_axes(torch_cuda, precision):
    print("frame clamp, hinges along each axis, both ways, flat and folded", precision, flush=True)
    tris, rest, x = hinges(36, 5, 1.0)
    x = x.reshape(-1, 4, 3)
    for k in range(36):   # the hinge along +-axis, the second face folded by a multiple of 50 degrees
        ax, fold = k % 3, np.deg2rad(50.0 * (k // 6))
        s = 1.0 if (k // 3) % 2 else -1.0
        u, m, n = (np.eye(3)[(ax + j) % 3] for j in range(3))
        x[k] = [0 * u, s * u, 0.5 * s * u + 0.8 * m, 0.3 * s * u - 0.7 * (np.cos(fold) * m + np.sin(fold) * n)]
    check(torch_cuda, tris, rest, x.reshape(-1, 3), [(4, (1.0, 1.0)), (5, (1.0, 1.0))], precision, 0.0)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_triangles_without_a_plane(torch_cuda, precision):
    print("frame clamp, collinear and collapsed triangles", precision, flush=True)
    r = np.random.default_rng(3)
    n = 24
    tris = np.arange(3 * n, dtype=np.int32).reshape(-1, 3)
    rest = (np.array([[0, 0, 0], [1, 0, 0], [0.4, 0.8, 0]])[None] + r.normal(0, 0.1, (n, 3, 3))).reshape(-1, 3)
    x = r.normal(size=(n, 3, 3))
    for k in range(n):
        d = x[k, 1] - x[k, 0]
        if k % 8 == 0:
            x[k, 2] = x[k, 0] + 0.3 * d          # on the line
        elif k % 8 == 1:
            x[k, 1] = x[k, 0]                    # first edge of no length
        elif k % 8 == 2:
            x[k, 2] = x[k, 0]                    # second edge of no length
        elif k % 8 == 3:
            x[k, 1] = x[k, 2] = x[k, 0]          # one point
        elif k % 8 == 4:
            x[k, 2] = x[k, 0] + 0.5 * d + 1e-9 * r.normal(size=3)   # almost on the line
        elif k % 8 == 5:
            x[k] = [[0, 0, 0], [0, 0, 1], [0, 0, -2]]
    check(torch_cuda, tris, rest, x.reshape(-1, 3), [(4, (1.0, 1.0))], precision, 0.0)
