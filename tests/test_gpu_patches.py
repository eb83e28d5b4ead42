"""Patches by recursive bisection and their default size: equal parts for any mesh size, components and non-manifold
pieces apart, patches over the LDS budget halved; the assembled result against the oracle each time."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
SHELL = [(4, (1.0, 1.0)), (5, (1.0, 1.0))]
ALL = 1 | 2 | 4


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch


def check(torch, tris, rest, x, precision, patch_faces=0, comp=None):
    _, prob = PR.build_gpu(tris, rest, rest.shape[0], 3, SHELL, precision, comp_offsets=comp, patch_faces=patch_faces)
    P = PR.build_oracle(tris, rest, rest.shape[0], 3, SHELL)
    ref = P.eval(np.ascontiguousarray(x).ravel(), ALL)
    e, g, h = (t.cpu().numpy() for t in prob.eval(torch.from_numpy(np.ascontiguousarray(x).ravel()).cuda(), ALL))
    rtol = PR.RTOL[precision]
    assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
    PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
    PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
    return prob.layout()


@pytest.mark.parametrize("n,target", [(2, 1), (2, 64), (5, 31), (30, 0), (30, 64), (33, 100), (70, 0), (70, 5000)])
def test_equal_parts(torch_cuda, n, target):
    print("patches of a grid", n, target, flush=True)
    m = meshgen.shell_cylinder(n)
    lay = check(torch_cuda, m.tris, m.rest, m.x, 1, target)
    faces = 2 * (n - 1) ** 2
    # as many parts as the target asks for, unless the LDS asks for more
    assert lay["n_patches"] >= -(-faces // lay["patch_faces"])
    if target and target <= 100:
        assert lay["patch_faces"] == target and lay["n_patches"] == -(-faces // target)


def test_components_keep_apart(torch_cuda):
    print("patches of components", flush=True)
    m = meshgen.icosphere_batch(n_meshes=3, mean_verts=700, vmin=600, vmax=900)
    lay = check(torch_cuda, m.tris, m.rest, m.x, 1, 200, m.comp_offsets)
    assert lay["n_patches"] >= sum(-(-2 * (b - a - 2) // 200) for a, b in zip(m.comp_offsets, m.comp_offsets[1:]))


@pytest.mark.parametrize("precision", [0, 1])
def test_a_few_patches_over_the_budget(torch_cuda, precision):
    # a closed fan of many faces around two poles next to a regular strip: the fan's patches touch more blocks
    print("patches over the LDS budget", precision, flush=True)
    k, (gt, gp) = 150, meshgen.grid(60)
    a = 2 * np.pi * np.arange(k) / k
    ring = np.stack([np.cos(a), np.sin(a), 0.1 * np.cos(7 * a)], 1)
    p = np.concatenate([ring, [[0, 0, 1.0], [0, 0, -1.0]]])
    i, j = np.arange(k), (np.arange(k) + 1) % k
    fan = np.concatenate([np.stack([i, j, np.full(k, k)], 1), np.stack([j, i, np.full(k, k + 1)], 1)])
    tris = np.concatenate([fan, gt + k + 2]).astype(np.int32)
    rest = np.concatenate([p, gp * 3.0 + [2, 0, 0]])
    x = rest + np.random.default_rng(8).normal(0, 1e-3, rest.shape)
    check(torch_cuda, tris, rest, x, precision, 512)
