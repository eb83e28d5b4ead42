"""What the FP32 clamp may not add to an element's rounding: a factor where no rotation is needed."""
from __future__ import annotations

import numpy as np
import pytest

from . import parity as PR

pytestmark = pytest.mark.gpu


def test_no_factor_without_rotations():
    """Triangles symmetric in their first two vertices, whose Dirichlet matrix is diagonal in the clamp's coordinates and
    positive: the clamp changes nothing. Each entry is rounded a few times, half up and half down, so over 12,000 diagonal
    entries the roundings leave a mean relative error below 2^-24 / sqrt(12000) times a few; a quarter of an ulp (2^-25,
    to which the hardware reciprocal of the scaling counts) is what a systematic part may not reach."""
    import torch
    print("[case] clamp without rotations", flush=True)
    r = np.random.default_rng(21)
    n = 4000
    w, h = r.uniform(0.2, 1.0, n), r.uniform(0.2, 1.0, n)
    rest = np.zeros((n, 3, 3))
    rest[:, 0, 0], rest[:, 1, 0], rest[:, 2, 1] = -w, w, h
    rest = rest.reshape(-1, 3)
    tris = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    x = r.normal(size=3 * n)
    _, prob = PR.build_gpu(tris, rest, 3 * n, 1, [(3, ())], 1)
    P = PR.build_oracle(tris, rest, 3 * n, 1, [(3, ())])
    ref = P.eval(x, 1 | 2 | 4)
    h32 = prob.eval(torch.from_numpy(x).cuda(), 1 | 2 | 4 | 8)[2].cpu().numpy().ravel().astype(np.float64)
    rp, ci = (t.cpu().numpy() for t in prob.pattern())
    dia = np.repeat(np.arange(3 * n), np.diff(rp)) == ci
    rel = h32[dia] / np.asarray(ref.hess).ravel()[dia] - 1.0
    print("mean relative error of the diagonal", rel.mean(), "rms", np.sqrt((rel**2).mean()), flush=True)
    assert abs(rel.mean()) < 2.0**-25
