"""The residual Jacobian at the sizes where its launch's blocks and waves end: element counts just below, at and
above 64 and 256, where a wave's run of rows is short or the next term begins, with vertices numbered at random."""
from __future__ import annotations

import numpy as np
import pytest

from .test_gpu_jacobian import build, check_jacobian, torch_cuda  # noqa: F401
from .test_gpu_rows import fan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("k", [3, 21, 22, 62, 63, 85, 86, 254, 255])      # 3k edges, k + 2 vertices
def test_block_and_wave_ends(torch_cuda, precision, k):  # noqa: F811
    print("[case] jacobian sizes", precision, k, flush=True)
    r = np.random.default_rng(k)
    tris, rest = fan(k)
    perm = r.permutation(k + 2)
    tris, rest = perm[tris].astype(np.int32), rest[np.argsort(perm)]
    vd = np.concatenate([r.uniform(0.5, 2.0, (k + 2, 1)), rest + r.normal(0, 0.2, rest.shape)], 1)
    _, prob, P, _ = build(torch_cuda, tris, rest, vd, precision)
    check_jacobian(torch_cuda, prob, P, rest + r.normal(0, 0.05, rest.shape), precision)
