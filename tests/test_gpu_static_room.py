"""The static scratch holds what it held when patches were grown one after another: an area problem on a 1380^2 grid
fitted 64 MiB then; the bisected patches share more entries (65.4 MiB)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import mad, meshgen

pytestmark = pytest.mark.gpu


def test_static_scratch_holds_a_large_area_problem():
    import torch
    print("[case] static scratch, 1380^2", flush=True)
    tris, rest = meshgen.grid(1380)
    prob = mad.Problem(mad.Mesh(tris, len(rest)), 3, mad.F32)
    prob.add_term(mad.TRI_AREA)
    prob.finalize()
    x = torch.from_numpy(np.ascontiguousarray(rest).ravel()).cuda()
    e, g, _ = prob.eval(x, mad.ENERGY | mad.GRAD)
    es, gs, _ = prob.eval_static(x, mad.ENERGY | mad.GRAD)
    assert bool((e == es).all())
    # a triangle adds at most half its longest edge to an entry, a partial sum of six of them is at most three such, and
    # each evaluation rounds five additions, in any order
    assert float((g - gs).abs().max()) <= 2 * 5 * 2.0**-24 * 3 * 0.5 * 2.0**0.5 / 1379
    assert prob.status() == (False, 0)
