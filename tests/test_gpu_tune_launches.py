"""The autotuner times a launch once: layouts that differ in nothing a launch reads share a time, and problems of edge
and vertex terms, which one kernel evaluates whatever the patches are, have one patch candidate."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import mad, meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
ALL = 1 | 2 | 4


@pytest.mark.parametrize("precision", [0, 1])
def test_edge_terms_have_one_patch_candidate(precision):
    import torch
    print("[case] autotune edges", precision, flush=True)
    tris, rest = meshgen.grid(20)
    prob = mad.Problem(mad.Mesh(tris, 400), 3, precision)
    prob.add_term(mad.SPRING, (7.0, 0.5), rest)
    prob.finalize()
    before = prob.layout()
    rep = prob.autotune(torch.from_numpy(1.1 * rest.ravel()).cuda(), ALL | 8, reps=2, force=True)
    assert sorted(c["scatter"] for c in rep["candidates"]) == ["atomic", "color", "patch"]
    assert all(c["ms"] > 0 for c in rep["candidates"])
    if rep["chosen"]["scatter"] == "patch":
        assert prob.layout() == before


@pytest.mark.parametrize("precision,mode,timed", [(1, ALL | 8, 10), (0, ALL | 8, 10), (0, 1 | 2, 6), (0, ALL, 10)])
def test_one_time_for_one_launch(precision, mode, timed):
    """timed: launches that differ (FP64 Hessians in 3D take their patches from a counter where asked to)"""
    import torch
    print("[case] autotune launches", precision, mode, flush=True)
    m = meshgen.shell_cylinder(n=30)
    _, prob = PR.build_gpu(m.tris, m.rest, m.n_verts, 3, [(4, (1.0, 1.0)), (5, (1.0, 1.0))], precision)
    rep = prob.autotune(torch.from_numpy(np.ascontiguousarray(m.x).ravel()).cuda(), mode, reps=3, force=True)
    patch = [c for c in rep["candidates"] if c["scatter"] == "patch"]
    assert len(patch) == (16 if precision == 1 else 8) and len(rep["candidates"]) == len(patch) + 2
    key = lambda c: (c["patch_faces"], c["wg_waves"])
    both = {}
    for c in patch:
        both.setdefault(key(c), {})[c["persistent"]] = c["ms"]
    counter = precision == 0 and mode & 4
    assert counter or all(b[0] == b[1] for b in both.values())
    assert len({c["ms"] for c in rep["candidates"]}) <= timed
