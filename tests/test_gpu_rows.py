"""Row-owned evaluation of edge and vertex terms against the oracle: rows longer than a wave (their units go through
it in passes), rows that grow past it by inserted pairs, components with an energy each, vertices on no triangle,
an edge of no length, several terms of each kind, raw and clamped with a floor, and the matrix-free product."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_00406_amd import mad, meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
ALL = 1 | 2 | 4


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch


def fan(k):
    """Two poles over a ring of k vertices: both poles' rows have k + 1 blocks."""
    a = 2 * np.pi * np.arange(k) / k
    p = np.concatenate([np.stack([np.cos(a), np.sin(a), 0.1 * np.cos(5 * a)], 1), [[0, 0, 1.0], [0, 0, -1.0]]])
    i, j = np.arange(k), (np.arange(k) + 1) % k
    t = np.concatenate([np.stack([i, j, np.full(k, k)], 1), np.stack([j, i, np.full(k, k + 1)], 1)])
    return t.astype(np.int32), p


def build(torch, tris, rest, precision, eps=0.0, comp=None, vertex_terms=True, reserve=0, seed=0):
    nv = rest.shape[0]
    r = np.random.default_rng(seed)
    mesh = mad.Mesh(tris, nv, comp)
    prob = mad.Problem(mesh, 3, precision, spd_eps=eps)
    P = O.Problem(tris, rest, nv, 3)
    for kind, okind, prm in ((mad.SPRING, O.SPRING, (7.0, 0.5)), (mad.EDGE_SQLEN, O.EDGE_SQLEN, ()),
                             (mad.RES_EDGE, O.RES_EDGE, (3.0,))):
        prob.add_term(kind, prm, rest if kind != mad.EDGE_SQLEN else None)
        P.add_term(okind, prm)
    if vertex_terms:
        for kind, okind, prm in ((mad.INERTIA, O.INERTIA, (0.3, 0.0, 0.5, -9.81)), (mad.RES_POSITION, O.RES_POSITION, ())):
            vd = np.concatenate([r.uniform(0.5, 2.0, (nv, 1)), rest + r.normal(0, 0.2, rest.shape)], 1)
            prob.add_vertex_term(kind, prm, torch.from_numpy(vd).cuda())
            P.add_term(okind, prm, vertex_data=vd)
    if reserve:
        prob.reserve_pairs(reserve)
    prob.finalize()
    P.build_pattern()
    return prob, P


def check(torch, prob, P, x, precision, mode, eps=0.0, ref=None):
    ref = P.eval(x.ravel(), mode, spd_eps=eps) if ref is None else ref
    e, g, h = (t.cpu().numpy() for t in prob.eval(torch.from_numpy(x.ravel().copy()).cuda(), mode))
    rtol = PR.RTOL[precision]
    assert abs(e[0] - ref.energy) <= rtol * ref.esum_abs
    if mode & 2:
        PR.assert_close("grad", g, ref.grad, ref.gscale, rtol)
    if mode & 4:
        PR.assert_close("hess", h, ref.hess, ref.hscale, rtol)
    assert prob.status() == (False, 0)
    return e, h


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("k", [3, 61, 63, 64, 130])
def test_long_rows(torch_cuda, precision, k):
    print("rows of", k + 1, "blocks", precision, flush=True)
    tris, rest = fan(k)
    x = rest + np.random.default_rng(k).normal(0, 0.2, rest.shape)
    prob, P = build(torch_cuda, tris, rest, precision)
    for mode in (1, 3, ALL, ALL | 8):
        check(torch_cuda, prob, P, x, precision, mode)
    v = np.random.default_rng(1).normal(size=x.size)
    for spd in (False, True):
        y, _, _ = prob.hvp(torch_cuda.from_numpy(x.ravel().copy()).cuda(), torch_cuda.from_numpy(v).cuda(), 8 if spd else 0)
        yr, ys = P.hvp(x.ravel(), v, spd=spd)
        PR.assert_close("hvp", y.cpu().numpy(), yr, ys, PR.RTOL[precision])


@pytest.mark.parametrize("precision", [0, 1])
def test_floor_and_bare_rows(torch_cuda, precision):
    print("eigenvalue floor, vertices on no triangle", precision, flush=True)
    tris, rest = meshgen.grid(12)
    rest = np.concatenate([[[5.0, 5, 5]] * 70, rest, [[9.0, 9, 9]]])   # 70 rows of one block first, one at the end
    x = rest + np.random.default_rng(4).normal(0, 0.05, rest.shape)
    prob, P = build(torch_cuda, tris + 70, rest, precision, eps=0.4, vertex_terms=False)
    _, h = check(torch_cuda, prob, P, x, precision, ALL | 8, eps=0.4)
    assert np.all(h[:70] == 0) and np.all(h[-1] == 0)


@pytest.mark.parametrize("precision", [0, 1])
def test_strained_springs_and_one_of_no_length(torch_cuda, precision):
    # (a spring at its rest length has no gradient but rounding, which no scale of its own can judge)
    print("coincident vertices", precision, flush=True)
    tris, rest = meshgen.grid(6)
    x = 1.3 * rest
    x[7] = x[8]
    prob = mad.Problem(mad.Mesh(tris, 36), 3, precision)
    prob.add_term(mad.SPRING, (7.0, 0.5), rest)
    prob.finalize()
    P = O.Problem(tris, rest, 36, 3)
    P.add_term(O.SPRING, (7.0, 0.5))
    P.build_pattern()
    for mode in (ALL, ALL | 8):
        check(torch_cuda, prob, P, x, precision, mode)


def test_components_and_inserted_pairs(torch_cuda):
    print("components, rows grown past a wave", flush=True)
    t, p = meshgen.grid(9)
    parts = [(t, p), fan(20), (t, p)]
    off = np.cumsum([0] + [len(q) for _, q in parts])
    tris = np.concatenate([a + o for (a, _), o in zip(parts, off)]).astype(np.int32)
    rest = np.concatenate([q for _, q in parts])
    x = rest + np.random.default_rng(6).normal(0, 0.05, rest.shape)
    prob, P = build(torch_cuda, tris, rest, 1, comp=off, reserve=400)
    e, h0 = check(torch_cuda, prob, P, x, 1, ALL | 8)
    for c, (a, q) in enumerate(parts):   # each component's energy: that of the others' sum left out
        assert e[1 + c] > 0
    assert abs(e[0] - e[1:].sum()) <= 1e-12 * np.abs(e).sum()
    rp0, ci0 = (q.cpu().numpy() for q in prob.pattern())
    pairs = np.array([[3, j] for j in range(40, 130)] + [[100, j] for j in range(0, 60)], np.int32)
    prob.insert_pairs(torch_cuda.from_numpy(pairs).cuda())
    rp, ci = (q.cpu().numpy() for q in prob.pattern())
    assert np.diff(rp).max() > 64
    e2, _, h = (q.cpu().numpy() for q in prob.eval(torch_cuda.from_numpy(x.ravel().copy()).cuda(), ALL | 8))
    assert np.array_equal(e2, e)   # the same sums: a row's lanes are added in the order of its columns
    old = {(r, c): h0[k] for r in range(len(rp0) - 1) for k, c in zip(range(rp0[r], rp0[r + 1]), ci0[rp0[r]:rp0[r + 1]])}
    for r in range(len(rp) - 1):
        for k in range(rp[r], rp[r + 1]):
            want = old.get((r, ci[k]), np.zeros((3, 3)))
            assert np.abs(h[k] - want).max() <= 1e-6 * (1 + np.abs(want).max())
