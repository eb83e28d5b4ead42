"""The FP64 redo queue is empty again after every evaluation that used it: evaluations one after another, one recorded
into a graph before any has run, the static scratch, the product, and a calm state after a stressed one."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import mad, meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
SHELL = [(4, (1.0, 1.0)), (5, (1.0, 1.0))]
CLAMPED = 1 | 2 | 4 | 8


@pytest.mark.parametrize("n", [3, 24])
@pytest.mark.parametrize("q", [1.0, 0.6])      # every element redone; those below that quality
def test_queue_is_left_empty(n, q):
    import torch
    print("[case] redo queue", n, q, flush=True)
    m = meshgen.shell_cylinder(n=n, seed=2002, noise="absolute")
    prob = mad.Problem(mad.Mesh(m.tris, m.n_verts), 3, mad.F32, degenerate_q=q)
    for k, prm in SHELL:
        prob.add_term(k, prm, m.rest)
    prob.finalize()
    P = PR.build_oracle(m.tris, m.rest, m.n_verts, 3, SHELL)
    states = [m.x, meshgen.shell_cylinder(n=n).x]
    xs = [torch.from_numpy(np.ascontiguousarray(x).ravel()).cuda() for x in states]
    refs = [P.eval(np.ascontiguousarray(x).ravel(), CLAMPED) for x in states]

    def check(out, i):
        torch.cuda.synchronize()
        e, g, h = (t.cpu().numpy() for t in out)
        assert abs(e[0] - refs[i].energy) <= PR.RTOL[1] * refs[i].esum_abs
        PR.assert_close("grad", g, refs[i].grad, refs[i].gscale, PR.RTOL[1])
        PR.assert_close("hess", h, refs[i].hess, refs[i].hscale, PR.RTOL[1])

    out, held = prob.outputs(xs[0].device), xs[0].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prob.eval(held, CLAMPED, out=out, stream=torch.cuda.current_stream())
    check(prob.eval(xs[0], CLAMPED), 0)
    for i in (1, 0, 1):
        held.copy_(xs[i])
        graph.replay()
        check(out, i)
        check(prob.eval(xs[i], CLAMPED), i)
    check(prob.eval_static(xs[0], CLAMPED), 0)
    v = torch.ones_like(xs[0])
    y0 = prob.hvp(xs[0], v, mad.SPD)[0].cpu().numpy()
    y1 = prob.hvp(xs[0], v, mad.SPD)[0].cpu().numpy()
    assert np.max(np.abs(y0 - y1)) <= 1e-5 * np.max(np.abs(y0))
    check(prob.eval(xs[1], CLAMPED), 1)
    assert not prob.status()[0]
