"""A clamped evaluation that ends in an error after its elements have run (here because the HIP runtime still holds
an error of the caller's) leaves no queued element behind: not for a graph recorded before it, and not for evaluations
between the recording of a graph and its first launch."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import mad, meshgen

from . import parity as PR

pytestmark = pytest.mark.gpu
SHELL = [(4, (1.0, 1.0)), (5, (1.0, 1.0))]
CLAMPED = 1 | 2 | 4 | 8


@pytest.mark.parametrize("record", ["before", "after"])
def test_no_element_stays_queued(record):
    import torch
    print("[case] failed call, graph recorded", record, flush=True)
    m = meshgen.shell_cylinder(n=24, seed=2002, noise="absolute")
    prob = mad.Problem(mad.Mesh(m.tris, m.n_verts), 3, mad.F32, degenerate_q=0.866)
    for k, prm in SHELL:
        prob.add_term(k, prm, m.rest)
    prob.finalize()
    ref = PR.build_oracle(m.tris, m.rest, m.n_verts, 3, SHELL).eval(np.ascontiguousarray(m.x).ravel(), CLAMPED)
    x = torch.from_numpy(np.ascontiguousarray(m.x).ravel()).cuda()

    def check(out):
        torch.cuda.synchronize()
        e, g, h = (t.cpu().numpy() for t in out)
        assert abs(e[0] - ref.energy) <= PR.RTOL[1] * ref.esum_abs
        PR.assert_close("grad", g, ref.grad, ref.gscale, PR.RTOL[1])
        PR.assert_close("hess", h, ref.hess, ref.hscale, PR.RTOL[1])

    def fail():
        torch.cuda.synchronize()
        assert mad.lib().hipSetDevice(1 << 20) != 0   # refused by the runtime, which keeps the error for the next call
        with pytest.raises(mad.MadError):
            prob.eval(x, CLAMPED, out=spare)
        torch.cuda.synchronize()

    check(prob.eval(x, CLAMPED))
    assert 0 < prob.status()[1] < 2 * m.tris.shape[0]      # some elements (of two and a half times the triangles) are redone
    out, spare, held = prob.outputs(x.device), prob.outputs(x.device), x.clone()
    graph = torch.cuda.CUDAGraph()
    if record == "after":
        fail()
    with torch.cuda.graph(graph):
        prob.eval(held, CLAMPED, out=out, stream=torch.cuda.current_stream())
    if record == "before":
        fail()
    else:
        check(prob.eval(x, CLAMPED))
    for _ in range(2):
        graph.replay()
        check(out)
        check(prob.eval(x, CLAMPED))
    assert not prob.status()[0]
