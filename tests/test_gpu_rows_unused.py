"""A vertex that no term reads does not make an evaluation non-finite, whichever scatter runs it; one that a term
reads does."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2509_00406_amd import mad, meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("scatter", [mad.SCATTER_ATOMIC, mad.SCATTER_PATCH, mad.SCATTER_COLOR])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_vertices_on_no_edge(value, scatter, precision):
    import torch
    print("[case] unused vertices", value, scatter, precision, flush=True)
    tris, rest = meshgen.grid(9)
    rest = np.concatenate([[[5.0, 5, 5]] * 3, rest, [[9.0, 9, 9]]])
    prob = mad.Problem(mad.Mesh((tris + 3).astype(np.int32), len(rest)), 3, precision, scatter=scatter)
    prob.add_term(mad.SPRING, (7.0, 0.5), rest)
    prob.finalize()
    for at, used in (((0, 2, -1), False), ((10,), True)):
        x = 1.2 * rest
        x[list(at)] = value
        xt = torch.from_numpy(x.ravel()).cuda()
        v = torch.ones_like(xt)
        for mode in (1, 2, 3, 7, 15):
            out = prob.eval(xt, mode)
            assert prob.status()[0] == used, (at, mode)
            if not used:
                assert all(bool(torch.isfinite(t).all()) for k, t in enumerate(out) if mode >> k & 1)
        for mode in (0, 8):
            y = prob.hvp(xt, v, mode)[0]
            assert prob.status()[0] == used, (at, "product", mode)
            assert used or bool(torch.isfinite(y).all())
