"""Giving a CSR operator the setting it reports changes nothing in FP64: the
same lanes sum every row in the same order."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5000, 40000, 110000, 161468])
def test_reported_setting_is_the_one_that_runs(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    g = synth.rgg_negative_laplacian(n, 1, 12.0)
    new = lambda: E.CsrOp(g.n, g.rowptr, g.colind, g.val)
    x = torch.as_tensor(synth.uniform_vector(g.n, 2), device="cuda:0")
    a, b = new(), new()
    b.set_tiles(*b.tiles())
    ya, yb = E.apply_op(a, 1.0, 0.3, x), E.apply_op(b, 1.0, 0.3, x)
    assert torch.equal(ya, yb), float((ya - yb).abs().max())
