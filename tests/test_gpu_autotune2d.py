"""The autotuner keeps what a 2D operator gains most from: where the loop runs
in one launch, or in passes of six products, it does not turn them off because
of how its pair sweep compares with single products; the result stays the
oracle's, also in a grid whose longest chain needs the whole of its room.
"""
import numpy as np
import pytest

import synth
from oracle import integrators as I
from oracle import operators as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(100, 100), (300, 200), (125, 2050)])
def test_tuned_2d_operator(shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    h = tuple(1.0 / (n + 1) for n in shape)
    A = O.stencil_matrix(shape, h, "dirichlet0", coef=1.0)
    a, b = O.gershgorin_interval(A)
    v = synth.uniform_vector(int(np.prod(shape)), 3)
    yo, _ = I.phi_action(A, 1, 13.0 / (b - a), v, 1e-12)
    op = E.StencilOp(shape, h, "dirichlet0", coef=1.0)
    print(f"tune {shape}", flush=True)
    entry = E.autotune.tune(op, "f64", reps=5, use_cache=False)
    assert entry["pairs"] and entry["passes_timed"] and op.pair_setting() >= 4
    for _ in range(6):
        y, s = E.phi_action(op, 1, 13.0 / (b - a), torch.as_tensor(v, device="cuda:0"), tol=1e-10)
        assert np.linalg.norm(y.cpu().numpy() - yo) <= 1e-10 * np.linalg.norm(yo)
