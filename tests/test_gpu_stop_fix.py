"""The term that a stop at the first product of a two-product launch leaves to
be taken back out of p belongs to that loop alone: the next substep, when it
runs in single products, must not find it.
"""
import numpy as np
import pytest

import synth
from oracle import integrators as I
from oracle import operators as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    return E


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_substep_after_a_stop_inside_a_pair(E, dtype):
    """Rough vectors teach the operator degree 8 for this substep length; a
    nearly constant vector over two such substeps then stops at every degree
    from 2 on in the first one, among them 5, the first product of the
    deferred products 4 and 5."""
    import torch
    shape = (131, 60)
    n = shape[0] * shape[1]
    h = tuple(1.0 / (m + 1) for m in shape)
    tabs = [np.cos(2 * np.pi * (np.arange(m) + 0.3) / m) for m in shape]
    field = (1.0 + 0.4 * tabs[1][:, None] * tabs[0][None, :]).reshape(-1)
    A = O.stencil_matrix(shape, h, "neumann0", coef=field)
    a, b = O.gershgorin_interval(A)
    z, tol = 1.5, 1e-6
    tau = z / (b - a)
    rough = synth.uniform_vector(n, 4)
    T = lambda x: torch.as_tensor(x, device="cuda:0")
    degrees = set()
    for eps in np.logspace(0, -6, 25):
        v = 1.0 + eps * rough
        yo, so = I.phi_action(A, 1, 2 * tau, v, tol, params=I.LejaParams(l_max=z * (1 + 1e-7)))
        assert so.substeps == 2
        degrees.add(so.degrees[0])
        op = E.StencilOp(shape, h, "neumann0", coef=field)
        for _ in range(6):
            E.phi_action(op, 1, tau, T(rough), tol=tol, dtype=dtype)
        print(f"fix {dtype} eps={eps:.1e} degrees {so.degrees}", flush=True)
        y, s = E.phi_action(op, 1, 2 * tau, T(v), tol=tol, dtype=dtype, params=E.LejaParams(l_max=z * (1 + 1e-7)))
        assert s["substeps"] == 2 and s["converged"] == 1
        # the Leja sums of both agree to rounding where they stop at the same
        # degree, and to the tolerance where a borderline test falls otherwise
        y = y.cpu().numpy()
        same = s["newton_steps"] == so.newton_steps
        bound = (1e-12 if dtype == "f64" else 5e-6) if same else 4 * tol
        assert np.max(np.abs(y - yo)) <= bound * np.max(np.abs(yo)), (eps, so.degrees)
    assert 5 in degrees
