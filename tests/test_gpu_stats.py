"""What a call reports does not depend on what the operator or the workspace
saw before: the first terms and the counts of a call with a known degree
against a fresh operator's launch by launch (params.profile).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    return E


def T(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


def make(E, name):
    """(new operator, points)"""
    if name == "csr":
        g = synth.rgg_negative_laplacian(3000, 1, 12.0)
        return (lambda: E.CsrOp(g.n, g.rowptr, g.colind, g.val)), g.n
    shape = {"resident": (100, 100), "const2d": (300, 300), "field2d": (140, 90), "const3d": (128, 12, 10),
             "field3d": (40, 20, 9)}[name]
    h = tuple(1.0 / n for n in shape)
    n = int(np.prod(shape))
    coef = 1.0 + 0.3 * synth.uniform_vector(n, 3) if name.startswith("field") else 1.0
    return (lambda: E.StencilOp(shape, h, "neumann0", coef=coef)), n


@pytest.mark.parametrize("name", ["resident", "const2d", "field2d", "const3d", "field3d", "csr"])
def test_first_terms_are_this_calls_own(E, name):
    """A constant vector stops at degree 2 under zero-flux boundaries: no
    third term, whatever earlier calls (enough of them to use every read-back
    slot) and the products past the stop had."""
    new, n = make(E, name)
    op = new()
    a, b = op.interval()
    tau = 13.0 / (b - a)
    rough, ones = T(synth.uniform_vector(n, 1)), T(np.ones(n))
    for _ in range(66):
        E.phi_action(op, 1, tau, rough, tol=1e-10)
    _, s = E.phi_action(op, 1, tau, ones, tol=1e-10)
    _, r = E.phi_action(new(), 1, tau, ones, tol=1e-10, params=E.LejaParams(profile=True))
    print(name, s["t_first"], r["t_first"], s["degree_last"], flush=True)
    assert s["degree_last"] == r["degree_last"] == 2
    scale = r["t_first"][0]
    assert np.allclose(s["t_first"], r["t_first"], rtol=1e-12, atol=1e-12 * scale)
    assert s["t_first"][3:] == [0.0, 0.0]


@pytest.mark.parametrize("fuse", [1, 2])
def test_tested_products_are_counted_alike(E, fuse):
    """An Euler step counts the products whose norms were reduced, not the
    norm of its start vector, whether the start vector is formed inside the
    first pair sweep (2) or not (1), tested launch by launch or afterwards."""
    new, n = make(E, "const3d")
    op = new()
    a, b = op.interval()
    tau = 13.0 / (b - a)
    u0 = 0.5 + 0.1 * synth.uniform_vector(n, 2)
    step = lambda o, **kw: E.expeuler_step(o, tau, T(u0), tol=1e-10, params=E.LejaParams(fuse_start=fuse, **kw))
    ref = new()
    for call in range(8):
        s, r = step(op), step(ref, profile=True)
        print(f"finalized {s['finalized']} of degree {s['degree_last']} (launch by launch {r['finalized']})", flush=True)
        assert s["fused_starts"] == fuse - 1 and s["degree_last"] == r["degree_last"]
        assert s["finalized"] == r["finalized"], call


@pytest.mark.parametrize("name", ["resident", "const2d", "field2d", "const3d", "field3d", "csr"])
def test_products_run_twice_are_reported(E, name):
    """A much earlier stop than every known one makes the loop run again: the
    call says how many products it ran for nothing; other calls say none."""
    new, n = make(E, name)
    op = new()
    a, b = op.interval()
    tau = 13.0 / (b - a)
    rough, ones = T(synth.uniform_vector(n, 1)), T(np.ones(n))
    for _ in range(8):
        _, s = E.phi_action(op, 1, tau, rough, tol=1e-10)
        assert s["rerun_products"] == 0
    _, s1 = E.phi_action(op, 1, tau, ones, tol=1e-10)
    print(f"{name}: degree {s['degree_last']}, then {s1['degree_last']}, run twice {s1['rerun_products']}", flush=True)
    assert s1["degree_last"] == 2 and s1["matvecs"] == 2
    if name == "resident":
        assert s1["rerun_products"] == 0
    else:
        assert 2 < s1["rerun_products"] <= s["degree_last"]
    _, s2 = E.phi_action(op, 1, tau, ones, tol=1e-10)
    assert s2["rerun_products"] == 0


@pytest.mark.parametrize("name", ["const2d", "field2d", "const3d", "field3d", "csr"])
def test_tolerances_and_storage_types_learn_apart(E, name):
    """Degrees known from a tight tolerance or from FP64 say nothing about a
    loose one or FP32: no such call runs its loop twice."""
    new, n = make(E, name)
    op = new()
    a, b = op.interval()
    tau = 13.0 / (b - a)
    v = T(synth.uniform_vector(n, 1))
    degrees = set()
    for tol, dtype in ((1e-12, "f64"), (1e-3, "f64"), (1e-12, "f64"), (1e-6, "f32"), (1e-3, "f32")):
        for _ in range(8):
            _, s = E.phi_action(op, 1, tau, v, tol=tol, dtype=dtype)
            assert s["rerun_products"] == 0, (tol, dtype)
        degrees.add(s["degree_last"])
        print(f"{name} tol {tol} {dtype}: degree {s['degree_last']}", flush=True)
    assert len(degrees) >= 3
