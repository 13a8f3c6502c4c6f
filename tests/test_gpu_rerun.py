"""Loops that stop earlier than their deferred stop tests reach are run again
up to the degree found.  Every early degree, against a fresh operator's launch
by launch (params.profile); and no loop runs twice because of what one other
vector needed.

Products and sums round the same however the launches are grouped, except that
FP32 pair sweeps of 3D operators leave a rounding of the last term in p: those
are bounded by the FP32 rounding of a sum of terms below its largest value
(2^-23 for the term added and taken out), times the ten terms at most.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

NAMES = ["const2d", "field2d", "const3d", "field3d", "csr"]


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
    if name == "csr":
        g = synth.rgg_negative_laplacian(3000, 1, 12.0)
        return (lambda: E.CsrOp(g.n, g.rowptr, g.colind, g.val)), g.n
    shape = {"const2d": (300, 150), "field2d": (140, 90), "const3d": (128, 12, 10), "field3d": (40, 20, 9)}[name]
    h = tuple(1.0 / n for n in shape)
    n = int(np.prod(shape))
    coef = 1.0 + 0.3 * synth.uniform_vector(n, 3) if name.startswith("field") else 1.0
    return (lambda: E.StencilOp(shape, h, "neumann0", coef=coef)), n


def check(name, dtype, y, z, where):
    y, z = y.cpu().numpy(), z.cpu().numpy()
    err = np.max(np.abs(y - z)) / np.max(np.abs(z))
    bound = 1e-13 if dtype == "f64" else (10 * 2.0**-23 if name.endswith("3d") or name == "const2d" else 0.0)
    assert err <= bound, (where, err)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", NAMES)
def test_every_early_stop(E, name, dtype):
    new, n = make(E, name)
    a, b = new().interval()
    tau = 13.0 / (b - a)
    tol = 1e-10 if dtype == "f64" else 1e-6
    rough = synth.uniform_vector(n, 1)
    degrees, rerun = set(), 0
    for eps in (1.0, 1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-7, 1e-9, 0.0):
        v = T(1.0 + eps * rough)
        op = new()
        for _ in range(5):
            E.phi_action(op, 1, tau, T(rough), tol=tol, dtype=dtype)
        print(f"early stop {name} {dtype} eps={eps}", flush=True)
        y, s = E.phi_action(op, 1, tau, v, tol=tol, dtype=dtype)
        z, r = E.phi_action(new(), 1, tau, v, tol=tol, dtype=dtype, params=E.LejaParams(profile=True))
        assert (s["degree_last"], s["matvecs"], s["converged"]) == (r["degree_last"], r["matvecs"], 1), eps
        # (a constant vector's terms are the roundings of a product's five or
        # seven weights, in FP64 or FP32)
        ulp = 2.0**-53 if dtype == "f64" else 2.0**-24
        assert abs(s["err_est"] - r["err_est"]) <= 1e-6 * r["err_est"] + 16 * ulp
        check(name, dtype, y, z, eps)
        degrees.add(s["degree_last"])
        rerun += s["rerun_products"]
        # two substeps of the same length and an Euler step of two substeps
        p2 = dict(l_max=13.0 * (1 + 1e-9))
        for k in (0, 1):
            y, s = E.phi_action(op, k, 2 * tau, v, tol=tol, dtype=dtype, params=E.LejaParams(**p2))
            z, r = E.phi_action(new(), k, 2 * tau, v, tol=tol, dtype=dtype, params=E.LejaParams(profile=True, **p2))
            assert s["substeps"] == 2 and s["matvecs"] == r["matvecs"], (eps, k)
            check(name, dtype, y, z, (eps, k))
    assert len(degrees) >= 5 and rerun > 0


@pytest.mark.parametrize("name", NAMES)
def test_one_other_vector_is_no_evidence(E, name):
    """A step length seen once, or thrice where nothing runs in chains, with a
    rough vector: a constant one then stops at degree 2 without a product run
    for nothing."""
    new, n = make(E, name)
    op = new()
    a, b = op.interval()
    rough, ones = T(synth.uniform_vector(n, 1)), T(np.ones(n))
    for q, seen in ((0.9, 0), (1.0, 1), (1.1, 1 if name.endswith("2d") else 3)):
        tau = q * 13.0 / (b - a)
        for _ in range(seen):
            E.phi_action(op, 1, tau, rough, tol=1e-10)
        _, s = E.phi_action(op, 1, tau, ones, tol=1e-10)
        assert s["degree_last"] == 2 and s["rerun_products"] == 0, seen


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", NAMES)
def test_steps_run_again(E, name, dtype):
    """Euler and Runge-Kutta steps whose loops stop early: the start vector is
    formed again (alone, or inside the first pair sweep) and u is untouched
    until the loop is accepted."""
    new, n = make(E, name)
    a, b = new().interval()
    tol = 1e-10 if dtype == "f64" else 1e-6
    rough = 0.5 + 0.1 * synth.uniform_vector(n, 1)
    rerun = 0
    for substeps in (1, 2):
        tau = substeps * 13.0 / (b - a)
        kw = dict(l_max=13.0 * (1 + 1e-9))
        for step in (E.expeuler_step, E.exprk2_step):
            for eps in (1e-2, 1e-6, 0.0):
                u0 = 0.5 + eps * 0.1 * synth.uniform_vector(n, 2)
                op = new()
                for _ in range(6):
                    step(op, tau, T(rough), tol=tol, dtype=dtype, params=E.LejaParams(**kw))
                print(f"step again {name} {dtype} {step.__name__} {substeps} eps={eps}", flush=True)
                u, z = T(u0), T(u0)
                s = step(op, tau, u, tol=tol, dtype=dtype, params=E.LejaParams(**kw))
                r = step(new(), tau, z, tol=tol, dtype=dtype, params=E.LejaParams(profile=True, fuse_start=1, **kw))
                assert s["substeps"] == r["substeps"] == substeps
                assert s["matvecs"] == r["matvecs"], (step.__name__, substeps, eps)
                # u's own rounding in FP64; FP32 vectors enter through tau p
                u, z = u.cpu().numpy(), z.cpu().numpy()
                err = np.max(np.abs(u - z)) / np.max(np.abs(z))
                assert err <= (1e-13 if dtype == "f64" else 10 * 2.0**-23), (step.__name__, substeps, eps, err)
                rerun += s["rerun_products"]
    assert rerun > 0
