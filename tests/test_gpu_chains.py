"""Chains of Newton products on 2D stencils (several products per pass) and
stop tests of several launches at once, against the oracle and against the
launch-by-launch path (params.profile, which keeps one test per launch).

The two paths take every product by the same formula, so with FP32 storage
they give the same bits; in FP64 a point differs by the rounding of at most a
few dozen terms of the Newton sum, bounded here by 1e-12 of the largest value.
"""
import numpy as np
import pytest

import synth
from oracle import integrators as I
from oracle import operators as O

pytestmark = pytest.mark.gpu

TOL_F64 = 1e-10


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


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def make(E, shape, bc, kind, amp=0.4):
    h = tuple(1.0 / (n + 1) for n in shape)
    tabs = [np.cos(2 * np.pi * (np.arange(n) + 0.3) / n) for n in shape]
    if kind == "const":
        return (lambda: E.StencilOp(shape, h, bc, coef=1.3)), O.stencil_matrix(shape, h, bc, coef=1.3)
    if kind == "dlap":
        return (lambda: E.StencilOp(shape, h, bc, coef=("dlap", 1.0))), O.dlap_matrix(shape, h, bc)
    field = (1.0 + amp * tabs[1][:, None] * tabs[0][None, :]).reshape(-1)
    A = O.stencil_matrix(shape, h, bc, coef=field)
    if kind == "separable":
        return (lambda: E.StencilOp(shape, h, bc, coef=("separable", 1.0, amp, *tabs))), A
    return (lambda: E.StencilOp(shape, h, bc, coef=field)), A


# strips: 64 V points less 2 halo columns of 4 to 8 points at inner ends; grids
# of up to 16,384 points run the whole loop in one workgroup (FP64, constant
# coefficient): rows of one wave (up to 64 or 128 points) and of several
SHAPES = [(128, 128), (128, 40), (124, 9), (250, 67), (248, 33), (129, 21), (57, 30), (113, 50), (2, 30), (1, 40),
          (40, 1), (64, 256), (65, 128), (600, 5), (1920, 2), (16, 400), (1000, 37), (300, 300), (113, 301), (64, 257),
          (130, 140), (57, 300)]


@pytest.mark.parametrize("kind", ["const", "field", "separable", "dlap"])
@pytest.mark.parametrize("bc", ["dirichlet0", "neumann0", "interior_only"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_chain_equals_separate_launches(E, kind, bc, dtype):
    for shape in SHAPES:
        new, A = make(E, shape, bc, kind)
        a, b = O.gershgorin_interval(A)
        iv = None if b > a else (-1.0, 0.0)
        tau = 25.0 / (b - a) if iv is None else 1e-3
        v = synth.uniform_vector(int(np.prod(shape)), 7)
        tol = 1e-10 if dtype == "f64" else 1e-6
        kw = {"interval": iv} if iv else {}
        print(f"chain {kind} {bc} {dtype} {shape}", flush=True)
        op, ref = new(), new()
        yo, _ = I.phi_action(A, 1, tau, v, 1e-12, interval=iv)
        for call in range(2):      # without and with a known degree
            y, s = E.phi_action(op, 1, tau, T(v), tol=tol, dtype=dtype, params=E.LejaParams(**kw))
            z, r = E.phi_action(ref, 1, tau, T(v), tol=tol, dtype=dtype, params=E.LejaParams(profile=True, **kw))
            y, z = y.cpu().numpy(), z.cpu().numpy()
            assert s["degree_last"] == r["degree_last"], (shape, call)
            if dtype == "f32":
                assert np.array_equal(y, z), (shape, call, np.max(np.abs(y - z)))
                assert relerr(y, yo) <= 2e-5, (shape, call)
            else:
                assert np.max(np.abs(y - z)) <= 1e-12 * np.max(np.abs(z)), (shape, call)
                assert relerr(y, yo) <= TOL_F64, (shape, call)


@pytest.mark.parametrize("shape,bc,kind", [((140, 90), "dirichlet0", "const"), ((131, 60), "neumann0", "field"),
                                           ((70, 12, 9), "neumann0", "field"), ((256, 10, 7), "dirichlet0", "const")])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_degree_hint_too_large_or_too_small(E, shape, bc, kind, dtype):
    """Inputs of very different smoothness on one operator: the degree known
    from the last call is wrong in both directions.  A stop before the
    deferred tests runs the loop again; every call gives what a fresh
    operator with a test per launch gives."""
    if len(shape) == 3:
        h = tuple(1.0 / (n + 1) for n in shape)
        coef = 1.0 if kind == "const" else 1.0 + 0.4 * synth.uniform_vector(int(np.prod(shape)), 3)
        new = lambda: E.StencilOp(shape, h, bc, coef=coef)
        A = O.stencil_matrix(shape, h, bc, coef=coef)
    else:
        new, A = make(E, shape, bc, kind)
    a, b = O.gershgorin_interval(A)
    n = int(np.prod(shape))
    grid = np.indices(tuple(reversed(shape)))
    smooth = np.ones(tuple(reversed(shape)))
    for ax, m in zip(grid, reversed(shape)):
        smooth = smooth * np.sin(np.pi * (ax + 1) / (m + 1))
    inputs = {"smooth": smooth.reshape(-1), "rough": synth.uniform_vector(n, 4)}
    op = new()
    degrees = set()
    for q in (18.0, 160.0):        # one and two substeps
        tau = q / (b - a)
        for name in ("rough", "smooth", "rough", "smooth", "smooth", "rough"):
            print(f"hint {shape} {kind} {dtype} q={q} {name}", flush=True)
            tol = 1e-10 if dtype == "f64" else 1e-6
            y, s = E.phi_action(op, 1, tau, T(inputs[name]), tol=tol, dtype=dtype)
            yo, so = I.phi_action(A, 1, tau, inputs[name], 1e-12)
            assert relerr(y.cpu().numpy(), yo) <= (TOL_F64 if dtype == "f64" else 2e-5), (q, name)
            z, r = E.phi_action(new(), 1, tau, T(inputs[name]), tol=tol, dtype=dtype,
                                params=E.LejaParams(profile=True))
            assert s["degree_last"] == r["degree_last"] and s["matvecs"] == r["matvecs"], (q, name)
            degrees.add(s["degree_last"])
            u = T(0.5 + 0.1 * inputs[name])
            st = E.expeuler_step(op, tau, u, tol=tol, dtype=dtype)
            uo, _ = I.expeuler_step(A, tau, 0.5 + 0.1 * inputs[name], 1e-12)
            assert relerr(u.cpu().numpy(), uo) <= (TOL_F64 if dtype == "f64" else 5e-6), (q, name)
            assert st["converged"] == 1
    assert len(degrees) >= 2


def test_hint_on_unstructured_matrix(E):
    """The same on a CSR operator (single products)."""
    g = synth.rgg_negative_laplacian(3000, 1, 12.0)
    import scipy.sparse as sp
    A = sp.csr_matrix((g.val, g.colind, g.rowptr), shape=(g.n, g.n))
    op = E.CsrOp(g.n, g.rowptr, g.colind, g.val)
    a, b = O.gershgorin_interval(A)
    for name, v in (("rough", synth.uniform_vector(g.n, 1)), ("constant", np.ones(g.n)),
                    ("rough", synth.uniform_vector(g.n, 2)), ("rough", synth.uniform_vector(g.n, 2))):
        print(f"hint csr {name}", flush=True)
        y, s = E.phi_action(op, 1, 60.0 / (b - a), T(v), tol=1e-10)
        yo, so = I.phi_action(A, 1, 60.0 / (b - a), v, 1e-10)
        assert abs(s["degree_last"] - so.degrees[-1]) <= 1
        assert relerr(y.cpu().numpy(), yo) <= TOL_F64


def test_hint_on_complex_matrix(E):
    """The same on a Hermitian operator: e^{-itH}v over substeps whose degree
    is known, and wrongly known, from earlier calls."""
    import scipy.sparse as sp
    g = synth.spin_bath_hamiltonian(9, 3, bath_bonds=10)
    H = sp.csr_matrix((g.val, g.colind, g.rowptr), shape=(g.n, g.n))
    op = E.CsrComplexOp(g.n, g.rowptr, g.colind, g.val)
    _, vec = np.linalg.eigh(H.toarray())
    inputs = {"eigenvector": vec[:, 0].astype(np.complex128), "rough": synth.complex_uniform_vector(g.n, 2)}
    for k in (0, 1):
        for name in ("rough", "rough", "eigenvector", "rough", "eigenvector", "eigenvector"):
            print(f"hint complex k={k} {name}", flush=True)
            y, s = E.skew_phi_action(op, k, 9.0, T(inputs[name]), tol=1e-10)
            fresh = E.CsrComplexOp(g.n, g.rowptr, g.colind, g.val)
            z, r = E.skew_phi_action(fresh, k, 9.0, T(inputs[name]), tol=1e-10)
            assert s["matvecs"] == r["matvecs"] and s["degree_last"] == r["degree_last"]
            # single products either way: the same bits
            assert np.array_equal(y.cpu().numpy(), z.cpu().numpy()), (k, name)
            yo, _ = I.skew_phi_action(H, k, 9.0, inputs[name], 1e-10)
            assert relerr(y.cpu().numpy(), yo) <= TOL_F64, (k, name)
