"""3D products whose rows go end to end: waves run over row ends, so x and y
neighbours may sit in another wave, another row or nowhere.

Each sum of seven terms differs from the oracle's by a few roundings of its
largest term; |A| |x| <= rho max|x| bounds the terms, so 16 roundings of
2^-53 rho max|x| bound the difference.
"""
import numpy as np
import pytest

from oracle import operators as O

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


# one row shorter than a lane's points, several rows per wave, rows one point
# past a wave, planes that end inside a wave and inside a workgroup, one plane
SHAPES = [(1, 9, 5), (2, 3, 4), (7, 40, 3), (65, 7, 9), (120, 5, 6), (130, 3, 5), (150, 130, 3), (150, 9, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", ["dirichlet0", "neumann0", "interior_only"])
@pytest.mark.parametrize("kind", ["const", "separable", "field", "dlap"])
def test_rows_end_to_end(E, shape, bc, kind):
    rng = np.random.default_rng(sum(shape))
    h = tuple(1.0 / (n + 1) for n in shape)
    tabs = [np.cos(2 * np.pi * (np.arange(n) + 0.3) / n) for n in shape]
    field = (1.0 + 0.4 * tabs[2][:, None, None] * tabs[1][None, :, None] * tabs[0]).reshape(-1)
    if kind == "dlap":
        op, A = E.StencilOp(shape, h, bc, coef=("dlap", 1.0)), O.dlap_matrix(shape, h, bc)
    else:
        coef = {"const": 1.3, "separable": ("separable", 1.0, 0.4, *tabs), "field": field}[kind]
        op, A = E.StencilOp(shape, h, bc, coef=coef), O.stencil_matrix(shape, h, bc,
                                                                      coef=1.3 if kind == "const" else field)
    x = rng.uniform(-1, 1, int(np.prod(shape)))
    rho = max(1.0, abs(A).sum(axis=1).max())
    for vec, waves, march in ((1, 4, 8), (2, 4, 8), (2, 2, 4)):
        op.set_tiles(vec, waves, march)
        y = E.apply_op(op, 1.0, 0.0, T(x)).cpu().numpy()
        assert np.abs(y - A @ x).max() <= 16 * 2.0**-53 * rho


@pytest.mark.parametrize("shape", [s for s in SHAPES if min(s) > 1])
@pytest.mark.parametrize("data", ["z1mz_xy", "sinpiz_expmxy"])
def test_boundary_data_on_rows_end_to_end(E, shape, data):
    rng = np.random.default_rng(sum(shape))
    h = tuple(1.0 / (n + 1) for n in shape)
    A, bf = O.stencil_matrix(shape, h, "dirichlet0", coef=1.3), O.dirichlet_boundary_term(shape, h, data, coef=1.3)
    op = E.StencilOp(shape, h, "dirichlet0", coef=1.3)
    x = rng.uniform(-1, 1, int(np.prod(shape)))
    op.set_boundary_data(data, "in_kernel")
    y = E.apply_op(op, 1.0, 0.0, T(x)).cpu().numpy()
    assert np.abs(y - (A @ x + bf)).max() <= 16 * 2.0**-53 * (abs(A).sum(axis=1).max() + np.abs(bf).max())
