"""CSR products at the sizes where the default lanes per row change: below and
above 2^15 rows, and around one, 1.2 and two passes of the grid.

A row has at most 8 entries of at most 1, so a product and its sum carry at
most 16 roundings of 2^-53 times 8 max|x|.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

PASS = 2048 * 64


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    return E


@pytest.mark.parametrize("n", [2**15 - 1, 2**15, PASS - 1, PASS, PASS + 1, 161468, 5 * 2 * PASS // 6, 2 * PASS * 5 // 6 - 1,
                               2 * PASS, 2 * PASS + 1])
def test_default_lanes(E, n):
    import torch
    rng = np.random.default_rng(n)
    # rows of up to 8 entries, some empty, at several distances
    offs = [0, 1, -1, 7, -63, 64, 1000, -4097]
    A = sum(sp.diags(rng.uniform(-1, 1, n - abs(o)) * (rng.random(n - abs(o)) < 0.7), o) for o in offs).tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    op = E.CsrOp(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    x = rng.uniform(-1, 1, n)
    y = E.apply_op(op, 1.0, 0.0, torch.as_tensor(x, device="cuda:0")).cpu().numpy()
    assert np.abs(y - A @ x).max() <= 16 * 2.0**-53 * 8
