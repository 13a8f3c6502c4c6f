"""3D products on both sides of the rule that lays rows end to end: where that
takes fewer workgroups per CU (150 x 130 x 100: 260 in rows of their own, 156
end to end; 16 x 250 x 250: 504 and 64), where rows of several waves leave many
lanes idle (71 x 36 x 32), where there are many workgroups (200 x 200 x 140:
500 and 395, with one point per lane 1000 and 785) and where rows stay apart
(48^3; 72 x 36 x 32; 200 x 64 x 40), with two points per lane and with one,
aligned and not.  The bound of tests/test_gpu_flat_rows.py: 16 roundings of the
largest term.
"""
import numpy as np
import pytest

from oracle import operators as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(150, 130, 100), (16, 250, 250), (48, 48, 48), (200, 64, 40), (71, 36, 32), (72, 36, 32),
                                   (200, 200, 140)])
@pytest.mark.parametrize("kind", ["const", "field"])
def test_both_layouts(shape, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    rng = np.random.default_rng(sum(shape))
    h = tuple(1.0 / n for n in shape)
    n = int(np.prod(shape))
    coef = 1.3 if kind == "const" else 1.0 + 0.4 * rng.random(n)
    op, A = E.StencilOp(shape, h, "neumann0", coef=coef), O.stencil_matrix(shape, h, "neumann0", coef=coef)
    x = rng.uniform(-1, 1, n)
    bound = 16 * 2.0**-53 * abs(A).sum(axis=1).max()
    want = A @ x
    room = torch.empty(2 * n + 2, dtype=torch.float64, device="cuda:0")
    for off in (0, 1):                 # 16-byte aligned, and by 8 bytes only
        xt = room[off:off + n]
        yt = room[off + n:off + 2 * n]
        xt.copy_(torch.as_tensor(x))
        print(f"layout {shape} {kind} offset {off}", flush=True)
        E.apply_op(op, 1.0, 0.0, xt, y=yt)
        assert np.abs(yt.cpu().numpy() - want).max() <= bound
    # the norms of both layouts end the loop at the oracle's degree
    from oracle import integrators as I
    a, b = O.gershgorin_interval(A)
    y, s = E.phi_action(op, 1, 13.0 / (b - a), torch.as_tensor(x, device="cuda:0"), tol=1e-8,
                        params=E.LejaParams(pairs=False))
    yo, so = I.phi_action(A, 1, 13.0 / (b - a), x, 1e-8)
    assert s["degree_last"] == so.degrees[-1]
    assert np.linalg.norm(y.cpu().numpy() - yo) <= 1e-10 * np.linalg.norm(yo)
