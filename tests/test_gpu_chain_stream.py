"""Chains with streaming stores (FP64 vectors that together exceed the
last-level cache; strips on whole cache lines, eight columns computed twice at
each inner end) against the launch-by-launch path, every boundary handling: a
width of whole strips and lines, and a ragged even one.

Both paths form every product and sum by the same operations up to the few
single products of the loop; a point differs by the rounding of at most a few
dozen terms of the Newton sum, bounded by 1e-12 of the largest value.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["dirichlet0", "neumann0", "interior_only"])
@pytest.mark.parametrize("shape", [(4096, 2750), (3010, 3737)])
def test_streaming_chains(shape, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1309_4616_amd as E
    h = tuple(1.0 / (n + 1) for n in shape)
    new = lambda: E.StencilOp(shape, h, bc, coef=1.3)
    op, n = new(), shape[0] * shape[1]
    kw = {}
    if bc == "interior_only":     # the outermost rows are zero: Gershgorin's upper end is 0 either way
        a, b = -8.0 * 1.3 / min(h) ** 2, 0.0
        kw = {"interval": (a, b)}
    else:
        a, b = op.interval()
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    v = torch.rand(n, generator=g, dtype=torch.float64, device="cuda:0") * 2 - 1
    for z in (13.0, 30.0, 60.0):
        print(f"stream {shape} {bc} z={z}", flush=True)
        for call in range(6):
            y, s = E.phi_action(op, 1, z / (b - a), v, tol=1e-10, params=E.LejaParams(**kw))
        x, r = E.phi_action(new(), 1, z / (b - a), v, tol=1e-10, params=E.LejaParams(profile=True, **kw))
        assert s["degree_last"] == r["degree_last"] and s["pair_launches"] > 0
        assert float((x - y).abs().max()) <= 1e-12 * float(x.abs().max()), z
