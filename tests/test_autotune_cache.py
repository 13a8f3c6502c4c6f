"""What a cached tile setting does to an operator (no GPU: a stand-in operator
records the calls)."""
import pytest

from paper_1309_4616_amd import autotune


class Recorder:
    def __init__(self, shape):
        self.shape = shape
        self.pairs = 1

    def set_tiles(self, *t):
        self.tiles = t

    def set_pairs(self, use):
        self.pairs = use


@pytest.mark.parametrize("shape,entry,pairs", [
    ((512, 300), {"pairs": True, "pair_rows": 32}, 32),
    ((512, 300), {"pairs": False}, 1),                        # the other passes had not been timed
    ((512, 300), {"pairs": None}, 1),                         # a coefficient without pair sweeps
    ((512, 300), {"pairs": False, "passes_timed": True}, False),
    ((64, 64, 64), {"pairs": False}, False),
    ((64, 64, 64), {"pairs": True}, True),
    ((64, 64, 64), {}, 1),
])
def test_cached_pair_setting(shape, entry, pairs):
    op = Recorder(shape)
    autotune._apply(op, {"tiles": [2, 4, 8], **entry})
    assert op.tiles == (2, 4, 8)
    assert op.pairs == pairs and type(op.pairs) is type(pairs)
