"""The march chunks where rounding up would leave one chunk too many for the
resident workgroups: fewer and longer chunks that fit, unless they are more than
half as long again.  Host only."""
import numpy as np
import pytest

from paper_2404_01249_amd import fa

SLOTS = (512, 1024, 512, 512)


@pytest.mark.parametrize("kind,shape,chunk,blocks", [
    (0, (97, 131, 203), 13, 504),      # 12 planes: nine chunks of 63 tiles
    (0, (100, 320, 320), 50, 400),     # 40 planes: 600 workgroups
    (0, (120, 240, 640), 71, 600),     # 120 planes would fit, but are too long
    (0, (128, 128, 128), 8, 512),      # fits as it is
    (1, (97, 131, 203), 7, 882),       # 6 planes: 1071
    (3, (512, 512, 512), 512, 512),
])
def test_chunk(kind, shape, chunk, blocks):
    assert fa.fa_plan_tiling(kind, [shape], 8, False) == ([chunk], [blocks])


def test_any_shape():
    rng = np.random.default_rng(2)
    for _ in range(400):
        kind, shape = int(rng.integers(0, 4)), tuple(int(v) for v in rng.integers(2, 400, 3))
        (z,), (b,) = fa.fa_plan_tiling(kind, [shape], 8, False)
        tiles = -(-shape[1] // (16 if shape[1] >= 16 else 8)) * -(-shape[2] // 32)
        rule = min(shape[0], max(-(-shape[0] * tiles // SLOTS[kind]), (1, 4, 4, 1)[kind]))
        assert b == tiles * -(-shape[0] // z) and rule <= z <= max(rule, rule * 3 // 2)
        assert z == rule or b <= SLOTS[kind] < tiles * -(-shape[0] // rule)
