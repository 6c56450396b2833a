"""The inverse's direction from voxels listed by cell equals, bit for bit, the
one from a global-atomic splat: both add the same fixed-point integers.  Covers
both tile sizes, tiles with remainders, grids of two nodes, cells with more
voxels than a list holds, and samples off the grid."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Inverse, synth

pytestmark = pytest.mark.gpu


def field(kind, shape):
    grid = np.stack(np.meshgrid(*[np.arange(n, dtype=np.float32) for n in shape], indexing="ij"))
    centre = (np.array(shape, np.float32).reshape(3, 1, 1, 1) - 1) / 2
    smooth = synth.smooth_field(shape, 7, sigma=2.0, max_norm=2.0).astype(np.float32)
    if kind == "smooth":
        return smooth
    if kind == "contracting":      # about 37 voxels to a cell in the middle, none outside
        return (0.7 * (centre - grid) + 0.1 * smooth).astype(np.float32)
    if kind == "one cell":         # every voxel to the same position
        return (centre + np.float32(0.3) - grid).astype(np.float32)
    if kind == "expanding":        # most samples off the grid
        return (1.5 * (grid - centre) + 0.1 * smooth).astype(np.float32)
    d = smooth.copy()              # a whole plane far outside, on both sides
    d[0, 0] += 1e6
    d[2, -1] -= 1e6
    return d


CASES = [((2, 2, 2), "smooth"), ((3, 17, 33), "smooth"), ((3, 17, 33), "expanding"), ((19, 23, 37), "contracting"),
         ((12, 9, 20), "one cell"), ((9, 20, 17), "outside"), ((70, 67, 69), "smooth"), ((70, 67, 69), "contracting"),
         ((70, 67, 69), "outside")]


@pytest.mark.parametrize("shape,kind", CASES)
def test_listed_splat_is_the_direct_splat(shape, kind):
    d = torch.from_numpy(field(kind, shape)).cuda()
    out = []
    for switch in (False, True):
        with Inverse(d, eta=0.5) as inv:
            inv.set_schedule([1.0], [4])
            inv.step(2)
            inv.set_splat(switch)
            g, loss = inv.eval_gradient()
            g = g.clone()
            inv.step(2)
            out.append((g, inv.field(), inv.loss_history(), loss))
    (g0, f0, h0, l0), (g1, f1, h1, l1) = out
    assert torch.equal(g0, g1) and torch.equal(f0, f1)
    # the same residuals summed in double in another order, rounded to float once
    assert np.all(np.abs(h0 - h1) <= np.spacing(np.abs(h1))) and abs(l0 - l1) <= np.spacing(np.float32(l1))
