"""The inverse of warps that send many voxels into few cells.  Such a level's
direction takes bricks of voxels; it equals the direct splat's bit for bit, on
both tile sizes, with boxes that fit LDS and larger ones, and with boxes over so
many tiles that it walks instead; its loss does not change from call to call;
and it costs about what a warp of no contraction does."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Inverse, fa, synth

pytestmark = pytest.mark.gpu


def field(kind, shape):
    rng = np.random.default_rng(8)
    grid = np.stack(np.meshgrid(*[np.arange(n, dtype=np.float32) for n in shape], indexing="ij"))
    size = np.array(shape, np.float32).reshape(3, 1, 1, 1)
    centre = (size - 1) / 2
    if kind == "half":         # most cells with about eight voxels, some with more
        return (0.5 * (centre - grid) + 0.3 * rng.standard_normal(grid.shape)).astype(np.float32)
    if kind == "contracting":
        return (0.8 * (centre - grid) + 0.1 * rng.standard_normal(grid.shape)).astype(np.float32)
    if kind == "corner":       # onto the grid's first cells and off it
        return (-0.95 * grid - 0.7 + 0.2 * rng.standard_normal(grid.shape)).astype(np.float32)
    if kind == "large boxes":  # each voxel somewhere in the middle eighth per axis
        return (centre + (rng.random(grid.shape) - 0.5) * np.minimum(size / 2, 12) - grid).astype(np.float32)
    assert kind == "two cells"  # neighbours to opposite corners: every box is the grid
    side = (grid.sum(0) % 2).astype(np.float32)
    return (0.4 + side * (size - 2) - grid).astype(np.float32)


KINDS = ["half", "contracting", "corner", "large boxes", "two cells"]
SHAPES = [(2, 3, 4), (5, 18, 33), (40, 20, 37), (70, 67, 69)]   # the last with tiles of 8 x 8 x 16


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", KINDS)
def test_is_the_direct_splat(kind, shape):
    d = torch.from_numpy(field(kind, shape)).cuda()
    out = []
    for switch in (False, True):
        with Inverse(d, eta=0.5) as inv:
            inv.set_schedule([1.0], [4])
            inv.step(2)
            inv.set_splat(switch)
            g, loss = inv.eval_gradient()
            again = inv.eval_gradient()
            assert torch.equal(g, again[0]) and loss == again[1]
            inv.step(2)
            out.append((g, inv.field(), inv.loss_history(), loss))
    (g0, f0, h0, l0), (g1, f1, h1, l1) = out
    assert torch.equal(g0, g1) and torch.equal(f0, f1)
    # the same residuals summed in double in another order, rounded to float once
    assert np.all(np.abs(h0 - h1) <= np.spacing(np.abs(h1))) and abs(l0 - l1) <= np.spacing(np.float32(l1))


def test_levels_and_new_schedules():
    shape = (70, 67, 69)
    want = {}
    with Inverse(torch.from_numpy(field("contracting", shape)).cuda(), eta=0.5) as inv:
        for direct in (True, False, False):
            inv.set_splat(direct)
            inv.set_schedule([2.0, 1.0], [3, 3])
            inv.run()
            assert torch.equal(inv.field(), want.setdefault("field", inv.field()))


def test_costs_no_multiple_of_a_smooth_warp():
    shape = (128, 128, 128)
    smooth = synth.smooth_field((32, 32, 32), 3, sigma=2.0, max_norm=2.0)
    smooth = torch.nn.functional.interpolate(torch.from_numpy(smooth)[None].cuda(), size=shape, mode="trilinear")[0]
    lib = fa.load_library()

    def us(d):
        with Inverse(d) as inv:
            inv.set_schedule([1.0], [1])
            g = torch.empty_like(d)
            best = 1e30
            for _ in range(5):
                t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                t[0].record()
                for _ in range(4):
                    assert lib.fa_inverse_eval_gradient(inv.handle, g.data_ptr(), None) == 0
                t[1].record()
                t[1].synchronize()
                best = min(best, 250.0 * t[0].elapsed_time(t[1]))
        return best

    base = us(smooth.contiguous())
    for factor in (0.8, 0.9):
        grid = torch.stack(torch.meshgrid(*[torch.arange(n, dtype=torch.float32, device="cuda") for n in shape],
                                          indexing="ij"))
        d = factor * (63.5 - grid) + 0.1 * smooth
        assert us(d.contiguous()) <= 6.0 * base   # 2 here, 13 and 33 where a few tiles had all of the work
