"""The state carried to the next level: trilinear samples of displacement and
moments at corner-aligned positions, the displacement in the new grid's voxels,
against the same in float64.  The grids have runs along n0 with remainders,
rows shorter and longer than a workgroup, and steps by more than one plane (a
finer level followed by a coarser one)."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Pair

pytestmark = pytest.mark.gpu

CASES = [((9, 11, 13), [2.0, 1.0]), ((9, 11, 13), [4.0, 1.3]), ((37, 12, 40), [1.6, 1.0]), ((6, 300, 33), [3.0, 1.0]),
         ((20, 18, 530), [2.0, 1.0]), ((70, 66, 130), [8.0, 1.0]), ((40, 33, 70), [1.0, 3.0]), ((5, 4, 6), [2.5, 1.0])]


def resampled(x, shape):
    for ax in range(3):
        n, m = x.shape[ax + 1], shape[ax]
        pos = torch.arange(m, dtype=torch.float64) * (n - 1) / (m - 1)
        i = pos.floor().long().clamp(max=n - 2)
        t = (pos - i).reshape([m if a == ax + 1 else 1 for a in range(4)])
        x = x.index_select(ax + 1, i) * (1 - t) + x.index_select(ax + 1, i + 1) * t
    return x


@pytest.mark.parametrize("shape,scales", CASES)
def test_state_at_the_next_level(shape, scales):
    g = torch.Generator().manual_seed(8)
    images = [torch.rand(shape, generator=g).cuda() for _ in range(2)]
    with Pair(*images) as pr:
        pr.set_schedule(scales, [0, 0])
        coarse = tuple(pr.level_shape())
        state = [torch.rand((3,) + coarse, generator=g) - 0.5 for _ in range(2)] + [torch.rand((3,) + coarse, generator=g)]
        pr.set_state(*[s.cuda() for s in state])
        pr.step(1)
        fine = tuple(pr.level_shape())
        assert fine != coarse
        for k, (got, s) in enumerate(zip(pr.state(), state)):
            want = resampled(s.double(), fine)
            rho = 1.0
            if k == 0:
                rho = max((f - 1) / (c - 1) for f, c in zip(fine, coarse))
                want = want * torch.tensor([(f - 1) / (c - 1) for f, c in zip(fine, coarse)]).reshape(3, 1, 1, 1)
            # values at most 1: about ten roundings of the sample, positions rounded at up to n
            tol = 2.0 ** -24 * (10 + sum(coarse)) * max(1.0, rho)
            assert (got.cpu().double() - want).abs().max().item() <= tol
