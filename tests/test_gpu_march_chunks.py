"""The march of the gradient kernel: a voxel's gradient does not depend on where
its chunk of planes begins, and a registration's chunks are those that
fa_plan_tiling states, at every window."""
import pytest
import torch

from paper_2404_01249_amd import Pair, fa, synth

pytestmark = pytest.mark.gpu


def images(shape):
    p = synth.blobs_pair(shape, seed=41, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
    return [torch.from_numpy(a).cuda() for a in (p.fixed, p.moving)]


@pytest.mark.parametrize("window", [3, 5, 7, 9])
@pytest.mark.parametrize("ty", [8, 16])
def test_gradient_is_the_same_for_every_chunk(window, ty):
    shape = (29, 37, 70)
    fixed, moving = images(shape)
    d = torch.from_numpy(synth.smooth_field(shape, 5, sigma=3.0, max_norm=2.0)).cuda()
    got = []
    for zc in (29, 1, 4, 13):
        with Pair(fixed, moving, window=window) as p:
            fa.fa_pair_set_tuning(p.handle, 0, ty, 32, zc, 1)
            p.set_schedule([1.0], [1])
            p.set_state(d)
            got.append(p.eval_gradient()[0])
    assert all(torch.equal(g, got[0]) for g in got[1:])


@pytest.mark.parametrize("window", [5, 7, 9])
@pytest.mark.parametrize("shape", [(97, 131, 203), (100, 200, 320), (96, 80, 112)])
def test_registration_takes_the_stated_chunks(window, shape):
    fixed, moving = (torch.rand(shape, device="cuda") for _ in range(2))
    with Pair(fixed, moving, window=window) as p:
        p.set_schedule([1.0], [1])
        ty, tx, zc, brick = fa.fa_pair_get_tiling(p.handle, 0, 0)
    assert not brick and fa.fa_plan_tiling(0, [shape], 4 * (window // 2), False)[0] == [zc]
