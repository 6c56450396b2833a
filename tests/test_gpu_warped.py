"""The warped image and its slope, which the warp smoothing leaves for the next
iteration's gradient, equal a fresh sample of the moving image at the same
displacement: a run is bitwise the run whose displacement is set anew, to its
own value, after every iteration (which discards them)."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Pair, synth

pytestmark = pytest.mark.gpu

# brick launches, an 8-row march, ragged 16-row tiles, tiles and chunks with
# remainders; a stationary warp width, the widest narrow one and a wide one
CASES = [
    ((9, 11, 13), 5, 0.5), ((33, 40, 50), 3, 0.5), ((70, 12, 400), 5, 0.5), ((67, 69, 71), 5, 0.0),
    ((48, 80, 90), 7, 1.0), ((41, 83, 97), 9, 2.0), ((40, 90, 95), 5, 2.5),
]


@pytest.mark.parametrize("shape,window,sigma_warp", CASES)
def test_kept_sample_is_a_fresh_one(shape, window, sigma_warp):
    p = synth.blobs_pair(shape, seed=11, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
    fixed, moving = (torch.from_numpy(a).cuda() for a in (p.fixed, p.moving))
    # displacements past the faces as well: samples off the grid on every side
    d0 = torch.from_numpy(synth.smooth_field(shape, 12, sigma=3.0, max_norm=4.0)).cuda()
    fields = []
    for anew in (False, True):
        with Pair(fixed, moving, window=window, sigma_warp=sigma_warp) as pr:
            pr.set_schedule([1.0], [4])
            pr.set_state(d0)
            for k in range(4):
                pr.step(1)
                # the step count is set in both runs, the displacement in one
                pr.set_state(pr.field() if anew else None, None, None, k + 1)
            fields.append((pr.field(), pr.loss_history()))
    assert torch.equal(fields[0][0], fields[1][0])
    assert np.array_equal(fields[0][1], fields[1][1])
