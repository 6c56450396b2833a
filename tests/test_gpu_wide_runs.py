"""The smoothing passes with a radius above 6 on axes of one full run of 64
positions, one position more, and several runs with a remainder, against the
oracle's iteration; tolerances of the registration step."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2404_01249_amd import Pair, synth

pytestmark = pytest.mark.gpu

TOL_G, TOL_L = 1e-4, 1e-5


@pytest.mark.parametrize("sigma", [2.5, 6.0, 8.0])
@pytest.mark.parametrize("shape", [(64, 65, 63), (65, 9, 130), (12, 131, 65)])
def test_one_iteration(shape, sigma):
    p = synth.blobs_pair(shape, seed=51, n_blobs=12, sigma_range=(2.0, 5.0), field_sigma=3.0, field_max=2.0)
    d = synth.smooth_field(shape, 52, sigma=3.0, max_norm=1.0).astype(np.float32)
    params = O.Params(eta=0.5, sigma_grad=sigma, sigma_warp=2.5, window=3)
    with Pair(torch.from_numpy(p.fixed).cuda(), torch.from_numpy(p.moving).cuda(), eta=0.5, sigma_grad=sigma,
              sigma_warp=2.5, window=3) as pr:
        pr.set_schedule([1.0], [1])
        pr.set_state(torch.from_numpy(d).cuda(), None, None, 0)
        pr.step(1)
        got, norm, loss = pr.state()[0].cpu().numpy().astype(np.float64), pr.step_norm(), pr.loss_history()[-1]
    zero = np.zeros((3,) + shape)
    want, _, _, want_loss, ex = O.iterate(p.fixed.astype(np.float64), p.moving.astype(np.float64), d.astype(np.float64),
                                          zero, zero, 1, params)
    step = want - d
    assert np.linalg.norm(got - d - step) <= TOL_G * np.linalg.norm(step)
    assert abs(norm - ex["M"]) <= TOL_G * ex["M"] and abs(loss - want_loss) <= TOL_L * abs(want_loss)
