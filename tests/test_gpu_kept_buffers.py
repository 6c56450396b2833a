"""Handles that keep their buffers from one run to the next (the inverse's
level fields and taps, the symmetric registration's inverse and tables) give
what a fresh handle gives, bit for bit, whether the next schedule has the same
grids, others, or more of them."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Inverse, Symmetric, synth

pytestmark = pytest.mark.gpu

SCHEDULES = [([2.0, 1.0], [3, 2]), ([2.0, 1.0], [1, 4]), ([1.0], [3]), ([3.0, 2.0, 1.0], [2, 2, 2]), ([2.0, 1.0], [3, 2])]


def test_inverse_schedules_in_turn():
    shape = (21, 26, 33)
    d = torch.from_numpy(synth.smooth_field(shape, 3, sigma=2.0, max_norm=2.0).astype(np.float32)).cuda()

    def run(inv, schedule):
        inv.set_schedule(*schedule)
        inv.run()
        return inv.field(), inv.loss_history()

    with Inverse(d, eta=0.4) as kept:
        for schedule in SCHEDULES:
            with Inverse(d, eta=0.4) as fresh:
                want = run(fresh, schedule)
            got = run(kept, schedule)
            assert torch.equal(got[0], want[0]) and np.array_equal(got[1], want[1])


def test_symmetric_finishes_in_turn():
    shape = (20, 24, 28)
    p = synth.blobs_pair(shape, seed=4, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
    fixed, moving = (torch.from_numpy(a).cuda() for a in (p.fixed, p.moving))

    def run(sym, k, schedule):
        sym.set_schedule(*SCHEDULES[k % 2])
        sym.run()
        d = sym.finish(*schedule, eta=0.2 + 0.1 * k, sigma_grad=1.0 + 0.5 * (k % 3))
        return d, sym.inverse_cost, sym.loss_history()

    with Symmetric(fixed, moving, eta=0.4) as kept:
        for k, schedule in enumerate(SCHEDULES):
            with Symmetric(fixed, moving, eta=0.4) as fresh:
                want = run(fresh, k, schedule)
            got = run(kept, k, schedule)
            assert torch.equal(got[0], want[0]) and got[1] == want[1] and np.array_equal(got[2], want[2])
