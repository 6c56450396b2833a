"""Levels of one iteration, which form no row pairs of the moving image: alone
they are bitwise the levels of a schedule that steps on from them, in a batch
the runs on their own, and a schedule of more iterations after them forms them."""
import numpy as np
import pytest
import torch

from paper_2404_01249_amd import Pair, run_batch, synth

pytestmark = pytest.mark.gpu


def pairs(shape, count):
    out = []
    for k in range(count):
        p = synth.blobs_pair(shape, seed=20 + k, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
        out.append([torch.from_numpy(a).cuda() for a in (p.fixed, p.moving)])
    return out


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("shape", [(20, 24, 28), (70, 66, 68)])   # bricks, marches
def test_batch_and_reschedule(shape, graphs):
    images = pairs(shape, 2)
    schedules = [([2.0, 1.0], [1, 1]), ([2.0, 1.0], [3, 2]), ([2.0, 1.0], [1, 3])]
    want = []
    for fixed, moving in images:
        per = []
        for schedule in schedules:
            with Pair(fixed, moving) as fresh:
                fresh.set_schedule(*schedule)
                fresh.run()
                per.append((fresh.field(), fresh.loss_history()))
        with Pair(fixed, moving) as kept:
            for schedule, (field, loss) in zip(schedules, per):
                kept.set_schedule(*schedule)
                kept.run()
                assert torch.equal(kept.field(), field) and np.array_equal(kept.loss_history(), loss)
        want.append(per)
    for k, schedule in enumerate(schedules):
        both = [Pair(fixed, moving) for fixed, moving in images]
        for p in both:
            p.set_schedule(*schedule)
        run_batch(both, graphs=graphs)
        for p, per in zip(both, want):
            assert torch.equal(p.field(), per[k][0])
            p.close()
