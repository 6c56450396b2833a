"""Where the warp smoothing finds row pairs of the moving image and where not:
the autotuner times the launch that samples them also for a level of a single
iteration, and a volume whose pairs 32-bit offsets do not reach is sampled by a
launch of its own, alone and in a batch."""
import pytest
import torch

from paper_2404_01249_amd import Pair, fa, run_batch, synth

pytestmark = pytest.mark.gpu


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_autotune_times_the_sampling_launch():
    shape = (90, 100, 117)
    fixed, moving = (torch.rand(shape, device="cuda") for _ in range(2))
    pairs = 2 * 4 * 94 * 104 * 121   # bytes of the row pairs
    fa.fa_autotune_clear()
    with Pair(fixed, moving) as p:
        p.set_schedule([1.0], [1])
        before = free_bytes()
        p.autotune(1)
        assert before - free_bytes() >= pairs   # they are there to be sampled
        p.run()
        with Pair(fixed, moving) as q:          # and serve a longer schedule as it stands
            q.set_schedule([1.0], [3])
            assert fa.fa_pair_get_tiling(q.handle, 0, 2) == fa.fa_pair_get_tiling(p.handle, 0, 2)
    fa.fa_autotune_clear()


def test_volume_without_row_pairs():
    shape = (2, 4100, 4100)   # a padded plane of 2^24 voxels and more
    gen = torch.Generator(device="cuda").manual_seed(2)
    images = [[torch.rand(shape, generator=gen, device="cuda") for _ in range(2)] for _ in range(2)]
    y = torch.linspace(0.0, 60.0, shape[1], device="cuda").view(1, -1, 1)
    x = torch.linspace(0.0, 45.0, shape[2], device="cuda").view(1, 1, -1)
    d0 = torch.stack([(0.4 * torch.sin(y) * torch.cos(x)).expand(shape), (1.5 * torch.cos(x + y)).expand(shape),
                      (1.5 * torch.sin(x - y)).expand(shape)]).contiguous()
    want = []
    for fixed, moving in images:
        got = []
        for anew in (False, True):
            with Pair(fixed, moving) as p:
                p.set_schedule([1.0], [3])
                p.set_state(d0)
                for k in range(3):
                    p.step(1)
                    p.set_state(p.field() if anew else None, None, None, k + 1)
                got.append(p.field())
        assert torch.equal(got[0], got[1])
        want.append(got[0])
    both = [Pair(fixed, moving) for fixed, moving in images]
    for p in both:
        p.set_schedule([1.0], [3])
        p.set_state(d0)
    run_batch(both)
    for p, w in zip(both, want):
        assert torch.equal(p.field(), w)
        p.close()
