"""LNCC calls whose gradient overlaps the moving image give what they give with
buffers apart: the image is sampled before the gradient's first store to it."""
import pytest
import torch

from paper_2404_01249_amd import fa, synth

pytestmark = pytest.mark.gpu


def evaluate(entry, shape, window, fixed, moving, d, grad):
    loss = torch.empty((), device="cuda")
    if entry == "noalloc":
        fa.fa_lncc_eval_noalloc(shape, window, 1e-5, fixed, moving, d, loss, grad)
    else:
        h = fa.fa_lncc_create(shape, window)
        fa.fa_lncc_eval(h, fixed, moving, d, loss, grad)
        torch.cuda.synchronize()
        fa.fa_lncc_destroy(h)
    return loss


@pytest.mark.parametrize("entry", ["eval", "noalloc"])
@pytest.mark.parametrize("shape,window", [((9, 20, 24), 5), ((97, 131, 203), 5), ((67, 69, 71), 9)])
def test_gradient_over_the_moving_image(entry, shape, window):
    p = synth.blobs_pair(shape, seed=51, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
    fixed, moving = (torch.from_numpy(a).cuda() for a in (p.fixed, p.moving))
    # samples far from their voxels, as a workgroup reads where others write
    d = torch.from_numpy(synth.smooth_field(shape, 5, sigma=3.0, max_norm=min(shape) / 3)).cuda()
    want = torch.empty((3,) + shape, device="cuda")
    loss = evaluate(entry, shape, window, fixed, moving, d, want)
    n = fixed.numel()
    # in the gradient's first and last component, across two, and over its ends
    for at in (0, 2 * n, n // 2 + 1, -n // 2, 3 * n - n // 3):
        room = torch.zeros(5 * n, device="cuda")
        grad = room[n:4 * n].view((3,) + shape)
        image = room[n + at:2 * n + at].view(shape)
        image.copy_(moving)
        got = evaluate(entry, shape, window, fixed, image, d, grad)
        assert torch.equal(got, loss) and torch.equal(grad, want), at


def test_no_room_for_a_copy():
    shape = (160, 192, 224)   # accepted, but not twice
    grad = torch.zeros((3,) + shape, device="cuda")
    fixed, loss = torch.zeros(shape, device="cuda"), torch.empty((), device="cuda")
    with pytest.raises(fa.FAError, match="overlaps"):
        fa.fa_lncc_eval_noalloc(shape, 5, 1e-5, fixed, grad[1], torch.zeros_like(grad), loss, grad)
