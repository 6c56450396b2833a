"""The evaluation kernels where their groups of voxels end: rows of the interior
shorter than, equal to and just past a thread's four voxels and a row of
threads; label arrays off a 16-byte boundary, runs of equal labels and tails;
grids of two nodes and samples off the grid for the pair loads."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2404_01249_amd import evaluate, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n2", [3, 4, 5, 6, 7, 9, 10, 11, 34, 35, 130, 258, 259, 263])
@pytest.mark.parametrize("n01", [(3, 3), (4, 11)])
def test_jacobian_rows(n01, n2):
    d = np.random.default_rng(n2).normal(0.0, 0.6, size=(3,) + n01 + (n2,)).astype(np.float32)
    got = evaluate.jacobian_det(torch.from_numpy(d).cuda()).cpu().numpy()
    assert np.array_equal(got, O.jacobian_det(d))
    assert evaluate.singular_fraction(torch.from_numpy(d).cuda()) == O.singular_fraction(d)


@pytest.mark.parametrize("offset", [0, 1, 16])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 4099, 70_001])
def test_overlap_runs_and_tails(n, offset):
    rng = np.random.default_rng(n)
    a = np.repeat(rng.integers(-2, 7, size=n), rng.integers(1, 40, size=n))[:n].astype(np.int8)
    b = np.where(rng.random(n) < 0.9, a, rng.integers(-2, 7, size=n)).astype(np.int8)
    dev = [torch.zeros(n + offset, dtype=torch.int8, device="cuda") for _ in range(2)]
    for t, x in zip(dev, (a, b)):
        t[offset:] = torch.from_numpy(x).cuda()
    got = evaluate.label_overlap(dev[0][offset:], dev[1][offset:], 6)
    assert np.array_equal(got, [[(a == r).sum(), (b == r).sum(), ((a == r) & (b == r)).sum()] for r in range(6)])


@pytest.mark.parametrize("shape", [(2, 2, 2), (2, 5, 3), (4, 3, 31), (3, 6, 97), (3, 4, 200)])
def test_compose_at_the_faces(shape):
    u = synth.smooth_field(shape, 5, sigma=1.0, max_norm=3.0).astype(np.float32)
    d = synth.smooth_field(shape, 6, sigma=1.0, max_norm=2.0).astype(np.float32)
    got = evaluate.compose(torch.from_numpy(u).cuda(), torch.from_numpy(d).cuda()).cpu().numpy().astype(np.float64)
    ref = O.compose(d.astype(np.float64), u.astype(np.float64))
    # about ten roundings of values below 2, one of the sum below 5
    assert np.abs(got - ref).max() <= 2.0 ** -24 * (10 * 2 + 5)
