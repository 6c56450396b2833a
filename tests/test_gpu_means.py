"""The intensity means that LNCC takes out of both images: with a constant of
1000 added, the fp32 window variances are right only if the means are, whatever
the number of workgroups that sum them (one, some of the counters' slots, all),
and call after call (the workgroups' counters start each call at zero)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2404_01249_amd import LNCC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 2, 2), (5, 7, 9), (16, 17, 33), (21, 20, 21), (32, 16, 17), (88, 80, 80)])
def test_loss_with_a_large_offset(shape):
    rng = np.random.default_rng(3)
    d = np.zeros((3,) + shape, np.float32)
    lncc = LNCC(shape, window=3)
    for offsets in ((1000.0, -1000.0), (-1000.0, 500.0), (0.0, 1000.0)):
        f, m = ((rng.random(shape) + c).astype(np.float32) for c in offsets)
        _, want = O.gateaux_gradient(f.astype(np.float64), m.astype(np.float64), d.astype(np.float64), 3, 1e-5)
        args = [torch.from_numpy(a).cuda() for a in (f, m, d)]
        got = [float(lncc.loss_and_grad(*args)[0]), float(lncc(*args)), float(lncc.loss_and_grad(*args)[0])]
        # fp32 variances of values below 1, of 27 terms each; 1e-4 leaves a factor of ten, a mean off by 1 gives 0.05
        assert all(abs(g - want) <= 1e-4 for g in got), (got, want)
    lncc.close()
