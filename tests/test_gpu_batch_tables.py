"""The launch tables of a batch whose registrations end one after another: each
end sends new tables, and what they take stays bounded while the call runs."""
import threading

import pytest
import torch

from paper_2404_01249_amd import Pair, run_batch

pytestmark = pytest.mark.gpu


def test_tables_stay_bounded():
    # 1500 bricks a launch on few voxels: the tables of 256 take 6 MB, of the 128
    # that run to the end 3 MB
    shape, count, steps = (5, 9, 6000), 256, 128
    iters = [min(1 + k, steps + 2) for k in range(count)]
    gen = torch.Generator(device="cuda").manual_seed(4)
    fixed, moving = (torch.rand(shape, generator=gen, device="cuda") for _ in range(2))
    pairs = [Pair(fixed, moving, eta=0.1 + 0.001 * k) for k in range(count)]
    for k, p in enumerate(pairs):
        p.set_schedule([1.0], [iters[k]])
    run_batch(pairs[:2])   # what a first batch allocates besides
    for k in range(2):
        pairs[k].set_schedule([1.0], [iters[k]])
    torch.cuda.synchronize()
    free = [torch.cuda.mem_get_info()[0]]
    done = threading.Event()

    def watch():
        while not done.is_set():
            free.append(torch.cuda.mem_get_info()[0])

    watcher = threading.Thread(target=watch)
    watcher.start()
    try:
        run_batch(pairs)
    finally:
        done.set()
        watcher.join()
    # two tables may be held at a time, not 128
    assert free[0] - min(free) <= 32 << 20, (free[0] - min(free), len(free))
    # registrations that ended early and late equal their runs alone
    for k in (0, 1, 100, 255):
        with Pair(fixed, moving, eta=0.1 + 0.001 * k) as alone:
            alone.set_schedule([1.0], [iters[k]])
            alone.run()
            assert torch.equal(alone.field(), pairs[k].field())
    for p in pairs:
        p.close()
