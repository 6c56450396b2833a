"""Iterations and gradients captured into a graph by the caller: a replay works
on the displacement that is there when it runs, whatever moved it (replays,
eager steps, a new state), and a capture that is never launched leaves nothing
behind that a later step would take for made.  Against eager runs, bit for bit."""
import pytest
import torch

from paper_2404_01249_amd import Inverse, Pair, fa, synth

pytestmark = pytest.mark.gpu

SHAPES = [(12, 20, 24), (67, 69, 71)]   # bricks, marches


def images(shape):
    p = synth.blobs_pair(shape, seed=31, n_blobs=8, sigma_range=(2.0, 4.0), field_sigma=3.0, field_max=2.0)
    return [torch.from_numpy(a).cuda() for a in (p.fixed, p.moving)]


def state(shape, seed):
    return torch.from_numpy(synth.smooth_field(shape, seed, sigma=3.0, max_norm=2.0)).cuda()


def trajectory(make, count, d0=None):
    """The fields after 0 .. count eager iterations."""
    with make() as h:
        h.set_schedule([1.0], [count + 1])
        if d0 is not None:
            h.set_state(d0)
        out = [h.field()]
        for _ in range(count):
            h.step(1)
            out.append(h.field())
    return out


def captured(h, call):
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=h.stream):
        call()
    return graph


def replay(h, graph):
    with torch.cuda.stream(h.stream):
        graph.replay()


def field(h):
    torch.cuda.synchronize()
    with torch.cuda.stream(h.stream):
        out = h.field()
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("iters", [2, 8])   # the captured iteration is the level's last, or one of many
def test_pair_replays(shape, iters):
    fixed, moving = images(shape)
    want = trajectory(lambda: Pair(fixed, moving), 5)
    d0 = state(shape, 3)
    moved = trajectory(lambda: Pair(fixed, moving), 3, d0)
    torch.cuda.synchronize()
    with Pair(fixed, moving, stream=torch.cuda.Stream()) as p:
        p.set_schedule([1.0], [iters])
        p.step(1)
        graph = captured(p, lambda: p.step(1))
        for k in range(4):
            replay(p, graph)
            assert torch.equal(field(p), want[2 + k])
        p.set_schedule([1.0], [iters])
        p.set_state(d0)
        replay(p, graph)
        assert torch.equal(field(p), moved[1])
        p.step(1)   # eager, after a replay
        assert torch.equal(field(p), moved[2])
        replay(p, graph)
        assert torch.equal(field(p), moved[3])


@pytest.mark.parametrize("shape", SHAPES)
def test_pair_capture_never_launched(shape):
    fixed, moving = images(shape)
    want = trajectory(lambda: Pair(fixed, moving), 2)
    torch.cuda.synchronize()
    with Pair(fixed, moving, stream=torch.cuda.Stream()) as p:
        p.set_schedule([1.0], [8])
        captured(p, lambda: p.step(1))
        for k in range(2):
            p.step(1)
            assert torch.equal(field(p), want[1 + k])


@pytest.mark.parametrize("shape", SHAPES)
def test_captured_gradient_follows_the_displacement(shape):
    fixed, moving = images(shape)
    torch.cuda.synchronize()
    with Pair(fixed, moving, stream=torch.cuda.Stream()) as p:
        p.set_schedule([1.0], [4])
        g = torch.empty((3,) + shape, device="cuda")
        torch.cuda.synchronize()
        p.eval_gradient()   # J is made for the initial displacement
        graph = captured(p, lambda: fa.load_library().fa_pair_eval_gradient(p.handle, g.data_ptr(), None))
        for seed in (3, 4, 5):
            p.set_state(state(shape, seed))
            replay(p, graph)
            torch.cuda.synchronize()
            assert torch.equal(g, p.eval_gradient()[0])
            torch.cuda.synchronize()


@pytest.mark.parametrize("shape", SHAPES)
def test_inverse_captures(shape):
    d = state(shape, 6)
    want = trajectory(lambda: Inverse(d), 6)
    torch.cuda.synchronize()
    with Inverse(d, stream=torch.cuda.Stream()) as inv:
        inv.set_schedule([1.0], [10])
        captured(inv, lambda: inv.step(1))   # never launched
        inv.step(2)
        assert torch.equal(field(inv), want[2])
        graph = captured(inv, lambda: inv.step(1))
        for k in range(3):
            replay(inv, graph)
            assert torch.equal(field(inv), want[3 + k])
        inv.step(1)
        assert torch.equal(field(inv), want[6])
