"""Steps taken two or three at a time on patches (needs a device): the same bits as
one step a call, which marches strips, at the patches' edges (24 x 8 nodes each for
two steps, 20 x 4 for three; up to 256 of these are taken), on lattices
smaller than one, with every kind of side, and around checking steps."""

import copy
import functools

import numpy as np
import pytest

from paper_2510_18688_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbf_mod():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2510_18688_amd import lbf
    lbf.load()
    return lbf


def _slab(nx, ny, px, py):
    case = W.slab_drop(nx, ny, 0.3 * min(nx, ny), 75.0, -1.0, h_s=min(4.0, 0.4 * ny))
    case.periodic_x, case.periodic_y = px, py
    return case


@functools.lru_cache(None)
def _walls():
    return W.porous_medium(nx=131, ny=67, seed=5, rmin=6.0, rmax=10.0, porosity=0.8)


CASES = {
    "one_node": lambda: _slab(1, 1, True, False),
    "one_node_periodic": lambda: _slab(1, 1, True, True),
    "smaller_periodic": lambda: _slab(5, 3, True, True),
    "one_patch": lambda: _slab(24, 8, True, False),
    "one_patch_walls": lambda: _slab(24, 8, False, False),
    "one_over": lambda: _slab(25, 9, True, True),
    "one_under": lambda: _slab(47, 23, False, True),
    "thin": lambda: _slab(130, 1, True, False),
    "walls": lambda: copy.deepcopy(_walls()),
    "three_steps": lambda: _slab(40, 12, True, False),
    "three_steps_over": lambda: _slab(41, 13, False, True),
    "most_three_steps": lambda: _slab(320, 64, True, False),
    "too_many_for_three": lambda: _slab(321, 64, True, False),
    "eight": lambda: _slab(8, 8, True, True),   # fewer go to strips
    "seven": lambda: _slab(7, 30, True, True),
}


@pytest.mark.parametrize("mdot,mrt", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("rb,check", [(0, 0), (4, 3)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_pairs_of_steps(lbf_mod, name, rb, check, mdot, mrt):
    import torch
    case = CASES[name]()
    case.mat.phi_src_mdot = mdot
    if mrt:
        case.mat.mrt, case.mat.s_b, case.mat.s_q, case.mat.s_g = 1, 1.5, 1.2, 1.4
    a = lbf_mod.Sim(case, row_block=rb, check_every=check)
    b = lbf_mod.Sim(case, row_block=rb, check_every=0)
    sa = torch.empty(a.state_bytes(), dtype=torch.uint8, device="cuda")
    sb = torch.empty_like(sa)
    for steps in (2, 3, 6, 11):
        a.step(steps)
        for _ in range(steps):
            b.step(1)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), steps


@pytest.mark.parametrize("thin", [False, True])
@pytest.mark.parametrize("mrt", [0, 1])
def test_batch_of_patches(lbf_mod, mrt, thin):
    """Batched pairs against the lattices stepped alone, one step a call; a lattice
    too thin for patches sends the whole batch to strips."""
    import torch
    names = ["walls", "eight", "one_over", "one_under"] + (["thin"] if thin else [])

    def sims():
        out = []
        for i, name in enumerate(names):
            case = CASES[name]()
            case.mat.phi_src_mdot = i % 2
            if mrt:
                case.mat.mrt, case.mat.s_b, case.mat.s_q, case.mat.s_g = 1, 1.5, 1.2, 1.4
            out.append(lbf_mod.Sim(case, row_block=(0, 4)[i % 2]))
        return out

    a, b = sims(), sims()
    batch = lbf_mod.Batch(a)
    for steps in (5, 37, 2, 70):
        batch.step(steps)
        for x, y in zip(a, b):
            for _ in range(steps):
                y.step(1)
            sx = torch.empty(x.state_bytes(), dtype=torch.uint8, device="cuda")
            sy = torch.empty_like(sx)
            x.save_state(sx)
            y.save_state(sy)
            assert torch.equal(sx, sy), (steps, x.nx, x.ny, x.case.mat.mrt)


@pytest.mark.parametrize("name", ["most_three_steps", "too_many_for_three", "seven"])
@pytest.mark.parametrize("steps", [2, 4, 6, 8, 10])
def test_captured_call_replays(lbf_mod, name, steps):
    """A captured call of an even number of steps ends in the buffer it began in,
    however its steps were grouped: replays continue from one another."""
    import torch
    stream = torch.cuda.Stream()
    a = lbf_mod.Sim(CASES[name](), check_every=0, stream=stream)
    b = lbf_mod.Sim(CASES[name](), check_every=0)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(steps)
    # (the fields, not the saved states: a replay does not turn the host's step count)
    for _ in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        b.step(steps)
        fa, fb = a.fields(), b.fields()
        for k in fa:
            assert (fa[k].view(np.uint32) == fb[k].view(np.uint32)).all(), k


def _same_fields(a, b, when):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        assert (fa[k].view(np.uint32) == fb[k].view(np.uint32)).all(), (when, k)


@pytest.mark.parametrize("name", ["most_three_steps", "too_many_for_three", "seven"])
@pytest.mark.parametrize("steps", [2, 4, 6, 8])
@pytest.mark.parametrize("check", [0, 9])
def test_replays_among_eager_calls(lbf_mod, name, steps, check):
    """Any call of an even number of steps ends in the buffer it began in, captured or
    not: a replay finds the fields set after the capture and what eager calls leave."""
    import torch
    case = CASES[name]()
    stream = torch.cuda.Stream()
    a = lbf_mod.Sim(case, check_every=check, stream=stream)
    b = lbf_mod.Sim(case, check_every=0)
    a.step(10)                       # levels 10 .. 17 hold no check
    a.step(0 if check else steps)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(steps)

    def replay():
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        b.step(steps)

    a.init_fields(case.phi, case.T)
    replay()
    _same_fields(a, b, "set after the capture")
    for n in (steps, 4, 12):
        a.step(n)
        b.step(n)
        _same_fields(a, b, ("eager", n))
        replay()
        _same_fields(a, b, ("replay after", n))


def test_replay_after_an_unstable_call(lbf_mod):
    """A call that a stability check ends leaves the state in the buffer that step by
    step it would, so that a replay continues from a state loaded after it."""
    import torch
    case = CASES["too_many_for_three"]()
    stream = torch.cuda.Stream()
    a = lbf_mod.Sim(case, check_every=4, stream=stream)
    b = lbf_mod.Sim(case, check_every=0)
    a.step(5)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(2)
    a.init_fields(case.phi, case.T)
    a.step(5)
    b.step(5)
    saved = torch.empty(a.state_bytes(), dtype=torch.uint8, device="cuda")
    a.save_state(saved)
    a.set_wall_temperature(0, np.full(a.nx, np.nan))
    with pytest.raises(lbf_mod.LbfError):
        a.step(9)                    # levels 5, 6, 7, then the check at 8
    a.set_wall_temperature(0, case.wall_profile(0))
    a.load_state(saved)
    with torch.cuda.stream(stream):
        graph.replay()
    stream.synchronize()
    b.step(2)
    # the replay turned the buffers twice: the state is where the host has it
    _same_fields(a, b, "replay")


@pytest.mark.parametrize("n, seg", [(4, 4), (6, 2), (8, 3), (10, 10)])
def test_recorded_run_keeps_the_turn(lbf_mod, n, seg):
    """A recorded run of an even number of steps ends in the buffer it began in,
    whatever its segments (replays after it)."""
    import torch
    case = CASES["too_many_for_three"]()
    case.mat.phi_src_mdot = 1
    stream = torch.cuda.Stream()
    a = lbf_mod.Sim(case, check_every=0, stream=stream, row_block=0)
    b = lbf_mod.Sim(case, check_every=0, row_block=0)
    tape = lbf_mod.Tape(a, n, seg)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(2)
    a.init_fields(case.phi, case.T)
    tape.forward()
    with torch.cuda.stream(stream):
        graph.replay()
    stream.synchronize()
    b.step(n + 2)
    _same_fields(a, b, (n, seg))


def _batch_pair(lbf_mod, stream):
    names = ["walls", "eight", "one_over", "one_under"]
    return ([lbf_mod.Sim(CASES[n](), check_every=0, stream=stream) for n in names],
            [lbf_mod.Sim(CASES[n](), check_every=0) for n in names])


@pytest.mark.parametrize("steps", [2, 4, 6])
def test_batch_replays_among_eager_calls(lbf_mod, steps):
    """A batched call of an even number of steps ends in the buffers it began in: graphs
    captured before it still replay from the state, and neither the capture nor a call
    after it needs new descriptors."""
    import torch
    stream = torch.cuda.Stream()
    a, b = _batch_pair(lbf_mod, stream)
    batch = lbf_mod.Batch(a)
    batch.step(2)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        batch.step(steps)

    def both(n, f):
        f()
        stream.synchronize()
        for x, y in zip(a, b):
            y.step(n)
            _same_fields(x, y, n)

    for y in b:
        y.step(2)
    with torch.cuda.stream(stream):
        for n in (2, 6, 34):
            both(steps, graph.replay)
            both(n, lambda: batch.step(n))
        both(steps, graph.replay)


@pytest.mark.parametrize("nx, ny", [(2048, 800), (1999, 801)])
def test_large_lattices(lbf_mod, nx, ny):
    """More than 8000 patches: pairs on patches, the steps between them on strips."""
    import torch
    a = lbf_mod.Sim(_slab(nx, ny, True, False), check_every=4)
    b = lbf_mod.Sim(_slab(nx, ny, True, False), check_every=0)
    sa = torch.empty(a.state_bytes(), dtype=torch.uint8, device="cuda")
    sb = torch.empty_like(sa)
    for steps in (7, 10):
        a.step(steps)
        for _ in range(steps):
            b.step(1)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), steps


@pytest.mark.parametrize("tile", [(64, 1), (64, 7), (128, 32), (256, 5), (256, 200), (512, 3), (512, 16)])
def test_tiles_step_by_step(lbf_mod, tile):
    """Every step a call's last, so that all of them march strips of the tile."""
    case = _slab(150, 70, True, False)
    a, b = lbf_mod.Sim(case, tile=tile), lbf_mod.Sim(case, tile=(64, 32))
    b.step(20)
    for _ in range(20):
        a.step(1)
    _same_fields(a, b, tile)
