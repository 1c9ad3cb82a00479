"""Coarse steps under the graph flag while one thread steps several simulations
in turn: replayed or launched, the same bits."""
import numpy as np
import pytest
import torch

from paper_2308_08085_amd import abi, workloads as W

from meshcheck import random_tags

pytestmark = pytest.mark.gpu


def _case(i, storage):
    if i == 2:
        return W.cylinder(2, 9, (64, 32), 8, 16, 3, 100.0, storage=storage, cap=3000, seed=50)
    if i == 3:  # three launches per coarse step: never replayed
        return W.cavity(3, 19, 16, 2, 100.0, storage=storage, cap=1200, seed=51)
    return W.cavity(2, 9, 32, 3 + i % 2, 100.0, storage=storage, cap=2000, seed=52 + i)


def _tags(g, seed):
    return random_tags(g.case, g.mesh(), np.random.default_rng(seed), 0.3, 0.2)


def _sim(case, stream=None):
    g = abi.AmrLbm(case, stream=stream)
    g.set_root_rho_u(case.initial_rho_u())
    for k in range(case.lmax - 1):
        g.tag(tags_in=_tags(g, k))
        g.adapt()
    return g


def _equal(graph, eager):
    for a, b in zip(graph, eager):
        assert np.array_equal(a.get_block_f_all(), b.get_block_f_all())
        assert np.array_equal(a.force(), b.force()) and np.array_equal(a.parity(), b.parity())


@pytest.mark.parametrize("storage", ["f64", "f16s"])
def test_simulations_stepped_in_turn(storage):
    """steps of odd and even counts, mesh changes, and changes of what a captured
    step holds, each followed by enough rounds to be replayed"""
    graph, eager = ([_sim(_case(i, storage)) for i in range(5)] for _ in range(2))

    def rounds(steps):
        for n in steps:
            for g in graph:
                g.step(n, graph=True)
            torch.cuda.synchronize()  # the next round finds every stream out of work
        for g in eager:
            g.step(sum(steps))
        _equal(graph, eager)

    rounds([2, 1, 1, 3, 2, 1])
    for k in range(2):
        for a, b in zip(graph, eager):
            t = _tags(a, 60 + k)
            assert np.array_equal(a.tag(tags_in=t), b.tag(tags_in=t))
            a.adapt(), b.adapt()
        rounds([1, 1, 1, 2, 1])
    for change in (lambda g: g.force_accumulation(False), lambda g: g.skip_parents(True),
                   lambda g: g.stream_bytes(0), lambda g: g.force_accumulation(True)):
        for g in graph + eager:
            change(g)
        rounds([1, 2, 1, 1])
    for g in graph + eager:
        g.close()


def test_batches_stepped_in_turn():
    """batches, whose captured steps outlive mesh changes, in both schedules"""
    def batch():
        st = torch.cuda.Stream()
        sims = [_sim(_case(i, "f32s"), st) for i in (0, 2, 3)]
        return abi.AmrBatch(sims), sims

    graph, eager = ([batch() for _ in range(3)] for _ in range(2))
    for schedule in (0, 1):
        for b, _ in graph + eager:
            b.set_tuning(threads=128, wg_per_cu=4, schedule=schedule)
        for it in range(3):
            for n in (1, 1, 2, 1, 3):
                for b, _ in graph:
                    b.step(n, graph=True)
                torch.cuda.synchronize()
            for b, _ in eager:
                b.step(8, graph=False)
            for (_, x), (_, y) in zip(graph, eager):
                _equal(x, y)
                for g, h in zip(x, y):
                    t = _tags(g, 70 + it)
                    assert np.array_equal(g.tag(tags_in=t), h.tag(tags_in=t))
                    g.adapt(), h.adapt()
    for b, sims in graph + eager:
        b.close()
        for g in sims:
            g.close()


def test_steps_inside_a_capture_of_the_caller():
    """with the flag, steps of several simulations go into the caller's own
    graph as launches; it is replayed with eager work in between"""
    a, b, ref = (_sim(_case(0, "f64")) for _ in range(3))
    for _ in range(3):
        a.step(2, graph=True)
        b.step(2, graph=True)
        torch.cuda.synchronize()
    ref.step(6)
    g = torch.cuda.CUDAGraph()
    b.step(1, graph=True)  # another simulation's steps are under way
    with torch.cuda.graph(g, stream=a.stream):
        a.step(2, graph=True)  # an even number: back to the same buffers
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.step(2)
        assert np.array_equal(a.get_block_f_all(), ref.get_block_f_all())
    for x in (a, b, ref):
        x.close()
