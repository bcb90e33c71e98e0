"""Several plane bins in one launch: the same state, fitness and counters, bit
for bit, as one launch per bin on one stream, at populations with two bins and
with all of them, ragged bins, in launches of fewer steps and replayed as a
graph, and on a part of the population (sim_rollout_split's GPU share)."""
import numpy as np
import pytest

from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import workloads as W

pytestmark = pytest.mark.gpu


def _result(pop, T, times=1, **options):
    sim = S.Simulator(pop, **options)
    for _ in range(times):
        sim.rollout(T)
    out = [sim.fitness(), *sim.get_state(), *sim.counters()]
    sim.close()
    return out


def _mixed():
    return W.concat([W.snake(5), W.boxes(3), W.random_trees(9), W.quadrupeds(2)])


@pytest.mark.parametrize("make,n_bins", [(lambda: W.concat([W.snake(6), W.boxes(7)]), 2), (_mixed, 4),
                                         (lambda: W.random_trees(301), 6)])
@pytest.mark.parametrize("options", [dict(), dict(steps_per_launch=33), dict(use_graph=True)])
def test_one_launch_equals_a_launch_per_bin(make, n_bins, options):
    pop = make()
    want = _result(pop, 120, streams=1)
    h = S.Handle(pop)
    assert len(h.bins()) >= n_bins
    h.close()
    for got, ref in zip(_result(pop, 120, times=3 if options.get("use_graph") else 1, **options), want):
        assert np.array_equal(got, ref, equal_nan=got.dtype.kind == "f")


def test_a_part_of_every_bin():
    pop = W.random_trees(64)
    a, b = S.Simulator(pop), S.Simulator(pop, streams=1)
    ra, rb = a.rollout_split(60, 13, 2), b.rollout_split(60, 13, 2)
    assert ra["n_gpu"] == rb["n_gpu"] == 51
    assert np.array_equal(a.fitness(), b.fitness())
    a.close()
    b.close()
