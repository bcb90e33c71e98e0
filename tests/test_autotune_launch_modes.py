"""The autotuner compares contact budgets within one launch mode: a budget that
the one launch of all bins has no kernel for is tried against a launch per bin,
and a layout that different options lead to is timed once (a cost model in the
place of the GPU)."""
import numpy as np

from paper_2502_11129_amd import autotune as A
from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import workloads as W


def _tune(monkeypatch, pop, cost):
    def timer(pop, T, reps, **opts):
        h = S.Handle(pop, **opts)
        bins, one, fac = h.bins(), h.one_launch(), h.bin_factorization()
        h.close()
        return cost({b[0]: b[2] for b in bins}, one, bins, opts, fac), bins
    monkeypatch.setattr(A, "_time_rollout", timer)
    return A.autotune(pop, T_pilot=100, reps=1)


def _layout(pop, o):
    h = S.Handle(pop, **o)
    bins, one, fac = h.bins(), h.one_launch(), h.bin_factorization()
    h.close()
    streams = 1 if one else min(o.get("streams") or len(bins), len(bins))
    return tuple(bins), tuple(fac), one, streams, o.get("steps_per_launch") or 1000, bool(o.get("use_graph"))


def test_two_budgets_that_pay_only_together_and_apart_are_found(monkeypatch):
    pop = W.random_trees(300)

    def cost(ncr, one, bins, opts, fac):
        # apart costs 15 % more; 2 contacts for 24 and for 28 DoFs save 10 % each there
        return (1.0 if one else 1.15) * (0.9 if ncr.get(24) == 2 else 1.0) * (0.9 if ncr.get(28) == 2 else 1.0) \
            + 0.01 * len(bins)
    best, trials = _tune(monkeypatch, pop, cost)
    assert best["ncr_by_nvc"].get(24) == 2 and best["ncr_by_nvc"].get(28) == 2
    assert best in [t["options"] for t in trials]
    layouts = [_layout(pop, t["options"]) for t in trials if not t.get("final")]
    assert len(set(layouts)) == len(layouts)             # nothing timed twice
    # a budget tried on top of the starting layouts' leaves a launch per bin only for another such
    apart = [t["options"] for t, l in zip(trials, layouts) if not l[2] and t["options"]["streams"] == 0]
    assert not apart


def test_the_one_launch_is_kept_where_it_is_fastest(monkeypatch):
    pop = W.random_trees(300)
    best, _ = _tune(monkeypatch, pop, lambda ncr, one, bins, opts, fac: (1.0 if one else 1.5) + 0.01 * len(bins))
    h = S.Handle(pop, **best)
    assert h.one_launch()
    h.close()


def test_populations_of_one_bin_and_without_the_one_launch(monkeypatch):
    for pop in (W.snake(4), W.box_and_ball(5), W.quadrupeds(3)):
        want = {b[:3] for b in S.Handle(pop).bins()}
        best, trials = _tune(monkeypatch, pop, lambda ncr, one, bins, opts, fac: 1.0)
        assert {b[:3] for b in S.Handle(pop, **best).bins()} == want
        assert all(np.isfinite(t["seconds"]) for t in trials)
