"""The contacts that a bin keeps in registers where no budget is asked for:
families of up to 16 DoFs take 16 where most robots of the bin can lie on more
than 8 corners (whatever their first orientation), or go out in one launch with
such a bin, else 8.  The budget never changes results."""
import numpy as np
import pytest

from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import workloads as W


def flat(n, hinges):
    """Chains of equal bricks lying on the plane, four corners of every body down."""
    b = W._Builder(W.ROOT_FREE)
    h = (W.BRICK_HALF,) * 3
    b.add_body(-1, h, W.BRICK_MASS)
    for j in range(hinges):
        b.add_body(j, h, W.BRICK_MASS, "+x", h, W.AXIS_Z, (0.6, 3.0, 0.1 * j))
    b.end_variant(1.0, [0, 0, W.BRICK_HALF + 1e-3, 1, 0, 0, 0] + [0.0] * hinges, [0.0] * (6 + hinges))
    return b.build("flat", 1000).subset(np.zeros(n, int))


def _budgets(pop, **o):
    h = S.Handle(pop, **o)
    out = {b[:2]: b[2] for b in h.bins()}
    h.close()
    return out


@pytest.mark.parametrize("n", [1, 63, 64, 65, 8193])
def test_robots_that_can_lie_on_many_corners_keep_16(n):
    for hinges, cap in ((2, 8), (3, 12), (10, 16)):
        assert _budgets(flat(n, hinges)) == {(cap, 16): 16}
        assert _budgets(flat(n, hinges), streams=1, time_launches=True) == {(cap, 16): 16}


def test_in_any_orientation_bend_and_root():
    p = flat(3, 4)
    for axis in ((1, 0, 0), (0, 1, 0), (0.6, 0, 0.8), (0.48, 0.6, 0.64)):
        q = p.q0.reshape(3, -1).copy()
        q[:, 3:7] = np.concatenate([[np.cos(0.6)], np.sin(0.6) * np.array(axis)])
        p.q0 = q.astype(np.float32).ravel()
        assert _budgets(p) == {(12, 16): 16}
    q[:, 7:] = [0.3, -0.5, 0.2, 0.4]                      # about the vertical: still flat
    p.q0 = q.astype(np.float32).ravel()
    assert _budgets(p) == {(12, 16): 16}
    up = W.chain(4, ["+x"] * 4, [W.AXIS_Y] * 4, theta0=[0.5, 0.4, -0.6, 0.5], root_type=W.ROOT_FREE)
    assert _budgets(up) == {(12, 16): 8}
    fixed = W.chain(5, ["+x"] * 5, [W.AXIS_Z] * 5)
    fixed.half_ext = np.full_like(fixed.half_ext, W.BRICK_HALF)
    assert _budgets(fixed) == {(8, 16): 16}


def test_others_keep_8():
    assert _budgets(W.boxes(9)) == {(8, 16): 8} and _budgets(flat(9, 1)) == {(8, 16): 8}
    assert _budgets(W.snake(16)) == _budgets(W.snake(8193)) == {(12, 16): 8}   # on the core's four and the end
    some = W.concat([flat(49, 3), W.snake(51)])
    assert _budgets(some) == {(12, 16): 8} and _budgets(W.concat([flat(51, 3), W.snake(49)])) == {(12, 16): 16}


def test_several_bins():
    small = W.concat([flat(40, 3), flat(30, 10)])
    assert _budgets(small) == _budgets(small, streams=2) == {(12, 16): 16, (16, 16): 16}
    # in a launch of all bins one bin of flat robots brings 16 for every small bin, apart each has its own
    mixed = W.concat([W.snake(40), flat(40, 10)])
    assert _budgets(mixed) == {(12, 16): 16, (16, 16): 16}
    assert _budgets(mixed, streams=2) == {(12, 16): 8, (16, 16): 16}
    with_large = W.concat([W.snake(9000), W.quadrupeds(2)])
    assert _budgets(with_large) == _budgets(with_large, streams=2) == {(12, 16): 8, (28, 32): 8}
    with_flat = W.concat([flat(9000, 3), W.quadrupeds(2)])
    assert _budgets(with_flat) == _budgets(with_flat, streams=2) == {(12, 16): 16, (28, 32): 8}
    assert set(_budgets(W.random_trees(300)).values()) == {8}
    for pop, o in ((with_large, {}), (with_flat, {}), (mixed, {}), (with_flat, dict(ncr_by_nvc={16: 8})),
                   (W.random_trees(300), dict(ncr_by_nvc={16: 8, 20: 4}))):
        h = S.Handle(pop, **o)
        assert h.one_launch()
        h.close()


def test_a_budget_asked_for_stays():
    p = flat(5, 3)
    assert _budgets(p, contacts_in_registers=2) == {(12, 16): 2}
    assert _budgets(p, ncr_by_nvc={12: 8}) == {(12, 16): 8}
    assert _budgets(p, ncr_by_nvc={16: 8}) == {(12, 16): 16}
    assert _budgets(W.box_and_ball(5)) == {(12, 16): 8}                   # kernels with a ball have no 16
    trees = W.random_trees(60)
    assert _budgets(trees, min_body_slots=32, single_launch=True)[16, 32] == 16
    with pytest.raises(S.SimError, match="nv capacity 16, 32 bodies, 8 contacts"):
        S.Handle(trees, min_body_slots=32, single_launch=True, ncr_by_nvc={16: 8})


@pytest.mark.gpu
@pytest.mark.parametrize("make", [lambda: flat(3, 2), lambda: flat(5, 3), lambda: flat(4, 10),
                                  lambda: W.concat([flat(6, 3), flat(3, 10), W.boxes(2)]),
                                  lambda: W.concat([W.snake(5), flat(3, 10), W.quadrupeds(3), flat(6, 2)]),
                                  lambda: W.concat([flat(6, 2), flat(5, 6), flat(3, 9), W.quadrupeds(3)])])
def test_every_budget_gives_the_same_bits(make):
    pop = make()

    def run(**o):
        sim = S.Simulator(pop, **o)
        sim.rollout(150)
        out = [sim.fitness(), *sim.get_state(), *sim.counters()]
        sim.close()
        return out
    want = run(contacts_in_registers=2)
    assert want[4].max() > 8 * 150                         # rows past a budget of 8 are exercised
    for o in (dict(), dict(streams=1), dict(ncr_by_nvc={8: 8, 12: 8, 16: 8}), dict(ncr_by_nvc={8: 16, 12: 16, 16: 16})):
        for a, b in zip(run(**o), want):
            assert np.array_equal(a, b)
