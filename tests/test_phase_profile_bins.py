"""The phase profiler runs a launch per bin: the kernels of the single launch have
no clocks, so options that lead there keep their bins and contacts in registers
but not the launch (host only)."""
import pytest

from paper_2502_11129_amd import phase_profile as P
from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import workloads as W


@pytest.mark.parametrize("options", [{}, dict(min_body_slots=32), dict(min_body_slots=32, single_launch=True),
                                     dict(ncr_by_nvc={16: 8, 20: 4}), dict(streams=2), dict(ncr_by_nvc={28: 2})])
def test_bins_are_launched_apart(options):
    for pop in (W.random_trees(200), W.quadrupeds(3)):
        want = S.Handle(pop, **options) if not (options.get("single_launch") and pop.n_variants == 3) else S.Handle(pop, min_body_slots=32)
        h = S.Handle(pop, **P.per_bin(pop, options))
        assert not h.one_launch() and h.bins() == want.bins()
        h.close()
        want.close()
    assert P.per_bin(W.random_trees(200), dict(streams=2)) == dict(streams=2)
