"""sim_fitness with a device pointer: the values and the order of the host call."""
import numpy as np
import pytest
import torch

from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import workloads as W

pytestmark = pytest.mark.gpu


# one variant; several bins whose packed order is not the user order, below,
# at and past one 256-thread block of the largest bin
@pytest.mark.parametrize("n", [1, 65, 1300])
def test_device_fitness_equals_host_fitness(n):
    pop = W.population_from_genotypes(W.random_genotypes(n, key=71))
    sim = S.Simulator(pop)
    sim.rollout(40)
    host = sim.fitness()
    assert n == 1 or len(set(sim.variant_bins().tolist())) > 1
    out = torch.full((n + 8,), -7.0, device="cuda")
    got = sim.fitness_device(out[:n])
    assert np.array_equal(got.cpu().numpy(), host)
    assert (out[n:] == -7.0).all()
    sim.close()
