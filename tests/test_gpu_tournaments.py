"""Tournaments beyond the four candidates that are read ahead of the survival
decision: eight candidates at a time, and a remainder.  Records are whole
numbers and copied doubles: equal to the oracle's for the same fitness."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset, oracle_config, records_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 3, 130])
@pytest.mark.parametrize("tsize", [7, 8, 9, 15, 16, 17, 63, 64])
def test_records_equal_the_oracle(m, tsize):
    """Few individuals: equal fitness (an individual drawn twice) at every
    place of a tournament."""
    gens = 4
    d = dataset(90, 20, 3, seed=m)
    s = gsgp.Settings(pop_size=m, pool_size=5, genome_len=15, n_generations_max=gens, seed=9 * m + tsize,
                      tournament_size=tsize, p_crossover=0.6, mutation_step=3.0)
    cfg = oracle_config(s)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    for g in range(1, gens + 1):
        F = R.fitness(0)[0]
        R.generation(1)
        assert records_equal(R.records(0, g, 1)[0], orc.select(cfg, g, F)), g
    R.close()


def test_a_large_tournament_is_no_chain_of_reads():
    """Survival with 64 candidates against the same with 4: 3.3 times as long
    when eight are read at a time, 4.2 times one after the other."""
    us = {}
    for tsize in (4, 64):
        s = gsgp.Settings(pop_size=256, pool_size=64, genome_len=15, n_generations_max=1300, seed=2,
                          tournament_size=tsize, p_crossover=1.0, precision=gsgp.FP32)
        R = gsgp.Runner(s, [dataset(1000, 250, 4, seed=1)])
        R.eval_population()
        us[tsize] = min(R.time_stages(200)["survive_ms"] for _ in range(6)) * 1e3
        R.close()
    print(us)
    assert us[64] <= 3.8 * us[4]
