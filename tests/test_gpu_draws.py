"""The variation draws against the oracle's for the same fitness, in both forms
of the tournament (up to four candidates read ahead of the survival decision,
one after the other beyond), with and without an elite copy, and with more
draws than a block has threads.  Whole numbers and copied doubles: equal."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset, oracle_config, records_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("m,r,tsize,pxo,ms_random", [
    (1, 1, 4, 0.5, 0), (2, 3, 1, 0.5, 1), (63, 65, 2, 0.0, 1), (65, 17, 3, 1.0, 0), (300, 200, 4, 0.3, 1),
    (300, 200, 5, 0.7, 0), (20000, 50, 4, 0.5, 1), (20000, 50, 6, 0.5, 1)])
def test_draws_equal_the_oracle(m, r, tsize, pxo, ms_random, precision):
    gens = 6
    d = dataset(90, 20, 3, seed=m)
    s = gsgp.Settings(pop_size=m, pool_size=r, genome_len=15, n_generations_max=gens, seed=5 * m + tsize,
                      tournament_size=tsize, p_crossover=pxo, ms_random=ms_random, mutation_step=3.0,
                      precision=gsgp.PRECISIONS[precision])
    cfg = oracle_config(s)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    copies = 0
    for g in range(1, gens + 1):
        F = R.fitness(0)[0]
        stats = R.generation(1)
        assert records_equal(R.records(0, g, 1)[0], orc.select(cfg, g, F)), g
        copies += int(stats[0, -1]["elite_copied"])
    assert copies or pxo > 0.0  # mutation by so large a step loses the best parent
    R.close()
