"""Blocks of generations slice by slice (FP32, pools beyond an XCD's L2 with a
population of 1,000 at least and some 200 blocks of 128 individuals x 512 cases)
against the same loop a generation at a time: every summary, fitness, record
and semantic value equal; and the choice between them and whole chunks."""
from __future__ import annotations

import time

import numpy as np
import pytest

from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset

pytestmark = pytest.mark.gpu


def _settings(m, r, gens, step, k=15):
    return gsgp.Settings(pop_size=m, pool_size=r, genome_len=k, n_generations_max=gens, seed=m + r,
                         tournament_size=0, p_crossover=0.0, ms_random=1, mutation_step=step, precision=gsgp.FP32)


# The smallest that go by slices, remainders of individuals and cases, test
# chunks, several runs of uneven size, and sums of squares beyond FP32.
@pytest.mark.parametrize("m,r,sizes,step,scale", [
    (1000, 2817, [(12_800, 0)], 0.1, 1.0),
    (1025, 2900, [(11_000, 2_300)], 5.0, 1.0),
    (1151, 3000, [(12_300, 700)], 0.5, 1e12),
    (1300, 3100, [(513, 64), (4_096, 0), (7_000, 1_500), (300, 0), (512, 512)], 3.0, 1.0),
])
def test_slices_equal_single_generations(m, r, sizes, step, scale):
    gens = 15 + 7 + 4
    data = [dataset(n_tr, n_te, 3, seed=m + i) for i, (n_tr, n_te) in enumerate(sizes)]
    for d in data:
        d.X_train *= scale
        d.X_test *= scale
    s = _settings(m, r, gens, step)
    A, B = gsgp.Runner(s, data), gsgp.Runner(s, data)
    A.eval_population()
    B.eval_population()
    for n in (15, 7, 4):
        A.generation(n, stats=False)
    for _ in range(gens):
        B.generation(1, stats=False)
    for i in range(len(data)):
        assert np.array_equal(A.stats(i, 0, gens + 1), B.stats(i, 0, gens + 1)), i
        for a, b in zip(A.fitness(i), B.fitness(i)):
            assert np.array_equal(a, b), i
        assert np.array_equal(A.records(i, 1, gens), B.records(i, 1, gens)), i
        assert np.array_equal(A.semantics(i, 0), B.semantics(i, 0)), i
    A.close()
    B.close()


def _generation_us(m, r, n):
    R = gsgp.Runner(_settings(m, r, 600, 0.1), [dataset(n, n // 4, 3, seed=1)])
    R.eval_population()
    best = np.inf
    for _ in range(13):
        R.stats(0, 0, 1)  # waits
        t = time.perf_counter()
        R.generation(45, stats=False)
        R.stats(0, 0, 1)
        best = min(best, time.perf_counter() - t)
    R.close()
    return best / 45 * 1e6


def test_a_large_pool_costs_a_small_population_little():
    """A small population reads few rows of any pool: 11 us a generation with
    2,000 of them or 40,000 (22 us slice by slice)."""
    small, large = _generation_us(128, 2_000, 5_000), _generation_us(128, 40_000, 5_000)
    print(f"{small:.1f} and {large:.1f} us")
    assert large <= 1.4 * small
