"""Getters that gather on the device: results of every size class (through
the mapped host memory, through the dead population buffer in one piece and
in several) against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp, synth

from .gpu_helpers import dataset, oracle_config

pytestmark = pytest.mark.gpu

# (m, r, n_train, n_test): the mapped memory holds 32,768 values.  m = 1 with
# a larger pool: the dead buffer holds less than the result (several pieces).
SIZES = [(3, 2, 5, 0), (4, 300, 700, 123), (1, 40, 2049, 511), (16, 16, 2047, 1), (64, 8, 513, 64)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("m,r,n_train,n_test", SIZES)
def test_semantics_of_every_size_class_match_the_oracle(m, r, n_train, n_test, precision):
    d = dataset(n_train, n_test, 4, seed=m + n_train)
    s = gsgp.Settings(pop_size=m, pool_size=r, n_generations_max=1, seed=11, precision=gsgp.PRECISIONS[precision])
    R = gsgp.Runner(s, [d])
    R.eval_population()
    X = np.concatenate([d.X_train, d.X_test])
    pop = orc.interpret(*orc.genomes(oracle_config(s), 4, orc.TAG_POPULATION, m), X)
    pool = orc.sigmoid(orc.interpret(*orc.genomes(oracle_config(s), 4, orc.TAG_POOL, r), X))
    if precision == "fp32":
        pop = pop.astype(np.float32).astype(np.float64)
    # the pool's exp may differ by 4 ulp (FP64), or round to a neighbour (FP32)
    tol = 4 * np.spacing(np.maximum(pool, 1e-300)) if precision == "fp64" else 1.2e-7 * pool + 1e-45
    n = n_train + n_test
    assert np.array_equal(R.semantics(0, 0), pop)
    assert np.all(np.abs(R.semantics(0, 1) - pool) <= tol)
    assert np.array_equal(R.semantics_rows(0, 0, m - 1, 1), pop[-1:])
    a = n // 3
    assert np.array_equal(R.semantics_cases(0, 0, a, n - a), pop[:, a:])
    assert np.array_equal(R.semantics_cases(0, 1, n - 1, 1), R.semantics(0, 1)[:, -1:])
    # reading leaves the run as it is
    B = gsgp.Runner(s, [d])
    B.eval_population()
    assert np.array_equal(R.generation(1), B.generation(1))
    assert np.array_equal(R.semantics(0, 0), B.semantics(0, 0))
    R.close()
    B.close()


@pytest.mark.parametrize("runs,gens", [(1, 1), (3, 300), (5, 2000)])
def test_summaries_and_fitness_in_one_or_several_pieces(runs, gens):
    """The mapped memory holds 8,192 summaries: 10,000 of them take two
    pieces; each run's own getter gives the same."""
    data = [dataset(40 + 7 * i, 9, 3, seed=i) for i in range(runs)]
    s = gsgp.Settings(pop_size=6, pool_size=5, genome_len=15, n_generations_max=gens, seed=5)
    R = gsgp.Runner(s, data)
    R.eval_population()
    got = R.generation(gens)
    for i in range(runs):
        assert np.array_equal(R.stats(i, 1, gens), got[i])
        train, test = R.fitness(i)
        last = got[i, -1]
        assert last["best_train_rmse"] == train.min() and last["best_index"] == int(np.argmin(train))
        assert last["best_test_rmse"] == test[last["best_index"]]
    R.close()


def test_fitness_beyond_the_mapped_memory():
    """2 x 17,000 values take the direct copies."""
    d = dataset(30, 10, 2, seed=3)
    s = gsgp.Settings(pop_size=17_000, pool_size=4, genome_len=7, n_generations_max=1, seed=9)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    train, test = R.fitness(0)
    S = R.semantics(0, 0)
    assert np.allclose(train, orc.rmse_rows(S[:, :30].copy(), d.y_train), rtol=1e-12, atol=0)
    assert np.allclose(test, orc.rmse_rows(S[:, 30:].copy(), d.y_test), rtol=1e-12, atol=0)
    R.close()
