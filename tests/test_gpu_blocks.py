"""Blocks of generations of the loop without selection against the same loop
a generation at a time (a supplied lineage takes that path) and against the
oracle: every summary, fitness, record and semantic value equal."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset, oracle_config, records_equal

pytestmark = pytest.mark.gpu


def _settings(m, r, gens, precision, step=0.1, ms_random=1, flags=0, k=31):
    return gsgp.Settings(pop_size=m, pool_size=r, genome_len=k, n_generations_max=gens, seed=7 * m + gens,
                         tournament_size=0, p_crossover=0.0, ms_random=ms_random, mutation_step=step,
                         precision=gsgp.PRECISIONS[precision], flags=flags)


def _same(A, B, runs, gens):
    for i in range(runs):
        assert np.array_equal(A.stats(i, 0, gens + 1), B.stats(i, 0, gens + 1)), i
        for a, b in zip(A.fitness(i), B.fitness(i)):
            assert np.array_equal(a, b), i
        assert np.array_equal(A.semantics(i, 0), B.semantics(i, 0)), i
        assert np.array_equal(A.records(i, 1, gens), B.records(i, 1, gens)), i


# A large step makes the best parent survive often (several copies in one
# block, copies of copies, the same individual overwritten again); small
# populations make the lines cross.
@pytest.mark.parametrize("precision", ["fp32", "fp32_kahan", "fp64"])
@pytest.mark.parametrize("m,r,n_train,n_test,step", [
    (1, 1, 70, 0, 0.1), (2, 3, 513, 64, 50.0), (3, 5, 1500, 300, 5.0), (17, 9, 64, 7, 2.0), (130, 40, 2048, 513, 0.5),
    (2100, 64, 300, 0, 3.0), (20000, 10, 900, 150, 3.0)])
def test_blocks_equal_single_generations(m, r, n_train, n_test, step, precision):
    gens = 7 + 5 + 4 + 16 + 2
    d = dataset(n_train, n_test, 3, seed=m)
    s = _settings(m, r, gens, precision, step)
    A, B = gsgp.Runner(s, [d]), gsgp.Runner(s, [d])
    A.eval_population()
    B.eval_population()
    for n in (7, 5, 4, 16, 2):  # blocks of up to 7 (15 from 2e7 values on) and single ones
        A.generation(n, stats=False)
    for g in range(gens):
        B.generation(1, stats=False)
    _same(A, B, 1, gens)
    assert m < 2 or A.stats(0, 1, gens)["elite_copied"].sum() > 3  # the copies were met
    # a supplied lineage goes a generation at a time
    C = gsgp.Runner(s, [d])
    C.eval_population()
    C.replay(A.records(0, 1, gens))
    _same(A, C, 1, gens)
    for R in (A, B, C):
        R.close()


# FP32 pools of more than 2,048 rows go slice by slice: blocks of 128
# individuals, whole chunks of 512 cases; products of features of 1e12 overflow
# the FP32 sums of squares.
@pytest.mark.parametrize("m,r,n_train,n_test,step,scale", [
    (1, 2049, 512, 0, 0.1, 1.0), (130, 2100, 1100, 600, 0.5, 1.0), (128, 3000, 1024, 512, 5.0, 1.0),
    (257, 2500, 513, 64, 0.5, 1e12)])
def test_sliced_blocks_equal_single_generations(m, r, n_train, n_test, step, scale):
    gens = 15 + 7 + 5 + 4 + 2
    d = dataset(n_train, n_test, 3, seed=m)
    d.X_train *= scale
    d.X_test *= scale
    s = _settings(m, r, gens, "fp32", step)
    A, B = gsgp.Runner(s, [d]), gsgp.Runner(s, [d])
    A.eval_population()
    B.eval_population()
    for n in (15, 7, 5, 4, 2):
        A.generation(n, stats=False)
    for g in range(gens):
        B.generation(1, stats=False)
    _same(A, B, 1, gens)
    for R in (A, B):
        R.close()


def test_blocks_of_several_runs_plain_and_guarded():
    data = [dataset(500 + 300 * i, 90 * i, 2 + i, seed=i) for i in range(4)]
    gens = 24
    out = []
    for flags in (0, gsgp.FLAG_NO_GRAPH, gsgp.FLAG_GUARDS):
        s = _settings(40, 20, gens, "fp32", 4.0, flags=flags)
        R = gsgp.Runner(s, data)
        R.eval_population()
        R.generation(gens)
        out.append(R)
    one = gsgp.Runner(_settings(40, 20, gens, "fp32", 4.0), data)
    one.eval_population()
    for _ in range(gens):
        one.generation(1)
    for R in out:
        _same(R, one, 4, gens)
        R.close()
    # restart, another shape, and a checkpoint in the middle of a block
    one.eval_population()
    one.generation(10)
    blob = one.checkpoint()
    one.generation(14)
    two = gsgp.Runner(_settings(40, 20, gens, "fp32", 4.0), data)
    two.restore(blob)
    two.set_launch(2, 8, 0, 0)
    two.generation(14)
    _same(one, two, 4, gens)
    one.close()
    two.close()


@pytest.mark.parametrize("ms_random", [0, 1])
def test_blocks_follow_the_oracle(ms_random):
    d = dataset(400, 150, 4, seed=5)
    gens = 21
    s = _settings(48, 32, gens, "fp64", 0.8, ms_random)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    R.generation(gens)
    res = orc.run(oracle_config(s), d.X_train, d.y_train, d.X_test, d.y_test, gens)
    assert records_equal(R.records(0, 1, gens), res.records)
    S = R.semantics(0, 0)
    want = np.concatenate([res.S_train, res.S_test], axis=1)
    assert np.max(np.abs(S - want) / np.maximum(np.abs(want), 1.0)) <= 1e-12
    assert np.max(np.abs(R.fitness(0)[0] - res.F) / res.F) <= 1e-12
    R.close()
