"""What an initialisation costs must not depend on what the data look like to
the interpreter: times of the same programs on two data sets that differ in one
respect, one after the other on the same GPU.  The bounds lie between what the
two cost when both are evaluated once and when one is evaluated twice."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp, synth

from .gpu_helpers import oracle_config

pytestmark = pytest.mark.gpu


def _data(n_train, n_test, l, seed, kind=""):
    """kind: "zeros" three features are 0 or 1, "large" products of features
    are clamped, "beyond" one value above 2^128."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, (n_train + n_test, l))
    y = X[:, 0] * X[:, 1]
    if kind == "zeros":
        X[:, :3] = rng.integers(0, 2, (n_train + n_test, 3))
    elif kind == "large":
        X *= 1e12
    elif kind == "beyond":
        X[3, 0] = 1e40
    return synth.Dataset(X[:n_train].copy(), y[:n_train].copy(), X[n_train:].copy(), y[n_train:].copy())


def _semantics_ms(settings, sets):
    """ComputeSemantics of a handle on each of `sets`, by turns; the least of 9."""
    handles = [gsgp.Runner(settings, data) for data in sets]
    best = [np.inf] * len(sets)
    for _ in range(10):
        for i, R in enumerate(handles):
            best[i] = min(best[i], R.time_eval()["compute_semantics_ms"])
    for R in handles:
        R.close()
    return best


@pytest.mark.parametrize("n_test", [0, 64])
def test_padding_columns_cost_no_second_evaluation(n_test):
    """The last tile of a run is the same work with and without padding."""
    s = gsgp.Settings(pop_size=512, pool_size=512, genome_len=255, n_generations_max=1, seed=3)
    whole, padded = _semantics_ms(s, [[_data(256 - n_test - d, n_test, 8, i) for i in range(64)] for d in (0, 3)])
    print(f"whole tiles {whole:.3f} ms, padded {padded:.3f} ms")
    assert padded <= 1.3 * whole


@pytest.mark.parametrize("kind", ["zeros", "large", "beyond"])
def test_data_outside_the_threaded_limits_cost_one_evaluation(kind):
    """Where most programs need the checked evaluator, they are not evaluated by
    the threaded one first.  (The checked one alone takes 1.2 to 1.35 times as
    long as the threaded one, both of them more than 1.75 times.)"""
    s = gsgp.Settings(pop_size=512, pool_size=512, genome_len=255, n_generations_max=1, seed=3)
    plain, other = _semantics_ms(s, [[_data(100_000, 25_000, 20, 1, k)] for k in ("", kind)])
    print(f"plain {plain:.3f} ms, {kind} {other:.3f} ms")
    assert other <= 1.55 * plain


@pytest.mark.parametrize("n_train,m,k", [(20_000, 256, 255), (70_000, 512, 63)])
@pytest.mark.parametrize("kind", ["zeros", "large", "beyond"])
def test_values_do_not_depend_on_the_evaluator(kind, n_train, m, k):
    """With one launch for all lists and with two, after the switch to the
    checked evaluator and before it: the oracle's bits."""
    d = _data(n_train, 1_000, 8, 2, kind)
    s = gsgp.Settings(pop_size=m, pool_size=m, genome_len=k, n_generations_max=1, seed=5)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    genomes = orc.genomes(oracle_config(s), 8, orc.TAG_POPULATION, m)
    X = np.concatenate([d.X_train, d.X_test])
    for c in (0, n_train // 2 + 11, n_train + 1_000 - 300):
        want = orc.interpret(*genomes, X[c:c + 300])
        assert np.array_equal(R.semantics_cases(0, 0, c, 300), want), c
    R.close()
