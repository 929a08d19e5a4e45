"""What an initialisation costs must not depend on what the data look like to
the interpreter: times of the same programs on two data sets that differ in one
respect, one after the other on the same GPU.  The bounds lie between what the
two cost when both are evaluated once and when one is evaluated twice."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2106_04034_amd import gsgp, synth

pytestmark = pytest.mark.gpu


def _data(n_train, n_test, l, seed):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, (n_train + n_test, l))
    y = X[:, 0] * X[:, 1]
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
