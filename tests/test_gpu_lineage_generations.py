"""Reconstruction of individuals of earlier generations than the current one:
the walk starts at their generation's records, summaries and scaling, while the
scratch it uses follows from the current one.  FP64 repeats the operations that
formed the stored semantics: equal, with local search to rounding."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset

pytestmark = pytest.mark.gpu


# Walks on the host (fewer than 64 individuals) and on the device, one and two
# individuals a thread; earlier generations of both parities, and the last
# generation of both.
@pytest.mark.parametrize("m,r,stops,flags", [
    (30, 20, (0, 5, 12, 13), 0),
    (64, 65, (0, 1, 2, 7, 70, 71), 0),
    (300, 200, (0, 3, 8, 20), 0),
    (1100, 300, (0, 4, 9, 11), 0),
    (30, 20, (0, 5, 12, 13), gsgp.FLAG_LOCAL_SEARCH),
    (300, 200, (0, 3, 8, 20), gsgp.FLAG_LOCAL_SEARCH),
])
def test_earlier_generations_repeat_their_semantics(m, r, stops, flags):
    d = dataset(900, 60, 3, seed=m)
    s = gsgp.Settings(pop_size=m, pool_size=r, genome_len=15, n_generations_max=stops[-1], seed=m, flags=flags,
                      mutation_step=2.0)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    X = np.concatenate([d.X_train, d.X_test])
    kept = {}
    for g in stops:
        if g > R.current_generation():
            R.generation(g - R.current_generation(), stats=False)
        st = R.stats(0, g, 1)[0]
        picks = {0, m - 1, int(st["best_index"])} | ({int(st["elite_dst"])} if st["elite_copied"] else set())
        kept[g] = [(i, R.semantics_rows(0, 0, i, 1)[0]) for i in picks]
    assert any(R.stats(0, 1, stops[-1])["elite_copied"])
    for g, rows in kept.items():
        for i, want in rows:
            got = R.reconstruct(0, g, i, X)
            if flags:
                assert np.allclose(got, want, rtol=1e-12, atol=1e-12 * np.abs(want).max()), (g, i)
            else:
                assert np.array_equal(got, want), (g, i)
            assert np.array_equal(R.reconstruct_static(0, g, i, X[:50]), got[:50]), (g, i)
    R.close()
