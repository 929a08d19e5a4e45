"""Lineage reconstruction over every route of the walk (on the host; on the
device from 64 individuals on, unless its nodes or maps do not fit) and of the
replay: 4, 2 and 1 cases per block with two generations of rows in LDS, and a
launch per generation beyond that.  On the training and test cases an
individual's reconstruction repeats the FP64 operations that formed its stored
semantics, in their order, so the values are equal."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,r,gens,flags", [
    (5, 3, 1, 0),              # one step
    (40, 300, 60, 0),          # the pool in LDS beside the rows
    (700, 3000, 25, 0),        # the pool too large for LDS
    (3000, 50, 16, 0),         # 4 or 2 cases a block
    (5000, 50, 16, 0),         # 2
    (12000, 50, 18, 0),        # 1
    (30000, 50, 18, 0),        # beyond LDS: a launch per generation
    (64, 64, 30, gsgp.FLAG_LOCAL_SEARCH),
    (256, 31, 40, gsgp.FLAG_LOCAL_SEARCH),
    (63, 300, 70, 0),          # the largest walked on the host
    (64, 65, 131, 0),          # the smallest on the device; more generations than a wave holds starts of
    (256, 300, 150, 0),        # the nodes of 150 generations exceed the buffer the device walk uses
    (1025, 1000, 13, 0),       # two individuals a thread
    (2300, 2400, 9, 0),        # four
    (8192, 8200, 9, 0),        # the largest walked on the device: eight
    (8193, 8200, 9, 0),        # just beyond them
])
def test_reconstruction_repeats_the_stored_semantics(m, r, gens, flags):
    d = dataset(21, 6, 3, seed=m)
    s = gsgp.Settings(pop_size=m, pool_size=r, genome_len=15, n_generations_max=gens, seed=m + gens, flags=flags)
    R = gsgp.Runner(s, [d])
    R.eval_population()
    stats = R.generation(gens)
    X = np.concatenate([d.X_train, d.X_test])
    for i in (int(stats[0, -1]["best_index"]), int(stats[0, -1]["elite_dst"]), m - 1):
        if i < 0:
            continue
        want = R.semantics_rows(0, 0, i, 1)[0]
        got = R.reconstruct(0, gens, i, X)
        if flags:  # the device fits its scaling from chunk sums, both sides apply the stored one
            assert np.allclose(got, want, rtol=1e-12, atol=1e-12 * np.abs(want).max())
        else:
            assert np.array_equal(got, want), (m, i)
        assert np.array_equal(R.reconstruct_static(0, gens, i, X), got)
        # any number of cases, each the same
        for n in (1, 7, 9):
            assert np.array_equal(R.reconstruct(0, gens, i, X[:n]), got[:n])
        # beyond 512 cases: up to 4 a block, the last one short
        assert np.array_equal(R.reconstruct(0, gens, i, np.tile(X, (21, 1))[:565]), np.tile(got, 21)[:565])
    # an earlier generation, and generation 0
    mid = R.reconstruct(0, gens // 2, 0, X)
    assert mid.shape == (27,) and np.isfinite(mid).all()
    R.close()
