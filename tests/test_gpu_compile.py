"""The genome compiler on genomes built to sit on its edges, and random ones
of every function density: semantics are the oracle's bits."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset

pytestmark = pytest.mark.gpu

L = 5


def _edge_genomes(k):
    """Rows of k genes: values left below the result at every distance from
    the end, functions before any push, skipped functions around the edges of
    64-gene chunks, single genes."""
    rows = []

    def add(genes):
        if len(genes) <= k:
            rows.append(list(genes) + [-1] * 0 + [0] * (k - len(genes)))  # trailing pushes never run
            rows.append([-2] * (k - len(genes)) + list(genes))            # functions before the first push

    add([0, 1, -1])
    add([0])
    add([0, 1])
    add([-5, -5, -4])
    for below in (1, 2, 3, 9, 61, 62, 63, 64, 65, 126, 130):
        add([i % L for i in range(below)] + [0, 1, -3])               # dead pushes below the result
        add([0, 1, -1] + [2] * below + [3, 4, -2, 1, -4])             # a dead function below it
        add([0] * below + [-1] * below)                               # everything consumed
        add([1] * below + [-1] * (below // 2) + [0, 2, -3])           # some consumed, the rest dead
        add([0, 1] + [-1] * below + [2, -3])                          # skipped functions in between
    return np.array(rows, np.int32)


@pytest.mark.parametrize("k", [1, 2, 3, 5, 63, 64, 65, 127, 128, 129, 200])
def test_edge_genomes_are_bit_exact(k):
    rng = np.random.default_rng(k)
    codes = _edge_genomes(k) if k > 1 else np.array([[0], [-1], [-5]], np.int32)
    # random genomes of several densities on top
    for p in (0.2, 0.45, 0.5, 0.55, 0.8, 0.97):
        g = rng.integers(0, L, size=(12, k)).astype(np.int32)
        g[rng.random((12, k)) < 0.3] = -5
        f = rng.random((12, k)) < p
        g[f] = rng.integers(-4, 0, size=int(f.sum()))
        codes = np.concatenate([codes, g])
    m, r = codes.shape[0], 3
    codes = np.concatenate([codes, codes[-r:]])
    consts = np.where(codes == -5, rng.uniform(-1, 1, codes.shape), 0.0)
    consts[codes == -5] = np.where(rng.random(int((codes == -5).sum())) < 0.1, 1e-7, consts[codes == -5])
    d = dataset(150, 37, L, seed=k)
    s = gsgp.Settings(pop_size=m, pool_size=r, genome_len=k, n_generations_max=1, seed=3)
    R = gsgp.Runner(s, [d])
    R.eval_population(codes, consts)
    X = np.concatenate([d.X_train, d.X_test])
    want = orc.interpret(codes[:m], consts[:m], X)
    got = R.semantics(0, 0)
    bad = np.nonzero((got != want).any(1))[0]
    assert bad.size == 0, (k, bad[:5], codes[bad[:1]])
    # the lineage evaluator reads the same compiled programs
    for i in range(0, m, 7):
        assert np.array_equal(R.reconstruct(0, 0, i, X), want[i]), i
    R.close()


def test_values_past_the_limits_take_the_checked_evaluator():
    """The threaded interpreter tests its limits once at the end of a program:
    results beyond FLT_MAX (clamped), infinite or NaN intermediates, values
    whose high word reads as an FP32 NaN or denormal, tiny and zero divisors and
    dividends, anywhere in a program and followed by harmless values, give the
    oracle's bits."""
    rng = np.random.default_rng(4)
    k, rows = 24, []
    big = [1e300, 1e307, 2e306, 1.5e308, -1e307, 3.5e38, 3.4028234663852886e38, 1e200]
    small = [1e-7, 9.99999e-7, 1e-6, -1e-6, 1.0000001e-6, 1e-300, 1e-310, 5e-324, 0.0, -0.0]

    def add(genes):
        g = np.full((2, k), 0.0)
        g[0, :] = 1  # trailing pushes never run
        for i, x in enumerate(genes):
            g[:, i] = (x, 0.0) if isinstance(x, int) else (-5, x)
        rows.append(g)

    for c in big + small + [0.5, -3.0, 1e19, 1e38]:
        for tail in ([], [1e-300, -3], [0.0, -3], [1e300, -4], [2, -4, 3, -1], [1e-20, -3, 1e-20, -3, 1e-20, -3]):
            add([0, c, -3] + tail)                      # x * c ...
            add([c, 1, -1] + tail)                      # c + x ...
            add([c, 1, -2, 0, -3] + tail)               # (c - x) * x ...
            add([0, c, -4] + tail)                      # x / c ...
            add([c, 1, -4] + tail)                      # c / x ...
            add([0, 1, -3, c, 2, -3, -4] + tail)        # x y / (c z) ...
            add([c, 0, -3, c, 1, -3, -2] + tail)        # c x - c y ...
            add([c, 0, -3, c, 0, -3, -4] + tail)        # c x / (c x) ...
    for _ in range(60):                                 # 0 / x, x / 0, and squares up to overflow
        i = int(rng.integers(L))
        add([i, i, -2, 1, -4])
        add([1, i, i, -2, -4])
        add([i, 1e100, -3] + [2, 1e100, -3, -3] * 3 + [1, -1])
    P = np.array(rows)
    codes, consts = P[:, 0].astype(np.int32), P[:, 1]
    m, r = codes.shape[0], 2
    codes, consts = np.concatenate([codes, codes[:r]]), np.concatenate([consts, consts[:r]])
    d = dataset(300, 20, L, seed=1)
    d.X_train[7, 0] = 0.0
    d.X_train[9, 1] = 1e-7
    d.X_train[11, 2] = -1e-300
    s = gsgp.Settings(pop_size=m, pool_size=r, genome_len=k, n_generations_max=1, seed=3)
    R = gsgp.Runner(s, [d])
    R.eval_population(codes, consts)
    X = np.concatenate([d.X_train, d.X_test])
    with np.errstate(all="ignore"):
        want = orc.interpret(codes[:m], consts[:m], X)
    got = R.semantics(0, 0)
    bad = np.nonzero((got != want).any(1))[0]
    assert bad.size == 0, (bad[:5], codes[bad[:1]], consts[bad[:1]])
    R.close()
