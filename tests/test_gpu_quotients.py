"""Quotients between 2^127 and FLT_MAX, in every form of the division and in
both evaluators: the short division's bits are the full one's (the oracle's)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2106_04034_amd import gsgp, synth

pytestmark = pytest.mark.gpu


def test_quotients_up_to_flt_max_are_bit_exact():
    rng = np.random.default_rng(8)
    n, k, top = 300, 20, 3.4028234663852886e38
    X = rng.uniform(1.0, 1.9, (n, 3))  # every case's quotient lies in the range
    rows = []

    def add(genes):
        """The genes alone, and after a zero dividend (0 / x + ...), which the
        threaded evaluator leaves to the checked one."""
        for g in (genes, [0, 0, -2, 1, -4] + genes + [-1]):
            c = np.zeros((2, k))
            c[0, :] = 1  # trailing pushes never run
            for i, x in enumerate(g):
                c[:, i] = (x, 0.0) if isinstance(x, int) else (-5, x)
            rows.append(c)

    for _ in range(40):
        a = rng.uniform(0.97, 1.0) * top * rng.choice([-1, 1])
        add([a, 0, -4])                            # constant / feature
        add([0, a / 2, -3, 2, -4])                 # (x a) / feature
        add([0, 1e30, -3, 1.9e30 / top, -4])       # (x c) / constant
        add([a, 0, -4, 1.0, -3, 0, -3, 0, -4])     # a product near FLT_MAX, divided
        add([0, a / 1.9, -3, 1, 1.0, -3, -4])      # / a value of the stack
        add([0, 1e-5, -3, 1e-5 / top, -4])         # a divisor below 1e-6: 1
    P = np.array(rows)
    codes, consts = P[:, 0].astype(np.int32), P[:, 1]
    m = codes.shape[0]
    codes, consts = np.concatenate([codes, codes[:2]]), np.concatenate([consts, consts[:2]])
    d = synth.Dataset(X[:200].copy(), X[:200, 0].copy(), X[200:].copy(), X[200:, 0].copy())
    R = gsgp.Runner(gsgp.Settings(pop_size=m, pool_size=2, genome_len=k, n_generations_max=1, seed=3), [d])
    R.eval_population(codes, consts)
    want = orc.interpret(codes[:m], consts[:m], X)
    assert ((np.abs(want) > 2.0**127) & (np.abs(want) < top)).all(1).sum() > 100
    assert np.array_equal(R.semantics(0, 0), want)
    R.close()
