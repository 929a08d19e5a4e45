"""Workspace guards around the calls that read a run: getters and the lineage
walk launch kernels that use the workspace too."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2106_04034_amd import gsgp

from .gpu_helpers import dataset

pytestmark = pytest.mark.gpu

CALLS = {
    "fitness": lambda R, d: R.fitness(0),
    "semantics": lambda R, d: R.semantics(0, 0),
    "one row": lambda R, d: R.semantics_rows(0, 1, 3, 1),
    "summaries": lambda R, d: R.stats(0, 0, 4),
    "reconstruct": lambda R, d: R.reconstruct(0, 5, 7, d.X_train[:9]),
    "reconstruct_static": lambda R, d: R.reconstruct_static(0, 5, 7, d.X_train[:9]),
}


@pytest.mark.parametrize("name", CALLS)
def test_reading_calls_check_the_guards(name):
    d = dataset(700, 60, 3, seed=4)
    R = gsgp.Runner(gsgp.Settings(pop_size=80, pool_size=50, genome_len=31, n_generations_max=5, seed=6,
                                  flags=gsgp.FLAG_GUARDS), [d])
    plain = gsgp.Runner(gsgp.Settings(pop_size=80, pool_size=50, genome_len=31, n_generations_max=5, seed=6), [d])
    for r in (R, plain):
        r.eval_population()
        r.generation(5)
    # every call leaves every guard as it is, and returns what it returns without guards
    for call in CALLS.values():
        for a, b in zip(call(R, d), call(plain, d)):
            assert np.array_equal(a, b)
    at = int(R._ws_ptr - R._ws.data_ptr() + R.guard_offsets()[4 + 3])  # after S[1]
    R._ws[at:at + 4] = 0
    R.torch.cuda.synchronize()
    with pytest.raises(gsgp.GSGPError) as e:
        CALLS[name](R, d)
    assert e.value.status == -2 and "S[1] of run 0" in str(e.value)
    R.close()
    plain.close()
