"""Merges of a few runs of which the last are shorter than the place of their first
sample (they have none, and nothing at that place may be read: it can lie behind the
last key), against the oracle, exactly."""
import numpy as np
import pytest

import synth
from tests.test_gpu_merge_tiles import _expect, _merge, _strings
from tests.test_gpu_parity import _runs_from_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[2400, 1], [2400, 48], [2400, 49], [3000, 40, 1], [1300] * 3 + [1, 50, 2, 1],
                                   [700] * 8 + [1] * 8, [200] * 15 + [62], [200] * 15 + [63]], ids=str)
def test_last_runs_short(sizes):
    k = len(sizes)
    rng = np.random.default_rng(k)
    strs = _strings("digits", sum(sizes), rng)
    print(f"[short runs] {sizes}", flush=True)
    runs = _runs_from_oracle(synth.from_list(strs), k, seed=k, assign=rng.permutation(np.repeat(np.arange(k), sizes)))
    src, ids, lcp, _ = _merge(runs, range(k), [0, k])
    e_src, e_ids, e_lcp = _expect(runs, [0, k])
    np.testing.assert_array_equal(ids, e_ids)
    np.testing.assert_array_equal(src, e_src)
    np.testing.assert_array_equal(lcp, e_lcp)
