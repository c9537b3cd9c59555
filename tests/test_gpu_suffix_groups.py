"""Suffix sorting by groups at the edges of its paths: texts around the sizes
where the first step's one group changes its sort (128, 512, 2048), groups
around eight members (sorted at once) and sixty-four (one tile), and long
repeats.  Order and LCPs against the oracle, exactly; the number of steps
against its closed form, the first t with 6 * 2^(t-1) > max LCP."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss

pytestmark = pytest.mark.gpu


def _text(kind, n, rng):
    if kind == "bytes":
        return rng.integers(0, 256, n)
    if kind == "binary":
        return rng.integers(97, 99, n)
    if kind == "unary":
        return np.full(n, 97)
    # a passage repeated k times among random letters: groups of k suffixes
    k = int(kind[6:])
    body = rng.integers(97, 123, 40)
    parts = []
    for _ in range(k):
        parts += [body, rng.integers(65, 91, max(1, n // k - 40))]
    return np.concatenate(parts)[:max(n, 40 * k)]


CASES = [(k, n) for k in ("bytes", "binary", "unary")
         for n in (1, 2, 3, 6, 7, 8, 9, 13, 127, 128, 129, 511, 513, 2047, 2049, 30_011)]
CASES += [(f"repeat{k}", n) for k in (2, 8, 9, 64, 65, 130, 700) for n in (2047, 2049, 30_011)]


@pytest.mark.parametrize("kind,n", CASES)
def test_suffix_groups(kind, n):
    rng = np.random.default_rng(n)
    text = _text(kind, n, rng).astype(np.uint8)
    print(f"[suffix groups] {kind} N={len(text)}", flush=True)
    sa, lcp, steps = ss.suffix_sort(torch.from_numpy(text).to("cuda:0"))
    torch.cuda.synchronize()
    esa, elcp = oracle.suffix_sort(text)
    np.testing.assert_array_equal(sa.cpu().numpy().view(np.uint32), esa)
    np.testing.assert_array_equal(lcp.cpu().numpy().view(np.uint32), elcp)
    t = 1
    while 6 * 2 ** (t - 1) <= int(elcp.max()):
        t += 1
    assert steps == t
