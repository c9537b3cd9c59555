"""The one-launch prefix doubling and the sort's short path for few strings, at
their limits (256 / 512 / 2048 strings) and one past them, against the oracle,
exactly."""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu


def _strings(kind, n, seed):
    rng = random.Random(seed)
    if kind == "short":      # empty strings, prefixes, duplicates, every byte value
        return [bytes(rng.choice((0, 65, 255)) for _ in range(rng.randint(0, 9))) for _ in range(n)]
    if kind == "deep":       # one long common prefix, then a few letters
        return [b"P" * 300 + bytes(rng.choice(b"ab") for _ in range(rng.randint(0, 14))) for _ in range(n)]
    if kind == "long":       # duplicates of long strings (thousands of limbs a round)
        base = [bytes(rng.randrange(256) for _ in range(rng.choice([63, 64, 65, 255, 1023, 5001]))) for _ in range(7)]
        return [rng.choice(base) + bytes([rng.randrange(3)] * rng.randint(0, 1)) for _ in range(n)]
    return [bytes(rng.randrange(32, 128) for _ in range(rng.randint(1, 80))) for _ in range(n)]


@pytest.mark.parametrize("kind", ["short", "deep", "long", "random"])
@pytest.mark.parametrize("n", [1, 2, 65, 257, 2047, 2048, 2049])
def test_few_strings_sort_and_doubling(kind, n):
    s = synth.from_list(_strings(kind, n, seed=n))
    print(f"[few strings] {kind} n={n} N={s.N}", flush=True)
    g = s.to("cuda:0")
    b, o = oracle.strings_np(s)
    ref = oracle.sort(b, o)
    for with_lcp in (True, False):
        perm, lcp = ss.sort(g.bytes, g.offsets, with_lcp=with_lcp)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(perm.cpu().numpy().view(np.uint32), ref)
        if with_lcp:
            np.testing.assert_array_equal(lcp.cpu().numpy().view(np.uint32), oracle.lcp(b, o, ref))
    for init_len, bits in ((8, 64), (4, 64), (12, 20), (256, 64), (8, 8)):
        d, rounds = ss.dist_prefix(g.bytes, g.offsets, init_len, bits)
        torch.cuda.synchronize()
        d_ref, r_ref, _ = oracle.dist_prefix(b, o, init_len, bits)
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), d_ref, err_msg=f"{init_len} {bits}")
        assert rounds == r_ref
