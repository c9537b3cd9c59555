"""The one-launch sort of few strings at its edges: counts around the wavefronts'
shares, strings equal over the 512 bytes that are compared at once and beyond,
zero bytes beside string ends, empty strings, copies.  Exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["zeros", "deep", "exact512", "short", "mixed"])
@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 63, 64, 65, 68, 129, 255, 256, 257])
def test_rank_sort(n, kind):
    rng = np.random.default_rng(n)
    print(f"[rank sort] n={n} {kind}", flush=True)
    def one():
        if kind == "zeros":      # ends and zero bytes read alike
            return b"ab" + bytes(int(rng.integers(0, 14))) + (b"" if rng.random() < 0.7 else b"\x01")
        if kind == "deep":       # equal far past the first 512 bytes
            return b"x" * int(rng.integers(500, 1600)) + bytes(rng.integers(0, 3, int(rng.integers(0, 4))).tolist())
        if kind == "exact512":
            return b"y" * int(rng.integers(510, 515)) + (b"" if rng.random() < 0.5 else b"z")
        if kind == "short":
            return bytes(rng.integers(97, 99, int(rng.integers(0, 5))).tolist())
        return bytes(rng.integers(0, 256, int(rng.integers(0, 700))).tolist())
    strs = [one() for _ in range(n)]
    s = synth.from_list(strs)
    g = s.to("cuda:0")
    perm, lcp = ss.sort(g.bytes, g.offsets)
    torch.cuda.synchronize()
    b, o = oracle.strings_np(s)
    ref = oracle.sort(b, o)
    np.testing.assert_array_equal(perm.cpu().numpy().view(np.uint32), ref)
    np.testing.assert_array_equal(lcp.cpu().numpy().view(np.uint32), oracle.lcp(b, o, ref))
