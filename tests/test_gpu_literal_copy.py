"""The literal copy by output words at its edges: literals of no, one and a few
bytes between long ones (a word that several literals share), all shorter or
all longer than a word, counts around one workgroup's 256 strings, output that
starts at every alignment.  Exact against the plain definition."""
import numpy as np
import pytest
import torch

import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("base", [0, 1, 7, 8, 15])
@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
@pytest.mark.parametrize("kind", ["mixed", "words", "long", "one"])
def test_literal_copy(kind, n, base):
    rng = np.random.default_rng(n + base)
    if kind == "mixed":    # many nearly empty literals beside one of thousands of bytes
        lens = np.where(rng.random(n) < 0.05, rng.integers(500, 6000, n), rng.integers(0, 4, n))
        lens[0] = 9000
    elif kind == "words":
        lens = rng.choice([15, 16, 17, 31, 32, 33, 47, 48, 49], n)
    elif kind == "long":
        lens = rng.integers(200, 400, n)
    else:                  # one literal holds everything
        lens = np.zeros(n, np.int64)
        lens[n // 2] = 70_001
    print(f"[literal copy] {kind} n={n} base={base}", flush=True)
    # the strings in any order with LCP 0 declared throughout: every literal is its string
    strs = [rng.integers(0, 256, int(x), dtype=np.uint8).tobytes() for x in lens]
    s = synth.from_list(strs)
    g = s.to(DEV)
    perm = rng.permutation(n).astype(np.int32)
    lcp = np.zeros(n, np.int32)
    total = int(lens.sum())
    out = dict(run_off=torch.empty(2, dtype=torch.int64, device=DEV), suf_off=torch.empty(n + 1, dtype=torch.int64, device=DEV),
               suf=torch.full((base + total + 3,), 0xEE, dtype=torch.uint8, device=DEV),
               **{k: torch.empty(n, dtype=torch.int32, device=DEV) for k in ("lcp", "len", "id")})
    fc = ss.partition_encode(g.bytes, g.offsets, torch.from_numpy(perm).to(DEV), torch.from_numpy(lcp).to(DEV), None,
                             torch.empty(0, dtype=torch.uint8, device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV),
                             out=out, suf_base=base)
    torch.cuda.synchronize()
    assert fc["total"] == total
    want = b"\xee" * base + b"".join(strs[p] for p in perm) + b"\xee" * 3
    assert out["suf"].cpu().numpy().tobytes() == want
