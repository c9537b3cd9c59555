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


@pytest.mark.parametrize("base", [0, 9])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 256, 1000])
@pytest.mark.parametrize("mean", [511, 512, 3000])
def test_long_literals(mean, n, base):
    """Around the mean length from which a workgroup takes 16 literals: empty and
    tiny ones among them, one that is much longer, every count around 16."""
    rng = np.random.default_rng(n + base + mean)
    lens = np.where(rng.random(n) < 0.2, rng.integers(0, 20, n), rng.integers(1, 2 * mean, n))
    lens[-1] = max(0, mean * n - int(lens[:-1].sum()))
    if lens.sum() > mean * n:
        lens = np.full(n, mean)
    assert int(lens.sum()) == mean * n
    print(f"[long literals] mean={mean} n={n} base={base}", flush=True)
    s = synth.from_list([rng.integers(0, 256, int(x), dtype=np.uint8).tobytes() for x in lens])
    g = s.to(DEV)
    perm = rng.permutation(n).astype(np.int32)
    out = dict(run_off=torch.empty(2, dtype=torch.int64, device=DEV), suf_off=torch.empty(n + 1, dtype=torch.int64, device=DEV),
               suf=torch.full((base + mean * n + 3,), 0xEE, dtype=torch.uint8, device=DEV),
               **{k: torch.empty(n, dtype=torch.int32, device=DEV) for k in ("lcp", "len", "id")})
    ss.partition_encode(g.bytes, g.offsets, torch.from_numpy(perm).to(DEV), torch.zeros(n, dtype=torch.int32, device=DEV), None,
                        torch.empty(0, dtype=torch.uint8, device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV),
                        out=out, suf_base=base)
    torch.cuda.synchronize()
    strs = s.as_list()
    assert out["suf"].cpu().numpy().tobytes() == b"\xee" * base + b"".join(strs[p] for p in perm) + b"\xee" * 3


def test_long_literals_time():
    """200 MB in 2,000 literals against a plain copy of as much (0.44 ms and 0.08): 256 literals
    a workgroup took 8 ms."""
    n, length = 2000, 100_000
    b = torch.randint(0, 256, (n * length,), dtype=torch.uint8, device=DEV)
    off = torch.arange(n + 1, dtype=torch.int64, device=DEV) * length
    perm = torch.randperm(n, device=DEV).to(torch.int32)
    lcp = torch.zeros(n, dtype=torch.int32, device=DEV)
    to = torch.empty_like(b)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for _ in range(3):
        ev[0].record()
        to.copy_(b)
        ev[1].record()
    torch.cuda.synchronize()
    plain = ev[0].elapsed_time(ev[1])
    def encode():
        ss.partition_encode(b, off, perm, lcp, None, torch.empty(0, dtype=torch.uint8, device=DEV),
                            torch.zeros(1, dtype=torch.int64, device=DEV))
    encode()
    ss.profile_enable(True)
    try:
        for _ in range(5):
            encode()
        torch.cuda.synchronize()
        took = ss.profile_report()["k_fc_copy"][0] / 5
    finally:
        ss.profile_enable(False)
    print(f"[long literals] copy {plain} ms, literals {took} ms", flush=True)
    assert took < 20 * plain
