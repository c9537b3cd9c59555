"""Device-driven sorts whose radix segments go to one workgroup each: sets below,
at and above the size that goes there at once, totals on both sides of the
lines between none, one and two levels over the whole device, segments that need
several levels (a short cutover, few letters, shared letters), one key for a
whole segment.  Exact against the oracle; the captured graph repeats it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("small_max", [128, 1024])
@pytest.mark.parametrize("kind", ["random", "few", "skewed", "copies"])
@pytest.mark.parametrize("sizes", [[32_768], [32_769], [20_000, 12_000, 700], [33_000, 3, 32_768, 2049], [2048, 2049, 2050, 257],
                                   [560_000, 40_000, 100], [200_000] + [4000] * 120])
def test_radix_by_workgroup(sizes, kind, small_max):
    if sum(sizes) // (2 * small_max) > 4096:
        small_max = 512
    rng = np.random.default_rng(sum(sizes) + small_max)
    print(f"[radix by workgroup] {sizes[:4]} of {len(sizes)} {kind} small_max={small_max}", flush=True)
    n = sum(sizes)
    if kind == "random":
        b = rng.integers(0, 256, (n, 9))
    elif kind == "few":
        b = rng.integers(97, 100, (n, 9))
    elif kind == "skewed":
        b = 97 + (26 * rng.random((n, 9)) ** 4).astype(np.int64)
    else:
        b = np.where(rng.random((n, 1)) < 0.9, 120, rng.integers(97, 123, (n, 9)))
    lens = np.where(rng.random(n) < 0.8, 9, rng.integers(0, 10, n))
    b = b.astype(np.uint8)
    strs = [b[i, :lens[i]].tobytes() for i in range(n)]
    s = synth.from_list(strs)
    off = np.concatenate([[0], np.cumsum(sizes)])
    g, so = s.to(DEV), torch.from_numpy(off).to(DEV)
    perm = torch.empty(n, dtype=torch.int32, device=DEV)
    lcp = torch.empty_like(perm)
    status = torch.full((2,), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ss.lib().ss_sort_workspace(n), dtype=torch.uint8, device=DEV)
    old = ss.set_tuning(ss.SS_TUNE_SMALL_MAX, small_max)
    try:
        def run():
            ss.sort_batch_device(g.bytes, g.offsets, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(9))
        run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run()
    finally:
        ss.set_tuning(ss.SS_TUNE_SMALL_MAX, old)
    first = perm.clone(), lcp.clone()
    for _ in range(3):
        perm.fill_(-1)
        lcp.fill_(-1)
        ws.random_(0, 255)  # nothing of a call may be left to the next
        graph.replay()
        torch.cuda.synchronize()
        assert status.tolist() == [0, 0]
        assert torch.equal(perm, first[0]) and torch.equal(lcp, first[1])
    p, l = perm.cpu().numpy().view(np.uint32), lcp.cpu().numpy().view(np.uint32)
    for j in range(len(sizes)):
        bb, o = oracle.strings_np(synth.from_list(strs[off[j]:off[j + 1]]))
        ref = oracle.sort(bb, o)
        np.testing.assert_array_equal(p[off[j]:off[j + 1]], ref, err_msg=f"set {j}")
        np.testing.assert_array_equal(l[off[j]:off[j + 1]], oracle.lcp(bb, o, ref), err_msg=f"set {j}")


@pytest.mark.parametrize("shares", [[0.5], [0.95], [0.3, 0.3, 0.3], [0.2, 0.14, 0.13, 0.1]])
@pytest.mark.parametrize("n", [9000, 40_000, 200_000])
def test_shared_keys(n, shares):
    """Large shares of a set's strings with one key each (strings that go on after
    it, equal strings, strings that end inside it), among random ones."""
    rng = np.random.default_rng(n + len(shares))
    print(f"[shared keys] n={n} {shares}", flush=True)
    heads = [b"http://", b"ftp", b"mailto:someone", b"\x00\xff\x00"][:len(shares)]
    pick = rng.choice(len(shares) + 1, n, p=shares + [1 - sum(shares)])
    tail = rng.integers(97, 123, (n, 6)).astype(np.uint8)
    strs = [(heads[k] + (tail[i].tobytes() if k % 2 == 0 else b"")) if k < len(shares) else tail[i].tobytes()
            for i, k in enumerate(pick)]
    s = synth.from_list(strs + [b"small set", b"a"])
    g = s.to(DEV)
    so = torch.tensor([0, n, n + 2], dtype=torch.int64, device=DEV)
    perm = torch.empty(n + 2, dtype=torch.int32, device=DEV)
    lcp = torch.empty_like(perm)
    status = torch.full((2,), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ss.lib().ss_sort_workspace(n + 2), dtype=torch.uint8, device=DEV)
    ss.sort_batch_device(g.bytes, g.offsets, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(20))
    torch.cuda.synchronize()
    assert status.tolist() == [0, 0]
    b, o = oracle.strings_np(synth.from_list(strs))
    ref = oracle.sort(b, o)
    np.testing.assert_array_equal(perm[:n].cpu().numpy().view(np.uint32), ref)
    np.testing.assert_array_equal(lcp[:n].cpu().numpy().view(np.uint32), oracle.lcp(b, o, ref))
    assert perm[n:].tolist() == [1, 0]
