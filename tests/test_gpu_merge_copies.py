"""Merges of few distinct strings: tiles of one key, larger than a tile holds, whose
strings end in the key, are equal past it, or differ past it, beside tiles that
are sorted.  Exact against the oracle; and a merge of copies takes no multiple of
the time of a merge of distinct strings."""
import statistics
import time

import numpy as np
import pytest
import torch

import paper_2404_16517_amd as ss
import synth
from tests.test_gpu_merge_tiles import _expect, _merge
from tests.test_gpu_parity import _runs_from_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _strings(kind, n, rng):
    if kind == "empty":
        return [b""] * n
    if kind == "ends":      # one short string, among its extensions and others
        return [b"ab" if x < 8 else b"ab" + b"c" * x if x < 9 else b"%03d" % rng.integers(1000) for x in rng.integers(0, 10, n)]
    if kind == "equal":     # one long string
        return [b"the same string, sixty bytes of it, in every run, every time"] * n
    if kind == "differ":    # one key, then everything differs; the first byte keeps the common prefix at 0
        return [b"SHAREDKEY-and-more-" + b"%05d" % x if x % 9 else b"%d" % (x % 10) for x in rng.integers(0, 99_999, n)]
    return [(b"SHAREDKEY" + b"x" * int(x)) if x < 3 else b"A" * int(x) for x in rng.integers(0, 6, n)]  # "mixed"


@pytest.mark.parametrize("kind", ["empty", "ends", "equal", "differ", "mixed"])
@pytest.mark.parametrize("k,n", [(1, 6000), (2, 2305), (8, 30_000), (300, 20_000), (600, 20_000)])
def test_merge_copies(kind, k, n):
    rng = np.random.default_rng(k + n)
    print(f"[merge copies] {kind} k={k} n={n}", flush=True)
    s = synth.from_list(_strings(kind, n, rng))
    runs = _runs_from_oracle(s, k, seed=k)
    for groups in ([0, k], [0, k // 2, k]) if k > 1 else ([0, k],):
        src, ids, lcp, ln = _merge(runs, rng.permutation(k), groups)
        e_src, e_ids, e_lcp = _expect(runs, groups)
        np.testing.assert_array_equal(ids, e_ids)
        np.testing.assert_array_equal(src, e_src)
        np.testing.assert_array_equal(lcp, e_lcp)
        by_id = np.empty(s.n, np.uint32)
        by_id[runs[3]] = runs[2]
        np.testing.assert_array_equal(ln, by_id[ids])


def test_merge_copies_time():
    """1M strings of 12 bytes in 8 runs: copies of one against distinct ones.  One
    workgroup moving the whole tile, and one update of one word per 16 strings,
    made the copies take 10 times as long."""
    n, k = 1_000_000, 8
    took = {}
    for kind in ("copies", "distinct"):
        g = torch.Generator(device=DEV).manual_seed(3)
        b = torch.randint(97, 123, (n, 12), dtype=torch.uint8, generator=g, device=DEV)
        if kind == "copies":
            b[:] = b[0].clone()
        so = torch.arange(k + 1, dtype=torch.int64, device=DEV) * (n // k)
        bytes_, off = b.view(-1), torch.arange(n + 1, dtype=torch.int64, device=DEV) * 12
        perm, lcp = ss.sort_batch(bytes_, off, so, global_ids=True)
        fc = ss.partition_encode_batch(bytes_, off, so, perm, lcp, None, torch.empty(0, dtype=torch.uint8, device=DEV),
                                       torch.zeros(1, dtype=torch.int64, device=DEV))
        go = torch.tensor([0, k], dtype=torch.int32, device=DEV)
        ws = torch.empty(ss.lib().ss_lcp_merge_workspace(n, n, k), dtype=torch.uint8, device=DEV)
        ts = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ss.lcp_merge(so[:-1], so[1:], go, fc["lcp"], fc["len"], fc["id"], fc["suf_off"], fc["suf"], ws=ws, n_out=n)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        took[kind] = statistics.median(ts[2:])
    print(f"[merge time] {took}", flush=True)
    assert took["copies"] < 3.5 * took["distinct"]
