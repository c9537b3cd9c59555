"""Tied segments of a merge: copies inside and across runs, prefixes, members that
leave the first one at the same or at different places and sides, segments around
8 members (ordered at once), 16 and 256, copies with one deviating member.  Exact
against the oracle; and what long or many equal neighbours of one run cost."""
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
PAIRS = ("every pair of a tied segment is compared: the kernels that left most comparisons out are taken back, after a "
         "GPU fault in a run that held them, whose cause was not found")
TAILS = [b"", b"a", b"ab", b"abc", b"abd", b"b", b"ba", b"bab", b"c", b"\x00", b"m" * 30, b"m" * 30 + b"a", b"m" * 29 + b"z"]


def _clusters(kind, rng):
    out = []
    for q in range(700 if kind == "mixed" else 60):
        head = b"%04d" % q + b"-the shared part"  # (the common prefix of all is empty: keys are its first 7 bytes)
        if kind == "mixed":       # 2 to 12 members of any sort
            out += [head + TAILS[t] for t in rng.integers(0, len(TAILS), int(rng.integers(2, 13)))]
        elif kind == "few tails":  # many equal ones among them
            out += [head + TAILS[t] for t in rng.choice(rng.integers(0, len(TAILS), 2), int(rng.integers(2, 10)))]
        else:                     # copies around the limits, one deviating in some clusters
            n = int(rng.choice([7, 8, 9, 10, 16, 17, 63, 64, 65, 255, 256, 257, 300]))
            members = [head + b"x" * 20] * n
            if q % 3:
                members[int(rng.integers(0, n))] = head + [b"x" * 19, b"x" * 21, b"x" * 19 + b"y", b"x" * 19 + b"a"][q % 4]
            out += members
    return out


@pytest.mark.parametrize("kind", ["mixed", "few tails", "copies"])
@pytest.mark.parametrize("k", [1, 2, 3, 8, 30])
def test_tied_members(kind, k):
    rng = np.random.default_rng(k)
    strs = _clusters(kind, rng)
    s = synth.from_list([strs[i] for i in rng.permutation(len(strs))])
    print(f"[tied members] {kind} k={k} n={s.n}", flush=True)
    runs = _runs_from_oracle(s, k, seed=k)
    for groups in ([0, k], [0, 1, k]) if k > 1 else ([0, k],):
        src, ids, lcp, ln = _merge(runs, rng.permutation(k), groups)
        e_src, e_ids, e_lcp = _expect(runs, groups)
        np.testing.assert_array_equal(ids, e_ids)
        np.testing.assert_array_equal(src, e_src)
        np.testing.assert_array_equal(lcp, e_lcp)
        by_id = np.empty(s.n, np.uint32)
        by_id[runs[3]] = runs[2]
        np.testing.assert_array_equal(ln, by_id[ids])


@pytest.mark.skip(reason=PAIRS)
def test_long_equal_neighbours_time():
    """Three strings of 5 MB, all but equal, in one of two runs whose other strings
    tie with them: the runs' LCPs order them.  Comparing the first with the third took
    30 ms."""
    g = torch.Generator(device=DEV).manual_seed(1)
    took = {}
    for size in (5_000_000, 30):
        lens = torch.tensor([size] * 3 + [30] * 3000, dtype=torch.int64, device=DEV)
        off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(lens, 0, out=off[1:])
        b = torch.randint(97, 99, (int(off[-1]),), dtype=torch.uint8, generator=g, device=DEV)
        b[size:2 * size] = b[:size]
        b[2 * size:3 * size] = b[:size]
        b[3 * size - 1] = 120
        n = lens.numel()
        so = torch.tensor([0, n // 2, n], dtype=torch.int64, device=DEV)
        perm, lcp = ss.sort_batch(b, off, so, global_ids=True)
        fc = ss.partition_encode_batch(b, off, so, perm, lcp, None, torch.empty(0, dtype=torch.uint8, device=DEV),
                                       torch.zeros(1, dtype=torch.int64, device=DEV))
        go = torch.tensor([0, 2], dtype=torch.int32, device=DEV)
        ts = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ss.lcp_merge(so[:-1], so[1:], go, fc["lcp"], fc["len"], fc["id"], fc["suf_off"], fc["suf"], n_out=n)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        took[size] = statistics.median(ts[2:])
    print(f"[long neighbours] {took}", flush=True)
    assert took[5_000_000] < 10 * took[30]


@pytest.mark.skip(reason=PAIRS)
def test_copies_time():
    """2M strings in two runs, each ten times, against 2M distinct ones: 4.5 times as
    long where all pairs are compared and larger segments sorted, 2.2 times where few are."""
    n = 2_000_000
    took = {}
    for copies in (10, 1):
        g = torch.Generator(device=DEV).manual_seed(2)
        b = torch.randint(97, 123, (n // copies, 40), dtype=torch.uint8, generator=g, device=DEV)
        if copies > 1:
            b = b[torch.randint(0, n // copies, (n,), generator=g, device=DEV)]
        bytes_, off = b.reshape(-1).contiguous(), torch.arange(n + 1, dtype=torch.int64, device=DEV) * 40
        so = torch.tensor([0, n // 2, n], dtype=torch.int64, device=DEV)
        perm, lcp = ss.sort_batch(bytes_, off, so, global_ids=True)
        fc = ss.partition_encode_batch(bytes_, off, so, perm, lcp, None, torch.empty(0, dtype=torch.uint8, device=DEV),
                                       torch.zeros(1, dtype=torch.int64, device=DEV))
        go = torch.tensor([0, 2], dtype=torch.int32, device=DEV)
        ws = torch.empty(ss.lib().ss_lcp_merge_workspace(n, n, 2), dtype=torch.uint8, device=DEV)
        ts = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ss.lcp_merge(so[:-1], so[1:], go, fc["lcp"], fc["len"], fc["id"], fc["suf_off"], fc["suf"], ws=ws, n_out=n)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        took[copies] = statistics.median(ts[2:])
    print(f"[copies time] {took}", flush=True)
    assert took[10] < 3.3 * took[1]
