"""The merge by key at its edges, against the oracle, exactly: numbers of runs
around the sampling steps' limits (16, 64, 512) and above the most a tile takes,
run sizes around one tile, groups of different kinds in one call, runs placed in
memory in another order than their numbers, keys with more copies than a tile
holds, ties of 2 to some hundred members."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth
from tests.test_gpu_parity import _runs_from_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def T(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a).view(dt).copy()).to(DEV)


def _strings(kind, n, rng):
    if kind == "digits":      # distinct keys mostly
        return [b"%08d" % x for x in rng.integers(0, 10 ** 8, n)]
    if kind == "copies":      # three strings, thousands of copies each, and some others
        base = [b"SAMESAME-one", b"SAMESAME-two-longer", b"SAMESAM"]
        return [base[x] if x < 3 else b"%04d" % x for x in rng.integers(0, 5, n)]
    if kind == "shared":      # one long prefix, ties past the key of every size
        return [b"Q" * 40 + bytes(rng.integers(97, 99, int(rng.integers(0, 12))).tolist()) for _ in range(n)]
    return synth.text_strings(n, seed=int(rng.integers(1 << 20)), median=12).as_list()


def _merge(runs, order, groups):
    """The library's merge of runs built by the oracle (run_off, ...), the runs
    placed in memory in the given order."""
    ro, lc, ln, idv, so, suf = runs
    k = len(ro) - 1
    begin, end = np.zeros(k, np.int64), np.zeros(k, np.int64)
    at, pos, sufp = 0, [], [0]
    parts = []
    for j in order:
        a, b = int(ro[j]), int(ro[j + 1])
        begin[j], end[j] = at, at + b - a
        at += b - a
        pos += range(a, b)
        for i in range(a, b):
            parts.append(suf[int(so[i]):int(so[i + 1])])
            sufp.append(sufp[-1] + int(so[i + 1] - so[i]))
    pos = np.array(pos, np.int64)
    sufm = np.concatenate(parts) if parts else np.zeros(0, np.uint8)
    go = np.array(groups, np.int32)
    out = ss.lcp_merge(torch.from_numpy(begin).to(DEV), torch.from_numpy(end).to(DEV), torch.from_numpy(go).to(DEV),
                       T(lc[pos], np.int32), T(ln[pos], np.int32), T(idv[pos], np.int32),
                       torch.tensor(sufp, dtype=torch.int64, device=DEV), torch.from_numpy(sufm.copy()).to(DEV),
                       with_len=True)
    torch.cuda.synchronize()
    return [x.cpu().numpy().view(np.uint64 if x.dtype == torch.int64 else np.uint32) for x in out]


def _expect(runs, groups):
    ro, lc, ln, idv, so, suf = runs
    src, ids, lcp = [], [], []
    for a, b in zip(groups[:-1], groups[1:]):
        p, q = int(ro[a]), int(ro[b])
        s, i, l = oracle.merge(ro[a:b + 1] - ro[a], lc[p:q], ln[p:q], idv[p:q], so[p:q + 1], suf)
        src.append(s + (np.uint64(a) << np.uint64(32)))
        ids.append(i)
        lcp.append(l)
    return np.concatenate(src), np.concatenate(ids), np.concatenate(lcp)


@pytest.mark.parametrize("kind", ["digits", "copies", "shared", "text"])
@pytest.mark.parametrize("k,n", [(1, 5000), (2, 2304), (2, 2305), (3, 7000), (16, 9000), (17, 9000), (64, 12_000),
                                 (65, 12_000), (512, 20_000), (513, 20_000), (700, 6000), (2048, 9000), (2048, 30_000), (2049, 9000)])
def test_merge_one_group(kind, k, n):
    rng = np.random.default_rng(k * 7 + n)
    print(f"[merge tiles] {kind} k={k} n={n}", flush=True)
    s = synth.from_list(_strings(kind, n, rng))
    runs = _runs_from_oracle(s, k, seed=k)
    src, ids, lcp, ln = _merge(runs, rng.permutation(k), [0, k])
    e_src, e_ids, e_lcp = _expect(runs, [0, k])
    np.testing.assert_array_equal(ids, e_ids)
    np.testing.assert_array_equal(src, e_src)
    np.testing.assert_array_equal(lcp, e_lcp)
    by_id = np.empty(s.n, np.uint32)
    by_id[runs[3]] = runs[2]
    np.testing.assert_array_equal(ln, by_id[ids])


@pytest.mark.parametrize("kind", ["digits", "copies", "shared", "text"])
def test_merge_groups_of_every_kind(kind):
    """Groups of no, one, few and many runs, small and large, in one call."""
    rng = np.random.default_rng(5)
    k = 600
    sizes = np.ones(k, int)
    sizes[:3] = (3000, 0, 2500)
    sizes[3] = 0
    sizes[20:60] = 150
    assign = np.repeat(np.arange(k), sizes)
    rng.shuffle(assign)
    s = synth.from_list(_strings(kind, len(assign), rng))
    runs = _runs_from_oracle(s, k, 0, assign=assign)
    groups = [0, 3, 4, 4, 5, 20, 60, 600]
    src, ids, lcp, _ = _merge(runs, rng.permutation(k), groups)
    e_src, e_ids, e_lcp = _expect(runs, groups)
    np.testing.assert_array_equal(ids, e_ids)
    np.testing.assert_array_equal(src, e_src)
    np.testing.assert_array_equal(lcp, e_lcp)


@pytest.mark.parametrize("k,n", [(2, 50), (5, 6000), (40, 9000)])
def test_unsorted_runs_lose_nothing(k, n):
    """Runs that break the sortedness precondition: the order is not specified,
    but every element comes out once."""
    rng = np.random.default_rng(n)
    strs = _strings("text", n, rng)
    ro = np.linspace(0, n, k + 1).astype(np.uint64)
    e = np.zeros(n, np.uint32)
    starts = set(int(x) for x in ro)
    for i in range(1, n):
        if i not in starts:
            a, b = strs[i - 1], strs[i]
            m = 0
            while m < min(len(a), len(b)) and a[m] == b[m]:
                m += 1
            e[i] = m
    d = np.array([len(x) for x in strs], np.uint32)
    suf = np.frombuffer(b"".join(x[int(m):] for x, m in zip(strs, e)), np.uint8)
    so = np.concatenate([[0], np.cumsum(d.astype(np.int64) - e)]).astype(np.uint64)
    _, ids, _, _ = _merge((ro, e, d, np.arange(n, dtype=np.uint32), so, suf), np.arange(k), [0, k])
    np.testing.assert_array_equal(np.sort(ids), np.arange(n))
