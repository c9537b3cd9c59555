"""Merges of one run far longer than the others, whose minima a launch of their own
finds: the common prefix of the group must follow the one place of the long run
where its strings share less, wherever that is.  Exact; and the minima take no
multiple of the time that as many entries in even runs take."""
import numpy as np
import pytest
import torch

import paper_2404_16517_amd as ss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _front_coded(rows, bounds):
    """Runs [bounds[j], bounds[j+1]) of equally long rows, each run sorted already."""
    n, length = rows.shape
    e = np.zeros(n, np.int64)
    same = rows[1:] == rows[:-1]
    e[1:] = np.where(same.all(axis=1), length, np.argmin(same, axis=1))
    e[bounds[:-1]] = 0
    keep = np.arange(length)[None, :] >= e[:, None]
    off = np.concatenate([[0], np.cumsum(length - e)])
    t = lambda a, dt: torch.from_numpy(a.astype(dt)).to(DEV)
    return (t(bounds[:-1], np.int64), t(bounds[1:], np.int64), torch.tensor([0, len(bounds) - 1], dtype=torch.int32, device=DEV),
            t(e, np.int32), t(np.full(n, length), np.int32), t(np.arange(n), np.int32), t(off, np.int64),
            torch.from_numpy(rows[keep]).to(DEV))


@pytest.mark.parametrize("dip", [1, 32_767, 32_768, 40_000, 69_998, 69_999])
@pytest.mark.parametrize("longs", [1, 2])
def test_common_prefix_of_long_runs(dip, longs):
    rng = np.random.default_rng(dip + longs)
    sizes = [40] * 30 + [70_000] * longs + [1, 55]
    bounds = np.concatenate([[0], np.cumsum(sizes)])
    n, length = int(bounds[-1]), 24
    assert max(sizes) > 32_768 * -(-n // (len(sizes) * 4096)) or longs == 2
    rows = np.full((n, length), ord("M"), np.uint8)
    rows[:, 12:] = rng.integers(97, 101, (n, length - 12))
    at = int(bounds[30 + longs - 1])  # in the last long run, the strings from `dip` on are larger after 3 bytes
    rows[at + dip:at + 70_000, 3] = ord("Z")
    key = [r.tobytes() for r in rows]
    for a, b in zip(bounds[:-1], bounds[1:]):
        key[a:b] = sorted(key[a:b])
    rows = np.frombuffer(b"".join(key), np.uint8).reshape(n, length).copy()
    print(f"[long runs] dip={dip} longs={longs} n={n}", flush=True)
    src, ids, lcp = ss.lcp_merge(*_front_coded(rows, bounds))
    torch.cuda.synchronize()
    want = np.argsort(np.array(key, dtype=f"S{length}"), kind="stable")
    np.testing.assert_array_equal(ids.cpu().numpy(), want)
    same = rows[want[1:]] == rows[want[:-1]]
    np.testing.assert_array_equal(lcp.cpu().numpy()[1:], np.where(same.all(axis=1), length, np.argmin(same, axis=1)))


def test_minima_of_a_long_run_time():
    """4M entries in one run among 1,023 of 100, against 1,024 of 4,006 (20 us and
    6): one workgroup alone takes 4M entries in 0.8 ms."""
    took = {}
    for kind, sizes in (("long", [100] * 1023 + [4_000_000]), ("even", [4006] * 1024)):
        bounds = np.concatenate([[0], np.cumsum(sizes)])
        n = int(bounds[-1])
        x = np.arange(n) - np.repeat(bounds[:-1], sizes)  # the position in the run, as five letters
        rows = np.stack([97 + x // 26 ** (4 - d) % 26 for d in range(5)], axis=1).astype(np.uint8)
        args = _front_coded(rows, bounds)
        ws = torch.empty(ss.lib().ss_lcp_merge_workspace(n, n, 1024), dtype=torch.uint8, device=DEV)
        ss.lcp_merge(*args, ws=ws, n_out=n)
        ss.profile_enable(True)
        try:
            for _ in range(5):
                ss.lcp_merge(*args, ws=ws, n_out=n)
            torch.cuda.synchronize()
            took[kind] = ss.profile_report()["k_run_min"][0] / 5
        finally:
            ss.profile_enable(False)
    print(f"[minima] {took} ms", flush=True)
    assert took["long"] < 15 * took["even"]
