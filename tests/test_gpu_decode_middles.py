"""Decoded bytes that lie between a string's head's literal and its own: around the
32 bytes up to which a string's own thread fetches them, chains of many pieces,
pieces and strings across chunks.  Byte for byte against the oracle; and long
strings made of such bytes take no multiple of the time of the same bytes from
one literal."""
import statistics
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _runs(kind, n, rng):
    i = np.arange(n)
    if kind == "near":  # head, an entry that keeps F bytes, one that keeps F + 30..35
        f = rng.integers(9, 40, n)
        d = np.full(n, 120)
        e = np.where(i % 3 == 0, rng.integers(0, 9, n), np.where(i % 3 == 1, f, np.roll(f, 1) + rng.integers(30, 36, n)))
    elif kind == "stairs":  # every string keeps some more of the one before
        d = rng.integers(280, 300, n)
        e = (i % 40) * 7
    elif kind == "long stairs":
        d = np.full(n, 30_000)
        e = (i % 50) * 600 - i % 7
    else:  # many thin pieces: long and short LCPs in turn
        d = np.full(n, 5000)
        e = np.where(i % 2 == 0, 4990, (i % 100) * 50)
    e = np.minimum(np.maximum(e, 0), np.minimum(d, np.concatenate([[0], d[:-1]])))
    suf_off = np.concatenate([[0], np.cumsum(d - e)]).astype(np.uint64)
    return np.array([0, n], np.uint64), e.astype(np.uint32), d.astype(np.uint32), suf_off, \
        rng.integers(0, 256, int(suf_off[-1])).astype(np.uint8)


def _device(run_off, e, d, suf_off, suf):
    T = lambda a, dt: torch.from_numpy(a.view(dt).copy()).to(DEV)
    return T(run_off, np.int64), T(e, np.int32), T(d, np.int32), T(suf_off, np.int64), torch.from_numpy(suf).to(DEV)


@pytest.mark.parametrize("kind,n", [("near", 3), ("near", 20_000), ("stairs", 5000), ("long stairs", 120), ("thin", 400)])
def test_decode_middles(kind, n):
    runs = _runs(kind, n, np.random.default_rng(n))
    print(f"[decode middles] {kind} n={n}", flush=True)
    rb, roff = oracle.fc_decode(*runs)
    args = _device(*runs)
    for shift in (0, 3):
        buf = torch.full((rb.size + 32,), 0xA5, dtype=torch.uint8, device=DEV)
        oo = torch.empty(n + 1, dtype=torch.int64, device=DEV)
        st = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        ss.fc_decode_noalloc(*args, oo, buf[shift:shift + rb.size], st)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        np.testing.assert_array_equal(oo.cpu().numpy().view(np.uint64), roff)
        got = buf.cpu().numpy()
        np.testing.assert_array_equal(got[shift:shift + rb.size], np.frombuffer(bytes(rb), np.uint8))
        assert (got[:shift] == 0xA5).all() and (got[shift + rb.size:] == 0xA5).all()


def test_decode_long_strings_time():
    """20,000 strings of 5,000 bytes: LCPs uniform (chains of some ten pieces)
    against 4,995 each (one literal).  One thread fetching a string's middle took
    7.7 times as long; dealt out they take 1.3 times."""
    n, length = 20_000, 5000
    rng = np.random.default_rng(1)
    took = {}
    for kind in ("uniform", "one"):
        e = rng.integers(0, length + 1, n) if kind == "uniform" else np.full(n, length - 5)
        e[0] = 0
        suf_off = np.concatenate([[0], np.cumsum(length - e)]).astype(np.uint64)
        args = _device(np.array([0, n], np.uint64), e.astype(np.uint32), np.full(n, length, np.uint32), suf_off,
                       np.full(int(suf_off[-1]), 97, np.uint8))
        ts = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ss.fc_decode(*args)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        took[kind] = statistics.median(ts[2:])
    print(f"[decode time] {took}", flush=True)
    assert took["uniform"] < 3 * took["one"]
