"""Runs of tied strings compared directly, at the limits of that path: 2 to 17
members (16 is the most it takes), ties of 0 to 1100 bytes past the keys (1024
is the most it compares), equal strings, prefixes and one deviating member.
Order and LCPs against the oracle, exactly."""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu


def _set(members, tie, seed):
    rng = random.Random(seed)
    out = []
    for q in range(40):
        base = b"%04d" % q + bytes(rng.choice(b"abc") for _ in range(28 + tie))
        kind = q % 4
        for m in range(members):
            if kind == 0:                               # all equal
                out.append(base)
            elif kind == 1:                             # one deviates at its last byte
                out.append(base[:-1] + b"z" if m == members // 2 else base)
            elif kind == 2:                             # one ends early
                out.append(base[:-1] if m == members - 1 else base)
            else:                                       # all end differently
                out.append(base + bytes([97 + (m * 7) % 23]))
    out += [b"%05d" % rng.randint(0, 99999) for _ in range(300)]
    rng.shuffle(out)
    return out


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("members", [2, 3, 8, 9, 16, 17])
@pytest.mark.parametrize("tie", [0, 1, 63, 64, 65, 1023, 1024, 1100])
def test_tied_runs(members, tie, batch):
    strs = _set(members, tie, seed=members * 2000 + tie)
    print(f"[tied runs] members={members} tie={tie} batch={batch}", flush=True)
    s = synth.from_list(strs)
    g = s.to("cuda:0")
    if batch:
        so = torch.tensor([0, s.n], dtype=torch.int64, device="cuda:0")
        perm, lcp = ss.sort_batch(g.bytes, g.offsets, so)
    else:
        perm, lcp = ss.sort(g.bytes, g.offsets)
    torch.cuda.synchronize()
    b, o = oracle.strings_np(s)
    ref = oracle.sort(b, o)
    np.testing.assert_array_equal(perm.cpu().numpy().view(np.uint32), ref)
    np.testing.assert_array_equal(lcp.cpu().numpy().view(np.uint32), oracle.lcp(b, o, ref))


def test_many_surviving_runs():
    """More runs that go on than 8 x 32 per workgroup of the largest grid (2048):
    what a workgroup collects is published in the middle of its runs and again at
    the end.  Triples that share 45 bytes and then differ, every 50th run of 17
    strings (passed on uncompared), in random input order."""
    groups, filler = 600_000, 40
    size = np.where(np.arange(groups) % 50 == 49, 17, 3)
    assert groups > 8 * 32 * 2048 and size.sum() < 2**31
    grp = np.repeat(np.arange(groups), size)
    last = np.arange(grp.size) - np.repeat(np.cumsum(size) - size, size)
    rank = np.random.default_rng(3).permutation(grp.size)  # input index i holds sorted string rank[i]
    digits = np.stack([grp // 26 ** (4 - d) % 26 for d in range(5)], axis=1)
    rows = np.full((grp.size, 6 + filler), 65, dtype=np.uint8)
    rows[:, :5] += digits.astype(np.uint8)
    rows[:, -1] += last.astype(np.uint8)
    want = np.empty(grp.size, dtype=np.int64)
    want[rank] = np.arange(grp.size)
    lcp_want = np.where(grp[1:] == grp[:-1], 5 + filler, np.argmax(digits[1:] != digits[:-1], axis=1))
    print(f"[surviving runs] groups={groups} n={grp.size}", flush=True)
    b = torch.from_numpy(rows[rank].reshape(-1)).to("cuda:0")
    o = torch.arange(grp.size + 1, dtype=torch.int64, device="cuda:0") * (6 + filler)
    perm, lcp = ss.sort(b, o)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(perm.cpu().numpy(), want)
    np.testing.assert_array_equal(lcp.cpu().numpy()[1:], lcp_want)
    assert lcp[0].item() == 0
