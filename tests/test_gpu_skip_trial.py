"""The skip pass's 16-byte trial of members: sets whose members differ from the
first string within 16 bytes, at its ends, past it, in changing shares, strings
that end inside the trial, prefixes and copies of the first string.  Exact
against the oracle, host- and device-driven."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _member(first, kind, rng):
    n = len(first)
    if kind == "near":
        k = int(rng.integers(0, min(n, 16)))
    elif kind == "edge":
        k = int(rng.integers(min(n - 1, 14), min(n, 18)))
    elif kind == "far":
        k = int(rng.integers(min(n - 1, 16), n))
    else:  # a prefix, a copy or an extension
        k = int(rng.integers(0, n + 1))
        return first[:k] if rng.random() < 0.5 else first + b"z" * int(rng.integers(0, 3))
    return first[:k] + bytes([rng.integers(1, 255)]) + bytes(rng.integers(97, 123, int(rng.integers(0, 12))).tolist())


@pytest.mark.parametrize("device_driven", [False, True])
@pytest.mark.parametrize("mix", [["near"], ["far"], ["edge"], ["prefix"], ["near", "far"], ["near", "near", "near", "far"],
                                 ["near", "edge", "far", "prefix"]])
@pytest.mark.parametrize("length", [1, 15, 16, 17, 40, 300])
def test_skip_trial(length, mix, device_driven):
    rng = np.random.default_rng(length * 7 + len(mix))
    print(f"[skip trial] length={length} mix={mix} device={device_driven}", flush=True)
    sizes = [1, 17, 64, 65, 257, 1500]
    strs = []
    for size in sizes:
        first = bytes(rng.integers(97, 123, length).tolist())
        strs += [first] + [_member(first, mix[int(rng.integers(0, len(mix)))], rng) for _ in range(size - 1)]
    s = synth.from_list(strs)
    off = np.concatenate([[0], np.cumsum(sizes)])
    g, so = s.to(DEV), torch.from_numpy(off).to(DEV)
    if device_driven:
        perm = torch.empty(s.n, dtype=torch.int32, device=DEV)
        lcp = torch.empty_like(perm)
        status = torch.full((2,), -1, dtype=torch.int32, device=DEV)
        ws = torch.empty(ss.lib().ss_sort_workspace(s.n), dtype=torch.uint8, device=DEV)
        ss.sort_batch_device(g.bytes, g.offsets, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(320))
        torch.cuda.synchronize()
        assert status.tolist() == [0, 0]
    else:
        perm, lcp = ss.sort_batch(g.bytes, g.offsets, so)
    torch.cuda.synchronize()
    p, l = perm.cpu().numpy().view(np.uint32), lcp.cpu().numpy().view(np.uint32)
    for j in range(len(sizes)):
        b, o = oracle.strings_np(synth.from_list(strs[off[j]:off[j + 1]]))
        ref = oracle.sort(b, o)
        np.testing.assert_array_equal(p[off[j]:off[j + 1]], ref, err_msg=f"set {j}")
        np.testing.assert_array_equal(l[off[j]:off[j + 1]], oracle.lcp(b, o, ref), err_msg=f"set {j}")
