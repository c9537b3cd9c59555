"""Radix digits made of the varying key bits, and the scatter through LDS: alphabets
whose varying bits lie together, apart, at the top or at the bottom of a byte,
strings that end inside the key, many duplicates, one string only; tiles and
chunks with remainders.  Exact against the oracle, host- and device-driven."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ALPHABETS = {
    "letters": b"abcdefghijklmnopqrstuvwxyz", "digits": b"0123456789", "acgt": b"ACGT", "bit0": b"@A", "bit7": b"\x00\x80",
    "alternate": bytes([0x00, 0x55, 0x11, 0x44, 0x41, 0x14]), "ends": bytes([0x01, 0x80, 0x81]), "all": bytes(range(256)),
    "one": b"x",
}


@pytest.mark.parametrize("device_driven", [False, True])
@pytest.mark.parametrize("bits,small_max,tile", [(8, 128, 1024), (8, 1024, 4096), (11, 512, 4096)])
@pytest.mark.parametrize("name", ALPHABETS)
def test_digits(name, bits, small_max, tile, device_driven):
    rng = np.random.default_rng(len(name) * 31 + bits)
    print(f"[digits] {name} bits={bits} small_max={small_max} tile={tile} device={device_driven}", flush=True)
    al = np.frombuffer(ALPHABETS[name], np.uint8)
    sizes = [20_011, 2049, 9000]
    strs = []
    for j, size in enumerate(sizes):
        pre = [b"", b"common prefix of a set ", b"\xff" * 9][j]
        lens = rng.integers([0, 5, 0][j], [10, 8, 20][j], size)
        strs += [pre + al[rng.integers(0, len(al), n)].tobytes() for n in lens]
    s = synth.from_list(strs)
    off = np.concatenate([[0], np.cumsum(sizes)])
    g, so = s.to(DEV), torch.from_numpy(off).to(DEV)
    tune = {ss.SS_TUNE_DIGIT_BITS: bits, ss.SS_TUNE_SMALL_MAX: small_max, ss.SS_TUNE_TILE: tile}
    old = {k: ss.set_tuning(k, v) for k, v in tune.items()}
    try:
        if device_driven:
            perm = torch.empty(s.n, dtype=torch.int32, device=DEV)
            lcp = torch.empty_like(perm)
            status = torch.full((2,), -1, dtype=torch.int32, device=DEV)
            ws = torch.empty(ss.lib().ss_sort_workspace(s.n), dtype=torch.uint8, device=DEV)
            ss.sort_batch_device(g.bytes, g.offsets, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(33))
            torch.cuda.synchronize()
            assert status.tolist() == [0, 0]
        else:
            perm, lcp = ss.sort_batch(g.bytes, g.offsets, so)
        torch.cuda.synchronize()
    finally:
        for k, v in old.items():
            ss.set_tuning(k, v)
    p, l = perm.cpu().numpy().view(np.uint32), lcp.cpu().numpy().view(np.uint32)
    for j in range(len(sizes)):
        b, o = oracle.strings_np(synth.from_list(strs[off[j]:off[j + 1]]))
        ref = oracle.sort(b, o)
        np.testing.assert_array_equal(p[off[j]:off[j + 1]], ref, err_msg=f"set {j}")
        np.testing.assert_array_equal(l[off[j]:off[j + 1]], oracle.lcp(b, o, ref), err_msg=f"set {j}")
