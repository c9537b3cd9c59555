"""Sorts whose lists are longer than one workgroup scans (4096 segments) or whose
histograms are longer than one range per workgroup (4M entries), and small sorts
with smaller radix tiles: 8-byte keys, exact against a stable sort of the keys."""
import numpy as np
import pytest
import torch

import paper_2404_16517_amd as ss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("sets,per,small_max,tile,device_driven", [
    (1, 1_400_000, 128, 1024, False), (1, 1_400_000, 128, 1024, True),      # many radix segments on later levels
    (5000, 300, 128, 4096, False), (5000, 300, 128, 4096, True),            # ... and on the first
    (4096, 300, 128, 4096, False), (4097, 300, 128, 4096, True),
    (1, 17_000_000, 1024, 1024, False),                                    # 4.2M histogram entries
    (100, 25_000, 1024, 4096, False), (800, 3000, 128, 4096, False), (40, 60_000, 128, 1024, False),  # narrow digits
    (1, 2049, 1024, 4096, False), (3, 30_000, 1024, 4096, False), (3, 30_000, 1024, 8192, True),  # small tiles
])
def test_long_lists(sets, per, small_max, tile, device_driven):
    n = sets * per
    print(f"[long lists] sets={sets} per={per} small_max={small_max} tile={tile} device={device_driven}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    b = torch.randint(0, 5 if per > 10_000_000 else 256, (n, 8), generator=g, device=DEV, dtype=torch.int64)
    key = torch.zeros(n, dtype=torch.int64, device=DEV)
    for j in range(8):
        key = (key << 8) | b[:, j]
    bytes_ = b.to(torch.uint8).reshape(-1).contiguous()
    off = torch.arange(n + 1, dtype=torch.int64, device=DEV) * 8
    so = torch.arange(sets + 1, dtype=torch.int64, device=DEV) * per
    old = ss.set_tuning(ss.SS_TUNE_SMALL_MAX, small_max), ss.set_tuning(ss.SS_TUNE_TILE, tile)
    try:
        if device_driven:
            perm = torch.empty(n, dtype=torch.int32, device=DEV)
            lcp = torch.empty_like(perm)
            status = torch.full((2,), -1, dtype=torch.int32, device=DEV)
            ws = torch.empty(ss.lib().ss_sort_workspace(n), dtype=torch.uint8, device=DEV)
            ss.sort_batch_device(bytes_, off, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(8))
            torch.cuda.synchronize()
            assert status.tolist() == [0, 0]
        else:
            perm, lcp = ss.sort_batch(bytes_, off, so)
        torch.cuda.synchronize()
    finally:
        ss.set_tuning(ss.SS_TUNE_SMALL_MAX, old[0])
        ss.set_tuning(ss.SS_TUNE_TILE, old[1])
    order = torch.sort((key ^ (-1 << 63)).reshape(sets, per), dim=1, stable=True).indices
    assert torch.equal(perm.reshape(sets, per).to(torch.int64), order)
    k = key.reshape(sets, per).gather(1, order)
    x = k[:, 1:] ^ k[:, :-1]
    want = torch.zeros(sets, per, dtype=torch.int32, device=DEV)
    for j in range(1, 9):  # shares j bytes: the top 8 j bits agree
        want[:, 1:] += (((x >> (64 - 8 * j)) if j < 8 else x) == 0).to(torch.int32)
    assert torch.equal(lcp.reshape(sets, per), want)
