"""The merge sort of segments in LDS at its edges: segment sizes around one
thread's 8 elements, the wavefront form's 512 and the workgroup form's 2048,
under every cutover, with keys that tie (duplicates, shared prefixes, strings
ending inside the key) and small sorts' smaller element tiles.  Exact against
the oracle, host- and device-driven."""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu
SIZES = [129, 136, 137, 255, 256, 257, 511, 512, 513, 1023, 1025, 2047, 2048, 2049]


def _strings(seed):
    """Sets of the sizes above: random letters, few letters (deep ties, exact
    duplicates, prefixes) and presorted or reversed numbers."""
    rng = random.Random(seed)
    sets = []
    for size in SIZES:
        kind = rng.randrange(3)
        if kind == 0:
            st = [bytes(rng.choice(b"ABCDEFGH") for _ in range(rng.randint(0, 14))) for _ in range(size)]
        elif kind == 1:
            st = [bytes(rng.choice(b"AB") for _ in range(rng.randint(0, 16))) for _ in range(size)]
        else:
            st = [b"%06d" % (i if rng.random() < 0.9 else rng.randrange(size)) for i in range(size)]
            if rng.random() < 0.5:
                st.reverse()
        sets.append(st)
    return sets


@pytest.mark.parametrize("device_driven", [False, True])
@pytest.mark.parametrize("small_max", [128, 256, 512, 1024])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_block_sort_sizes(seed, small_max, device_driven):
    sets = _strings(seed)
    s = synth.from_list([x for st in sets for x in st])
    off = np.concatenate([[0], np.cumsum([len(st) for st in sets])])
    print(f"[block sort] seed={seed} small_max={small_max} device={device_driven}", flush=True)
    g = s.to("cuda:0")
    so = torch.from_numpy(off).to("cuda:0")
    old = ss.set_tuning(ss.SS_TUNE_SMALL_MAX, small_max)
    try:
        if device_driven:
            perm = torch.empty(s.n, dtype=torch.int32, device="cuda:0")
            lcp = torch.empty_like(perm)
            status = torch.full((2,), -1, dtype=torch.int32, device="cuda:0")
            ws = torch.empty(ss.lib().ss_sort_workspace(s.n), dtype=torch.uint8, device="cuda:0")
            ss.sort_batch_device(g.bytes, g.offsets, so, perm, lcp, status, ws, ss.sort_batch_device_rounds(16))
            torch.cuda.synchronize()
            assert status.tolist() == [0, 0]
        else:
            perm, lcp = ss.sort_batch(g.bytes, g.offsets, so)
        torch.cuda.synchronize()
    finally:
        ss.set_tuning(ss.SS_TUNE_SMALL_MAX, old)
    p, l = perm.cpu().numpy().view(np.uint32), lcp.cpu().numpy().view(np.uint32)
    for j, st in enumerate(sets):
        b, o = oracle.strings_np(synth.from_list(st))
        ref = oracle.sort(b, o)
        np.testing.assert_array_equal(p[off[j]:off[j + 1]], ref, err_msg=f"set {j} of {len(st)}")
        np.testing.assert_array_equal(l[off[j]:off[j + 1]], oracle.lcp(b, o, ref), err_msg=f"set {j}")
