"""Prefix doubling of few strings: one launch up to 256 KB, the general rounds
above (one workgroup would hash it all alone), by the recorded kernels; results
on both sides of the line against the oracle, exactly."""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2404_16517_amd as ss
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,length,one_launch", [(2048, 128, True), (2, 131_072, True), (16, 16_384, True), (1000, 262, True),
                                                 (1000, 263, False), (2000, 500, False), (65, 5000, False), (2, 131_073, False)])
def test_line_between_one_launch_and_rounds(n, length, one_launch):
    rng = random.Random(n + length)
    head = bytes(rng.randrange(97, 123) for _ in range(length - 6))
    strs = [head[:rng.choice([length - 6, length // 2])] for _ in range(n)]
    strs = [h + bytes(rng.choice(b"ab") for _ in range(length - len(h))) if len(h) == length - 6 else h + head[len(h):] + b"tail.."
            for h in strs]
    s = synth.from_list(strs)
    assert s.N == n * length and (s.N <= 256 << 10) == one_launch
    print(f"[line] n={n} length={length}", flush=True)
    g = s.to("cuda:0")
    ss.profile_enable(True)
    try:
        d, rounds = ss.dist_prefix(g.bytes, g.offsets)
        torch.cuda.synchronize()
        names = ss.profile_report().keys()
    finally:
        ss.profile_enable(False)
    assert ("k_pd_small" in names) == one_launch, sorted(names)
    b, o = oracle.strings_np(s)
    d_ref, r_ref, _ = oracle.dist_prefix(b, o, 8, 64)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), d_ref)
    assert rounds == r_ref
