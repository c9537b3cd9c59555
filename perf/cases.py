"""The workloads this library is measured on: what they are, how their inputs
are made and how a program calls them.

Each case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (device inputs drawn from a seed, workspaces it keeps, for the
captured sort its graph), ``run`` is one pass through the package's entry
points, ``work`` the bytes that pass cannot do without.  Every output is a
whole number or a byte, so two correct implementations agree exactly and no
reference in wider arithmetic is needed.

Three kinds of strings, the ones the benchmark and the tests use:
  dn       fixed length over 'A'..'Z': a common run of 'A', the base-26 code of
           a random permutation, random letters (a chosen D/N ratio)
  text     log-normal lengths (median 40), Zipf(1.1) bytes over 96 printable
           codes, 20 % exact copies of other strings
  letters  uniform lengths in [8, 256], uniform letters (sets of them)
"""
from __future__ import annotations

import math
import random

import torch

import paper_2404_16517_amd as ss

DEV = "cuda:0"


# ------------------------------------------------------------------- cases

def listed() -> list[dict]:
    return [
        # the sample sort inside every splitter selection: 16 processing
        # elements with three samples each (latency of one small call)
        {"name": "sort_samples", "op": "sort", "kind": "dn", "n": 48, "length": 500, "ratio": 0.5},
        # the smallest served request: sort + LCP, exact and approximate
        # distinguishing prefixes of a thousand text strings
        {"name": "job_text_1k", "op": "job", "kind": "text", "n": 1000},
        # one processing element's array at the small configuration
        {"name": "sort_dn_100k", "op": "sort", "kind": "dn", "n": 100_000, "length": 100, "ratio": 0.5},
        # a large served request of text, its size odd
        {"name": "job_text_4m", "op": "job", "kind": "text", "n": 4_000_003},
        # many independent sets of 10^3..10^5 strings in one call
        {"name": "sort_sets_512", "op": "sets", "sets": 512, "lo": 1000, "hi": 100_000},
        # the same through a captured graph, small sets (nothing read back)
        {"name": "graph_sets_64", "op": "graph", "sets": 64, "lo": 100, "hi": 10_000},
        # one sorted array of full text strings into 16 front-coded buckets
        {"name": "encode_text_4m", "op": "encode", "kind": "text", "n": 4_000_003, "p": 16},
        # 256 sorted front-coded runs of 64-byte strings into one sequence
        {"name": "merge_dn_256runs", "op": "merge", "kind": "dn", "n": 8_000_000, "length": 64, "ratio": 0.3,
         "p": 256, "buckets": 1},
        # every bucket's runs from 16 processing elements, text
        {"name": "merge_text_16x16", "op": "merge", "kind": "text", "n": 4_000_000, "p": 16, "buckets": 16},
        # front-coded runs back to strings
        {"name": "decode_text_2m", "op": "decode", "kind": "text", "n": 2_000_003, "p": 16},
        # suffix array and LCPs of one text
        {"name": "suffix_text_8mb", "op": "suffix", "kind": "text", "n": 8_000_001},
        # the whole single-level prefix-doubling merge sort of 8 GB of strings
        {"name": "pdms_dn_16m", "op": "pdms", "kind": "dn", "n": 16_000_000, "length": 500, "ratio": 0.5, "p": 16},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_strings(rng: random.Random, n: int) -> dict:
    if rng.random() < 0.5:
        return {"kind": "text", "n": n}
    return {"kind": "dn", "n": n, "length": rng.choice([64, 100, 100, 250, 333, 500]),
            "ratio": rng.choice([0.3, 0.5, 0.7, 0.9])}


def draw(rng: random.Random) -> dict:
    op = rng.choice(["sort", "sort", "job", "sets", "graph", "encode", "merge", "decode", "suffix", "pdms"])
    if op == "sort":
        return {"op": op, **_draw_strings(rng, _log_int(rng, 24, 4_000_000))}
    if op == "job":
        return {"op": op, **_draw_strings(rng, _log_int(rng, 1000, 4_000_000))}
    if op == "sets":
        return {"op": op, "sets": _log_int(rng, 16, 512), "lo": 1000, "hi": 100_000}
    if op == "graph":
        return {"op": op, "sets": _log_int(rng, 16, 512), "lo": 100, "hi": 10_000}
    if op == "suffix":
        return {"op": op, "kind": "text", "n": _log_int(rng, 10_000, 8_000_000)}
    if op == "merge":
        if rng.random() < 0.4:
            p, buckets = rng.choice([2, 5, 16, 64, 100, 256]), 1
        else:
            p = buckets = rng.choice([4, 7, 16, 24])
        return {"op": op, **_draw_strings(rng, _log_int(rng, 200_000, 4_000_000)), "p": p, "buckets": buckets}
    if op == "pdms":
        return {"op": op, **_draw_strings(rng, _log_int(rng, 100_000, 6_000_000)), "p": rng.choice([4, 8, 16])}
    return {"op": op, **_draw_strings(rng, _log_int(rng, 100_000, 3_000_000)), "p": rng.choice([1, 4, 16])}


# ------------------------------------------------------------------ inputs

# Contents follow the seed; lengths, set sizes and which strings are copies
# follow the case, so that every seed gives outputs of the same shapes.

def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


def _offsets(lens: torch.Tensor) -> torch.Tensor:
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=off[1:])
    return off


def _digits(n: int) -> int:
    k = 1
    while 26 ** k < n:
        k += 1
    return k


def _filler(c: dict) -> int:
    return max(0, int(math.floor(c["ratio"] * c["length"] + 0.5)) - _digits(c["n"]))


def _dn(c: dict, g: torch.Generator):
    n, length, k, fill = c["n"], c["length"], _digits(c["n"]), _filler(c)
    pi = torch.randperm(n, generator=g, device=DEV)
    out = torch.empty((n, length), dtype=torch.uint8, device=DEV)
    out[:, :fill] = 65
    for d in range(k):
        out[:, fill + d] = (65 + (pi // 26 ** (k - 1 - d)) % 26).to(torch.uint8)
    for a in range(0, n, 1 << 20):
        b = min(n, a + (1 << 20))
        out[a:b, fill + k:] = torch.randint(65, 91, (b - a, length - fill - k), dtype=torch.uint8, generator=g,
                                            device=DEV)
    return out.view(-1), torch.arange(n + 1, dtype=torch.int64, device=DEV) * length


def _zipf_bytes(count: int, g: torch.Generator) -> torch.Tensor:
    w = 1.0 / torch.arange(1, 97, dtype=torch.float64) ** 1.1
    top = (torch.cumsum(w, 0) / w.sum() * 65536).round().long()
    table = (32 + torch.searchsorted(top, torch.arange(65536), right=True).clamp_(max=95)).to(torch.uint8).to(DEV)
    out = torch.empty(count, dtype=torch.uint8, device=DEV)
    for a in range(0, count, 1 << 27):
        b = min(count, a + (1 << 27))
        out[a:b] = table[torch.randint(0, 65536, (b - a,), dtype=torch.int32, generator=g, device=DEV)]
    return out


def _text(n: int, g: torch.Generator):
    f = _gen(n)
    lens = torch.randn(n, generator=f, device=DEV).add_(math.log(40.0)).exp_().round_().clamp_(1, 4096).long()
    idx = torch.arange(n, device=DEV)
    copy = torch.rand(n, generator=f, device=DEV) < 0.2
    copy[0] = False
    src = (torch.rand(n, generator=f, device=DEV, dtype=torch.float64) * idx).long()  # an earlier string
    copy &= ~copy[src]  # ... that is no copy itself
    dst = idx[copy]
    src = src[copy]
    lens[dst] = lens[src]
    off = _offsets(lens)
    data = _zipf_bytes(int(off[-1]), g)
    if dst.numel():
        cl = lens[dst]
        at = torch.arange(int(cl.sum()), device=DEV) - torch.repeat_interleave(torch.cumsum(cl, 0) - cl, cl)
        data[torch.repeat_interleave(off[dst], cl) + at] = data[torch.repeat_interleave(off[src], cl) + at]
    return data, off


def _strings(c: dict, g: torch.Generator):
    return _dn(c, g) if c["kind"] == "dn" else _text(c["n"], g)


def _sets(c: dict, g: torch.Generator):
    r = random.Random(c["sets"])
    sizes = [_log_int(r, c["lo"], c["hi"]) for _ in range(c["sets"])]
    so = torch.tensor([0] + sizes, dtype=torch.int64, device=DEV).cumsum(0)
    off = _offsets(torch.randint(8, 257, (sum(sizes),), generator=_gen(c["sets"]), device=DEV))
    data = torch.randint(65, 91, (int(off[-1]),), dtype=torch.uint8, generator=g, device=DEV)
    return data, off, so


def _ws(nbytes: int) -> torch.Tensor:
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV)


def _bounds(n: int, p: int) -> torch.Tensor:
    return torch.tensor([n * i // p for i in range(p + 1)], dtype=torch.int64, device=DEV)


def _splitters(b, o, perm, so, r: int, max_len: int):
    """r - 1 splitters from three samples per sorted array (more of a single one)."""
    samp = ss.select_splitters_batch(perm, so, 4 if so.numel() > 2 else 4 * r, check=False)
    sb, sof = ss.gather_strings(b, o, samp, cap_hint=samp.numel() * max_len, sync=False)
    sperm, _ = ss.sort(sb, sof, with_lcp=False)
    ids = ss.select_splitters(sperm, r)
    return ss.gather_strings(sb, sof, ids, cap_hint=max(ids.numel(), 1) * max_len, sync=False)


def _encode_all(s):
    return ss.partition_encode_batch(s["b"], s["o"], s["so"], s["perm"], s["lcp"], s["dist"], s["fb"], s["fo"],
                                     ws=s["ws"])


def prepare(c: dict, seed: int) -> dict:
    g = _gen(seed)
    L = ss.lib()
    op = c["op"]
    s = {"op": op, "c": c}
    if op == "suffix":
        s["text"] = _zipf_bytes(c["n"], g)
        q = c["n"] // 16  # a repeated passage, as real texts have
        s["text"][3 * q:3 * q + 2000] = s["text"][q:q + 2000].clone()
        s["ws"] = _ws(L.ss_suffix_sort_workspace(c["n"]))
        return s
    if op in ("sets", "graph"):
        s["b"], s["o"], s["so"] = _sets(c, g)
        n = s["o"].numel() - 1
        s["ws"] = _ws(L.ss_sort_workspace(n))
        if op == "graph":
            s["perm"] = torch.zeros(n, dtype=torch.int32, device=DEV)
            s["lcp"] = torch.zeros(n, dtype=torch.int32, device=DEV)
            s["status"] = torch.zeros(2, dtype=torch.int32, device=DEV)
            torch.cuda.synchronize()
            s["graph"] = ss.Graph.capture(
                lambda: ss.sort_batch_device(s["b"], s["o"], s["so"], s["perm"], s["lcp"], s["status"], s["ws"], 3),
                torch.cuda.Stream())
        return s
    b, o = _strings(c, g)
    s["b"], s["o"] = b, o
    n = o.numel() - 1
    if op == "sort":
        s["ws"] = _ws(L.ss_sort_workspace(n))
        return s
    if op == "job":
        s["ws"] = _ws(max(L.ss_sort_workspace(n), L.ss_dist_prefix_workspace(n)))
        return s
    p = c["p"]
    s["so"] = _bounds(n, p)
    s["max_len"] = int((o[1:] - o[:-1]).max())
    if op == "pdms":
        s["ws_sort"] = _ws(L.ss_sort_workspace(n))
        s["ws_pd"] = _ws(L.ss_dist_prefix_workspace(n))
        s["ws_pe"] = _ws(L.ss_partition_encode_workspace(n))
        s["ws_merge"] = _ws(L.ss_lcp_merge_workspace(n, n, p * p))
        s["seed"] = _ws(L.ss_sort_seed_bytes(n))
        s["group_off"] = torch.arange(0, p * p + 1, p, dtype=torch.int32, device=DEV)
        return s
    # encode: one sorted array and its splitters.  merge, decode: every
    # processing element's array sorted, split and front-coded.  dn strings send
    # their distinguishing prefixes, text strings travel whole (encode, decode)
    # or by distinguishing prefix (merge)
    if op == "encode":
        s["so"] = _bounds(n, 1)
    s["perm"], s["lcp"] = ss.sort_batch(b, o, s["so"], global_ids=True)
    short = c["kind"] == "dn" or op == "merge"
    s["dist"] = ss.dist_prefix(b, o)[0] if short else None
    r = c.get("buckets", p)
    s["fb"], s["fo"] = _splitters(b, o, s["perm"], s["so"], r, s["max_len"])
    if op == "encode":  # the buffers a program encodes into
        u32 = [torch.empty(n, dtype=torch.int32, device=DEV) for _ in range(3)]
        s["out"] = {"run_off": torch.empty(r + 1, dtype=torch.int64, device=DEV), "lcp": u32[0], "len": u32[1],
                    "id": u32[2], "suf_off": torch.empty(n + 1, dtype=torch.int64, device=DEV),
                    "suf": torch.zeros(b.numel(), dtype=torch.uint8, device=DEV)}
        return s
    s["ws"] = _ws(L.ss_partition_encode_workspace(n))
    s["fc"] = _encode_all(s)
    ro = s["fc"]["run_off"].view(p, r + 1)
    if op == "decode":
        s["run_off"] = torch.cat([ro[:, :-1].reshape(-1), ro[-1:, -1]])
        return s
    s["rb"], s["re"] = ro[:, :-1].t().contiguous().view(-1), ro[:, 1:].t().contiguous().view(-1)
    s["go"] = torch.arange(0, p * r + 1, p, dtype=torch.int32, device=DEV)
    s["ws"] = _ws(L.ss_lcp_merge_workspace(n, n, p * r))
    for k in ("b", "o", "perm", "lcp", "dist"):
        s.pop(k)
    return s


# --------------------------------------------------------------- one pass

def run(s: dict):
    op = s["op"]
    if op == "sort":
        return ss.sort(s["b"], s["o"], ws=s["ws"])
    if op == "sets":
        return ss.sort_batch(s["b"], s["o"], s["so"], ws=s["ws"])
    if op == "graph":
        s["graph"].launch()
        return s["perm"], s["lcp"], s["status"]
    if op == "job":
        perm, lcp = ss.sort(s["b"], s["o"], ws=s["ws"])
        dist = ss.dist_exact(s["o"], perm, lcp)
        dpx, rounds = ss.dist_prefix(s["b"], s["o"], 8, 64, ws=s["ws"])
        return perm, lcp, dist, dpx, rounds
    if op == "encode":
        fc = ss.partition_encode(s["b"], s["o"], s["perm"], s["lcp"], s["dist"], s["fb"], s["fo"], out=s["out"])
        return {**s["out"], "total": fc["total"]}  # (bytes past the total stay zero)
    if op == "merge":
        fc = s["fc"]
        return ss.lcp_merge(s["rb"], s["re"], s["go"], fc["lcp"], fc["len"], fc["id"], fc["suf_off"], fc["suf"],
                            ws=s["ws"], n_out=s["c"]["n"], with_len=True)
    if op == "decode":
        fc = s["fc"]
        return ss.fc_decode(s["run_off"], fc["lcp"], fc["len"], fc["suf_off"], fc["suf"])
    if op == "suffix":
        return ss.suffix_sort(s["text"], ws=s["ws"])
    # pdms: prefix doubling's first pass leaves the sorts' seed; every
    # element's array sorted; the other rounds; splitters; buckets and front
    # coding; each bucket's runs merged; exact distinguishing prefixes
    b, o, so, p = s["b"], s["o"], s["so"], s["c"]["p"]
    ss.dist_prefix_first_seed(b, o, 8, 64, ws=s["ws_pd"], seed=s["seed"], set_off=so)
    perm, lcp = ss.sort_batch_seeded(b, o, so, s["seed"], ws=s["ws_sort"], global_ids=True)
    dpx, rounds = ss.dist_prefix_rounds(b, o, s["ws_pd"], 8, 64)
    fb, fo = _splitters(b, o, perm, so, p, s["max_len"])
    fc = ss.partition_encode_batch(b, o, so, perm, lcp, dpx, fb, fo, ws=s["ws_pe"])
    ro = fc["run_off"].view(p, p + 1)
    rb, re = ro[:, :-1].t().reshape(-1), ro[:, 1:].t().reshape(-1)
    _, order, mlcp, mlen = ss.lcp_merge(rb, re, s["group_off"], fc["lcp"], fc["len"], fc["id"], fc["suf_off"],
                                        fc["suf"], ws=s["ws_merge"], n_out=s["c"]["n"], with_len=True,
                                        with_src=False)
    ss.join_group_lcps(b, o, order, mlcp, rb, re, s["group_off"])
    dist = ss.dist_exact_bounded(None, mlcp, mlen)
    return order, mlcp, dist, dpx, rounds


# -------------------------------------------------------------- its bytes

def _dist_bytes(c: dict) -> tuple[float, float]:
    """Mean distinguishing prefix and mean length of one string."""
    n = max(c.get("n", 2), 2)
    if c.get("kind") == "dn":
        return _filler(c) + _digits(n), c["length"]
    if c.get("kind") == "text":
        # a third of the strings have an equal one and count whole (mean
        # length 66); the others differ after some log(n) bytes
        return 0.33 * 66 + 0.67 * (1 + math.log(n) / 2.7), 66.0
    return 1 + math.log(n, 26), 132.0


def work(c: dict) -> dict:
    op = c["op"]
    if op in ("sets", "graph"):
        n = c["sets"] * (c["hi"] - c["lo"]) / math.log(c["hi"] / c["lo"])
        d, _ = _dist_bytes({"n": n / c["sets"]})
        return {"bytes": n * (d + 8 + 8), "flops": 0}
    n = c["n"]
    if op == "suffix":
        return {"bytes": n * (1 + 4 + 4), "flops": 0}
    d, length = _dist_bytes(c)
    if op == "sort":  # distinguishing bytes and offsets in; order and LCPs out
        return {"bytes": n * (d + 16), "flops": 0}
    if op == "job":  # ... and both kinds of dist
        return {"bytes": n * (d + 24), "flops": 0}
    sent = 1.0 * _digits(n) / 2 + 1 if c["kind"] == "dn" else (length - 3 if op in ("encode", "decode") else d - 3)
    if op == "encode":  # literals in and out; offset, order, LCP in; e, d, id, offset out
        return {"bytes": n * (2 * sent + 16 + 20), "flops": 0}
    if op == "merge":  # e, d, id, offset, a few literal bytes in; source, id, LCP, length out
        return {"bytes": n * (20 + min(sent, 8) + 20), "flops": 0}
    if op == "decode":  # e, d, offset, literals in; offset and strings out
        return {"bytes": n * (16 + sent + 8 + (d if c["kind"] == "dn" else length)), "flops": 0}
    # pdms: distinguishing bytes and offsets in; order, LCPs, both dists out;
    # the literals written once and read once
    return {"bytes": n * (d + 8 + 16 + 2 * sent), "flops": 0}
