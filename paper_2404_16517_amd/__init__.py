"""Python binding of libstrsort (the C-ABI in include/strsort.h).

Argument marshalling only: every step runs in the HIP kernels of the shared
library.  PyTorch supplies device memory (tensors on a ROCm device) and the
current stream.  32-bit unsigned outputs are returned in ``torch.int32``
tensors holding the same bits; 64-bit unsigned ones in ``torch.int64``.
Strings are a ``uint8`` byte tensor plus an ``int64`` offsets tensor of n+1
entries (string i = bytes[offsets[i]:offsets[i+1]]).

There is no CPU fallback: without the built library or a GPU every call raises.
"""
from __future__ import annotations

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libstrsort.so")

SS_TUNE_SMALL_MAX = 1
SS_TUNE_TILE = 2
SS_TUNE_DIGIT_BITS = 3
SS_TUNE_DEDUP = 4
SS_TUNE_DEDUP_LOG_BUCKETS = 5
SS_ERR_CAPACITY = -5


class StrsortError(RuntimeError):
    pass


_lib = None


def lib():
    """The loaded shared library (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise StrsortError(f"{LIB_PATH} is missing: build it with `python -m paper_2404_16517_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        P, U32, U64, I32, SZ = ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64, ctypes.c_int, ctypes.c_size_t
        sig = {
            "ss_last_error": ([], ctypes.c_char_p),
            "ss_version": ([], I32),
            "ss_sort_workspace": ([U64], SZ),
            "ss_sort": ([P, U64, P, U64, P, P, P, SZ, P], I32),
            "ss_sort_seeded": ([P, U64, P, U64, P, P, P, P, SZ, P], I32),
            "ss_sort_seed_bytes": ([U64], SZ),
            "ss_dist_prefix_first_seed": ([P, U64, P, U64, P, U32, U32, U32, U32, P, P, SZ, P], I32),
            "ss_sort_batch_seeded": ([P, U64, P, U64, P, U32, P, P, P, U32, P, SZ, P], I32),
            "ss_sort_batch": ([P, U64, P, U64, P, U32, P, P, U32, P, SZ, P], I32),
            "ss_sort_batch_device_rounds": ([U32], U32),
            "ss_sort_batch_device": ([P, U64, P, U64, P, U32, P, P, U32, U32, P, P, SZ, P], I32),
            "ss_graph_begin": ([P], I32),
            "ss_graph_end": ([P, P], I32),
            "ss_graph_launch": ([P, P], I32),
            "ss_graph_nodes": ([P], SZ),
            "ss_graph_destroy": ([P], None),
            "ss_lcp": ([P, U64, P, U64, P, P, P], I32),
            "ss_dist_exact": ([P, U64, P, P, P, P], I32),
            "ss_dist_prefix_workspace": ([U64], SZ),
            "ss_dist_prefix": ([P, U64, P, U64, U32, U32, P, P, P, SZ, P], I32),
            "ss_dist_prefix_first": ([P, U64, P, U64, U32, U32, P, SZ, P], I32),
            "ss_dist_prefix_rounds": ([P, U64, P, U64, U32, U32, P, P, P, SZ, P], I32),
            "ss_doubling_keys": ([P, U64, P, U64, U32, U32, U32, U32, P, P, SZ, P], I32),
            "ss_select_splitters": ([U64, P, U32, P, P], I32),
            "ss_select_splitters_batch_workspace": ([], SZ),
            "ss_select_splitters_batch": ([P, U64, P, U32, U32, P, P, SZ, P], I32),
            "ss_gather_workspace": ([U64], SZ),
            "ss_select_splitters_chars_batch_workspace": ([U64], SZ),
            "ss_select_splitters_chars_batch": ([P, P, P, U64, P, U32, U32, P, P, SZ, P], I32),
            "ss_gather_strings": ([P, U64, P, U64, P, U64, P, P, U64, P, P, SZ, P], I32),
            "ss_bucket_bounds": ([P, U64, P, U64, P, P, U64, P, U32, P, P], I32),
            "ss_partition_encode_workspace": ([U64], SZ),
            "ss_partition_encode": ([P, U64, P, U64, P, P, P, P, U64, P, U32, P, P, P, P, P, P, U64, U64, P, P, SZ,
                                     P], I32),
            "ss_partition_encode_batch": ([P, U64, P, U64, P, U32, P, P, P, P, U64, P, U32, P, P, P, P, P, P, U64, U64,
                                           P, P, SZ, P], I32),
            "ss_fc_decode_workspace": ([U64], SZ),
            "ss_profile_enable": ([I32], None),
            "ss_profile_only": ([ctypes.c_char_p], None),
            "ss_profile_query": ([ctypes.c_char_p, P, P, P], I32),
            "ss_profile_names": ([ctypes.c_char_p, SZ], SZ),
            "ss_fc_decode": ([U32, P, P, P, P, P, U64, P, P, U64, P, SZ, P], I32),
            "ss_fc_decode_noalloc": ([U32, P, P, P, P, P, U64, P, P, U64, P, P], I32),
            "ss_lcp_merge_workspace": ([U64, U64, U32], SZ),
            "ss_lcp_merge": ([U32, P, P, U32, P, U64, P, P, P, P, P, P, P, P, P, U64, P, P, SZ, P], I32),
            "ss_dist_exact_bounded": ([P, P, P, U64, P, P], I32),
            "ss_join_group_lcps": ([P, U64, P, P, U64, U32, P, P, U32, P, P, P], I32),
            "ss_set_tuning": ([I32, I32], I32),
            "ss_suffix_sort_workspace": ([U64], SZ),
            "ss_suffix_sort": ([P, U64, P, P, P, P, SZ, P], I32),
        }
        for name, (args, res) in sig.items():
            f = getattr(L, name)
            f.argtypes = args
            f.restype = res
        _lib = L
    return _lib


# Addresses and streams go to the library as plain integers: building a stream
# object and a pointer object per argument took a third of the host time of a
# small call (sorting 48 strings: 9.6 us a call with them, 6.8 without; the kernel 5.2).

def _p(t: torch.Tensor | None):
    return t.data_ptr() if t is not None and t.numel() else None


def _stream(device) -> int:
    return torch._C._cuda_getCurrentRawStream(device.index)


def _check(rc: int):
    if rc != 0:
        msg = lib().ss_last_error().decode(errors="replace")
        raise StrsortError(f"strsort error {rc}: {msg}")


def _dev_strings(bytes_: torch.Tensor, offsets: torch.Tensor):
    if not bytes_.is_cuda or not offsets.is_cuda:
        raise StrsortError("strings must be on a GPU device")
    if bytes_.dtype != torch.uint8 or offsets.dtype != torch.int64:
        raise StrsortError("bytes must be uint8 and offsets int64")
    if not bytes_.is_contiguous() or not offsets.is_contiguous():
        raise StrsortError("bytes and offsets must be contiguous")
    return bytes_, offsets, offsets.numel() - 1


def _ws(nbytes: int, device) -> torch.Tensor:
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device=device)


def _u32(n: int, device) -> torch.Tensor:
    return torch.empty(max(n, 0), dtype=torch.int32, device=device)


def set_tuning(param: int, value: int) -> int:
    old = lib().ss_set_tuning(param, value)
    if old < 0:
        _check(old)
    return old


# ---------------------------------------------------------------- sorting

def sort(bytes_, offsets, with_lcp: bool = True, ws: torch.Tensor | None = None):
    """Stable sort + LCP array.  Returns (perm int32[n], lcp int32[n] or None)."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    perm = _u32(n, dev)
    lcp = _u32(n, dev) if with_lcp else None
    need = lib().ss_sort_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    _check(lib().ss_sort(_p(b), b.numel(), _p(o), n, _p(perm), _p(lcp), _p(ws), ws.numel(), _stream(dev)))
    return perm, lcp


SS_BATCH_GLOBAL_IDS = 1
SS_BATCH_CONTINUE = 2


def sort_batch(bytes_, offsets, set_off: torch.Tensor, with_lcp: bool = True, ws=None, global_ids: bool = False,
               out=None):
    """Independent sorts of the sets [set_off[j], set_off[j+1]) in one launch sequence.
    Returns (perm int32[n], lcp int32[n] or None); perm holds indices within
    each set, or indices of the whole array with ``global_ids``.  With
    ``out=(perm, lcp)`` (and the same ``ws``) it finishes an incomplete
    device-driven sort instead of starting over."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    so = set_off.to(device=dev, dtype=torch.int64).contiguous()
    cont = out is not None
    if cont:
        perm, lcp = out
    else:
        perm = _u32(n, dev)
        lcp = _u32(n, dev) if with_lcp else None
    need = lib().ss_sort_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    flags = (SS_BATCH_GLOBAL_IDS if global_ids else 0) | (SS_BATCH_CONTINUE if cont else 0)
    _check(lib().ss_sort_batch(_p(b), b.numel(), _p(o), n, _p(so), so.numel() - 1, _p(perm), _p(lcp),
                               flags, _p(ws), ws.numel(), _stream(dev)))
    return perm, lcp


def sort_batch_device_rounds(max_len: int) -> int:
    """Rounds after which the device-driven sort is complete for strings of at most max_len bytes."""
    return int(lib().ss_sort_batch_device_rounds(max_len))


def sort_batch_device(bytes_, offsets, set_off, perm, lcp_, status, ws, rounds: int, global_ids: bool = False,
                      cont: bool = False):
    """Device-driven batch sort into caller-supplied buffers (nothing is read
    back or allocated, so it can be captured in a Graph).  ``status``: int32
    device tensor of 2 words (unresolved segments, malformed set_off)."""
    b, o, n = _dev_strings(bytes_, offsets)
    if perm.numel() < n or (lcp_ is not None and lcp_.numel() < n) or status.numel() < 2:
        raise StrsortError("perm/lcp need n entries and status 2")
    _check(lib().ss_sort_batch_device(_p(b), b.numel(), _p(o), n, _p(set_off), set_off.numel() - 1, _p(perm),
                                      _p(lcp_), (SS_BATCH_GLOBAL_IDS if global_ids else 0) |
                                      (SS_BATCH_CONTINUE if cont else 0), rounds, _p(status),
                                      _p(ws), ws.numel(), _stream(b.device)))


class Graph:
    """A captured launch sequence of library calls (ss_graph_*), replayed with one launch."""

    def __init__(self, handle: ctypes.c_void_p):
        self._h = handle

    @classmethod
    def capture(cls, fn, stream: "torch.cuda.Stream") -> "Graph":
        """Record the library calls ``fn()`` makes on ``stream`` (made current
        while it runs); every buffer they use must already exist."""
        sp = ctypes.c_void_p(stream.cuda_stream)
        with torch.cuda.stream(stream):
            _check(lib().ss_graph_begin(sp))
            h = ctypes.c_void_p()
            try:
                fn()
            finally:
                rc = lib().ss_graph_end(sp, ctypes.byref(h))
        _check(rc)
        return cls(h)

    def launch(self, stream: "torch.cuda.Stream | None" = None):
        st = stream.cuda_stream if stream is not None else torch.cuda.current_stream().cuda_stream
        _check(lib().ss_graph_launch(self._h, ctypes.c_void_p(st)))

    def nodes(self) -> int:
        return int(lib().ss_graph_nodes(self._h))

    def close(self):
        if self._h:
            lib().ss_graph_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def lcp(bytes_, offsets, perm):
    """LCP array of the order ``perm`` (perm values index ``offsets``)."""
    b, o, _ = _dev_strings(bytes_, offsets)
    n = perm.numel()
    out = _u32(n, b.device)
    _check(lib().ss_lcp(_p(b), b.numel(), _p(o), n, _p(perm.contiguous()), _p(out), _stream(b.device)))
    return out


def dist_exact_bounded(perm, lcp_, d, n_strings=None):
    """Exact distinguishing prefixes from a per-position bound d (dist <= d <=
    len), e.g. the merged fc_len values: by input index (``perm`` given), or
    by sorted position (``perm`` None)."""
    n = lcp_.numel()
    if d.numel() != n or (perm is not None and perm.numel() != n):
        raise StrsortError("perm, lcp and d must have the same length")
    if perm is None:
        out = torch.empty(n, dtype=torch.int32, device=lcp_.device)
    else:
        size = n if n_strings is None else int(n_strings)
        out = torch.zeros(max(size, 0), dtype=torch.int32, device=perm.device)
    _check(lib().ss_dist_exact_bounded(_p(perm.contiguous()) if perm is not None else None, _p(lcp_.contiguous()),
                                       _p(d.contiguous()), n, _p(out), _stream(lcp_.device)))
    return out


def dist_exact(offsets, perm, lcp_, out=None):
    """Exact distinguishing prefixes by input index (sized like ``offsets``),
    into ``out`` when given (nothing is allocated then)."""
    n = perm.numel()
    if lcp_.numel() != n:
        raise StrsortError("perm and lcp must have the same length")
    if out is None:
        out = torch.zeros(max(offsets.numel() - 1, 0), dtype=torch.int32, device=offsets.device)
    _check(lib().ss_dist_exact(_p(offsets), n, _p(perm.contiguous()), _p(lcp_.contiguous()), _p(out),
                               _stream(offsets.device)))
    return out


def dist_prefix(bytes_, offsets, init_len: int = 8, hash_bits: int = 64, ws=None):
    """Prefix doubling.  Returns (dist_approx int32[n] by input index, rounds)."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    out = _u32(n, dev)
    need = lib().ss_dist_prefix_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    rounds = ctypes.c_uint32(0)
    _check(lib().ss_dist_prefix(_p(b), b.numel(), _p(o), n, init_len, hash_bits, _p(out), ctypes.byref(rounds),
                                _p(ws), ws.numel(), _stream(dev)))
    return out, int(rounds.value)


def dist_prefix_first(bytes_, offsets, init_len: int = 8, hash_bits: int = 64, ws=None):
    """The first hash pass of prefix doubling; returns the workspace that
    dist_prefix_rounds continues from."""
    b, o, n = _dev_strings(bytes_, offsets)
    need = lib().ss_dist_prefix_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, b.device)
    _check(lib().ss_dist_prefix_first(_p(b), b.numel(), _p(o), n, init_len, hash_bits, _p(ws), ws.numel(),
                                      _stream(b.device)))
    return ws


def dist_prefix_first_seed(bytes_, offsets, init_len: int = 8, hash_bits: int = 64, first_pass: str = "auto",
                           ws=None, seed=None, set_off: torch.Tensor | None = None):
    """dist_prefix_first that also leaves the sort's first-round seed (for
    the sets of set_off, or one set).  Returns (ws, seed); pass ws to
    dist_prefix_rounds and seed to sort_seeded / sort_batch_seeded."""
    b, o, n = _dev_strings(bytes_, offsets)
    nsets = 0
    if set_off is not None:
        set_off = set_off.to(device=b.device, dtype=torch.int64).contiguous()
        nsets = set_off.numel() - 1
    need = lib().ss_dist_prefix_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, b.device)
    sneed = lib().ss_sort_seed_bytes(n)
    if seed is None or seed.numel() < sneed:
        seed = _ws(sneed, b.device)
    _check(lib().ss_dist_prefix_first_seed(_p(b), b.numel(), _p(o), n, _p(set_off), nsets, init_len, hash_bits,
                                           FIRST_PASS_MODES[first_pass], _p(seed), _p(ws), ws.numel(),
                                           _stream(b.device)))
    return ws, seed


def sort_batch_seeded(bytes_, offsets, set_off: torch.Tensor, seed, with_lcp: bool = True, ws=None,
                      global_ids: bool = False):
    """sort_batch() whose first round uses the seed of dist_prefix_first_seed
    on the same strings and set_off (the seed is overwritten)."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    if seed.numel() < lib().ss_sort_seed_bytes(n):
        raise StrsortError("seed too small")
    set_off = set_off.to(device=dev, dtype=torch.int64).contiguous()
    perm = _u32(n, dev)
    lcp = _u32(n, dev) if with_lcp else None
    need = lib().ss_sort_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    flags = SS_BATCH_GLOBAL_IDS if global_ids else 0
    _check(lib().ss_sort_batch_seeded(_p(b), b.numel(), _p(o), n, _p(set_off), set_off.numel() - 1, _p(seed),
                                      _p(perm), _p(lcp), flags, _p(ws), ws.numel(), _stream(dev)))
    return perm, lcp


def sort_seeded(bytes_, offsets, seed, with_lcp: bool = True, ws: torch.Tensor | None = None):
    """sort() whose first round uses the seed of dist_prefix_first_seed on the
    same strings (the seed is overwritten)."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    if seed.numel() < lib().ss_sort_seed_bytes(n):
        raise StrsortError("seed too small")
    perm = _u32(n, dev)
    lcp = _u32(n, dev) if with_lcp else None
    need = lib().ss_sort_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    _check(lib().ss_sort_seeded(_p(b), b.numel(), _p(o), n, _p(seed), _p(perm), _p(lcp), _p(ws), ws.numel(),
                                _stream(dev)))
    return perm, lcp


def dist_prefix_rounds(bytes_, offsets, ws, init_len: int = 8, hash_bits: int = 64):
    """The remaining rounds after dist_prefix_first (same workspace).
    Returns (dist_approx int32[n] by input index, rounds)."""
    b, o, n = _dev_strings(bytes_, offsets)
    out = _u32(n, b.device)
    rounds = ctypes.c_uint32(0)
    _check(lib().ss_dist_prefix_rounds(_p(b), b.numel(), _p(o), n, init_len, hash_bits, _p(out),
                                       ctypes.byref(rounds), _p(ws), ws.numel(), _stream(b.device)))
    return out, int(rounds.value)


FIRST_PASS_MODES = {"auto": 0, "plain": 1, "deep": 2}


def doubling_keys(bytes_, offsets, init_len: int, rounds: int, hash_bits: int = 64, first_pass: str = "auto",
                  ws=None):
    """Keys of the first ``rounds`` prefix-doubling rounds of every string
    (all strings active): int64 tensor [rounds, n] of the masked keys."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    out = torch.empty((max(rounds, 0), max(n, 0)), dtype=torch.int64, device=dev)
    need = lib().ss_dist_prefix_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    _check(lib().ss_doubling_keys(_p(b), b.numel(), _p(o), n, init_len, hash_bits, rounds,
                                  FIRST_PASS_MODES[first_pass], _p(out), _p(ws), ws.numel(), _stream(dev)))
    return out


# ------------------------------------------------- splitters and coding

def select_splitters(perm: torch.Tensor, r: int):
    n = perm.numel()
    ids = _u32(max(r - 1, 0), perm.device)
    _check(lib().ss_select_splitters(n, _p(perm.contiguous()), r, _p(ids), _stream(perm.device)))
    return ids


def select_splitters_batch(perm: torch.Tensor, set_off: torch.Tensor, r: int, check: bool = True):
    """Regular samples of every set of a batch; (num_sets * (r-1),) uint32.
    check=False: set_off is not validated and nothing is read back."""
    n = perm.numel()
    so = set_off.to(device=perm.device, dtype=torch.int64).contiguous()
    k = max(so.numel() - 1, 0)
    ids = _u32(max(k * (r - 1), 0), perm.device)
    ws = _ws(lib().ss_select_splitters_batch_workspace(), perm.device) if check else None
    _check(lib().ss_select_splitters_batch(_p(perm.contiguous()), n, _p(so), k, r, _p(ids),
                                           _p(ws), ws.numel() if check else 0, _stream(perm.device)))
    return ids


def select_splitters_chars_batch(perm: torch.Tensor, offsets: torch.Tensor, set_off: torch.Tensor, r: int,
                                 weights: torch.Tensor | None = None):
    """Character-based regular samples of every set (r - 1 per set), by string
    lengths or by ``weights`` (per input index); (num_sets * (r-1),) uint32."""
    n = perm.numel()
    dev = perm.device
    so = set_off.to(device=dev, dtype=torch.int64).contiguous()
    k = max(so.numel() - 1, 0)
    ids = _u32(max(k * (r - 1), 0), dev)
    ws = _ws(lib().ss_select_splitters_chars_batch_workspace(n), dev)
    _check(lib().ss_select_splitters_chars_batch(_p(perm.contiguous()), _p(offsets),
                                                 _p(weights.contiguous()) if weights is not None else None, n,
                                                 _p(so), k, r, _p(ids), _p(ws), ws.numel(), _stream(dev)))
    return ids


def gather_strings(bytes_, offsets, ids: torch.Tensor, cap_hint: int | None = None, sync: bool = True):
    """Strings ids[0..m) as a new string array (bytes, offsets).  The byte
    buffer starts at ``cap_hint`` bytes (default 1 KiB per string) and is
    regrown once to the exact total if that is too small.  sync=False:
    nothing is read back; the whole buffer of cap_hint bytes is returned and
    strings that would not fit are left out (offsets[m] > cap_hint says so)."""
    b, o, n = _dev_strings(bytes_, offsets)
    dev = b.device
    m = ids.numel()
    out_off = torch.empty(m + 1, dtype=torch.int64, device=dev)
    ws = _ws(lib().ss_gather_workspace(m), dev)
    idc = ids.contiguous()
    cap = int(cap_hint) if cap_hint is not None else 1024 * m
    if not sync:
        out = torch.empty(max(cap, 1), dtype=torch.uint8, device=dev)
        _check(lib().ss_gather_strings(_p(b), b.numel(), _p(o), n, _p(idc), m, _p(out_off), _p(out), cap, None,
                                       _p(ws), ws.numel(), _stream(dev)))
        return out, out_off
    total = ctypes.c_uint64(0)
    for _ in range(2):
        out = torch.empty(max(cap, 1), dtype=torch.uint8, device=dev)
        rc = lib().ss_gather_strings(_p(b), b.numel(), _p(o), n, _p(idc), m, _p(out_off), _p(out), cap,
                                     ctypes.byref(total), _p(ws), ws.numel(), _stream(dev))
        if rc != SS_ERR_CAPACITY:
            break
        cap = int(total.value)
    _check(rc)
    return out[:int(total.value)], out_off


def bucket_bounds(bytes_, offsets, perm, spl_bytes, spl_offsets):
    """Bucket bounds (r+1 entries) of the sorted order ``perm`` (its values
    index ``offsets``; it may cover any part of the string array) for the
    r-1 splitters (spl_bytes, spl_offsets)."""
    b, o, _ = _dev_strings(bytes_, offsets)
    n = perm.numel()
    r = spl_offsets.numel()  # r-1 splitters
    out = torch.empty(r + 1, dtype=torch.int64, device=b.device)
    _check(lib().ss_bucket_bounds(_p(b), b.numel(), _p(o), n, _p(perm.contiguous()), _p(spl_bytes),
                                  spl_bytes.numel(), _p(spl_offsets), r, _p(out), _stream(b.device)))
    return out


def partition_encode(bytes_, offsets, perm, lcp_, dist, spl_bytes, spl_offsets, suf_cap: int | None = None,
                     out: dict | None = None, suf_base: int = 0, n: int | None = None):
    """Buckets + front coding.  Returns a dict of device tensors:
    run_off (r+1), lcp, len, id (n, int32 bits), suf_off (n+1), suf (uint8), total (int).

    ``out`` may supply preallocated output tensors (same keys, ``suf`` being the
    whole shared literal buffer); literals are then written at ``suf_base``.
    ``n`` (default: offsets.numel()-1) is the number of sorted positions in
    ``perm``; perm values index ``offsets``."""
    b, o, n_all = _dev_strings(bytes_, offsets)
    n = n_all if n is None else n
    dev = b.device
    r = spl_offsets.numel()
    if out is None:
        cap = b.numel() if suf_cap is None else suf_cap
        out = dict(run_off=torch.empty(r + 1, dtype=torch.int64, device=dev), lcp=_u32(n, dev), len=_u32(n, dev),
                   id=_u32(n, dev), suf_off=torch.empty(n + 1, dtype=torch.int64, device=dev),
                   suf=torch.empty(max(cap, 1), dtype=torch.uint8, device=dev))
    cap = out["suf"].numel()
    ws = _ws(lib().ss_partition_encode_workspace(n), dev)
    total = ctypes.c_uint64(0)
    _check(lib().ss_partition_encode(_p(b), b.numel(), _p(o), n, _p(perm.contiguous()), _p(lcp_.contiguous()),
                                     _p(dist.contiguous()) if dist is not None else None, _p(spl_bytes),
                                     spl_bytes.numel(), _p(spl_offsets), r, _p(out["run_off"]), _p(out["lcp"]),
                                     _p(out["len"]), _p(out["id"]), _p(out["suf_off"]), _p(out["suf"]), suf_base, cap,
                                     ctypes.byref(total), _p(ws), ws.numel(), _stream(dev)))
    t = int(total.value)
    res = dict(out)
    res["total"] = t
    if suf_base == 0:
        res["suf"] = out["suf"][:t]
    return res


def partition_encode_batch(bytes_, offsets, set_off, perm, lcp_, dist, spl_bytes, spl_offsets, ws=None):
    """Buckets + front coding of several sorted arrays (sets of positions
    [set_off[b], set_off[b+1]) of perm/lcp) with common splitters, one call.
    Returns a dict: run_off (sets*(r+1), absolute), lcp, len, id, suf_off, suf, total."""
    b, o, _ = _dev_strings(bytes_, offsets)
    dev = b.device
    n = perm.numel()
    so = set_off.to(device=dev, dtype=torch.int64).contiguous()
    B = so.numel() - 1
    r = spl_offsets.numel()
    out = dict(run_off=torch.empty(B * (r + 1), dtype=torch.int64, device=dev), lcp=_u32(n, dev), len=_u32(n, dev),
               id=_u32(n, dev), suf_off=torch.empty(n + 1, dtype=torch.int64, device=dev),
               suf=torch.empty(max(b.numel(), 1), dtype=torch.uint8, device=dev))
    need = lib().ss_partition_encode_workspace(n)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    total = ctypes.c_uint64(0)
    _check(lib().ss_partition_encode_batch(_p(b), b.numel(), _p(o), n, _p(so), B, _p(perm.contiguous()),
                                           _p(lcp_.contiguous()), _p(dist.contiguous()) if dist is not None else None,
                                           _p(spl_bytes), spl_bytes.numel(), _p(spl_offsets), r, _p(out["run_off"]),
                                           _p(out["lcp"]), _p(out["len"]), _p(out["id"]), _p(out["suf_off"]),
                                           _p(out["suf"]), 0, out["suf"].numel(), ctypes.byref(total), _p(ws),
                                           ws.numel(), _stream(dev)))
    out["total"] = int(total.value)
    return out


# -------------------------------------------------------------- profiling

def profile_enable(on: bool = True):
    """Record HIP events around the library's main kernels (clears old records)."""
    lib().ss_profile_enable(1 if on else 0)


def profile_only(name: str | None = None):
    """Record only the launches of kernel `name` (None: all)."""
    lib().ss_profile_only(name.encode() if name else None)


def profile_report() -> dict:
    """{kernel: (ms, algorithmic bytes, launches)} for the records so far."""
    L = lib()
    need = L.ss_profile_names(None, 0)
    buf = ctypes.create_string_buffer(need + 1)
    L.ss_profile_names(buf, need + 1)
    out = {}
    for name in filter(None, buf.value.decode().split(",")):
        ms, by, cnt = ctypes.c_double(), ctypes.c_double(), ctypes.c_uint32()
        if L.ss_profile_query(name.encode(), ctypes.byref(ms), ctypes.byref(by), ctypes.byref(cnt)) == 0:
            out[name] = (ms.value, by.value, cnt.value)
    return out


def fc_decode(run_off, fc_lcp, fc_len, suf_off, suf):
    """Decode front-coded runs.  Returns (bytes uint8, offsets int64[n+1])."""
    dev = fc_lcp.device
    n = fc_lcp.numel()
    k = run_off.numel() - 1
    out_off = torch.empty(n + 1, dtype=torch.int64, device=dev)
    total = int(fc_len.to(torch.int64).sum()) if n else 0
    out = torch.empty(max(total, 1), dtype=torch.uint8, device=dev)
    ws = _ws(lib().ss_fc_decode_workspace(n), dev)
    _check(lib().ss_fc_decode(k, _p(run_off), _p(fc_lcp), _p(fc_len), _p(suf_off), _p(suf), n, _p(out_off),
                              _p(out), total, _p(ws), ws.numel(), _stream(dev)))
    return out[:total], out_off


SS_FC_DECODE_NOALLOC_MAX = 1 << 22


def fc_decode_noalloc(run_off, fc_lcp, fc_len, suf_off, suf, out_offsets, out_bytes, status):
    """ss_fc_decode_noalloc into caller-supplied outputs (the library allocates
    nothing).  ``status`` is an int32 device tensor of one element: 0 decoded,
    1 malformed runs, 2 capacity (``out_bytes.numel()``) exceeded."""
    dev = fc_lcp.device
    n = fc_lcp.numel()
    k = run_off.numel() - 1
    _check(lib().ss_fc_decode_noalloc(k, _p(run_off), _p(fc_lcp), _p(fc_len), _p(suf_off), _p(suf), n,
                                      _p(out_offsets), _p(out_bytes), out_bytes.numel(), _p(status), _stream(dev)))


def lcp_merge(run_begin, run_end, group_off, fc_lcp, fc_len, fc_id, suf_off, suf, ws=None, n_out=None,
              with_len=False, with_src=True):
    """LCP-aware merge of the runs [run_begin[j], run_end[j]) of shared
    front-coded arrays, one merged sequence per group of runs
    (group g = runs group_off[g]..group_off[g+1]-1).  ``n_out`` (the total run
    size), when the caller knows it, saves computing it here.
    Returns (src int64[n_out] or None without ``with_src``, id int32[n_out],
    lcp int32[n_out]), and the merged fc_len values as a fourth array with
    ``with_len``."""
    dev = fc_lcp.device
    n_fc = fc_lcp.numel()
    rb = run_begin.to(device=dev, dtype=torch.int64).contiguous()
    re_ = run_end.to(device=dev, dtype=torch.int64).contiguous()
    go = group_off.to(device=dev, dtype=torch.int32).contiguous()
    k = rb.numel()
    if n_out is None:
        n_out = int((re_ - rb).sum()) if k else 0
    need = lib().ss_lcp_merge_workspace(n_out, n_fc, k)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    src = torch.empty(max(n_out, 0), dtype=torch.int64, device=dev) if with_src else None
    idv, lc = _u32(n_out, dev), _u32(n_out, dev)
    ln = _u32(n_out, dev) if with_len else None
    got = ctypes.c_uint64(0)
    _check(lib().ss_lcp_merge(k, _p(rb), _p(re_), go.numel() - 1, _p(go), n_fc, _p(fc_lcp), _p(fc_len), _p(fc_id),
                              _p(suf_off), _p(suf), _p(src) if with_src else None, _p(idv), _p(lc),
                              _p(ln) if with_len else None, n_out,
                              ctypes.byref(got), _p(ws), ws.numel(), _stream(dev)))
    if got.value != n_out:
        raise StrsortError(f"runs hold {got.value} entries, n_out = {n_out}")
    return (src, idv, lc, ln) if with_len else (src, idv, lc)


def join_group_lcps(bytes_, offsets, order, lcp_, run_begin, run_end, group_off):
    """Set lcp_ (in place) at the first position of every merged group to the
    LCP with the last string of the groups before it."""
    b, o, _ = _dev_strings(bytes_, offsets)
    dev = b.device
    rb = run_begin.to(device=dev, dtype=torch.int64).contiguous()
    re_ = run_end.to(device=dev, dtype=torch.int64).contiguous()
    go = group_off.to(device=dev, dtype=torch.int32).contiguous()
    if not lcp_.is_contiguous() or lcp_.numel() != order.numel():
        raise StrsortError("lcp must be contiguous and sized like order")
    _check(lib().ss_join_group_lcps(_p(b), b.numel(), _p(o), _p(order.contiguous()), order.numel(), rb.numel(),
                                    _p(rb), _p(re_), go.numel() - 1, _p(go), _p(lcp_), _stream(dev)))
    return lcp_


def lcp_merge_runs(run_off, fc_lcp, fc_len, fc_id, suf_off, suf, ws=None):
    """Merge contiguous runs [run_off[j], run_off[j+1]) into one sequence."""
    ro = run_off.to(dtype=torch.int64)
    k = ro.numel() - 1
    go = torch.tensor([0, k], dtype=torch.int32, device=fc_lcp.device)
    return lcp_merge(ro[:-1], ro[1:], go, fc_lcp, fc_len, fc_id, suf_off, suf, ws=ws)


# ---------------------------------------------------------------- suffixes

def suffix_sort(text: torch.Tensor, with_lcp: bool = True, ws=None):
    """Suffix array (and LCP array) of a uint8 device tensor.
    Returns (sa int32[N], lcp int32[N] or None, steps)."""
    if not text.is_cuda or text.dtype != torch.uint8 or not text.is_contiguous():
        raise StrsortError("text must be a contiguous uint8 GPU tensor")
    N = text.numel()
    dev = text.device
    sa = _u32(N, dev)
    lc = _u32(N, dev) if with_lcp else None
    need = lib().ss_suffix_sort_workspace(N)
    if ws is None or ws.numel() < need:
        ws = _ws(need, dev)
    steps = ctypes.c_uint32(0)
    _check(lib().ss_suffix_sort(_p(text), N, _p(sa), _p(lc), ctypes.byref(steps), _p(ws), ws.numel(),
                                _stream(dev)))
    return sa, lc, int(steps.value)
