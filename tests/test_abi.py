"""The C-ABI library loads, exports every symbol the header declares, and
rejects bad arguments on the host before any GPU work (CPU only)."""
import ctypes
import os
import re

import pytest

from paper_2503_11367_amd import binding as mb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x1000          # non-null, 256-aligned, never dereferenced on an error path


def header_symbols():
    text = open(os.path.join(ROOT, "include", "mmattn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mmattn_[a-z_]+)\s*\(", text)))


def test_exports_match_header():
    L = mb.lib()
    syms = header_symbols()
    assert set(syms) >= {"mmattn_mask_encode", "mmattn_tile_map", "mmattn_balance", "mmattn_fwd",
                         "mmattn_bwd", "mmattn_workspace_size", "mmattn_version"}
    for s in syms:
        assert hasattr(L, s), s
    assert b"gfx950" in L.mmattn_version()


def spans_arr(items):
    arr = (mb.Span * max(len(items), 1))()
    for i, it in enumerate(items):
        arr[i] = mb.Span(*it)
    return arr


def encode_rc(spans, offs, S, bits=FAKE, ws=FAKE, ws_bytes=1 << 20):
    arr = spans_arr(spans)
    off = (ctypes.c_int64 * len(offs))(*offs)
    return mb.lib().mmattn_mask_encode(ctypes.addressof(arr) if spans else 0, len(spans),
                                       ctypes.addressof(off), len(offs) - 1, S, bits, ws, ws_bytes, 0)


def test_encode_validation():
    assert encode_rc([], [0, 64], 64, bits=0) == -1
    assert encode_rc([], [0, 64], 0) == -2
    assert encode_rc([], [0, 32], 64) == -5                      # last offset != S
    assert encode_rc([], [0, 40, 40, 64], 64) == -5              # empty sample
    assert encode_rc([(8, 8, 1, 0), (12, 4, 1, 0)], [0, 64], 64) == -5      # overlap
    assert encode_rc([(20, 8, 1, 0), (4, 4, 1, 0)], [0, 64], 64) == -5      # unsorted
    assert encode_rc([(60, 8, 1, 0)], [0, 64], 64) == -5                    # past the end
    assert encode_rc([(28, 8, 1, 0)], [0, 32, 64], 64) == -5                # crosses samples
    assert encode_rc([(8, 8, 0, 0)], [0, 64], 64) == -5                     # modality 0 is text
    assert encode_rc([(8, 8, 8, 0)], [0, 64], 64) == -5                     # one attend bit per modality
    assert encode_rc([(8, 8, 1, 4)], [0, 64], 64) == -5                     # unknown flag bit
    assert encode_rc([(8, 8, 1, 2 | 1)], [0, 64], 64) == -5                 # no bidirectional term, no causal bit
    assert encode_rc([(8, 8, 1, 2 | (2 << 8))], [0, 64], 64) == -5          # ... or own modality denied
    assert encode_rc([(8, 8, 1, 0)], [0, 64], 64, ws=0) == -4
    # a look-back window (flags bits 16-31, here the largest) passes the layout checks
    assert encode_rc([(8, 8, 1, 2 | (0xFFFF << 16) - (1 << 32))], [0, 64], 64, ws=0) == -4
    assert encode_rc([(8, 8, 1, 4 | (100 << 16))], [0, 64], 64, ws=0) == -5
    assert encode_rc([(8, 8, 1, 0)], [0, 64], 64, ws_bytes=8) == -4
    assert encode_rc([(8, 8, 1, 0)], [0, 64], 64, ws=FAKE + 8) == -4        # misaligned


def test_tile_map_validation():
    f = mb.lib().mmattn_tile_map
    assert f(0, 512, 64, 64, FAKE, FAKE, FAKE, 0) == -1
    assert f(FAKE, 512, 64, 64, FAKE, 0, FAKE, 0) == -1
    assert f(FAKE, 500, 64, 64, FAKE, FAKE, FAKE, 0) == -2
    assert f(FAKE, 512, 0, 64, FAKE, FAKE, FAKE, 0) == -2
    assert f(FAKE, 512, 64, 48, FAKE, FAKE, FAKE, 0) == -2
    assert f(FAKE, 1 << 20, 8, 64, FAKE, FAKE, FAKE, 0) == -3     # too many q-tiles


def test_balance_validation():
    f = mb.lib().mmattn_balance
    assert f(0, 8, 2, FAKE, FAKE, FAKE, FAKE, 0) == -1
    assert f(FAKE, 0, 2, FAKE, FAKE, FAKE, FAKE, 0) == -2
    assert f(FAKE, 8, 0, FAKE, FAKE, FAKE, FAKE, 0) == -2
    assert f(FAKE, 1 << 20, 2, FAKE, FAKE, FAKE, FAKE, 0) == -3
    assert f(FAKE, 8, 5000, FAKE, FAKE, FAKE, FAKE, 0) == -3


def fwd_rc(q=FAKE, k=FAKE, v=FAKE, bits=FAKE, blocks=FAKE, n_blocks=4, block=128, S=1024, Hq=4,
           Hkv=2, D=128, scale=0.1, dtype=0, o=FAKE, lse=FAKE, ws=FAKE, ws_bytes=1 << 30):
    return mb.lib().mmattn_fwd(q, k, v, bits, blocks, n_blocks, block, S, Hq, Hkv, D, scale, dtype,
                               o, lse, ws, ws_bytes, 0)


def test_fwd_validation():
    assert fwd_rc(q=0) == -1 and fwd_rc(o=0) == -1 and fwd_rc(blocks=0) == -1
    assert fwd_rc(Hq=3) == -2                 # Hq % Hkv
    assert fwd_rc(S=1000) == -2               # S % block
    assert fwd_rc(n_blocks=9) == -2           # more blocks than the sequence has
    assert fwd_rc(scale=0.0) == -2
    assert fwd_rc(D=96) == -3
    assert fwd_rc(dtype=1) == -3
    assert fwd_rc(block=8, S=1024) == -3      # block % 16
    assert fwd_rc(S=1 << 23, n_blocks=(65535 * 64) // 128 + 1) == -3      # share too long for one launch
    assert fwd_rc(q=FAKE + 2) == -2           # alignment
    assert fwd_rc(ws=0) == -4
    assert fwd_rc(ws_bytes=16) == -4
    # an empty share is valid, needs no per-row buffers and launches nothing
    assert fwd_rc(n_blocks=0, q=0, blocks=0, o=0, lse=0, ws=0, ws_bytes=0) == 0
    assert fwd_rc(n_blocks=0, k=0) == -1 and fwd_rc(n_blocks=-1) == -2


def test_fwd_heads_validation():
    f = mb.lib().mmattn_fwd_heads

    def rc(begin, count, n_blocks=4, ws_bytes=1 << 30):
        return f(FAKE, FAKE, FAKE, FAKE, FAKE, n_blocks, 128, 1024, 8, 4, 128, 0.1, 0, begin, count, 0,
                 FAKE, FAKE, FAKE, ws_bytes, 0)
    assert rc(-1, 1) == -2 and rc(0, 0) == -2 and rc(3, 2) == -2 and rc(4, 1) == -2
    assert rc(0, 5) == -2
    assert rc(1, 2, ws_bytes=64) == -4
    assert rc(1, 2, n_blocks=0) == 0              # empty share: nothing to do
    # one workspace serves every window, and is at least the whole-launch one
    w_all = mb.workspace_size(mb.OP_FWD, 1024, 4, 128, 8, 4, 128)
    w_win = mb.workspace_size(mb.OP_FWD_HEADS, 1024, 4, 128, 8, 4, 128)
    assert w_win >= w_all > 0


def test_fwd_staged_validation():
    f = mb.lib().mmattn_fwd_staged

    def rc(hps=1, k_src=FAKE, copy=FAKE, stream=0, ws_bytes=1 << 30):
        return f(FAKE, k_src, FAKE, FAKE, FAKE, FAKE, FAKE, 4, 128, 1024, 8, 4, 128, 0.1, 0, hps,
                 FAKE, FAKE, FAKE, ws_bytes, copy, stream)
    assert rc(k_src=0) == -1
    assert rc(hps=0) == -2 and rc(hps=3) == -2
    assert rc(copy=0, stream=0) == -2             # the two streams must differ
    assert rc(ws_bytes=64) == -4


def test_bwd_validation():
    f = mb.lib().mmattn_bwd
    args = [FAKE, FAKE, FAKE, FAKE, FAKE, 4, 128, 1024, 4, 2, 128, 0.1, 0,
            FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 30, 0]
    bad = list(args); bad[15] = 0
    assert f(*bad) == -1
    bad = list(args); bad[8] = 3
    assert f(*bad) == -2
    bad = list(args); bad[20] = 16
    assert f(*bad) == -4


def test_workspace_size_monotone():
    a = mb.workspace_size(mb.OP_FWD, 8192, 64, 128, 32, 8, 128)
    b = mb.workspace_size(mb.OP_FWD, 16384, 128, 128, 32, 8, 128)
    assert 0 < a < b
    assert mb.workspace_size(mb.OP_TILE_MAP, 8192, 0, 0) == 0
    assert mb.workspace_size(mb.OP_ENCODE, 8192, 4, 1) >= 4 * 24 + 16


@pytest.mark.parametrize("S,n_blocks,Hq,Hkv,D", [(512, 4, 8, 8, 128), (512, 1, 64, 8, 64), (256, 2, 16, 2, 128),
                                                 (8192, 64, 16, 16, 128), (4096, 32, 32, 8, 128), (4096, 32, 32, 8, 64)])
def test_no_partial_buffers_where_no_list_is_cut(S, n_blocks, Hq, Hkv, D):
    """Up to eight key tiles, or 512 work items or more (pairs of heads, where they are even):
    no list is cut, so the workspaces hold no partial results."""
    tiles, out_fp32 = n_blocks * (S // 64), n_blocks * 128 * Hq * D * 4
    plan = 5 * tiles + 256 * 16 + Hkv * 64 * 4 + 8 * n_blocks * 128       # lists, norms, tables, alignment
    assert mb.workspace_size(mb.OP_FWD, S, n_blocks, 128, Hq, Hkv, D) <= plan
    if S <= 512:
        # the backward's copies of Q and dO (bf16) and its rows' constants; its pool of dK, dV partials
        # belongs to the pass over keys
        pool = (S // 128) * (Hq // Hkv) * 2 * 128 * Hkv * D * 4
        rows = 2 * out_fp32 // 2 + 4 * n_blocks * 128 * (4 * Hq + 3)
        assert mb.workspace_size(mb.OP_BWD, S, n_blocks, 128, Hq, Hkv, D) <= rows + pool + plan + 4 * tiles + 256 * 16
    # one that is cut has room for slices of at least four tiles
    assert mb.workspace_size(mb.OP_FWD, 2048, 2, 128, 2, 1, 128) >= 8 * 256 * 2 * (128 + 2) * 4


def test_current_stream_without_the_raw_handle(monkeypatch):
    """A torch without the raw-handle function: the Stream object's handle is used; likewise
    before CUDA is initialised, and for a stream given as an object or a handle."""
    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(mb.torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(mb.torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(mb.torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(mb, "_raw_stream", None)
    assert mb._stream(None) == 77
    monkeypatch.setattr(mb, "_raw_stream", lambda device: 100 + device)
    assert mb._stream(None) == 103
    monkeypatch.setattr(mb.torch.cuda, "is_initialized", lambda: False)
    assert mb._stream(None) == 77
    assert mb._stream(Stream) == 77 and mb._stream(5) == 5


def test_span_list_packing():
    """mask_encode's span list as one by one: lists longer than one packing call, values that need
    converting or wrapping, flags in whatever answers flags[i]."""
    import numpy as np
    rng = np.random.default_rng(3)

    def plain(spans, flags):
        arr = (mb.Span * max(len(spans), 1))()
        for i, (st, ln, mod) in enumerate(spans):
            arr[i] = mb.Span(int(st), int(ln), int(mod), int(flags[i]) if flags is not None else 0)
        return bytes(arr)

    for n in (0, 1, 255, 256, 257, 1000):
        spans = [tuple(int(x) for x in rng.integers(0, 1 << 31, 3)) for _ in range(n)]
        flags = [int(x) for x in rng.integers(-(1 << 31), 1 << 31, n)]
        for f in (None, flags, tuple(flags), np.array(flags), dict(enumerate(flags)), flags + [7]):
            assert bytes(mb._span_array(spans, f)) == plain(spans, f), (n, type(f))
        for odd in ((1.9, 2, 1), (np.int64(5), True, 2), ("7", 8, 1), (1, 2, 1 << 33), (0, 5, 1)):
            assert bytes(mb._span_array(spans + [odd], None)) == plain(spans + [odd], None), odd
        big = flags + [0x80000001]
        assert bytes(mb._span_array(spans + [(1, 2, 1)], big)) == plain(spans + [(1, 2, 1)], big)
    for bad in ([1], 5):
        with pytest.raises((IndexError, TypeError)):
            mb._span_array([(0, 1, 1), (4, 1, 1)], bad)


def test_span_list_packing_keeps_nothing_of_long_lists():
    """Long lists of many different lengths: a compiled format of each would stay in the process (5 MB
    for 40000 spans).  Formats of at most 256 spans, 100 of them: below 4 MB."""
    import tracemalloc
    tracemalloc.start()
    try:
        before = tracemalloc.get_traced_memory()[0]
        for n in range(40000, 40010):
            mb._span_array([(1, 2, 1)] * n, None)
        assert tracemalloc.get_traced_memory()[0] - before < 4 << 20
    finally:
        tracemalloc.stop()


def test_balance_read_validation():
    f = mb.lib().mmattn_balance_read
    ok = dict(W=FAKE, nB=8, P=2, rob=FAKE, load=FAKE, off=FAKE, blocks=FAKE, box=FAKE, size=48, ticket=1, h=FAKE, ho=FAKE,
              st=0)
    rc = lambda **k: f(*dict(ok, **k).values())                                 # noqa: E731
    assert all(rc(**{n: 0}) == -1 for n in ("W", "rob", "load", "off", "blocks", "box", "h", "ho"))
    assert rc(nB=0) == -2 and rc(P=0) == -2 and rc(nB=1 << 20) == -3 and rc(P=5000) == -3
    assert rc(box=FAKE + 4) == -2 and rc(size=47) == -4
