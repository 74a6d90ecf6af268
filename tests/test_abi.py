"""C ABI checks that need no GPU: the library loads, exports every function
include/hga.h declares, sizes workspaces, and rejects invalid arguments on the
host (these calls return before any HIP call, so no device is touched)."""

import ctypes
import os
import re

import pytest

from paper_2607_15105_amd import hga

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000  # a 16-byte aligned non-null address; never dereferenced on these paths


def _declared():
    src = open(os.path.join(ROOT, "include", "hga.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(hga_\w+)\s*\(", src)))


def test_library_exports_every_declared_function():
    names = _declared()
    assert {"hga_build_summaries", "hga_route", "hga_attend_fwd", "hga_route_attend_fwd",
            "hga_attend_bwd", "hga_workspace_size", "hga_status_string"} <= set(names)
    L = hga.lib()
    for n in names:
        assert hasattr(L, n), n


def _cfg(**kw):
    base = dict(n_q_heads=32, n_kv_heads=8, head_dim=128)
    base.update(kw)
    import torch
    dtype = base.pop("dtype", torch.bfloat16)
    return hga.make_config(dtype=dtype, **base)


def test_workspace_sizes():
    c = _cfg()
    # routing keeps its descriptors and scores in LDS
    assert hga.workspace_size(c, hga.OP_ROUTE, 0, 2048) == 0
    # backward: D of every (row, query head), rounded up to 256 bytes, then
    # the dK/dV partials of 2 query-head subsets while the routable history
    # at the call's first block is under 6 k_c chunks
    dvec = lambda n_q: -(-n_q * 32 * 4 // 256) * 256
    part = lambda p, rows: 2 * p * rows * 8 * 128 * 4
    assert hga.workspace_size(c, hga.OP_BWD, 0, 2048, 0) == dvec(2048) + part(2, 2048)
    assert hga.workspace_size(c, hga.OP_BWD, 1024, 1024, 512) == dvec(1024) + part(2, 1536)
    assert hga.workspace_size(c, hga.OP_BWD, 3072, 1024, 3072) == dvec(1024) + part(2, 1024)  # 45 < 48
    assert hga.workspace_size(c, hga.OP_BWD, 4096, 1024, 4096) == dvec(1024)  # 61 history chunks
    assert hga.workspace_size(c, hga.OP_BWD, 15360, 1024, 15360) == dvec(1024)
    assert hga.workspace_size(_cfg(n_q_heads=8), hga.OP_BWD, 0, 1024, 0) == 1024 * 8 * 4  # G = 1: no split
    assert hga.workspace_size(c, hga.OP_BWD, 0, 100) == 0          # not a block multiple
    assert hga.workspace_size(c, hga.OP_BWD, 1024, 1024, 2048) == 0  # grad_begin after q_begin
    assert hga.workspace_size(_cfg(head_dim=96), hga.OP_ROUTE, 0, 64) == 0
    # the caller's choice of dK/dV work items per (chunk, kv head)
    assert hga.workspace_size(_cfg(bwd_kv_parts=1), hga.OP_BWD, 0, 2048, 0) == dvec(2048)
    assert hga.workspace_size(_cfg(bwd_kv_parts=2), hga.OP_BWD, 15360, 1024, 15360) == dvec(1024) + part(2, 1024)
    assert hga.workspace_size(_cfg(n_q_heads=8, bwd_kv_parts=2), hga.OP_BWD, 0, 1024, 0) == 1024 * 8 * 4
    assert hga.workspace_size(_cfg(bwd_kv_parts=3), hga.OP_BWD, 0, 1024, 0) == 0  # invalid
    assert hga.workspace_size(_cfg(bwd_kv_parts=-1), hga.OP_BWD, 0, 1024, 0) == 0


def test_status_strings():
    L = hga.lib()
    for code, text in hga.STATUS.items():
        assert L.hga_status_string(code).decode() == text


def _route(cfg, q_begin=0, n_q=2048, ws_bytes=1 << 20, q=FAKE, cap=None, strides=None):
    L = hga.lib()
    cap_c = cap if cap is not None else (q_begin + n_q) // 64
    cap_g = (q_begin + n_q) // cfg.group_size
    return L.hga_route(ctypes.byref(cfg), q, strides or hga.Strides(32 * 128, 128), q_begin, n_q, FAKE, cap_c,
                       FAKE, cap_g, FAKE, FAKE, FAKE, FAKE, ws_bytes, None)


@pytest.mark.parametrize("kw,status", [
    (dict(n_q_heads=30), -1),              # Hq not a multiple of Hkv
    (dict(n_q_heads=24), -2),              # GQA 3 unsupported
    (dict(head_dim=96), -2),
    (dict(chunk_size=32), -2),
    (dict(group_size=3), -1),
    (dict(top_chunks=-1), -1),
    (dict(top_groups=65), -2),
    (dict(sink_tokens=32), -1),
    (dict(local_tokens=0), -1),
])
def test_invalid_configs_are_rejected(kw, status):
    assert _route(_cfg(**kw)) == status


def test_invalid_ranges_and_buffers_are_rejected():
    c = _cfg()
    assert _route(c, n_q=100) == -1               # not a block multiple
    assert _route(c, q_begin=-64) == -1
    assert _route(c, q=0) == -1                   # null Q
    assert _route(c, q=FAKE + 2) == -1            # misaligned Q
    assert _route(c, cap=10) == -1                # summary table too small
    # a context beyond 8,192 chunks is routed in rounds, not refused: with a
    # summary table too small for it the call still fails on that argument
    assert _route(c, n_q=64 * 8193, cap=8192) == -1
    assert _route(c, n_q=0) == -1                 # empty: n_q > 0 is required
    assert _route(c, q_begin=64, n_q=-64) == -1
    # positions beyond 2^31 and strides of 4 GB or more: row offsets are
    # 32 x 32-bit products in the kernels
    assert _route(c, q_begin=(1 << 31) - 64, n_q=128) == -1
    assert _route(c, strides=hga.Strides(1 << 31, 128)) == -1   # 4 GB per token in bf16
    assert _route(c, strides=hga.Strides(32 * 128, 1 << 31)) == -1
    L = hga.lib()
    Skv = hga.Strides(8 * 128, 128)
    assert L.hga_build_summaries(ctypes.byref(c), FAKE, Skv, (1 << 31) - 64, (1 << 31) + 64,
                                 FAKE, 1 << 26, FAKE, 1 << 29, None) == -1
    # an empty or reversed key range
    assert L.hga_build_summaries(ctypes.byref(c), FAKE, Skv, 128, 128, FAKE, 64, FAKE, 512, None) == -1
    assert L.hga_build_summaries(ctypes.byref(c), FAKE, Skv, 128, 64, FAKE, 64, FAKE, 512, None) == -1
    import torch
    assert _route(_cfg(dtype=torch.float32)) == -2  # fp32 is built for head_dim 64


def test_backward_rejects_grad_begin_after_q_begin():
    c = _cfg()
    L = hga.lib()
    S = hga.Strides(32 * 128, 128)
    Skv = hga.Strides(8 * 128, 128)
    st = L.hga_attend_bwd(ctypes.byref(c), FAKE, S, FAKE, Skv, FAKE, Skv, FAKE, S, None, FAKE, S, FAKE,
                          1024, 1024, 2048, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 30, None)
    assert st == -1


@pytest.mark.parametrize("hq,hkv,short,longer", [(16, 2, 1024, 4032), (8, 2, 2048, 2112), (8, 1, 512, 512),
                                                 (32, 8, 256, 448), (32, 8, 1024, 1024)])
def test_backward_takes_a_buffer_of_two_subsets_or_of_a_longer_call(hq, hkv, short, longer):
    """What a call that splits its dK/dV work asks of its buffer is two query-head
    subsets, also where the library would take more: a buffer sized for a longer
    call, which may split less, does for a shorter one. o_f32 is misaligned, which is
    looked at after the buffer: no call gets as far as a launch."""
    c = _cfg(n_q_heads=hq, n_kv_heads=hkv)
    L = hga.lib()
    S, Skv = hga.Strides(hq * 128, 128), hga.Strides(hkv * 128, 128)
    status = lambda size: L.hga_attend_bwd(ctypes.byref(c), FAKE, S, FAKE, Skv, FAKE, Skv, FAKE, S, FAKE + 4, FAKE, S,
                                           FAKE, 0, short, 0, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, size, None)
    two = -(-short * hq * 4 // 256) * 256 + 2 * 2 * short * hkv * 128 * 4
    assert status(hga.workspace_size(c, hga.OP_BWD, 0, short, 0)) == -1
    assert status(hga.workspace_size(c, hga.OP_BWD, 0, longer, 0)) == -1
    assert status(two) == -1
    assert status(two - 1) == -3


def test_gather_rejects_short_or_unaligned_slots():
    c = _cfg()  # Ws 64 + Wl 128 + 16 groups of 8 = 320 rows per slot at least
    L = hga.lib()
    Skv = hga.Strides(8 * 128, 128)
    S = hga.Strides(32 * 128, 128)
    assert hga.gathered_rows(c) == 320
    gather = lambda r_cap, kc=FAKE: L.hga_gather_routed(ctypes.byref(c), FAKE, Skv, FAKE, Skv, 0, 1024, FAKE,
                                                        FAKE, kc, FAKE, r_cap, None)
    assert gather(256) == -1       # too few rows
    assert gather(352) == -1       # not a multiple of 64
    assert gather(320, kc=0) == -1
    fwd = lambda r_cap: L.hga_attend_gathered_fwd(ctypes.byref(c), FAKE, S, FAKE, FAKE, r_cap, 0, 1024,
                                                  FAKE, FAKE, S, FAKE, None, None)
    assert fwd(256) == -1
    assert fwd(330) == -1


def test_noalloc_backward_rejects_calls_beyond_its_scratch_on_the_host():
    """A backward whose workspace would exceed the library's static scratch
    returns HGA_ERR_WORKSPACE before any HIP call (no device is touched)."""
    c = _cfg()
    L = hga.lib()
    S = hga.Strides(32 * 128, 128)
    Skv = hga.Strides(8 * 128, 128)
    assert hga.workspace_size(c, hga.OP_BWD, 0, 4096, 0) > hga.NOALLOC_SCRATCH_BYTES
    st = L.hga_attend_bwd_noalloc(ctypes.byref(c), FAKE, S, FAKE, Skv, FAKE, Skv, FAKE, S, None, FAKE, S,
                                  FAKE, 0, 4096, 0, FAKE, FAKE, FAKE, FAKE, FAKE, None)
    assert st == -3
    # grad_begin after q_begin is still an argument error
    st = L.hga_attend_bwd_noalloc(ctypes.byref(c), FAKE, S, FAKE, Skv, FAKE, Skv, FAKE, S, None, FAKE, S,
                                  FAKE, 1024, 1024, 2048, FAKE, FAKE, FAKE, FAKE, FAKE, None)
    assert st == -1


def test_row_calls_take_any_position_and_reject_empty_ranges():
    """Per-query routing accepts unaligned positions and counts; empty or
    negative ranges are argument errors returned before any HIP call."""
    c = _cfg()
    L = hga.lib()
    S = hga.Strides(32 * 128, 128)
    route = lambda q_begin, n_q: L.hga_route_rows(ctypes.byref(c), FAKE, S, q_begin, n_q, FAKE, 1 << 20,
                                                  FAKE, 1 << 23, FAKE, FAKE, FAKE, None)
    assert route(100, 0) == -1
    assert route(-1, 5) == -1
    # no chunk limit: beyond 8,192 chunks a too-small summary table is still refused
    assert L.hga_route_rows(ctypes.byref(c), FAKE, S, 64, 64 * 8193, FAKE, 8192, FAKE, 1 << 23, FAKE, FAKE,
                            FAKE, None) == -1
    Skv = hga.Strides(8 * 128, 128)
    fwd = lambda q_begin, n_q: L.hga_attend_rows_fwd(ctypes.byref(c), FAKE, S, FAKE, Skv, FAKE, Skv, q_begin,
                                                     n_q, FAKE, FAKE, FAKE, S, FAKE, None, None)
    assert fwd(7, 0) == -1
    assert fwd(-64, 3) == -1
    Sq = hga.Strides(32 * 128, 128)
    bwd = lambda n_q, grad_begin: L.hga_attend_rows_bwd(ctypes.byref(c), FAKE, Sq, FAKE, Skv, FAKE, Skv, FAKE, Sq,
                                                        None, FAKE, Sq, FAKE, 2000, n_q, grad_begin, FAKE, FAKE,
                                                        FAKE, FAKE, FAKE, FAKE, 1 << 30, None)
    assert bwd(4097, 1920) == -2    # beyond the rows of one backward call
    assert bwd(16, 2048) == -1      # grad_begin after q_begin
    assert bwd(16, 100) == -1       # grad_begin not a multiple of C
    assert hga.rows_workspace_size(c, 4097) == 0
    assert hga.rows_workspace_size(c, 1000) == -(-1000 * 32 * 4 // 256) * 256


def test_tier_entry_points_reject_bad_arguments_on_the_host():
    c = _cfg()
    L = hga.lib()
    assert L.hga_host_device_view(None) is None
    cache = hga.GroupCache(FAKE, FAKE, FAKE, FAKE, 0, 256)      # no slots
    assert L.hga_group_cache_clear(ctypes.byref(c), ctypes.byref(cache), None) == -2
    cache = hga.GroupCache(FAKE, FAKE, FAKE, FAKE, 4097, 256)   # beyond the slot limit
    assert L.hga_group_cache_clear(ctypes.byref(c), ctypes.byref(cache), None) == -2
    cache = hga.GroupCache(FAKE, FAKE, FAKE, FAKE, 32, 256)
    S = hga.Strides(32 * 128, 128)
    # the slot map must cover the chunk table: chunk_cap 255 != 256
    st = L.hga_route_cached(ctypes.byref(c), FAKE, S, 0, 1024, FAKE, 255, FAKE, 2048, ctypes.byref(cache),
                            FAKE, FAKE, FAKE, FAKE, FAKE, 0, None)
    assert st == -1
    Skv = hga.Strides(8 * 128, 128)
    # history that ends after the call's first query, or off a chunk boundary
    g = lambda hist_end: L.hga_gather_tiered(ctypes.byref(c), FAKE, FAKE, Skv, hist_end, FAKE, FAKE, Skv, 1024,
                                             1024, FAKE, FAKE, FAKE, FAKE, 320, None)
    assert g(2048) == -1
    assert g(100) == -1


def test_prepared_calls_marshal_and_check_like_direct_calls():
    """A PreparedCall (the form a launch loop issues) converts its arguments
    once and reports the library's status like a direct call: here a config
    the library refuses on the host before reading any pointer."""
    c = _cfg(head_dim=96)
    args = (ctypes.byref(c), FAKE, hga.Strides(32 * 128, 128), 0, 2048, FAKE, 32, FAKE, 256,
            FAKE, FAKE, FAKE, FAKE, 1 << 20, None)
    pc = hga.PreparedCall("hga_route", args)
    assert pc.name == "hga_route"
    with pytest.raises(hga.HgaError) as e:
        pc()
    assert e.value.status == -2 == hga.lib().hga_route(*args)
    with pytest.raises(hga.HgaError):
        pc()  # issued again: the same result
