"""The routing's top-k selections at the sizes where their form changes: one
and four entries per lane, the cut by lane maxima, a round shared by sixteen
waves; with a quarter of the chunks bit-identical copies of others, so that
ties at the boundary are decided by the index. Exact equality with the oracle,
near-ties included."""

from dataclasses import replace

import pytest
import torch

from oracle import hga_oracle as orc
from paper_2607_15105_amd import hga, synth
from tests import parity as P
from tests.test_gpu_rows import _gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def _wl(cands, n_q, first, **kw):
    """A call whose first row lies in the block with `cands` candidate chunks
    (one sink chunk, a two-chunk local window), `first` rows into it."""
    q0 = 64 * (cands + 2) + first
    T = -(-(q0 + n_q) // 64) * 64
    kw = {"top_chunks": 8, "top_groups": 16, "n_q_heads": 4, "n_kv_heads": 2, **kw}
    return synth.Workload("selection", T=T, head_dim=64, dtype="bf16", seed=41 + cands, q_begin=q0, n_q=n_q,
                          grad_begin=0, key_offset="normal", tie_copies=min(cands // 4, (cands - 7) // 2, 300), **kw)


def _check(wl, rows, Kn=None, Qn=None):
    hc, cfg = P.hcfg_of(wl), P.cfg_of(wl)
    end = wl.q_begin + wl.n_q
    if Kn is None:
        Kn, Qn = synth.keys(wl, 0, end), synth.queries(wl, wl.q_begin, end)
    K, Q = P.to_dev(Kn), P.to_dev(Qn)
    cs, gs = hga.alloc_summaries(hc, -(-end // 64) * 64)
    hga.build_summaries(hc, K, 0, end, cs, gs)
    if rows:
        sc, sg, ns = hga.alloc_route_rows(hc, wl.n_q)
        hga.route_rows(hc, Q, wl.q_begin, cs, gs, sc, sg, ns)
    else:
        rb = hga.alloc_route(hc, wl.q_begin, wl.n_q)
        hga.route(hc, Q, wl.q_begin, cs, gs, rb.sel_chunks, rb.sel_groups, rb.n_sel_groups, rb.workspace)
        sc, sg, ns = rb.sel_chunks, rb.sel_groups, rb.n_sel_groups
    torch.cuda.synchronize()
    ocs, ogs = orc.summaries(Kn, cfg, end)
    ro = (orc.route_rows if rows else orc.route)(Qn, ocs, ogs, cfg, wl.q_begin, wl.n_q)
    run = P.GpuRun(cs, gs, sc.cpu().numpy(), sg.cpu().numpy(), ns.cpu().numpy(), None, None)
    rep = P.compare_routing(wl, run, ro, ogs, Qn, rows=rows)
    print(f"[selection] exact={rep.exact} near_ties={rep.near_ties} mismatches={rep.mismatches}", flush=True)
    assert rep.mismatches == 0 and rep.near_ties == 0, rep.detail


@pytest.mark.parametrize("kc,kg", [(8, 16), (16, 64), (64, 13)])
@pytest.mark.parametrize("cands", [9, 64, 65, 256, 257, 289, 512, 513, 700])
def test_one_row(cands, kc, kg):
    """A decode step: four waves up to 512 candidates, sixteen beyond."""
    _check(_wl(cands, 1, 37, top_chunks=kc, top_groups=kg), True)


@pytest.mark.parametrize("cands", [63, 255, 511])
def test_rows_four_per_workgroup(cands):
    """Rows of two blocks, so of two candidate counts, four per workgroup."""
    _check(_wl(cands, 600, 50), True)


@pytest.mark.parametrize("cands,n_q,n_kv", [(64, 64, 2), (257, 128, 2), (700, 64, 2), (255, 4224, 4), (640, 8448, 2)])
def test_blocks(cands, n_q, n_kv):
    """Block routing with one and with several blocks per workgroup."""
    _check(_wl(cands, n_q, 0, n_kv_heads=n_kv, n_q_heads=2 * n_kv), False)


@pytest.mark.parametrize("cands", [257, 700, 4200])
def test_rows_one_per_workgroup(cands):
    """More (row, kv head) pairs than CUs, but too few rows for four per
    workgroup: one to two passes of 256 candidates, and two rounds of 4,096."""
    _check(_wl(cands, 40, 20, n_kv_heads=8, n_q_heads=8), True)


@pytest.mark.parametrize("kc,kg", [(8, 16), (16, 64), (64, 16), (64, 64)])
@pytest.mark.parametrize("steps", [1, 32])
@pytest.mark.parametrize("cands,n_q,rows", [(60, 1, True), (250, 40, True), (700, 1, True), (700, 600, True),
                                            (60, 64, False), (250, 64, False), (700, 64, False), (700, 8448, False)])
def test_equal_scores_and_shared_keys(cands, n_q, rows, steps, kc, kg):
    """Scores that are all equal (steps 1: the selection goes by position
    alone) and scores of 32 values 2^-20 apart at 256, which all round to one
    float: the routing's 32-bit keys cannot tell them apart."""
    wl = replace(_wl(cands, n_q, 0, top_chunks=kc, top_groups=kg), tie_copies=0)
    end, g = wl.q_begin + wl.n_q, wl.group_size
    tok = torch.arange(end)
    K = torch.zeros(end, 2, 64)
    K[:, :, 0] = 256.0
    K[:, 0, 1] = (tok // 64 * 7 % 32 % steps).float() * 2.0 ** -20
    K[:, 1, 1] = (tok // 64 * 13 % 32 % steps).float() * 2.0 ** -20
    K[:, :, 2] = ((tok // g * 5 % 8 % steps).float() * 2.0 ** -24)[:, None]
    Q = torch.zeros(wl.n_q, 4, 64)
    Q[:, :, :3] = 1.0
    K, Q = (x.to(torch.bfloat16).view(torch.int16).numpy().view("uint16") for x in (K, Q))
    _check(wl, rows, K, Q)
