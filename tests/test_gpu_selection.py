"""The routing's top-k selections at the sizes where their form changes: one
and four entries per lane, the cut by lane maxima, a round shared by sixteen
waves; with a quarter of the chunks bit-identical copies of others, so that
ties at the boundary are decided by the index. Exact equality with the oracle,
near-ties included."""

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


def _check(wl, rows):
    hc, cfg = P.hcfg_of(wl), P.cfg_of(wl)
    end = wl.q_begin + wl.n_q
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
@pytest.mark.parametrize("cands", [9, 64, 65, 256, 257, 289, 700])
def test_one_row(cands, kc, kg):
    """A decode step: four waves up to 256 candidates, sixteen beyond."""
    _check(_wl(cands, 1, 37, top_chunks=kc, top_groups=kg), True)


@pytest.mark.parametrize("cands", [63, 255, 511])
def test_rows_four_per_workgroup(cands):
    """Rows of two blocks, so of two candidate counts, four per workgroup."""
    _check(_wl(cands, 600, 50), True)


@pytest.mark.parametrize("cands,n_q,n_kv", [(64, 64, 2), (257, 128, 2), (700, 64, 2), (255, 4224, 4), (640, 8448, 2)])
def test_blocks(cands, n_q, n_kv):
    """Block routing with one and with several blocks per workgroup."""
    _check(_wl(cands, n_q, 0, n_kv_heads=n_kv, n_q_heads=2 * n_kv), False)
