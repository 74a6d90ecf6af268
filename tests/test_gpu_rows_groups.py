"""Per-query attention on groups of rows (hga_attend_rows_fwd, bf16): the
four forms a call can take (a wave per group, four waves per group, four or
twelve waves per row), with partial first and last groups, for every head ratio; and
what a row does not attend stays out of its result, infinities and NaN too,
although the rows of a group share products."""

from dataclasses import replace

import pytest
import torch

from paper_2607_15105_amd import hga, synth
from tests import parity as P
from tests.test_gpu_rows import _gpu, _rows_bwd_check, _rows_check  # noqa: F401

pytestmark = pytest.mark.gpu


# 232 keys a row: four waves per row up to 640 (row, kv head) pairs (256 with
# eight heads), then four waves per group, and from 1,024 (group, kv head) pairs
# a wave per group
@pytest.mark.parametrize("n_q,q_begin", [(1, 1787), (63, 1500), (66, 1537), (99, 1501), (515, 1501)])
@pytest.mark.parametrize("G,d", [(1, 64), (2, 64), (4, 128), (8, 64)])
def test_rows_forms(G, d, n_q, q_begin):
    wl = synth.Workload("rows_forms", T=2048, n_q_heads=8 * G, n_kv_heads=8, head_dim=d, dtype="bf16", seed=31,
                        q_begin=q_begin, n_q=n_q, grad_begin=0, key_offset="normal", top_groups=13, local_tokens=64)
    _rows_check(wl, 1)


def _fwd(wl, V, x):
    O = torch.empty_like(x["Q"])
    lse = torch.empty(wl.n_q, wl.n_q_heads, device="cuda")
    hga.attend_rows_fwd(x["hc"], x["Q"], x["K"], V, wl.q_begin, x["sg"], x["ns"], O, lse)
    torch.cuda.synchronize()
    return O, lse


@pytest.mark.parametrize("n_q", [12, 130, 600])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_rows_not_attending_a_non_finite_value_keep_their_result(n_q, bad):
    """An infinity or a NaN in the V row of a token of the call itself (later
    rows attend it, earlier rows of its group do not) and of a token that
    some rows select."""
    wl = replace(synth.WORKLOADS["qwen3_8b_2k"], q_begin=1410, n_q=n_q)
    hc = P.hcfg_of(wl)
    end = wl.q_begin + n_q
    x = {"hc": hc, "K": P.to_dev(synth.keys(wl, 0, end)), "Q": P.to_dev(synth.queries(wl, wl.q_begin, end))}
    V = P.to_dev(synth.values(wl, 0, end))
    cs, gs = hga.alloc_summaries(hc, -(-end // 64) * 64)
    hga.build_summaries(hc, x["K"], 0, end, cs, gs)
    sc, x["sg"], x["ns"] = hga.alloc_route_rows(hc, n_q)
    hga.route_rows(hc, x["Q"], wl.q_begin, cs, gs, sc, x["sg"], x["ns"])
    O, lse = _fwd(wl, V, x)
    G, g = wl.n_q_heads // wl.n_kv_heads, wl.group_size
    own = wl.q_begin + 6                                   # position of row 6
    sel = int(x["sg"][3, 0, 0])                            # a group that row 3 selects for kv head 0
    V2 = V.clone()
    V2[own, :, 1] = bad
    V2[sel * g + 1, 0, 5] = bad
    O2, lse2 = _fwd(wl, V2, x)
    rows = torch.arange(n_q, device="cuda")
    blk = (wl.q_begin + rows) // 64 * 64 + 64
    sees_own = ((rows >= 6) & (own >= blk - wl.local_tokens))[:, None] | (x["sg"] == own // g).any(-1)
    sees_sel = (x["sg"] == sel).any(-1)
    sees_sel[:, 1:] = False
    assert (sel + 1) * g <= wl.q_begin - 127               # outside every row's windows
    clean = ~(sees_own | sees_sel)
    assert clean[:6].any() and sees_sel[:6, 0].any() and (n_q < 100 or clean[100:].any())
    o, o2 = (t.float().view(n_q, wl.n_kv_heads, G, -1) for t in (O, O2))
    assert torch.isfinite(o2[clean]).all()
    assert (o - o2)[clean].abs().max() <= 2 ** -8 * o[clean].abs().max()
    assert not torch.isfinite(o2[..., 1][sees_own]).any()
    assert not torch.isfinite(o2[..., 5][sees_sel]).any()
    assert (lse - lse2).abs().max() <= 1e-5


# dQ: four waves per row up to 512 pairs, four per group, a wave per group
@pytest.mark.parametrize("n_q,q_begin", [(3, 1665), (66, 1537), (515, 1501)])
@pytest.mark.parametrize("G,d", [(1, 64), (2, 64), (4, 128), (8, 64)])
def test_rows_backward_forms(G, d, n_q, q_begin):
    wl = synth.Workload("rows_bwd_forms", T=2048, n_q_heads=8 * G, n_kv_heads=8, head_dim=d, dtype="bf16", seed=33,
                        q_begin=q_begin, n_q=n_q, grad_begin=q_begin // 64 * 64 - 64, key_offset="normal",
                        top_groups=13, local_tokens=64)
    _rows_bwd_check(wl, repeat=True)


@pytest.mark.parametrize("n_q", [12, 130, 600])
def test_rows_dq_of_rows_not_attending_a_non_finite_key(n_q):
    """An infinity in the K row of a token of the call and of a token that
    some rows select: dQ of the rows that attend neither stays what it is,
    with D from the bf16 O and from the float32 O."""
    wl = replace(synth.WORKLOADS["qwen3_8b_2k"], q_begin=1410, n_q=n_q, grad_begin=1408)
    hc, end = P.hcfg_of(wl), 1410 + n_q
    K, V = P.to_dev(synth.keys(wl, 0, end)), P.to_dev(synth.values(wl, 0, end))
    Q, dO = P.to_dev(synth.queries(wl, 1410, end)), P.to_dev(synth.grad_output(wl, 1410, end))
    cs, gs = hga.alloc_summaries(hc, -(-end // 64) * 64)
    hga.build_summaries(hc, K, 0, end, cs, gs)
    sc, sg, ns = hga.alloc_route_rows(hc, n_q)
    hga.route_rows(hc, Q, 1410, cs, gs, sc, sg, ns)
    O, lse = torch.empty_like(Q), torch.empty(n_q, wl.n_q_heads, device="cuda")
    o32 = torch.empty(n_q, wl.n_q_heads, wl.head_dim, device="cuda")
    hga.attend_rows_fwd(hc, Q, K, V, 1410, sg, ns, O, lse, o32)
    ws = torch.empty(hga.rows_workspace_size(hc, n_q), dtype=torch.uint8, device="cuda")

    def dq(k, o):
        out = torch.empty(n_q, wl.n_kv_heads, wl.n_q_heads // wl.n_kv_heads, wl.head_dim, device="cuda")
        dk = torch.empty(end - 1408, wl.n_kv_heads, wl.head_dim, device="cuda")
        hga.attend_rows_bwd(hc, Q, k, V, O, dO, lse, 1410, 1408, sg, ns, out, dk, torch.empty_like(dk), ws, o)
        torch.cuda.synchronize()
        return out

    g, own, sel = wl.group_size, 1416, int(sg[3, 0, 0])
    bad = K.clone()
    bad[own, :, 1] = float("inf")
    bad[sel * g + 1, 0, 5] = float("inf")
    rows = torch.arange(n_q, device="cuda")
    blk = (1410 + rows) // 64 * 64 + 64
    sees = ((rows >= 6) & (own >= blk - wl.local_tokens))[:, None] | (sg == own // g).any(-1)
    sees[:, 0] |= (sg[:, 0] == sel).any(-1)
    clean = ~sees
    assert clean[:6].any() and sees[:6, 0].any()
    for o in (o32, None):
        x, y = dq(K, o), dq(bad, o)
        assert (x - y)[clean].abs().max() <= 1e-5 * x[clean].abs().max()
        assert not torch.isfinite(y[sees].sum(-1)).any()
    assert (dq(K, None) - dq(K, o32)).abs().max() <= 2e-2


# three of the forms, by rows: four waves per row, four per group, a wave per group
@pytest.mark.parametrize("tails", [False, True])
@pytest.mark.parametrize("n_q", [20, 90, 600])
def test_rows_float32_output_keeps_the_weights(n_q, tails):
    """The float32 copy of O against float64 on the same routing: P enters P.V
    as a bf16 hi + lo pair, so no weight is off by more than 2^-17 (7.6e-6);
    the scores' float32 sums add about 1e-6. A P rounded to bf16 gives 1.2e-3
    and more. The LSE: half a unit of its own rounding, and the sums'."""
    wl = synth.Workload("rows_o32", T=2048, n_q_heads=32, n_kv_heads=8, head_dim=128, dtype="bf16", seed=35,
                        q_begin=1400, n_q=n_q, grad_begin=0, key_offset="student_t" if tails else "normal")
    hc, end = P.hcfg_of(wl), wl.q_begin + n_q
    K, V, Q = (P.to_dev(x) for x in (synth.keys(wl, 0, end), synth.values(wl, 0, end),
                                     synth.queries(wl, wl.q_begin, end)))
    cs, gs = hga.alloc_summaries(hc, -(-end // 64) * 64)
    hga.build_summaries(hc, K, 0, end, cs, gs)
    sc, sg, ns = hga.alloc_route_rows(hc, n_q)
    hga.route_rows(hc, Q, wl.q_begin, cs, gs, sc, sg, ns)
    O, lse = torch.empty_like(Q), torch.empty(n_q, 32, device="cuda")
    o32 = torch.empty(n_q, 32, 128, device="cuda")
    hga.attend_rows_fwd(hc, Q, K, V, wl.q_begin, sg, ns, O, lse, o32)
    # every row's set as a mask over the context, in float64
    pos = wl.q_begin + torch.arange(n_q, device="cuda")
    tok = torch.arange(end, device="cuda")
    ls = pos // 64 * 64 + 64 - wl.local_tokens
    see = ((tok < wl.sink_tokens) | (tok >= ls[:, None]))[:, None].repeat(1, 8, 1)
    see |= (tok[None, None, :, None] // wl.group_size == sg[:, :, None, :]).any(-1)
    see &= (tok <= pos[:, None])[:, None]
    worst = 0.0
    for h in range(8):
        q = Q[:, 4 * h:4 * h + 4].double()
        s = torch.matmul(q, K[:, h].double().T) / 128 ** 0.5
        s.masked_fill_(~see[:, h][:, None], -float("inf"))
        want = torch.matmul(torch.softmax(s, -1), V[:, h].double())
        worst = max(worst, float((o32[:, 4 * h:4 * h + 4] - want).norm() / want.norm()))
        assert (lse[:, 4 * h:4 * h + 4] - torch.logsumexp(s, -1)).abs().max() <= 3e-6
    assert worst <= 1e-5


@pytest.mark.parametrize("n_q,q_begin", [(1, 1787), (33, 1503)])
@pytest.mark.parametrize("G,d", [(1, 128), (4, 64), (4, 128), (8, 128)])
def test_rows_long_lists(G, d, n_q, q_begin):
    """More than 16 steps of 32 keys a row, few rows: twelve waves per row, and
    eight for dQ up to 256 pairs; with 264 pairs four."""
    wl = synth.Workload("rows_long", T=2048, n_q_heads=8 * G, n_kv_heads=8, head_dim=d, dtype="bf16", seed=37,
                        q_begin=q_begin, n_q=n_q, grad_begin=q_begin // 64 * 64 - 64, key_offset="normal",
                        group_size=16, top_chunks=16, top_groups=64, local_tokens=64)
    _rows_bwd_check(wl, repeat=True)
