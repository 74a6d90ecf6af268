"""The backward's dK/dV partition by the library's choice: calls with few heads
or rows and little history split over one, two, four or eight query-head
subsets, against the oracle and against the unsplit call."""

import pytest
import torch

from paper_2607_15105_amd import hga, synth
from tests import parity as P
from tests.test_gpu_parity import _full_check

pytestmark = pytest.mark.gpu


def _wl(G, n_kv, n_q, q_begin, d, dtype):
    return synth.Workload("bwd_parts", T=q_begin + n_q, n_q_heads=G * n_kv, n_kv_heads=n_kv, head_dim=d, dtype=dtype,
                          seed=51, q_begin=q_begin, n_q=n_q, grad_begin=q_begin, key_offset="normal")


def _parts(wl):
    ws = hga.workspace_size(P.hcfg_of(wl), hga.OP_BWD, wl.q_begin, wl.n_q, wl.grad_begin)
    dvec = -(-wl.n_q * wl.n_q_heads * 4 // 256) * 256
    rows = wl.q_begin + wl.n_q - wl.grad_begin
    return (ws - dvec) // (2 * rows * wl.n_kv_heads * wl.head_dim * 4) or 1


@pytest.mark.parametrize("G,n_kv,n_q,q_begin,d,dtype,parts", [
    (4, 2, 512, 0, 64, "fp32", 4),
    (8, 1, 512, 0, 64, "bf16", 8),
    (8, 2, 1024, 0, 128, "bf16", 8),    # 256 + 64 workgroups, chains of 32 steps and more
    (4, 2, 2048, 0, 64, "bf16", 4),     # 256 + 64 as well
    (4, 8, 512, 0, 64, "bf16", 2),      # as many, but chains of 16 steps
    (2, 2, 256, 128, 128, "bf16", 2),
    (1, 4, 256, 0, 64, "bf16", 1),
    (4, 2, 256, 4096, 64, "bf16", 1),   # history
    (4, 8, 256, 0, 128, "bf16", 2),     # dQ is as long as the chains
    (4, 4, 1024, 2048, 128, "bf16", 2),  # the sink chunk is not active: short chains, 320 workgroups
    (8, 1, 1024, 512, 64, "bf16", 8),   # nor here, but every block picks the few candidates
])
def test_library_choice(G, n_kv, n_q, q_begin, d, dtype, parts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = _wl(G, n_kv, n_q, q_begin, d, dtype)
    assert _parts(wl) == parts
    _full_check(wl, backward=True)


def test_a_buffer_sized_for_a_longer_call_takes_a_shorter_one():
    """8/1 heads from token 0: 2,048 rows split into eight subsets and 4,032
    rows into two, in half the bytes. In the longer call's buffer the shorter
    call splits into two, as where the caller asks for two."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = _wl(8, 1, 2048, 0, 64, "bf16")
    hc = P.hcfg_of(wl)
    two = hga.make_config(8, 1, 64, group_size=wl.group_size, top_chunks=wl.top_chunks, top_groups=wl.top_groups,
                          sink_tokens=wl.sink_tokens, local_tokens=wl.local_tokens, bwd_kv_parts=2)
    small, full = (hga.workspace_size(hc, hga.OP_BWD, 0, n, 0) for n in (4032, 2048))
    assert hga.workspace_size(two, hga.OP_BWD, 0, 2048, 0) < small < full
    K, V, Q, dO = (P.to_dev(f(wl, 0, 2048)) for f in (synth.keys, synth.values, synth.queries, synth.grad_output))
    cs, gs = hga.alloc_summaries(hc, 2048)
    rb = hga.alloc_route(hc, 0, 2048)
    O, lse = torch.empty_like(Q), torch.empty(2048, 8, device="cuda")
    hga.build_summaries(hc, K, 0, 2048, cs, gs)
    hga.route_attend_fwd(hc, Q, K, V, 0, cs, gs, rb.sel_chunks, rb.sel_groups, rb.n_sel_groups, O, lse, rb.workspace)

    def grads(cfg, size):
        ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        out = [torch.empty(2048, h, 64, device="cuda") for h in (8, 1, 1)]
        hga.attend_bwd(cfg, Q, K, V, O, dO, lse, 0, 0, rb.sel_groups, rb.n_sel_groups, *out, ws[:size])
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xFF).all())  # nothing past the buffer's end
        return out

    a, b, c = grads(hc, small), grads(two, small), grads(hc, full)
    for x, y, z in zip(a, b, c):
        assert torch.equal(x, y)
        # sums of the same terms in another order: 84 units of float32 rounding
        assert (x - z).abs().max() <= 1e-5 * z.abs().max()
