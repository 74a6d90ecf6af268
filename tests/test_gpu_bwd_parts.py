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
])
def test_library_choice(G, n_kv, n_q, q_begin, d, dtype, parts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = _wl(G, n_kv, n_q, q_begin, d, dtype)
    assert _parts(wl) == parts
    _full_check(wl, backward=True)
