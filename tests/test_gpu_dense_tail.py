"""Full-sequence attention whose last, small round of workgroups runs as a launch of its own with two or four key groups: either, one
workgroup left and as many as there may be, a last block of rows that fills one of its four parts or a few rows of one, grouped-query heads and
tensors in [B, rows, H, d] storage.  Tolerances: tests/parity_util.py."""
import math

import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("batch,q_heads,kv_heads,L", [
    (1, 257, 257, 289 - 64),                               # one group of rows a head, up to 256 positions: no second launch
    (1, 129, 129, 290), (5, 20, 4, 530), (5, 20, 4, 577), (5, 20, 4, 768), (1, 86, 43, 600), (2, 53, 53, 1090),      # four groups
    (3, 28, 4, 900), (3, 28, 4, 769), (4, 32, 8, 641), (1, 48, 8, 1602), (2, 28, 4, 1200),                           # two, and where two were the choice
])
def test_last_round(batch, q_heads, kv_heads, L):
    print(f"[case] dense tail B={batch} {q_heads}/{kv_heads} L={L}", flush=True)
    torch.manual_seed(L + q_heads)
    for strided in (False, True):
        make = lambda h: torch.randn((batch, L, h, 128) if strided else (batch, h, L, 128), device=DEV).bfloat16()
        q, k, v, out = (make(h) for h in (q_heads, kv_heads, kv_heads, q_heads))
        out.fill_(float("nan"))
        if strided:
            q, k, v, out = (x.permute(0, 2, 1, 3) for x in (q, k, v, out))
        shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=0, block_len=32,
                             dtype=B.SDLLM_BF16, kv_stride=B.strides_of(k))
        B.sdllm_dense_attn(shape, q, k, v, out)
        torch.cuda.synchronize()
        group = q_heads // kv_heads
        for b in range(batch):
            for h in range(0, q_heads, 1 if q_heads < 64 else 7):
                a = (q[b, h].float() @ k[b, h // group].float().T) / math.sqrt(128)
                ref = (torch.softmax(a, -1) @ v[b, h // group].float()).double().cpu().numpy()
                U.assert_close(out[b, h], ref, "bf16", f"b={b} h={h} L={L}")
        assert not out.isnan().any()
