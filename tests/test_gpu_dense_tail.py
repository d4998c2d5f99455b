"""Full-sequence attention whose last, small round of workgroups runs as a launch of its own with two or four key groups: either, with one
workgroup left and as many as there may be, with as few tiles as it takes and one fewer, a last block of rows that fills one of its four parts or
a few rows of one, grouped-query heads and tensors in [B, rows, H, d] storage.  Tolerances: tests/parity_util.py."""
import math

import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


# groups: key groups of the main launch, of the last one (0: none)
@pytest.mark.parametrize("batch,q_heads,kv_heads,L,groups", [
    (1, 257, 257, 225, (1, 0)), (1, 129, 129, 290, (2, 0)), (5, 20, 4, 577, (2, 0)), (1, 107, 107, 712, (1, 0)), (4, 32, 8, 641, (1, 0)), (1, 56, 8, 1152, (2, 0)),
    (1, 171, 57, 647, (1, 4)), (1, 257, 257, 257, (1, 4)), (1, 288, 32, 270, (1, 4)), (5, 20, 4, 768, (1, 4)), (1, 160, 32, 512, (1, 4)), (1, 205, 41, 1100, (1, 4)),
    (1, 107, 107, 738, (1, 2)), (1, 128, 16, 738, (1, 2)), (3, 28, 4, 900, (1, 2)), (3, 28, 4, 769, (1, 2)), (1, 48, 8, 1602, (1, 2)),
    (2, 28, 4, 1200, (1, 4)), (1, 56, 8, 1153, (1, 4)),                                     # where two throughout were the choice without it
])
def test_last_round(batch, q_heads, kv_heads, L, groups):
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
        assert (B.sdllm_launch_plan(shape, B.SDLLM_CALL_DENSE).key_groups, B.sdllm_dense_tail_groups(shape)) == groups
        B.sdllm_dense_attn(shape, q, k, v, out)
        torch.cuda.synchronize()
        group = q_heads // kv_heads
        for b in range(batch):
            for h in range(0, q_heads, 1 if q_heads < 64 else 7):
                a = (q[b, h].float() @ k[b, h // group].float().T) / math.sqrt(128)
                ref = (torch.softmax(a, -1) @ v[b, h // group].float()).double().cpu().numpy()
                U.assert_close(out[b, h], ref, "bf16", f"b={b} h={h} L={L}")
        assert not out.isnan().any()
