"""Full-sequence attention with the keys of a head shared out between two or four groups of a workgroup's waves: sequence
lengths around the stage (two or four tiles) and row-block edges, groups without a tile, and a grid that takes each
variant.  Tolerances: tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U
from tests.test_gpu_general import _hide

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("batch,q_heads,kv_heads,L,groups", [
    # tile counts that leave 0, 1, 2 and 3 groups of the last stage without a tile, a last tile of one key
    (1, 2, 1, 97, 4), (1, 2, 1, 128, 4), (1, 2, 1, 161, 4), (1, 3, 1, 161, 4), (2, 4, 2, 255, 4), (1, 2, 2, 385, 4), (1, 4, 4, 1025, 4),
    (1, 2, 1, 289, 4), (1, 2, 1, 323, 4), (1, 28, 4, 513, 4),
    (2, 12, 4, 705, 2), (1, 28, 4, 735, 2), (2, 12, 4, 1057, 2), (1, 28, 4, 769, 2),
    (1, 2, 1, 129, 1), (8, 28, 4, 200, 1),                                                          # whole rows
])
def test_dense_attn_key_groups(batch, q_heads, kv_heads, L, groups):
    print(f"[case] dense_attn key groups B={batch} {q_heads}/{kv_heads} L={L}", flush=True)
    torch.manual_seed(L + q_heads)
    q, k, v = ((g * torch.randn(batch, h, L, 128, device=DEV)).bfloat16() for g, h in ((2.0, q_heads), (1.0, kv_heads), (1.0, kv_heads)))
    out = torch.full_like(q, float("nan"))
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=0, block_len=32,
                         dtype=B.SDLLM_BF16)
    assert B.sdllm_launch_plan(shape, B.SDLLM_CALL_DENSE).key_groups == groups
    B.sdllm_dense_attn(shape, q, k, v, out)
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, k, v), "bf16", f"L={L}")


@pytest.mark.parametrize("batch,q_heads,kv_heads,L", [(1, 2, 1, 300), (1, 28, 4, 735)])
def test_tiles_of_infinitely_low_keys(batch, q_heads, kv_heads, L):
    # whole tiles without weight, among them the first of a key group
    print(f"[case] dense_attn key groups, -inf tiles L={L}", flush=True)
    torch.manual_seed(L)
    q, k, v = (torch.randn(batch, h, L, 128, device=DEV).bfloat16() for h in (q_heads, kv_heads, kv_heads))
    kept = _hide(k, q, [*range(32, 64), *range(96, 128)])
    out = torch.zeros_like(q)
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=0, block_len=32,
                         dtype=B.SDLLM_BF16)
    B.sdllm_dense_attn(shape, q, k, v, out)
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, k[:, :, kept], v[:, :, kept]), "bf16", f"L={L}")
