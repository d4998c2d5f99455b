"""Key splits of a head merged by a launch of their own: counts on either side of what one thread folds at once (4, 8, 12, 16, 24, 32) and
more, heads of several batch elements, and output rows in any layout.  Tolerances: tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("batch,q_heads,kv_heads,n_cached,splits", [
    (4, 28, 4, 1520, 2), (1, 28, 4, 300, 3), (3, 4, 2, 560, 4), (1, 28, 4, 740, 5), (1, 4, 4, 700, 8), (3, 4, 2, 700, 6), (1, 8, 2, 1100, 8),
    (2, 4, 2, 1200, 8), (1, 28, 4, 2159, 8), (1, 28, 4, 2280, 9), (1, 6, 3, 1500, 12), (1, 3, 3, 2100, 12), (2, 2, 1, 2600, 12), (1, 16, 2, 3560, 13),
    (1, 8, 8, 4000, 16), (3, 4, 2, 4840, 17), (2, 2, 1, 4400, 24), (2, 4, 2, 7140, 25), (2, 28, 4, 19200, 32), (1, 16, 2, 29000, 8), (1, 28, 4, 38500, 64),
])
def test_merge_of_key_splits(batch, q_heads, kv_heads, n_cached, splits):
    print(f"[case] merge B={batch} {q_heads}/{kv_heads} n_cached={n_cached}", flush=True)
    torch.manual_seed(n_cached + q_heads)
    d, b = 128, 32
    q = (2.0 * torch.randn(batch, q_heads, b, d, device=DEV)).bfloat16()
    kc, vc = (torch.randn(batch, kv_heads, n_cached, d, device=DEV).bfloat16() for _ in range(2))
    kb, vb = (torch.randn(batch, kv_heads, b, d, device=DEV).bfloat16() for _ in range(2))
    ref = U.oracle_attention_batch(q, torch.cat([kc, kb], 2), torch.cat([vc, vb], 2))
    for out in (torch.full((batch, q_heads, b, d), float("nan"), device=DEV, dtype=torch.bfloat16),
                torch.full((batch, b, q_heads, d + 8), float("nan"), device=DEV, dtype=torch.bfloat16)[..., :d].permute(0, 2, 1, 3)):
        shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=d, seq_len=65536, block_off=8192, block_len=b,
                             dtype=B.SDLLM_BF16, cache_rows=n_cached, out_stride=B.strides_of(out))
        assert (B.sdllm_burst_splits(shape, B.SDLLM_CALL_SPARSE, n_cached) or B.sdllm_launch_plan(shape, B.SDLLM_CALL_SPARSE, n_cached).key_splits) == splits
        ws = torch.full((B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached),), 0xff, dtype=torch.uint8, device=DEV)
        B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
        torch.cuda.synchronize()
        U.assert_close(out, ref, "bf16", f"B={batch} {q_heads}/{kv_heads} n_cached={n_cached}")
