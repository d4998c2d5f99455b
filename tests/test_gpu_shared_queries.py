"""Query rows that reach a workgroup's waves through LDS: one to eight waves (which share eight requests out), waves and splits
without a tile, workgroups that have LDS of their own for the rows and such that lend a tile's, and rows, heads and batches in
any order in memory, among them rows further apart than 32 bits of bytes reach.  Tolerances: tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _call(batch, q_heads, kv_heads, n_cached, q):
    head_dim, block = 128, 32
    kc, vc = (torch.randn(batch, kv_heads, max(1, n_cached), head_dim, device=DEV).bfloat16() for _ in range(2))
    kb, vb = (torch.randn(batch, kv_heads, block, head_dim, device=DEV).bfloat16() for _ in range(2))
    out = torch.full((batch, q_heads, block, head_dim), float("nan"), device=DEV, dtype=torch.bfloat16)
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=head_dim, seq_len=16384, block_off=8192, block_len=block,
                         dtype=B.SDLLM_BF16, cache_rows=max(1, n_cached), q_stride=B.strides_of(q))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q, torch.cat([kc[:, :, :n_cached], kb], 2), torch.cat([vc[:, :, :n_cached], vb], 2))
    U.assert_close(out, ref, "bf16", f"B={batch} {q_heads}/{kv_heads} n_cached={n_cached}")


@pytest.mark.parametrize("batch,q_heads,kv_heads,n_cached", [
    (1, 7, 1, 0), (1, 7, 1, 40), (1, 14, 2, 100), (2, 28, 4, 300), (8, 28, 4, 1700),      # tiles fetched into LDS, 1 to 8 waves
    (1, 28, 4, 1100), (1, 4, 4, 1000), (1, 8, 8, 8000), (3, 32, 32, 900),               # key splits, the last one shorter
    (12, 28, 4, 250), (20, 28, 4, 100), (18, 32, 8, 70), (20, 30, 10, 33),               # two and four workgroups to a CU
    (9, 30, 10, 20), (5, 32, 32, 20),                                                    # fewer tiles than waves
])
def test_queries_in_any_layout(batch, q_heads, kv_heads, n_cached):
    print(f"[case] shared queries B={batch} {q_heads}/{kv_heads} n_cached={n_cached}", flush=True)
    torch.manual_seed(n_cached + q_heads)
    q = 2.0 * torch.randn(batch, 32, q_heads, 128, device=DEV).bfloat16()
    _call(batch, q_heads, kv_heads, n_cached, q.permute(0, 2, 1, 3))                      # [B, rows, H, d] storage
    _call(batch, q_heads, kv_heads, n_cached, q.permute(0, 2, 1, 3).contiguous())


def test_query_rows_far_apart():
    # rows 144 MB apart: 29 rows on, the offset is beyond 2^32 bytes
    print("[case] shared queries, far rows", flush=True)
    torch.manual_seed(5)
    q = torch.zeros(32, 72 * 1024 * 1024, device=DEV, dtype=torch.bfloat16)[:, :7 * 128].unflatten(1, (7, 128))
    q.copy_(2.0 * torch.randn(32, 7, 128, device=DEV))
    for n_cached in (300, 1500):
        _call(1, 7, 1, n_cached, q.permute(1, 0, 2)[None])
