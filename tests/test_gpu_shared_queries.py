"""Query rows that reach a workgroup's waves through LDS, in each of the three kernels that fetch them so: one to eight waves (which share
eight requests out), waves without a tile, workgroups that have LDS of their own for the rows and such that lend a tile's, and
rows, heads and batches in any order in memory, among them rows further apart than 32 bits of bytes reach.  Tolerances: tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _route(shape, n_cached):
    """Kernel and waves of a sparse step."""
    splits = B.sdllm_burst_splits(shape, B.SDLLM_CALL_SPARSE, n_cached)
    if splits:
        return "burst", max(8, -(-(-(-n_cached // 32) + 1) // splits))
    plan = B.sdllm_launch_plan(shape, B.SDLLM_CALL_SPARSE, n_cached)
    return {B.SDLLM_KERNEL_STREAM: "stream", B.SDLLM_KERNEL_PER_HEAD: "per_head"}[plan.kernel], plan.waves


def _call(batch, q_heads, kv_heads, n_cached, q, route):
    head_dim, block = 128, 32
    kc, vc = (torch.randn(batch, kv_heads, max(1, n_cached), head_dim, device=DEV).bfloat16() for _ in range(2))
    kb, vb = (torch.randn(batch, kv_heads, block, head_dim, device=DEV).bfloat16() for _ in range(2))
    out = torch.full((batch, q_heads, block, head_dim), float("nan"), device=DEV, dtype=torch.bfloat16)
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=head_dim, seq_len=16384, block_off=8192, block_len=block,
                         dtype=B.SDLLM_BF16, cache_rows=max(1, n_cached), q_stride=B.strides_of(q))
    assert _route(shape, n_cached) == route
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q, torch.cat([kc[:, :, :n_cached], kb], 2), torch.cat([vc[:, :, :n_cached], vb], 2))
    U.assert_close(out, ref, "bf16", f"B={batch} {q_heads}/{kv_heads} n_cached={n_cached}")


@pytest.mark.parametrize("batch,q_heads,kv_heads,n_cached,route", [
    (1, 7, 1, 0, ("burst", 8)), (1, 7, 1, 40, ("burst", 8)), (1, 14, 2, 100, ("burst", 8)), (1, 14, 2, 260 - 32, ("burst", 9)), (1, 28, 4, 1100, ("burst", 8)),
    (1, 4, 4, 1000, ("burst", 8)), (1, 8, 8, 8000, ("burst", 9)), (5, 32, 32, 20, ("burst", 8)),            # all tiles at once
    (2, 28, 4, 300, ("stream", 5)), (2, 28, 4, 500, ("stream", 6)), (8, 28, 4, 1700, ("stream", 8)),        # tiles fetched into LDS
    (3, 32, 32, 900, ("per_head", 8)), (2, 28, 4, 1250, ("per_head", 7)), (4, 8, 8, 3000, ("per_head", 6)),  # key splits, the last one shorter
    (12, 28, 4, 250, ("per_head", 4)), (20, 28, 4, 100, ("per_head", 2)), (18, 32, 8, 70, ("per_head", 2)), (20, 30, 10, 33, ("per_head", 2)),   # two and four workgroups to a CU
    (9, 30, 10, 0, ("per_head", 1)), (9, 30, 10, 20, ("per_head", 2)), (9, 30, 10, 64, ("per_head", 3)), (1, 32, 32, 3000, ("per_head", 6)),
])
def test_queries_in_any_layout(batch, q_heads, kv_heads, n_cached, route):
    print(f"[case] shared queries B={batch} {q_heads}/{kv_heads} n_cached={n_cached}", flush=True)
    torch.manual_seed(n_cached + q_heads)
    q = 2.0 * torch.randn(batch, 32, q_heads, 128, device=DEV).bfloat16()
    _call(batch, q_heads, kv_heads, n_cached, q.permute(0, 2, 1, 3), route)                      # [B, rows, H, d] storage
    _call(batch, q_heads, kv_heads, n_cached, q.permute(0, 2, 1, 3).contiguous(), route)


def test_query_rows_far_apart():
    # rows 144 MB apart: 29 rows on, the offset is beyond 2^32 bytes
    print("[case] shared queries, far rows", flush=True)
    torch.manual_seed(5)
    q = torch.zeros(32, 72 * 1024 * 1024, device=DEV, dtype=torch.bfloat16)[:, :28 * 128].unflatten(1, (28, 128))
    q.copy_(2.0 * torch.randn(32, 28, 128, device=DEV))
    for heads, kv_heads, n_cached, route in ((7, 1, 300, ("burst", 8)), (7, 1, 1500, ("burst", 8)), (28, 4, 285, ("stream", 5)), (28, 4, 2600, ("per_head", 6))):
        _call(1, heads, kv_heads, n_cached, q[:, :heads].permute(1, 0, 2)[None], route)
