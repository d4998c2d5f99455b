"""The attention kernel that fetches tiles straight into LDS, at the sizes where its pipeline and its launch rule can go
wrong: waves with two or three tiles and with many, a ragged last tile of either key segment, key splits, more heads than CUs,
and the scoring statistics when the block's own keys share tiles with candidates.  Sparse steps of fewer than ten tiles run another kernel
(tests/test_gpu_burst.py), as do some of ten and more that bring a workspace.  Tolerances: tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests import parity_util as U
from tests.test_gpu_general import _hide
from tests.test_gpu_parity import _run_block

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _workspace(shape, n_cached):
    """What the call asks for, or none where the kernel for small calls would then take it."""
    splits = B.sdllm_burst_splits(shape, B.SDLLM_CALL_SPARSE, n_cached)
    assert splits != 1                                      # a call that it takes without a workspace
    return None if splits else torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("batch,q_heads,kv_heads,n_cached,waves,touches", [
    (1, 28, 4, 257, 5, 0), (1, 28, 4, 288, 5, 0), (2, 28, 4, 300, 5, 0), (2, 28, 4, 500, 6, 0), (3, 16, 2, 479, 5, 0), (9, 16, 2, 1500, 6, 0),
    (1, 7, 1, 289, 5, 0), (1, 14, 2, 512, 6, 0), (3, 6, 2, 671, 6, 0),                              # without a workspace
    (1, 32, 32, 270, 5, 0), (3, 8, 8, 281, 5, 0), (4, 8, 8, 400, 5, 0),                             # multi-head calls small enough to go unsplit
    (8, 28, 4, 1633, 8, 0), (5, 28, 4, 2111, 8, 0),         # one workgroup per head, eight waves
    (10, 28, 4, 1185, 4, 0),                                # more heads than CUs: four waves
    # heads bring tiles into L2 for each other; ragged last tiles in both segments, waves with a tile less than others
    (8, 28, 4, 3301, 8, 1), (6, 28, 4, 3107, 8, 1), (9, 16, 2, 3333, 8, 1), (10, 28, 4, 1733, 4, 1), (17, 16, 2, 1543, 4, 1),
])
def test_stream_sparse_attn(batch, q_heads, kv_heads, n_cached, waves, touches):
    print(f"[case] stream sparse_attn B={batch} {q_heads}/{kv_heads} n_cached={n_cached}", flush=True)
    torch.manual_seed(n_cached + batch)
    b, d, rows = 32, 128, max(1, n_cached)
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=d, seq_len=16384, block_off=8192,
                         block_len=b, dtype=B.SDLLM_BF16, cache_rows=rows)
    plan = B.sdllm_launch_plan(shape, B.SDLLM_CALL_SPARSE, n_cached)
    assert (plan.kernel, plan.key_splits, plan.waves, plan.touches_ahead) == (B.SDLLM_KERNEL_STREAM, 1, waves, touches)
    q = (2.0 * torch.randn(batch, q_heads, b, d, device=DEV)).bfloat16()
    kc, vc = (torch.randn(batch, kv_heads, rows, d, device=DEV).bfloat16() for _ in range(2))
    kb, vb = (torch.randn(batch, kv_heads, b, d, device=DEV).bfloat16() for _ in range(2))
    out = torch.full_like(q, float("nan"))
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, _workspace(shape, n_cached))
    torch.cuda.synchronize()
    k_all = torch.cat([kc[:, :, :n_cached], kb], 2)
    v_all = torch.cat([vc[:, :, :n_cached], vb], 2)
    U.assert_close(out, U.oracle_attention_batch(q, k_all, v_all), "bf16", f"n_cached={n_cached}")


@pytest.mark.parametrize("q_heads,kv_heads,batch,prompt,splits,touches,modes", [
    (14, 2, 1, 233, 1, 0, {}),                                             # block off the tile grid on both sides
    (7, 1, 2, 64, 1, 0, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),      # few candidate tiles, long mixed tail
    (28, 4, 2, 3111, 4, 0, {}),                                            # statistics from key splits
    (28, 4, 2, 12433, 4, 1, {}),                                           # ... whose heads bring tiles into L2 for each other
    (14, 2, 1, 0, 1, 0, {}),                                               # no prefix
    (28, 4, 12, 1171, 1, 0, {}),                                           # more heads than CUs
    (28, 4, 22, 1109, 1, 0, {}),                                           # more than two four-wave workgroups per CU
])
def test_stream_statistics_at_the_cache_update_step(q_heads, kv_heads, batch, prompt, splits, touches, modes):
    w = wl.WORKLOADS["dream7b_gqa"].scaled(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, prompt=prompt, gen=160)
    plan = B.sdllm_launch_plan(U.shape_for(w, 2, **modes), B.SDLLM_CALL_UPDATE)
    assert (plan.kernel, plan.key_splits, plan.touches_ahead) == (B.SDLLM_KERNEL_STREAM, splits, touches)
    _run_block(w, block_index=2, n_steps=3, **modes)


@pytest.mark.parametrize("batch,q_heads,kv_heads,n_cached", [(1, 7, 1, 300), (1, 7, 1, 600), (2, 28, 4, 290), (1, 32, 32, 270), (10, 28, 4, 1200)])
def test_tiles_of_infinitely_low_keys(batch, q_heads, kv_heads, n_cached):
    # whole tiles without weight, among them the first of a wave
    print(f"[case] stream, -inf tiles B={batch} {q_heads}/{kv_heads} n_cached={n_cached}", flush=True)
    torch.manual_seed(n_cached)
    q = torch.randn(batch, q_heads, 32, 128, device=DEV).bfloat16()
    kc, vc, kb, vb = (torch.randn(batch, kv_heads, n, 128, device=DEV).bfloat16() for n in (n_cached, n_cached, 32, 32))
    kept = _hide(kc, q, [*range(32, 64), *range(96, 128)])
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=4096, block_off=2048, block_len=32,
                         dtype=B.SDLLM_BF16, cache_rows=n_cached)
    assert B.sdllm_launch_plan(shape, B.SDLLM_CALL_SPARSE, n_cached).kernel == B.SDLLM_KERNEL_STREAM
    out = torch.zeros_like(q)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, _workspace(shape, n_cached))
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, torch.cat([kc[:, :, kept], kb], 2), torch.cat([vc[:, :, kept], vb], 2)), "bf16", "kept keys")
