"""Column pass of block lengths other than 32 on the kernels for 32 query rows: one block and two, rows that are not there, groups that just
fit and such that do not, a single block with many rows of the grid, both normalisations, either side of the block, strided queries, and the
same inside a cache-update step.  Tolerance as in tests/test_gpu_score_heads.py: sums of at most 512 fp32 weights."""
import math

import pytest
import torch

from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests.test_gpu_parity import _run_block

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("mode", [B.SDLLM_LOGIT_MEAN, B.SDLLM_SOFTMAX_MEAN])
# The last two have more than eight heads or blocks to a KV head.
@pytest.mark.parametrize("batch,q_heads,kv_heads,block,L,off", [
    (1, 4, 2, 1, 97, 40), (2, 6, 2, 8, 300, 100), (1, 14, 2, 16, 700, 333), (1, 8, 1, 31, 230, 0), (16, 4, 4, 24, 200, 77),
    (1, 2, 2, 33, 133, 50), (2, 4, 4, 40, 500, 460), (1, 8, 2, 48, 1700, 801), (3, 6, 2, 63, 400, 31), (1, 2, 2, 64, 96, 32),
    (2, 32, 32, 64, 300, 100), (1, 4, 1, 64, 2090, 700), (30, 8, 2, 64, 333, 90), (1, 5, 1, 64, 300, 64), (1, 9, 1, 16, 300, 64),
])
def test_scores(batch, q_heads, kv_heads, block, L, off, mode):
    print(f"[case] score blocks B={batch} {q_heads}/{kv_heads} b={block} L={L} off={off} mode={mode}", flush=True)
    torch.manual_seed(L + block)
    q = (2.0 * torch.randn(batch, block, q_heads, 128, device=DEV)).bfloat16().permute(0, 2, 1, 3)   # [B, rows, H, d] storage
    k = torch.randn(batch, kv_heads, L, 128, device=DEV).bfloat16()
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=off, block_len=block,
                         dtype=B.SDLLM_BF16, score_mode=mode, q_stride=B.strides_of(q))
    on_blocks = q_heads // kv_heads * -(-block // 32) <= 8 and (mode == B.SDLLM_SOFTMAX_MEAN or block % 32 == 0)
    assert B.sdllm_column_kernel(shape) == (B.SDLLM_COLUMNS_BLOCKS if on_blocks else B.SDLLM_COLUMNS_GENERAL)
    idx = torch.zeros(batch, kv_heads, B.sdllm_retained_count(shape)[0], dtype=torch.int32, device=DEV)
    pooled, score = (torch.full((batch, kv_heads, L - block), float("nan"), device=DEV) for _ in range(2))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SCORE_SELECT), dtype=torch.uint8, device=DEV)
    B.sdllm_score_select(shape, q, k, idx, pooled, score, ws)
    torch.cuda.synchronize()
    keys = torch.cat([k[:, :, :off], k[:, :, off + block:]], 2).double()
    group = q_heads // kv_heads
    for g in range(kv_heads):
        a = q[:, g * group:(g + 1) * group].double().flatten(1, 2) @ keys[:, g].transpose(1, 2).contiguous() / math.sqrt(128)
        ref = (torch.softmax(a, -1) if mode == B.SDLLM_SOFTMAX_MEAN else a).mean(1)
        err = (score[:, g].double() - ref).norm() / ref.norm()
        assert err < 1e-5, f"head {g}: relative error {err:.2e}"


@pytest.mark.parametrize("q_heads,kv_heads,block,batch,prompt,modes", [
    (8, 2, 64, 2, 500, {}), (6, 2, 48, 1, 333, {}), (14, 2, 16, 1, 700, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),
    (4, 4, 64, 1, 1000, dict(score_mode=B.SDLLM_LOGIT_MEAN)),
])
def test_cache_update_step(q_heads, kv_heads, block, batch, prompt, modes):
    import dataclasses
    w = wl.WORKLOADS["dream7b_gqa"].scaled(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, prompt=prompt, gen=4 * block)
    w = dataclasses.replace(w, block=block)
    _run_block(w, block_index=1, n_steps=3, **modes)


@pytest.mark.parametrize("mode", [B.SDLLM_LOGIT_MEAN, B.SDLLM_SOFTMAX_MEAN])
@pytest.mark.parametrize("batch,q_heads,kv_heads,block", [(1, 3, 1, 40), (2, 7, 1, 20), (64, 1, 1, 5), (1, 2, 1, 64)])
def test_infinitely_low_keys(batch, q_heads, kv_heads, block, mode):
    # such keys weigh nothing (softmax) or -inf (logits), a whole tile of them as well, and the others keep their scores
    print(f"[case] score blocks, -inf keys B={batch} {q_heads}/{kv_heads} b={block} mode={mode}", flush=True)
    torch.manual_seed(block)
    L, off = 300, 131
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=off, block_len=block,
                         dtype=B.SDLLM_BF16, score_mode=mode)
    if mode == B.SDLLM_SOFTMAX_MEAN or block % 32 == 0:
        assert B.sdllm_column_kernel(shape) == B.SDLLM_COLUMNS_BLOCKS
    q = torch.randn(batch, q_heads, block, 128, device=DEV).bfloat16()
    k = torch.randn(batch, 1, L, 128, device=DEV).bfloat16()
    low = [*range(32, 64), 100, L - 1]
    q[..., 0] = q[..., 0].abs() + 0.25
    k[:, :, low, 0] = float("-inf")
    idx = torch.zeros(batch, 1, B.sdllm_retained_count(shape)[0], dtype=torch.int32, device=DEV)
    pooled, score = (torch.full((batch, 1, L - block), float("nan"), device=DEV) for _ in range(2))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SCORE_SELECT), dtype=torch.uint8, device=DEV)
    B.sdllm_score_select(shape, q, k, idx, pooled, score, ws)
    torch.cuda.synchronize()
    low[-1] -= block                                           # as candidates
    kept = [c for c in range(L - block) if c not in low]
    assert (score[:, 0, low] == (0.0 if mode == B.SDLLM_SOFTMAX_MEAN else float("-inf"))).all()
    keys = torch.cat([k[:, 0, :off], k[:, 0, off + block:]], 1)[:, kept].double()
    a = q.double().flatten(1, 2) @ keys.transpose(1, 2).contiguous() / math.sqrt(128)
    ref = (torch.softmax(a, -1) if mode == B.SDLLM_SOFTMAX_MEAN else a).mean(1)
    err = (score[:, 0, kept].double() - ref).norm() / ref.norm()
    assert err < 1e-5, f"relative error {err:.2e}"
