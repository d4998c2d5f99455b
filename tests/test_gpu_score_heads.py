"""Column pass of the scoring with a wave per query head: every group size, step counts from one to beyond the ring of tiles in
LDS, ragged last tiles on both sides of the block, candidates on one side only, streams without a tile of their own; and the waves that
walk the heads, which take the pass over where the rows are many.
Tolerance: a score sums at most 256 logits or weights in fp32, each from a 128-term fp32 dot product of bf16 values (error
about 2^-24 * sqrt(128 * 256) of its size, 1e-5 with a factor of five)."""
import math

import pytest
import torch

from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests.test_gpu_parity import _run_block

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _reference(q, k, group, off, softmax):
    keys = torch.cat([k[:, :, :off], k[:, :, off + 32:]], 2).double()
    out = []
    for g in range(k.shape[1]):
        a = q[:, g * group:(g + 1) * group].double().flatten(1, 2) @ keys[:, g].transpose(1, 2) / math.sqrt(128)
        out.append((torch.softmax(a, -1) if softmax else a).mean(1))
    return torch.stack(out, 1)


@pytest.mark.parametrize("batch,q_heads,kv_heads,L,off", [
    (1, 4, 2, 33, 0), (1, 4, 2, 97, 32), (2, 6, 2, 800, 415), (1, 8, 2, 1056, 1024), (1, 5, 1, 230, 31), (1, 6, 1, 2090, 700),
    (1, 7, 1, 64, 32), (1, 7, 1, 65, 1), (1, 14, 2, 4300, 2111), (8, 28, 4, 700, 333), (3, 8, 1, 3001, 0), (2, 16, 2, 7001, 6000),
    (70, 8, 4, 500, 100), (70, 28, 4, 300, 101), (103, 28, 4, 230, 64),   # more rows than CUs: a workgroup walks all tiles
    (20, 8, 4, 330, 0), (8, 24, 8, 500, 77), (6, 16, 4, 300, 90), (24, 16, 4, 1501, 1400), (48, 20, 4, 900, 31), (20, 28, 4, 1633, 800),   # waves that walk the heads
])
@pytest.mark.parametrize("mode", [B.SDLLM_LOGIT_MEAN, B.SDLLM_SOFTMAX_MEAN])
def test_scores_of_grouped_heads(batch, q_heads, kv_heads, L, off, mode):
    print(f"[case] score heads B={batch} {q_heads}/{kv_heads} L={L} off={off} mode={mode}", flush=True)
    torch.manual_seed(L + off)
    q = (2.0 * torch.randn(batch, q_heads, 32, 128, device=DEV)).bfloat16()
    k = torch.randn(batch, kv_heads, L, 128, device=DEV).bfloat16()
    _check_scores(q, k, off, mode)


def _check_scores(q, k, off, mode):
    batch, q_heads = q.shape[:2]
    kv_heads, L = k.shape[1:3]
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=off, block_len=32,
                         dtype=B.SDLLM_BF16, score_mode=mode, q_stride=B.strides_of(q), kv_stride=B.strides_of(k))
    kt = B.sdllm_retained_count(shape)[0]
    idx = torch.zeros(batch, kv_heads, kt, dtype=torch.int32, device=DEV)
    pooled, score = (torch.full((batch, kv_heads, L - 32), float("nan"), device=DEV) for _ in range(2))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SCORE_SELECT), dtype=torch.uint8, device=DEV)
    B.sdllm_score_select(shape, q, k, idx, pooled, score, ws)
    torch.cuda.synchronize()
    ref = _reference(q, k, q_heads // kv_heads, off, mode == B.SDLLM_SOFTMAX_MEAN)
    err = (score.double() - ref).norm() / ref.norm()
    assert err < 1e-5, f"relative error {err:.2e}"


# Queries and keys stored [B, rows, H, d], and query rows further apart than 32 bits of bytes reach: both kernels of the pass.
@pytest.mark.parametrize("batch,q_heads,kv_heads,L,off", [(1, 14, 2, 2300, 1111), (3, 8, 4, 777, 100), (24, 16, 4, 1501, 1400), (20, 20, 4, 1433, 8)])
@pytest.mark.parametrize("mode", [B.SDLLM_LOGIT_MEAN, B.SDLLM_SOFTMAX_MEAN])
def test_scores_of_tensors_stored_by_rows(batch, q_heads, kv_heads, L, off, mode):
    print(f"[case] score heads, stored by rows B={batch} {q_heads}/{kv_heads} L={L} off={off} mode={mode}", flush=True)
    torch.manual_seed(L)
    q = (2.0 * torch.randn(batch, 32, q_heads, 128, device=DEV)).bfloat16().permute(0, 2, 1, 3)
    k = torch.randn(batch, L, kv_heads, 128, device=DEV).bfloat16().permute(0, 2, 1, 3)
    _check_scores(q, k, off, mode)


@pytest.mark.parametrize("kv_heads,L", [(1, 1500), (10, 12900)])
def test_scores_of_query_rows_far_apart(kv_heads, L):
    # rows 144 MB apart: 29 rows on, the offset is beyond 2^32 bytes
    print(f"[case] score heads, far rows, {kv_heads} KV heads L={L}", flush=True)
    torch.manual_seed(L)
    heads = 7 * kv_heads
    q = torch.zeros(32, 72 * 1024 * 1024, device=DEV, dtype=torch.bfloat16)[:, :heads * 128].unflatten(1, (heads, 128))
    q.copy_(2.0 * torch.randn(32, heads, 128, device=DEV))
    k = torch.randn(1, kv_heads, L, 128, device=DEV).bfloat16()
    _check_scores(q.permute(1, 0, 2)[None], k, 200, B.SDLLM_LOGIT_MEAN)


# With the statistics left by the dense attention (key splits or not, one or two kernels): index sets and cache against the oracle.
@pytest.mark.parametrize("q_heads,kv_heads,batch,prompt,modes", [
    (4, 2, 1, 70, {}), (6, 2, 2, 333, {}), (8, 2, 1, 1500, {}), (10, 2, 1, 64, {}), (12, 2, 1, 701, {}), (14, 2, 1, 2600, {}),
    (16, 2, 3, 300, {}), (28, 4, 2, 900, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),
    (16, 8, 32, 200, {}), (16, 4, 24, 1400, {}), (28, 4, 24, 1300, {}), (28, 4, 65, 70, {}),   # many rows: either kernel
])
def test_cache_update_with_grouped_heads(q_heads, kv_heads, batch, prompt, modes):
    w = wl.WORKLOADS["dream7b_gqa"].scaled(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, prompt=prompt, gen=160)
    _run_block(w, block_index=1, n_steps=3, **modes)
