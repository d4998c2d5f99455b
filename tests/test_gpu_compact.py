"""The gather at the edges of its blocks, which copy 16, 32 or 64 rows of one (batch, KV head): row counts on either side of them, every
row size, caches with room to spare and strided sources.  Byte for byte."""
import pytest
import torch

from paper_2508_02558_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("batch,heads,kept", [(1, 1, 1), (2, 3, 15), (1, 7, 16), (3, 2, 17), (2, 1, 31), (1, 5, 32), (2, 2, 33), (1, 3, 63), (2, 2, 64),
                                              (1, 2, 65), (3, 5, 129)])
def test_gather(dtype, d, batch, heads, kept):
    print(f"[case] compact {dtype} d={d} B={batch} heads={heads} kept={kept}", flush=True)
    torch.manual_seed(kept + d)
    t, code = (torch.bfloat16, B.SDLLM_BF16) if dtype == "bf16" else (torch.float32, B.SDLLM_F32)
    seq = 32 + kept                                            # everything behind the block is kept
    k, v = (torch.randn(batch, seq, heads, d, device=DEV).to(t).permute(0, 2, 1, 3) for _ in range(2))   # [B, rows, H, d] storage
    kc, vc = (torch.full((batch, heads, kept + 3, d), float("nan"), device=DEV, dtype=t) for _ in range(2))
    shape = B.make_shape(batch=batch, n_q_heads=heads, n_kv_heads=heads, head_dim=d, seq_len=seq, block_off=0, block_len=32, dtype=code,
                         retention=1.0, cache_rows=kept + 3, kv_stride=B.strides_of(k))
    assert B.sdllm_retained_count(shape)[0] == kept
    idx = torch.randint(0, seq, (batch, heads, kept), device=DEV, dtype=torch.int32)
    B.sdllm_compact_kv(shape, k, v, idx, kc, vc)
    torch.cuda.synchronize()
    rows = idx.long()[..., None].expand(-1, -1, -1, d)
    for src, dst in ((k, kc), (v, vc)):
        assert torch.equal(dst[:, :, :kept], src.gather(2, rows))
        assert dst[:, :, kept:].isnan().all()                  # nothing behind the retained rows


def test_more_blocks_than_a_launch_has():
    # one row of each of 16 793 600 heads, a block each: 16 385 more than have fewer than 2^32 threads
    print("[case] compact, 16.8 million heads of one row", flush=True)
    batch, heads, d = 65600, 256, 64
    k, v = (torch.randint(-30000, 30000, (batch, heads, 2, d), device=DEV, dtype=torch.int16) for _ in range(2))
    kc, vc = (torch.zeros(batch, heads, 1, d, device=DEV, dtype=torch.int16) for _ in range(2))
    shape = B.make_shape(batch=batch, n_q_heads=heads, n_kv_heads=heads, head_dim=d, seq_len=2, block_off=0, block_len=1, dtype=B.SDLLM_BF16,
                         retention=1.0, cache_rows=1, kv_stride=B.strides_of(k))
    assert B.sdllm_retained_count(shape)[0] == 1
    idx = torch.randint(0, 2, (batch, heads, 1), device=DEV, dtype=torch.int32)
    B.sdllm_compact_kv(shape, k, v, idx, kc, vc)
    torch.cuda.synchronize()
    for src, dst in ((k, kc), (v, vc)):
        assert torch.equal(dst[:, :, 0], torch.where(idx == 0, src[:, :, 0], src[:, :, 1]))
