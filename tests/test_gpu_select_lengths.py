"""Selection of segments on either side of every 1024 candidates up to 8192 (the keys of a thread), with ties across them: index sets of
sdllm_score_select against the oracle's ranking of the scores that the same call returns, entry by entry."""
import numpy as np
import pytest
import torch

from oracle import sdllm_oracle as orc
from paper_2508_02558_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("prefix", [1, 1023, 1024, 1025, 2048, 2049, 3072, 3073, 4097, 5120, 5121, 6145, 7168, 7169, 8192])
def test_lengths(prefix, ties):
    print(f"[case] select prefix={prefix} ties={ties}", flush=True)
    torch.manual_seed(prefix)
    suffix, heads = 77, 2
    seq = prefix + 32 + suffix
    q = torch.randn(1, heads, 32, 128, device=DEV).bfloat16()
    k = torch.randn(1, heads, seq, 128, device=DEV).bfloat16()
    if ties:   # five distinct keys, so that whole runs of scores are equal
        k = k[:, :, torch.randint(0, 5, (seq,), device=DEV)].contiguous()
    shape = B.make_shape(batch=1, n_q_heads=heads, n_kv_heads=heads, head_dim=128, seq_len=seq, block_off=prefix, block_len=32,
                         dtype=B.SDLLM_BF16, retention=0.4, pool_kernel=3)
    kt, kp, ks = B.sdllm_retained_count(shape)
    idx = torch.full((1, heads, kt), -1, dtype=torch.int32, device=DEV)
    pooled, score = (torch.full((1, heads, seq - 32), float("nan"), device=DEV) for _ in range(2))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SCORE_SELECT), dtype=torch.uint8, device=DEV)
    B.sdllm_score_select(shape, q, k, idx, pooled, score, ws)
    torch.cuda.synchronize()
    pos = orc.candidate_positions(seq, prefix, 32)
    for h in range(heads):
        want = []
        for begin, length, keep in ((0, prefix, kp), (prefix, suffix, ks)):
            s = score[0, h, begin:begin + length].cpu().numpy()
            padded = np.concatenate([[-np.inf], s, [-np.inf]])
            p = np.maximum(np.maximum(padded[:-2], padded[1:-1]), padded[2:])
            assert (pooled[0, h, begin:begin + length].cpu().numpy() == p).all()
            order = np.lexsort((np.arange(length), -p))            # larger first, the lower position among equals
            want.append(begin + np.sort(order[:keep]))
        assert (idx[0, h].cpu().numpy() == pos[np.concatenate(want)]).all()
