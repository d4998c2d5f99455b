"""Full-sequence attention by key groups and step count: sequences of up to eight tiles, whose stages are loaded through registers, and
the first step counts of the rings (5 steps in LDS with one key group, 4 with two), where the prologue, the steady iterations and the
ones that fetch nothing more meet; ragged last tiles, a last step that one group has no tile of.  Tensors are stored [B, L, H, d] and
passed as [B, H, L, d] views, so that rows, heads and batches lie in another order than the results are computed in.  Tolerances:
tests/parity_util.py; the oracle sees the first, a middle and the last head."""
import pytest
import torch

from oracle import sdllm_oracle as orc
from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests import parity_util as U
from tests.test_gpu_general import _hide

pytestmark = pytest.mark.gpu
DEV = "cuda"

SHORT = [(8, 28, 4, 1, 1), (8, 28, 4, 33, 1), (8, 28, 4, 65, 1), (8, 28, 4, 97, 1), (8, 28, 4, 128, 1), (8, 32, 8, 129, 1), (8, 28, 4, 161, 1),
         (8, 28, 4, 193, 1), (8, 28, 4, 225, 1), (8, 32, 8, 256, 1), (4, 28, 4, 225, 2), (4, 32, 32, 256, 2)]
RINGS = [(8, 28, 4, 257, 1), (8, 28, 4, 289, 1), (8, 28, 4, 320, 1), (8, 28, 4, 321, 1), (8, 28, 4, 353, 1), (4, 32, 32, 385, 1), (8, 28, 4, 417, 1),
         (2, 28, 4, 257, 2), (2, 28, 4, 289, 2), (2, 28, 4, 320, 2), (2, 28, 4, 321, 2), (2, 28, 4, 353, 2), (2, 32, 8, 385, 2), (2, 28, 4, 417, 2)]


def _stored_by_rows(batch, heads, L, gain=1.0):
    return (gain * torch.randn(batch, L, heads, 128, device=DEV)).bfloat16().permute(0, 2, 1, 3)


def _run(q, k, v, groups):
    batch, q_heads, L, _ = q.shape
    shape = B.make_shape(batch=batch, n_q_heads=q_heads, n_kv_heads=k.shape[1], head_dim=128, seq_len=L, block_off=0, block_len=min(32, L),
                         dtype=B.SDLLM_BF16, kv_stride=B.strides_of(k))
    assert B.sdllm_launch_plan(shape, B.SDLLM_CALL_DENSE).key_groups == groups
    out = torch.full((batch, L, q_heads, 128), float("nan"), device=DEV, dtype=torch.bfloat16).permute(0, 2, 1, 3)
    B.sdllm_dense_attn(shape, q, k, v, out)
    torch.cuda.synchronize()
    return out


def _check(out, q, k, v):
    batch, q_heads = q.shape[:2]
    group = q_heads // k.shape[1]
    assert torch.isfinite(out.float()).all()
    for b, h in ((0, 0), (batch // 2, q_heads // 2 + 1), (batch - 1, q_heads - 1)):
        ref = orc.attention(wl.to_f64(q[b, h:h + 1]), wl.to_f64(k[b, h // group][None]), wl.to_f64(v[b, h // group][None]))
        U.assert_close(out[b, h:h + 1], ref, "bf16", f"batch {b} head {h} L={q.shape[2]}")


@pytest.mark.parametrize("batch,q_heads,kv_heads,L,groups", SHORT + RINGS)
def test_step_counts(batch, q_heads, kv_heads, L, groups):
    print(f"[case] dense_attn steps B={batch} {q_heads}/{kv_heads} L={L}", flush=True)
    torch.manual_seed(L + q_heads)
    q, k, v = _stored_by_rows(batch, q_heads, L, 2.0), _stored_by_rows(batch, kv_heads, L), _stored_by_rows(batch, kv_heads, L)
    _check(_run(q, k, v, groups), q, k, v)


# Every tile from the second on holds a key of a larger logit than all before it, in the first half of its keys and in the second by
# turns: sums and accumulators that are not zero are scaled down in every step of up to eleven, in every second or third of more.
@pytest.mark.parametrize("batch,q_heads,kv_heads,L,groups", [(8, 28, 4, 225, 1), (4, 32, 32, 256, 2), (8, 28, 4, 300, 1), (1, 28, 4, 1181, 1),
                                                             (2, 28, 4, 321, 2), (1, 28, 4, 735, 2)])
def test_rising_maxima(batch, q_heads, kv_heads, L, groups):
    print(f"[case] dense_attn rising maxima B={batch} {q_heads}/{kv_heads} L={L}", flush=True)
    torch.manual_seed(L)
    along = torch.nn.functional.normalize(torch.randn(128, device=DEV), dim=0)
    q, k, v = _stored_by_rows(batch, q_heads, L, 0.5), _stored_by_rows(batch, kv_heads, L), _stored_by_rows(batch, kv_heads, L)
    q.copy_(q.float() + 8.0 * along)
    tiles = (L + 31) // 32
    for t in range(1, tiles):
        at = min(L - 1, 32 * t + (5 if t % 2 else 21))
        k[:, :, at] = (along * (10.0 + 120.0 * t / tiles)).bfloat16()        # logits from 7 to about 90
    _check(_run(q, k, v, groups), q, k, v)


@pytest.mark.parametrize("batch,q_heads,kv_heads,L,groups", [(8, 28, 4, 200, 1), (8, 28, 4, 300, 1), (4, 32, 32, 256, 2), (2, 28, 4, 321, 2)])
def test_tiles_of_infinitely_low_keys(batch, q_heads, kv_heads, L, groups):
    # whole tiles without weight, among them the first of the sequence and of a key group
    print(f"[case] dense_attn steps, -inf tiles B={batch} {q_heads}/{kv_heads} L={L}", flush=True)
    torch.manual_seed(L)
    q, k, v = _stored_by_rows(batch, q_heads, L), _stored_by_rows(batch, kv_heads, L), _stored_by_rows(batch, kv_heads, L)
    kept = _hide(k, q, [*range(0, 64), *range(128, 160)])
    _check(_run(q, k, v, groups), q, k[:, :, kept], v[:, :, kept])
