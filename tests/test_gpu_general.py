"""The general kernels (fp32, head_dim 64, block lengths other than 32, large groups, far-apart rows) against the oracle,
at the sizes where their tiling can go wrong: 32-row blocks with 1 to 32 valid rows, one and two row blocks, tiles with a
ragged end on either side of the block, keys split over workgroups, more query blocks than one LDS stage of the scoring
holds.  Tolerances are those of tests/parity_util.py."""
import pytest
import torch

from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests import parity_util as U
from tests.test_abi_host import sequential_step_bytes
from tests.test_gpu_parity import _run_block

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype,d,block,q_heads,kv_heads,batch,prompt,modes", [
    ("bf16", 128, 1, 2, 2, 1, 33, {}),                     # one valid row of 32
    ("bf16", 128, 33, 4, 2, 1, 200, {}),                   # second row block with one row
    ("bf16", 128, 64, 9, 1, 1, 161, {}),                   # 18 query blocks: several LDS stages of queries
    ("bf16", 128, 64, 4, 4, 2, 1500, dict(select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR)),   # keys split
    ("bf16", 128, 32, 9, 1, 2, 100, {}),                   # 32-row dense kernel, general scoring (group > 8)
    ("bf16", 64, 32, 8, 2, 3, 500, dict(score_mode=B.SDLLM_LOGIT_MEAN)),
    ("bf16", 64, 24, 14, 2, 1, 1300, {}),                  # keys split, padding rows in every query block
    ("bf16", 64, 48, 2, 2, 1, 0, {}),                      # no prefix
    ("f32", 64, 32, 2, 2, 1, 2300, {}),                    # keys split
    ("f32", 64, 64, 14, 2, 1, 77, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),
    ("f32", 128, 40, 6, 2, 2, 130, {}),                    # six heads x two row blocks, more than one LDS stage
    ("f32", 128, 8, 4, 1, 1, 700, dict(score_mode=B.SDLLM_LOGIT_MEAN)),
])
def test_general_block(dtype, d, block, q_heads, kv_heads, batch, prompt, modes):
    w = wl.WORKLOADS["llada8b_layer"].scaled(dtype=dtype, head_dim=d, block=block, n_q_heads=q_heads, n_kv_heads=kv_heads,
                                             batch=batch, prompt=prompt, gen=3 * block)
    _run_block(w, block_index=1, n_steps=3, **modes)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [1, 31, 33, 64, 97, 300])
def test_general_dense_attn_row_and_tile_edges(dtype, d, L):
    print(f"[case] general dense_attn {dtype} d={d} L={L}", flush=True)
    torch.manual_seed(L)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v = (torch.randn(2, h, L, d, device=DEV).to(t) for h in (6, 2, 2))
    out = torch.zeros_like(q)
    shape = B.make_shape(batch=2, n_q_heads=6, n_kv_heads=2, head_dim=d, seq_len=L, block_off=0, block_len=min(32, L), dtype=U.DT[dtype])
    B.sdllm_dense_attn(shape, q, k, v, out)
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, k, v), dtype, f"L={L}")


@pytest.mark.parametrize("dtype,d,block,n_cached", [("bf16", 64, 16, 1300), ("f32", 64, 32, 1000), ("f32", 128, 50, 700)])
def test_general_sparse_attn_without_a_workspace(dtype, d, block, n_cached):
    # shapes whose keys are split over workgroups when there is room for the partials run unsplit when there is none
    print(f"[case] general sparse_attn, no workspace: {dtype} d={d} b={block} n={n_cached}", flush=True)
    torch.manual_seed(n_cached)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    shape = B.make_shape(batch=1, n_q_heads=2, n_kv_heads=1, head_dim=d, seq_len=4096, block_off=2048, block_len=block,
                         dtype=U.DT[dtype], cache_rows=n_cached)
    need = B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached)
    assert need > 256
    q = torch.randn(1, 2, block, d, device=DEV).to(t)
    kc, vc = (torch.randn(1, 1, n_cached, d, device=DEV).to(t) for _ in range(2))
    kb, vb = (torch.randn(1, 1, block, d, device=DEV).to(t) for _ in range(2))
    ref = U.oracle_attention_batch(q, torch.cat([kc, kb], 2), torch.cat([vc, vb], 2))
    room = torch.empty(need + 16, dtype=torch.uint8, device=DEV)
    for ws in (None, room[:need], room[:need - 1], room[1:1 + need]):
        out = torch.full_like(q, float("nan"))
        B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
        torch.cuda.synchronize()
        U.assert_close(out, ref, dtype, "no workspace" if ws is None else f"workspace of {ws.numel()} at {ws.storage_offset()}")


def test_rows_too_far_apart_for_32_bit_offsets():
    print("[case] cache rows 32 MiB apart", flush=True)
    torch.manual_seed(5)
    n, d, step = 70, 128, 1 << 24
    store = torch.empty(n * step, dtype=torch.bfloat16, device=DEV)
    kc = store.as_strided((1, 1, n, d), (0, 0, step, 1), 0)
    vc = store.as_strided((1, 1, n, d), (0, 0, step, 1), d)
    kc.copy_(torch.randn(1, 1, n, d, device=DEV))
    vc.copy_(torch.randn(1, 1, n, d, device=DEV))
    q, kb, vb = (torch.randn(1, 1, 32, d, device=DEV).bfloat16() for _ in range(3))
    shape = B.make_shape(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d, seq_len=4096, block_off=2048, block_len=32,
                         dtype=B.SDLLM_BF16, cache_stride=(0, 0, step))
    out = torch.zeros_like(q)
    B.sdllm_sparse_attn(shape, q, kc, vc, n, kb, vb, out, None)
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, torch.cat([kc, kb], 2), torch.cat([vc, vb], 2)), "bf16", "far rows")


@pytest.mark.parametrize("d", [64, 128])
def test_probabilities_keep_24_bits_with_bf16_tensors(d):
    # Row i: key 1 has probability x_i / (2 + x_i), keys 0 and 2 have 1 / (2 + x_i), the others none.  Column i of V is
    # 1 for key 1, minus the first 16 bits of x_i for keys 0 and 2, so out[i, i] is what x_i has below them.  Bound, in units
    # of 2^-24 relative to x_i: 2 for the exponential, 1 for its argument, 8 for the sums of terms near 1, 16 in all; then
    # the rounding of the result to bf16.  Sixteen-bit probabilities are off by up to 64.
    print(f"[case] 24-bit probabilities d={d}", flush=True)
    b = 31
    i = torch.arange(b)
    q, k, v = (torch.zeros(1, 1, b, d, dtype=torch.float64) for _ in range(3))
    q[..., 0], q[..., 1] = (i + 1) / 8, 64
    k[0, 0, 1, 0] = -1
    k[0, 0, 3:, 1] = -256
    x = torch.exp(-(i + 1).double() / 64)
    hi = x.bfloat16().double()
    lo = (x - hi).bfloat16().double()
    v[0, 0, 0, :b], v[0, 0, 1, :b], v[0, 0, 2, :b] = -hi, 1, -lo
    shape = B.make_shape(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d, seq_len=64, block_off=0, block_len=b, dtype=B.SDLLM_BF16,
                         softmax_scale=0.125)
    qb, kb, vb = (t.bfloat16().to(DEV) for t in (q, k, v))
    out = torch.zeros_like(qb)
    B.sdllm_sparse_attn(shape, qb, None, None, 0, kb, vb, out, None)
    torch.cuda.synchronize()
    got, want = out[0, 0, i, i].double().cpu(), (x - hi - lo) / (2 + x)
    assert ((got - want).abs() <= 16 * 2.0 ** -24 * x / (2 + x) + 2.0 ** -9 * want.abs()).all()


@pytest.mark.parametrize("dtype,d,block,n_cached", [
    ("f32", 64, 1, 0), ("f32", 128, 33, 70), ("f32", 128, 33, 1300),                              # the last with key splits
    ("bf16", 64, 1, 0), ("bf16", 128, 1, 0), ("bf16", 64, 33, 70), ("bf16", 128, 48, 1300),
])
def test_infinite_values_stay_infinite(dtype, d, block, n_cached):
    # a key of positive weight with an infinity in V: that column is infinite, the others are not touched
    print(f"[case] infinities in V: {dtype} d={d} b={block} n={n_cached}", flush=True)
    torch.manual_seed(d + n_cached)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    shape = B.make_shape(batch=1, n_q_heads=2, n_kv_heads=1, head_dim=d, seq_len=4096, block_off=2048, block_len=block,
                         dtype=U.DT[dtype], cache_rows=max(1, n_cached))
    q = torch.randn(1, 2, block, d, device=DEV).to(t)
    kc, vc = (torch.randn(1, 1, max(1, n_cached), d, device=DEV).to(t) for _ in range(2))
    kb, vb = (torch.randn(1, 1, block, d, device=DEV).to(t) for _ in range(2))
    vb[0, 0, -1, 3], vb[0, 0, 0, d - 1] = float("inf"), float("-inf")
    if n_cached:
        vc[0, 0, n_cached // 2, 17], vc[0, 0, n_cached - 1, 40] = float("-inf"), float("inf")
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    out = torch.zeros_like(q)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q, torch.cat([kc[:, :, :n_cached], kb], 2), torch.cat([vc[:, :, :n_cached], vb], 2))
    inf = torch.from_numpy(ref).isinf()
    assert inf.any() and torch.equal(out.cpu().double()[inf], torch.from_numpy(ref)[inf])
    U.assert_close(torch.where(inf.to(DEV), torch.zeros_like(out), out), torch.where(inf, 0.0, torch.from_numpy(ref)).numpy(), dtype, "finite columns")


@pytest.mark.parametrize("dtype,d,block,q_heads", [("bf16", 64, 24, 4), ("bf16", 128, 40, 9), ("f32", 64, 8, 2), ("f32", 128, 50, 6)])
@pytest.mark.parametrize("mode", [B.SDLLM_SOFTMAX_MEAN, B.SDLLM_LOGIT_MEAN])
def test_scores_of_infinitely_low_keys(dtype, d, block, q_heads, mode):
    # query blocks with padding rows: a key whose logits are all -inf weighs nothing (softmax) or -inf (logits), and the
    # other candidates keep their scores
    print(f"[case] -inf keys in the scoring: {dtype} d={d} b={block} mode={mode}", flush=True)
    torch.manual_seed(block)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    L, off = 300, 131
    shape = B.make_shape(batch=1, n_q_heads=q_heads, n_kv_heads=1, head_dim=d, seq_len=L, block_off=off, block_len=block,
                         dtype=U.DT[dtype], score_mode=mode)
    q = torch.randn(1, q_heads, block, d, device=DEV).to(t)
    q[..., 0] = q[..., 0].abs() + 0.25
    k = torch.randn(1, 1, L, d, device=DEV).to(t)
    k[0, 0, 100, 0] = k[0, 0, L - 1, 0] = float("-inf")
    low = [100, L - 1 - block]                                  # as candidates
    gl = U.GpuLayer(shape, DEV)
    _, _, score = gl.score_select(q, k)
    got = score[0, 0].double().cpu()
    kept = torch.ones(L - block, dtype=torch.bool)
    kept[low] = False
    cand = torch.cat([k[0, 0, :off], k[0, 0, off + block:]])
    a = torch.stack([q[0, h].double().cpu() @ cand[kept.to(DEV)].double().cpu().T / d ** 0.5 for h in range(q_heads)])
    want = (torch.softmax(a, -1) if mode == B.SDLLM_SOFTMAX_MEAN else a).mean((0, 1))
    assert (got[low] == (0.0 if mode == B.SDLLM_SOFTMAX_MEAN else float("-inf"))).all()
    torch.testing.assert_close(got[kept], want, rtol=2e-5, atol=1e-12 if mode == B.SDLLM_SOFTMAX_MEAN else 2e-5)


def _hide(k, q, keys):
    """Makes the logits of `keys` -inf for every query; returns the others."""
    q[..., 0] = q[..., 0].abs() + 0.25
    k[:, :, keys, 0] = float("-inf")
    return [i for i in range(k.shape[2]) if i not in set(keys)]


@pytest.mark.parametrize("dtype,d,block,n_cached", [("bf16", 64, 32, 500), ("bf16", 128, 48, 1300), ("f32", 64, 16, 500), ("f32", 128, 32, 300)])
def test_tiles_of_infinitely_low_keys(dtype, d, block, n_cached):
    # whole tiles without weight, among them the first of a wave
    print(f"[case] -inf tiles: {dtype} d={d} b={block} n={n_cached}", flush=True)
    torch.manual_seed(block + d)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    shape = B.make_shape(batch=1, n_q_heads=2, n_kv_heads=1, head_dim=d, seq_len=4096, block_off=2048, block_len=block,
                         dtype=U.DT[dtype], cache_rows=n_cached)
    q = torch.randn(1, 2, block, d, device=DEV).to(t)
    kc, vc = (torch.randn(1, 1, n_cached, d, device=DEV).to(t) for _ in range(2))
    kb, vb = (torch.randn(1, 1, block, d, device=DEV).to(t) for _ in range(2))
    kept = _hide(kc, q, [*range(64, 130), *range(224, 256)])
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    out = torch.zeros_like(q)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q, torch.cat([kc[:, :, kept], kb], 2), torch.cat([vc[:, :, kept], vb], 2)), dtype, "kept keys")


# Cache-update steps whose key splits are merged in the compaction's launch: both types, row blocks that are not full, more than
# one block of rows per head, no softmax in the score.
@pytest.mark.parametrize("dtype,d,block,q_heads,kv_heads,batch,prompt,modes", [
    ("bf16", 128, 64, 8, 8, 1, 1300, {}), ("bf16", 128, 24, 14, 2, 1, 900, {}), ("bf16", 64, 32, 4, 2, 1, 1500, {}),
    ("bf16", 128, 48, 4, 4, 2, 1200, dict(score_mode=B.SDLLM_LOGIT_MEAN)), ("f32", 64, 32, 4, 4, 1, 700, {}), ("f32", 128, 17, 4, 2, 2, 600, {}),
    ("f32", 64, 64, 2, 2, 1, 800, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),
])
def test_update_steps_merge_their_splits_with_the_compaction(dtype, d, block, q_heads, kv_heads, batch, prompt, modes):
    w = wl.WORKLOADS["llada8b_layer"].scaled(dtype=dtype, head_dim=d, block=block, n_q_heads=q_heads, n_kv_heads=kv_heads,
                                             batch=batch, prompt=prompt, gen=4 * block)
    assert B.sdllm_launch_plan(U.shape_for(w, 1, **modes), B.SDLLM_CALL_UPDATE).key_splits > 1
    _run_block(w, block_index=1, n_steps=3, **modes)


# The same steps with a workspace in which the partials and the scoring buffers take turns: the merge is a launch of its own then.
@pytest.mark.parametrize("dtype,d,block,q_heads,kv_heads,L,rows,mode", [
    ("bf16", 128, 64, 8, 8, 1500, 32, B.SDLLM_SOFTMAX_MEAN), ("bf16", 64, 32, 4, 2, 1600, 32, B.SDLLM_LOGIT_MEAN),
    ("f32", 128, 40, 6, 2, 900, 16, B.SDLLM_SOFTMAX_MEAN),
])
def test_update_step_in_less_workspace(dtype, d, block, q_heads, kv_heads, L, rows, mode):
    print(f"[case] update step, less workspace: {dtype} d={d} b={block} L={L}", flush=True)
    torch.manual_seed(L)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    shape = B.make_shape(batch=1, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=d, seq_len=L, block_off=500, block_len=block,
                         dtype=U.DT[dtype], score_mode=mode)
    kt = B.sdllm_retained_count(shape)[0]
    q, k, v = (torch.randn(1, h, n, d, device=DEV).to(t) for h, n in ((q_heads, block), (kv_heads, L), (kv_heads, L)))
    results = []
    for nbytes in (B.sdllm_workspace_bytes(shape, B.SDLLM_OP_BLOCK_STEP), sequential_step_bytes(shape, rows)):
        room = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
        idx = torch.zeros(1, kv_heads, kt, dtype=torch.int32, device=DEV)
        kc, vc = (torch.zeros(1, kv_heads, L - block, d, device=DEV, dtype=t) for _ in range(2))
        out = torch.zeros_like(q)
        assert B.sdllm_block_step(shape, 1, 1, q, k, v, idx, kc, vc, out, room[:nbytes]) == B.SDLLM_STATE_UPDATE
        torch.cuda.synchronize()
        assert (room[nbytes:] == 0x5A).all()
        results.append((out, idx, kc, vc))
    assert all(torch.equal(a, b) for a, b in zip(*results))
    U.assert_close(results[1][0], U.oracle_attention_batch(q, k, v), dtype, "dense rows")
