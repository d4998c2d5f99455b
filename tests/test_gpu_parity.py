"""GPU-vs-oracle parity of the HIP path, element by element, through the C ABI.

Index sets: bit-exact outside the tie band (entries whose oracle pooled score lies within 1e-4
relative of the k-th value are reported as ties and may differ).  Compaction: bit-exact.
Attention outputs: max-abs <= 2e-2 and mean-abs <= 2e-3 for bf16 tensors with fp32 accumulation,
1e-5 / 1e-6 for fp32 tensors.
"""
import numpy as np
import pytest
import torch

from oracle import sdllm_oracle as orc
from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import workloads as wl
from tests import parity_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _note(msg):
    print(msg, flush=True)


def _run_block(w, layer=0, block_index=0, n_steps=4, delay=1, **modes):
    """A whole decoding block through sdllm_block_step against the oracle, every step."""
    _note(f"[case] block_step workload={w.name} B={w.batch} Hq={w.n_q_heads} Hkv={w.n_kv_heads} "
          f"L={w.seq_len} block={block_index} modes={modes}")
    inp = wl.make_block_inputs(w, layer, block_index, n_steps)
    shape = U.shape_for(w, block_index, **modes)
    o, b = inp["block_off"], w.block
    gl = U.GpuLayer(shape, DEV)
    k_full = inp["k_full"].to(DEV)
    v_full = inp["v_full"].to(DEV)
    q_all, kb_all, vb_all = inp["q"].to(DEV), inp["k_blk"].to(DEV), inp["v_blk"].to(DEV)
    cache_gpu = None
    ties = 0
    for t in range(n_steps):
        state = orc.cache_state(t, delay)
        q = q_all[t].contiguous()
        if state < 2:
            k_full[:, :, o:o + b] = kb_all[t]
            v_full[:, :, o:o + b] = vb_all[t]
            st = gl.block_step(t, delay, q, k_full, v_full)
            ref = U.oracle_attention_batch(q, k_full, v_full)
            U.assert_close(gl.out, ref, w.dtype, f"dense step {t}")
            if state == 1:
                idx_gpu = gl.idx[:, :, :gl.k_total].cpu().numpy().astype(np.int64)
                idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q, k_full)
                for bi in range(w.batch):
                    for g in range(w.n_kv_heads):
                        ties += U.compare_index_rows(idx_gpu[bi, g], idx_orc[bi, g], pooled_orc[bi, g], w.seq_len, o, b,
                                                     U.ranked_segments(shape))
                # compaction is a byte copy of the rows the GPU itself selected
                ig = torch.from_numpy(idx_gpu).to(DEV)
                want_k = torch.gather(k_full, 2, ig[..., None].expand(-1, -1, -1, w.head_dim))
                want_v = torch.gather(v_full, 2, ig[..., None].expand(-1, -1, -1, w.head_dim))
                assert torch.equal(gl.k_cache[:, :, :gl.k_total], want_k)
                assert torch.equal(gl.v_cache[:, :, :gl.k_total], want_v)
                # ... and equals the oracle's gather of the same rows (Sec. 3.3, fourth equation), value for value:
                # a bf16 or fp32 element is exactly representable in the oracle's float64
                for bi in range(w.batch):
                    kc, vc = orc.compact_kv(wl.to_f64(k_full[bi]), wl.to_f64(v_full[bi]), idx_gpu[bi])
                    assert np.array_equal(wl.to_f64(gl.k_cache[bi, :, :gl.k_total]), kc), f"K_c batch {bi}"
                    assert np.array_equal(wl.to_f64(gl.v_cache[bi, :, :gl.k_total]), vc), f"V_c batch {bi}"
                cache_gpu = (want_k, want_v)
        else:
            kb, vb = kb_all[t].contiguous(), vb_all[t].contiguous()
            st = gl.block_step(t, delay, q, kb, vb)
            # end to end with the GPU's own index set (the oracle attends to the same rows)
            ref = U.oracle_attention_batch(q, torch.cat([cache_gpu[0], kb], 2), torch.cat([cache_gpu[1], vb], 2))
            U.assert_close(gl.out, ref, w.dtype, f"sparse step {t}")
        assert st == state
    _note(f"[done] ties in band: {ties}")
    return ties


def test_tiny_fp32_block():
    _run_block(wl.WORKLOADS["tiny"])


@pytest.mark.parametrize("modes", [
    dict(score_mode=B.SDLLM_LOGIT_MEAN),
    dict(select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR),
    dict(select_mode=B.SDLLM_JOINT, score_mode=B.SDLLM_LOGIT_MEAN, k_rounding=B.SDLLM_FLOOR),
    dict(pool_mode=B.SDLLM_AVG_POOL),
    dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY),
])
def test_tiny_fp32_modes(modes):
    _run_block(wl.WORKLOADS["tiny"], n_steps=3, **modes)


@pytest.mark.parametrize("delay", [0, 2, 3])
def test_tiny_delay_sweep(delay):
    _run_block(wl.WORKLOADS["tiny"].scaled(steps_per_block=6), n_steps=6, delay=delay)


@pytest.mark.parametrize("r,s", [(0.1, 1), (0.3, 5), (0.7, 7), (0.9, 9), (0.0, 3), (1.0, 3)])
def test_tiny_retention_and_kernel_sweep(r, s):
    _run_block(wl.WORKLOADS["tiny"].scaled(retention=r, pool_kernel=s), n_steps=3)


def test_llada_layer_bf16_block():
    # the LLaDA-8B-shaped single layer at full size: 32 heads, prompt 1024, first block
    _run_block(wl.WORKLOADS["llada8b_layer"], n_steps=3)


@pytest.mark.parametrize("modes", [dict(), dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY), dict(pool_mode=B.SDLLM_AVG_POOL)])
def test_many_heads_unsplit_update_step_off_grid(modes):
    # 160 heads: one workgroup per head and no key splits, so the cache-update step's dense launch also
    # sweeps K for the saliency scores; the block starts at an odd offset (tiles straddle the block on
    # both sides), once in the middle of the generation and once at its end (no suffix)
    w = wl.WORKLOADS["llada8b_layer"].scaled(batch=5, prompt=1013)
    _run_block(w, layer=1, block_index=3, n_steps=3, **modes)
    if not modes:
        _run_block(w, layer=2, block_index=w.n_blocks - 1, n_steps=3)


def test_llada_layer_last_block_has_no_suffix():
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=4)
    _run_block(w, block_index=w.n_blocks - 1, n_steps=3)


def test_last_block_with_exactly_sized_score_buffers():
    # The last block of a generation has no suffix, so the suffix segment of every row is empty; the
    # optional score / pooled outputs are exactly [B, Hkv, N] floats placed at the very end of a buffer
    # whose following bytes hold NaN.  Nothing may be written behind them and the index set must not
    # depend on where the score rows live.
    _note("[case] last block, exactly sized score_out / pooled_out")
    for pool_kernel, prompt in ((3, 1024), (5, 9000)):   # register-resident and LDS-resident select
        w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=4, prompt=prompt, pool_kernel=pool_kernel)
        bi = w.n_blocks - 1
        inp = wl.make_block_inputs(w, 0, bi, 2, device=DEV)
        shape = U.shape_for(w, bi)
        gl = U.GpuLayer(shape, DEV)
        assert shape.seq_len - shape.block_off - shape.block_len == 0
        q = inp["q"][1].contiguous()
        idx_ws, _, _ = gl.score_select(q, inp["k_full"], want_scores=False)
        n = w.batch * w.n_kv_heads * gl.n_cand
        guard = 64
        buf_s = torch.full((n + guard,), float("nan"), device=DEV)
        buf_p = torch.full((n + guard,), float("nan"), device=DEV)
        gl.idx.fill_(-1)
        B.sdllm_score_select(shape, q, inp["k_full"], gl.idx, buf_p[:n], buf_s[:n], gl.ws)
        torch.cuda.synchronize()
        assert (gl.idx[:, :, :gl.k_total].cpu().numpy() == idx_ws).all()
        assert torch.isnan(buf_s[n:]).all() and torch.isnan(buf_p[n:]).all()
        assert torch.isfinite(buf_s[:n]).all() and torch.isfinite(buf_p[:n]).all()
        idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q, inp["k_full"])
        for g in range(w.n_kv_heads):
            U.compare_index_rows(idx_ws[0, g], idx_orc[0, g], pooled_orc[0, g], w.seq_len, inp["block_off"], w.block,
                                 U.ranked_segments(shape))


def test_block_at_sequence_start_has_no_prefix():
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=4, prompt=0, gen=512)
    _run_block(w, block_index=0, n_steps=3)


def test_dream_gqa_bf16_block():
    _run_block(wl.WORKLOADS["dream7b_gqa"], n_steps=3)


def test_dream_gqa_modes():
    w = wl.WORKLOADS["dream7b_gqa"].scaled(prompt=1000, gen=96)   # ragged: 1000 and 64 candidates per side
    _run_block(w, n_steps=3, select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR)
    _run_block(w, n_steps=3, score_mode=B.SDLLM_LOGIT_MEAN, evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)


def test_bf16_head_dim_64_and_short_block_take_the_generic_path():
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=2, head_dim=64, prompt=200, gen=64)
    _run_block(w, n_steps=3)
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=2, n_kv_heads=2, prompt=100, gen=48, block=16)
    _run_block(w, n_steps=3)


def test_batched_block():
    w = wl.WORKLOADS["llada8b_sweep"].scaled(batch=3, n_q_heads=4, n_kv_heads=4, prompt=300, gen=64)
    _run_block(w, n_steps=3)


# ------------------------------------------------------------------ sdllm_sparse_attn on its own
@pytest.mark.parametrize("n_cached", [0, 1, 31, 32, 33, 77, 1000, 2165])
def test_sparse_attn_ragged_cache_lengths(n_cached):
    _note(f"[case] sparse_attn n_cached={n_cached}")
    torch.manual_seed(n_cached)
    Bt, Hq, Hkv, b, d = 2, 8, 4, 32, 128
    shape = B.make_shape(batch=Bt, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=4096, block_off=2048,
                         block_len=b, dtype=B.SDLLM_BF16, cache_rows=max(1, n_cached))
    q = torch.randn(Bt, Hq, b, d, device=DEV).bfloat16()
    kc = torch.randn(Bt, Hkv, max(1, n_cached), d, device=DEV).bfloat16()
    vc = torch.randn_like(kc.float()).bfloat16()
    kb = torch.randn(Bt, Hkv, b, d, device=DEV).bfloat16()
    vb = torch.randn(Bt, Hkv, b, d, device=DEV).bfloat16()
    out = torch.zeros(Bt, Hq, b, d, device=DEV, dtype=torch.bfloat16)
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    B.sdllm_sparse_attn(shape, q, kc if n_cached else None, vc if n_cached else None, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q, torch.cat([kc[:, :, :n_cached], kb], 2), torch.cat([vc[:, :, :n_cached], vb], 2))
    U.assert_close(out, ref, "bf16", f"n_cached={n_cached}")


def test_sparse_attn_strided_views_and_explicit_scale():
    _note("[case] sparse_attn strided views")
    torch.manual_seed(5)
    Bt, Hq, Hkv, b, d, n = 2, 4, 2, 32, 128, 150
    # tensors stored [B, n, H, d] and passed as [B, H, n, d] views
    q = torch.randn(Bt, b, Hq, d, device=DEV).bfloat16().permute(0, 2, 1, 3)
    kc = torch.randn(Bt, 200, Hkv, d, device=DEV).bfloat16().permute(0, 2, 1, 3)
    vc = torch.randn(Bt, 200, Hkv, d, device=DEV).bfloat16().permute(0, 2, 1, 3)
    kb = torch.randn(Bt, b, Hkv, d, device=DEV).bfloat16().permute(0, 2, 1, 3)
    vb = torch.randn(Bt, b, Hkv, d, device=DEV).bfloat16().permute(0, 2, 1, 3)
    out = torch.zeros(Bt, b, Hq, d, device=DEV, dtype=torch.bfloat16).permute(0, 2, 1, 3)
    shape = B.make_shape(batch=Bt, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=1024, block_off=512, block_len=b,
                         dtype=B.SDLLM_BF16, softmax_scale=0.05, q_stride=B.strides_of(q),
                         cache_stride=B.strides_of(kc), blk_stride=B.strides_of(kb), out_stride=B.strides_of(out))
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n), dtype=torch.uint8, device=DEV)
    B.sdllm_sparse_attn(shape, q, kc, vc, n, kb, vb, out, ws)
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q, torch.cat([kc[:, :, :n], kb], 2), torch.cat([vc[:, :, :n], vb], 2), scale=0.05)
    U.assert_close(out, ref, "bf16", "strided")


def test_r_one_reproduces_dense_attention_and_zero_queries_pick_lowest_positions():
    _note("[case] r=1 and all-ties")
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=4, prompt=256, gen=96, retention=1.0)
    inp = wl.make_block_inputs(w, n_steps=2)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    q = inp["q"][1].to(DEV).contiguous()
    k, v = inp["k_full"].to(DEV), inp["v_full"].to(DEV)
    o, b = inp["block_off"], w.block
    idx, _, _ = gl.score_select(q, k)
    cand = orc.candidate_positions(w.seq_len, o, b)
    assert (idx == cand[None, None]).all()
    gl.compact(k, v)
    out = gl.sparse_attn(q, k[:, :, o:o + b].contiguous(), v[:, :, o:o + b].contiguous()).clone()
    gl.block_step(0, 1, q, k, v)   # dense
    assert (out.float() - gl.out.float()).abs().max().item() <= 2e-2
    U.assert_close(out, U.oracle_attention_batch(q, k, v), "bf16", "r=1 sparse == dense")
    # all-zero queries: every candidate ties, the lowest positions of each segment win
    w2 = w.scaled(retention=0.5)
    shape2 = U.shape_for(w2)
    gl2 = U.GpuLayer(shape2, DEV)
    idx2, pooled2, score2 = gl2.score_select(torch.zeros_like(q), k)
    n_pre, n_suf = o, w.seq_len - o - b
    want = np.concatenate([np.arange(n_pre // 2), o + b + np.arange(n_suf // 2)])
    assert (idx2 == want[None, None]).all()
    np.testing.assert_allclose(score2.cpu().numpy(), 1.0 / (n_pre + n_suf), rtol=1e-5)


@pytest.mark.parametrize("prompt,gen,block_index,modes", [
    (9000, 96, 0, {}),                                                            # 9 chunks of 1024, ragged
    (12288, 64, 0, dict(pool_mode=B.SDLLM_AVG_POOL)),                              # exactly 12 chunks, avg pooling
    (20000, 96, 1, dict(select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR)),     # joint ranking across the seam
    (30000, 64, 0, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),                   # suffix kept whole
])
def test_select_long_segments(prompt, gen, block_index, modes):
    # segments of more than 8192 candidates are ranked by the kernel that keeps its keys in LDS
    _note(f"[case] long-segment select prompt={prompt} modes={modes}")
    for pool_kernel in (1, 3, 5, 7):   # windows 1, 3 and 5 have compile-time paths, 7 takes the generic pooling
        w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=2, n_kv_heads=2, prompt=prompt, gen=gen, pool_kernel=pool_kernel,
                                                 retention=0.3)
        inp = wl.make_block_inputs(w, 0, block_index, 2, device=DEV)
        shape = U.shape_for(w, block_index, **modes)
        gl = U.GpuLayer(shape, DEV)
        q = inp["q"][1].contiguous()
        idx_gpu, pooled, _ = gl.score_select(q, inp["k_full"])
        idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q, inp["k_full"])
        for begin, length, k in U.ranked_segments(shape):
            if k >= 0:   # pooled values are defined for ranked candidates only
                np.testing.assert_allclose(pooled[:, :, begin:begin + length].cpu().double().numpy(),
                                           pooled_orc[:, :, begin:begin + length], rtol=2e-5, atol=1e-12)
        for g in range(w.n_kv_heads):
            U.compare_index_rows(idx_gpu[0, g], idx_orc[0, g], pooled_orc[0, g], w.seq_len, inp["block_off"], w.block,
                                 U.ranked_segments(shape))
        # and once more without the optional pooled/score outputs (the keys then never leave the chip)
        gl.idx.fill_(-1)
        B.sdllm_score_select(shape, q, inp["k_full"], gl.idx, None, None, gl.ws)
        torch.cuda.synchronize()
        assert (gl.idx[:, :, :gl.k_total].cpu().numpy() == idx_gpu).all()


@pytest.mark.parametrize("prompt,modes", [
    (3000, {}),                                                                   # one workgroup per segment
    (20000, {}),                                                                  # pooling spread over 10 workgroups
    (20000, dict(select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR)),           # one joint segment across the seam
    (70000, dict(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)),                         # 35 pooling workgroups, suffix kept whole
])
def test_exact_ties_across_workgroup_boundaries(prompt, modes):
    # Keys that take only five distinct values, in runs of 37 positions: every score is one of five
    # levels, each level holds a fifth of the candidates, and the k-th value falls inside a level whose
    # members are spread over the whole segment.  The retained members of that level must be exactly
    # its lowest positions, which the emission can only get right if its counts of equal entries are
    # exact across every pooling-workgroup (2048) and emission-workgroup (1024) boundary.  Identical keys
    # give bit-identical scores on both sides, so the index sets are compared entry by entry.
    _note(f"[case] exact ties prompt={prompt} modes={modes}")
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=2, n_kv_heads=2, prompt=prompt, gen=96, retention=0.3)
    inp = wl.make_block_inputs(w, 0, 1, 2, device=DEV)
    shape = U.shape_for(w, 1, **modes)
    gl = U.GpuLayer(shape, DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(prompt)
    levels = torch.randn(w.batch, w.n_kv_heads, 5, w.head_dim, device=DEV, generator=g).bfloat16()
    which = (torch.arange(w.seq_len, device=DEV) // 37) % 5
    k_full = levels[:, :, which]
    q = inp["q"][1].contiguous()
    idx_gpu, pooled, _ = gl.score_select(q, k_full)
    idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q, k_full)
    for begin, length, k in U.ranked_segments(shape):
        if k >= 0:
            assert np.unique(pooled_orc[:, :, begin:begin + length]).size <= 5 * w.n_kv_heads
            assert torch.unique(pooled[:, :, begin:begin + length]).numel() <= 5 * w.n_kv_heads
    assert idx_gpu.shape == idx_orc.shape
    assert (idx_gpu == idx_orc).all(), f"{int((idx_gpu != idx_orc).sum())} entries differ"
    # all-zero queries: one level for everybody, the threshold bin holds the whole segment
    idx0, _, _ = gl.score_select(torch.zeros_like(q), k_full)
    want = []
    for begin, length, k in U.ranked_segments(shape):
        cand = orc.candidate_positions(w.seq_len, inp["block_off"], w.block)[begin:begin + length]
        want.append(cand if k < 0 else cand[:k])
    assert (idx0 == np.concatenate(want)[None, None]).all()


@pytest.mark.parametrize("prompt,gen,batch", [
    (9217, 9248, 1),     # prefix 9 chunks + 1 candidate, suffix exactly 9 chunks: both segments take the two-launch path
    (8193, 64, 3),       # one candidate beyond the single-workgroup limit; short suffix; several rows
    (16384, 12320, 2),   # prefix exactly 16 chunks (two per wave of the finish kernel), suffix 12 chunks + 32
])
def test_select_with_both_segments_long(prompt, gen, batch):
    # chunk counts that are odd, even, and one over a boundary, on both sides of the block at once
    _note(f"[case] both segments long: prompt={prompt} gen={gen} batch={batch}")
    w = wl.WORKLOADS["llada8b_layer"].scaled(batch=batch, n_q_heads=2, n_kv_heads=2, prompt=prompt, gen=gen, retention=0.4)
    inp = wl.make_block_inputs(w, 0, 0, 2, device=DEV)
    shape = U.shape_for(w, 0)
    gl = U.GpuLayer(shape, DEV)
    q = inp["q"][1].contiguous()
    idx_gpu, pooled, _ = gl.score_select(q, inp["k_full"])
    idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q, inp["k_full"])
    np.testing.assert_allclose(pooled.cpu().double().numpy(), pooled_orc, rtol=3e-5, atol=1e-12)
    ties = 0
    for bi in range(batch):
        for g in range(w.n_kv_heads):
            ties += U.compare_index_rows(idx_gpu[bi, g], idx_orc[bi, g], pooled_orc[bi, g], w.seq_len, inp["block_off"], w.block,
                                         U.ranked_segments(shape))
    _note(f"[done] ties in band: {ties}")


def test_select_at_the_longest_supported_segment():
    # a prefix of 1 046 528 candidates = 1022 chunks, just under the two-launch path's limit of 1024: the
    # per-chunk tables of the finish kernel are nearly full and every one of its 256 workgroups adds up
    # 1022 bin lists
    _note("[case] 1M-candidate segment")
    w = wl.WORKLOADS["dream_long"].scaled(n_q_heads=1, n_kv_heads=1, prompt=1022 * 1024, gen=64, retention=0.1, sink=16)
    inp = wl.make_block_inputs(w, n_steps=2, device=DEV)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    q = inp["q"][1].contiguous()
    idx, _, score = gl.score_select(q, inp["k_full"])
    idx_orc, pooled_orc, score_orc = U.oracle_score_select(shape, q, inp["k_full"])
    np.testing.assert_allclose(score.cpu().double().numpy(), score_orc, rtol=1e-4, atol=1e-14)
    ties = U.compare_index_rows(idx[0, 0], idx_orc[0, 0], pooled_orc[0, 0], w.seq_len, inp["block_off"], w.block,
                                U.ranked_segments(shape))
    _note(f"[done] ties in band: {ties}")


def test_scores_match_oracle_values():
    _note("[case] score / pooled values")
    # every group size has its own instantiation of the two scoring passes (the stand-alone entry
    # point runs its own row-statistics pass; inside a block step the dense attention supplies them)
    groups = [("llada8b_layer", dict(n_q_heads=2 * G, n_kv_heads=2, prompt=97 + 61 * G, gen=64)) for G in (2, 3, 4, 5, 6, 8)]
    for name, kw in [("llada8b_layer", dict(n_q_heads=4, n_kv_heads=4, prompt=500, gen=128)),
                     ("dream7b_gqa", dict(prompt=700, gen=96)), ("tiny", {})] + groups:
        w = wl.WORKLOADS[name].scaled(**kw)
        inp = wl.make_block_inputs(w, n_steps=2)
        for mode in (B.SDLLM_SOFTMAX_MEAN, B.SDLLM_LOGIT_MEAN):
            shape = U.shape_for(w, score_mode=mode)
            gl = U.GpuLayer(shape, DEV)
            q = inp["q"][1].to(DEV).contiguous()
            k = inp["k_full"].to(DEV)
            _, pooled, score = gl.score_select(q, k)
            _, pooled_orc, score_orc = U.oracle_score_select(shape, q, k)
            sg, pg = score.cpu().double().numpy(), pooled.cpu().double().numpy()
            if mode == B.SDLLM_SOFTMAX_MEAN:
                np.testing.assert_allclose(sg, score_orc, rtol=2e-5, atol=1e-12)
                np.testing.assert_allclose(pg, pooled_orc, rtol=2e-5, atol=1e-12)
                np.testing.assert_allclose(sg.sum(-1), 1.0, rtol=1e-5)
            else:
                np.testing.assert_allclose(sg, score_orc, rtol=0, atol=2e-5)
                np.testing.assert_allclose(pg, pooled_orc, rtol=0, atol=2e-5)


def _check_selected_rows(gl, shape, w, q, k_full, o, b, rows):
    """Index sets of the batch elements `rows` after a cache-update step, against the oracle."""
    idx_gpu = gl.idx[rows, :, :gl.k_total].cpu().numpy().astype(np.int64)
    idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q[rows], k_full[rows])
    for i in range(len(rows)):
        for g in range(w.n_kv_heads):
            U.compare_index_rows(idx_gpu[i, g], idx_orc[i, g], pooled_orc[i, g], w.seq_len, o, b, U.ranked_segments(shape))


def _runs_shared_kernel(w, *calls, block_index=0):
    """Whether every one of the calls (sparse steps over the retained keys) takes the shared-tile grouped-query kernel."""
    shape = U.shape_for(w, block_index)
    k_total, _, _ = B.sdllm_retained_count(shape)
    return all(B.sdllm_launch_plan(shape, c, k_total if c == B.SDLLM_CALL_SPARSE else 0).kernel == B.SDLLM_KERNEL_SHARED_TILE for c in calls)


def _at_shared_kernel_batch(w, *calls):
    """`w` at the smallest batch from which on it does."""
    batch = 1
    while not (_runs_shared_kernel(w.scaled(batch=batch), *calls) and _runs_shared_kernel(w.scaled(batch=2 * batch), *calls)):
        batch += 1
    return w.scaled(batch=batch)


def test_grouped_query_kernel_at_large_batch():
    # enough heads x key tiles switches sdllm_sparse_attn / the dense step to the shared-tile grouped-query kernel
    _note("[case] grouped-query shared-tile kernel")
    both = (B.SDLLM_CALL_SPARSE, B.SDLLM_CALL_UPDATE)
    w = _at_shared_kernel_batch(wl.WORKLOADS["dream7b_gqa"].scaled(prompt=300, gen=64), *both)   # ragged tiles; 150 + 16 retained keys
    inp = wl.make_block_inputs(w, n_steps=3, device=DEV)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    assert gl.k_total == 166
    o, b = inp["block_off"], w.block
    q1 = inp["q"][1].contiguous()
    assert gl.block_step(1, 1, q1, inp["k_full"], inp["v_full"]) == 1
    bs = [0, 7, w.batch - 1]
    U.assert_close(gl.out[bs], U.oracle_attention_batch(q1[bs], inp["k_full"][bs], inp["v_full"][bs]), "bf16", "dense gqa")
    _check_selected_rows(gl, shape, w, q1, inp["k_full"], o, b, bs)
    q2, kb, vb = inp["q"][2].contiguous(), inp["k_blk"][2].contiguous(), inp["v_blk"][2].contiguous()
    assert gl.block_step(2, 1, q2, kb, vb) == 2
    kt = gl.k_total
    ref = U.oracle_attention_batch(q2[bs], torch.cat([gl.k_cache[bs, :, :kt], kb[bs]], 2),
                                   torch.cat([gl.v_cache[bs, :, :kt], vb[bs]], 2))
    U.assert_close(gl.out[bs], ref, "bf16", "sparse gqa")
    del inp, gl
    # every group size the shared-tile kernel serves has its own workgroup shape (waves, pieces per
    # thread, tiles per LDS stage, one or two head splits); prompts chosen so that tile counts are odd
    # and even, with ragged last tiles.  Groups of 3, 5 and 6 heads run the one-workgroup-per-head
    # kernel at any size; they go through the same checks at a batch of that order.
    for G, Hkv, prompt in ((2, 3, 1000), (3, 2, 33), (4, 2, 905), (5, 1, 100), (6, 1, 257), (7, 1, 64), (8, 1, 70)):
        w2 = w.scaled(n_q_heads=G * Hkv, n_kv_heads=Hkv, prompt=prompt, gen=64)
        if G in (2, 4, 7, 8):
            w2 = _at_shared_kernel_batch(w2, *both)
        else:
            w2 = w2.scaled(batch=200)
            assert not any(_runs_shared_kernel(w2, c) for c in both)
        inp2 = wl.make_block_inputs(w2, n_steps=3, device=DEV)
        gl2 = U.GpuLayer(U.shape_for(w2), DEV)
        q = inp2["q"][1].contiguous()
        gl2.block_step(1, 1, q, inp2["k_full"], inp2["v_full"])
        last = w2.batch - 1
        bs2 = [0, last]
        U.assert_close(gl2.out[bs2], U.oracle_attention_batch(q[bs2], inp2["k_full"][bs2], inp2["v_full"][bs2]), "bf16", f"dense G={G}")
        _check_selected_rows(gl2, gl2.shape, w2, q, inp2["k_full"], inp2["block_off"], w2.block, bs2)
        q2, kb, vb = inp2["q"][2].contiguous(), inp2["k_blk"][2].contiguous(), inp2["v_blk"][2].contiguous()
        gl2.block_step(2, 1, q2, kb, vb)
        kt = gl2.k_total
        ref = U.oracle_attention_batch(q2[bs2], torch.cat([gl2.k_cache[bs2, :, :kt], kb[bs2]], 2),
                                       torch.cat([gl2.v_cache[bs2, :, :kt], vb[bs2]], 2))
        U.assert_close(gl2.out[bs2], ref, "bf16", f"sparse G={G}")
        del inp2, gl2


@pytest.mark.parametrize("batch,q_heads,prompt,modes", [
    (2, 28, 20000, {}),                                              # block on a tile boundary
    (2, 28, 20011, {}),                                              # the block's keys share two tiles with candidates
    (2, 28, 20011, {"evict_scope": B.SDLLM_EVICT_PREFIX_ONLY}),      # the suffix is not scored either
    (3, 32, 10643, {}),                                              # groups of eight
])
def test_grouped_query_kernel_with_key_splits(batch, q_heads, prompt, modes):
    # few (batch, KV head) rows but long keys: the shared-tile kernel then splits every row's keys over
    # many workgroups (ragged last split, fp32 partials, combine) in both the dense and the sparse step;
    # at the cache-update step it also supplies the scoring pass's row statistics, so the index sets
    # checked here depend on its candidate-only (max, sum) in every split
    w = wl.WORKLOADS["dream7b_gqa"].scaled(batch=batch, n_q_heads=q_heads, prompt=prompt, gen=64, retention=0.99)
    assert _runs_shared_kernel(w, B.SDLLM_CALL_SPARSE, B.SDLLM_CALL_FULL, B.SDLLM_CALL_UPDATE)
    assert B.sdllm_launch_plan(U.shape_for(w), B.SDLLM_CALL_UPDATE).key_splits > 1
    _run_block(w, n_steps=3, **modes)


@pytest.mark.parametrize("heads,kv_heads,batch", [
    (8, 8, 40),    # 320 heads: four-wave workgroups, two per CU
    (8, 8, 70),    # 560 heads: two-wave workgroups, four per CU
    (6, 2, 60),    # 360 grouped-query heads (G = 3, always one workgroup per head): four waves
    (6, 2, 100),   # 600 of them: two waves
])
def test_more_heads_than_compute_units(heads, kv_heads, batch):
    # with more heads than CUs the one-workgroup-per-head attention runs smaller workgroups so that
    # several fit a CU; few tiles per wave and a ragged last tile
    w = wl.WORKLOADS["llada8b_layer"].scaled(batch=batch, n_q_heads=heads, n_kv_heads=kv_heads, prompt=333, gen=64)
    _run_block(w, n_steps=3)


def test_fused_row_statistics_ignore_dominant_block_keys():
    # At the cache-update step the dense attention also supplies the scoring softmax's row statistics,
    # which run over the candidates only.  Here every query's own block key dominates its attention
    # row by about e^90 (k = 8 q): statistics taken relative to the attention's reference, or
    # including the block's keys, would underflow to zero scores.  Multi-head, grouped-query per-head
    # and grouped-query shared-tile kernels, block off the tile grid.
    _note("[case] fused row statistics under dominant block keys")
    base = wl.WORKLOADS["dream7b_gqa"].scaled(prompt=333, gen=64)
    cases = [wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=4, n_kv_heads=4, prompt=300, gen=64), base,
             _at_shared_kernel_batch(base, B.SDLLM_CALL_UPDATE)]   # dense step: 13 tiles
    for w in cases:
        inp = wl.make_block_inputs(w, n_steps=2, device=DEV)
        shape = U.shape_for(w)
        gl = U.GpuLayer(shape, DEV)
        o, b, G = inp["block_off"], w.block, w.group
        k_full, v_full = inp["k_full"], inp["v_full"]
        rows = sorted({0, w.batch - 1})
        for t in range(2):
            q = inp["q"][t].contiguous()
            k_full[:, :, o:o + b] = 8 * q[:, ::G]          # exact in bf16 (power of two)
            v_full[:, :, o:o + b] = inp["v_blk"][t]
            assert gl.block_step(t, 1, q, k_full, v_full) == t
            U.assert_close(gl.out[rows], U.oracle_attention_batch(q[rows], k_full[rows], v_full[rows]), w.dtype, f"dense step {t}")
        _check_selected_rows(gl, shape, w, q, k_full, o, b, rows)


@pytest.mark.parametrize("prompt", [700, 9300])   # selection in one workgroup per segment / in two launches
def test_block_step_replays_identically_from_a_hip_graph(prompt):
    # the library only enqueues kernels (no allocation, no memset, no host sync), so a block step can
    # be captured; every replay must reproduce the eager result, with eager work in between
    _note(f"[case] HIP graph capture / replay, prompt {prompt}")
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=8, n_kv_heads=8, prompt=prompt, gen=96)
    inp = wl.make_block_inputs(w, n_steps=3, device=DEV)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    q1, q2 = inp["q"][1].contiguous(), inp["q"][2].contiguous()
    kb, vb = inp["k_blk"][2].contiguous(), inp["v_blk"][2].contiguous()
    gl.block_step(1, 1, q1, inp["k_full"], inp["v_full"])
    eager_idx, eager_kc = gl.idx.clone(), gl.k_cache.clone()
    gl.block_step(2, 1, q2, kb, vb)
    eager_out = gl.out.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.sdllm_block_step(shape, 1, 1, q1, inp["k_full"], inp["v_full"], gl.idx, gl.k_cache, gl.v_cache, gl.out, gl.ws)
        B.sdllm_block_step(shape, 2, 1, q2, kb, vb, gl.idx, gl.k_cache, gl.v_cache, gl.out, gl.ws)
    for rep in range(3):
        gl.idx.fill_(-1); gl.k_cache.zero_(); gl.out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(gl.idx, eager_idx), rep
        assert torch.equal(gl.k_cache, eager_kc), rep
        assert torch.equal(gl.out, eager_out), rep
        # eager work between replays
        gl.block_step(0, 1, q1, inp["k_full"], inp["v_full"])


def test_very_long_segment_takes_the_streaming_select_variant():
    # more than 36 864 candidates in one segment: the select kernel re-reads the pooled row instead
    # of holding it in registers; the scoring runs on the MFMA path with a single head
    _note("[case] 40k-candidate segment")
    w = wl.WORKLOADS["dream_long"].scaled(n_q_heads=2, n_kv_heads=1, prompt=40000, gen=64, retention=0.3, sink=16)
    inp = wl.make_block_inputs(w, n_steps=2, device=DEV)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    q = inp["q"][1].contiguous()
    idx, pooled, score = gl.score_select(q, inp["k_full"])
    idx_orc, pooled_orc, score_orc = U.oracle_score_select(shape, q, inp["k_full"])
    np.testing.assert_allclose(score.cpu().double().numpy(), score_orc, rtol=3e-5, atol=1e-12)
    ties = U.compare_index_rows(idx[0, 0], idx_orc[0, 0], pooled_orc[0, 0], w.seq_len, inp["block_off"], w.block,
                                U.ranked_segments(shape))
    _note(f"[done] ties in band: {ties}")
    # same result without asking for the pooled row back
    idx2, _, _ = gl.score_select(q, inp["k_full"], want_scores=False)
    assert (idx2 == idx).all()


def test_compaction_never_leaves_the_source_tensor():
    # positions outside [0, L) in the index buffer are clamped, not followed
    _note("[case] compact with out-of-range indices")
    w = wl.WORKLOADS["llada8b_layer"].scaled(n_q_heads=2, n_kv_heads=2, prompt=96, gen=64)
    shape = U.shape_for(w)
    gl = U.GpuLayer(shape, DEV)
    k = torch.randn(w.batch, w.n_kv_heads, w.seq_len, w.head_dim, device=DEV).bfloat16()
    v = torch.randn_like(k.float()).bfloat16()
    idx = torch.randint(0, w.seq_len, (w.batch, w.n_kv_heads, gl.k_total), device=DEV, dtype=torch.int32)
    idx[0, 0, 0] = -7
    idx[0, 1, 3] = 2 ** 30
    B.sdllm_compact_kv(shape, k, v, idx, gl.k_cache, gl.v_cache)
    torch.cuda.synchronize()
    clamped = idx.long().clamp(0, w.seq_len - 1)
    want = torch.gather(k, 2, clamped[..., None].expand(-1, -1, -1, w.head_dim))
    assert torch.equal(gl.k_cache[:, :, :gl.k_total], want)


def test_block_step_on_sequence_major_views():
    # every tensor stored [B, rows, H, d] (the layout a fused QKV projection produces) and passed as
    # [B, H, rows, d] views through the stride fields; GQA so that scoring, selection, compaction and
    # both attention kernels all see non-trivial strides
    _note("[case] block_step on [B, rows, H, d] storage")
    w = wl.WORKLOADS["dream7b_gqa"].scaled(batch=2, prompt=500, gen=96)
    inp = wl.make_block_inputs(w, n_steps=3, device=DEV)
    o, b, d = inp["block_off"], w.block, w.head_dim

    def seq_major(t):   # same values, [B, rows, H, d] storage
        return t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)

    k_full, v_full = seq_major(inp["k_full"]), seq_major(inp["v_full"])
    q = [seq_major(inp["q"][t]) for t in range(3)]
    kb, vb = seq_major(inp["k_blk"][2]), seq_major(inp["v_blk"][2])
    base = U.shape_for(w)
    k_total, _, _ = B.sdllm_retained_count(base)
    k_cache = torch.zeros(w.batch, k_total + 5, w.n_kv_heads, d, device=DEV, dtype=torch.bfloat16).permute(0, 2, 1, 3)
    v_cache = torch.zeros_like(k_cache.permute(0, 2, 1, 3)).permute(0, 2, 1, 3)
    out = torch.zeros(w.batch, b, w.n_q_heads, d, device=DEV, dtype=torch.bfloat16).permute(0, 2, 1, 3)
    shape = B.make_shape(batch=w.batch, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, head_dim=d, seq_len=w.seq_len,
                         block_off=o, block_len=b, dtype=B.SDLLM_BF16, retention=w.retention, pool_kernel=w.pool_kernel,
                         q_stride=B.strides_of(q[0]), kv_stride=B.strides_of(k_full), blk_stride=B.strides_of(kb),
                         cache_stride=B.strides_of(k_cache), out_stride=B.strides_of(out))
    idx = torch.zeros(w.batch, w.n_kv_heads, k_total, device=DEV, dtype=torch.int32)
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_BLOCK_STEP), dtype=torch.uint8, device=DEV)
    assert B.sdllm_block_step(shape, 1, 1, q[1], k_full, v_full, idx, k_cache, v_cache, out, ws) == 1
    torch.cuda.synchronize()
    U.assert_close(out, U.oracle_attention_batch(q[1], k_full, v_full), "bf16", "dense, strided")
    idx_orc, pooled_orc, _ = U.oracle_score_select(shape, q[1], k_full)
    ig = idx.cpu().numpy().astype(np.int64)
    for bi in range(w.batch):
        for g in range(w.n_kv_heads):
            U.compare_index_rows(ig[bi, g], idx_orc[bi, g], pooled_orc[bi, g], w.seq_len, o, b, U.ranked_segments(shape))
    ex = idx.long()[..., None].expand(-1, -1, -1, d)
    assert torch.equal(k_cache[:, :, :k_total], torch.gather(k_full, 2, ex))
    assert torch.equal(v_cache[:, :, :k_total], torch.gather(v_full, 2, ex))
    assert B.sdllm_block_step(shape, 2, 1, q[2], kb, vb, idx, k_cache, v_cache, out, ws) == 2
    torch.cuda.synchronize()
    ref = U.oracle_attention_batch(q[2], torch.cat([k_cache[:, :, :k_total], kb], 2), torch.cat([v_cache[:, :, :k_total], vb], 2))
    U.assert_close(out, ref, "bf16", "sparse, strided")


@pytest.mark.parametrize("Bt,Hq,Hkv,n_cached", [(1, 4, 4, 700), (2, 14, 2, 333), (2, 28, 4, 500), (2, 28, 4, 1300), (160, 28, 4, 300)])
def test_attention_with_peaked_softmax_and_late_maxima(Bt, Hq, Hkv, n_cached):
    # logits with a spread of several dozen (softmax close to one-hot) and, per row, a dominant key
    # planted in a late tile: the running softmax reference has to jump by far more than its slack
    # after many tiles have been accumulated, in the kernel for small calls, the one that streams tiles into LDS (500 keys), the
    # per-head one with key splits (1300) and (last case) the shared-tile grouped-query kernel
    _note(f"[case] peaked softmax B={Bt} Hq={Hq} Hkv={Hkv} n_cached={n_cached}")
    torch.manual_seed(77 + n_cached)
    b, d = 32, 128
    shape = B.make_shape(batch=Bt, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=4096, block_off=2048,
                         block_len=b, dtype=B.SDLLM_BF16, cache_rows=n_cached)
    q = (4.0 * torch.randn(Bt, Hq, b, d, device=DEV)).bfloat16()
    kc = (4.0 * torch.randn(Bt, Hkv, n_cached, d, device=DEV)).bfloat16()
    vc = torch.randn(Bt, Hkv, n_cached, d, device=DEV).bfloat16()
    kb = (4.0 * torch.randn(Bt, Hkv, b, d, device=DEV)).bfloat16()
    vb = torch.randn(Bt, Hkv, b, d, device=DEV).bfloat16()
    # a key aligned with the first query head's row 0, three quarters of the way through the cache
    G = Hq // Hkv
    kc[:, :, (3 * n_cached) // 4] = (1.5 * q[:, ::G, 0].float()).bfloat16()
    out = torch.zeros(Bt, Hq, b, d, device=DEV, dtype=torch.bfloat16)
    ws = torch.empty(B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n_cached), dtype=torch.uint8, device=DEV)
    B.sdllm_sparse_attn(shape, q, kc, vc, n_cached, kb, vb, out, ws)
    torch.cuda.synchronize()
    bs = [0, Bt - 1] if Bt > 2 else list(range(Bt))
    ref = U.oracle_attention_batch(q[bs], torch.cat([kc[bs], kb[bs]], 2), torch.cat([vc[bs], vb[bs]], 2))
    U.assert_close(out[bs], ref, "bf16", "peaked softmax")
    assert torch.isfinite(out.float()).all()
