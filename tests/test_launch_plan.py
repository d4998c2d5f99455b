"""Which kernel an attention call runs, on either side of the lines of the launch rules.  The lines and what was measured
on both sides of them stand at the rules in csrc/api.hip; here they are pinned, and the GPU tests that are meant for one
kernel ask sdllm_launch_plan whether they reach it."""
import pytest

from paper_2508_02558_amd import binding as B

GENERAL, PER_HEAD, SHARED, STREAM = (B.SDLLM_KERNEL_GENERAL, B.SDLLM_KERNEL_PER_HEAD, B.SDLLM_KERNEL_SHARED_TILE,
                                     B.SDLLM_KERNEL_STREAM)
SPARSE, FULL, UPDATE, DENSE = B.SDLLM_CALL_SPARSE, B.SDLLM_CALL_FULL, B.SDLLM_CALL_UPDATE, B.SDLLM_CALL_DENSE


def plan(call, batch, q_heads, kv_heads, tiles, **more):
    """`tiles` 32-key tiles per head: for a sparse step one of them is the block's."""
    shape = dict(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=32 * tiles, block_off=0, block_len=32,
                 dtype=B.SDLLM_BF16)
    shape.update(more)
    return B.sdllm_launch_plan(B.make_shape(**shape), call, 32 * (tiles - 1) if call == SPARSE else 0)


def route(*args, **more):
    p = plan(*args, **more)
    return p.kernel, p.key_splits


def test_types_and_sizes_that_only_the_general_kernel_takes():
    for more in (dict(dtype=B.SDLLM_F32), dict(head_dim=64), dict(block_len=16), dict(block_len=33)):
        assert plan(SPARSE, 1, 4, 2, 10, **more).kernel == GENERAL
        assert plan(FULL, 1, 4, 2, 10, **more).kernel == GENERAL
    for more in (dict(dtype=B.SDLLM_F32), dict(head_dim=64)):
        assert plan(DENSE, 1, 4, 2, 10, **more).kernel == GENERAL
    assert plan(DENSE, 1, 4, 2, 10, block_len=16).kernel == B.SDLLM_KERNEL_DENSE


@pytest.mark.parametrize("heads,L,groups", [(2, 129, 1), (2, 161, 4), (2, 97, 4), (28, 735, 2), (28, 1277, 1), (8, 1277, 4), (256, 4352, 1)])
def test_key_groups_of_whole_sequences(heads, L, groups):
    shape = B.make_shape(batch=1, n_q_heads=heads, n_kv_heads=heads, head_dim=128, seq_len=L, block_off=0, block_len=32, dtype=B.SDLLM_BF16)
    assert B.sdllm_launch_plan(shape, DENSE).key_groups == groups


def test_a_call_or_plan_that_is_not_there_is_rejected():
    for call, n_cached in ((-1, 0), (4, 0), (SPARSE, -1)):
        with pytest.raises(B.SdllmError):
            B.sdllm_launch_plan(B.make_shape(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, seq_len=64, block_off=0, block_len=32,
                                             dtype=B.SDLLM_BF16), call, n_cached)


@pytest.mark.parametrize("batch,q_heads,kv_heads,tiles,full,update", [
    (1, 28, 4, 13, (STREAM, 1), (STREAM, 1)),
    (1, 28, 4, 20, (STREAM, 1), (PER_HEAD, 2)),
    (1, 12, 4, 22, (STREAM, 1), (PER_HEAD, 3)),
    (2, 28, 4, 30, (STREAM, 1), (PER_HEAD, 2)),
    (4, 28, 4, 38, (STREAM, 1), (PER_HEAD, 2)),
    (8, 16, 2, 24, (STREAM, 1), (STREAM, 1)),
    (1, 8, 8, 16, (STREAM, 1), (PER_HEAD, 2)),
])
def test_key_splits_of_an_update_step_whose_merge_costs_nothing(batch, q_heads, kv_heads, tiles, full, update):
    assert route(FULL, batch, q_heads, kv_heads, tiles) == full
    for mode in (B.SDLLM_SOFTMAX_MEAN, B.SDLLM_LOGIT_MEAN):
        assert route(UPDATE, batch, q_heads, kv_heads, tiles, block_off=64, score_mode=mode) == update
    # nothing to compact: the merge is a launch of its own
    assert route(UPDATE, batch, q_heads, kv_heads, tiles, block_off=64, retention=0.0) == full
