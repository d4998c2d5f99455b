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


def dense_groups(heads, L, **more):
    shape = dict(batch=1, n_q_heads=heads, n_kv_heads=heads, head_dim=128, seq_len=L, block_off=0, block_len=32, dtype=B.SDLLM_BF16)
    shape.update(more)
    shape = B.make_shape(**shape)
    return B.sdllm_launch_plan(shape, DENSE).key_groups, B.sdllm_dense_tail_groups(shape)


# Beyond 256 positions, where the ring kernels' costs decide: the sizes at which they and those of the kernels before them differ, with the
# groups of a last round that is a launch of its own, whose other rounds have one group.
@pytest.mark.parametrize("heads,L,groups", [(84, 800, (1, 2)), (140, 800, (2, 0)), (112, 1025, (2, 0)), (56, 1277, (1, 4)), (64, 1277, (1, 4)),
                                            (40, 1537, (1, 4)), (40, 1793, (1, 4)), (32, 2049, (1, 4)), (8, 2049, (2, 0)), (28, 1181, (1, 0)),
                                            (84, 1277, (1, 0)), (28, 300, (4, 0)), (56, 300, (2, 0)), (224, 300, (1, 0))])
def test_key_groups_of_the_ring_kernels(heads, L, groups):
    assert dense_groups(heads, L) == groups


# Workgroups left after whole rounds of 256 (1, 64, 65, 128, 129) and the tiles from which that pays
@pytest.mark.parametrize("heads,L,groups", [(205, 1100, (1, 4)), (160, 512, (1, 4)), (160, 300, (2, 0)), (107, 768, (1, 2)), (128, 768, (1, 2)), (128, 736, (1, 0)),
                                            (77, 1100, (1, 0)), (192, 600, (2, 0)), (256, 1200, (1, 0)), (160, 256, (1, 0)),
                                            # a last block of at most 128 rows, without which two groups throughout need a round less
                                            (56, 1152, (2, 0)), (56, 1153, (1, 4)), (24, 2599, (2, 0)), (60, 3120, (2, 0)), (112, 1153, (1, 4))])
def test_last_round_of_whole_sequences(heads, L, groups):
    assert dense_groups(heads, L) == groups
    assert dense_groups(heads, L, head_dim=64)[1] == dense_groups(heads, L, dtype=B.SDLLM_F32)[1] == 0      # the general kernel


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


# Groups of 7 and 8 heads: the shared-tile kernel from the second tile count on, not yet at the first (short of the line by no
# more than its slope).  Sparse steps and dense rows alike.
@pytest.mark.parametrize("batch,q_heads,kv_heads,below,from_", [
    (5, 28, 4, 128, 129), (6, 28, 4, 127, 128), (10, 16, 2, 123, 124), (7, 28, 4, 138, 139), (8, 28, 4, 149, 150), (9, 28, 4, 160, 161),
    (8, 32, 4, 162, 163),                                                                  # up to one workgroup per CU
    (3, 28, 4, 482, 483), (4, 28, 4, 299, 300), (8, 16, 2, 324, 325), (2, 28, 4, 598, 599), (3, 32, 4, 312, 313),   # with key splits
    (10, 28, 4, 65, 66), (12, 28, 4, 65, 66), (16, 28, 4, 74, 75), (18, 28, 4, 83, 84), (32, 16, 2, 85, 86),          # up to two
    (19, 28, 4, 39, 40), (20, 32, 4, 39, 40), (32, 28, 4, 39, 40), (17, 32, 4, 39, 40),    # up to four, filling the chip
    (22, 28, 4, 49, 50), (24, 32, 4, 49, 50), (26, 28, 4, 49, 50),                         # ... and not
])
def test_shared_tile_kernel_from_the_measured_line_on(batch, q_heads, kv_heads, below, from_):
    for call in (SPARSE, FULL):
        assert plan(call, batch, q_heads, kv_heads, below).kernel != SHARED
        assert plan(call, batch, q_heads, kv_heads, from_).kernel == SHARED


@pytest.mark.parametrize("batch,q_heads,kv_heads", [(37, 28, 4), (33, 32, 4), (129, 8, 1), (65, 16, 2), (150, 7, 1)])
def test_shared_tile_kernel_always_beyond_four_heads_per_cu(batch, q_heads, kv_heads):
    for tiles in (2, 5, 20, 35, 60):
        for call in (SPARSE, FULL, UPDATE):
            assert route(call, batch, q_heads, kv_heads, tiles, block_off=min(64, 32 * tiles - 32)) == (SHARED, 1)


def test_shared_tile_kernel_at_update_steps():
    for batch, q_heads, kv_heads, below, from_ in ((20, 32, 4, 29, 30), (32, 28, 4, 29, 30), (22, 28, 4, 45, 46), (24, 32, 4, 45, 46)):
        assert plan(UPDATE, batch, q_heads, kv_heads, below, block_off=64).kernel != SHARED
        assert plan(UPDATE, batch, q_heads, kv_heads, from_, block_off=64).kernel == SHARED


def test_scratch_beyond_a_callers_gives_way_up_to_5000_tiles():
    # 34 x 16/2 heads x 48 tiles: 26 MB of partials on the faster kernel, none on the other.  A null pointer is enough to see
    # that the plan is accepted: nothing but the missing output is wrong with these calls.
    import ctypes
    shape = B.make_shape(batch=34, n_q_heads=16, n_kv_heads=2, head_dim=128, seq_len=4096, block_off=0, block_len=32, dtype=B.SDLLM_BF16)
    n = 32 * 47
    need = B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SPARSE_ATTN, n)
    assert B.sdllm_launch_plan(shape, SPARSE, n).kernel == SHARED and need > B.SDLLM_STATIC_SCRATCH_BYTES
    fake, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(None)
    call = lambda k: B.load().sdllm_sparse_attn_noalloc(ctypes.byref(shape), fake, fake, fake, k, fake, fake, null, null)
    assert call(32 * 200) == B.SDLLM_ERR_STATIC_LIMIT
    assert call(n) in (B.SDLLM_ERR_INVALID_ARG, B.SDLLM_ERR_HIP)   # past the limit check (without a GPU the array has no address)


@pytest.mark.parametrize("call", [SPARSE, FULL])
def test_small_calls_stay_unsplit_up_to_the_measured_line(call):
    for batch, q_heads, kv_heads, last in ((1, 8, 2, 22), (1, 12, 4, 22), (1, 28, 4, 22), (1, 32, 8, 22), (2, 28, 4, 33), (2, 32, 8, 33),
                                           (4, 28, 4, 48), (4, 24, 4, 48), (8, 16, 2, 48), (3, 32, 8, 38), (8, 12, 4, 38), (4, 32, 8, 38)):
        assert route(call, batch, q_heads, kv_heads, last) == (STREAM, 1)
        kernel, splits = route(call, batch, q_heads, kv_heads, last + 1)
        assert kernel == PER_HEAD and splits > 1


def test_stream_kernel_with_more_heads_than_cus():
    for batch, q_heads, kv_heads, tiles, want in ((10, 28, 4, 35, PER_HEAD), (10, 28, 4, 36, STREAM), (17, 16, 2, 36, STREAM), (9, 32, 4, 36, PER_HEAD),
                                                  (12, 28, 4, 52, PER_HEAD), (9, 32, 4, 52, STREAM), (26, 16, 2, 51, PER_HEAD),
                                                  (26, 16, 2, 52, STREAM), (20, 28, 4, 36, PER_HEAD), (20, 16, 4, 60, PER_HEAD)):
        for call in (SPARSE, FULL):
            assert plan(call, batch, q_heads, kv_heads, tiles).kernel == want
    # with the scoring's statistics
    for batch, q_heads, kv_heads, tiles, want in ((12, 28, 4, 36, STREAM), (12, 28, 4, 35, PER_HEAD), (22, 28, 4, 40, STREAM), (20, 16, 4, 60, PER_HEAD)):
        assert plan(UPDATE, batch, q_heads, kv_heads, tiles, block_off=64).kernel == want
        assert plan(UPDATE, batch, q_heads, kv_heads, tiles, block_off=64, score_mode=B.SDLLM_LOGIT_MEAN).kernel == PER_HEAD


def test_launches_of_the_general_kernel_stay_below_two_to_the_32_threads():
    # all rows of 65 535 fp32 heads of 64 x 8224 positions (an output of 138 GB): 33 684 990 workgroups
    p = plan(DENSE, 65535, 1, 1, 257, dtype=B.SDLLM_F32, head_dim=64)
    assert p.kernel == GENERAL and 65535 * 514 * p.waves * 64 < 1 << 32
    assert plan(DENSE, 1, 8, 8, 256, dtype=B.SDLLM_F32, head_dim=64).waves > 1


# Small calls that go to the kernel that fetches all tiles of a workgroup at once, ahead of the routes above, with how many splits.
@pytest.mark.parametrize("batch,q_heads,kv_heads,tiles,splits", [
    (1, 1, 1, 1, 1), (8, 28, 4, 9, 1), (8, 32, 8, 9, 1), (9, 32, 8, 2, 0), (8, 32, 32, 6, 1), (8, 32, 32, 7, 0), (7, 32, 32, 9, 0),
    (1, 136, 136, 9, 1), (1, 137, 137, 9, 0), (1, 176, 176, 8, 1), (1, 177, 177, 8, 0), (1, 200, 200, 7, 1), (1, 201, 201, 7, 0), (1, 240, 240, 5, 1),
    (8, 32, 32, 5, 0), (1, 216, 216, 4, 1), (8, 32, 32, 4, 0), (8, 32, 32, 3, 1), (8, 32, 32, 1, 1), (8, 32, 16, 9, 1),
    (1, 16, 2, 10, 4), (1, 28, 4, 10, 0), (1, 28, 4, 11, 3), (1, 32, 32, 10, 0), (1, 32, 32, 11, 0), (1, 40, 40, 11, 0), (1, 44, 44, 12, 3), (1, 56, 56, 14, 0), (1, 56, 56, 15, 3),
    (2, 32, 32, 15, 0), (2, 32, 32, 16, 2), (1, 72, 72, 21, 0), (5, 16, 16, 21, 0), (5, 16, 16, 22, 0), (3, 32, 32, 28, 0),
    (1, 28, 28, 12, 3), (1, 28, 28, 13, 0), (1, 28, 28, 15, 3), (1, 32, 32, 14, 0), (1, 32, 32, 15, 3), (1, 38, 38, 14, 0), (1, 40, 40, 12, 3),
    # multi-head with many bytes
    (1, 18, 18, 100, 12), (1, 20, 20, 64, 8), (1, 20, 20, 65, 0), (1, 28, 28, 45, 6), (1, 28, 28, 46, 0), (1, 32, 32, 40, 5), (1, 32, 32, 41, 0), (1, 42, 42, 43, 5), (1, 42, 42, 44, 0),
    (2, 32, 32, 32, 4), (2, 32, 32, 33, 0), (1, 48, 24, 17, 0), (1, 48, 24, 18, 3),
    (1, 40, 8, 14, 0), (1, 40, 8, 15, 3), (2, 28, 4, 17, 0), (2, 28, 4, 18, 3), (3, 16, 2, 16, 0), (3, 16, 2, 17, 3), (2, 32, 8, 23, 0), (2, 32, 8, 24, 3), (5, 16, 2, 24, 0),
    (1, 28, 4, 69, 8), (1, 28, 4, 81, 9), (1, 28, 4, 82, 0), (1, 32, 8, 72, 8), (1, 32, 8, 73, 0), (1, 2, 2, 288, 32), (1, 2, 2, 289, 0),
    (1, 1, 1, 40, 14), (1, 1, 1, 56, 14), (1, 1, 1, 140, 24),      # as many as the merge folds at once
])
def test_small_calls_whose_tiles_are_fetched_at_once(batch, q_heads, kv_heads, tiles, splits):
    shape = dict(batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=128, seq_len=32 * tiles, block_off=0, block_len=32, dtype=B.SDLLM_BF16)
    assert B.sdllm_burst_splits(B.make_shape(**shape), SPARSE, 32 * (tiles - 1)) == splits
    assert B.sdllm_burst_splits(B.make_shape(**shape), FULL) == splits
    for call in (UPDATE, DENSE):
        assert B.sdllm_burst_splits(B.make_shape(**shape), call) == 0
    for more in (dict(dtype=B.SDLLM_F32), dict(head_dim=64), dict(block_len=16)):
        assert B.sdllm_burst_splits(B.make_shape(**{**shape, **more}), SPARSE, 32 * (tiles - 1)) == 0
    if splits > 1:   # never more partials than the static scratch holds
        assert batch * q_heads * splits * 16640 <= B.SDLLM_STATIC_SCRATCH_BYTES


# Column pass of other block lengths: blocks as heads of the kernels for 32 rows, with one block per KV head from 64 of them on
@pytest.mark.parametrize("batch,heads,kv_heads,L,more,kernel", [
    (1, 8, 8, 600, dict(block_len=32), B.SDLLM_COLUMNS_32), (1, 14, 2, 600, dict(block_len=16), B.SDLLM_COLUMNS_BLOCKS),
    (2, 32, 32, 1280, dict(block_len=64), B.SDLLM_COLUMNS_BLOCKS), (1, 5, 1, 300, dict(block_len=64), B.SDLLM_COLUMNS_GENERAL),
    (1, 8, 8, 600, dict(block_len=64, score_mode=B.SDLLM_LOGIT_MEAN), B.SDLLM_COLUMNS_BLOCKS),
    (1, 8, 8, 600, dict(block_len=48, score_mode=B.SDLLM_LOGIT_MEAN), B.SDLLM_COLUMNS_GENERAL),
    (1, 8, 8, 600, dict(block_len=64, head_dim=64), B.SDLLM_COLUMNS_GENERAL), (1, 8, 8, 600, dict(block_len=64, dtype=B.SDLLM_F32), B.SDLLM_COLUMNS_GENERAL),
    (7, 8, 8, 600, dict(block_len=16), B.SDLLM_COLUMNS_GENERAL), (8, 8, 8, 100, dict(block_len=16), B.SDLLM_COLUMNS_BLOCKS),
    (7, 8, 8, 600, dict(block_len=33), B.SDLLM_COLUMNS_BLOCKS),
])
def test_column_pass_of_other_block_lengths(batch, heads, kv_heads, L, more, kernel):
    shape = dict(batch=batch, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, seq_len=L, block_off=L // 2, dtype=B.SDLLM_BF16)
    assert B.sdllm_column_kernel(B.make_shape(**{**shape, **more})) == kernel
