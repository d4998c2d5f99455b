"""Host-side checks of the C ABI that need no GPU: exported symbols, struct layout, the host
logic (retained counts, cache-state schedule, workspace sizing) and argument rejection."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

from oracle import sdllm_oracle as orc
from paper_2508_02558_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INCLUDE = os.path.join(ROOT, "include")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2508_02558_amd.build import build_library
        build_library(verbose=False)
    return B.load()


def _declared_functions():
    names = set()
    for header in sorted(os.listdir(INCLUDE)):
        if header.endswith(".h"):
            text = open(os.path.join(INCLUDE, header)).read()
            text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
            names.update(re.findall(r"\b(sdllm_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_every_declared_symbol_is_exported(lib):
    declared = _declared_functions()
    assert set(declared) == set(B.EXPORTED)
    for name in declared:
        assert hasattr(lib, name), name


def test_struct_layout_matches_the_header(tmp_path):
    src = tmp_path / "layout.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "sdllm.h"\n'
                   'int main(void){printf("%zu %zu %zu %zu %zu\\n", sizeof(sdllm_shape_t),'
                   ' offsetof(sdllm_shape_t, softmax_scale), offsetof(sdllm_shape_t, retention),'
                   ' offsetof(sdllm_shape_t, q_stride), offsetof(sdllm_shape_t, out_stride));return 0;}\n')
    exe = tmp_path / "layout"
    subprocess.check_call(["gcc", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    got = [int(x) for x in subprocess.check_output([str(exe)]).split()]
    S = B.sdllm_shape_t
    assert got == [ctypes.sizeof(S), S.softmax_scale.offset, S.retention.offset, S.q_stride.offset, S.out_stride.offset]


def _shape(**kw):
    base = dict(batch=1, n_q_heads=2, n_kv_heads=2, head_dim=64, seq_len=160, block_off=64, block_len=32,
                dtype=B.SDLLM_F32, retention=0.5, pool_kernel=3)
    base.update(kw)
    return B.make_shape(**base)


def test_retained_count_agrees_with_golden_table_and_oracle(lib, golden):
    for r, n, ceil_k, floor_k in golden("retained_count_table.txt"):
        n = int(n)
        # prefix of n tokens, block right after it, no suffix
        for rounding, want in ((B.SDLLM_CEIL, int(ceil_k)), (B.SDLLM_FLOOR, int(floor_k))):
            s = _shape(seq_len=n + 32, block_off=n, retention=float(r), k_rounding=rounding)
            kt, kp, ks = B.sdllm_retained_count(s)
            assert (kt, kp, ks) == (want, want, 0)
    s = _shape()
    assert B.sdllm_retained_count(s) == (64, 32, 32)
    s = _shape(select_mode=B.SDLLM_JOINT, k_rounding=B.SDLLM_FLOOR)
    assert B.sdllm_retained_count(s) == (64, -1, -1)
    s = _shape(evict_scope=B.SDLLM_EVICT_PREFIX_ONLY)
    assert B.sdllm_retained_count(s) == (32 + 64, 32, 64)
    for r in (0.0, 0.1, 0.3, 0.7, 0.9, 1.0):
        for n in (0, 1, 7, 10, 33):
            s = _shape(seq_len=n + 32 + 5, block_off=n, retention=r)
            assert B.sdllm_retained_count(s)[1:] == (orc.retained_count(n, r), orc.retained_count(5, r))


def test_cache_state_schedule(lib, golden):
    for delay, states in golden("cache_state_table.txt"):
        for i, st in enumerate(states.split()):
            assert B.sdllm_cache_state(i, int(delay)) == int(st)
    with pytest.raises(B.SdllmError):
        B.sdllm_cache_state(-1, 1)


def test_invalid_shapes_are_rejected(lib):
    bad = [dict(batch=0), dict(n_q_heads=3), dict(block_off=140), dict(retention=1.5), dict(retention=-0.1),
           dict(pool_kernel=2), dict(pool_kernel=0), dict(dtype=7), dict(score_mode=3), dict(select_mode=2),
           dict(k_rounding=5), dict(pool_mode=2), dict(evict_scope=2), dict(q_stride=(4096, 2048, 63)),
           dict(softmax_scale=-1.0), dict(retention=float("nan"))]
    for kw in bad:
        with pytest.raises(B.SdllmError) as ei:
            B.sdllm_retained_count(_shape(**kw))
        assert ei.value.status == B.SDLLM_ERR_INVALID_ARG, kw
    for kw in (dict(head_dim=96), dict(block_len=65, seq_len=300)):
        with pytest.raises(B.SdllmError) as ei:
            B.sdllm_retained_count(_shape(**kw))
        assert ei.value.status == B.SDLLM_ERR_UNSUPPORTED, kw
    assert B.error_string(0) == "ok" and "workspace" in B.error_string(B.SDLLM_ERR_WORKSPACE)
    assert B.sdllm_version() >= 100


def test_null_pointers_and_small_workspace_are_rejected_before_any_launch(lib):
    s = _shape()
    z = ctypes.c_void_p(None)
    sp = ctypes.byref(s)
    assert lib.sdllm_score_select(sp, z, z, z, z, z, z, 0, z) == B.SDLLM_ERR_INVALID_ARG
    assert lib.sdllm_compact_kv(sp, z, z, z, z, z, z) == B.SDLLM_ERR_INVALID_ARG
    assert lib.sdllm_sparse_attn(sp, z, z, z, 4, z, z, z, z, 0, z) == B.SDLLM_ERR_INVALID_ARG
    assert lib.sdllm_block_step(sp, 0, 1, z, z, z, z, z, z, z, z, 0, z, None) == B.SDLLM_ERR_WORKSPACE
    # a fake but aligned pointer value is enough to get past the pointer checks (nothing is enqueued
    # when the workspace is too small)
    fake = ctypes.c_void_p(0x1000)
    assert lib.sdllm_score_select(sp, fake, fake, fake, z, z, fake, 16, z) == B.SDLLM_ERR_WORKSPACE
    assert lib.sdllm_score_select(sp, fake, fake, fake, z, z, ctypes.c_void_p(0x1008), 1 << 30, z) == B.SDLLM_ERR_WORKSPACE
    assert lib.sdllm_sparse_attn(sp, ctypes.c_void_p(0x1004), z, z, 0, fake, fake, fake, z, 0, z) == B.SDLLM_ERR_INVALID_ARG
    assert lib.sdllm_sparse_attn(sp, fake, z, z, -1, fake, fake, fake, z, 0, z) == B.SDLLM_ERR_INVALID_ARG


@pytest.mark.parametrize("heads,kv_heads,n_cached,splits", [(32, 32, 1120, 5), (28, 4, 1760, 8)])
def test_a_sparse_step_asks_for_the_same_workspace_whichever_kernel_would_take_it(lib, heads, kv_heads, n_cached, splits):
    # the kernel for small calls would make do with four and seven splits here
    s = B.make_shape(batch=1, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, seq_len=16384, block_off=8192, block_len=32, dtype=B.SDLLM_BF16)
    assert B.sdllm_launch_plan(s, B.SDLLM_CALL_SPARSE, n_cached).key_splits == splits > B.sdllm_burst_splits(s, B.SDLLM_CALL_SPARSE, n_cached)
    fake, need = ctypes.c_void_p(0x1000), heads * splits * 32 * (128 + 2) * 4
    assert B.sdllm_workspace_bytes(s, B.SDLLM_OP_SPARSE_ATTN, n_cached) == need
    for ws, n in ((fake, need - 1), (fake, need * (splits - 1) // splits), (ctypes.c_void_p(0), need)):
        assert lib.sdllm_sparse_attn(ctypes.byref(s), fake, fake, fake, n_cached, fake, fake, fake, ws, n, ctypes.c_void_p(0)) == B.SDLLM_ERR_WORKSPACE


def test_noalloc_entry_rejects_requests_beyond_its_static_scratch(lib):
    # batch 8 of a 28/4-head shape with 8000 cached keys runs the shared-tile kernel with 8 key splits:
    # 1792 partial slots of 16.25 KB, far beyond the 8 MiB array.  Rejected on the host, nothing enqueued.
    s = B.make_shape(batch=8, n_q_heads=28, n_kv_heads=4, head_dim=128, seq_len=20000, block_off=12000, block_len=32,
                     dtype=B.SDLLM_BF16, cache_rows=8000)
    assert B.sdllm_workspace_bytes(s, B.SDLLM_OP_SPARSE_ATTN, 8000) > B.SDLLM_STATIC_SCRATCH_BYTES
    fake = ctypes.c_void_p(0x1000)
    z = ctypes.c_void_p(None)
    assert lib.sdllm_sparse_attn_noalloc(ctypes.byref(s), fake, fake, fake, 8000, fake, fake, fake, z) == B.SDLLM_ERR_STATIC_LIMIT
    assert "static scratch" in B.error_string(B.SDLLM_ERR_STATIC_LIMIT)
    assert lib.sdllm_sparse_attn_noalloc(ctypes.byref(s), fake, fake, fake, -1, fake, fake, fake, z) == B.SDLLM_ERR_INVALID_ARG


def test_static_scratch_is_visible_in_the_device_image(lib, tmp_path):
    # hipGetSymbolAddress looks the array up by name in the gfx950 code object: it has to be a GLOBAL
    # symbol there (a LOCAL one makes the runtime abort on the first sdllm_sparse_attn_noalloc call)
    obj = os.path.join(ROOT, "paper_2508_02558_amd", "_build", "api.o")
    objdump, readelf = "/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readelf"
    if not (os.path.exists(obj) and os.path.exists(objdump) and os.path.exists(readelf)):
        pytest.skip("needs the build directory and the LLVM binutils")
    local = tmp_path / "api.o"
    local.write_bytes(open(obj, "rb").read())
    subprocess.check_call([objdump, "--offloading", str(local)], cwd=tmp_path, stdout=subprocess.DEVNULL)
    images = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert images, os.listdir(tmp_path)
    syms = subprocess.check_output([readelf, "--dyn-syms", str(tmp_path / images[0])], text=True)
    rows = [ln.split() for ln in syms.splitlines() if ln.strip().endswith("scratch")]
    assert rows and all(r[4] == "GLOBAL" and int(r[2]) == B.SDLLM_STATIC_SCRATCH_BYTES for r in rows), syms


def test_segments_beyond_the_selection_limit_are_rejected_before_any_launch(lib):
    # a prefix of more than 1M candidates: the selection's per-chunk tables end there
    s = B.make_shape(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, seq_len=1_200_000 + 32, block_off=1_200_000, block_len=32,
                     dtype=B.SDLLM_BF16)
    fake = ctypes.c_void_p(0x1000)
    z = ctypes.c_void_p(None)
    assert lib.sdllm_score_select(ctypes.byref(s), fake, fake, fake, z, z, fake, 1 << 40, z) == B.SDLLM_ERR_UNSUPPORTED
    ok = B.make_shape(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, seq_len=1_000_000 + 32, block_off=1_000_000, block_len=32,
                      dtype=B.SDLLM_BF16)
    assert B.sdllm_workspace_bytes(ok, B.SDLLM_OP_SCORE_SELECT) > 3 * 4 * 1_000_000   # scores + two key buffers


def test_workspace_sizes(lib):
    s = _shape()
    for op in (B.SDLLM_OP_SCORE_SELECT, B.SDLLM_OP_COMPACT_KV, B.SDLLM_OP_SPARSE_ATTN, B.SDLLM_OP_BLOCK_STEP):
        assert B.sdllm_workspace_bytes(s, op, 64) >= 256
    # split-KV partials of the MFMA path: a batch-1 LLaDA-shaped call needs room for them
    big = B.make_shape(batch=1, n_q_heads=32, n_kv_heads=32, head_dim=128, seq_len=4352, block_off=4096,
                       block_len=32, dtype=B.SDLLM_BF16)
    kt, _, _ = B.sdllm_retained_count(big)
    assert kt == 2160
    assert B.sdllm_workspace_bytes(big, B.SDLLM_OP_SPARSE_ATTN, kt) > 32 * 32 * 128 * 4
    assert B.sdllm_workspace_bytes(big, B.SDLLM_OP_BLOCK_STEP) >= B.sdllm_workspace_bytes(big, B.SDLLM_OP_SCORE_SELECT)
    with pytest.raises(B.SdllmError):
        B.sdllm_workspace_bytes(s, 9)


def sequential_step_bytes(shape, q_rows_per_block):
    """What a block step of the general kernels needs when the partials of its key splits are merged before the scoring."""
    up = lambda n: (n + 255) // 256 * 256
    blocks = shape.batch * shape.n_q_heads * -(-shape.block_len // q_rows_per_block)
    def partials(plan):
        if plan.key_splits == 1:
            return 0
        return up(blocks * plan.key_splits * q_rows_per_block * shape.head_dim * 4) + up(blocks * plan.key_splits * 2 * q_rows_per_block * 4)
    kt = B.sdllm_retained_count(shape)[0]
    update = B.sdllm_launch_plan(shape, B.SDLLM_CALL_UPDATE)
    parts = max(partials(update), partials(B.sdllm_launch_plan(shape, B.SDLLM_CALL_FULL)), partials(B.sdllm_launch_plan(shape, B.SDLLM_CALL_SPARSE, kt)))
    stats = up(blocks * update.key_splits * 2 * q_rows_per_block * 4) if shape.score_mode == B.SDLLM_SOFTMAX_MEAN else 0
    return up(max(parts, B.sdllm_workspace_bytes(shape, B.SDLLM_OP_SCORE_SELECT))) + stats


@pytest.mark.parametrize("kw,rows", [
    (dict(dtype=B.SDLLM_BF16, head_dim=128, block_len=64, n_q_heads=8, n_kv_heads=8, seq_len=1500), 32),
    (dict(dtype=B.SDLLM_BF16, head_dim=64, block_len=32, n_q_heads=4, n_kv_heads=2, seq_len=1600, score_mode=B.SDLLM_LOGIT_MEAN), 32),
    (dict(dtype=B.SDLLM_F32, head_dim=128, block_len=40, n_q_heads=6, n_kv_heads=2, seq_len=900), 16),
])
def test_block_step_takes_a_workspace_without_room_for_partials_and_scores_side_by_side(lib, kw, rows):
    s = B.make_shape(batch=1, block_off=500, **kw)
    assert B.sdllm_launch_plan(s, B.SDLLM_CALL_UPDATE).key_splits > 1
    less, full = sequential_step_bytes(s, rows), B.sdllm_workspace_bytes(s, B.SDLLM_OP_BLOCK_STEP)
    assert less < full
    fake, z = ctypes.c_void_p(0x1000), ctypes.c_void_p(None)
    # past the size check the missing queries are the error
    step = lambda n: lib.sdllm_block_step(ctypes.byref(s), 1, 1, z, fake, fake, fake, fake, fake, fake, fake, n, z, None)
    assert step(full) == step(less) == B.SDLLM_ERR_INVALID_ARG
    assert step(less - 1) == B.SDLLM_ERR_WORKSPACE
    # the 32-row kernels need it all, where it is no more than they need (with 8 heads the kernel for small calls would use more)
    m = B.make_shape(batch=1, n_q_heads=32, n_kv_heads=32, head_dim=128, seq_len=1500, block_off=500, block_len=32, dtype=B.SDLLM_BF16)
    assert B.sdllm_launch_plan(m, B.SDLLM_CALL_UPDATE).key_splits > 1
    need = B.sdllm_workspace_bytes(m, B.SDLLM_OP_BLOCK_STEP)
    assert lib.sdllm_block_step(ctypes.byref(m), 1, 1, z, fake, fake, fake, fake, fake, fake, fake, need - 1, z, None) == B.SDLLM_ERR_WORKSPACE


# Heads and cached keys of which a block step used to ask for less than its sparse step had a use for.  least: what it did ask for.
@pytest.mark.parametrize("heads,kv_heads,seq_len,least", [(16, 2, 700, 828672), (14, 2, 1500, 1452544), (8, 8, 300, 14848), (8, 8, 4500, 1261312),
                                                          (1, 1, 2500, 147712), (28, 4, 2500, 3896064), (32, 32, 4500, 4962816)])
def test_block_step_asks_for_room_for_every_split_of_a_small_call_and_takes_less(lib, heads, kv_heads, seq_len, least):
    s = B.make_shape(batch=1, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, seq_len=seq_len, block_off=200, block_len=32, dtype=B.SDLLM_BF16)
    kept, need = B.sdllm_retained_count(s)[0], B.sdllm_workspace_bytes(s, B.SDLLM_OP_BLOCK_STEP)
    splits = [B.sdllm_burst_splits(s, call, kept) for call in (B.SDLLM_CALL_SPARSE, B.SDLLM_CALL_FULL)]
    assert need >= max(n if n > 1 else 0 for n in splits) * heads * 32 * (128 + 2) * 4
    assert need >= B.sdllm_workspace_bytes(s, B.SDLLM_OP_SPARSE_ATTN, kept)
    fake, z = ctypes.c_void_p(0x1000), ctypes.c_void_p(None)
    step = lambda n: lib.sdllm_block_step(ctypes.byref(s), 1, 1, z, fake, fake, fake, fake, fake, fake, fake, n, z, None)
    assert step(need) == step(least) == B.SDLLM_ERR_INVALID_ARG       # past the size check the missing queries are the error
    assert step(least - 1) == B.SDLLM_ERR_WORKSPACE


def test_current_stream_with_and_without_torchs_private_function(monkeypatch):
    import types
    import torch
    cuda = types.SimpleNamespace(current_device=lambda: 3, current_stream=lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(torch, "cuda", cuda)
    for private, handle in ((lambda device: 40 + device, 43), (None, 77)):
        monkeypatch.setattr(B, "_torch", None)
        monkeypatch.setattr(B, "_raw_stream", None)
        monkeypatch.setattr(torch, "_C", types.SimpleNamespace(**({"_cuda_getCurrentRawStream": private} if private else {})))
        assert B._stream(None) == handle
    monkeypatch.undo()
    assert B._stream(5) == 5 and B._stream(0) is None


def test_product_path_never_imports_the_oracle():
    pkg = os.path.join(ROOT, "paper_2508_02558_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith(".py"):
                text = open(os.path.join(dirpath, f)).read()
                assert not re.search(r"^\s*(from|import)\s+oracle\b", text, flags=re.M), f
                assert "sdllm_oracle" not in text, f
    text = open(os.path.join(ROOT, "oracle", "sdllm_oracle.py")).read()
    assert "paper_2508_02558_amd" not in text and "ctypes" not in text
