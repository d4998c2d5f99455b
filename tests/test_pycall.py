"""The entry points called without ctypes: every argument arrives where the C prototype has it, errors come back as they do through
ctypes, and nothing is called with arguments that could not be had."""
import ctypes
import importlib.util
import os
import sysconfig

import pytest

from paper_2508_02558_amd import binding as B
from paper_2508_02558_amd import build

pytestmark = pytest.mark.skipif(B._pycall is None, reason="built without the interpreter's headers")
vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t


class Tensor:
    def __init__(self, at, numel=0):
        self.at, self.n = at, numel

    def data_ptr(self):
        return self.at

    def numel(self):
        return self.n

    def element_size(self):
        return 2


def recorder(restype, *argtypes):
    seen = []

    @ctypes.CFUNCTYPE(restype, *argtypes)
    def f(*args):
        seen.append(args)
        if len(args) == 14:
            args[13][0] = 2
        return f.status
    f.status = 0
    return f, seen, ctypes.cast(f, vp).value


def test_block_step_arguments():
    f, seen, at = recorder(i32, vp, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp, ctypes.POINTER(i32))
    t = [Tensor(0x7f0000000000 + 16 * i, 3) for i in range(8)]
    t[7].n = 1 << 40
    assert B._pycall.block_step(at, 0x55, 7, 3, *t, 0xabc) == 2
    assert seen[0][:13] == (0x55, 7, 3, *(x.at for x in t), 1 << 41, 0xabc)
    assert B._pycall.block_step(at, 0x55, -1, 3, *t[:3], None, None, None, t[6], None, 0) == 2
    assert seen[1][:13] == (0x55, -1, 3, *(x.at for x in t[:3]), None, None, None, t[6].at, None, 0, None)
    f.status = -3
    assert B._pycall.block_step(at, 0x55, 7, 3, *t, 0) == -3


def test_sparse_and_dense_arguments():
    f, seen, at = recorder(i32, vp, vp, vp, vp, i32, vp, vp, vp, vp, sz, vp)
    q, k, v, kb, vb, out, ws = (Tensor(0x1000 * i, 5) for i in range(1, 8))
    assert B._pycall.sparse_attn(at, 9, q, k, v, 77, kb, vb, out, ws, 0x10) == 0
    assert seen[0] == (9, q.at, k.at, v.at, 77, kb.at, vb.at, out.at, ws.at, 10, 0x10)
    rows = []

    @ctypes.CFUNCTYPE(i32, vp, vp, ctypes.POINTER(ctypes.c_int64), vp, vp, vp, ctypes.POINTER(ctypes.c_int64), vp)
    def dense(shape, q_, qs, k_, v_, o_, os_, stream):
        rows.append((shape, q_, qs[:3], k_, v_, o_, os_[:3], stream))
        return -1
    at = ctypes.cast(dense, vp).value
    assert B._pycall.dense_attn(at, 9, q, (1 << 40, 2, 3), k, v, out, (4, 5, 6), 0) == -1
    assert rows == [(9, q.at, [1 << 40, 2, 3], k.at, v.at, out.at, [4, 5, 6], None)]


def test_nothing_is_called_with_arguments_that_cannot_be_had():
    f, seen, at = recorder(i32, vp, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp, ctypes.POINTER(i32))
    t = Tensor(0x100, 1)
    for args in ((at, 5, 0, 1, t, t, 3.5, t, t, t, t, t, 0), (at, 5, "0", 1, t, t, t, t, t, t, t, t, 0), (at, 5, 0, 1, t, t, t, t, t, t, t, object(), 0),
                 (at, 5, 0, 1, t), (at, 5, 0, 1, Tensor("x"), t, t, t, t, t, t, t, 0)):
        with pytest.raises((AttributeError, TypeError)):
            B._pycall.block_step(*args)
    assert not seen


def test_refusals_are_the_same_with_and_without(monkeypatch):
    shape = B.make_shape(batch=1, n_q_heads=2, n_kv_heads=2, head_dim=64, seq_len=160, block_off=64, block_len=32, dtype=B.SDLLM_F32)
    odd = B.make_shape(batch=1, n_q_heads=2, n_kv_heads=2, head_dim=96, seq_len=160, block_off=64, block_len=32, dtype=B.SDLLM_F32)
    t, ws = Tensor(0x1000, 4), Tensor(0x10000, 1 << 24)
    t.stride = lambda: (8, 8, 64, 1)

    def refusals():
        got = []
        for s in (shape, odd):
            for call in (lambda: B.sdllm_block_step(s, 0, 1, None, t, t, t, t, t, t, ws, stream=1), lambda: B.sdllm_block_step(s, -1, 1, t, t, t, t, t, t, t, ws, stream=1),
                         lambda: B.sdllm_block_step(s, 2, 1, t, t, t, t, t, t, t, None, stream=1), lambda: B.sdllm_sparse_attn(s, None, t, t, 4, t, t, t, ws, stream=1),
                         lambda: B.sdllm_dense_attn(s, t, None, t, t, stream=1)):
                with pytest.raises(B.SdllmError) as e:
                    call()
                got.append(str(e.value))
        with pytest.raises(Exception):
            B.sdllm_sparse_attn(None, t, t, t, 4, t, t, t, ws, stream=1)
        return got
    with_it = refusals()
    monkeypatch.setattr(B, "_pycall", None)
    assert refusals() == with_it


def test_built_by_the_librarys_compiler_for_this_interpreter(monkeypatch, tmp_path):
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert B._pycall.__file__.endswith("_pycall" + suffix)
    stale = tmp_path / "_pycall.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "PYCALL_PATH", str(tmp_path / ("_pycall" + suffix)))
    monkeypatch.setenv("CXX", str(tmp_path / "no-compiler"))
    if os.path.isabs(build.HIPCC):
        monkeypatch.setenv("PATH", str(tmp_path))                  # no other compiler either
    build._build_pycall()
    assert not stale.exists()                                      # one that every interpreter would load
    spec = importlib.util.spec_from_file_location("_pycall", build.PYCALL_PATH)
    assert importlib.util.module_from_spec(spec).block_step
