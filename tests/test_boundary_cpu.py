"""Host-side checks of the C-ABI boundary that need no GPU: the library loads, exports every symbol
the public header declares, and rejects bad arguments before touching the device."""
import ctypes
import os
import re
import shutil
import struct
import sysconfig

import pytest

import paper_2504_00970_amd as skv
from paper_2504_00970_amd import _build, binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "sentencekv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(skv_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = binding._lib()
    names = _declared()
    assert len(names) >= 12
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(skv.EXPORTS) == names


def test_strerror_covers_every_status():
    lib = binding._lib()
    msgs = {lib.skv_strerror(c).decode() for c in (0, -1, -2, -3, -4)}
    assert len(msgs) == 5 and lib.skv_strerror(-99).decode() == "unknown status"


@pytest.mark.parametrize("field,value", [("head_dim", 64), ("n_q_heads", 30), ("kv_dtype", 7), ("max_budget", 0),
                                         ("n_kv_heads", 0), ("max_batch", 0), ("n_q_heads", 8 * 16), ("semvec_dtype", 3), ("kv_dtype", 2), ("max_batch", 4097)])
def test_create_rejects_bad_descriptors_before_touching_the_gpu(field, value):
    kw = dict(n_layers=1, n_q_heads=32, n_kv_heads=8, max_tokens=64, max_sentences=8, max_budget=16)
    kw[field] = value
    with pytest.raises(skv.SkvError) as e:
        skv.Context(skv.Desc(**kw))
    assert e.value.status == skv.SKV_EINVAL


def test_null_context_and_null_out_pointer_are_invalid_arguments():
    lib = binding._lib()
    assert lib.skv_create(None, None, None) == skv.SKV_EINVAL
    assert lib.skv_score(None, 0, None, None, 0, None) == skv.SKV_EINVAL
    assert lib.skv_attend(None, None, None, None, None, 0, None, None) == skv.SKV_EINVAL
    assert lib.skv_set_stream(None, None) == skv.SKV_EINVAL
    assert lib.skv_workspace_bytes(None) == 0
    assert lib.skv_query_update(None, 1, None, None, None, 8, None, None, None) == skv.SKV_EINVAL
    assert lib.skv_build_semvec_layers(None, None, 0, None, 0, None) == skv.SKV_EINVAL
    assert lib.skv_token_importance_work_bytes(None, 100, 8) == -1
    assert lib.skv_token_importance(None, None, None, 100, 8, None, None, 0) == skv.SKV_EINVAL
    assert lib.skv_retain(None, None, 1, 1, None, 1, None, None, None, None) == skv.SKV_EINVAL
    assert lib.skv_compact_pool(None, None, None, 1, None, 1, None, None, None) == skv.SKV_EINVAL
    assert lib.skv_merge_lse(None, 1, None, None, None, None, None, None) == skv.SKV_EINVAL
    lib.skv_destroy(None)      # no-op


_NATIVE = [n for n in skv.EXPORTS if n in ("skv_segment", "skv_build_semvec", "skv_build_semvec_layers", "skv_token_importance", "skv_retain",
                                           "skv_compact_pool", "skv_query_update", "skv_score", "skv_select", "skv_gather", "skv_attend",
                                           "skv_decode_step", "skv_merge_lse")]


@pytest.mark.parametrize("through", ["native", "ctypes"])
@pytest.mark.parametrize("name", _NATIVE)
def test_python_calls_refuse_arguments_in_each_others_place(name, through):
    """An integer is no pointer and a tensor no number (the context is null: nothing is looked at beyond the arguments' types)."""
    import torch
    lib = binding._lib()
    call, kinds = getattr(binding._CALLS if through == "native" else binding._CtypesCalls(lib), name), binding._SIGNATURES[name][1]
    args = [None if k is ctypes.c_void_p else 1 for k in kinds]
    assert call(*args) == skv.SKV_EINVAL
    for i, k in enumerate(kinds):
        bad = list(args)
        address = i == 0 or (name == "skv_segment" and i == len(kinds) - 1)
        bad[i] = torch.zeros(1, dtype=torch.int32) if address or k is not ctypes.c_void_p else 4096
        with pytest.raises(TypeError):
            call(*bad)
        if not address and k is ctypes.c_void_p:
            bad[i] = torch.zeros(4, 4).t()
            with pytest.raises(AssertionError):
                call(*bad)
            bad[i] = torch.zeros(4, 4)
            assert call(*bad) == skv.SKV_EINVAL
    with pytest.raises(TypeError):
        call(*args[:-1])


def test_build_notices_what_the_call_module_depends_on(tmp_path, monkeypatch):
    """An edited calls.cpp or header, another torch, another Python or no module at all: build(force=False) compiles it anew."""
    binding._lib()
    assert _build.calls_fit()
    calls = tmp_path / "_calls.so"
    shutil.copy(_build.CALLS, calls)
    monkeypatch.setattr(_build, "CALLS", str(calls))
    newest = max(os.path.getmtime(p) for p in (os.path.join(_build.CSRC, "calls.cpp"), os.path.join(_build.INCLUDE, "sentencekv.h")))
    os.utime(calls, (newest + 1, newest + 1))
    assert not _build.calls_stale()
    os.utime(calls, (newest - 1, newest - 1))
    assert _build.calls_stale()
    os.utime(calls, (newest + 1, newest + 1))
    with monkeypatch.context() as m:
        m.setattr("torch.__version__", "0.0.1")
        assert not _build.calls_fit() and _build.calls_stale()
    with monkeypatch.context() as m:
        m.setattr(sysconfig, "get_python_version", lambda: "3.1")
        assert _build.calls_stale()
    calls.unlink()
    assert _build.calls_stale()
    started = []
    monkeypatch.setattr(_build, "stale", lambda lib="": False)
    monkeypatch.setattr(_build, "_start", lambda cmd, verbose: started.append(cmd))
    monkeypatch.setattr(_build, "_finish_calls", lambda proc: True)
    _build.build(force=False)
    assert len(started) == 1 and any("calls.cpp" in part for part in started[0])


def test_calls_go_through_ctypes_where_the_module_cannot_be_built(tmp_path, monkeypatch):
    lib = binding._lib()
    monkeypatch.setattr(_build, "CALLS", str(tmp_path / "_calls.so"))
    monkeypatch.setattr(_build, "_host_compiler", lambda: str(tmp_path / "no-compiler"))
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "_CALLS", None)
    with pytest.warns(UserWarning, match="ctypes"):
        assert binding._lib() is not lib
    assert isinstance(binding._CALLS, binding._CtypesCalls)
    assert binding._CALLS.skv_attend(None, None, None, None, None, 0, None, None) == skv.SKV_EINVAL


def test_product_package_does_not_reach_into_the_oracle():
    pkg = os.path.join(ROOT, "paper_2504_00970_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                src = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in src.lower(), f


def _kernels(path):
    """Metadata of the gfx950 kernels in a library: the code objects of its bundles carry it as a note (type 32, msgpack)."""
    msgpack = pytest.importorskip("msgpack")
    data, kernels, at = open(path, "rb").read(), [], 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (entries,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<3Q", data, p)
            name, p = data[p + 24:p + 24 + length], p + 24 + length
            if b"gfx950" not in name:
                continue
            elf = data[at + offset:at + offset + size]
            headers, = struct.unpack_from("<Q", elf, 0x20)
            each, n = struct.unpack_from("<2H", elf, 0x36)
            for i in range(n):
                kind, _, begin, _, _, length = struct.unpack_from("<2I4Q", elf, headers + i * each)
                end = begin + length
                while kind == 4 and begin < end:                                            # PT_NOTE
                    name_size, desc_size, note = struct.unpack_from("<3I", elf, begin)
                    begin += 12 + (name_size + 3) // 4 * 4
                    if note == 32:
                        kernels += msgpack.unpackb(elf[begin:begin + desc_size])["amdhsa.kernels"]
                    begin += (desc_size + 3) // 4 * 4
        at += 24
    return kernels


def test_no_kernel_spills_registers():
    """A spilled register is a trip through memory in kernels that are bound by such trips, and in those that load keys it waits behind the keys."""
    kernels = _kernels(_build.build(force=False))
    assert len(kernels) > 100
    assert [k[".name"] for k in kernels if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]] == []
