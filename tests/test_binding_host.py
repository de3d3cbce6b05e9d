"""The extension module of the Python binding on the host: a build of it that takes the null stream, with callbacks in the
library's place.  Nothing is launched and no device is needed."""
import ctypes as C
import importlib
import importlib.util
import os
import subprocess
import sys
import sysconfig
import types
from dataclasses import replace

import pytest
import torch

from paper_2502_15075_amd import build, kvq

P, I32, I64, F, SZ = C.c_void_p, C.c_int32, C.c_int64, C.c_float, C.c_size_t
# the five entry points, in the order in which bind() takes them
SIGNATURES = {
    "quantize_append": (P, P, P, P, C.c_int, I64, I64, I64, I32, I32, P),
    "decode_attention": (P, P, P, C.c_int, I32, I32, F, P, C.c_int, P, SZ, P),
    "decode_attention_varlen": (P, P, P, C.c_int, I32, P, I32, F, P, C.c_int, P, SZ, P),
    "decode_step": (P, P, P, P, C.c_int, I64, I64, I32, P, C.c_int, I32, F, P, C.c_int, P, SZ, P),
    "decode_step_varlen": (P, P, P, P, C.c_int, I64, I64, P, I32, P, C.c_int, I32, F, P, C.c_int, P, SZ, P),
}


@pytest.fixture(scope="module")
def binding(tmp_path_factory):
    """A module of its own: its entry points and its process are not those of the module that kvq.py has loaded."""
    so = str(tmp_path_factory.mktemp("binding") / "_kvq_binding.so")
    r = subprocess.run(build.binding_command(so, "-DKVQ_CURRENT_STREAM()=nullptr"), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    spec = importlib.util.spec_from_file_location("_kvq_binding", so)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


class Library:
    """Callbacks in the library's place: calls are noted with their arguments, and `body` (if any) runs inside of each."""

    def __init__(self, binding):
        self.calls, self.body = [], None
        self.functions = [C.CFUNCTYPE(C.c_int, *sig)(self._entry(name)) for name, sig in SIGNATURES.items()]
        binding.bind(*[C.cast(f, C.c_void_p).value for f in self.functions], kvq.Layout, kvq.Cache)
        binding.ready()

    def _entry(self, name):
        def call(*args):
            self.calls.append((name, args))
            if self.body is not None:
                self.body(*args)
            return 0
        return call


def host_cache(layout, cls=kvq.Cache):
    """A cache in host memory (its addresses go nowhere but to the callbacks)."""
    return cls(layout, device="cpu", fill=0)


def plain_arguments(layout, cache):
    """For each function arguments that it takes."""
    B, H, Hq = layout.batch, layout.kv_heads, 2 * layout.kv_heads
    rows, one = torch.zeros(B, H, 3, 128, dtype=torch.float16), torch.zeros(B, H, 128, dtype=torch.float16)
    q, out = torch.zeros(B, Hq, 128, dtype=torch.float16), torch.zeros(B, Hq, 128)
    ws, lens = torch.zeros(64, dtype=torch.uint8), torch.ones(B, dtype=torch.int32)
    return {
        "quantize_append": [layout, cache, rows, rows.clone(), 5],
        "decode_attention": [layout, cache, q, 7, 0.5, out, ws],
        "decode_attention_varlen": [layout, cache, q, lens, 7, 0.5, out, ws],
        "decode_step": [layout, cache, one, one.clone(), 6, q, 0.5, out, ws],
        "decode_step_varlen": [layout, cache, one, one.clone(), lens, 6, q, 0.5, out, ws],
    }


@pytest.mark.parametrize("name", SIGNATURES)
def test_structs_of_a_call_outlive_a_new_page_table(binding, name):
    """While a call is inside the library the interpreter's lock is free: what another thread does to the cache, here a new page
    table, must not change or free what the call reads."""
    lib = Library(binding)
    L = kvq.Layout(2, 2, 256, page_tokens=64, n_pages=8)
    cache = host_cache(L)
    cache.page_table = torch.zeros(2, 4, dtype=torch.int32)
    want_layout, want_cache = bytes(L.c()), bytes(cache.c())
    seen = []

    def body(layout, planes, *_):
        cache.page_table = torch.ones(2, 4, dtype=torch.int32)          # drops the struct that was kept ...
        held = [(C.c_uint64 * (len(want_cache) // 8))(*[0x11] * (len(want_cache) // 8)) for _ in range(2000)]   # ... and takes its place
        seen.append((C.string_at(layout, len(want_layout)), C.string_at(planes, len(want_cache)), len(held)))

    lib.body = body
    assert getattr(binding, name)(*plain_arguments(L, cache)[name]) == 0
    assert len(seen) == 1
    assert seen[0][0] == want_layout
    assert seen[0][1] == want_cache


@pytest.mark.parametrize("name", SIGNATURES)
def test_a_new_layout_and_cache_are_taken_at_once(binding, name):
    """The first call that a layout and a cache are handed to is taken like any other: nobody has built their structs before."""
    lib = Library(binding)
    L = kvq.Layout(2, 2, 256 + 64 * list(SIGNATURES).index(name))
    cache = host_cache(replace(L))
    seen = []
    lib.body = lambda layout, planes, *_: seen.append((C.string_at(layout, C.sizeof(kvq._CLayout)), C.string_at(planes, C.sizeof(kvq._CCache))))
    assert L._c is None and cache._struct is None
    assert getattr(binding, name)(*plain_arguments(L, cache)[name]) == 0
    assert seen == [(bytes(L.c()), bytes(cache.c()))]


@pytest.mark.parametrize("name", SIGNATURES)
def test_a_class_that_builds_its_own_struct_is_asked_for_it(binding, name):
    """A subclass with a c() of its own, and any other object that has one, is asked on every call, whatever has been kept."""
    class Moving(kvq.Cache):
        shift = 0

        def c(self):
            st = kvq._CCache.from_buffer_copy(kvq.Cache.c(self))
            st.k_codes += self.shift
            return st

    class Longer(kvq.Layout):
        def c(self):
            st = kvq._CLayout.from_buffer_copy(kvq.Layout.c(self))
            st.max_seq += 1
            return st

    class Other:                                             # no Cache at all
        def __init__(self, cache):
            self.cache = cache

        def c(self):
            return self.cache.c()

    lib = Library(binding)
    seen = []
    lib.body = lambda layout, planes, *_: seen.append((kvq._CLayout.from_address(layout).max_seq, kvq._CCache.from_address(planes).k_codes))
    L, cache = Longer(2, 2, 256), host_cache(kvq.Layout(2, 2, 256), Moving)
    base = kvq.Cache.c(cache).k_codes                        # (kept now)
    for shift in (0, 64, 128):
        cache.shift = shift
        assert getattr(binding, name)(*plain_arguments(L, cache)[name]) == 0
        assert getattr(binding, name)(*plain_arguments(L, Other(cache))[name]) == 0
        assert seen[-2:] == [(257, base + shift)] * 2


def test_a_struct_that_cannot_be_built_is_left_to_the_caller(binding):
    """An error in c() is none of the module's, an interrupt is passed on."""
    class Broken(kvq.Cache):
        error = ValueError

        def c(self):
            raise self.error

    lib = Library(binding)
    L = kvq.Layout(2, 2, 256)
    cache = host_cache(L, Broken)
    args = plain_arguments(L, cache)["quantize_append"]
    assert binding.quantize_append(*args) is None
    cache.error = KeyboardInterrupt
    with pytest.raises(KeyboardInterrupt):
        binding.quantize_append(*args)
    assert lib.calls == []


def test_the_module_that_is_built_is_the_one_that_is_loaded():
    """Named for this interpreter, made for this torch, and what the calls go through."""
    kvq.load()
    assert os.path.samefile(kvq._fast.__file__, build.BINDING) and build.BINDING.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert kvq._fast.torch_version == torch.__version__
    assert kvq._fast_append is kvq._fast.quantize_append and kvq._fast_step_varlen is kvq._fast.decode_step_varlen


@pytest.mark.parametrize("there", [None, types.SimpleNamespace(), types.SimpleNamespace(torch_version="0.1")])
def test_the_library_works_without_the_module(monkeypatch, there):
    """None that can be imported, one from before it said what it was made for, one for another torch: load() says so and the
    Python statements serve every call."""
    name = "_kvq_binding"
    package = importlib.import_module("paper_2502_15075_amd")
    monkeypatch.setitem(sys.modules, f"{package.__name__}.{name}", there)
    monkeypatch.delattr(package, name, raising=False)
    if there is not None:
        monkeypatch.setattr(package, name, there, raising=False)
    for fast in ("_fast_append", "_fast_attention", "_fast_attention_varlen", "_fast_step", "_fast_step_varlen"):
        monkeypatch.setattr(kvq, fast, kvq._not_loaded)
    monkeypatch.setattr(kvq, "_fast", None)
    monkeypatch.setattr(kvq, "_lib", None)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        kvq.load()
    assert kvq._fast is None and kvq._fast_append is kvq._not_loaded and kvq._fast_step is kvq._not_loaded
    L = kvq.Layout(2, 2, 64)
    assert kvq.cache_bytes(L) == [4 * 64 * 64, 4 * 64 * 8, 4 * 64 * 32, 4 * 64 * 8]
    cache, rows = host_cache(L), torch.zeros(2, 2, 4, 128, dtype=torch.float16)
    monkeypatch.setattr(kvq, "_stream_ptr", lambda: 0)       # (no device: what the library refuses before it launches anything)
    with pytest.raises(kvq.KvqError) as e:
        kvq.quantize_append(L, cache, rows, rows, 61)
    assert e.value.status == kvq.ERR_CAPACITY


@pytest.mark.parametrize("command", [["false"], ["/nonexistent/compiler"], None])
def test_a_build_without_the_modules_compiler_goes_on(monkeypatch, tmp_path, command):
    """A compiler that fails or is not there, torch headers that are not: said, and the module of an earlier build goes."""
    def make(out, *extra):
        if command is None:
            raise ImportError("no torch headers")
        return command
    old = tmp_path / "_kvq_binding.so"
    old.write_bytes(b"")
    monkeypatch.setattr(build, "BINDING", str(old))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "binding_command", make)
    assert build._build_binding() != "" and not old.exists()


class Wrapped(torch.Tensor):
    """A tensor subclass: what its attributes say is its own business."""


# what takes the place of one argument: other kinds of object, numbers of other types and beyond 32 bits, tensors that are not plain
JUNK = {
    "None": None, "text": "x", "object": object(), "int": 3, "big int": 1 << 40, "negative big int": -(1 << 31) - 1, "bool": True, "float": 2.5,
    "list": [1], "scalar tensor": torch.tensor(1.0), "double": torch.zeros(2, 2, 128, dtype=torch.float64), "int64": torch.zeros(2, dtype=torch.int64),
    "sparse": torch.zeros(2, 2, 3, 128).to_sparse(), "subclass": torch.zeros(2, 2, 3, 128).as_subclass(Wrapped),
    "strided": torch.zeros(2, 2, 128, 3, dtype=torch.float16).transpose(2, 3), "rank 5": torch.zeros(1, 2, 2, 3, 128, dtype=torch.float16),
    "strided lengths": torch.ones(2, 2, dtype=torch.int32)[:, 0], "lengths of other batch": torch.ones(3, dtype=torch.int32),
}
# the arguments after layout and cache: R rows, Q query, O output, W workspace, L lengths, I integer, S scale
SLOTS = {"quantize_append": "RRI", "decode_attention": "QISOW", "decode_attention_varlen": "QLISOW", "decode_step": "RRIQSOW",
         "decode_step_varlen": "RRLIQSOW"}
PLAIN = {"I": ("int",), "S": ("float",), "L": (),
         # the library looks at the bytes of a workspace, the binding at nothing but its being a plain tensor or None
         "W": ("None", "scalar tensor", "double", "int64", "strided", "rank 5", "strided lengths", "lengths of other batch")}


@pytest.mark.parametrize("name", SIGNATURES)
def test_an_argument_that_is_not_plain_leaves_the_call_to_the_caller(binding, name):
    """Each argument in turn replaced by something else, all others plain: None comes back, nothing is raised and the library is not
    called.  (Where the replacement is plain too, it is.)"""
    lib = Library(binding)
    L = kvq.Layout(2, 2, 256)
    cache = host_cache(L)
    args = plain_arguments(L, cache)[name]
    assert getattr(binding, name)(*args) == 0 and len(lib.calls) == 1
    for slot in range(len(args)):
        for what, junk in JUNK.items():
            lib.calls.clear()
            kind = "LC"[slot] if slot < 2 else SLOTS[name][slot - 2]
            taken = slot >= 2 and what in PLAIN.get(kind, ())
            got = getattr(binding, name)(*args[:slot], junk, *args[slot + 1:])
            assert got == (0 if taken else None), (slot, what)
            assert len(lib.calls) == (1 if taken else 0), (slot, what)
    for wrong in (args[:-1], args + [None]):
        assert getattr(binding, name)(*wrong) is None
    assert getattr(binding, name)(cache, L, *args[2:]) is None                # (each where the other belongs)
    with torch.device("cpu"):                                                 # a function mode: torch's own calls may mean something else
        assert getattr(binding, name)(*args) is None


def test_the_library_gets_what_the_arguments_say(binding):
    """Addresses, types, strides, sizes and numbers as the C functions take them."""
    lib = Library(binding)
    L = kvq.Layout(2, 2, 256)
    a = plain_arguments(L, host_cache(L))
    big = torch.zeros(2, 5, 2, 256, dtype=torch.bfloat16)
    k, v = big.transpose(1, 2)[:, :, 1:4, :128], big.transpose(1, 2)[:, :, 2:5, 128:]
    assert binding.quantize_append(*a["quantize_append"][:2], k, v, 9) == 0
    assert lib.calls[-1][1][2:] == (k.data_ptr(), v.data_ptr(), kvq.KVQ_BF16, 5 * 2 * 256, 256, 2 * 256, 9, 3, None)
    args = a["decode_attention"]
    assert binding.decode_attention(*args) == 0
    q, n, scale, out, ws = args[2:]
    assert lib.calls[-1][1][2:] == (q.data_ptr(), kvq.KVQ_F16, 4, n, scale, out.data_ptr(), kvq.KVQ_F32, ws.data_ptr(), 64, None)
    args = a["decode_attention_varlen"]
    assert binding.decode_attention_varlen(*args[:-1], None) == 0
    q, lens, n, scale, out, _ = args[2:]
    assert lib.calls[-1][1][2:] == (q.data_ptr(), kvq.KVQ_F16, 4, lens.data_ptr(), n, scale, out.data_ptr(), kvq.KVQ_F32, None, 0, None)
    args = a["decode_step"]
    k4, v4 = torch.zeros(2, 2, 1, 256, dtype=torch.float16)[..., :128], torch.ones(2, 2, 1, 256, dtype=torch.float16)[..., :128]
    assert binding.decode_step(*args[:2], k4, v4, *args[4:]) == 0
    pos, q, scale, out, ws = args[4:]
    assert lib.calls[-1][1][2:] == (k4.data_ptr(), v4.data_ptr(), kvq.KVQ_F16, 512, 256, pos, q.data_ptr(), kvq.KVQ_F16, 4, scale,
                                    out.data_ptr(), kvq.KVQ_F32, ws.data_ptr(), 64, None)
    args = a["decode_step_varlen"]
    assert binding.decode_step_varlen(*args) == 0
    k, v, pos, most, q, scale, out, ws = args[2:]
    assert lib.calls[-1][1][2:] == (k.data_ptr(), v.data_ptr(), kvq.KVQ_F16, 256, 128, pos.data_ptr(), most, q.data_ptr(), kvq.KVQ_F16, 4,
                                    scale, out.data_ptr(), kvq.KVQ_F32, ws.data_ptr(), 64, None)
