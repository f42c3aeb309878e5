"""The native argument marshalling of the binding (csrc/marshal.c) without a GPU: what it hands to the
library for ordinary calls, and that it leaves everything else to the binding's own checks."""
import ctypes
import os
import subprocess
import sys

import pytest
import torch

from paper_2502_06728_amd import binding

vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
COMPRESS = ctypes.CFUNCTYPE(i32, vp, i64, vp, i32, vp, vp, i32, vp, i32, vp, vp)
STEP = ctypes.CFUNCTYPE(i32, vp, i64, i32, vp, i32, i64, vp, i32, i64, vp, i32, vp, vp)
ADAMW = ctypes.CFUNCTYPE(i32, vp, vp, i64, i32, vp, i32, i64, vp, i32, i64, vp, i32, vp, vp, vp, vp, vp)
NAMES = ("detonation_compress_packed", "detonation_decompress_step_packed",
         "detonation_decompress_adamw_step_packed")


class OnDevice:
    """A tensor that says it is on the device."""
    is_cuda = True

    def __init__(self, t):
        self.t, self.dtype = t, t.dtype

    def is_contiguous(self):
        return self.t.is_contiguous()

    def numel(self):
        return self.t.numel()

    def data_ptr(self):
        return self.t.data_ptr()


@pytest.fixture
def calls():
    """The library's entry points replaced by recorders; `calls.status` is what they return."""
    lib = binding.load()

    class Calls(list):
        status = 0

    got = Calls()

    def record(adamw):
        def f(cfg, *rest):
            c = ctypes.cast(cfg, ctypes.POINTER(binding.deto_config)).contents
            fields = tuple(getattr(c, name) for name, _ in c._fields_)
            if adamw:
                o = ctypes.cast(rest[0], ctypes.POINTER(binding.deto_adamw)).contents
                fields += tuple(getattr(o, name) for name, _ in o._fields_)
                rest = rest[1:]
            got.append((fields, rest))
            return got.status
        return f

    fns = (COMPRESS(record(False)), STEP(record(False)), ADAMW(record(True)))
    dtypes = (torch.float32, torch.bfloat16, torch.float16, torch.int32, torch.uint8)
    binding._marshal.setup(*(ctypes.cast(f, vp).value for f in fns), *dtypes, lambda: 3, lambda d: 40 + d)
    yield got
    binding._marshal.setup(*(ctypes.cast(getattr(lib, n), vp).value for n in NAMES), *dtypes,
                           torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)


def on(n, dtype=torch.float32):
    return OnDevice(torch.zeros(n, dtype=dtype))


N, S, K = 1000, 64, 20          # 16 chunks, 320 entries, 32 words
C = -(-N // S)


@pytest.mark.parametrize("stream,handle", [(None, 43), (7, 7)])
@pytest.mark.parametrize("packed,vt,it,codes", [(False, torch.float32, torch.int32, (0, 0)),
                                                (True, torch.bfloat16, torch.uint8, (1, 1)),
                                                (True, torch.float16, torch.int32, (2, 0)),
                                                (True, torch.int32, torch.uint8, (3, 1))])
def test_ordinary_calls(calls, packed, vt, it, codes, stream, handle):
    cfg = binding.Config(chunk=S, topk=K, sign=True, dct=True, decay=0.5, lr=0.25, weight_decay=2.0,
                         seed=-1, step=2**63 + 1)
    want = (S, K, 0, 3, 0.5, 0.25, 2.0, 2**64 - 1, 2**63 + 1)
    R, words = 3, C * 2 if vt == torch.int32 else C * K
    g, m = on(N, torch.bfloat16), on(N)
    idx, val = on(R * C * K, it), on(R * words, vt)
    comp = binding.detonation_compress_packed if packed else binding.detonation_compress
    comp(cfg, g, m, idx, val, stream=stream)
    fields, a = calls.pop()
    assert fields == want
    assert a == (N, g.data_ptr(), 1, m.data_ptr(), idx.data_ptr(), codes[1], val.data_ptr(), codes[0],
                 None, handle)
    dec = binding.detonation_decompress_step_packed if packed else binding.detonation_decompress_step
    dec(cfg, R, idx, val, g, stream=stream)
    fields, a = calls.pop()
    assert fields == want
    assert a == (N, R, idx.data_ptr(), codes[1], C * K, val.data_ptr(), codes[0], words, g.data_ptr(),
                 1, None, handle)
    ada = (binding.detonation_decompress_adamw_step_packed if packed
           else binding.detonation_decompress_adamw_step)
    ea, es, mx = on(N), on(N), on(N)
    ada(cfg, binding.AdamW(0.5, 0.25, 0.125, True, 9), R, idx, val, m, ea, es, mx, stream=stream)
    fields, a = calls.pop()
    assert fields == want + (0.5, 0.25, 0.125, 1, 9)
    assert a == (N, R, idx.data_ptr(), codes[1], C * K, val.data_ptr(), codes[0], words, m.data_ptr(),
                 0, ea.data_ptr(), es.data_ptr(), mx.data_ptr(), None, handle)
    calls.status = 2
    with pytest.raises(binding.DetonationError):
        comp(cfg, g, m, idx, val)


def test_everything_else_is_left_to_the_checks(calls):
    cfg = binding.Config(chunk=S, topk=K)
    idx, val = on(2 * C * K, torch.int32), on(2 * C * K)
    c, d = binding._marshal.compress, binding._marshal.decompress
    good = [cfg, None, on(N), on(N), idx, val, False, None]
    assert c(*good) == 0
    for at, bad in [(0, binding.Config(chunk=S, topk=S + 1)), (0, binding.Config(chunk=0, topk=0)),
                    (0, binding.Config(chunk=S, topk=K, seed="x")), (1, N + 1), (1, -1), (1, 2.0),
                    (2, on(N - 1)), (2, on(N, torch.float16)), (2, torch.zeros(N)), (2, None),
                    (2, OnDevice(torch.zeros(2 * N)[::2])), (3, on(N, torch.bfloat16)), (4, None),
                    (4, on(C * K, torch.uint8)), (4, on(C * K - 1, torch.int32)), (5, on(C * K - 1)),
                    (5, on(C * K, torch.bfloat16)), (5, None), (7, "stream")]:
        call = list(good)
        call[at] = bad
        assert c(*call) == -1, (at, bad)
    good = [cfg, None, 2, idx, val, on(N), False, None]
    assert d(*good) == 0
    for at, bad in [(2, 0), (2, 3), (2, 2.0), (3, None), (5, on(N, torch.float16)), (5, on(N), )]:
        call = list(good)
        call[at] = bad
        assert d(*call) == (0 if at == 5 and bad.dtype == torch.float32 else -1), (at, bad)
    moments = [binding.AdamW(amsgrad=True), on(N), on(N), None]
    assert d(*good, *moments) == -1                       # the maximum is required
    assert d(*good, binding.AdamW(amsgrad=2), on(N), on(N), on(N)) == -1
    assert d(*good, binding.AdamW(), on(N), on(N), None) == 0
    assert d(*good, binding.AdamW(), on(N), on(N - 1), None) == -1
    with pytest.raises(ValueError, match="contiguous device tensors"):
        binding.detonation_compress(cfg, torch.zeros(N), torch.zeros(N), idx.t, val.t)
    with pytest.raises(ValueError, match="at least"):
        binding.detonation_compress(cfg, on(N), on(N), idx, on(3))


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as it is before its first call."""
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_marshal", None)
    return monkeypatch


def goes_through_the_checks():
    cfg = binding.Config(chunk=S, topk=K)
    assert binding.version() >= 1007 and binding.payload_entries(cfg, N) == C * K
    idx, val = torch.zeros(C * K, dtype=torch.int32), torch.zeros(C * K)
    for f in (binding.detonation_compress, binding.detonation_compress_packed):
        with pytest.raises(ValueError, match="contiguous device tensors"):
            f(cfg, torch.zeros(N), torch.zeros(N), idx, val)
        with pytest.raises(ValueError, match="at least"):
            f(cfg, on(N), on(N), on(C * K, torch.int32), on(3))
    for f in (binding.detonation_decompress_step, binding.detonation_decompress_step_packed):
        with pytest.raises(ValueError, match="at least"):
            f(cfg, 2, on(C * K, torch.int32), on(C * K), on(N))


def test_works_without_the_compiled_marshalling(unloaded, tmp_path):
    """Not compiled for this interpreter, or not loadable by it."""
    unloaded.setattr(binding, "MARSHAL_PATH", str(tmp_path / "absent.so"))
    goes_through_the_checks()
    assert not hasattr(binding._marshal, "setup")
    (tmp_path / "broken.so").write_bytes(b"no library")
    unloaded.setattr(binding, "MARSHAL_PATH", str(tmp_path / "broken.so"))
    unloaded.setattr(binding, "_marshal", None)
    goes_through_the_checks()


def test_works_without_torch_stream_functions(unloaded):
    unloaded.delattr(torch._C, "_cuda_getCurrentRawStream")
    goes_through_the_checks()


def test_loading_the_library_needs_no_torch():
    code = ("import sys; from paper_2502_06728_amd import binding as b; "
            "assert b.version() >= 1007 and b.payload_entries(b.Config(), 100) == 16; "
            "assert 'torch' not in sys.modules; import torch; assert hasattr(b._marshalling(), 'setup')")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=os.path.dirname(os.path.dirname(__file__)))


def test_building_needs_no_c_compiler(monkeypatch, tmp_path, capsys):
    from paper_2502_06728_amd import build
    target = tmp_path / "m.so"
    monkeypatch.setattr(build, "MARSHAL", str(target))
    for cc in ("false", "no-such-compiler"):
        target.write_bytes(b"of an earlier build")
        monkeypatch.setenv("CC", cc)
        build._build_marshal(False)
        assert not target.exists() and "not compiled" in capsys.readouterr().err


def test_a_class_with_its_own_c_is_asked(monkeypatch):
    """A Config or AdamW of the caller's that computes what it passes on (a schedule, say)."""
    class Halved(binding.Config):
        def c(self):
            c = super().c()
            c.lr *= 0.5
            return c

    class Later(binding.AdamW):
        def c(self):
            o = super().c()
            o.step += 1
            return o

    seen = []

    class Lib:
        def __getattr__(self, name):
            def f(*args):
                seen.append((name, [a._obj for a in args if hasattr(a, "_obj")]))
                return 0
            return f

    binding.load()
    monkeypatch.setattr(binding, "load", lambda: Lib())
    monkeypatch.setattr(binding, "payload_entries", lambda cfg, n: C * K)
    idx, val = on(C * K, torch.int32), on(C * K)
    cfg, opt = Halved(chunk=S, topk=K, lr=1.0), Later(step=4)
    plain = binding.Config(chunk=S, topk=K)
    for pk in ("", "_packed"):
        getattr(binding, "detonation_compress" + pk)(cfg, on(N), on(N), idx, val, stream=7)
        getattr(binding, "detonation_decompress_step" + pk)(cfg, 1, idx, val, on(N), stream=7)
        ada = getattr(binding, "detonation_decompress_adamw_step" + pk)
        ada(cfg, binding.AdamW(), 1, idx, val, on(N), on(N), on(N), stream=7)
        assert [c[0].lr for _, c in seen] == [0.5] * 3
        seen.clear()
        ada(plain, opt, 1, idx, val, on(N), on(N), on(N), stream=7)
        assert [c[1].step for _, c in seen] == [5]
        seen.clear()
