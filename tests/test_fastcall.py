"""The module that takes ordinary calls to the library without ctypes: what it refuses, that a refusal calls nothing,
and that both ways hand the library the same arguments.  A recording C function stands in for the library's."""
import ctypes

import pytest
import torch

from paper_2502_00425_amd import binding as mq

P, I32, I64, F32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float
TYPES = {
    "prefill": [P, I64, P, P, P, P, I64] + [I32] * 4 + [F32, F32, I32, P, I64, P],
    "prefill_static": [P, I64, P, P, P, P, I64] + [I32] * 4 + [F32, F32, I32, P],
    "decode": [P, I64, P, P, P, I64] + [I32] * 4 + [F32, F32, I32, P],
    "decode_grouped": [P, I64, I32, I32, I32, F32, F32, I32, P, I32, P],
    "gemv_grouped": [P, I32, I32, I32, F32, F32, P, I32, P],
    "quant": [P, I64, P, P, I32, I32, I32, F32, F32, I32, P],
    "weight_only": [P, I64, P, P, I64, I32, I32, I32, P],
}
STREAM = 0x1230


@pytest.fixture
def both(monkeypatch):
    """-> (the module, what its calls handed over, the binding on the same recorders)"""
    seen, keep = [], []

    def recorder(name):
        def fn(*a):
            a = list(a)
            if "grouped" in name:
                at, count = len(a) - 3, a[-2]
                a[at] = bytes((ctypes.c_char * (40 * count)).from_address(a[at])) if count else b""
                a[at] = b"".join(a[at][40 * i:40 * i + 36] for i in range(count))       # without the padding
            seen.append((name, a))
            return 0
        f = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES[name])(fn)
        keep.append(f)
        return f

    entries = {n: recorder(n) for n in TYPES}
    loader = mq.importlib.machinery.ExtensionFileLoader("mquant_fastcall", mq.FAST_PATH)
    mod = mq.importlib.util.module_from_spec(mq.importlib.util.spec_from_file_location("mquant_fastcall", mq.FAST_PATH,
                                                                                       loader=loader))
    loader.exec_module(mod)
    assert mod is not mq._fast
    assert mod.quant(*[None] * 7) is NotImplemented                                     # before setup
    mod.setup(lambda: True, lambda: 0, lambda d: STREAM, *(ctypes.cast(entries[n], P).value for n in TYPES))

    class Lib:
        mquant_status_string = staticmethod(lambda st: b"")
    for n, c in zip(TYPES, ("w4a8_linear_prefill", "w4a8_linear_prefill_static", "w4a8_linear_decode",
                            "w4a8_linear_decode_grouped", "w4a8_gemv_grouped", "hadamard_quant_act", "w4g128_gemm")):
        setattr(Lib, "mquant_" + c, staticmethod(entries[n]))
    monkeypatch.setattr(mq, "lib", Lib)
    monkeypatch.setattr(mq, "_stream", lambda: STREAM)
    yield mod, seen, monkeypatch


def calls():
    x = torch.zeros((3, 512), dtype=torch.float16)
    wide = torch.zeros((3, 600), dtype=torch.float16)[:, 8:264]
    xq, perm = torch.zeros((3, 512), dtype=torch.int8), torch.zeros(3, dtype=torch.int32)
    w, ws, y = torch.zeros(64, dtype=torch.uint8), torch.zeros(256, dtype=torch.float16), torch.zeros((3, 256), dtype=torch.float16)
    work = torch.zeros(300, dtype=torch.uint8)
    lin = [(w, ws, 256, y), (w, None, 256, wide)]
    return {
        "prefill": lambda **k: mq.w4a8_linear_prefill(x, perm, w, ws, 256, 2, 0.5, 0.1, 512, work, out=k.get("out", wide)),
        "prefill_static": lambda **k: mq.w4a8_linear_prefill_static(x, None, w, ws, 256, k.get("n_vis", 2), 0.5, 0.1, 512, y),
        "decode": lambda **k: mq.w4a8_linear_decode(x, w, ws, 256, 0, k.get("s", 0.5), 0.1, 512, out=y),
        "decode_grouped": lambda **k: mq.w4a8_linear_decode_grouped(x, k.get("lin", lin), 0, 0.5, 0.1, 512),
        "gemv_grouped": lambda **k: mq.w4a8_gemv_grouped(xq, k.get("lin", lin), 1, 0.5, 0.1),
        "quant": lambda **k: mq.hadamard_quant_act(x, 1, 0.5, 0.1, 512, perm_dev=k.get("perm", perm), out=xq),
        "weight_only": lambda **k: mq.w4g128_gemm(x, w, 256, out=wide),
    }


@pytest.mark.parametrize("name", list(TYPES))
def test_the_same_arguments_either_way(both, name):
    mod, seen, mp = both
    call = calls()[name]
    mp.setattr(mq, "_fast", mod)
    call()
    slow = type("Slow", (), {"__getattr__": lambda s, _: lambda *a: NotImplemented})()
    mp.setattr(mq, "_fast", slow)
    call()
    assert len(seen) == 2 and seen[0] == seen[1] and seen[0][0] == name
    assert seen[0][1][-1] == STREAM


def test_the_unusual_goes_the_other_way(both):
    """Whole numbers where a fraction is usual, a layout or type that the checks refuse: the module calls nothing, and the
    result or the error is that of the other way."""
    mod, seen, mp = both
    mp.setattr(mq, "_fast", mod)
    c = calls()
    c["decode"](s=1)                                                   # an int as a scale: ctypes takes it
    assert seen.pop()[1][10] == 1.0
    t = torch.zeros((3, 256), dtype=torch.float16)
    c["decode_grouped"](lin=[[t, t, 256, t]])                          # a list instead of a tuple
    assert seen.pop()[0] == "decode_grouped" and not seen              # from here on nothing is called
    with pytest.raises(mq.MQuantError):
        c["prefill"](out=torch.zeros((256, 3), dtype=torch.float16).t())
    with pytest.raises(mq.MQuantError):
        c["quant"](perm=torch.zeros(6, dtype=torch.int32)[::2])
    with pytest.raises(mq.MQuantError):
        c["gemv_grouped"](lin=[(t, t, 2 ** 31, t)])
    assert mod.quant(1, 2, 3) is NotImplemented and mod.prefill() is NotImplemented
    assert mod.prefill_static(*[None] * 10) is NotImplemented and mod.gemv_grouped(None, [], 0, 1.0, 1.0) is NotImplemented
    assert mod.gemv_grouped(t, [(t, t)], 0, 1.0, 1.0) is NotImplemented
    mod.setup(lambda: False, lambda: 0, lambda d: STREAM, *[1] * 7)    # no GPU initialised yet
    assert mod.weight_only(t, t, 4, t) is NotImplemented
    assert not seen


def test_errors_of_the_library_are_raised(both):
    mod, seen, mp = both
    bad = ctypes.CFUNCTYPE(ctypes.c_int, *TYPES["weight_only"])(lambda *a: mq.ERR_BAD_SHAPE)
    mod.setup(lambda: True, lambda: 0, lambda d: STREAM, *[1] * 6, ctypes.cast(bad, P).value)
    mp.setattr(mq, "_fast", mod)
    with pytest.raises(mq.MQuantError) as e:
        calls()["weight_only"]()
    assert e.value.status == mq.ERR_BAD_SHAPE


@pytest.mark.parametrize("where", ["initialized", "device", "stream", "shape", "stride", "data_ptr", "is_contiguous"])
@pytest.mark.parametrize("error,raised", [(KeyboardInterrupt, True), (SystemExit, True), (MemoryError, True), (RuntimeError, False)])
def test_interrupts_are_not_swallowed(both, where, error, raised):
    """What a program raises over a call (Ctrl-C surfaces in the functions of torch that the module calls) reaches the
    caller, as it does through ctypes; an error of a method leaves the call to the other way.  Nothing is launched."""
    mod, seen, _ = both

    def fail(*a):
        raise error

    class X:
        shape = property(fail) if where == "shape" else (3, 512)
        stride = fail if where == "stride" else lambda self: (512, 1)
        data_ptr = fail if where == "data_ptr" else lambda self: 4096
        is_contiguous = fail if where == "is_contiguous" else lambda self: True
    mod.setup(fail if where == "initialized" else lambda: True, fail if where == "device" else lambda: 0,
              fail if where == "stream" else lambda d: STREAM, *[1] * 7)
    t = X()
    calls = [lambda: mod.quant(t, 1, 0.5, 0.1, 512, t, t), lambda: mod.prefill_static(t, t, t, t, 256, 2, 0.5, 0.1, 512, t),
             lambda: mod.gemv_grouped(t, [(t, t, 256, t)], 1, 0.5, 0.1)]
    for call in calls:
        if raised:
            with pytest.raises(error):
                call()
        else:
            assert call() is NotImplemented
    assert not seen


def test_without_the_module(both, monkeypatch, tmp_path):
    """An interpreter for which it is not built: every call takes the other way."""
    mod, seen, mp = both
    mp.setattr(mq, "FAST_PATH", str(tmp_path / "none.so"))
    mp.setattr(mq, "_fast", mq._load_fast())
    for name, call in calls().items():
        call()
        assert seen.pop()[0] == name


def test_the_module_belongs_to_one_build_and_interpreter(monkeypatch, tmp_path):
    from paper_2502_00425_amd import build as hip_build
    assert hip_build.CALL_LIB == mq.FAST_PATH and not hip_build.is_stale()
    assert hip_build.sysconfig.get_config_var("SOABI") in mq.FAST_PATH
    ids = {hip_build.source_hash(hip_build.CALL_SOURCES)}
    with monkeypatch.context() as m:
        m.setattr(hip_build, "CC_FLAGS", hip_build.CC_FLAGS + ["-g"])
        ids.add(hip_build.source_hash(hip_build.CALL_SOURCES))
    with monkeypatch.context() as m:
        m.setattr(hip_build.sysconfig, "get_config_var", lambda _: "cpython-399-other")
        ids.add(hip_build.source_hash(hip_build.CALL_SOURCES))
    assert len(ids) == 3
    # no compiler: the libraries are whole without the module, and one of other sources does not stay
    monkeypatch.setattr(hip_build, "CALL_LIB", str(tmp_path / "m.so"))
    monkeypatch.setenv("CC", "no-such-compiler")
    monkeypatch.setenv("HIPCC", "/no/such/hipcc")
    assert not hip_build.is_stale() and hip_build.ensure_fresh() == hip_build.LIB
    (tmp_path / "m.so").write_bytes(b"")
    assert hip_build.is_stale()
    hip_build.ensure_fresh()
    assert not (tmp_path / "m.so").exists() and not hip_build.is_stale()
    # with one the module is built without hipcc
    monkeypatch.delenv("CC")
    assert hip_build.is_stale()
    hip_build.ensure_fresh()
    assert (tmp_path / "m.so").exists() and not hip_build.is_stale()
