"""The launching calls' argument marshalling in C against the general way through ctypes: both reach the library with the same
arguments (a recording stand-in here, so no GPU), and what the first does not know goes the second way."""
import ctypes
import os
import subprocess
import sys
import sysconfig
import textwrap
import threading

import numpy as np
import pytest
import torch

import paper_2604_26666_amd as fact
from paper_2604_26666_amd import binding

NAMES = ("fact_gemm", "fact_gemm_batched", "fact_gemm_splitk", "fact_block_mlp", "fact_block_mlp_f16", "fact_attention", "fact_block_forward")


class General:
    """In the place of the C functions: nothing is known, every call goes through ctypes."""

    def __getattr__(self, name):
        return lambda *a: None


@pytest.fixture(scope="module")
def recorded():
    if not os.path.exists(fact.lib_path()):
        from paper_2604_26666_amd import build
        build.build()
    real, fast = binding.lib(), binding._fast_calls()
    calls, keep = [], []

    def value(x):
        if isinstance(x, ctypes.POINTER(binding._CEpilogue)):
            return tuple(getattr(x[0], f) for f, _ in binding._CEpilogue._fields_) if x else None
        if isinstance(x, ctypes.POINTER(binding._CBlock)):
            return tuple(getattr(x[0], f) for f, _ in binding._CBlock._fields_)
        if isinstance(x, ctypes.POINTER(ctypes.c_int64)):
            return tuple(x[:3])
        return x

    class Stub:
        pass

    stub, table = Stub(), {}
    for n in NAMES:
        proto = ctypes.CFUNCTYPE(ctypes.c_int, *getattr(real, n).argtypes)
        f = proto(lambda *a, n=n: calls.append((n,) + tuple(value(x) for x in a)) or 7)
        keep.append(f)
        setattr(stub, n, f)
        table[n] = ctypes.cast(f, ctypes.c_void_p).value
    streams = (torch.cuda.is_initialized, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
    fast.init(table, fact.Epilogue, fact.Block, streams)
    binding._lib = stub

    def run(name, *a, **k):
        calls.clear()
        out = []
        for way in (fast, General()):
            binding._fast = way
            assert getattr(fact, name)(*a, **k) == 7
            out.append(calls[-1])
        assert len(calls) == 2
        binding._fast = fast
        return out

    yield run
    binding._lib, binding._fast = real, None
    binding._fast_calls()


T = lambda *s: torch.zeros(*s, dtype=torch.bfloat16)
S = 0x7F00DEADBEE0


def test_gemm(recorded):
    A, B, C, bias = T(3, 5), T(5, 7), T(3, 7), T(7)
    ep = fact.Epilogue(bias=bias, residual=C, ldr=7, stride_r=2 ** 40, act=1, out_f32=1, f16=1)
    for e in (None, ep, fact.Epilogue(residual=0x1000)):
        for tb in (0, 1, True):
            one, two = recorded("fact_gemm", 3, 7, 5, A, 5, B, 7, tb, C, 7, e, S)
            assert one == two and one[4] == A.data_ptr() and one[8] == int(tb) and one[12] == S
    one, two = recorded("fact_gemm", -1, 2 ** 62, 0, None, 1, 2 ** 63 + 8, 1, 0, None, 1, stream=0)
    assert one == two
    one, two = recorded("fact_gemm_batched", 2, 3, 7, 5, A, 5, 15, B, 7, 35, 0, C, 7, 21, ep, S)
    assert one == two and len(one) == 17
    for split in (0, 9):
        one, two = recorded("fact_gemm_splitk", 3, 7, 5, A, 5, B, 7, 0, C, 7, ep, split, bias, 2 ** 40, S)
        assert one == two


def test_blocks_and_attention(recorded):
    t = [T(4) for _ in range(13)]
    for name in ("fact_block_mlp", "fact_block_mlp_f16"):
        one, two = recorded(name, 2, 3, 4, t[0], t[1], None, t[2], 1, t[3], t[4], None, t[5], t[6], t[7], 99, S)
        assert one == two and one[0] == name
    a = (1, 2, 3, 1, 64, t[0].data_ptr(), (1, 2, 3), t[1], [4, 5, 6], t[2], (7, 8, 9), t[3], (10, 11, 12))
    one, two = recorded("fact_attention", *a, 0, 0.25, S)
    assert one == two and one[7] == (1, 2, 3) and one[13] == (10, 11, 12)
    one, two = recorded("fact_attention", *a, stream=S)
    assert one == two
    names = ("norm1_g", "norm1_b", "Wqkv", "bqkv", "Wo", "bo", "norm2_g", "norm2_b", "W1", "W1u", "b1", "W2", "b2")
    b = fact.Block(1, 2, 3, 4, 5, 64, 7, 1, 2, rope=1, eps=1e-5, rope_base=500000.0, **dict(zip(names, t)))
    some = fact.Block(1, 2, 3, 4, 5, 64, 7, 0, 1, Wqkv=t[0], Wo=None, b2=0x2000)
    for blk in (b, some):
        one, two = recorded("fact_block_forward", blk, t[0], t[1], t[2], 77, S)
        assert one == two and one[0] == "fact_block_forward"


def test_what_c_does_not_know_goes_through_ctypes(recorded):
    A = T(4)

    class Wrapped:                                           # data_ptr() of a number that is no int
        def data_ptr(self):
            return np.int64(A.data_ptr())

    class Stream:
        cuda_stream = S

    class Ep(fact.Epilogue):
        pass

    one, two = recorded("fact_gemm", 3, 7, 5, Wrapped(), 5, A, 7, np.int32(1), A, 7, Ep(bias=A), Stream())
    assert one == two and one[4] == A.data_ptr() and one[12] == S and one[8] == 1
    one, two = recorded("fact_attention", 1, 2, 3, 1, 64, A, np.array([1, 2, 3]), A, (4, 5, 6), A, (7, 8, 9), A, (10, 11, 12), 1, 1, S)
    assert one == two and one[7] == (1, 2, 3)
    one, two = recorded("fact_block_forward", fact.Block(1, 2, 3, 4, 5, 64, 7, 0, 1, eps=1, Wqkv=A), A, A, A, 77, S)
    assert one == two


def test_the_same_errors(recorded):
    A = T(4)
    for bad, error in (((3, 7, 5, "A", 5, A, 7, 1, A, 7), AttributeError), ((3.0, 7, 5, A, 5, A, 7, 1, A, 7), ctypes.ArgumentError),
                       ((3, 7, 5, A, 5, A, 7, None, A, 7), TypeError)):
        with pytest.raises(error):
            fact.fact_gemm(*bad, None, S)
    with pytest.raises(TypeError):
        fact.fact_gemm(3, 7, 5, A)


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["default", "side", "nested", "thread", "thread with a stream"])
def test_no_stream_is_the_current_one(recorded, where):
    A = T(4)
    torch.cuda.synchronize()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    got = []

    def seen(want):
        one, two = recorded("fact_gemm", 3, 7, 5, A, 5, A, 7, 1, A, 7)
        blk = recorded("fact_block_forward", fact.Block(1, 2, 3, 4, 5, 64, 7, 0, 1, Wqkv=A), A, A, A, 77)
        got.extend((x[-1] or 0, want) for x in (one, two, *blk))
        assert torch.cuda.current_stream().cuda_stream == want and binding._fast.gemm(3, 7, 5, A, 5, A, 7, 1, A, 7, None, None) == 7

    def threads(s):
        with torch.cuda.stream(s):
            seen(s.cuda_stream)

    if where == "default":
        seen(0)
    elif where == "side":
        with torch.cuda.stream(side):
            seen(side.cuda_stream)
        seen(0)
    elif where == "nested":
        with torch.cuda.stream(side):
            with torch.cuda.stream(other):
                seen(other.cuda_stream)
            seen(side.cuda_stream)
    else:
        with torch.cuda.stream(side):                       # a new thread starts on the default stream
            t = threading.Thread(target=seen, args=(0,)) if where == "thread" else threading.Thread(target=threads, args=(other,))
            t.start()
            t.join()
            seen(side.cuda_stream)
    assert len(got) == (4 if where == "default" else 8) and all(a == b for a, b in got), got


def test_an_interrupt_ends_the_call(recorded):
    A = T(4)

    class Interrupted:
        times = 0

        def data_ptr(self):
            self.times += 1
            if self.times == 1:
                raise KeyboardInterrupt
            return A.data_ptr()

    i = Interrupted()
    for call in (lambda: fact.fact_gemm(3, 7, 5, i, 5, A, 7, 1, A, 7, None, S), lambda: fact.fact_gemm(3, 7, 5, A, 5, A, 7, 1, A, 7, fact.Epilogue(bias=i), S),
                 lambda: fact.fact_block_forward(fact.Block(1, 2, 3, 4, 5, 64, 7, 0, 1, Wqkv=i), A, A, A, 77, S)):
        i.times = 0
        with pytest.raises(KeyboardInterrupt):
            call()
        assert i.times == 1


def python(code, **env):
    return subprocess.run([sys.executable, "-c", textwrap.dedent(code)], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                          env={**os.environ, **env}, capture_output=True, text=True, timeout=240)


@pytest.mark.parametrize("absent", ["torch", "paper_2604_26666_amd._pycall"])
def test_addresses_and_streams_need_neither_torch_nor_the_extension(recorded, absent):
    # a module that is None in sys.modules cannot be imported; the calls are refused by the library, not by the binding
    r = python(f"""
        import sys
        sys.modules[{absent!r}] = None
        import paper_2604_26666_amd as fact
        p = 4096
        assert fact.fact_gemm(0, 8, 8, p, 8, p, 8, 1, p, 8, fact.Epilogue(bias=p), 0) == -2
        assert fact.fact_attention(0, 8, 1, 1, 64, p, (8, 64, 64), p, (8, 64, 64), p, (8, 64, 64), p, (8, 64, 64), 1, 0.0, 0) == -2
    """)
    assert r.returncode == 0, r.stderr


def test_torch_that_comes_later_brings_its_streams(recorded):
    r = python("""
        import sys
        import paper_2604_26666_amd as fact
        p = 4096
        assert fact.fact_gemm(0, 8, 8, p, 8, p, 8, 1, p, 8, None, 0) == -2 and "torch" not in sys.modules
        import torch
        torch.cuda.current_stream = lambda: type("S", (), {"cuda_stream": 0})()
        assert fact.fact_gemm(0, 8, 8, p, 8, p, 8, 1, p, 8) == -2
        bound = []
        from paper_2604_26666_amd import _pycall, binding
        init = _pycall.init
        _pycall.init = lambda *a: (bound.append(a[3]), init(*a))
        assert fact.fact_gemm(0, 8, 8, p, 8, p, 8, 1, p, 8) == -2 and fact.fact_gemm(0, 8, 8, p, 8, p, 8, 1, p, 8) == -2
        assert len(bound) == 1 and bound[0] is not None
    """)
    assert r.returncode == 0, r.stderr


def test_the_extension_carries_its_interpreters_tag(recorded):
    from paper_2604_26666_amd import _pycall, build
    assert build.PYCALL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.samefile(_pycall.__file__, build.PYCALL)
