"""The extension module that carries a layer's calls to the library: the same results, errors and refusals as through ctypes."""
import ctypes
import threading
import time

import numpy as np
import pytest
import torch

from paper_2603_08185_amd import binding as serq

DEV = "cuda:0"
NAMES = ["quantize_act", "swiglu_quantize_act", "mx_quantize_act", "mx_swiglu_quantize_act", "quantize_act_asym", "linear",
         "mx_linear", "g128_linear"]


class _General:
    """In place of the module: every call takes the general way."""

    def __getattr__(self, name):
        return lambda *a: None


class _Seen:
    """Passes on to the module and notes what came back."""

    def __init__(self, mod):
        self.mod, self.codes = mod, []

    def __getattr__(self, name):
        def call(*a):
            rc = getattr(self.mod, name)(*a)
            self.codes.append(rc)
            return rc
        return call


def test_refuses_what_is_not_plain():
    serq.lib()
    f = serq._fast
    x = torch.zeros((2, 64), dtype=torch.bfloat16)
    u = torch.zeros(128, dtype=torch.uint8)
    s = torch.zeros(2)
    assert f.quantize_act(x, None, 8, u, s) is None                       # not in device memory
    assert f.swiglu_quantize_act(x, x, None, 8, u, s) is None
    assert f.mx_quantize_act(x, None, u, u) is None
    assert f.mx_swiglu_quantize_act(x, x, None, u, u) is None
    assert f.quantize_act_asym(x, None, 8, u, s, s) is None
    for bad in (8.0, None, "8", True, np.int64(8), 1 << 40, 1 << 70):     # an int is a plain one and fits
        assert f.linear(u, s, bad, u, s, 0, 0, None, 2, 1, 32, 64, x, None, 0) is None
        assert f.g128_linear(u, s, None, bad, u, u, s, 0, 0, None, 2, 1, 32, 128, x, 0) is None
        assert f.mx_linear(u, u, u, u, 0, bad, None, None, 1, 32, 64, x, None, 0) is None
    assert f.linear(u, s, 8, u, s, 0, 0, None, 2, 1, 32, 64, x.double(), None, 0) is None   # no such type of output
    assert f.linear([1], s, 8, u, s, 0, 0, None, 2, 1, 32, 64, x, None, 0) is None
    with pytest.raises(ValueError):                                       # and the general way names the error
        serq.quantize_act(x, None, 8, u, s)
    with pytest.raises(TypeError):
        f.linear(u)
    with pytest.raises(TypeError):
        f.bind(1, 2)
    with pytest.raises(ValueError):
        f.bind(*([0] * len(NAMES)))


def test_packing_and_sizes_do_without_the_module(monkeypatch, tmp_path):
    (tmp_path / "broken.so").write_bytes(b"not a library")
    for path in (tmp_path / "missing.so", tmp_path / "broken.so"):
        for name in ("_lib", "_fast", "_fast_error"):
            monkeypatch.setattr(serq, name, None)
        monkeypatch.setattr(serq, "FASTCALL_PATH", str(path))
        assert serq.lib().serq_packed_weight_bytes(64, 128) == 64 * 128 // 2
        x, u, s = torch.zeros((1, 128), dtype=torch.bfloat16), torch.zeros(128, dtype=torch.uint8), torch.zeros(1)
        for call in (lambda: serq.quantize_act(x, None, 8, u, s), lambda: serq.linear(u, s, 8, u, s, 1, 64, 128, Y=x)):
            with pytest.raises(ImportError, match="build it with"):       # and no silent other way for a layer's calls
                call()


def _calls(dt, M, K=384, N=96, r=32):
    g = torch.Generator().manual_seed(M)
    wide = torch.randn((M + 1, K + 64), generator=g).to(dt).to(DEV)
    X, U = wide[:M, :K], torch.randn((M, K), generator=g).to(dt).to(DEV)  # rows with a stride of their own, and dense ones
    W, s = torch.randn((N, K), generator=g).to(dt).to(DEV), torch.rand(K, generator=g).to(DEV) + 0.5
    L, G, Q = serq.pack_weights(W, s, r, r_dtype=dt), serq.g128_pack_weights(W, s, r, r_dtype=dt), serq.mx_pack_weights(W, s, r)
    big = torch.zeros((M + 1, N + 16), dtype=dt, device=DEV)
    u8 = lambda n: torch.zeros(max(n, 16), dtype=torch.uint8, device=DEV)
    f32, i32 = (lambda: torch.zeros(M, device=DEV)), (lambda: torch.zeros(M, dtype=torch.int32, device=DEV))
    xs = serq.lib().serq_mx_act_scale_bytes(M, K)

    def run():
        out = []
        for ab in (4, 8):
            out += [*serq.quantize_act(X, L.s_inv, ab, u8(M * K), f32()), *serq.quantize_act(U, None, ab, u8(M * K), f32()),
                    *serq.swiglu_quantize_act(X, U, L.s_inv, ab, u8(M * K), f32()),
                    *serq.quantize_act_asym(X, G.s_inv, ab, u8(M * K), f32(), i32())]
            xq, sc = serq.quantize_act(U, L.s_inv, ab)
            for kw in (dict(), dict(Rp=L.Rp, r=r, r_dtype=dt), dict(Rp=serq.pack_lowrank_q4(L.R), r=r, r_dtype=serq.I4)):
                out.append(serq.linear(xq, sc, ab, L.Wq, L.wscale, M, N, K, ws=serq.workspace(M, N, K, r, ab, DEV), **kw).clone())
                out.append(serq.linear(xq, sc, ab, L.Wq, L.wscale, M, N, K, Y=big[:M, 8:8 + N], **kw).clone())
            xq, sc, z = serq.quantize_act_asym(U, G.s_inv, ab)
            for zz, rp in ((z, G.Rp), (None, None)):
                out.append(serq.g128_linear(xq, sc, zz, ab, G.Wq, G.gscale, G.wsum, M, N, K, Rp=rp, r=r if rp is not None else 0,
                                            r_dtype=dt, out_dtype=torch.float32))
        out += [*serq.mx_quantize_act(X, Q.s_inv, u8(M * K), u8(xs)), *serq.mx_swiglu_quantize_act(X, U, None, u8(M * K), u8(xs))]
        xq, xsc = serq.mx_quantize_act(U, Q.s_inv)
        out.append(serq.mx_linear(xq, xsc, Q.Wq, Q.wsc, M, N, K, Rq=Q.Rq, rsc=Q.rsc, r=r, ws=serq.mx_workspace(M, N, K, DEV)))
        out.append(serq.mx_linear(xq, xsc, Q.Wq, Q.wsc, M, N, K, Y=big[:M, 8:8 + N]).clone())
        return out
    return run


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("M", [0, 1, 40])
def test_same_as_the_general_way(dt, M, monkeypatch):
    run = _calls(dt, M)
    seen = _Seen(serq._fast)
    monkeypatch.setattr(serq, "_fast", seen)
    fast = run()
    assert seen.codes and all(c == 0 for c in seen.codes)                 # none was refused
    monkeypatch.setattr(serq, "_fast", _General())
    general = run()
    assert len(fast) == len(general)
    for a, b in zip(fast, general):
        assert a.shape == b.shape and torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_current_stream_and_errors(monkeypatch):
    run = _calls(torch.bfloat16, 7)
    want = run()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    x = torch.randn((3, 128), device=DEV).bfloat16()
    xq, sc = torch.zeros(3 * 128, dtype=torch.uint8, device=DEV), torch.zeros(3, device=DEV)
    with torch.cuda.graph(g, stream=st):                                  # recorded only if it goes to the current stream
        serq.quantize_act(x, None, 8, xq, sc)
    assert not xq.any()
    g.replay()
    torch.cuda.synchronize()
    assert xq.any() and all(torch.equal(a, b) for a, b in zip(want, run()))
    for fast in (serq._fast, _General()):
        monkeypatch.setattr(serq, "_fast", fast)
        for call, code in ((lambda: serq.quantize_act(x, None, 5, xq, sc), -2), (lambda: serq.quantize_act(x[:, :100], None, 8, xq, sc), -3),
                           (lambda: serq.linear(xq, sc, 8, xq, sc, 3, 48, 128, Y=x), -3),
                           (lambda: serq.g128_linear(xq, sc, None, 8, xq, xq, sc, 3, 64, 64, Y=x), -3),
                           (lambda: serq.mx_linear(xq, xq, xq, xq, 3, 64, 128, Y=x, r=33), -3)):
            with pytest.raises(serq.SerqError) as e:
                call()
            assert e.value.code == code
        with pytest.raises(ValueError):
            serq.quantize_act(x.t(), None, 8, xq, sc)
        with pytest.raises(ValueError):
            serq.swiglu_quantize_act(x, x[:2], None, 8, xq, sc)
        with pytest.raises(KeyError):
            serq.quantize_act(x.double(), None, 8, xq, sc)
        with pytest.raises(KeyError):
            serq.linear(xq, sc, 8, xq, sc, 3, 64, 128, r_dtype=torch.int32, Y=x)


# The entry point is a wait of the C library here (for a semaphore in the first operand, until the time in the second): it can only
# end in time if the thread that posts gets the interpreter lock.
@pytest.mark.gpu
@pytest.mark.parametrize("name", ["linear", "mx_linear", "g128_linear"])
def test_interpreter_lock_is_free_during_the_call(name):
    L, f, libc = serq.lib(), serq._fast, ctypes.CDLL(None, use_errno=True)
    real = [ctypes.cast(getattr(L, n), ctypes.c_void_p).value for n in serq._FAST]
    wait = ctypes.cast(libc.sem_timedwait, ctypes.c_void_p).value
    sem, until = torch.zeros(16, dtype=torch.int64), torch.zeros(2, dtype=torch.int64)
    until[0] = int(time.clock_gettime(time.CLOCK_REALTIME)) + 4
    libc.sem_init(ctypes.c_void_p(sem.data_ptr()), 0, 0)
    y = torch.zeros((1, 64), dtype=torch.bfloat16)
    args = {"linear": (sem, until, 8, sem, sem, 0, 0, None, 2, 1, 64, 128, y, None, 0),
            "mx_linear": (sem, until, sem, sem, 0, 0, None, None, 1, 64, 128, y, None, 0),
            "g128_linear": (sem, until, None, 8, sem, sem, sem, 0, 0, None, 2, 1, 64, 128, y, 0)}[name]
    inside = threading.Event()

    def post():
        inside.wait()
        time.sleep(0.2)                                                   # the call has begun
        libc.sem_post(ctypes.c_void_p(sem.data_ptr()))

    t = threading.Thread(target=post)
    t.start()
    try:
        f.bind(*(wait if n == "serq_" + name else r for n, r in zip(serq._FAST, real)))
        inside.set()
        assert getattr(f, name)(*args) == 0                               # -1: timed out
    finally:
        f.bind(*real)
        inside.set()
        t.join()
