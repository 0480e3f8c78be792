"""The binding's native call path (one C++ call per layer) and what the Python
path behind it takes over: other Python threads run while it allocates and
launches, unused options are not looked at, and memory that only speeds a call
up is done without where there is none."""
import ctypes
import gc
import sys
import threading

import pytest
import torch

from tests._gpu import log

pytestmark = pytest.mark.gpu


def _x(rows, k, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(rows, k, generator=g, device="cuda").to(torch.bfloat16)


def _calls():
    import paper_2605_31035_amd as M
    from paper_2605_31035_amd._lib import native
    x, w = _x(16, 256), M.mixfp4_quantize(_x(64, 256, 1))
    a, small = M.mixfp4_quantize(x), M.mixfp4_quantize(x[:1, :64])
    sync = torch.zeros(4, dtype=torch.int32, device="cuda")
    return {"quantize": lambda: native.quantize(x, None, 0, 0, None, 0, 0),
            "gemm": lambda: native.gemm(a, w, True),
            "decode_step": lambda: native.decode_step(x, w, sync),
            "dequantize": lambda: native.dequantize(*small)}


def _flat(r):
    return [t for v in r for t in _flat(v)] if isinstance(r, tuple) else [r]


@pytest.mark.parametrize("rows,k,opt", [
    (3, 64, dict()), (65, 4096, dict()), (48, 320, dict(mode="e1m2", rounding="stochastic", seed=7)),
    (2048, 128, dict(hadamard_block=128)), (64, 96, dict(transpose=True, hadamard_block=16)),
    (33, 256, dict(mode="four_six", offset=1 << 40, rounding="stochastic", seed=-1))])
def test_native_equals_python(rows, k, opt):
    """The Python path (here with outputs given) and the native one."""
    import paper_2605_31035_amd as M
    from paper_2605_31035_amd._lib import native
    x = _x(rows, k + 8)[:, :k]
    flags = (M._MODES[opt.get("mode", "mixfp4")] | (M.STOCHASTIC if "rounding" in opt else 0)
             | (M.TRANSPOSE if "transpose" in opt else 0))
    log(f"native quantize {rows}x{k} {opt}")
    got = native.quantize(x, None, flags, opt.get("hadamard_block", 0), None, opt.get("seed", 0),
                          opt.get("offset", 0))
    want = M.mixfp4_quantize(x, codes=torch.empty_like(got[0]), **opt)
    given = M.mixfp4_quantize(x, got[2], scales=torch.empty_like(got[1]), **opt)
    for g, w, s in zip(got, want, given):
        assert torch.equal(g, w) and torch.equal(g, s)
    assert torch.equal(native.dequantize(*got), M.mixfp4_dequantize(_Sub(got[0]), *got[1:]))


@pytest.mark.parametrize("m", [1, 16, 17, 100])
def test_native_gemm_equals_python(m):
    import paper_2605_31035_amd as M
    from paper_2605_31035_amd._lib import native
    x, w = _x(m, 576), M.mixfp4_quantize(_x(272, 576, 1))
    a = M.mixfp4_quantize(x)
    log(f"native gemm m={m}")
    for auto in (False, True):
        want = M.mixfp4_gemm(list(a), list(w), workspace="auto" if auto else None)
        assert torch.equal(native.gemm(a, w, auto), want)
    if m <= 16:
        sync = torch.zeros(4, dtype=torch.int32, device="cuda")
        got = native.decode_step(x, w, sync)
        want = M.mixfp4_decode_step(x, list(w), sync=sync)
        for g, v in zip(_flat(got), _flat(want)):
            assert torch.equal(g, v)


class _Sub(torch.Tensor):
    """A subclass: its owner may want to see the call."""

    def __new__(cls, t):
        return t.as_subclass(cls)


class _Seen(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


class _Dispatched(torch.utils._python_dispatch.TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_what_is_declined():
    """The native functions return None, and leave the rest to Python, for what
    they do not take as it is."""
    import paper_2605_31035_amd as M
    from paper_2605_31035_amd._lib import native
    x, w = _x(16, 256), M.mixfp4_quantize(_x(64, 256, 1))
    a = M.mixfp4_quantize(x)
    sync = torch.zeros(4, dtype=torch.int32, device="cuda")
    log("native: declined arguments")

    def quantize(v, s=None, block=0, signs=None, seed=0):
        return native.quantize(v, s, 1 if s is not None else 0, block, signs, seed, 0)
    assert quantize(x) is not None and quantize(torch.nn.Parameter(x)) is not None
    for v in (_Sub(x), x.cpu(), x.float(), x.t(), x[0], x[:, :24], x[:0], x[:, ::2], None, 1.0,
              torch.empty_like(x, device="meta")):
        assert quantize(v) is None, v
    one = torch.ones(1, device="cuda")
    for s in (one.cpu(), one.double(), torch.ones(2, device="cuda"), _Sub(one), 1.0):
        assert quantize(x, s) is None, s
    signs = torch.ones(16, dtype=torch.int8, device="cuda")
    assert quantize(x, block=16, signs=signs) is not None
    for g in (signs.cpu(), signs.int(), signs[:8], torch.ones(32, dtype=torch.int8, device="cuda")[::2]):
        assert quantize(x, block=16, signs=g) is None, g
    for bad in (dict(block=17), dict(block=512), dict(block=-16), dict(block="16"),
                dict(block=0.0), dict(signs=signs), dict(seed=None), dict(seed=0.5)):
        assert quantize(x, **bad) is None, bad
    assert native.gemm(a, w, True) is not None and native.decode_step(x, w, sync) is not None
    for o in (list(a), a[:2], (a[0], a[1].cpu(), a[2]), (a[0].int(), *a[1:]), (a[0], a[1][:8], a[2]),
              (a[0].t().contiguous().t(), *a[1:]), (_Sub(a[0]), *a[1:]), (a[0][:, :64], *a[1:]), None):
        assert native.gemm(o, w, True) is None and native.gemm(w, o, False) is None, o
        assert native.decode_step(x, o, sync) is None, o
    for v in (_x(17, 256), _x(16, 240), _x(16, 264)[:, :256], x.float(), x.cpu()):
        assert native.decode_step(v, w, sync) is None
    assert native.decode_step(x, w, sync[:3]) is None and native.decode_step(x, w, None) is None
    for d in ((a[0].cpu(), a[1]), (a[0], a[1][:, :8]), (a[0][:, :64], a[1]), (_Sub(a[0]), a[1]), (1, 2)):
        assert native.dequantize(*d, None) is None
    for mode in (_Seen(), _Dispatched()):
        with mode:
            assert quantize(x) is None and native.gemm(a, w, True) is None
            assert native.decode_step(x, w, sync) is None and native.dequantize(*a) is None
            got = M.mixfp4_quantize(x)
        for g, v in zip(got, a):
            assert torch.equal(g, v)


@pytest.mark.parametrize("name", ["quantize", "gemm", "decode_step", "dequantize"])
@pytest.mark.parametrize("second_thread", [False, True])
def test_current_stream_is_used(name, second_thread):
    """Behind a wait on a stream of its own, while the default stream stays idle;
    the current stream is a thread's own."""
    call = _calls()[name]
    want, side, out = _flat(call()), torch.cuda.Stream(), {}
    torch.cuda.synchronize()

    def work():
        with torch.cuda.stream(side):
            torch.cuda._sleep(200_000_000)              # about 0.1 s
            out["got"] = call()
            out["behind"] = not side.query()
            out["idle"] = torch.cuda.default_stream().query()
    log(f"native {name} on a stream, second thread: {second_thread}")
    if second_thread:
        t = threading.Thread(target=work)
        t.start()
        t.join()
    else:
        work()
    assert out["behind"] and out["idle"]
    side.synchronize()
    for g, w in zip(_flat(out["got"]), want):
        assert torch.equal(g, w)


@pytest.mark.parametrize("name", ["quantize", "gemm", "decode_step", "dequantize"])
def test_other_threads_run(name):
    """With a switch interval that the interpreter never reaches, a thread that
    waits for it only gets it when a call lets go of it.  The outputs are kept
    until the end, and are small: freeing a tensor or taking more memory from
    the device lets go of it as well."""
    call = _calls()[name]
    gate, ran, kept = threading.Lock(), [], []
    gate.acquire()

    def other():
        gate.acquire()
        ran.append(True)

    log(f"native {name} beside another thread")
    t = threading.Thread(target=other)
    t.start()
    before = sys.getswitchinterval()
    gc.collect()
    gc.disable()
    sys.setswitchinterval(60.0)
    try:
        gate.release()
        for _ in range(50):
            for _ in range(100):
                kept.append(call())
            if ran:
                break
    finally:
        sys.setswitchinterval(before)
        gc.enable()
    seen = bool(ran)
    t.join()
    torch.cuda.synchronize()
    assert seen and all(r is not None for r in kept)


@pytest.mark.parametrize("unused", [dict(seed=None, offset=None), dict(seed=1.5),
                                    dict(hadamard_block=0.0),
                                    dict(hadamard_signs=torch.ones(16, dtype=torch.int8))])
def test_unused_options_are_not_looked_at(unused):
    """Rounding to nearest without rotation or transposition takes no draws, no
    block and no signs: what stands in their place does not matter."""
    import paper_2605_31035_amd as M
    x = _x(5, 64)
    log(f"unused options {unused}")
    for g, w in zip(M.mixfp4_quantize(x, **unused), M.mixfp4_quantize(x)):
        assert torch.equal(g, w)


@pytest.fixture
def scarce():
    """Limits this process to so many bytes of new device memory."""
    def limit(spare):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        total = torch.cuda.get_device_properties(0).total_memory
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + spare) / total)
    yield limit
    torch.cuda.set_per_process_memory_fraction(1.0)


@pytest.mark.parametrize("m,n,k", [(40, 4096, 8032), (300, 2048, 16384)])
def test_auto_without_room_for_its_workspace(scarce, m, n, k):
    """workspace="auto" computes mixfp4_gemm's product where the route's
    workspace cannot be had (two passes with 70 MB, A decoded with 17 MB)."""
    import paper_2605_31035_amd as M
    a, w = M.mixfp4_quantize(_x(m, k)), M.mixfp4_quantize(_x(n, k, 1))
    want, need = M.mixfp4_gemm(a, w), ctypes.c_int64(0)
    assert M.lib.mixfp4_gemm_auto_workspace_size(m, n, k, ctypes.byref(need)) == 0
    assert need.value >= 16 << 20
    log(f"auto without memory {m}x{n}x{k}")
    scarce(8 << 20)
    with pytest.raises(torch.OutOfMemoryError):
        M.mixfp4_gemm(a, w, workspace=True)
    assert torch.equal(M.mixfp4_gemm(a, w, workspace="auto").cpu(), want.cpu())


@pytest.mark.parametrize("opt", [dict(), dict(hadamard_block=128), dict(transpose=True)])
def test_quantize_without_room_for_scratch(scarce, opt):
    """Codes and scales fit exactly; nothing is left for scratch."""
    import paper_2605_31035_amd as M
    x = _x(8192, 4096)
    want = M.mixfp4_quantize(x, **opt)
    out = dict(codes=torch.empty_like(want[0]), scales=torch.empty_like(want[1]),
               scale_out=torch.empty_like(want[2]))
    log(f"quantize without memory {opt}")
    scarce(0)
    held = []                                   # what is left of the segments in use
    for size in (1 << 20, 1 << 16, 1 << 12, 512):
        try:
            while True:
                held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass
    for g, w in zip(M.mixfp4_quantize(x, **out, **opt), want):
        assert torch.equal(g.cpu(), w.cpu())    # the comparison takes memory too
