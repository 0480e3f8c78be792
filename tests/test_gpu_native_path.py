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
