"""The binding's native call path (one C++ call per layer): it lets other
Python threads run while it allocates and launches."""
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
