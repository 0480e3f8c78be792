"""GPU parity of mixfp4_gemm(workspace="auto") on the direct GEMM (A decoded
once, W decoded between the MFMAs) against the oracle's fp64 GEMM of the
exactly dequantized operands: |C - C_ref| <= 1e-5 * sum|a*w| + 1e-6
element-wise, the tolerance of mixfp4_gemm."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from oracle import gemm as G
from oracle import quant as Q
from tests._gpu import dev_f32, dev_u8, host, log

pytestmark = pytest.mark.gpu


def _dev(q):
    return (dev_u8(q.codes), dev_u8(q.scales), dev_f32(q.s32))


def _rows(q, rows):
    return Q.Quantized(codes=q.codes[rows], scales=q.scales[rows], s32=q.s32, t=None,
                       sf_code=None, si_code=None, delta=None)


def _check(c, qa, qw, m, n):
    rng = np.random.default_rng(m * n)
    rows = np.unique(np.concatenate([[0, m - 1], rng.integers(0, m, 48)]))
    cols = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 200)]))
    a_hat, w_hat = G.operands(_rows(qa, rows), _rows(qw, cols))
    c_ref, bound = G.gemm(a_hat, w_hat)
    ok, worst = G.within_tolerance(c[np.ix_(rows, cols)], c_ref, bound)
    assert ok.all(), f"{(~ok).sum()} elements out of tolerance, worst ratio {worst}"
    assert np.isfinite(c).all()


def _need(m, n, k):
    import paper_2605_31035_amd as M
    b = ctypes.c_int64(0)
    assert M.lib.mixfp4_gemm_auto_workspace_size(m, n, k, ctypes.byref(b)) == 0
    return b.value


def _auto_against_oracle(m, n, k):
    import paper_2605_31035_amd as M
    if n * k < 1 << 22:
        qa, qw = Q.quantize(W.adversarial(m + 3 * k, m, k)), Q.quantize(W.adversarial(n + k, n, k))
        a, w = _dev(qa), _dev(qw)
    else:                                                       # quantized on the device
        from tests._gpu import gpu_quantize
        a = gpu_quantize(W.adversarial(m + 3 * k, m, k))
        w = gpu_quantize(W.adversarial(n + k, n, k))
        qa, qw = (Q.Quantized(codes=host(x[0]), scales=host(x[1]), s32=host(x[2])[0], t=None,
                              sf_code=None, si_code=None, delta=None) for x in (a, w))
    out = torch.full((m, n), float("nan"), device="cuda")
    c = M.mixfp4_gemm(a, w, out=out, workspace="auto")
    again = M.mixfp4_gemm(a, w, workspace="auto")
    torch.cuda.synchronize()
    assert torch.equal(c, again)
    _check(host(c), qa, qw, m, n)


def test_direct_falls_back():
    """Too little workspace, or W scales that are not word aligned: what
    mixfp4_gemm computes."""
    import paper_2605_31035_amd as M
    m, n, k = 70, 300, 512
    qa, qw = Q.quantize(W.adversarial(5, m, k)), Q.quantize(W.adversarial(6, n, k))
    a, w = _dev(qa), _dev(qw)
    ref = M.mixfp4_gemm(a, w)
    need = _need(m, n, k)
    out = torch.full((m, n), float("nan"), device="cuda")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    p = ctypes.c_void_p

    def call(scales, nbytes):
        assert M.lib.mixfp4_gemm_auto(
            p(a[0].data_ptr()), p(a[1].data_ptr()), p(a[2].data_ptr()), p(w[0].data_ptr()),
            p(scales.data_ptr()), p(w[2].data_ptr()), m, n, k, p(out.data_ptr()),
            p(ws.data_ptr()), nbytes, None) == 0
        torch.cuda.synchronize()
        return out
    assert torch.equal(call(w[1], need - 1), ref)
    odd = torch.empty(n * (k // 16) + 4, dtype=torch.uint8, device="cuda")[1:1 + n * (k // 16)]
    odd.copy_(w[1].reshape(-1))
    assert odd.data_ptr() % 4 == 1
    _check(host(call(odd, need)), qa, qw, m, n)


# One row or more per tile configuration (rows x columns of a workgroup),
# with ragged edges, every K remainder of 256 and shares of K that differ by a
# step.
@pytest.mark.parametrize("m,n,k", [
    (17, 33, 576), (64, 4090, 576), (33, 130, 704), (500, 1001, 832),      # 32 x 32
    (31, 14300, 3008), (17, 16300, 4096),                  # 32 x 64
    (100, 4090, 4096), (128, 4090, 3008),                  # 64 x 32
    (33, 9001, 640), (64, 8200, 1024), (129, 4001, 640), (500, 1999, 832),  # 64 x 64
    (33, 17003, 1024), (33, 17003, 1280),                  # 64 x 128
    (65, 8235, 704),                                       # 128 x 64
    (67, 16907, 3072), (647, 10782, 512), (131, 24372, 1536),              # 128 x 128
    (133, 18715, 1280), (500, 11001, 2048),                # 128 x 256, K halved over the waves
    (257, 22173, 576), (300, 21903, 640),                  # 128 x 256, two workgroups per CU
])
def test_direct_tiles(m, n, k):
    log(f"direct gemm m={m} n={n} k={k}")
    assert _need(m, n, k) == (m + 255) // 256 * 256 * k * 2     # A decoded, W packed
    _auto_against_oracle(m, n, k)


# Short K and many rows or columns: one launch of the fused kernel, no workspace.
@pytest.mark.parametrize("m,n,k", [
    (17, 33, 256), (33, 130, 320), (31, 8200, 320), (129, 17003, 320), (33, 9001, 320),
    (64, 28672, 576), (129, 17003, 256), (65, 8200, 576), (509, 11001, 320), (65, 17003, 384),
    (509, 16300, 256), (500, 11001, 1024), (129, 28672, 320), (509, 28672, 576),
    (768, 4096, 1024), (1024, 2048, 512),
    (17, 33, 544), (17, 8192, 1056), (100, 600, 800)])          # K % 64 = 32
def test_short_k_takes_no_workspace(m, n, k):
    log(f"auto without workspace m={m} n={n} k={k}")
    assert _need(m, n, k) == 0
    _auto_against_oracle(m, n, k)


@pytest.mark.parametrize("m,n,k", [(70, 300, 1056), (17, 2048, 4000)])
def test_k_of_32_takes_two_passes(m, n, k):
    """K % 64 = 32 where W's decode is the smaller cost: both operands decoded,
    bit for bit as with the workspace given."""
    import paper_2605_31035_amd as M
    assert _need(m, n, k) == M.mixfp4_gemm_workspace_size(m, n, k) > 0
    qa, qw = Q.quantize(W.adversarial(m, m, k)), Q.quantize(W.adversarial(n, n, k))
    a, w = _dev(qa), _dev(qw)
    c = M.mixfp4_gemm(a, w, workspace="auto")
    assert torch.equal(c, M.mixfp4_gemm(a, w, workspace=True))
    _check(host(c), qa, qw, m, n)


@pytest.mark.parametrize("m,n,k,two", [(2048, 4096, 512, True), (1300, 100, 1024, False),
                                       (4096, 4096, 4096, True), (200, 1000, 1056, True)])
def test_unaligned_w_scales(m, n, k, two):
    """W's scale bytes off a word: the direct GEMM does not read them; products
    that pay for two passes still take them (they write the workspace)."""
    import paper_2605_31035_amd as M
    from tests._gpu import gpu_quantize
    log(f"unaligned W scales {m}x{n}x{k}")
    a, w = gpu_quantize(W.adversarial(m, m, k)), gpu_quantize(W.adversarial(n, n, k))
    buf = torch.empty(w[1].numel() + 1, dtype=torch.uint8, device="cuda")
    shifted = buf[1:].view(w[1].shape).copy_(w[1])
    assert shifted.data_ptr() % 4 == 1
    ws = torch.zeros(M.mixfp4_gemm_workspace_size(m, n, k), dtype=torch.uint8, device="cuda")
    c = torch.full((m, n), float("nan"), device="cuda")
    p = M._ptr
    assert M.lib.mixfp4_gemm_auto(p(a[0]), p(a[1]), p(a[2]), p(w[0]), p(shifted), p(w[2]), m, n, k,
                                  p(c), p(ws), ws.numel(), M._stream(c.device)) == 0
    assert bool(ws.any()) == two
    want = M.mixfp4_gemm(a, w, workspace=True if two else None)
    assert torch.equal(c, want)
    assert torch.equal(M.mixfp4_gemm(a, (w[0], shifted, w[2]), workspace="auto"), want)
