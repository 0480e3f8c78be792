"""Rotation edges: tensors whose last row of 16 lanes holds a single Hadamard
block, sums on bf16 midpoints (exact ties and inexact ones), and non-finite
inputs, whose tensor scale is that of the rotated tensor."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import hadamard as HD
from oracle import quant as Q
from tests._gpu import dev_bf16, host, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,rows,k", [(128, 1, 128), (128, 3, 128), (128, 5, 384), (128, 37, 640),
                                      (64, 3, 64), (256, 3, 256), (16, 3, 48)])
def test_rotate_then_quantize_tails(b, rows, k):
    import paper_2605_31035_amd as M
    rng = np.random.default_rng(rows * k)
    # small integers: sums with few bits, many exactly halfway between two
    # bf16 values; scaled by 2^20 in places, so that others need more than 24
    x = rng.integers(-255, 256, (rows, k)).astype(np.float32)
    x[:, ::7] *= np.float32(2.0 ** 20)
    bits = W.f32_to_bf16_bits(x)
    signs = rng.choice([-1, 1], size=b)
    log(f"rotation tails b={b} rows={rows} k={k}")
    sg = torch.from_numpy(signs.astype(np.int8)).cuda()
    rot = HD.hadamard(bits, b, signs)
    y = M.mixfp4_hadamard(dev_bf16(bits), b, sg)
    np.testing.assert_array_equal(host(y.view(torch.int16)).view(np.uint16), rot)
    codes, scales, s32 = M.mixfp4_quantize(dev_bf16(bits), hadamard_block=b, hadamard_signs=sg)
    ref = Q.quantize(rot)
    assert host(s32)[0] == ref.s32
    np.testing.assert_array_equal(host(codes), ref.codes)
    np.testing.assert_array_equal(host(scales), ref.scales)


@pytest.mark.parametrize("b", [16, 64, 128])
@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("bad", [[np.inf], [np.inf, -np.inf], [np.nan]])
def test_scale_of_non_finite(b, transpose, bad):
    """s32 is formed from max|bits| of the rotated tensor, also where an
    infinity spreads over its block or cancels to NaN."""
    import paper_2605_31035_amd as M
    if transpose and b > 64:
        pytest.skip("a transposed rotation takes at most 64 rows")
    rng = np.random.default_rng(b)
    x = torch.from_numpy(rng.standard_normal((256, 256)).astype(np.float32)).cuda().bfloat16()
    for i, v in enumerate(bad):
        x[2 * i * transpose, 2 * i] = v
    log(f"rotation of non-finite values b={b} transpose={transpose} {bad}")
    got = M.mixfp4_quantize(x, hadamard_block=b, transpose=transpose)[2]
    rot = M.mixfp4_hadamard(x.t().contiguous() if transpose else x, b)
    mag = int((rot.view(torch.int16).to(torch.int32) & 0x7FFF).max())
    amax = torch.tensor([mag], dtype=torch.int32).to(torch.int16).view(torch.bfloat16).float()
    want = amax / 2688 if bool(amax > 0) else torch.ones(1)
    assert float(got) == float(want)


@pytest.mark.parametrize("b,rows,k,pad,mode,rounding", [
    (128, 1025, 128, 0, "mixfp4", "nearest"), (256, 515, 256, 16, "four_six", "nearest"),
    (128, 347, 384, 16, "mixfp4", "stochastic"), (256, 257, 512, 0, "e2m1", "stochastic"),
    (64, 300, 448, 0, "mixfp4", "nearest")])
def test_rotated_copy_in_scratch(b, rows, k, pad, mode, rounding):
    """The scratch with room for the rotated tensor (rows * k > 2^17), against
    the same call on the rotated tensor and with the maxima's scratch only."""
    import paper_2605_31035_amd as M
    x = torch.from_numpy(W.adversarial(rows, rows, k + pad).view(np.int16)).cuda().view(
        torch.bfloat16)[:, :k]
    sg = torch.from_numpy(np.random.default_rng(b).choice([-1, 1], b).astype(np.int8)).cuda()
    log(f"rotated copy b={b} {rows}x{k} pad={pad} {mode} {rounding}")
    opt = dict(mode=mode, rounding=rounding, seed=5, offset=7)
    got = M.mixfp4_quantize(x, hadamard_block=b, hadamard_signs=sg, **opt)
    want = M.mixfp4_quantize(M.mixfp4_hadamard(x, b, sg), **opt)
    twice = M.mixfp4_quantize(x, tensor_scale=got[2], hadamard_block=b, hadamard_signs=sg, **opt)
    for g, w, t in zip(got, want, twice):
        assert torch.equal(g, w) and torch.equal(g, t)


def _butterflies_fp64(x, b):
    """Fast Walsh-Hadamard in fp64, stages in ascending order of the element bit."""
    v = x.astype(np.float64).reshape(-1, b).copy()
    for bit in range(b.bit_length() - 1):
        t = v.reshape(-1, b >> (bit + 1), 2, 1 << bit)
        v = np.stack([t[:, :, 0] + t[:, :, 1], t[:, :, 0] - t[:, :, 1]], 2).reshape(-1, b)
    return v.reshape(x.shape)


@pytest.mark.parametrize("b", [16, 64, 256])
def test_stage_order_beyond_the_exact_span(b):
    """Magnitudes 2^60 apart: large values that cancel in one stage and swallow
    small ones in another, so the fp64 sums depend on the order of the stages,
    which is that of the element bits.  b a power of 4: the scale is exact and
    the sums are rounded once to bf16."""
    import paper_2605_31035_amd as M
    x = np.zeros((b.bit_length() * (b.bit_length() - 1), b), np.float32)
    r = 0
    for i in range(b.bit_length() - 1):                # the bit in which the large values differ
        for j in range(b.bit_length() - 1):            # the bit of the small one
            if i != j:
                x[r, 0] = x[r, 1 << i] = 2.0 ** 60
                x[r, 1 << j] = 3.0
                r += 1
    log(f"stage order b={b}")
    y = M.mixfp4_hadamard(dev_bf16(W.f32_to_bf16_bits(x)), b)
    m, e = np.frexp(_butterflies_fp64(x, b) / np.sqrt(b))
    want = np.ldexp(np.rint(m * 256.0), e - 8)           # 8 significant bits, ties to even
    np.testing.assert_array_equal(host(y.float()).astype(np.float64), want)
