"""Stochastic rounding where a draw lands exactly between two codes: block
scales of 1 (block maximum 6 or 7, tensor scale 1) and elements that are odd
multiples of 1/512 of the lattice step, so that w == 511 - 2u for one draw in
256; codes bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import quant as Q
from tests._gpu import dev_bf16, dev_f32, host, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,omode,top", [("e2m1", "e2m1", 6.0), ("e1m2", "e1m2", 7.0),
                                            ("mixfp4", "select", 6.0), ("mixfp4", "select", 7.0),
                                            ("four_six", "four_six", 6.0)])
@pytest.mark.parametrize("transpose", [False, True])
def test_ties(mode, omode, top, transpose):
    import paper_2605_31035_amd as M
    rng = np.random.default_rng(int(top) + len(mode))
    rows, k = 256, 1024
    x = (2 * rng.integers(0, 128, (rows, k)) + 1) / (1024.0 if top == 6.0 else 512.0)
    x = x.astype(np.float32) * rng.choice([-1.0, 1.0], (rows, k)).astype(np.float32)
    x.reshape(rows, -1, 16)[:, :, 3] = top
    bits = W.f32_to_bf16_bits(x)
    log(f"stochastic ties {mode} top={top} transpose={transpose}")
    ref = Q.quantize(bits, s32=1.0, mode=omode, rounding="stochastic", seed=77, offset=5)
    xd = dev_bf16(bits)
    codes, scales, _ = M.mixfp4_quantize(xd.t().contiguous() if transpose else xd, dev_f32(1.0),
                                         mode=mode, rounding="stochastic", seed=77, offset=5,
                                         transpose=transpose)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(scales), ref.scales)
    np.testing.assert_array_equal(host(codes), ref.codes)
