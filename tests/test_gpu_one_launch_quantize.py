"""The one-launch quantizer (tensor scale and codes of at most 2^17 elements in
one kernel) on both sides of every size at which its workgroup changes: 256
threads with 1, 4 or 8 blocks in flight, 512 threads, where two workgroups
share a turn's blocks, 1024 threads, where four do, and the two-pass call
beyond.  Every format and both roundings, contiguous and strided rows, bit for
bit against the oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import quant as Q
from tests._gpu import dev_bf16, host, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("blocks", [1, 255, 256, 257, 1024, 1025, 2048, 2049, 3000, 4096, 4097,
                                    6100, 8192, 8193])
def test_one_launch_sizes(blocks, pad):
    import paper_2605_31035_amd as M
    k = 16 * next(d for d in (4, 3, 1) if blocks % d == 0)
    rows = blocks * 16 // k
    bits = W.adversarial(blocks, rows, k)
    # the maximum in the last block, which only the last turn reads
    bits[-1, -1] = W.f32_to_bf16_bits(np.abs(W.bf16_bits_to_f32(bits)).max(keepdims=True)[0] * 2)[0]
    x = torch.zeros((rows, k + pad), dtype=torch.bfloat16, device="cuda")
    x[:, :k] = dev_bf16(bits)
    x = x[:, :k]
    log(f"one launch: {blocks} blocks, pad {pad}")
    for mode, omode in (("mixfp4", "select"), ("e2m1", "e2m1"), ("e1m2", "e1m2"),
                        ("four_six", "four_six")):
        for rounding in ("nearest", "stochastic"):
            opt = dict(rounding=rounding, seed=(1 << 40) + 3, offset=(5 << 33) + 1)
            codes, scales, s32 = M.mixfp4_quantize(x, mode=mode, **opt)
            ref = Q.quantize(bits, mode=omode, **opt)
            assert host(s32)[0] == ref.s32, (mode, rounding)
            np.testing.assert_array_equal(host(scales), ref.scales, err_msg=f"{mode} {rounding}")
            np.testing.assert_array_equal(host(codes), ref.codes, err_msg=f"{mode} {rounding}")
