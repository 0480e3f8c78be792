"""Sizes on both sides of the ranges in which the maximum pass loads X without
the non-temporal hint: the tensor scale is that of the whole X (its maximum is
the last element), and the codes are those of the call with that scale given."""
import pytest
import torch

from tests._gpu import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,mb", [(kind, mb) for kind, edges in (
    ("2d", (31, 32, 104, 105, 137, 138, 160, 161)), ("decode", (31, 32, 72, 73)),
    ("transpose", (31, 32, 112, 113)), ("variant", (31, 32, 124, 125)), ("1d", (32, 128)))
    for mb in edges])
def test_kept_ranges(kind, mb):
    import paper_2605_31035_amd as M
    g = torch.Generator(device="cuda")
    g.manual_seed(mb)
    x = torch.randn(mb * 128, 4096, generator=g, device="cuda", dtype=torch.bfloat16)
    x[-1, -1] = 31.0
    log(f"kept range {kind} {mb} MB")

    def call(s):
        if kind == "2d":
            a, t = M.mixfp4_quantize_2d(x, s)
            return (*a, *t[:2])
        if kind == "decode":
            out = torch.zeros((mb + 1) // 2 << 21, dtype=torch.uint8, device="cuda")   # padded rows
            return (*M.mixfp4_quantize_decode(x, s, out=out)[0], out)
        if kind == "variant":
            v = M.mixfp4_quantize_variant(x, tensor_scale=s)
            return v.codes, v.scales, v.s32
        return M.mixfp4_quantize(x, s, transpose=kind == "transpose")
    got = call(None)
    assert torch.equal(got[2], x.abs().max().float().reshape(1) / 2688)
    for a, b in zip(got, call(got[2])):
        assert torch.equal(a, b)
