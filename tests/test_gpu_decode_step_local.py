"""The one-launch decode step where every workgroup quantizes A itself: up to
four blocks of A per thread (256 threads: 1024 blocks; 128 where K splits over
two waves; 512 on two sets of waves), one more block than that, K tails, an
all-zero A and tensor scales outside the direct division range."""
import pytest
import torch

import workloads as W
from tests._gpu import dev_bf16, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [
    (1, 17, 64), (1, 4096, 192), (4, 300, 4096), (5, 300, 4096), (16, 100, 1024), (16, 100, 1088),
    (5, 40, 1536), (6, 40, 1536), (3, 11008, 4160), (16, 28672, 2048), (9, 28672, 4096)])
@pytest.mark.parametrize("scale", [1.0, 0.0, 2.0 ** -120, 2.0 ** 118])
def test_local_step(m, n, k, scale):
    import paper_2605_31035_amd as M
    log(f"local step m={m} n={n} k={k} scale={scale}")
    x = dev_bf16(W.adversarial(m + k, m, k))
    x = x if scale == 1.0 else (x.float() / 30000 * scale).bfloat16()
    w = M.mixfp4_quantize(dev_bf16(W.adversarial(n, n, k)))
    sync = torch.zeros(4, dtype=torch.int32, device="cuda")
    c, a = M.mixfp4_decode_step(x, w, sync=sync)
    q = M.mixfp4_quantize(x)
    for got, ref in zip(a, q):
        assert torch.equal(got, ref)
    assert torch.equal(c, M.mixfp4_gemm(q, w))
    assert int(sync.abs().sum()) == 0
