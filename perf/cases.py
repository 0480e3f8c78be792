"""Work that a user of this framework has it do, as cases that can be timed and
checked: MixFP4 quantization of activations, weights and gradients, the
quantized linear layer from one token to a large prefill, and its backward
pass, each through the package's public functions.

`listed()` are fixed cases, `draw(rng)` gives more of the same ranges,
`prepare(case, seed)` makes what a program holds before the call, `run(state)`
is one pass, `work(case)` the bytes and operations the pass cannot do without,
`tolerance(case)` how far a correct result may be off, and `exact(case, seed)`
the result in 64 bits from plain torch.
"""
import math

import torch

import paper_2605_31035_amd as M

MODES = ("mixfp4", "e2m1", "e1m2", "four_six")
BITS = 0.5625                                  # bytes of codes and scales per element
# weight shapes [n, k] of the repository's workloads and benchmark
LAYERS = ((4096, 4096), (11008, 4096), (4096, 11008), (14336, 4096), (8192, 8192), (28672, 8192))
LARGEST = 16384 * 8192 * 8192


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # a few tokens' activation, quantized on its own: the smallest call
        dict(name="token_quantize", kind="quantize", rows=3, k=4096, mode="mixfp4", given=False,
             sr=False, block=0),
        # the activation of an ordinary prefill, tensor scale computed on the device
        dict(name="act_quantize", kind="quantize", rows=1537, k=4096, mode="mixfp4", given=False,
             sr=False, block=0),
        # a large tensor with a calibrated (static) tensor scale
        dict(name="large_quantize", kind="quantize", rows=16384, k=16384, mode="mixfp4", given=True,
             sr=False, block=0),
        # fake quantization as accuracy studies run it: rotate, quantize, decode to fp32
        dict(name="rotated_roundtrip", kind="roundtrip", rows=4096, k=4096, mode="mixfp4", block=128),
        # a weight in 16 x 16 tiles for both passes of training
        dict(name="weight_2d", kind="weight2d", n=11008, k=4096),
        # one token through one layer in one launch
        dict(name="token_step", kind="step", m=1, n=11008, k=4096),
        # a full decode batch through a large layer: the weight is read once
        dict(name="decode_linear", kind="linear", m=16, n=28672, k=8192),
        # batched decoding of more sequences than one matrix tile holds
        dict(name="batch_linear", kind="linear", m=64, n=14336, k=4096),
        # a chunk of a chunked prefill, with an odd number of tokens
        dict(name="chunk_linear", kind="linear", m=509, n=11008, k=4096),
        # the prefill of a 7B-class layer
        dict(name="prefill_linear", kind="linear", m=2048, n=11008, k=4096),
        # a large prefill on decoded operands, quantization and both decodes included
        dict(name="large_linear", kind="two_pass", m=16384, n=8192, k=8192),
        # the backward pass of a 7B-class layer: DGRAD and WGRAD with stochastic
        # rounding and the random Hadamard rotation
        dict(name="backward", kind="backward", tokens=2048, n=11008, k=4096, block=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _layer(rng):
    """[n, k] of a layer: one of the repository's, or sizes between them."""
    if rng.random() < 0.5:
        return rng.choice(LAYERS)
    n = 16 * _log_int(rng, 64, 1792) if rng.random() < 0.75 else _log_int(rng, 1024, 28672)
    step = 16 if rng.random() < 0.125 else 64
    return n, step * _log_int(rng, 1024 // step, 14336 // step)


def draw(rng):
    kind = rng.choice(("quantize", "quantize", "roundtrip", "weight2d", "step", "linear", "linear",
                       "linear", "linear", "two_pass", "backward"))
    if kind in ("quantize", "roundtrip"):
        k = 16 * _log_int(rng, 64, 1024)
        block = 0
        if rng.random() < 0.3:
            block = rng.choice((16, 32, 64, 128, 256))
            k = max(block, k // block * block)
        rows = min(_log_int(rng, 1, 16384), (1 << 27) // k)
        mode = rng.choice(("mixfp4", "mixfp4", "mixfp4") + MODES[1:])
        if kind == "roundtrip":
            return dict(kind=kind, rows=rows, k=k, mode=mode, block=block)
        return dict(kind=kind, rows=rows, k=k, mode=mode, given=rng.random() < 0.3,
                    sr=rng.random() < 0.25, block=block)
    if kind == "weight2d":
        return dict(kind=kind, n=16 * _log_int(rng, 64, 896), k=16 * _log_int(rng, 64, 896))
    n, k = _layer(rng)
    if kind == "step":
        return dict(kind=kind, m=rng.randint(1, 16), n=n, k=(k + 63) // 64 * 64)
    if kind == "linear":
        return dict(kind=kind, m=min(_log_int(rng, 1, 8192), LARGEST // (n * k)), n=n, k=k)
    if kind == "two_pass":
        return dict(kind=kind, m=min(_log_int(rng, 512, 16384), LARGEST // (n * k)), n=n,
                    k=(k + 31) // 32 * 32)
    tokens = 64 * rng.randint(4, 64)
    return dict(kind=kind, tokens=tokens, n=(n + 63) // 64 * 64, k=(k + 63) // 64 * 64,
                block=rng.choice((16, 16, 32, 64)))


# --------------------------------------------------------------------------
# inputs: the distributions of the repository's workloads, made on the GPU
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _student(g, nu, rows, k):
    z = _normal(g, rows, k)
    chi = sum(_normal(g, rows, k).square_() for _ in range(nu))
    return z.mul_(chi.div_(nu).rsqrt_())


def _scaled_channels(g, x, count, factor):
    x[:, torch.randperm(x.shape[1], generator=g, device="cuda")[:count]] *= factor
    return x


def _activation(g, rows, k):
    """Heavy-tailed activations with a few outlier channels."""
    return _scaled_channels(g, _student(g, 4, rows, k), 8, 50.0).to(torch.bfloat16)


def _weight(g, n, k):
    return _normal(g, n, k).mul_(0.02).to(torch.bfloat16)


def _gradient(g, rows, n):
    return _scaled_channels(g, _student(g, 3, rows, n).mul_(1e-4), 16, 20.0).to(torch.bfloat16)


def _signs(g, block):
    return torch.randint(0, 2, (block,), generator=g, device="cuda", dtype=torch.int8) * 2 - 1


def _inputs(case, seed):
    """The tensors of one case, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind in ("quantize", "roundtrip"):
        t = dict(x=_activation(g, case["rows"], case["k"]))
        if case["block"]:
            t["signs"] = _signs(g, case["block"])
        if case.get("given"):
            # a calibrated scale: somewhat above what this tensor alone would give
            t["s32"] = (t["x"].abs().max().float() * 1.1 / 2688).reshape(1)
        return t
    if kind == "weight2d":
        return dict(w=_weight(g, case["n"], case["k"]))
    if kind == "backward":
        return dict(x=_activation(g, case["tokens"], case["k"]), w=_weight(g, case["n"], case["k"]),
                    dy=_gradient(g, case["tokens"], case["n"]), signs=_signs(g, case["block"]))
    return dict(x=_activation(g, case["m"], case["k"]), w=_weight(g, case["n"], case["k"]))


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"], st["seed"] = case, seed
    if case["kind"] in ("linear", "step", "two_pass"):
        st["w"] = M.mixfp4_quantize(st["w"])            # weights are quantized offline
    elif case["kind"] == "backward":
        st["wt"] = M.mixfp4_quantize_2d(st.pop("w"))[1]   # kept from the forward pass
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "quantize":
        return M.mixfp4_quantize(st["x"], st.get("s32"), mode=case["mode"],
                                 rounding="stochastic" if case["sr"] else "nearest",
                                 seed=st["seed"], hadamard_block=case["block"],
                                 hadamard_signs=st.get("signs"))
    if kind == "roundtrip":
        codes, scales, s32 = M.mixfp4_quantize(st["x"], mode=case["mode"], hadamard_block=case["block"],
                                               hadamard_signs=st.get("signs"))
        return codes, scales, s32, M.mixfp4_dequantize(codes, scales, s32)
    if kind == "weight2d":
        return M.mixfp4_quantize_2d(st["w"])
    if kind == "step":
        return M.mixfp4_decode_step(st["x"], st["w"])
    if kind == "linear":
        a = M.mixfp4_quantize(st["x"])
        return M.mixfp4_gemm(a, st["w"], workspace="auto"), a
    if kind == "two_pass":
        a, dec = M.mixfp4_quantize_decode(st["x"])
        return M.mixfp4_gemm_decoded(dec, M.mixfp4_decode_operand(st["w"])), a
    dy, signs, block = st["dy"], st["signs"], case["block"]
    qdy = M.mixfp4_quantize(dy, rounding="stochastic", seed=st["seed"])
    dx = M.mixfp4_gemm(qdy, st["wt"], workspace="auto")
    qdyt = M.mixfp4_quantize(dy, rounding="stochastic", seed=st["seed"], offset=1,
                             hadamard_block=block, hadamard_signs=signs, transpose=True)
    qxt = M.mixfp4_quantize(st["x"], hadamard_block=block, hadamard_signs=signs, transpose=True)
    return dx, M.mixfp4_gemm(qdyt, qxt, workspace="auto")


def work(case):
    kind = case["kind"]
    if kind == "quantize":
        return dict(bytes=case["rows"] * case["k"] * (2 + BITS), flops=0)
    if kind == "roundtrip":
        return dict(bytes=case["rows"] * case["k"] * (2 + BITS + 4), flops=0)
    if kind == "weight2d":
        return dict(bytes=case["n"] * case["k"] * (2 + 2 * BITS), flops=0)
    if kind == "backward":
        t, n, k = case["tokens"], case["n"], case["k"]
        return dict(bytes=2 * t * (n + k) + BITS * n * k + 4 * (t * k + n * k), flops=4 * t * n * k)
    m, n, k = case["m"], case["n"], case["k"]
    return dict(bytes=m * k * (2 + BITS) + BITS * n * k + 4 * m * n, flops=2 * m * n * k)


def tolerance(case):
    """Codes and scales are exact.  Products differ by the order of their fp32 sums (2.5e-8 to
    6e-8 from the 64-bit result; two orders are up to about 1e-7 apart)."""
    if case["kind"] in ("quantize", "roundtrip", "weight2d"):
        return "exact"
    return dict(rel=4e-7, max=5e-6)


# --------------------------------------------------------------------------
# the same in 64 bits, from Algorithm 1 and plain torch
# --------------------------------------------------------------------------
def _rne_grid(y, int4):
    """Round magnitudes to the E2M1 or INT4 grid, nearest, ties to the even code."""
    if int4:
        return torch.round(y).clamp_(max=7.0)
    step = torch.where(y < 2, 0.5, torch.where(y < 4, 1.0, 2.0))
    return (torch.round(y / step) * step).clamp_(max=6.0)


def _stochastic_grid(y, int4, u):
    """App. D on the local lattice: y + (eps - 1/2) d to the nearer neighbour, ties to the
    even code, eps = (u + 1/2) / 256."""
    step = torch.where(int4 | (y >= 2) & (y < 4), 1.0, torch.where(y < 2, 0.5, 2.0))
    lo = torch.floor(y / step)
    z = 512 * (y / step - lo) + 2 * u + 1
    up = (z > 512) | (z == 512) & (lo % 2 == 1)
    return torch.minimum((lo + up) * step, torch.where(int4, 7.0, 6.0).to(y))


def _philox_bytes(first, count, seed, offset):
    """The draws of blocks [first, first + count): Philox4x32-10, 16 bytes each."""
    mask = 0xFFFFFFFF
    g = torch.arange(first, first + count, device="cuda", dtype=torch.int64)
    c = [g & mask, g >> 32, torch.full_like(g, offset & mask), torch.full_like(g, offset >> 32)]
    k0, k1 = seed & mask, (seed >> 32) & mask

    def mul(a, b):
        hi = ((a >> 16) * b + (((a & 0xFFFF) * b) >> 16)) >> 16
        return hi & mask, (a * b) & mask
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    w = torch.stack(c, 1)
    return torch.stack([(w >> s) & 0xFF for s in (0, 8, 16, 24)], 2).reshape(count, 16).double()


def _branch(ax, bm, div, int4):
    s8 = (bm / div).float().clamp(max=448.0).to(torch.float8_e4m3fn).double()
    y = torch.where(s8 > 0, (ax / s8).float().double(), 0.0)
    return s8, y, s8 * _rne_grid(y, int4)


def _dequantized(x, s32, mode="mixfp4", draws=None, tile=1):
    """Algorithm 1 on a bf16 [rows, k] tensor and its decode, in fp64; blocks of 16 along k
    (of `tile` rows).  `draws`: (seed, offset) of stochastic rounding."""
    rows, k = x.shape
    out = torch.empty((rows, k), dtype=torch.float64, device=x.device)
    per = max(1, (1 << 24) // (k * tile)) * tile
    for r0 in range(0, rows, per):
        xb = x[r0:r0 + per].double()
        n = xb.shape[0]
        xb = (xb / s32.double()).float().double()
        xb = xb.reshape(n // tile, tile, k // 16, 16).transpose(1, 2).reshape(-1, tile * 16)
        ax = xb.abs()
        bm = ax.amax(1, keepdim=True).float().double()
        s1, y1, d1 = _branch(ax, bm, 6.0, False)
        s2, y2, d2 = _branch(ax, bm, 4.0 if mode == "four_six" else 7.0, mode != "four_six")
        delta = ((d2 - d1) * ((2 * ax - d1) - d2)).sum(1, keepdim=True)   # Err 1 - Err 2, exact
        second = delta > 0 if mode == "four_six" else delta >= 0
        if mode in ("e2m1", "e1m2"):
            second = torch.full_like(second, mode == "e1m2")
        if draws is None:
            d = torch.where(second, d2, d1)
        else:
            u = _philox_bytes(r0 * (k // 16), n * (k // 16), *draws)
            u = torch.where(torch.signbit(xb), 255 - u, u)
            int4 = (second & (mode != "four_six")).expand_as(ax)
            d = torch.where(second, s2, s1) * _stochastic_grid(torch.where(second, y2, y1), int4, u)
        d = torch.copysign(d, xb) * s32.double()
        out[r0:r0 + per] = d.reshape(n // tile, k // 16, tile, 16).transpose(1, 2).reshape(n, k)
    return out


def _scale(x):
    a = x.abs().max().double()
    return torch.where(a > 0, a / 2688, 1.0).float().reshape(1)


def _rotated(x, block, signs):
    """x diag(signs) H / sqrt(block) along k, rounded once to bf16 (through fp32 with round to odd)."""
    h = torch.ones((1, 1), dtype=torch.float64, device=x.device)
    while h.shape[0] < block:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    y = ((x.double().reshape(-1, block) * signs.double()) @ h / math.sqrt(block)).reshape(x.shape)
    f = y.float()
    low = torch.where(f.double().abs() > y.abs(), torch.nextafter(f, torch.zeros_like(f)), f)
    bits = torch.where(low.double() != y, low.view(torch.int32) | 1, low.view(torch.int32))
    return bits.view(torch.float32).to(torch.bfloat16)


def _product(a, w):
    return torch.cat([a @ w[j:j + 4096].T for j in range(0, w.shape[0], 4096)], 1)


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "weight2d":
        s = t["w"].abs().max().double() / 2688
        return (None, None, s.reshape(1)), (None, None, s.reshape(1))
    if kind in ("quantize", "roundtrip"):
        x = _rotated(t["x"], case["block"], t["signs"]) if case["block"] else t["x"]
        s64 = t["s32"].double() if case.get("given") else (x.abs().max().double() / 2688).reshape(1)
        if kind == "quantize":
            return None, None, s64
        return None, None, s64, _dequantized(x, _scale(x), case["mode"])
    if kind == "backward":
        x, dy, w, block, signs = t["x"], t["dy"], t["w"], case["block"], t["signs"]
        wd = _dequantized(w, _scale(w), tile=16)
        dx = _dequantized(dy, _scale(dy), draws=(seed, 0)) @ wd
        dyt, xt = (_rotated(v.T.contiguous(), block, signs) for v in (dy, x))
        dw = _product(_dequantized(dyt, _scale(dyt), draws=(seed, 1)), _dequantized(xt, _scale(xt)))
        return dx, dw
    c = _product(_dequantized(t["x"], _scale(t["x"])), _dequantized(t["w"], _scale(t["w"])))
    return c, (None, None, t["x"].abs().max().double().reshape(1) / 2688)
