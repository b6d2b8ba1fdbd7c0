"""The calls whose speed counts: what a user of the package runs, from the smallest layer to whole networks.

A case is a dict with a ``kind`` and sizes.  Kinds, each through the package's public entry points:

  pack     Sign + packing of a real matrix (how inputs and weights enter the packed domain)
  dense    one hidden layer on packed bits: product, BatchNorm, Sign in one call
  product  the +-1 matrix product with its int32 result
  norm     Sign(BatchNorm(.)) of int32 pre-activations (the second half of an unfused layer)
  pixels   the first layer on 8-bit inputs: bit planes, then the fused layer
  conv     one binary convolution layer (optionally with its 2 x 2 max pooling) on packed NHWC bits
  mlp      a whole fully connected network from real inputs to int32 scores
  convnet  the binary ConvNet body from packed feature maps to int32 scores

Inputs are drawn on the GPU from the seed alone: +-1 values with equal probability, N(0, 1) real inputs, uniform
bytes, and BatchNorm parameters of a trained network's spread (a tenth of the channels with a negative gamma).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1602_02830_amd as bnn

DEV = "cuda:0"
EPS = 1e-4
MLP_SIZES = (784, 4096, 4096, 4096, 10)
# Binary ConvNet body: (input channels, filters, height = width, pooled) per convolution, then the dense sizes.
CONVNET_CONVS = ((128, 128, 32, True), (128, 256, 16, False), (256, 256, 16, True), (256, 512, 8, False),
                 (512, 512, 8, True))
CONVNET_DENSE = (4 * 4 * 512, 1024, 1024, 10)

MAX_WORK = 8192 ** 3            # multiply-adds of the largest listed product
MAX_REALS = 32768 * 8192        # elements of the largest listed real matrix


def listed():
    return [
        # One dense layer at a small batch: interactive inference, bound by the call itself.
        {"name": "dense_64x1024x1024", "kind": "dense", "M": 64, "N": 1024, "K": 1024},
        # The hidden layer of the 3 x 4096 MLP over a whole 10 000-image test set.
        {"name": "dense_10000x4096x4096", "kind": "dense", "M": 10000, "N": 4096, "K": 4096},
        # A product whose sizes fit nothing: K one past a multiple of 32 words, rows packed without padding.
        {"name": "product_1000x1000x4097", "kind": "product", "M": 1000, "N": 1000, "K": 4097},
        # The large square binary product, int32 result.
        {"name": "product_8192x8192x8192", "kind": "product", "M": 8192, "N": 8192, "K": 8192},
        # BatchNorm + Sign as a pass of its own, for programs that keep the pre-activations.
        {"name": "norm_10000x4096", "kind": "norm", "M": 10000, "N": 4096},
        # Packing a gigabyte of reals.
        {"name": "pack_32768x8192", "kind": "pack", "M": 32768, "K": 8192},
        # First layer of the MLP on the images' bytes.
        {"name": "pixels_10000x4096x784", "kind": "pixels", "M": 10000, "N": 4096, "K": 784},
        # A layer in the middle of the ConvNet at its inference batch.
        {"name": "conv_256x16x16_256to256", "kind": "conv", "B": 256, "HW": 16, "Cin": 256, "Cout": 256, "stride": 1,
         "pool": 0},
        # A pooled layer on 28 x 28 feature maps: image rows that do not divide a power of two.
        {"name": "conv_128x28x28_128to256_pool", "kind": "conv", "B": 128, "HW": 28, "Cin": 128, "Cout": 256,
         "stride": 1, "pool": 2},
        # Whole networks: one training-size minibatch, the whole test set, the ConvNet body.
        {"name": "mlp_batch100", "kind": "mlp", "M": 100, "bytes_in": False},
        {"name": "mlp_batch10000", "kind": "mlp", "M": 10000, "bytes_in": False},
        {"name": "convnet_batch256", "kind": "convnet", "B": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, step):
    """A size in [lo, hi], spread over its logarithm; half of the time a multiple of `step`."""
    v = _log_int(rng, lo, hi)
    return max(step, v // step * step) if rng.random() < 0.5 else v


def draw(rng):
    while True:
        kind = rng.choice(["pack", "dense", "dense", "product", "product", "norm", "pixels", "conv", "conv", "mlp",
                           "convnet"])
        if kind == "pack":
            case = {"kind": kind, "M": _log_int(rng, 64, 32768), "K": _size(rng, 512, 8192, 128)}
        elif kind in ("dense", "product"):
            case = {"kind": kind, "M": _size(rng, 64, 16384, 64), "N": _size(rng, 256, 8192, 128),
                    "K": _size(rng, 512, 8192, 512)}
        elif kind == "norm":
            case = {"kind": kind, "M": _log_int(rng, 256, 20000), "N": _size(rng, 256, 8192, 128)}
        elif kind == "pixels":
            case = {"kind": kind, "M": _log_int(rng, 100, 10000), "N": _size(rng, 512, 4096, 128),
                    "K": rng.choice([784, 1024, 3072, rng.randint(300, 3072)])}
        elif kind == "conv":
            stride = rng.choice([1, 1, 1, 2])
            hw = rng.choice([8, 16, 32, rng.randint(7, 32), rng.randint(7, 56)])
            pool = 2 if stride == 1 and hw % 2 == 0 and rng.random() < 0.4 else 0
            case = {"kind": kind, "B": _log_int(rng, 8, 256), "HW": hw, "Cin": rng.choice([64, 128, 128, 256, 256, 512]),
                    "Cout": rng.choice([64, 128, 256, 512, 33 * rng.randint(2, 12)]), "stride": stride, "pool": pool}
        elif kind == "mlp":
            case = {"kind": kind, "M": _log_int(rng, 64, 10000), "bytes_in": rng.random() < 0.4}
        else:
            case = {"kind": kind, "B": _log_int(rng, 16, 256)}
        reals = case["M"] * case["K"] if kind == "pack" else case["M"] * case["N"] if kind == "norm" else 0
        # the first layer on bytes weighs eight planes
        weight = 8 if kind == "pixels" else 1
        if reals <= MAX_REALS and weight * work(case)["flops"] <= 2 * MAX_WORK:
            return case


# ---- inputs ------------------------------------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + salt)


def _pm1(g, *shape):
    """+-1 as float32."""
    return torch.randint(0, 2, shape, generator=g, device=DEV).mul_(2).sub_(1).float()


def _bn(seed, salt, N, K):
    """(gamma, beta, mean, var), float32 [N], for pre-activations of fan-in K."""
    r = np.random.default_rng([int(seed), salt])
    gamma = 1.0 + 0.1 * r.standard_normal(N)
    gamma = np.where(r.random(N) < 0.1, -gamma, gamma)
    beta = 0.1 * r.standard_normal(N)
    mean = 0.25 * math.sqrt(K) * r.standard_normal(N)
    var = K * r.uniform(0.5, 1.5, N)
    return tuple(a.astype(np.float32) for a in (gamma, beta, mean, var))


def _byte_bn(bn):
    """BatchNorm of a first layer on bytes: the sums are wider by the bytes' root mean square (about 147.5)."""
    gamma, beta, mean, var = bn
    return gamma, beta, (147.5 * mean).astype(np.float32), (147.5 ** 2 * var).astype(np.float32)


def _draws(case, seed):
    """The plain values behind a case: what prepare() packs and exact() computes with."""
    kind = case["kind"]
    g = _gen(seed, 1)
    if kind == "pack":
        return {"x": torch.randn(case["M"], case["K"], generator=g, device=DEV)}
    if kind in ("dense", "product"):
        d = {"a": _pm1(g, case["M"], case["K"]), "w": _pm1(g, case["N"], case["K"])}
        if kind == "dense":
            d["bn"] = _bn(seed, 2, case["N"], case["K"])
        return d
    if kind == "norm":
        # sums of 4096 +-1 products: even numbers of standard deviation 64
        s = torch.randn(case["M"], case["N"], generator=g, device=DEV).mul_(32).round_().mul_(2).to(torch.int32)
        return {"s": s, "bn": _bn(seed, 2, case["N"], 4096)}
    if kind == "pixels":
        x = torch.randint(0, 256, (case["M"], case["K"]), generator=g, device=DEV, dtype=torch.uint8)
        return {"x": x, "w": _pm1(g, case["N"], case["K"]), "bn": _byte_bn(_bn(seed, 2, case["N"], case["K"]))}
    if kind == "conv":
        x = _pm1(g, case["B"], case["HW"], case["HW"], case["Cin"])
        w = _pm1(g, case["Cout"], 3, 3, case["Cin"])
        return {"x": x, "w": w, "bn": _bn(seed, 2, case["Cout"], 9 * case["Cin"])}
    if kind == "mlp":
        layers = list(zip(MLP_SIZES[:-1], MLP_SIZES[1:]))
        bns = [_bn(seed, 10 + l, n, k) for l, (k, n) in enumerate(layers[:-1])]
        if case["bytes_in"]:
            x = torch.randint(0, 256, (case["M"], MLP_SIZES[0]), generator=g, device=DEV, dtype=torch.uint8)
            bns[0] = _byte_bn(bns[0])
        else:
            x = torch.randn(case["M"], MLP_SIZES[0], generator=g, device=DEV)
        return {"x": x, "ws": [_pm1(g, n, k) for k, n in layers], "bns": bns}
    x = _pm1(g, case["B"], 32, 32, CONVNET_CONVS[0][0])
    convs = [(_pm1(g, cout, 3, 3, cin), _bn(seed, 10 + l, cout, 9 * cin), pooled)
             for l, (cin, cout, _hw, pooled) in enumerate(CONVNET_CONVS)]
    layers = list(zip(CONVNET_DENSE[:-1], CONVNET_DENSE[1:]))
    return {"x": x, "convs": convs, "ws": [_pm1(g, n, k) for k, n in layers],
            "bns": [_bn(seed, 30 + l, n, k) for l, (k, n) in enumerate(layers[:-1])]}


# ---- the path ----------------------------------------------------------------------------------------------

def _words(n):
    return (n + 31) // 32


def _folded(bn, K):
    thr, flip = bnn.bn_fold(*bn, EPS, K)
    return torch.from_numpy(thr).to(DEV), torch.from_numpy(flip.view(np.int32)).to(DEV)


def _packed_maps(x):
    """+-1 NHWC -> packed NHWC words."""
    b, h, w, c = x.shape
    return bnn.pack_sign(x.reshape(-1, c)).view(b, h, w, _words(c))


def prepare(case, seed):
    kind = case["kind"]
    d = _draws(case, seed)
    st = {"kind": kind}
    if kind == "pack":
        st["x"] = d["x"]
        st["out"] = torch.empty(case["M"], _words(case["K"]), dtype=torch.int32, device=DEV)
    elif kind in ("dense", "product"):
        st["K"] = case["K"]
        st["a"], st["w"] = bnn.pack_sign(d["a"]), bnn.pack_sign(d["w"])
        if kind == "dense":
            st["thr"], st["flip"] = _folded(d["bn"], case["K"])
            st["out"] = torch.empty(case["M"], _words(case["N"]), dtype=torch.int32, device=DEV)
        else:
            st["out"] = torch.empty(case["M"], case["N"], dtype=torch.int32, device=DEV)
    elif kind == "norm":
        st["s"] = d["s"]
        st["thr"], st["flip"] = _folded(d["bn"], 4096)
        st["out"] = torch.empty(case["M"], _words(case["N"]), dtype=torch.int32, device=DEV)
    elif kind == "pixels":
        st["K"], st["x"], st["w"] = case["K"], d["x"], bnn.pack_sign(d["w"])
        st["thr"], st["flip"] = _folded(d["bn"], 255 * case["K"])
        st["planes"] = torch.empty(case["M"], 8 * _words(case["K"]), dtype=torch.int32, device=DEV)
        st["out"] = torch.empty(case["M"], _words(case["N"]), dtype=torch.int32, device=DEV)
    elif kind == "conv":
        st["x"] = _packed_maps(d["x"])
        st["net"] = bnn.BinaryConvLayer(d["w"], d["bn"], EPS, case["B"], case["HW"], case["HW"],
                                        stride=case["stride"], pad=1, fused=True, implicit=True, pool=case["pool"])
    elif kind == "mlp":
        st["x"] = d["x"]
        st["net"] = bnn.BinaryMLP(d["ws"], d["bns"], EPS, case["M"], fused=True, input_uint8=case["bytes_in"])
    else:
        st["x"] = _packed_maps(d["x"])
        st["net"] = bnn.BinaryConvNet(d["convs"], d["ws"], d["bns"], EPS, case["B"], 32, 32)
    return st


def run(st):
    kind = st["kind"]
    if kind == "pack":
        return bnn.pack_sign(st["x"], out=st["out"])
    if kind == "dense":
        return bnn.xnor_gemm_bn_sign_pack(st["a"], st["w"], st["K"], st["thr"], st["flip"], out=st["out"])
    if kind == "product":
        return bnn.xnor_gemm(st["a"], st["w"], st["K"], out=st["out"])
    if kind == "norm":
        return bnn.bn_sign_pack(st["s"], st["thr"], st["flip"], out=st["out"])
    if kind == "pixels":
        planes = bnn.pack_bitplanes(st["x"], out=st["planes"])
        return bnn.bitplane_gemm_bn_sign_pack(planes, st["w"], st["K"], st["thr"], st["flip"], out=st["out"])
    return st["net"].forward(st["x"])


# ---- what the path cannot do without -----------------------------------------------------------------------

def _layer_work(M, N, K, bits_in, bits_out):
    """One product with weights of one bit: bytes in, weights and thresholds, bytes out."""
    out = 4 * M * _words(N) + 4 * N if bits_out == 1 else 4 * M * N
    return {"bytes": M * K * bits_in // 8 + N * K // 8 + out, "flops": 2 * M * N * K}


def work(case):
    kind = case["kind"]
    if kind == "pack":
        return {"bytes": 4 * case["M"] * case["K"] + 4 * case["M"] * _words(case["K"]), "flops": 0}
    if kind == "norm":
        return {"bytes": 4 * case["M"] * case["N"] + 4 * case["M"] * _words(case["N"]) + 4 * case["N"], "flops": 0}
    if kind in ("dense", "product"):
        return _layer_work(case["M"], case["N"], case["K"], 1, 1 if kind == "dense" else 32)
    if kind == "pixels":
        return _layer_work(case["M"], case["N"], case["K"], 8, 1)
    if kind == "conv":
        return _conv_work(case["B"], case["HW"], case["Cin"], case["Cout"], case["stride"], case["pool"])
    if kind == "mlp":
        M, b, f = case["M"], 4 * case["M"] * MLP_SIZES[-1], 0
        b += M * MLP_SIZES[0] * (1 if case["bytes_in"] else 4)
        for k, n in zip(MLP_SIZES[:-1], MLP_SIZES[1:]):
            b += n * k // 8
            f += 2 * M * n * k
        return {"bytes": b, "flops": f}
    B, b, f = case["B"], case["B"] * (32 * 32 * 128 // 8 + 4 * CONVNET_DENSE[-1]), 0
    for cin, cout, hw, _pooled in CONVNET_CONVS:
        b += 9 * cin * cout // 8
        f += 2 * B * hw * hw * cout * 9 * cin
    for k, n in zip(CONVNET_DENSE[:-1], CONVNET_DENSE[1:]):
        b += n * k // 8
        f += 2 * B * n * k
    return {"bytes": b, "flops": f}


def _conv_work(B, hw, cin, cout, stride, pool):
    ho = (hw - 1) // stride + 1
    po = ho // 2 if pool else ho
    b = 4 * B * hw * hw * _words(cin) + 9 * cin * cout // 8 + 4 * B * po * po * _words(cout) + 4 * cout
    return {"bytes": b, "flops": 2 * B * ho * ho * cout * 9 * cin}


def tolerance(case):
    return "exact"              # every output is a whole number or packed bits


# ---- the same results in plain 64-bit torch ----------------------------------------------------------------

_SHIFTS = None


def _pack_plain(bits):
    """Booleans [rows][n] -> int32 words, element k at bit k % 32 of word k / 32."""
    global _SHIFTS
    if _SHIFTS is None:
        _SHIFTS = torch.arange(32, device=DEV, dtype=torch.int64)
    rows, n = bits.shape
    out = torch.empty(rows, _words(n), dtype=torch.int32, device=DEV)
    step = max(1, (1 << 24) // max(1, n))
    for r in range(0, rows, step):
        part = bits[r:r + step]
        full = torch.zeros(part.shape[0], 32 * _words(n), dtype=torch.int64, device=DEV)
        full[:, :n] = part
        words = (full.view(part.shape[0], -1, 32) << _SHIFTS).sum(-1)
        out[r:r + step] = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
    return out


def _sign_bn(s, bn):
    """Sign(BatchNorm(s)) as booleans, s float64 [rows][N]."""
    gamma, beta, mean, var = (torch.from_numpy(a).to(DEV).double() for a in bn)
    return gamma * ((s - mean) / torch.sqrt(var + EPS)) + beta >= 0


def _pm(bits):
    return bits.double().mul_(2).sub_(1)


def _conv_plain(x, w, stride):
    """x float64 NHWC, padded with +1 on every side; w [Cout][3][3][Cin]."""
    b, h, ww, c = x.shape
    p = torch.ones(b, h + 2, ww + 2, c, dtype=torch.float64, device=DEV)
    p[:, 1:-1, 1:-1] = x
    ho, wo = (h - 1) // stride + 1, (ww - 1) // stride + 1
    s = torch.zeros(b * ho * wo, w.shape[0], dtype=torch.float64, device=DEV)
    for ky in range(3):
        for kx in range(3):
            tap = p[:, ky:ky + stride * (ho - 1) + 1:stride, kx:kx + stride * (wo - 1) + 1:stride].reshape(-1, c)
            s += tap @ w[:, ky, kx].double().t()
    return s.view(b, ho, wo, -1)


def _pool_plain(s):
    b, h, w, c = s.shape
    return s.view(b, h // 2, 2, w // 2, 2, c).amax(dim=(2, 4))


def exact(case, seed):
    kind = case["kind"]
    d = _draws(case, seed)
    if kind == "pack":
        return _pack_plain(d["x"] >= 0)
    if kind == "norm":
        return _pack_plain(_sign_bn(d["s"].double(), d["bn"]))
    if kind in ("dense", "product"):
        s = d["a"].double() @ d["w"].double().t()
        return _pack_plain(_sign_bn(s, d["bn"])) if kind == "dense" else s.to(torch.int32)
    if kind == "pixels":
        return _pack_plain(_sign_bn(d["x"].double() @ d["w"].double().t(), d["bn"]))
    if kind == "conv":
        s = _conv_plain(d["x"].double(), d["w"], case["stride"])
        s = _pool_plain(s) if case["pool"] else s
        b, h, w, c = s.shape
        return _pack_plain(_sign_bn(s.reshape(-1, c), d["bn"])).view(b, h, w, -1)
    if kind == "mlp":
        a = d["x"].double() if case["bytes_in"] else _pm(d["x"] >= 0)
        for w, bn in zip(d["ws"][:-1], d["bns"]):
            a = _pm(_sign_bn(a @ w.double().t(), bn))
        return (a @ d["ws"][-1].double().t()).to(torch.int32)
    a = d["x"].double()
    for w, bn, pooled in d["convs"]:
        s = _conv_plain(a, w, 1)
        s = _pool_plain(s) if pooled else s
        a = _pm(_sign_bn(s.reshape(-1, s.shape[-1]), bn)).view(s.shape)
    a = a.reshape(a.shape[0], -1)
    for w, bn in zip(d["ws"][:-1], d["bns"]):
        a = _pm(_sign_bn(a @ w.double().t(), bn))
    return (a @ d["ws"][-1].double().t()).to(torch.int32)
