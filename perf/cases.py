"""Performance cases: the layers that programs call through the public entry points, over the sizes they use.

A case names one entry point (`call`) and its sizes; `listed()` gives fixed cases, `draw()` more of the same ranges.
Inputs are synthetic (x ~ N(0, 1), W ~ N(0, 1 / C_in) per real component), drawn on the GPU from the seed alone.
"""
import math

import torch

from paper_2504_11681_amd import binding

# call       entry point                                       x, y        W
# auto1d     spectral_conv1d_auto: per-shape dispatch          c64         [C_in, C_out], any length up to 4096
# real1d     spectral_conv1d_real                              float32     [C_in, C_out]
# fno1d      fno1d_real                                        float32     [C_in, C_out, K1]
# rect2d     spectral_conv2d_rect                              c64         [C_in, C_out]
# permode2d  spectral_conv2d_permode                           c64         [C_in, C_out, K1, K2]
# fno2d      fno2d_real                                        float32     [C_in, C_out, 2 K1, K2]
# grid2d     spectral_conv2d_rect_staged: grids whose sides    c64         [C_in, C_out]
#            are not powers of two
REAL_CALLS = ("real1d", "fno1d", "fno2d")


def case(call, B, C_in, C_out, N1, N2, K1, K2, name=None):
    c = {"call": call, "B": B, "C_in": C_in, "C_out": C_out, "N1": N1, "N2": N2, "K1": K1, "K2": K2}
    return c if name is None else dict(c, name=name)


def line(call, B, C_in, C_out, N, K, name=None):
    return case(call, B, C_in, C_out, 1, N, 1, K, name)


def listed():
    return [
        # one small layer of a model stepped a few samples at a time: launch and latency only
        line("auto1d", 4, 16, 16, 64, 16, "1d_b4_c16_n64"),
        # a training-size batch of a small 1-D model: still under one workgroup per CU
        line("auto1d", 64, 64, 64, 256, 64, "1d_b64_c64_n256"),
        # the production 1-D layer that the headline figure is quoted on
        line("auto1d", 256, 128, 128, 1024, 128, "1d_b256_c128_n1024"),
        # the widest cell of the hidden-dimension sweep, half of the spectrum kept: most arithmetic per byte
        line("auto1d", 512, 256, 256, 256, 128, "1d_b512_c256_n256_k128"),
        # long pencils: one eighth of the spectrum of 4096-point signals
        line("auto1d", 64, 128, 128, 4096, 512, "1d_b64_c128_n4096"),
        # a sampled signal whose length is no power of two, ragged channel and mode counts
        line("auto1d", 64, 40, 56, 1000, 50, "1d_b64_c40_56_n1000"),
        # real-valued fields, shared weights
        line("real1d", 256, 128, 128, 1024, 128, "real1d_b256_c128_n1024"),
        # the Fourier layer of a 1-D FNO: real field, few modes, own weights per mode, small batch
        line("fno1d", 32, 64, 64, 1024, 16, "fno1d_b32_c64_n1024_m16"),
        # the production 2-D layer (the largest case)
        case("rect2d", 32, 64, 64, 256, 256, 64, 64, "2d_b32_c64_n256"),
        # high-resolution images, few samples
        case("rect2d", 4, 32, 32, 512, 512, 64, 64, "2d_b4_c32_n512"),
        # the Fourier layer of a 2-D FNO on 64 x 64 real fields, both low-frequency blocks, 12 modes per axis
        case("fno2d", 256, 64, 64, 64, 64, 12, 12, "fno2d_b256_c64_n64_m12"),
        # a simulation grid whose sides are odd (85 x 85 points, 12 modes per axis)
        case("grid2d", 32, 32, 32, 85, 85, 12, 12, "grid2d_b32_c32_n85"),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def odd_length(rng, lo, hi):
    while True:
        n = log_int(rng, lo, hi)
        if n & (n - 1):
            return n


MOST_BYTES = 1 << 30        # of one drawn case: half of the largest listed one
MOST_DIRECT = 1.2e10        # multiply-adds that direct sums over odd lengths may take (about the listed 85 x 85 grid's)


def direct_sums(c):
    n = 0.0
    for N, pencils in ((c["N2"], c["N1"]), (c["N1"], c["N2"])):
        if N & (N - 1):
            n += c["B"] * (c["C_in"] + c["C_out"]) * float(pencils) * N * N
    return n


def draw(rng):
    call = rng.choice(("auto1d", "auto1d", "long", "odd", "real1d", "fno1d", "rect2d", "rect2d", "permode2d", "fno2d", "grid2d"))
    if call in ("auto1d", "real1d"):
        N = rng.choice((64, 128, 256, 512, 1024))
        c = line(call, log_int(rng, 4, 512), log_int(rng, 8, 256), log_int(rng, 8, 256), N,
                 log_int(rng, max(8, N // 16), min(256, N // 2)))
    elif call == "long":
        N = rng.choice((2048, 4096))
        c = line("auto1d", log_int(rng, 4, 64), log_int(rng, 16, 128), log_int(rng, 16, 128), N, log_int(rng, N // 16, N // 4))
    elif call == "odd":
        N = odd_length(rng, 48, 2000)
        c = line("auto1d", log_int(rng, 4, 64), log_int(rng, 8, 128), log_int(rng, 8, 128), N, log_int(rng, 8, max(9, min(128, N // 4))))
    elif call == "fno1d":
        N = rng.choice((64, 128, 256, 1024))
        c = line(call, log_int(rng, 4, 256), log_int(rng, 8, 128), log_int(rng, 8, 128), N, log_int(rng, 8, min(128, N // 2)))
    elif call == "grid2d":
        N1, N2 = odd_length(rng, 40, 480), odd_length(rng, 40, 480)
        c = case(call, log_int(rng, 2, 32), log_int(rng, 4, 64), log_int(rng, 4, 64), N1, N2,
                 log_int(rng, 8, min(32, N1 // 4)), log_int(rng, 8, min(32, N2 // 4)))
    else:
        sides = (64, 128, 256, 512) if call == "rect2d" else (64, 128, 256)
        N1, N2 = rng.choice(sides), rng.choice(sides)
        c = case(call, log_int(rng, 2, 64), log_int(rng, 4, 64), log_int(rng, 4, 64), N1, N2,
                 log_int(rng, 4, min(32, N1 // 4)), log_int(rng, 8, min(64, N2 // 2)))
    while c["B"] > 1 and (work(c)["bytes"] > MOST_BYTES or direct_sums(c) > MOST_DIRECT):
        c["B"] = (c["B"] + 1) // 2
    return c


def modes(c):
    """Retained modes of the truncated spectrum (fno2d keeps both low-frequency blocks of the first axis)."""
    return (2 * c["K1"] if c["call"] == "fno2d" else c["K1"]) * c["K2"]


def weight_shape(c):
    k = {"fno1d": (c["K2"],), "permode2d": (c["K1"], c["K2"]), "fno2d": (2 * c["K1"], c["K2"])}.get(c["call"], ())
    return (c["C_in"], c["C_out"]) + k


def field_shape(c, C):
    return (c["B"], C, c["N2"]) if c["N1"] == 1 else (c["B"], C, c["N1"], c["N2"])


def inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = torch.float32 if c["call"] in REAL_CALLS else torch.complex64
    x = torch.empty(field_shape(c, c["C_in"]), dtype=dtype, device="cuda")
    (x if dtype == torch.float32 else torch.view_as_real(x)).normal_(0.0, 1.0, generator=g)
    W = torch.empty(weight_shape(c), dtype=torch.complex64, device="cuda")
    torch.view_as_real(W).normal_(0.0, 1.0 / math.sqrt(c["C_in"]), generator=g)
    return x, W


def prepare(c, seed):
    x, W = inputs(c, seed)
    y = torch.empty(field_shape(c, c["C_out"]), dtype=x.dtype, device="cuda")
    return {"call": c["call"], "K1": c["K1"], "K2": c["K2"], "x": x, "W": W, "y": y}


def run(s):
    call, x, W, y = s["call"], s["x"], s["W"], s["y"]
    if call == "auto1d":
        return binding.spectral_conv1d_auto(x, W, y, s["K2"])
    if call == "real1d":
        return binding.spectral_conv1d_real(x, W, y, s["K2"])
    if call == "fno1d":
        return binding.fno1d_real(x, W, y)
    if call == "rect2d":
        return binding.spectral_conv2d_rect(x, W, y, s["K1"], s["K2"])
    if call == "permode2d":
        return binding.spectral_conv2d_permode(x, W, y)
    if call == "fno2d":
        return binding.fno2d_real(x, W, y)
    return binding.spectral_conv2d_rect_staged(x, W, y, s["K1"], s["K2"])


def work(c):
    """x and W read once, y written once; the contraction over the channels and transforms pruned to the kept modes."""
    real = c["call"] in REAL_CALLS
    pts, m, both = c["N1"] * c["N2"], modes(c), c["C_in"] + c["C_out"]
    weights = 8 * c["C_in"] * c["C_out"] * (m if len(weight_shape(c)) > 2 else 1)
    per_line = 5.0 * c["N2"] * math.log2(max(2, c["K2"]))
    per_field = c["N1"] * per_line + (c["K2"] * 5.0 * c["N1"] * math.log2(max(2, m // c["K2"])) if c["N1"] > 1 else 0.0)
    return {"bytes": (4 if real else 8) * c["B"] * pts * both + weights,
            "flops": 8.0 * c["B"] * m * c["C_in"] * c["C_out"] + c["B"] * both * per_field * (0.5 if real else 1.0)}


def tolerance(c):
    """Four times the distance from the float64 result that was measured: at most 4e-7 with 32-bit sums of transforms by
    butterflies, and growing with the length where a transform is one long 32-bit sum (8.4e-7 at 1000 points)."""
    side = max([N for N in (c["N1"], c["N2"]) if N & (N - 1)], default=0)
    rel = 1.6e-6 * max(1.0, side / 400.0)
    return {"rel": rel, "max": 12 * rel}


def waves(N, freqs, sign):
    """[N, len(freqs)] complex128: exp(sign 2 pi i n k / N), the phase reduced with whole numbers."""
    n = torch.arange(N, device="cuda", dtype=torch.int64)
    k = torch.tensor(freqs, device="cuda", dtype=torch.int64)
    phase = ((n[:, None] * k[None, :]) % N).to(torch.float64) * (sign * 2.0 * math.pi / N)
    return torch.polar(torch.ones_like(phase), phase)


def exact(c, seed):
    """The definition in float64: the kept bins as sums, the contraction, the inverse from the kept bins."""
    x, W = inputs(c, seed)
    x, W = x.to(torch.complex128), W.to(torch.complex128)
    B, Ci, Co, N1, N2, K2 = c["B"], c["C_in"], c["C_out"], c["N1"], c["N2"], c["K2"]
    real = c["call"] in REAL_CALLS
    f1 = list(range(-c["K1"], c["K1"])) if c["call"] == "fno2d" else list(range(c["K1"]))
    X = x.reshape(-1, N2) @ waves(N2, range(K2), -1)                                        # [B Ci N1, K2]
    X = X.reshape(B * Ci, N1, K2).transpose(1, 2).reshape(-1, N1) @ waves(N1, f1, -1)       # [B Ci K2, f1]
    X = X.reshape(B, Ci, K2, len(f1)).permute(0, 3, 2, 1).contiguous()                      # [B, f1, K2, Ci]
    if W.dim() == 2:
        Y = X.reshape(-1, Ci) @ W
    else:
        M = len(f1) * K2
        Wm = W.reshape(Ci, Co, M).permute(2, 0, 1).contiguous()                             # [M, Ci, Co]
        Xm = X.reshape(B, M, Ci).transpose(0, 1).contiguous()                               # [M, B, Ci]
        Y = torch.matmul(Xm, Wm).transpose(0, 1).contiguous()
    Y = Y.reshape(B, len(f1), K2, Co).permute(0, 3, 2, 1).contiguous()                      # [B, Co, K2, f1]
    if real:
        Y[:, :, 0] *= 0.5
    y = Y.reshape(-1, len(f1)) @ waves(N1, f1, +1).T.contiguous()                           # [B Co K2, N1]
    y = y.reshape(B * Co, K2, N1).transpose(1, 2).reshape(-1, K2) @ waves(N2, range(K2), +1).T.contiguous()
    y = (2.0 * y.real if real else y) / float(N1 * N2)
    return y.reshape(field_shape(c, Co)).contiguous()
