"""The calls a program makes through this library, at the sizes and options it makes them with, for measuring.

Each listed case stands for one kind of work; `draw` gives more calls of the same kinds over their whole ranges.
All outputs are integers, or fp32 values of a fixed sequence of correctly rounded operations, so every correct
implementation gives the same bytes.
"""
import math

import torch

from paper_2101_05615_amd import qgemm as q

DEV = "cuda:0"


def listed():
    return [
        # the smallest call: one little layer of a recommender or a detector head, where the launch is everything
        {"name": "tiny_64x64x128", "kind": "tiny", "M": 64, "N": 64, "K": 128, "per_channel": False, "b_zp": False,
         "bias": True, "relu": False},
        # a serving loop at small batch: one token of 16 users through a fully connected layer (weights stream)
        {"name": "fc_small_batch_16x4096x4096", "kind": "fc_small", "M": 16, "N": 4096, "K": 4096, "per_channel": False,
         "b_zp": True, "bias": False, "relu": True},
        # the same kind of layer at a batch of a few hundred rows (a prompt, a bigger batch)
        {"name": "fc_batch_256x8192x8192", "kind": "fc_batch", "M": 256, "N": 8192, "K": 8192, "per_channel": True,
         "b_zp": False, "bias": True, "relu": False},
        # large compute-bound product, the headline of bench.py: per-channel zero points and scales, bias, ReLU
        {"name": "square_8192x8192x8192", "kind": "large", "M": 8192, "N": 8192, "K": 8192, "per_channel": True,
         "b_zp": True, "bias": True, "relu": True},
        # one layer of a recommender's MLP over a big batch: many rows, few columns, short K
        {"name": "mlp_32768x512x1024", "kind": "mlp", "M": 32768, "N": 512, "K": 1024, "per_channel": True,
         "b_zp": False, "bias": False, "relu": False},
        # extents off every tile and alignment, rows cut out of wider matrices
        {"name": "ragged_999x1531x2047", "kind": "ragged", "M": 999, "N": 1531, "K": 2047, "per_channel": True,
         "b_zp": True, "bias": True, "relu": False},
        # fp32 activations in, fp32 result out: a quantized layer inside an fp32 model
        {"name": "fp32_ends_2048x4096x4096", "kind": "fp32", "M": 2048, "N": 4096, "K": 4096, "per_channel": True,
         "b_zp": False, "bias": True, "relu": True},
        # outlier-aware weights (4-bit bulk and a sparse rest) at small batch
        {"name": "outlier_16x8192x8192", "kind": "outlier", "M": 16, "N": 8192, "K": 8192, "per_channel": True,
         "b_zp": False, "bias": True, "relu": False, "frac": 0.005},
        # group convolution of a ResNeXt-like network: 32 groups of 4 channels
        {"name": "group_conv_32x56x56x128_g32", "kind": "gconv", "Nb": 32, "H": 56, "W": 56, "G": 32, "Cg": 4, "Og": 4,
         "R": 3, "stride": 1, "bias": False, "relu": False},
        # depthwise convolution of a mobile network
        {"name": "depthwise_32x56x56x128", "kind": "gconv", "Nb": 32, "H": 56, "W": 56, "G": 128, "Cg": 1, "Og": 1,
         "R": 3, "stride": 1, "bias": True, "relu": True},
        # inner 3 x 3 layer of a ResNet
        {"name": "conv_32x28x28x128_128", "kind": "conv", "Nb": 32, "H": 28, "W": 28, "Cin": 128, "Cout": 128, "R": 3,
         "pad": 1, "stride": 1, "bias": True, "relu": True},
        # first layer of a ResNet: RGB image, 7 x 7, stride 2
        {"name": "first_layer_8x224x224x3_64", "kind": "conv", "Nb": 8, "H": 224, "W": 224, "Cin": 3, "Cout": 64, "R": 7,
         "pad": 3, "stride": 2, "bias": True, "relu": True},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _extent(rng, lo, hi):
    """A layer width: mostly a multiple of 64, 32 or 16 as networks have them, now and then any number."""
    v = _log_int(rng, lo, hi)
    m = rng.choice([64, 64, 32, 16, 1])
    return max(min(lo, m), min(hi, (v + m // 2) // m * m)) if m > 1 else v


def _options(rng):
    return {"per_channel": rng.random() < 0.6, "b_zp": rng.random() < 0.4, "bias": rng.random() < 0.7,
            "relu": rng.random() < 0.5}


def draw(rng):
    kind = rng.choice(["tiny", "fc_small", "fc_batch", "large", "mlp", "ragged", "fp32", "outlier", "gconv", "gconv",
                       "conv", "first"])
    if kind == "tiny":
        return {"kind": kind, "M": _log_int(rng, 1, 64), "N": _log_int(rng, 16, 256), "K": _log_int(rng, 16, 512),
                **_options(rng)}
    if kind == "fc_small":
        return {"kind": kind, "M": _log_int(rng, 1, 64), "N": _extent(rng, 512, 8192), "K": _extent(rng, 512, 8192),
                **_options(rng)}
    if kind == "fc_batch":
        return {"kind": kind, "M": _log_int(rng, 65, 1024), "N": _extent(rng, 1024, 8192),
                "K": _extent(rng, 1024, 8192), **_options(rng)}
    if kind == "large":
        return {"kind": kind, "M": _extent(rng, 2048, 8192), "N": _extent(rng, 2048, 8192),
                "K": _extent(rng, 2048, 8192), **_options(rng)}
    if kind == "mlp":
        return {"kind": kind, "M": _log_int(rng, 4096, 65536), "N": _extent(rng, 64, 1024), "K": _extent(rng, 64, 2048),
                **_options(rng)}
    if kind == "ragged":
        return {"kind": kind, "M": _log_int(rng, 100, 4000) | 1, "N": _log_int(rng, 100, 4000) | 1,
                "K": _log_int(rng, 100, 4000) | 1, **_options(rng)}
    if kind == "fp32":
        return {"kind": kind, "M": _log_int(rng, 16, 4096), "N": _extent(rng, 512, 4096), "K": _extent(rng, 512, 4096),
                **_options(rng)}
    if kind == "outlier":
        return {"kind": kind, "M": _log_int(rng, 1, 64), "N": _extent(rng, 1024, 8192), "K": _extent(rng, 1024, 8192),
                "frac": rng.choice([0.001, 0.005, 0.01]), **_options(rng)}
    side = _log_int(rng, 7, 56)
    images = _log_int(rng, 1, 32)
    flags = {"bias": rng.random() < 0.7, "relu": rng.random() < 0.5}
    if kind == "gconv":
        # channels per group of depthwise, ResNeXt-like and wide-group layers; 32 to 512 channels in all
        cg = rng.choice([1, 1, 4, 4, 8, 16, 32])
        c = min(512, max(32, 32 * _log_int(rng, 1, 16)))
        return {"kind": kind, "Nb": images, "H": side, "W": max(7, side + rng.choice([0, 0, 0, -3, 5])), "G": c // cg,
                "Cg": cg, "Og": cg, "R": 3, "stride": rng.choice([1, 1, 2]), **flags}
    if kind == "conv":
        r = rng.choice([1, 3, 3, 3, 5])
        return {"kind": "conv", "Nb": images, "H": side, "W": max(7, side + rng.choice([0, 0, 0, -3, 5])),
                "Cin": rng.choice([32, 64, 96, 128, 256]), "Cout": rng.choice([32, 64, 96, 128, 256]), "R": r,
                "pad": r // 2, "stride": rng.choice([1, 1, 2]), **flags}
    r = rng.choice([3, 5, 7])
    side = _log_int(rng, 96, 256)
    return {"kind": "conv", "Nb": _log_int(rng, 1, 16), "H": side, "W": side + rng.choice([0, 0, -7, 16]),
            "Cin": rng.choice([1, 3, 3, 3, 4]), "Cout": rng.choice([16, 32, 48, 64]), "R": r, "pad": r // 2,
            "stride": rng.choice([1, 2, 2]), **flags}


# ---------------------------------------------------------------------------- inputs


def _is_gemm(case):
    return "M" in case


def _draw_inputs(case, seed):
    """Everything a call takes, in its natural layout, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    h = torch.Generator()
    h.manual_seed(seed * 104729 + 3)

    def ints(lo, hi, shape, dtype):
        return torch.randint(lo, hi, shape, generator=g, device=DEV, dtype=dtype)

    s = {"case": case}
    if _is_gemm(case):
        M, N, K = case["M"], case["N"], case["K"]
        kind = case["kind"]
        s["a_zp"], s["c_zp"] = 128, 0 if case["relu"] else 128
        std_a, std_b = 74.0, 74.0
        if kind == "mlp":      # activations behind a ReLU, weights of a trained layer
            s["a_zp"] = 0
            s["A"] = torch.randn((M, K), generator=g, device=DEV).mul_(40).abs_().round_().clamp_(max=255).to(torch.uint8)
            B = torch.randn((K, N), generator=g, device=DEV).mul_(30).round_().clamp_(-128, 127).to(torch.int8)
            std_a, std_b = 40.0, 30.0
        elif kind == "fp32":   # a little of it beyond the quantizer's range, which saturates
            s["alpha"], s["inv"] = 0.05, 1.0 / 0.05
            s["A"] = torch.randn((M, K), generator=g, device=DEV).mul_(2.2)
            B = ints(-128, 128, (K, N), torch.int8)
            std_a = 44.0
        elif kind == "outlier":  # narrow bulk and a few large entries, as outlier-aware quantization makes them
            s["A"] = ints(0, 256, (M, K), torch.uint8)
            B = torch.randn((K, N), generator=g, device=DEV).mul_(2.5).round_()
            big = torch.rand((K, N), generator=g, device=DEV) < case["frac"]
            B = torch.where(big, torch.randn((K, N), generator=g, device=DEV).mul_(40).round_(), B)
            B = B.clamp_(-128, 127).to(torch.int8)
            std_b = 4.0
        elif kind == "ragged":   # rows cut out of a wider matrix
            s["A"] = ints(0, 256, (M, K + 5), torch.uint8)[:, 2:K + 2]
            B = ints(-128, 128, (K, N + 3), torch.int8)[:, 1:N + 1]
        else:
            s["A"] = ints(0, 256, (M, K), torch.uint8)
            B = ints(-128, 128, (K, N), torch.int8)
        s["B"] = B
        depth = K
        nz = N if case["per_channel"] else 1
        s["b_zp"] = torch.randint(-8, 9, (nz,), generator=h, dtype=torch.int32).numpy() if case["b_zp"] else \
            torch.zeros(1, dtype=torch.int32).numpy()
    else:
        R = case["R"]
        cin = case["Cin"] if case["kind"] == "conv" else case["G"] * case["Cg"]
        N = case["Cout"] if case["kind"] == "conv" else case["G"] * case["Og"]
        s["a_zp"], s["c_zp"] = 128, 0 if case["relu"] else 128
        s["A"] = ints(0, 256, (case["Nb"], case["H"], case["W"], cin), torch.uint8)
        if case["kind"] == "conv":
            s["B"] = ints(-128, 128, (R, R, cin, N), torch.int8)
            depth = R * R * cin
        else:
            s["B"] = ints(-128, 128, (case["G"], R, R, case["Cg"], case["Og"]), torch.int8)
            depth = R * R * case["Cg"]
        s["b_zp"] = torch.zeros(1, dtype=torch.int32).numpy()
        std_a, std_b = 74.0, 74.0
        nz = N
    s["N"] = N
    s["bias"] = ints(-1000, 1001, (N,), torch.int32) if case["bias"] else None
    # outputs mostly inside 0..255
    s["scales"] = (torch.rand(nz, generator=g, device=DEV).sub_(0.5).exp2_() * (40.0 / (math.sqrt(depth) * std_a * std_b)))
    return s


def prepare(case, seed):
    s = _draw_inputs(case, seed)
    A = s["A"]
    if _is_gemm(case):
        M, N = case["M"], case["N"]
        B = s.pop("B")
        if case["kind"] == "outlier":
            Bp = q.pack_b_outlier(B, s["b_zp"])
        else:
            Bp = q.pack_b(B, s["b_zp"])
        s["Bp"] = Bp
        if case["kind"] in ("fc_small", "fc_batch"):   # a serving loop marshals its calls once
            s["ws"] = q.gemm_workspace(M, Bp)
            out = torch.empty((M, N), dtype=torch.uint8, device=DEV)
            s["call"] = q.PreparedGemm(A, s["a_zp"], Bp, s["bias"], s["scales"], s["c_zp"], case["relu"], out,
                                       workspace=s["ws"])
        elif case["kind"] == "ragged":
            s["out"] = torch.empty((M, N + 7), dtype=torch.uint8, device=DEV)[:, 3:N + 3]
        elif case["kind"] == "fp32":
            s["ws"] = torch.empty(q.gemm_f32_workspace_bytes(M, Bp), dtype=torch.uint8, device=DEV)
        return s
    R, stride = case["R"], case["stride"]
    pad = case["pad"] if case["kind"] == "conv" else R // 2
    ho = (case["H"] + 2 * pad - R) // stride + 1
    wo = (case["W"] + 2 * pad - R) // stride + 1
    out = torch.empty((case["Nb"], ho, wo, s["N"]), dtype=torch.uint8, device=DEV)
    if case["kind"] == "conv":
        s["Bp"] = q.pack_conv_dense_w(s.pop("B"), s["b_zp"])
        s["call"] = q.PreparedConvDense(A, s["Bp"], s["a_zp"], s["bias"], s["scales"], s["c_zp"], case["relu"], pad, stride,
                                        out)
    else:
        s["Bp"] = q.pack_conv_w(s.pop("B"), s["b_zp"])
        s["call"] = q.PreparedConv(A, s["Bp"], s["a_zp"], s["bias"], s["scales"], s["c_zp"], case["relu"], pad, stride, out)
    return s


def run(s):
    if "call" in s:
        s["call"].launch()
        return s["call"].out
    case = s["case"]
    if case["kind"] == "fp32":
        return q.gemm_f32s8_dequant_f32(s["A"], s["inv"], s["a_zp"], s["Bp"], s["bias"], s["scales"], case["relu"],
                                        workspace=s["ws"])
    return q.gemm_u8s8_requant(s["A"], s["a_zp"], s["Bp"], s["bias"], s["scales"], s["c_zp"], case["relu"],
                               out=s.get("out"))


def work(case):
    if _is_gemm(case):
        M, N, K = case["M"], case["N"], case["K"]
        a, b, c = M * K, K * N, M * N
        if case["kind"] == "fp32":
            a, c = 4 * a, 4 * c
        if case["kind"] == "outlier":   # 4 bits for every weight, 4 bytes for every outlier
            b = b // 2 + int(4 * case["frac"] * b)
        return {"bytes": a + b + c + 8 * N, "flops": 2.0 * M * N * K}
    R, stride = case["R"], case["stride"]
    conv = case["kind"] == "conv"
    pad = case["pad"] if conv else R // 2
    ho = (case["H"] + 2 * pad - R) // stride + 1
    wo = (case["W"] + 2 * pad - R) // stride + 1
    cin = case["Cin"] if conv else case["G"] * case["Cg"]
    cout = case["Cout"] if conv else case["G"] * case["Og"]
    depth = R * R * (cin if conv else case["Cg"])
    return {"bytes": case["Nb"] * (case["H"] * case["W"] * cin + ho * wo * cout) + depth * cout + 8 * cout,
            "flops": 2.0 * case["Nb"] * ho * wo * cout * depth}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The same results from 64-bit arithmetic (a product on a rounding tie in fp32 may round the other way here)."""
    s = _draw_inputs(case, seed)
    A, B, N = s["A"].double(), s["B"].double(), s["N"]
    bz = torch.from_numpy(s["b_zp"]).to(DEV).double()
    if _is_gemm(case):
        if case["kind"] == "fp32":
            A = (A * s["inv"]).round_().clamp_(-s["a_zp"], 255 - s["a_zp"])
        else:
            A -= s["a_zp"]
        x = A @ (B - bz)
    else:
        R, stride = case["R"], case["stride"]
        conv = case["kind"] == "conv"
        pad = case["pad"] if conv else R // 2
        A = torch.nn.functional.pad(A - s["a_zp"], (0, 0, pad, pad, pad, pad))
        if not conv:   # as a dense filter with blocks of zeros
            G, cg, og = case["G"], case["Cg"], case["Og"]
            full = torch.zeros((R, R, G, cg, G, og), dtype=torch.float64, device=DEV)
            at = torch.arange(G, device=DEV)
            full[:, :, at, :, at, :] = B
            B = full.reshape(R, R, G * cg, G * og)
        ho = (A.shape[1] - R) // stride + 1
        wo = (A.shape[2] - R) // stride + 1
        x = torch.zeros((A.shape[0] * ho * wo, N), dtype=torch.float64, device=DEV)
        for kh in range(R):
            for kw in range(R):
                a = A[:, kh:kh + (ho - 1) * stride + 1:stride, kw:kw + (wo - 1) * stride + 1:stride]
                x += a.reshape(-1, A.shape[3]) @ B[kh, kw]
        x = x.reshape(A.shape[0], ho, wo, N)
    if s["bias"] is not None:
        x += s["bias"].double()
    x *= s["scales"].double()
    if case.get("kind") == "fp32":
        return x.clamp_(min=0) if case["relu"] else x
    lo = 0 if case["relu"] else -s["c_zp"]
    return (x.round_().clamp_(lo, 255 - s["c_zp"]) + s["c_zp"]).to(torch.uint8)
