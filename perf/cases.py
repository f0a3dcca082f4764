"""The framework's work in real use, as cases that can be timed and checked.

A case is a dict of plain values:

  kind      "decode"   decompress one resident stream into a BF16 tensor
                       (codec.decode_block)
            "forward"  decompress a transformer block and multiply it by its
                       activations (codec.block_forward, or its variant that
                       takes no workspace with "noalloc")
            "gemm"     the products of a block that is already decompressed
                       (codec.block_gemm)
            "gemv"     one token straight from the compressed block
                       (codec.block_gemv)
            "encode"   compress a BF16 tensor held by the host into the
                       caller's buffers (codec.build_codebook, df11_encode,
                       codec.build_tables)
  n         weights, for decode and encode
  hidden, kv, ffn      sizes of the block's seven matrices, for the others
  tokens    activation rows
  dist      "gaussian" (one standard deviation per matrix, as trained linear
            layers have) or "heavy" (Student t with 3 degrees of freedom, some
            outliers and exact zeros)
  threads   chunks per stream block; 0 takes the library's choice for the size
"""
import ctypes
import math

import numpy as np
import torch

from paper_2504_11651_amd import codec

# Mean Huffman code length of an exponent in bits: Gaussian weights need about
# 2.6 whatever their standard deviation, a block with seven of them 2.65, the
# heavy-tailed mixture 2.85.
CODE_BITS = {"gaussian": 2.64, "heavy": 2.85}
PIECE = 1 << 26  # weights drawn at once


def listed():
    b8 = {"hidden": 4096, "kv": 1024, "ffn": 14336, "dist": "gaussian"}
    return [
        # the smallest useful stream: one 1024 x 4096 key or value projection,
        # or a 1,024-row slice of an LM head; latency and the launch count
        {"name": "decode_4m", "kind": "decode", "n": 1024 * 4096, "dist": "gaussian", "threads": 0},
        # one 4096 x 4096 projection
        {"name": "decode_16m", "kind": "decode", "n": 4096 * 4096, "dist": "gaussian", "threads": 0},
        # a middle-sized tensor that ends inside every unit of the format,
        # with the long codes of heavy tails
        {"name": "decode_heavy_100m", "kind": "decode", "n": 100_000_007, "dist": "heavy", "threads": 0},
        # a Llama-3-8B-sized transformer block, one stream
        {"name": "decode_8b", "kind": "decode", "n": 218_103_808, "dist": "gaussian", "threads": 0},
        # a Llama-3.1-70B-sized transformer block, the benchmark's headline
        {"name": "decode_70b", "kind": "decode", "n": 855_638_016, "dist": "gaussian", "threads": 0},
        # generating one token: the block is decompressed into the workspace
        # and consumed by its seven products
        {"name": "forward_8b_t1", "kind": "forward", "tokens": 1, "noalloc": False, "threads": 0, **b8},
        # a batch of decoding sequences
        {"name": "forward_8b_t16", "kind": "forward", "tokens": 16, "noalloc": False, "threads": 0, **b8},
        # the largest batch of a call: a prefill chunk of 64 tokens
        {"name": "forward_8b_t64", "kind": "forward", "tokens": 64, "noalloc": False, "threads": 0, **b8},
        # products of a block that stays decompressed, an odd batch
        {"name": "gemm_8b_t5", "kind": "gemm", "tokens": 5, **b8},
        # the same at a batch that fills three of four token slices and a bit
        {"name": "gemm_8b_t49", "kind": "gemm", "tokens": 49, **b8},
        # one token without a decompressed copy of the block
        {"name": "gemv_8b", "kind": "gemv", "tokens": 1, "threads": 64, **b8},
        # compressing one 4096 x 4096 projection when a model is converted
        {"name": "encode_16m", "kind": "encode", "n": 4096 * 4096, "dist": "gaussian", "threads": 0},
    ]


def draw(rng):
    """One more case of the listed ones' ranges."""
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "decode", "forward", "forward", "gemm", "gemv", "encode"])
    dist = rng.choice(["gaussian", "gaussian", "heavy"])
    if kind == "decode":
        return {"kind": kind, "n": log_uniform(1_000_003, 500_000_003), "dist": dist,
                "threads": rng.choice([0, 0, 0, 0, 64, 128, 256, 512, 1024])}
    if kind == "encode":
        return {"kind": kind, "n": log_uniform(1_000_003, 40_000_003), "dist": dist,
                "threads": rng.choice([0, 0, 64, 128])}
    # grouped-query blocks: rows are multiples of 16 and columns of 64, not of
    # the kernels' larger tiles
    hidden = 64 * rng.randint(32, 72)
    case = {"kind": kind, "hidden": hidden, "kv": hidden // rng.choice([1, 2, 4, 8]) // 16 * 16,
            "ffn": 64 * int(hidden * rng.uniform(2.5, 3.6) / 64), "dist": dist,
            "tokens": 1 if kind == "gemv" else log_uniform(1, 64)}
    if kind == "gemv":
        case["threads"] = 64
    if kind == "forward":
        case["threads"] = rng.choice([0, 0, 0, 64, 128, 256])
        case["noalloc"] = rng.choice([False, False, True])
    return case


def shapes(case):
    """(offset, rows, cols) of q, k, v, o, gate, up and down in the block."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    out, off = [], 0
    for rows, cols in ((h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f)):
        out.append((off, rows, cols))
        off += rows * cols
    return out


def weight_count(case):
    if "n" in case:
        return case["n"]
    off, rows, cols = shapes(case)[-1]
    return off + rows * cols


def weights(case, seed):
    """The case's BF16 weights on the GPU."""
    n = weight_count(case)
    parts = [r * c for _, r, c in shapes(case)] if "n" not in case else [n]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")

    def normal(k):
        return torch.randn(k, generator=gen, device="cuda", dtype=torch.float32)

    at = 0
    for size in parts:
        sigma = 0.02 if len(parts) == 1 else \
            0.008 + 0.032 * float(torch.rand(1, generator=gen, device="cuda"))
        while size:
            k = min(size, PIECE)
            v = normal(k) * sigma
            if case["dist"] == "heavy":
                # Student t with 3 degrees of freedom: N / sqrt(chi2_3 / 3)
                chi = normal(k).square_()
                chi += normal(k).square_()
                chi += normal(k).square_()
                v *= (3.0 / chi).sqrt_()
                u = torch.rand(k, generator=gen, device="cuda")
                big = torch.exp2(6.0 * torch.rand(k, generator=gen, device="cuda"))
                v = torch.where(u < 1e-4, torch.copysign(big, v), v)
                v = torch.where(u > 0.99, torch.zeros_like(v), v)
            out[at:at + k] = v
            at += k
            size -= k
    return out


def activations(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed + 1_000_003)
    return [torch.randn((case["tokens"], c), generator=gen, device="cuda").to(torch.bfloat16)
            for _, _, c in shapes(case)]


def host_bits(w):
    return w.view(torch.int16).cpu().numpy().view(np.uint16)


def layout(case, n):
    return codec.make_layout(8, case["threads"], 11) if case["threads"] else codec.default_layout(n)


def prepare(case, seed):
    """What a program holds before the call: resident compressed weights,
    activations, output and workspace buffers."""
    kind, n = case["kind"], weight_count(case)
    w = weights(case, seed)
    if kind == "encode":
        # room for codes of 4 bits on average, whatever the weights
        return {"kind": kind, "w": host_bits(w), "layout": layout(case, n),
                "exp": np.zeros(n // 2 + 65536, np.uint8), "sm": np.zeros((n + 15) // 16 * 16 + 16, np.uint8),
                "gaps": np.zeros(n // 24 + 65536, np.uint8), "block_pos": np.zeros(n // 1024 + 1024, np.uint32)}
    st = {"kind": kind}
    if kind != "gemm":
        st["stream"] = codec.to_device(codec.encode(host_bits(w), layout=layout(case, n)))
    if kind == "decode":
        st["out"] = torch.empty_like(w)
        return st
    mats = shapes(case)
    st["mats"] = mats
    st["x"] = activations(case, seed)
    st["y"] = [torch.empty((case["tokens"], r), dtype=torch.float32, device="cuda")
               for _, r, _ in mats]
    if kind == "gemm":
        st["w"] = w
    if kind == "forward":
        st["noalloc"] = case["noalloc"]
        st["out"] = torch.empty_like(w)
    if kind == "gemv":
        need = codec.gemv_workspace_bytes(st["stream"], mats)
    else:
        need = codec.gemm_workspace_bytes(mats, case["tokens"])
    if kind == "forward" and case["noalloc"] and need > codec.STATIC_SCRATCH_BYTES:
        st["noalloc"] = False  # more partial sums than the library's own array holds
    st["workspace"] = torch.empty(max(need // 4, 4), dtype=torch.float32, device="cuda")
    return st


def run(st):
    """One pass.  Decompressed weights are returned as 16-bit patterns."""
    kind = st["kind"]
    if kind == "decode":
        return codec.decode_block(st["stream"], st["out"]).view(torch.int16)
    if kind == "encode":
        book = codec.build_codebook(st["w"])
        sizes, args = codec.Sizes(), []
        for key in ("exp", "sm", "gaps", "block_pos"):
            args += [st[key].ctypes.data, st[key].nbytes]
        rc = codec.lib().df11_encode(st["w"].ctypes.data, st["w"].size, ctypes.byref(book),
                                     ctypes.byref(st["layout"]), *args, ctypes.byref(sizes))
        if rc != codec.DF11_OK:
            raise RuntimeError(codec.strerror(rc))
        return {"exp": st["exp"], "sm": st["sm"], "gaps": st["gaps"],
                "block_pos": st["block_pos"].view(np.int32), "total_bits": int(sizes.total_bits),
                "tables": codec.build_tables(book, st["layout"].lut_bits)}
    if kind == "gemm":
        return codec.block_gemm(st["w"], st["mats"], st["x"], st["y"], st["workspace"])
    if kind == "gemv":
        return codec.block_gemv(st["stream"], st["mats"], st["x"], st["y"], st["workspace"])
    if st["noalloc"]:
        y = codec.block_forward_noalloc(st["stream"], st["out"], st["mats"], st["x"], st["y"])
    else:
        y = codec.block_forward(st["stream"], st["out"], st["mats"], st["x"], st["y"],
                                st["workspace"])
    return {"weights": st["out"].view(torch.int16), "y": y}


def work(case):
    """Bytes and operations of one pass: the compressed stream (a byte of sign
    and mantissa, the exponent's code and its share of a 5-bit gap per 64 bits
    for each weight), the decompressed weights where they are an input or an
    output, activations and results; two operations per weight and token."""
    kind, n = case["kind"], weight_count(case)
    packed = n * (1 + CODE_BITS[case["dist"]] / 8 * (1 + 5 / 64))
    if kind in ("decode", "encode"):
        return {"bytes": packed + 2 * n}
    t = case["tokens"]
    io = sum(2 * t * c + 4 * t * r for _, r, c in shapes(case))
    held = {"forward": packed + 2 * n, "gemm": 2 * n, "gemv": packed}[kind]
    return {"bytes": held + io, "flops": 2 * t * n}


def tolerance(case):
    if case["kind"] in ("decode", "encode"):
        return "exact"
    # sums of up to 14,336 exact BF16 products in 32 bits: against 64 bits the
    # products differ by 0.8e-7 to 4.0e-7 over the token counts (largest
    # difference 3.0e-6 of the root mean square); four times that
    return {"rel": 1.6e-6, "max": 1.2e-5}


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        return None  # a stream of codes and tables: its bytes are compared
    w = weights(case, seed)
    if kind == "decode":
        return w.view(torch.int16)
    y = [x.double() @ w[off:off + r * c].view(r, c).double().t()
         for (off, r, c), x in zip(shapes(case), activations(case, seed))]
    return {"weights": w.view(torch.int16), "y": y} if kind == "forward" else y
