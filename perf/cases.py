"""Performance cases of the SFC-CA GEMM library: the calls its users make.

Every case is one call of a public entry point of
``paper_2601_16294_amd.sfcgemm`` on operands that already lie on the GPU.  The
families, and what each stands for:

  small     the paper's smallest cubes: latency, launches and the host path
  square    large and ordinary square-ish bf16 products, bf16 output
  ragged    sides that are no multiple of a block, aligned rows, fp32 output
  odd       any sides at all (rows not 16-byte aligned), as a batch of tokens
            or a vocabulary of odd size gives them; fp32 and bf16 output
  kdom      K-dominant shapes, the layer count left to the library
  shortk    short contractions (the sweep's K = 512 edge): the store of C counts
  prefill   activations times weights, decoder projections (4096 / 14336)
  decode    a few tokens times weights: the weights are read once, from memory
  serve     the entry point that allocates nothing, mixed batch of tokens
  fp8       OCP 8-bit operands, either format, fp32 or bf16 output

Operands may be column slices of wider matrices (``pad`` extra columns), as a
fused projection weight is.
"""
import math

import torch

from paper_2601_16294_amd import sfcgemm as sg

_FP8 = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}
_OUT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(family, M, N, K, out, ca=1, dist="normal", pad=0, fa="", fb=""):
    return {"family": family, "M": M, "N": N, "K": K, "out": out, "ca": ca, "dist": dist, "pad": pad, "fa": fa,
            "fb": fb}


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # the paper's smallest cube, one layer: latency
        named("small512_f32", "small", 512, 512, 512, "f32", dist="uniform"),
        # a small product of odd sides (tokens x odd head width)
        named("odd333x517x421_bf16", "odd", 333, 517, 421, "bf16", ca=0),
        # a few tokens times an up-projection: reads 112 MiB of weights
        named("decode16x14336x4096_bf16", "decode", 16, 14336, 4096, "bf16", ca=0, dist="weights"),
        # a mixed batch of 256 tokens in a serving loop that may not allocate
        named("serve256x4096x4096_bf16", "serve", 256, 4096, 4096, "bf16", ca=0, dist="weights"),
        # ragged edges on both sides, fp32 output
        named("ragged3000x7000x2048_f32", "ragged", 3000, 7000, 2048, "f32", dist="uniform"),
        # no side a multiple of anything: unaligned rows of A, B and C
        named("odd3001x5003x2047_f32", "odd", 3001, 5003, 2047, "f32", dist="uniform"),
        # short contraction of the sweep: C dominates the traffic
        named("shortk8192x4096x512_bf16", "shortk", 8192, 4096, 512, "bf16", ca=0, dist="uniform"),
        # communication-avoiding shape, the library picks the layers
        named("kdom1024x1024x65536_f32", "kdom", 1024, 1024, 65536, "f32", ca=0, dist="normal0.1"),
        # 4096 tokens times an up-projection
        named("prefill4096x14336x4096_bf16", "prefill", 4096, 14336, 4096, "bf16", dist="weights"),
        # the headline square product
        named("square8192_bf16", "square", 8192, 8192, 8192, "bf16"),
        # 8-bit operands: the same prefill, and a ragged mixed-format product
        named("fp8_prefill4096x14336x4096_bf16", "fp8", 4096, 14336, 4096, "bf16", fa="e4m3", fb="e4m3"),
        named("fp8_ragged3000x7008x2048_f32", "fp8", 3000, 7008, 2048, "f32", ca=0, fa="e5m2", fb="e4m3"),
    ]


def _log(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(mult, int(round(v / mult)) * mult)


_MAX_FLOPS = 2.0 * 8192 ** 3


def draw(rng):
    """One more call of the families above, sizes spread over their ranges."""
    family = rng.choice(["small", "square", "ragged", "odd", "odd", "kdom", "shortk", "prefill", "decode", "decode",
                         "serve", "fp8"])
    out = rng.choice(["f32", "bf16"])
    pad = rng.choice([0, 0, 64])
    while True:
        if family == "small":
            c = _case(family, _log(rng, 64, 1024, 8), _log(rng, 64, 1024, 8), _log(rng, 64, 1024, 8), out,
                      ca=rng.choice([0, 1]), dist="uniform", pad=pad)
        elif family == "square":
            c = _case(family, _log(rng, 1024, 8192, 64), _log(rng, 1024, 8192, 64), _log(rng, 1024, 8192, 64),
                      "bf16", ca=rng.choice([0, 1]), pad=pad)
        elif family == "ragged":
            c = _case(family, _log(rng, 500, 6000), _log(rng, 500, 8000, 8), _log(rng, 500, 6000, 8), "f32",
                      dist="uniform", pad=pad)
        elif family == "odd":
            c = _case(family, _log(rng, 100, 6000), _log(rng, 100, 6000), _log(rng, 100, 6000), out,
                      ca=rng.choice([0, 1]), dist="uniform")
        elif family == "kdom":
            c = _case(family, _log(rng, 128, 2048, 64), _log(rng, 128, 2048, 64), _log(rng, 8192, 65536, 64), out,
                      ca=0, dist="normal0.1", pad=pad)
        elif family == "shortk":
            c = _case(family, _log(rng, 1024, 8192, 64), _log(rng, 1024, 8192, 64), _log(rng, 64, 512, 8), out,
                      ca=rng.choice([0, 1]), dist="uniform", pad=pad)
        elif family == "prefill":
            c = _case(family, _log(rng, 512, 8192), rng.choice([4096, 6144, 14336]), rng.choice([4096, 14336]),
                      "bf16", dist="weights", pad=pad)
        elif family == "decode":
            c = _case(family, _log(rng, 1, 64), _log(rng, 1024, 16384, 64), _log(rng, 1024, 16384, 64), "bf16",
                      ca=0, dist="weights", pad=pad)
        elif family == "serve":
            m = _log(rng, 64, 1024)
            n = _log(rng, 512, 8192, 64)
            # the library's static workspace bounds the layer copies of ca = 0
            c = _case(family, m, n, _log(rng, 1024, 8192, 64), "bf16", ca=0 if m * n <= 1 << 20 else 1,
                      dist="weights", pad=pad)
        else:
            c = _case(family, _log(rng, 512, 8192, 1), _log(rng, 512, 14336, 16), _log(rng, 512, 8192, 16), out,
                      ca=rng.choice([0, 1]), pad=pad, fa=rng.choice(["e4m3", "e5m2"]), fb=rng.choice(["e4m3", "e5m2"]))
        # no dearer than the headline product (8-bit operands run at twice the rate)
        if 2.0 * c["M"] * c["N"] * c["K"] <= _MAX_FLOPS:
            return c


def _matrix(gen, rows, cols, std, uniform, dtype, pad):
    """rows x cols of `dtype`, a column slice of a matrix `pad` columns wider."""
    x = torch.empty((rows, cols + pad), dtype=torch.float32, device="cuda")
    if uniform:
        x.uniform_(-1.0, 1.0, generator=gen)
    else:
        x.normal_(0.0, std, generator=gen)
    return x.to(dtype)[:, :cols]


def _operands(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    uniform = case["dist"] == "uniform"
    std = {"normal0.1": (0.1, 0.1), "weights": (1.0, 0.02)}.get(case["dist"], (1.0, 1.0))
    ta = _FP8[case["fa"]] if case["fa"] else torch.bfloat16
    tb = _FP8[case["fb"]] if case["fb"] else torch.bfloat16
    A = _matrix(gen, case["M"], case["K"], std[0], uniform, ta, case["pad"])
    B = _matrix(gen, case["K"], case["N"], std[1], uniform, tb, case["pad"])
    return A, B


def prepare(case, seed):
    A, B = _operands(case, seed)
    C = torch.empty((case["M"], case["N"]), dtype=_OUT[case["out"]], device="cuda")
    return {"A": A, "B": B, "C": C, "case": case}


def run(state):
    case, A, B, C = state["case"], state["A"], state["B"], state["C"]
    if case["family"] == "fp8":
        sg.sfc_gemm_f8_ex(A, B, C, ca_layers=case["ca"], a_format=case["fa"], b_format=case["fb"])
    elif case["family"] == "serve":
        sg.sfc_gemm_noalloc_ex(A, B, C, ca_layers=case["ca"])
    elif case["out"] == "bf16":
        sg.sfc_gemm_bf16out(A, B, C, ca_layers=case["ca"])
    else:
        sg.sfc_gemm(A, B, C, ca_layers=case["ca"])
    return C


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    e = 1 if case["family"] == "fp8" else 2
    return {"bytes": e * (M * K + K * N) + (4 if case["out"] == "f32" else 2) * M * N, "flops": 2 * M * N * K}


def tolerance(case):
    # About four times the start's own distance from the 64-bit product: bf16
    # output is one rounding of the fp32 sum (1.7e-3 in the 2-norm, at most 2^-8
    # of the value); fp32 output carries the rounding of fp32 sums over K (1e-7
    # to 4e-7); the 8-bit matrix instruction adds its 64 products with fewer bits
    # (1.1e-5).
    if case["out"] == "bf16":
        return {"rel": 6.6e-3, "max": 1.6e-2}
    if case["family"] == "fp8":
        return {"rel": 4.5e-5, "max": 4e-4}
    return {"rel": 2e-6, "max": 1e-5}


def exact(case, seed):
    A, B = _operands(case, seed)
    if case["fa"]:
        A, B = A.to(torch.float32), B.to(torch.float32)
    # row bands keep the 64-bit copies small
    Bd = B.to(torch.float64)
    step = max(1, (1 << 28) // max(1, case["K"]))
    return torch.cat([A[i:i + step].to(torch.float64) @ Bd for i in range(0, case["M"], step)])
