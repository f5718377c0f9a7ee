"""The work that a program built on this library has it do, as cases that can be timed and compared.

Five kinds of work, all through the package's public entry points:
  layer     one linear layer's forward, y = S_m V_m^T (scale .* (W~ (V_n S_n x))): at B = 1 (token by
            token generation) qtip_rht_decode_matvec + qtip_rht_f32, at B > 1 (several sequences at
            once, or a prompt) qtip_rht + qtip_decode_matmat + qtip_rht_f32;
  step      the input transform and the product alone, qtip_rht + qtip_decode_matvec: bench.py's step;
  quantize  a weight matrix to code streams, qtip_quantize_gpu;
  ldl       the block LDL decomposition of a proxy Hessian, qtip_block_ldl;
  ldlq      a weight matrix to code streams with feedback, qtip_quantize_ldlq.
Sizes are those of qtip_synth.WORKLOADS and of bench.py, and ragged ones beside them.
"""
import math
from types import SimpleNamespace

import torch

import paper_2406_11235_amd as q

CODES = {"1MAD": q.CODE_1MAD, "3INST": q.CODE_3INST, "HYB": q.CODE_HYB, "HYB2": q.CODE_HYB2,
         "LUT14": q.CODE_LUT, "HYB1": q.CODE_HYB1}
# standard deviation of the values of a code (tables are drawn from N(0, 1))
CODE_SD = {"1MAD": 1.0, "3INST": 1.2437}
MAX_WEIGHTS = 8192 * 28672
MAX_PREFILL = 14336 * 4096 * 997


def code_shape(code):
    """(L, V, T_x, T_y) of a code."""
    return (14, 1, 32, 8) if code == "LUT14" else (16, 2 if code in ("HYB", "HYB2") else 1, 16, 16)


def layer(name, m, n, code, k, B, block_n, block_m, row_scale=False, kind="layer"):
    case = {"kind": kind, "m": m, "n": n, "code": code, "k": k, "B": B,
            "block_n": block_n, "block_m": block_m, "row_scale": row_scale}
    return {"name": name} | case if name else case


def listed():
    return [
        # the smallest layer, with a scale per row: launches and latency are most of it
        layer("layer_1024_3inst_k2_b1", 1024, 1024, "3INST", 2, 1, 1024, 1024, row_scale=True),
        # an attention projection while generating token by token
        layer("layer_4096_3inst_k2_b1", 4096, 4096, "3INST", 2, 1, 4096, 4096),
        # an FFN up projection while generating, 3-bit 1MAD
        layer("layer_14336x4096_1mad_k3_b1", 14336, 4096, "1MAD", 3, 1, 2048, 2048),
        # the benchmark's step on a 70B-class FFN shape
        layer("step_8192x28672_3inst_k2", 8192, 28672, "3INST", 2, 1, 4096, 4096, kind="step"),
        # the same shape as a whole layer in the code with the small table
        layer("layer_8192x28672_hyb_k2_b1", 8192, 28672, "HYB", 2, 1, 4096, 4096),
        # the lookup-only code on a shape that divides into nothing large
        layer("layer_4128x14464_lut14_k2_b1", 4128, 14464, "LUT14", 2, 1, 128, 32),
        # a handful of sequences generated together, 4-bit HYB
        layer("layer_8192_hyb_k4_b4", 8192, 8192, "HYB", 4, 4, 4096, 4096),
        # many sequences generated together
        layer("layer_8192_hyb_k4_b64", 8192, 8192, "HYB", 4, 64, 4096, 4096),
        # a prompt of no round length
        layer("prefill_14336x4096_3inst_k2_b997", 14336, 4096, "3INST", 2, 997, 2048, 2048),
        # a matrix quantized block by block on its own
        {"name": "quantize_2048_3inst_k2", "kind": "quantize", "m": 2048, "n": 2048, "code": "3INST", "k": 2},
        # the decomposition that comes before quantizing with feedback
        {"name": "ldl_2048_g16", "kind": "ldl", "n": 2048, "g": 16},
        # a matrix quantized with feedback: one column block after the other
        {"name": "ldlq_2048x1024_3inst_k2", "kind": "ldlq", "m": 2048, "n": 1024, "code": "3INST", "k": 2},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(size, unit):
    return max(1, round(size / unit)) * unit


def _block(size):
    """The Hadamard block of a dimension: the largest power of two in it, at most 4096."""
    return min(4096, size & -size)


def draw(rng):
    what = rng.choices(("b1", "step", "batch", "prefill", "quantize", "ldl", "ldlq"), (30, 6, 22, 16, 10, 6, 10))[0]
    if what == "ldl":
        return {"kind": "ldl", "n": _multiple(_log_uniform(rng, 256, 2048), 16),
                "g": rng.choice((8, 16, 16))}
    code = rng.choices(tuple(CODES), (2, 4, 4, 1, 1, 1))[0]
    k = rng.choice((2, 2, 3, 4))
    if what in ("quantize", "ldlq"):
        m = _multiple(_log_uniform(rng, 128, 2048), 32)
        n = _multiple(_log_uniform(rng, 128, 2048 if what == "quantize" else 1024), 16)
        return {"kind": what, "m": m, "n": n, "code": code, "k": k}
    # a power of two in every dimension that the Hadamard blocks are cut from, times anything
    unit_m, unit_n = 1 << rng.randint(5, 12), 1 << rng.randint(5, 12)
    hi = 14336 if what in ("batch", "prefill") else 28672
    m = _multiple(_log_uniform(rng, 768, hi), unit_m)
    n = _multiple(_log_uniform(rng, 768, hi), unit_n)
    while m * n > MAX_WEIGHTS:
        m = max(unit_m, _multiple(m / 2, unit_m))
    B = 1
    if what == "batch":
        B = round(_log_uniform(rng, 2, 64))
    elif what == "prefill":
        B = round(_log_uniform(rng, 65, min(1024, max(66, MAX_PREFILL / (m * n)))))
    return layer(None, m, n, code, k, B, _block(n), _block(m), row_scale=rng.random() < 0.25,
                 kind="step" if what == "step" else "layer")


def _lut(code, g):
    count = {"HYB": 1024, "HYB2": 1024, "LUT14": 1 << 14, "HYB1": 64}.get(code)
    return None if count is None else torch.randn(count, device="cuda", generator=g).half()


def _signs(n, g):
    return (torch.randint(0, 2, (n,), device="cuda", generator=g, dtype=torch.int8) * 2 - 1)


def _correlated(n, g):
    """Inputs of a layer that go strongly together, as a layer's inputs do: 2 n samples of n values."""
    X = torch.randn(2 * n, n, dtype=torch.float64, device=g.device, generator=g)
    return 0.9 * X[:, :1] + 0.1 * X


def _hessian(n, g):
    X = _correlated(n, g)
    return X.T @ X / (2 * n) + 1e-3 * torch.eye(n, dtype=torch.float64, device=g.device)


def _feedback(n, ty, seed):
    """L - I of H = L D L^T in ty x ty blocks, made on the host from a Cholesky factor, and rounded to few
    enough bits that the last ones of that factor do not matter."""
    C = torch.linalg.cholesky(_hessian(n, torch.Generator(device="cpu").manual_seed(seed)))
    blocks = torch.stack([C[i:i + ty, i:i + ty] for i in range(0, n, ty)])
    inverse = torch.linalg.inv(blocks)
    L = torch.cat([C[:, i:i + ty] @ inverse[i // ty] for i in range(0, n, ty)], dim=1)
    index = torch.arange(n) // ty
    L[index[:, None] <= index[None, :]] = 0
    return L.half().float().cuda()


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    s = SimpleNamespace(**case)
    if s.kind == "ldl":
        s.H = _hessian(s.n, g)
        s.A = torch.empty(s.n, s.n, device="cuda")
        s.D = torch.empty(s.n // s.g, s.g, s.g, dtype=torch.float64, device="cuda")
        s.ws = torch.empty(q.qtip_block_ldl_workspace(s.n), dtype=torch.uint8, device="cuda")
        return s
    s.L, s.V, tx, ty = code_shape(s.code)
    s.id = CODES[s.code]
    s.lut = _lut(s.code, g)
    tiles = s.m * s.n // 256
    if s.kind in ("quantize", "ldlq"):
        s.W = torch.randn(s.m, s.n, device="cuda", generator=g) * CODE_SD.get(s.code, 1.0)
        s.codes = torch.zeros(tiles, 8 * s.k, dtype=torch.int32, device="cuda")
        s.err = torch.zeros(tiles, device="cuda")
        if s.kind == "quantize":
            size = q.qtip_quantize_gpu_workspace(s.k, s.V, min(tiles, 4096))
        else:
            s.A = _feedback(s.n, ty, seed)
            s.What = torch.empty(s.m, s.n, device="cuda")
            size = q.qtip_quantize_ldlq_workspace(s.m, s.n, s.k, s.V, s.m // 16)
        s.ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        return s
    s.codes = torch.randint(-2**31, 2**31, (tiles, 8 * s.k), dtype=torch.int32, device="cuda", generator=g)
    s.x = torch.randn(s.B, s.n, device="cuda", generator=g).half()
    s.signs_n, s.signs_m = _signs(s.n, g), _signs(s.m, g)
    s.scale = (torch.rand(s.m, device="cuda", generator=g) + 0.5).half() if s.row_scale else None
    s.xt = torch.empty_like(s.x)
    s.z = torch.empty(s.B, s.m, device="cuda")
    s.y = torch.empty(s.B, s.m, dtype=torch.float16, device="cuda")
    return s


def run(s):
    if s.kind == "layer":
        if s.B == 1:
            q.qtip_rht_decode_matvec(s.codes, s.L, s.k, s.V, s.id, s.lut, s.m, s.n, s.x, s.signs_n, s.block_n,
                                     s.scale, s.z, s.xt)
        else:
            q.qtip_rht(s.x, s.signs_n, s.n, s.block_n, s.B, 0, s.xt)
            q.qtip_decode_matmat(s.codes, s.L, s.k, s.V, s.id, s.lut, s.m, s.n, s.xt, s.B, s.scale, s.z)
        q.qtip_rht_f32(s.z, s.signs_m, s.m, s.block_m, s.B, 1, s.y)
        return s.y
    if s.kind == "step":
        q.qtip_rht(s.x, s.signs_n, s.n, s.block_n, 1, 0, s.xt)
        q.qtip_decode_matvec(s.codes, s.L, s.k, s.V, s.id, s.lut, s.m, s.n, s.xt, s.z)
        return s.z
    if s.kind == "quantize":
        q.qtip_quantize_gpu(s.W, s.m, s.n, s.L, s.k, s.V, s.id, s.lut, s.codes, s.err, s.ws, s.ws.numel())
        return s.codes, s.err
    if s.kind == "ldl":
        q.qtip_block_ldl(s.H, s.n, s.g, s.A, s.D, s.ws, s.ws.numel())
        return s.A, s.D
    q.qtip_quantize_ldlq(s.W, s.A, s.m, s.n, s.L, s.k, s.V, s.id, s.lut, s.codes, s.What, s.err, s.ws,
                         s.ws.numel())
    return s.codes, s.What, s.err


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "ldl":
        # H's lower triangle once, A and D once; n^3 / 3 multiply-adds
        return {"bytes": 4 * n * n + 4 * n * n + 8 * n * case["g"], "flops": 2 * n**3 / 3}
    m, k = case["m"], case["k"]
    L, V, _, ty = code_shape(case["code"])
    table = {"HYB": 2048, "HYB2": 2048, "LUT14": 2 << 14, "HYB1": 128}.get(case["code"], 0)
    codes = m * n * k // 8
    if kind in ("quantize", "ldlq"):
        # two passes of 256 / V steps over 2^L states; at V = 1 a state is a difference, a multiply-add and
        # a minimum, at V = 2 an addition and a minimum
        flops = m * n / 256 * 2 * (256 // V) * 2**L * (4 if V == 1 else 2)
        size = 4 * m * n + codes + 4 * (m * n // 256) + table
        if kind == "ldlq":
            size += 4 * m * n + 4 * n * (n - ty) // 2  # What; A below its diagonal blocks
            flops += m * n * (n - ty)
        return {"bytes": size, "flops": flops}
    B = case["B"]
    size = codes + table + B * 2 * n + n + (2 * m if case["row_scale"] else 0)
    flops = 2 * B * m * n + B * n * (math.log2(case["block_n"]) + 2)
    if kind == "step":
        return {"bytes": size + 4 * m, "flops": flops}
    return {"bytes": size + m + B * 2 * m, "flops": flops + B * m * (math.log2(case["block_m"]) + 2)}


def tolerance(case):
    if case["kind"] in ("quantize", "ldlq"):
        return "exact"  # every rounding of the search and of the feedback is part of the interface
    if case["kind"] == "ldl":
        return {"rel": 1e-6}  # binary64, A rounded to binary32
    if case["kind"] == "step":
        return {"rel": 1e-4}  # binary32 sums over activations rounded to binary16
    return {"rel": 1e-3}  # the same, rounded to binary16
