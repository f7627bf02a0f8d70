"""The work that a user of this library has it do, through its public entry points: what is timed when the
library's speed is measured, and what its results are compared with.

`listed()` holds one case per kind of use, `draw(rng)` more cases of the same ranges.  All results are whole
numbers with one correct value, so the tolerance is "exact" everywhere.

Kinds of use and the ranges they stand for (M rows of activations, N output columns, K depth):
  skinny    decoding and recurrent gates, M = 1 .. 32: the smallest calls, and weights streamed from memory
  mid       decoding with many sequences or short prompts, M = 33 .. 256
  large     prompts, training-sized batches and plain square products, M, N up to 8192, odd sizes and unaligned
            rows among them
  ffn       the two fully connected layers of a transformer block, u8 in and out, one behind the other
  s16       16-bit operands, small and large
  unpacked  both operands are inputs of the call (nothing was packed beforehand)
  batched   many independent products of odd sizes in one call
  pack      laying out a weight when a model is loaded
"""
import math

import numpy as np
import torch

import paper_1910_00178_amd as ng
from paper_1910_00178_amd.workloads import batched_shapes

# entry points of one product; the kinds above draw from them
OPS = ("s32", "u8", "channel", "s8s8", "u8u8", "s16", "unpacked")


def _gemm(name, use, op, M, N, K, za=128, zb=0, pitch="padded", **more):
    case = {"use": use, "op": op, "M": M, "N": N, "K": K, "za": za, "zb": zb, "pitch": pitch, **more}
    return {"name": name, **case} if name else case


def listed():
    return [
        # LSTM gates of one sequence (a step's input times the stacked gate weights): the smallest call
        _gemm("gates_1x4096x1024", "skinny", "s32", 1, 4096, 1024, za=0, values="uniform"),
        # decoding 16 sequences through a wide layer with per-column scales and bias: the weight is a stream
        _gemm("decode_16x16384x4096_channel", "skinny", "channel", 16, 16384, 4096),
        # decoding 64 sequences, weights with a zero-point
        _gemm("decode_64x4096x4096", "mid", "s32", 64, 4096, 4096, zb=3),
        # the two layers of a 768 / 3072 transformer block on 1024 tokens, u8 activations throughout
        {"name": "ffn_1024x768x3072", "use": "ffn", "op": "channel", "M": 1024, "D": 768, "H": 3072, "pitch": "padded"},
        # unsigned weights (zero-point near 128: the row sums of A are always needed)
        _gemm("u8u8_2048x4096x1024", "large", "u8u8", 2048, 4096, 1024, zb=131),
        # odd sizes in every direction, rows as long as K: no row but the first is aligned
        _gemm("ragged_2047x3071x1537", "large", "s32", 2047, 3071, 1537, zb=-3, pitch="tight"),
        # the largest: a square product on uniform operands
        _gemm("square_8192", "large", "s32", 8192, 8192, 8192, za=0, values="uniform"),
        # 16-bit activations through a small layer, and a large 16-bit product
        _gemm("s16_512x768x768", "s16", "s16", 512, 768, 768, za=37, zb=-21),
        _gemm("s16_4096", "s16", "s16", 4096, 4096, 4096, za=0, zb=0),
        # both operands computed at run time (attention scores and the like), ragged outputs
        _gemm("unpacked_777x1000x320", "unpacked", "unpacked", 777, 1000, 320),
        # 64 products of odd sizes from 1 to thousands, every one with its own zero-points
        {"name": "batched_64", "use": "batched", "op": "batched", "count": 64, "mmax": 2048, "nmax": 4096, "kmax": 4096, "shapes": 0},
        # loading a weight of 64 MiB
        {"name": "pack_16384x4096", "use": "pack", "op": "pack", "N": 16384, "K": 4096, "pitch": "padded"},
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm; every other one a multiple of 64 where the range has room."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if hi >= 128 and rng.random() < 0.5:
        n = max(64, (n + 32) // 64 * 64)
    return max(lo, min(hi, n))


def draw(rng):
    use = rng.choice(("skinny", "skinny", "mid", "mid", "large", "large", "ffn", "s16", "s16", "unpacked", "batched", "pack"))
    pitch = rng.choice(("padded", "padded", "tight"))
    if use == "ffn":
        D = rng.choice((256, 512, 768, 1000, 1024, 1536))
        return {"use": use, "op": "channel", "M": _log(rng, 32, 4096), "D": D, "H": 4 * D, "pitch": pitch}
    if use == "batched":
        mmax = rng.choice((16, 128, 512, 2048))
        return {"use": use, "op": "batched", "count": rng.randint(8, 64), "mmax": mmax, "nmax": rng.choice((1024, 4096)),
                "kmax": rng.choice((1024, 4096)), "shapes": rng.randint(1, 999)}
    if use == "pack":
        return {"use": use, "op": rng.choice(("pack", "pack", "pack_u8", "pack_s16")), "N": _log(rng, 64, 16384), "K": _log(rng, 64, 8192),
                "pitch": pitch}
    if use == "skinny":
        op = rng.choice(("s32", "s32", "u8", "channel", "s8s8", "u8u8", "unpacked"))
        M, N, K = rng.choice((1, 1, 2, 4, 7, 8, 13, 16, 25, 32)), _log(rng, 256, 32768), _log(rng, 128, 8192)
    elif use == "mid":
        op = rng.choice(("s32", "s32", "u8", "channel", "s8s8", "u8u8"))
        M, N, K = _log(rng, 33, 256), _log(rng, 256, 16384), _log(rng, 128, 8192)
    elif use == "large":
        op = rng.choice(("s32", "s32", "u8", "channel", "s8s8", "u8u8"))
        M, N, K = _log(rng, 257, 8192), _log(rng, 256, 8192), _log(rng, 64, 8192)
    elif use == "s16":
        op, pitch = "s16", "padded"         # this entry point takes aligned rows only
        M, N, K = _log(rng, 1, 4096), _log(rng, 64, 4096), _log(rng, 64, 4096)
    else:
        op = "unpacked"
        M, N, K = _log(rng, 1, 2048), _log(rng, 64, 4096), _log(rng, 64, 4096)
    while M * N * K > (1 << 37):            # below the largest listed case whatever the route costs
        N, K = max(64, N // 2), max(64, K // 2)
    za = rng.choice((0, 37, 128, 128)) if op != "s8s8" else rng.choice((0, 0, -5))
    zb = rng.choice((0, 0, 3, -3)) if op not in ("u8u8", "s16") else 128 + rng.choice((0, 3, -7)) if op == "u8u8" else rng.choice((0, -21))
    more = {"columns": 1} if op == "channel" and rng.random() < 0.25 else {}   # a zero-point of its own per column
    return _gemm(None, use, op, M, N, K, za=za, zb=zb, pitch=pitch, **more)


# ---- inputs ------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _rows(gen, rows, K, pitch, dtype, values, element_align):
    """`rows` rows of K values; the buffer's rows are as long as K or padded to 16 bytes."""
    ld = K if pitch == "tight" else -(-K // element_align) * element_align
    info = torch.iinfo(dtype)
    if values == "uniform":
        return torch.randint(info.min, info.max + 1, (rows, ld), generator=gen, device="cuda", dtype=dtype), ld
    # quantised activations and weights: Gaussian, clipped to the type
    mean = 128.0 if dtype == torch.uint8 else 0.0
    sd = {torch.uint8: 40.0, torch.int8: 30.0, torch.int16: 5000.0}[dtype]
    x = torch.empty((rows, ld), dtype=dtype, device="cuda")
    for r in range(0, rows, 4096):
        part = torch.randn((min(4096, rows - r), ld), generator=gen, device="cuda").mul_(sd).add_(mean).round_().clamp_(info.min, info.max)
        x[r:r + 4096] = part.to(dtype)
    return x, ld


def _types(op):
    if op == "s16":
        return torch.int16, torch.int16
    return (torch.int8 if op == "s8s8" else torch.uint8), (torch.uint8 if op == "u8u8" else torch.int8)


def _operands(case, seed):
    gen = _gen(seed)
    ta, tb = _types(case["op"])
    align = 8 if case["op"] == "s16" else 16
    values = case.get("values", "layer")
    A, lda = _rows(gen, case["M"], case["K"], case["pitch"], ta, values, align)
    B, ldb = _rows(gen, case["N"], case["K"], case["pitch"], tb, values, align)
    return gen, A, lda, B, ldb


def _column_terms(gen, N, K, with_zb):
    """Scales that put the outputs of Gaussian operands over the whole range of u8, bias, zero-points."""
    scales = (torch.rand(N, generator=gen, device="cuda") * 0.5 + 0.75) * (40.0 / (40.0 * 30.0 * math.sqrt(K)))
    bias = torch.randint(-2000, 2000, (N,), generator=gen, device="cuda", dtype=torch.int32)
    zbv = torch.randint(-8, 9, (N,), generator=gen, device="cuda", dtype=torch.int32) if with_zb else None
    return scales.float(), bias, zbv


def _scale(K):
    return float(np.float32(40.0 / (40.0 * 30.0 * math.sqrt(K))))


def _ffn_layers(case, seed):
    gen = _gen(seed)
    M, D, H = case["M"], case["D"], case["H"]
    X, ldx = _rows(gen, M, D, case["pitch"], torch.uint8, "layer", 16)
    layers = []
    for N, K, relu, zc in ((H, D, 1, 0), (D, H, 0, 128)):
        W, ldw = _rows(gen, N, K, case["pitch"], torch.int8, "layer", 16)
        layers.append((N, K, W, ldw, relu, zc) + _column_terms(gen, N, K, False)[:2])
    return X, ldx, layers


def _batch(case, seed):
    gen = _gen(seed)
    out = []
    for M, N, K, za, zb in batched_shapes(case["count"], case["mmax"], case["nmax"], case["kmax"], case["shapes"]):
        A = torch.randint(0, 256, (M, K), generator=gen, device="cuda", dtype=torch.uint8)
        B = torch.randint(-128, 128, (N, K), generator=gen, device="cuda", dtype=torch.int8)
        out.append((M, N, K, za, zb, A, B))
    return out


# ---- what a program keeps: the context, packed weights, workspaces, outputs ---------------------------------

_contexts = {}


def _ctx():
    d = torch.cuda.current_device()
    if d not in _contexts:
        _contexts[d] = ng.ngemm_create(d)
    return _contexts[d]


class _Weight:
    """A packed operand: the library's descriptor and the buffer that it refers to."""

    def __init__(self, B, ldb, K, N):
        size, pack = {torch.int16: (ng.ngemm_packed_b_bytes_s16, ng.ngemm_pack_b_s16),
                      torch.uint8: (ng.ngemm_packed_b_bytes, ng.ngemm_pack_b_u8),
                      torch.int8: (ng.ngemm_packed_b_bytes, ng.ngemm_pack_b)}[B.dtype]
        n = size(K, N)
        self.buf = torch.empty(n, dtype=torch.uint8, device="cuda")
        self.handle = pack(_ctx(), K, N, B, ldb, self.buf, n)

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            ng.ngemm_packed_b_free(self.handle)


def prepare(case, seed):
    s = {"case": case, "ctx": _ctx()}
    use, op = case["use"], case["op"]
    if use == "ffn":
        X, ldx, layers = _ffn_layers(case, seed)
        s.update(X=X, ldx=ldx, layers=[], M=case["M"])
        for N, K, W, ldw, relu, zc, scales, bias in layers:
            ldc = N if case["pitch"] == "tight" else -(-N // 16) * 16
            wsb = ng.ngemm_workspace_bytes(case["M"], N, K)
            s["layers"].append({"w": _Weight(W, ldw, K, N), "N": N, "relu": relu, "zc": zc, "scales": scales, "bias": bias, "ldc": ldc,
                                "C": torch.zeros((case["M"], ldc), dtype=torch.uint8, device="cuda"),
                                "ws": torch.empty(wsb, dtype=torch.uint8, device="cuda"), "wsb": wsb})
        return s
    if use == "batched":
        items, s["C"], s["keep"] = [], [], []
        for M, N, K, za, zb, A, B in _batch(case, seed):
            w, C = _Weight(B, K, K, N), torch.empty((M, N), dtype=torch.int32, device="cuda")
            items.append((M, A, K, za, zb, w.handle, C, N))
            s["C"].append(C)
            s["keep"] += [A, w]
        s["problems"] = ng.make_problems(items)
        return s
    if use == "pack":
        dt = {"pack": torch.int8, "pack_u8": torch.uint8, "pack_s16": torch.int16}[op]
        s["B"], s["ldb"] = _rows(_gen(seed), case["N"], case["K"], case["pitch"], dt, "layer", 8 if op == "pack_s16" else 16)
        s["bytes"] = (ng.ngemm_packed_b_bytes_s16 if op == "pack_s16" else ng.ngemm_packed_b_bytes)(case["K"], case["N"])
        s["packed"] = torch.empty(s["bytes"], dtype=torch.uint8, device="cuda")
        return s
    M, N, K = case["M"], case["N"], case["K"]
    gen, A, lda, B, ldb = _operands(case, seed)
    s.update(A=A, lda=lda, C=torch.empty((M, N), dtype=torch.uint8 if op in ("u8", "channel") else torch.int32, device="cuda"))
    if op == "unpacked":
        s.update(B=B, ldb=ldb)
        s["wsb"] = ng.ngemm_unpacked_workspace_bytes(M, N, K)
    else:
        s["w"] = _Weight(B, ldb, K, N)
        s["wsb"] = ng.ngemm_workspace_bytes(M, N, K)
    if op == "channel":
        s["scales"], s["bias"], s["zbv"] = _column_terms(gen, N, K, bool(case.get("columns")))
    s["ws"] = torch.empty(s["wsb"], dtype=torch.uint8, device="cuda")
    return s


# ---- one pass ----------------------------------------------------------------------------------------------

def run(s):
    case, ctx = s["case"], s["ctx"]
    use, op = case["use"], case["op"]
    if use == "ffn":
        x, ldx, za = s["X"], s["ldx"], 128
        for q in s["layers"]:
            ng.ngemm_run_u8s8u8_requant_channel(ctx, s["M"], x, ldx, za, q["w"].handle, 0, None, q["scales"], q["bias"], q["relu"], q["zc"],
                                                q["C"], q["ldc"], q["ws"], q["wsb"])
            x, ldx, za = q["C"], q["ldc"], q["zc"]
        return [q["C"] for q in s["layers"]]
    if use == "batched":
        ng.ngemm_run_batched_u8s8s32(ctx, s["problems"])
        return s["C"]
    if use == "pack":
        pack = {"pack": ng.ngemm_pack_b, "pack_u8": ng.ngemm_pack_b_u8, "pack_s16": ng.ngemm_pack_b_s16}[op]
        ng.ngemm_packed_b_free(pack(ctx, case["K"], case["N"], s["B"], s["ldb"], s["packed"], s["bytes"]))
        return s["packed"]
    M, N, K, za, zb = case["M"], case["N"], case["K"], case["za"], case["zb"]
    A, lda, C, ws, wsb = s["A"], s["lda"], s["C"], s["ws"], s["wsb"]
    if op == "unpacked":
        ng.ngemm_run_u8s8s32_unpacked(ctx, M, N, K, A, lda, za, s["B"], s["ldb"], zb, C, N, ws, wsb)
    elif op == "u8":
        ng.ngemm_run_u8s8u8_requant(ctx, M, A, lda, za, s["w"].handle, zb, _scale(K), 128, C, N, ws, wsb)
    elif op == "channel":
        ng.ngemm_run_u8s8u8_requant_channel(ctx, M, A, lda, za, s["w"].handle, zb, s["zbv"], s["scales"], s["bias"], 0, 128, C, N, ws, wsb)
    else:
        call = {"s32": ng.ngemm_run_u8s8s32, "s8s8": ng.ngemm_run_s8s8s32, "u8u8": ng.ngemm_run_u8u8s32, "s16": ng.ngemm_run_s16s16s32}[op]
        call(ctx, M, A, lda, za, s["w"].handle, zb, C, N, ws, wsb)
    return C


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def work(case):
    use, op = case["use"], case["op"]
    if use == "ffn":
        M, D, H = case["M"], case["D"], case["H"]
        return {"bytes": 2 * M * D + 2 * M * H + 2 * D * H + 8 * (D + H), "flops": 4 * M * D * H}
    if use == "batched":
        sh = batched_shapes(case["count"], case["mmax"], case["nmax"], case["kmax"], case["shapes"])
        return {"bytes": sum(M * K + N * K + 4 * M * N for M, N, K, _, _ in sh), "flops": sum(2 * M * N * K for M, N, K, _, _ in sh)}
    size = 2 if op in ("s16", "pack_s16") else 1
    if use == "pack":
        return {"bytes": 2 * size * case["N"] * case["K"] + 4 * case["N"], "flops": 0}
    M, N, K = case["M"], case["N"], case["K"]
    out = (1 if op in ("u8", "channel") else 4) * M * N
    return {"bytes": size * (M * K + N * K) + out + (8 * N if op == "channel" else 0), "flops": 2 * M * N * K}


def tolerance(case):
    return "exact"


# ---- the same from plain torch in 64 bits --------------------------------------------------------------------

def _sums(A, za, B, zb):
    """sum_k (A[i][k] - za) (B[j][k] - zb), row blocks at a time: float64 is exact far beyond these sums."""
    Bd = (B.to(torch.float64) - zb).t().contiguous()
    rows = [(A[r:r + 1024].to(torch.float64) - za) @ Bd for r in range(0, A.shape[0], 1024)]
    return torch.cat(rows).to(torch.int64)


def _wrap32(v):
    return ((v + (1 << 31)) % (1 << 32)) - (1 << 31)


def _requant(c, scales, zc, relu):
    """Whole sums to u8 as the header states it: binary32 conversion, one binary32 product, ties to even."""
    q = torch.round(_wrap32(c).to(torch.float32) * scales).to(torch.float64) + zc
    return (q.clamp_min(float(zc)) if relu else q).clamp(0.0, 255.0).to(torch.uint8)


def _packed(B, K, N, shift):
    """The documented layout: 32 columns x 32 bytes of depth per fragment, 16 bytes per lane, then the column sums."""
    Np = -(-N // 32) * 32
    if B.dtype == torch.int16:
        # two byte planes per 32 elements: the signed high byte of b - 128, then its low byte shifted to signed
        Kp = -(-K // 32) * 32
        b = torch.zeros((Np, Kp), dtype=torch.int64, device=B.device)
        b[:N, :K] = B[:, :K].to(torch.int64) - 128
        hi, lo = (b + 128) >> 8, ((b + 128) & 255) - 128
        hi[N:], lo[N:], hi[:, K:], lo[:, K:] = 0, 0, 0, 0
        planes = torch.stack([hi.view(Np, Kp // 32, 32), lo.view(Np, Kp // 32, 32)], dim=2).reshape(Np, 2 * Kp)
        sums, b8, Kp = b.sum(dim=1), planes, 2 * Kp
    else:
        Kp = -(-K // 64) * 64
        b8 = torch.zeros((Np, Kp), dtype=torch.int64, device=B.device)
        b8[:N, :K] = B[:, :K].to(torch.int64) - shift
        sums = b8.sum(dim=1)
    frag = b8.to(torch.int8).view(Np // 32, 32, Kp // 32, 2, 16).permute(0, 2, 3, 1, 4).contiguous().view(torch.uint8).reshape(-1)
    return torch.cat([frag, sums.to(torch.int32).view(torch.uint8).reshape(-1)])


def exact(case, seed):
    use, op = case["use"], case["op"]
    if use == "ffn":
        x, _, layers = _ffn_layers(case, seed)
        out, za = [], 128
        for N, K, W, _, relu, zc, scales, bias in layers:
            q = _requant(_sums(x[:, :K], za, W[:, :K], 0) + bias, scales, zc, relu)
            ldc = N if case["pitch"] == "tight" else -(-N // 16) * 16
            C = torch.zeros((case["M"], ldc), dtype=torch.uint8, device=q.device)
            C[:, :N] = q
            out.append(C)
            x, za = q, zc
        return out
    if use == "batched":
        return [_sums(A, za, B, zb).to(torch.int32) for _, _, _, za, zb, A, B in _batch(case, seed)]
    if use == "pack":
        dt = {"pack": torch.int8, "pack_u8": torch.uint8, "pack_s16": torch.int16}[op]
        B, _ = _rows(_gen(seed), case["N"], case["K"], case["pitch"], dt, "layer", 8 if op == "pack_s16" else 16)
        return _packed(B, case["K"], case["N"], 128 if op == "pack_u8" else 0)
    K = case["K"]
    gen, A, _, B, _ = _operands(case, seed)
    if op == "channel":
        scales, bias, zbv = _column_terms(gen, case["N"], K, bool(case.get("columns")))
        zb = case["zb"] if zbv is None else zbv.to(torch.float64)[:, None]
        return _requant(_sums(A[:, :K], case["za"], B[:, :K], zb) + bias, scales, 128, 0)
    c = _sums(A[:, :K], case["za"], B[:, :K], case["zb"])
    if op == "u8":
        return _requant(c, torch.tensor(_scale(K), dtype=torch.float32, device=c.device), 128, 0)
    return _wrap32(c).to(torch.int32)
