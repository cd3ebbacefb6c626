"""The work that a program which serves or prepares block-pruned BERT weights has libbsr do.

Every case is a dict of plain values; `prepare` makes what such a program holds before the call
(weights pruned on the GPU, activations, the prepared call with its plan), `run` is one pass
through the library's public entry points, `exact` the same result in fp64 by plain torch.

Kinds of case:
  products   one or several BSR products Y = X W^T + b, issued as a serving loop issues them (one
             prepared call, with per-matrix plans where the block shape has them), or as a script
             does (bsr_spmm on tensors).
  attention  scaled dot-product attention of a batch of sequences.
  block      the BERT attention block on pruned weights: Q, K, V products, attention, O product.
  prune      a dense weight pruned to its k best blocks.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2106_08846_amd import bsr

DEVICE = "cuda:0"
W_SIGMA = 0.02      # BERT's initialiser scale, for weights and biases
SKEW_SIGMA = 0.5    # spread of ln(block-row scale) of a skewed weight

# Matrix-core block shapes, vector-ALU block shapes (the shapes of the paper's sweep and the
# library's other kernels).
SHAPES_MFMA = [(32, 1), (16, 1), (16, 16), (32, 32)]
SHAPES_VALU = [(1, 1), (8, 1), (1, 32), (4, 4), (8, 8), (1, 8), (4, 1), (2, 2)]

# The most floating-point work and memory traffic of one pass (the eight products of two
# BERT-large layers at 6144 tokens).
MAX_FLOPS = 10.4e9
MAX_BYTES = 4.2e8


def _products(name, layers, R, C, density, T, dtype="f32", call="prepared", plan=True,
              arith="native", skew=False):
    """`layers`: "NxK*count+..." -- the count products of one term share their X."""
    c = {"kind": "products", "layers": layers, "R": R, "C": C, "density": density, "T": T,
         "dtype": dtype, "call": call, "plan": plan, "arith": arith, "skew": skew}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one 768x768 projection of a 128-token request, straight from a
        # script (arguments checked and marshalled on every call).
        _products("linear_768_4x4_T128", "768x768*1", 4, 4, 0.1, 128, call="plain"),
        # A whole attention block for one 128-token request (three launches in a row): the
        # latency of a single-request server.
        {"kind": "block", "R": 32, "C": 1, "density": 0.1, "hidden": 768, "batch": 1, "seq": 128,
         "name": "block_base_32x1_1x128"},
        # Fused QKV of a batch of 8 x 512 tokens at the sparsest and the densest of the
        # densities in use; fp32 and bf16.
        _products("qkv_32x1_d5_T4096", "2304x768*1", 32, 1, 0.05, 4096),
        _products("qkv_32x1_d40_bf16_T4096", "2304x768*1", 32, 1, 0.4, 4096, dtype="bf16"),
        # BERT-large attention projections of a batch of 16 x 384 tokens, skewed block-rows: two
        # layers' Q, K, V, O in one call (the largest work), and one layer in square blocks.
        _products("large_32x1_skew_T6144", "1024x1024*4+1024x1024*4", 32, 1, 0.1, 6144,
                  skew=True),
        _products("large_32x32_skew_T6144", "1024x1024*4", 32, 32, 0.1, 6144, skew=True),
        # The two feed-forward layers of BERT-base at 4096 tokens, in the small blocks that keep
        # more of a model's accuracy, and a ragged bf16 batch.
        _products("ffn_8x8_T4096", "3072x768*1+768x3072*1", 8, 8, 0.1, 4096),
        _products("ffn_1x32_T4096", "3072x768*1+768x3072*1", 1, 32, 0.1, 4096),
        _products("ffn_4x4_bf16_T777", "3072x768*1+768x3072*1", 4, 4, 0.2, 777, dtype="bf16"),
        # Attention of BERT-large between the projections, 16 sequences of 384 tokens.
        {"kind": "attention", "heads": 16, "batch": 16, "seq": 384, "name": "attention_16x384"},
        # Pruning: one BERT-large projection in the headline shape, and a feed-forward weight
        # element by element (unstructured).
        {"kind": "prune", "N": 1024, "K": 1024, "R": 32, "C": 1, "density": 0.1, "norm": "l2",
         "per_row": False, "name": "prune_1024_32x1"},
        {"kind": "prune", "N": 3072, "K": 768, "R": 1, "C": 1, "density": 0.1, "norm": "l2",
         "per_row": False, "name": "prune_3072x768_1x1"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, step):
    """A layer width that `step` divides: one of BERT's, or any up to 3072."""
    if rng.random() < 0.6:
        w = rng.choice([768, 1024, 2304, 3072])
        if w % step == 0:
            return w
    return step * max(1, _log_int(rng, 64, 3072) // step)


def draw(rng: random.Random):
    u = rng.random()
    if u < 0.12:
        return {"kind": "attention", "heads": rng.choice([8, 12, 16]),
                "batch": _log_int(rng, 1, 16), "seq": _log_int(rng, 24, 512)}
    if u < 0.22:
        R, C = rng.choice(SHAPES_MFMA + [(4, 4), (8, 8), (1, 32)])
        return {"kind": "block", "R": R, "C": C, "density": round(rng.uniform(0.05, 0.3), 3),
                "hidden": 768, "batch": _log_int(rng, 1, 8), "seq": _log_int(rng, 32, 512)}
    if u < 0.36:
        R, C = rng.choice(SHAPES_MFMA + SHAPES_VALU)
        return {"kind": "prune", "N": min(_width(rng, R), 3072 // R * R),
                "K": min(_width(rng, C), 768 // C * C), "R": R, "C": C,
                "density": round(rng.uniform(0.05, 0.4), 3), "norm": rng.choice(["l2", "l2", "l1"]),
                "per_row": rng.random() < 0.25}
    R, C = rng.choice([(32, 1)] * 3 + SHAPES_MFMA + SHAPES_VALU)
    dtype = "bf16" if rng.random() < 0.35 and R * C > 1 else "f32"
    N, K = _width(rng, R), _width(rng, C)
    if dtype == "bf16" and K % 2:
        K += C          # bf16 rows of an even length, as every model has
    n = rng.choice([1, 1, 1, 2, 3, 4, 8])
    layers = f"{N}x{K}*{n}" if rng.random() < 0.7 or n % 2 else f"{N}x{K}*{n // 2}+{N}x{K}*{n // 2}"
    plan = rng.random() < 0.8
    split = dtype == "f32" and plan and (R, C) == (32, 1) and rng.random() < 0.25
    c = _products(None, layers, R, C, round(rng.uniform(0.05, 0.4), 3), _log_int(rng, 1, 6144),
                  dtype=dtype, call="plain" if rng.random() < 0.2 else "prepared", plan=plan,
                  arith="split" if split else "native", skew=rng.random() < 0.4)
    w = work(c)
    over = max(w["flops"] / MAX_FLOPS, w["bytes"] / MAX_BYTES)
    if (R, C) in SHAPES_VALU:
        over *= 2       # these shapes' ceiling is the vector ALUs', half the matrix cores'
    if over > 1.0:
        c["T"] = max(1, int(c["T"] / over) - 1)
    return c


# ------------------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(1_000_003 * int(seed) + 12345)


def _normal(g, shape, sigma):
    return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32) * sigma


def _weight(g, N, K, R, skew):
    W = _normal(g, (N, K), W_SIGMA)
    if skew:   # block-rows of very different magnitude keep very different numbers of blocks
        s = torch.exp(_normal(g, (N // R,), SKEW_SIGMA))
        W = (W.view(N // R, R * K) * s[:, None]).view(N, K).contiguous()
    return W


def _terms(case):
    """[(N, K, count)] of a products case."""
    out = []
    for t in case["layers"].split("+"):
        shape, count = t.split("*")
        N, K = shape.split("x")
        out.append((int(N), int(K), int(count)))
    return out


def _product_inputs(case, seed):
    """[(X, [(W dense, bias), ...]), ...], fp32."""
    g = _gen(seed)
    out = []
    for N, K, count in _terms(case):
        X = _normal(g, (case["T"], K), 1.0)
        out.append((X, [(_weight(g, N, K, case["R"], case["skew"]), _normal(g, (N,), W_SIGMA))
                        for _ in range(count)]))
    return out


def _qkv_inputs(case, seed):
    g = _gen(seed)
    T, H = case["batch"] * case["seq"], case["heads"] * 64
    return [_normal(g, (T, H), 1.0) for _ in range(3)]


def _block_inputs(case, seed):
    g = _gen(seed)
    H, T = case["hidden"], case["batch"] * case["seq"]
    return (_normal(g, (T, H), 1.0),
            [(_normal(g, (H, H), W_SIGMA), _normal(g, (H,), W_SIGMA)) for _ in range(4)])


def _keep(N, K, R, C, density, per_row=False):
    """Blocks kept at a density: floor(density * blocks + 1/2), per block-row when per_row."""
    Nb, Kb = N // R, K // C
    if per_row:
        return Nb * min(Kb, int(math.floor(density * Kb + 0.5)))
    return min(Nb * Kb, int(math.floor(density * Nb * Kb + 0.5)))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "prune":
        W = _weight(_gen(seed), case["N"], case["K"], case["R"], False)
        return {"case": case, "W": W}
    if kind == "attention":
        q, k, v = _qkv_inputs(case, seed)
        return {"case": case, "q": q, "k": k, "v": v, "o": torch.empty_like(q)}
    if kind == "block":
        X, ws = _block_inputs(case, seed)
        args = []
        for W, b in ws:
            args += [bsr.bsr_prune_from_dense(W, case["R"], case["C"], density=case["density"]), b]
        call = bsr.AttentionBlockCall(X, *args, case["batch"], case["seq"], case["hidden"] // 64)
        return {"case": case, "call": call}
    products, plans = [], []
    for X, ws in _product_inputs(case, seed):
        Xd = bsr.bsr_cast_f32_bf16(X) if case["dtype"] == "bf16" else X
        for W, b in ws:
            M = bsr.bsr_prune_from_dense(W, case["R"], case["C"], density=case["density"])
            if case["dtype"] == "bf16":
                M = M.to_bf16()
            planned = case["plan"] and (case["R"], case["C"]) == (32, 1) and case["call"] != "plain"
            arith = bsr.ARITH_BF16X3 if case["arith"] == "split" else bsr.ARITH_AUTO
            plans.append(bsr.bsr_plan_prepare(M, arith=arith) if planned else None)
            Y = torch.empty((case["T"], M.n_rows), dtype=torch.float32, device=DEVICE)
            products.append((Xd, M, b, Y))
    if case["call"] == "plain":
        return {"case": case, "products": products}
    return {"case": case, "call": bsr.SpmmBatchCall(
        products, plans=plans if any(p is not None for p in plans) else None)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "products":
        if case["call"] == "plain":
            return [bsr.bsr_spmm(X, M, b) for X, M, b, _ in state["products"]]
        return state["call"]()
    if kind == "block":
        return state["call"]()
    if kind == "attention":
        return bsr.bsr_attention(state["q"], state["k"], state["v"], case["batch"], case["seq"],
                                 case["heads"], O=state["o"])
    M = bsr.bsr_prune_from_dense(state["W"], case["R"], case["C"], density=case["density"],
                                 norm=case["norm"], per_row=case["per_row"])
    return [M.indptr, M.indices[:M.nnzb], M.data[:M.nnzb]]


# --------------------------------------------------------------------------------- accounting

def _product_work(N, K, R, C, density, T, bf16=False):
    k, xs = _keep(N, K, R, C, density), 2 if bf16 else 4
    flops = 2.0 * k * R * C * T
    w_bytes = k * R * C * xs + 4 * k + 4 * (N // R + 1) + 4 * N
    return flops, w_bytes, T * K * xs, 4.0 * T * N


def work(case):
    kind = case["kind"]
    if kind == "prune":
        N, K, R, C = case["N"], case["K"], case["R"], case["C"]
        k = _keep(N, K, R, C, case["density"], case["per_row"])
        return {"bytes": 4.0 * N * K + 4.0 * k * R * C + 4.0 * k + 4.0 * (N // R + 1),
                "flops": 2.0 * N * K}
    if kind == "attention":
        T, H = case["batch"] * case["seq"], case["heads"] * 64
        return {"bytes": 16.0 * T * H, "flops": 4.0 * T * case["seq"] * H}
    if kind == "block":
        H, T = case["hidden"], case["batch"] * case["seq"]
        f, wb, xb, yb = _product_work(H, H, case["R"], case["C"], case["density"], T)
        # X in, Y out, and the three projections and the context once each way between stages.
        return {"bytes": 4 * wb + 10.0 * 4 * T * H, "flops": 4 * f + 4.0 * T * case["seq"] * H}
    flops = bts = 0.0
    for N, K, count in _terms(case):
        f, wb, xb, yb = _product_work(N, K, case["R"], case["C"], case["density"], case["T"],
                                      case["dtype"] == "bf16")
        flops += count * f
        bts += xb + count * (wb + yb)
    return {"bytes": bts, "flops": flops}


def tolerance(case):
    """Everything is accumulated and returned in fp32 (bf16 cases round their inputs, which both
    sides share, and multiply exactly), so another summation order shows a few 1e-7; the pruning
    is a selection and a copy."""
    if case["kind"] == "prune":
        return "exact"
    if case["kind"] == "block":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 2e-6, "max": 5e-5}


# -------------------------------------------------------------------------- the fp64 reference

def _prune_exact(W, R, C, k, norm="l2", per_row=False):
    """indptr, indices, data of the k best blocks (key descending, block id ascending)."""
    N, K = W.shape
    Nb, Kb = N // R, K // C
    blocks = W.view(Nb, R, Kb, C).permute(0, 2, 1, 3).reshape(Nb * Kb, R * C)
    x = blocks.double()
    keys = (x * x).sum(1) if norm == "l2" else x.abs().sum(1)
    if per_row:
        ids = torch.sort(keys.view(Nb, Kb), dim=1, descending=True, stable=True).indices
        kept = ids[:, : k // Nb] + torch.arange(Nb, device=W.device)[:, None] * Kb
        kept = kept.reshape(-1)
    else:
        kept = torch.sort(keys, descending=True, stable=True).indices[:k]
    kept = torch.sort(kept).values
    counts = torch.bincount(kept // Kb, minlength=Nb)
    indptr = torch.zeros(Nb + 1, dtype=torch.int32, device=W.device)
    indptr[1:] = torch.cumsum(counts, 0).to(torch.int32)
    return indptr, (kept % Kb).to(torch.int32), blocks[kept].view(-1, R, C), kept


def _masked(W, R, C, density):
    """W with only its kept blocks."""
    N, K = W.shape
    kept = _prune_exact(W, R, C, _keep(N, K, R, C, density))[3]
    mask = torch.zeros((N // R) * (K // C), dtype=W.dtype, device=W.device)
    mask[kept] = 1.0
    mask = mask.view(N // R, 1, K // C, 1).expand(-1, R, -1, C).reshape(N, K)
    return W * mask


def _attention_exact(q, k, v, batch, seq, heads):
    def split(x):
        return x.view(batch, seq, heads, 64).permute(0, 2, 1, 3).reshape(-1, seq, 64)
    q, k, v = split(q), split(k), split(v)
    out = torch.empty_like(q)
    for i in range(q.shape[0]):
        out[i] = torch.softmax((q[i] @ k[i].t().contiguous()) * 0.125, dim=1) @ v[i]
    return out.view(batch, heads, seq, 64).permute(0, 2, 1, 3).reshape(batch * seq, heads * 64)


def exact(case, seed):
    kind = case["kind"]
    if kind == "prune":
        W = _weight(_gen(seed), case["N"], case["K"], case["R"], False)
        k = _keep(case["N"], case["K"], case["R"], case["C"], case["density"], case["per_row"])
        return list(_prune_exact(W, case["R"], case["C"], k, case["norm"], case["per_row"])[:3])
    if kind == "attention":
        q, k, v = (t.double() for t in _qkv_inputs(case, seed))
        return _attention_exact(q, k, v, case["batch"], case["seq"], case["heads"])
    if kind == "block":
        X, ws = _block_inputs(case, seed)
        d = [_masked(W, case["R"], case["C"], case["density"]).double() for W, _ in ws]
        b = [bias.double() for _, bias in ws]
        q, k, v = (X.double() @ d[i].t().contiguous() + b[i] for i in range(3))
        ctx = _attention_exact(q, k, v, case["batch"], case["seq"], case["hidden"] // 64)
        return ctx @ d[3].t().contiguous() + b[3]
    out = []
    for X, ws in _product_inputs(case, seed):
        if case["dtype"] == "bf16":
            X = X.bfloat16()
        for W, b in ws:
            M = _masked(W, case["R"], case["C"], case["density"])
            if case["dtype"] == "bf16":
                M = M.bfloat16()
            out.append(X.double() @ M.double().t().contiguous() + b.double())
    return out
