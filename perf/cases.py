"""The work that programs built on libabft have it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``prepare`` makes what a program holds before the calls (operands,
output and verdict buffers, a context, the weight checksum where the program encodes its weights
once), ``run`` makes one pass through the C ABI as the binding exposes it, on the current stream.

Kinds
  linear     one Linear layer, C = A W^T (+ bias), protected or plain
  attention  the per-head products Q K^T ("qk") or attn V ("av") of a batch of heads
  block      the six GEMM classes of a transformer block, one call after the other
  repair     a bit of a stored output flips; verify, then correct

Shapes are those of ViT-B/16 (197 tokens, hidden 768, 12 heads, MLP 3072) and ViT-L/16 at 384^2 (577
tokens, hidden 1024, 16 heads, MLP 4096), value distributions those of abft_inputs.py: uniform int8;
activations N(0, 1), weights N(0, 0.02), softmax rows for attention probabilities.
"""
from __future__ import annotations

import math
import weakref

import torch

import paper_2310_03841_amd as ab

TORCH_TYPE = {"i8": torch.int8, "bf16": torch.bfloat16, "f16": torch.float16}
ES = {"i8": 1, "bf16": 2, "f16": 2}
OS = {"i8": 4, "bf16": 2, "f16": 2}
MAX_K = 4096                       # deepest K of a protected GEMM


# ---------------------------------------------------------------------------------- the cases
def _linear(name, dtype, M, N, K, trans_b=True, mode="detect", cached=False, bias=False, stored=False):
    c = dict(kind="linear", dtype=dtype, M=M, N=N, K=K, trans_b=trans_b, mode=mode, cached=cached, bias=bias,
             stored=stored)
    return dict(c, name=name) if name else c


def _attention(name, dtype, product, tokens, head_dim, items):
    c = dict(kind="attention", dtype=dtype, product=product, tokens=tokens, head_dim=head_dim, items=items)
    return dict(c, name=name) if name else c


def _block(name, dtype, tokens, heads, images, cached):
    c = dict(kind="block", dtype=dtype, tokens=tokens, heads=heads, images=images, cached=cached)
    return dict(c, name=name) if name else c


def _repair(name, dtype, M, N, K):
    c = dict(kind="repair", dtype=dtype, M=M, N=N, K=K)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a single image through an attention projection, weights not encoded: bound by latency
        _linear("proj_i8_1image", "i8", 197, 768, 768),
        # the wide layer of an MLP for a single image in a server: bias, weight checksum kept
        _linear("fc1_bf16_1image_bias", "bf16", 197, 3072, 768, cached=True, bias=True),
        # the same layer for a large batch, nothing cached: the benchmark workload
        _linear("fc1_bf16_b64", "bf16", 12608, 3072, 768),
        # the narrow, deep layer of an MLP at an ordinary batch, weight checksum kept
        _linear("fc2_f16_b32_cached", "f16", 6304, 768, 3072, cached=True),
        # odd sizes in every dimension, right operand stored K x N (a product of two activations)
        _linear("odd_bf16_kn", "bf16", 1537, 1001, 713, trans_b=False),
        # a layer left unprotected (selective protection runs such layers beside protected ones)
        _linear("proj_bf16_b32_plain", "bf16", 6304, 768, 768, mode="off"),
        # the output is checked again after it has lain in memory: stored-side sums, then verify
        _linear("fc1_bf16_b32_stored_verify", "bf16", 6304, 3072, 768, bias=True, stored=True),
        # a flipped bit in the stored output of a layer: found, located, repaired
        _repair("repair_fc2_i8_b32", "i8", 6304, 768, 3072),
        # attention products of a batch of 32 images
        _attention("qk_bf16_b32", "bf16", "qk", 197, 64, 384),
        _attention("av_bf16_b32", "bf16", "av", 197, 64, 384),
        # a whole transformer block for one image
        _block("block_bf16_1image", "bf16", 197, 12, 1, True),
        # a whole block of the larger model for a large batch, quantised
        _block("block_i8_large_b64", "i8", 577, 16, 64, True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size of [lo, hi], spread over its logarithm; half of the time a multiple of 64 as layers have."""
    n = _log(rng, lo, hi)
    if hi >= 64 and rng.random() < 0.5:
        n = max(64, (n + 32) // 64 * 64)
    return min(max(n, lo), hi)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "attention", "attention", "block", "repair"])
    dtype = rng.choice(["i8", "bf16", "f16"])
    if kind == "linear":
        M, N, K = _size(rng, 16, 12608), _size(rng, 64, 4096), _size(rng, 64, MAX_K)
        mode = rng.choice(["detect", "detect", "detect", "correct", "off"])
        # the re-sum of a rounded output only makes sense where its rounding stays below the tolerance
        stored = (dtype != "i8" and mode == "detect" and rng.random() < 0.3 and N <= 4 * K and M <= 8 * K)
        return _linear(None, dtype, M, N, K, trans_b=rng.random() < 0.8, mode=mode,
                       cached=mode != "off" and rng.random() < 0.5, bias=rng.random() < 0.4, stored=stored)
    if kind == "attention":
        tokens, hd = rng.randint(50, 577), rng.choice([32, 48, 64, 64, 80, 128])
        items = _log(rng, 3, 1024)
        items = max(3, min(items, int(4e8 / (tokens * tokens + tokens * hd))))
        return _attention(None, dtype, rng.choice(["qk", "av"]), tokens, hd, items)
    if kind == "block":
        tokens, heads = rng.randint(50, 577), rng.randint(3, 16)
        images = _log(rng, 1, 64)
        return _block(None, dtype, tokens, heads, images, rng.random() < 0.5)
    return _repair(None, dtype, _size(rng, 64, 12608), _size(rng, 64, 4096), _size(rng, 64, MAX_K))


# ---------------------------------------------------------------------------------- one GEMM
def _pad(n, elem_bytes):
    q = 16 // elem_bytes
    return (n + q - 1) // q * q


def _values(gen, kind, dtype, *shape):
    """Operand values on the GPU; the last dimension is padded to whole 16 bytes."""
    ld = _pad(shape[-1], ES[dtype])
    full = shape[:-1] + (ld,)
    if dtype == "i8":
        return torch.randint(-128, 128, full, generator=gen, device="cuda", dtype=torch.int8)
    x = torch.empty(full, device="cuda", dtype=torch.float32).normal_(0.0, 0.02 if kind == "weight" else 1.0,
                                                                      generator=gen)
    if kind == "softmax":
        x[..., shape[-1]:] = -math.inf
        x = torch.softmax(x, dim=-1)
    return x.to(TORCH_TYPE[dtype])


def _check(rc, where):
    if rc != ab.ABFT_OK:
        raise ab.AbftError(rc, where)


class _Gemm:
    """One layer of a program: its operands, its context, its output and verdict buffers."""

    def __init__(self, gen, dtype, M, N, K, batch=1, trans_b=True, mode="detect", cached=False, bias=False,
                 stored=False, a_kind="act", b_kind="weight"):
        self.code = ab.DTYPE_CODE[dtype]
        self.A = _values(gen, a_kind, dtype, batch, M, K)
        self.B = _values(gen, b_kind, dtype, batch, *((N, K) if trans_b else (K, N)))
        self.bias = None
        if bias and dtype == "i8":
            self.bias = torch.randint(-1000, 1001, (N,), generator=gen, device="cuda", dtype=torch.int32)
        elif bias:
            self.bias = torch.empty(N, device="cuda", dtype=torch.float32).normal_(0.0, 0.1, generator=gen)
        ldc = _pad(N, OS[dtype])
        # zeros, so that the pad beyond N, which the library never writes, is the same everywhere
        self.C = torch.zeros((batch, M, ldc), device="cuda",
                             dtype=torch.int32 if dtype == "i8" else TORCH_TYPE[dtype])
        self.row_flag = torch.zeros(batch * M, device="cuda", dtype=torch.uint8)
        self.col_flag = torch.zeros(batch * N, device="cuda", dtype=torch.uint8)
        self.counts = torch.zeros(8, device="cuda", dtype=torch.int32)
        self.shape = ab.make_shape(M, N, K, batch=batch, lda=self.A.shape[-1], ldb=self.B.shape[-1], ldc=ldc,
                                   transB=trans_b)
        self.result = ab.make_result(self.row_flag, self.col_flag, self.counts)
        self.ctx = ab.abft_create(batch * M, batch * N, batch * ((K + 127) // 128 * 128), batch)
        weakref.finalize(self, ab.abft_destroy, self.ctx)
        self.plain = mode == "off"
        self.mode = {"off": ab.ABFT_OFF, "detect": ab.ABFT_DETECT, "correct": ab.ABFT_DETECT_CORRECT}[mode]
        if cached:
            # what the binding documents as the offline weight checksum: once per weight
            _check(ab.abft_encode_b(self.ctx, self.B, self.code, self.shape), "abft_encode_b")
            self.mode |= ab.ABFT_B_CHECKSUM_CACHED
        if stored:
            self.mode |= ab.ABFT_STORED_SUMS
        self.stored = stored

    def __call__(self):
        r = None if self.plain else self.result
        if self.bias is not None:
            _check(ab.abft_gemm_bias(self.ctx, self.A, self.B, self.bias, self.C, self.code, self.mode, self.shape, r),
                   "abft_gemm_bias")
        else:
            _check(ab.abft_gemm(self.ctx, self.A, self.B, self.C, self.code, self.mode, self.shape, r), "abft_gemm")
        if self.stored:
            self.verify()
        return self.out()

    def verify(self):
        _check(ab.abft_verify(self.ctx, self.C, self.code, self.shape, self.result), "abft_verify")

    def out(self):
        return (self.C,) if self.plain else (self.C, self.row_flag, self.col_flag, self.counts)


def _block_layers(c):
    """(M, N, K, batch, trans_b, cached, a_kind, b_kind) of the six GEMM classes of a block."""
    heads, tokens, hidden = c["heads"], c["tokens"], 64 * c["heads"]
    rows, items, mlp = c["images"] * tokens, c["images"] * heads, 4 * hidden
    cached = c["cached"]
    return [
        (rows, 3 * hidden, hidden, 1, True, cached, "act", "weight"),
        (tokens, tokens, 64, items, True, False, "act", "act"),
        (tokens, 64, tokens, items, False, False, "softmax", "act"),
        (rows, hidden, hidden, 1, True, cached, "act", "weight"),
        (rows, mlp, hidden, 1, True, cached, "act", "weight"),
        (rows, hidden, mlp, 1, True, cached, "act", "weight"),
    ]


def _attention_shape(c):
    """(M, N, K, trans_b) of an attention product."""
    t, hd = c["tokens"], c["head_dim"]
    return (t, t, hd, True) if c["product"] == "qk" else (t, hd, t, False)


# ---------------------------------------------------------------------------------- the interface
class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if c["kind"] == "linear":
        s.run = _Gemm(gen, c["dtype"], c["M"], c["N"], c["K"], trans_b=c["trans_b"], mode=c["mode"],
                      cached=c["cached"], bias=c["bias"], stored=c["stored"])
    elif c["kind"] == "attention":
        M, N, K, trans_b = _attention_shape(c)
        s.run = _Gemm(gen, c["dtype"], M, N, K, batch=c["items"], trans_b=trans_b,
                      a_kind="softmax" if c["product"] == "av" else "act", b_kind="act")
    elif c["kind"] == "block":
        layers = [_Gemm(gen, c["dtype"], M, N, K, batch=batch, trans_b=trans_b, cached=cached, a_kind=ak, b_kind=bk)
                  for M, N, K, batch, trans_b, cached, ak, bk in _block_layers(c)]
        s.run = lambda: [layer() for layer in layers]
    elif c["kind"] == "repair":
        gemm = _Gemm(gen, c["dtype"], c["M"], c["N"], c["K"])
        gemm()                                         # the output that lies in memory when the bit flips
        row, col, bit = (int(torch.randint(0, n, (1,), generator=gen, device="cuda")) for n in (c["M"], c["N"], 32))
        if c["dtype"] != "i8":
            bit = 14                                   # the top exponent bit: far above any tolerance

        def repair():
            _check(ab.abft_inject(gemm.ctx, gemm.C, gemm.code, gemm.shape, 0, row, col, bit), "abft_inject")
            gemm.verify()
            _check(ab.abft_correct(gemm.ctx, gemm.A, gemm.B, gemm.C, gemm.code, gemm.shape, gemm.result),
                   "abft_correct")
            return gemm.out()
        s.run = repair
    else:
        raise ValueError(c["kind"])
    return s


def run(state):
    return state.run()


def _gemm_work(dtype, M, N, K, batch, bias=False, protected=True):
    nbytes = batch * ((M * K + N * K) * ES[dtype] + M * N * OS[dtype]) + (4 * N if bias else 0)
    return nbytes + (batch * (M + N) + 32 if protected else 0), 2.0 * M * N * K * batch


def work(case):
    c = case
    if c["kind"] == "linear":
        b, f = _gemm_work(c["dtype"], c["M"], c["N"], c["K"], 1, c["bias"], c["mode"] != "off")
        if c["stored"]:                                # the stored output is read back once, flags written again
            b += c["M"] * c["N"] * OS[c["dtype"]] + c["M"] + c["N"]
    elif c["kind"] == "attention":
        M, N, K, _ = _attention_shape(c)
        b, f = _gemm_work(c["dtype"], M, N, K, c["items"])
    elif c["kind"] == "block":
        parts = [_gemm_work(c["dtype"], M, N, K, batch) for M, N, K, batch, *_ in _block_layers(c)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    else:
        # one read of the stored output, the flags, and one 32 x 32 tile from its operand rows
        b = c["M"] * c["N"] * OS[c["dtype"]] + c["M"] + c["N"] + 64 * c["K"] * ES[c["dtype"]]
        f = 2.0 * 32 * 32 * c["K"]
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """int8: C, flags and counts are whole numbers of exact arithmetic.  Floating point: C is one
    rounding of an fp32 sum, so two correct implementations differ by one unit in the last place
    where their sums fall on two sides of a rounding boundary."""
    if case["dtype"] == "i8":
        return "exact"
    return TOLERANCE[case["dtype"]]


# Measured against the product summed in 64 bits and rounded once to the output type, over the listed
# shapes and three more: bf16 rel <= 3.9e-5, max <= 7.8e-3 (one unit in the last place); f16 rel <=
# 1.4e-5, max <= 9.8e-4.  Four times that, and for rel in the smallest outputs drawn (1024 values)
# room for four such roundings.
TOLERANCE = {"bf16": {"rel": 5e-4, "max": 3.2e-2}, "f16": {"rel": 6e-5, "max": 4e-3}}
