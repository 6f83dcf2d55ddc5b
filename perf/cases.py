"""The work this library is measured by: its four operations through the ctypes binding, as a program calls them.

A program creates a `tf.Problem` per shape and keeps it, together with the variant it runs. The variant here is the
library's static pick (`tf.proposal` with nothing tried but the baseline: the first proposal of the variant loop),
which needs no measurement and is the same every time; then `Problem.run` is called once per product.

    listed()            the cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, the problem handle, the chosen variant, the output buffer
    run(state)          one call; returns the output
    work(case)          bytes and operations the call cannot do without
    tolerance(case)     what another correct implementation of the same precision may differ by
"""
import math

import torch

from paper_2512_09196_amd import tf

_EPI = {"gelu_erf": tf.TF_EPI_BIAS_GELU_ERF, "gelu_tanh": tf.TF_EPI_BIAS_GELU_TANH, "bias": tf.TF_EPI_BIAS,
        "fp32": tf.TF_EPI_NONE_F32}


def _gemm(name, M, N, K, epi="gelu_erf", b_as_nk=False, dist="normal"):
    c = {"op": "gemm", "M": M, "N": N, "K": K, "epi": epi, "b_as_nk": b_as_nk, "dist": dist}
    return dict(c, name=name) if name else c


def _vecmat(name, M, N, K):
    c = {"op": "vecmat", "M": M, "N": N, "K": K}
    return dict(c, name=name) if name else c


def _bgemm(name, batch, M, N, K):
    c = {"op": "bgemm_tn", "batch": batch, "M": M, "N": N, "K": K}
    return dict(c, name=name) if name else c


def _sine(name, n):
    c = {"op": "sine", "n": n}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest product of the benchmark: a launch and little else
        _gemm("gemm_256", 256, 256, 256, dist="uniform"),
        # an ordinary square product
        _gemm("gemm_2048", 2048, 2048, 2048, dist="uniform"),
        # the up-projection of a feed-forward layer on 4096 tokens (prefill, forward of training): the largest product
        _gemm("gemm_mlp_up", 4096, 11008, 4096),
        # the same kind of layer while decoding: few rows, the weights are read once
        _gemm("gemm_decode", 16, 8192, 8192),
        # few outputs, a very long sum (K has to be split over the chip)
        _gemm("gemm_tall_k", 1024, 1024, 16384, dist="uniform"),
        # weights stored output-major, a batch of tokens that fills no whole tile, the tanh form of the activation
        _gemm("gemm_nk_prefill", 1500, 4096, 4096, epi="gelu_tanh", b_as_nk=True),
        # decoding with output-major weights and a projection without activation
        _gemm("gemm_nk_decode", 5, 11008, 4096, epi="bias", b_as_nk=True),
        # whole 16-byte rows, but no dimension a multiple of a tile and K no multiple of a K tile
        _gemm("gemm_ragged", 1160, 3080, 1864, epi="bias"),
        # odd dimensions throughout (rows start at any two-byte address), fp32 result
        _gemm("gemm_odd", 509, 1021, 763, epi="fp32"),
        # one matrix per row: the batched vector-matrix product at a memory-filling size
        _vecmat("vecmat_large", 32, 4096, 4096),
        # gradient of the second operand, one product per chunk of a sequence
        _bgemm("bgemm_tn_chunks", 32, 1024, 1024, 256),
        # element-wise sine over a quarter of a gigabyte
        _sine("sine_large", 1 << 26),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiple(x, m):
    return max(m, (x + m // 2) // m * m)


# no drawn case costs more than the largest listed ones
_MAX_FLOPS = 2 * 4096 * 11008 * 4096
_MAX_BYTES = 1 << 30


def draw(rng):
    while True:
        c = _draw_one(rng)
        w = work(c)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            return c


def _draw_one(rng):
    kind = rng.choice(["dense", "dense", "dense", "decode", "decode", "tall", "odd", "vecmat", "bgemm", "sine"])
    nk = rng.random() < 0.4
    epi = rng.choice(["gelu_erf", "gelu_erf", "gelu_tanh", "bias", "fp32"])
    dist = rng.choice(["normal", "uniform"])
    # half of the sizes are round, the others only keep rows of whole 16-byte pieces
    step = 64 if rng.random() < 0.5 else 8
    if kind == "dense":
        return _gemm(None, _log_int(rng, 64, 4096), _multiple(_log_int(rng, 256, 11008), step),
                     _multiple(_log_int(rng, 256, 8192), step), epi, nk, dist)
    if kind == "decode":
        return _gemm(None, rng.randint(1, 32), _multiple(_log_int(rng, 1024, 11008), step),
                     _multiple(_log_int(rng, 1024, 8192), step), epi, nk, dist)
    if kind == "tall":
        return _gemm(None, _log_int(rng, 64, 1024), _multiple(_log_int(rng, 256, 1024), step),
                     _multiple(_log_int(rng, 8192, 16384), step), epi, nk, dist)
    if kind == "odd":
        return _gemm(None, _log_int(rng, 32, 1024), _log_int(rng, 33, 2048) | 1, _log_int(rng, 33, 1024) | 1, epi, nk, dist)
    if kind == "vecmat":
        return _vecmat(None, rng.randint(1, 32), _log_int(rng, 256, 4096), _multiple(_log_int(rng, 256, 4096), 8))
    if kind == "bgemm":
        return _bgemm(None, rng.randint(2, 64), _multiple(_log_int(rng, 128, 1024), 8),
                      _multiple(_log_int(rng, 128, 1024), 8), _multiple(_log_int(rng, 64, 512), 64))
    return _sine(None, _log_int(rng, 100003, 1 << 26))


def _normal(gen, shape, sigma, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=gen).to(dtype)


def _uniform(gen, shape, scale, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-scale, scale, generator=gen).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op = case["op"]
    B = bias = None
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        nk = case["b_as_nk"]
        b_shape = (N, K) if nk else (K, N)
        if case["dist"] == "uniform":           # both operands scaled by 1/sqrt(K), a bias of order one
            A = _uniform(gen, (M, K), K ** -0.5)
            B = _uniform(gen, b_shape, K ** -0.5)
            bias = _normal(gen, (N,), 1.0)
        else:                                   # activations of order one, weights and bias of a trained layer's size
            A = _normal(gen, (M, K), 1.0)
            B = _normal(gen, b_shape, 0.02)
            bias = _normal(gen, (N,), 0.01)
        epi = _EPI[case["epi"]]
        Y = torch.empty((M, N), dtype=torch.float32 if epi == tf.TF_EPI_NONE_F32 else torch.bfloat16, device="cuda")
        prob = tf.Problem(M, N, K, epi=epi, trans_b=nk)
    elif op == "vecmat":
        M, N, K = case["M"], case["N"], case["K"]
        A = _normal(gen, (M, K), 1.0)
        B = _uniform(gen, (M, N, K), K ** -0.5)
        Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
        prob = tf.Problem(M, N, K, op=tf.TF_OP_BATCHED_VECMAT)
    elif op == "bgemm_tn":
        M, N, K = case["M"], case["N"], case["K"]
        A = _normal(gen, (case["batch"], K, M), 1.0)
        B = _uniform(gen, (case["batch"], K, N), K ** -0.5)
        Y = torch.empty((case["batch"], M, N), dtype=torch.float32, device="cuda")
        prob = tf.Problem(M, N, K, op=tf.TF_OP_BATCHED_GEMM_TN, batch=case["batch"])
    else:
        A = _normal(gen, (case["n"],), 10.0, torch.float32)
        Y = torch.empty_like(A)
        prob = tf.Problem(1, case["n"], 0, op=tf.TF_OP_ELEMENTWISE_SIN)
    family = prob.variants()
    tried = [v.id == 0 for v in family]         # the baseline is what the pick is meant to beat
    pick = tf.proposal(prob.desc, tf.hw_query(0), family, tried, 0, tf.TF_BN_UNKNOWN)
    return {"prob": prob, "variant": max(pick, 0), "A": A, "B": B, "bias": bias, "Y": Y}


def run(state):
    state["prob"].run(state["variant"], state["A"], state["B"], state["bias"], state["Y"])
    return state["Y"]


def work(case):
    op = case["op"]
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + K * N + N) + M * N * (4 if case["epi"] == "fp32" else 2), "flops": 2 * M * N * K}
    if op == "vecmat":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + M * N * K) + 4 * M * N, "flops": 2 * M * N * K}
    if op == "bgemm_tn":
        b, M, N, K = case["batch"], case["M"], case["N"], case["K"]
        return {"bytes": b * (2 * K * (M + N) + 4 * M * N), "flops": 2 * b * M * N * K}
    return {"bytes": 8 * case["n"], "flops": case["n"]}


def tolerance(case):
    # Measured against the same operation in double precision on the same inputs; about four times what was seen.
    op = case["op"]
    if op == "gemm" and case["epi"] != "fp32":
        return {"rel": 6e-3}                    # one rounding to bf16: seen 1.4e-3 to 1.7e-3
    if op == "sine":
        return {"rel": 2e-7}                    # seen 3.0e-8 (the polynomial's own error is of that order too)
    return {"rel": 2e-6}                        # sums in fp32: seen 2.5e-8 to 1.7e-7, up to 8.1e-7 where K is 16384
