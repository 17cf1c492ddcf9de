"""What a user of this library has it do, as cases that can be timed and checked.

A case is one pass through the public entry points: ``gemm`` on row-major torch
tensors, the BLAS-shaped calls of ``Handle`` on column-major buffers, or a batch of
uneven problems.  Entries are drawn on the device as (u - 0.5) exp(phi g), u uniform,
g normal (the generator of ``workloads.py``), real and imaginary parts alike.

Fields of a case (plain values):
  entry   "gemm" (row-major tensors, result in a new tensor), "blas" (column-major
          buffers with leading dimensions, result in a given C) or "batch"
  type    "z" complex128, "c" complex64, "d" float64, "s" float32
  m, n, k shape of the product; batch: count, lo, hi instead (log-uniform sizes)
  moduli, mode, algo   the handle's configuration
  ta, tb, pad, beta    blas only: op(A), op(B), extra rows of every leading dimension,
          real beta (alpha is then 1.5, with an imaginary part for complex types)
  verify  blas only: the Freivalds check (the call then waits for its verdict)
  phi     spread of the values
"""
from __future__ import annotations

import math
import random

import torch

import paper_2512_08321_amd as ozc

DTYPE = {"z": torch.complex128, "c": torch.complex64, "d": torch.float64, "s": torch.float32}


def _case(name, entry, type, m=0, n=0, k=0, moduli=14, mode="fast", algo="karatsuba", ta="N",
          tb="N", pad=0, beta=0.0, verify=False, phi=0.5, count=0, lo=0, hi=0):
    return {"name": name, "entry": entry, "type": type, "m": m, "n": n, "k": k, "moduli": moduli,
            "mode": mode, "algo": algo, "ta": ta, "tb": tb, "pad": pad, "beta": beta,
            "verify": verify, "phi": phi, "count": count, "lo": lo, "hi": hi}


def listed():
    return [
        # a small block of a dense solver: launches and latency are the whole call
        _case("zgemm 64", "gemm", "z", 64, 64, 64),
        # the paper's method in its plain form on a small product (expanded products)
        _case("zgemm 256 expanded", "gemm", "z", 256, 256, 256, algo="4m"),
        # a ragged update C := alpha A^T B + beta C in single precision, padded buffers
        _case("cgemm ragged update", "blas", "c", 333, 777, 555, moduli=8, ta="T", pad=3, beta=0.5),
        # an ordinary product whose result is certified before it is used
        _case("zgemm 1000 verified", "blas", "z", 1000, 900, 1100, ta="C", verify=True),
        # real double precision, rectangular
        _case("dgemm 1536x2048x1000", "gemm", "d", 1536, 2048, 1000),
        # real single precision, larger and short in k (a panel update)
        _case("sgemm 3000x3000x700", "gemm", "s", 3000, 3000, 700, moduli=8),
        # an inner-product shape: little output, very long k
        _case("zgemm 384x320x40000", "gemm", "z", 384, 320, 40000),
        # accurate scaling at a middle size, wide values
        _case("zgemm 2048 accurate", "gemm", "z", 2048, 2048, 2048, moduli=13, mode="accurate", phi=2.0),
        # many independent products of uneven shapes in one call
        _case("zgemm batch", "batch", "z", count=64, lo=64, hi=2048, phi=2.0),
        # single-precision complex at the size of the moduli sweeps, fewest useful moduli
        _case("cgemm 4096", "gemm", "c", 4096, 4096, 4096, moduli=6),
        # double-precision complex at the size of the moduli sweeps
        _case("zgemm 4096", "gemm", "z", 4096, 4096, 4096),
        # the benchmark's product
        _case("zgemm 16384", "gemm", "z", 16384, 16384, 16384),
    ]


def _log_int(rng, lo, hi):
    """Log-uniform integer, half of them off the multiples of 64."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        x = (x + 32) // 64 * 64
    return max(lo, min(hi, x))


def draw(rng: random.Random):
    if rng.random() < 0.15:
        lo = rng.choice([64, 100, 128])
        return _drawn("batch", rng.choice("zzc"), rng, count=rng.randint(8, 64), lo=lo,
                      hi=rng.randint(4 * lo, 2048))
    type = rng.choice("zzzccds")
    shape = rng.random()
    if shape < 0.2:    # long inner dimension
        m, n, k = _log_int(rng, 64, 1024), _log_int(rng, 64, 1024), _log_int(rng, 4096, 65536)
    elif shape < 0.4:  # short inner dimension
        m, n, k = _log_int(rng, 512, 8192), _log_int(rng, 512, 8192), _log_int(rng, 64, 512)
    else:              # all dimensions alike in range
        m, n, k = (_log_int(rng, 64, 8192) for _ in range(3))
    if rng.random() < 0.5:
        return _drawn("gemm", type, rng, m=m, n=n, k=k)
    complex_type = type in "zc"
    return _drawn("blas", type, rng, m=m, n=n, k=k, ta=rng.choice("NTC"), tb=rng.choice("NTC"),
                  pad=rng.choice([0, 0, 1, 8]), beta=rng.choice([0.0, 0.0, 0.5]),
                  verify=complex_type and rng.random() < 0.25)


def _drawn(entry, type, rng, **kw):
    c = _case("", entry, type, moduli=rng.randint(12, 18) if type in "zd" else rng.randint(6, 9),
              mode=rng.choice(["fast", "fast", "accurate"]),
              algo=rng.choice(["karatsuba", "karatsuba", "karatsuba", "4m"]),
              phi=round(rng.uniform(0.0, 2.0), 2), **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _matrix(rows, cols, dtype, phi, gen):
    """rows x cols device tensor, entries (u - 0.5) exp(phi g)."""
    real = torch.float64 if dtype in (torch.complex128, torch.float64) else torch.float32
    out = torch.empty((rows, cols), dtype=dtype, device="cuda")
    for part in ([out.real, out.imag] if dtype.is_complex else [out]):
        x = torch.rand((rows, cols), dtype=real, device="cuda", generator=gen).sub_(0.5)
        g = torch.randn((rows, cols), dtype=real, device="cuda", generator=gen)
        part.copy_(x.mul_(g.mul_(phi).exp_()))
    return out


def _batch_shapes(case, seed):
    # the shapes belong to the case, the values to the seed
    rng = random.Random(1000 * case["count"] + case["hi"])
    span = (math.log(case["lo"]), math.log(case["hi"]))
    return [tuple(int(round(math.exp(rng.uniform(*span)))) for _ in range(3))
            for _ in range(case["count"])]


def _scalars(case):
    if case["beta"] == 0.0:
        return 1.0, 0.0
    return (1.5 - 0.25j if case["type"] in "zc" else 1.5), case["beta"]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype, phi = DTYPE[case["type"]], case["phi"]
    mat = lambda r, c: _matrix(r, c, dtype, phi, gen)
    if case["entry"] == "batch":
        # column-major m x k, k x n, m x n: row-major tensors of the transposed shape
        return [(mat(k, m), mat(n, k), torch.zeros((n, m), dtype=dtype, device="cuda"))
                for m, n, k in _batch_shapes(case, seed)]
    m, n, k = case["m"], case["n"], case["k"]
    if case["entry"] == "gemm":
        return mat(m, k), mat(k, n)
    pad = case["pad"]
    A = mat(k, m + pad) if case["ta"] == "N" else mat(m, k + pad)
    B = mat(n, k + pad) if case["tb"] == "N" else mat(k, n + pad)
    C = mat(n, m + pad) if case["beta"] else torch.zeros((n, m + pad), dtype=dtype, device="cuda")
    return A, B, C


def prepare(case, seed):
    state = {"case": case, "inputs": _inputs(case, seed)}
    if case["entry"] == "gemm":
        return state
    h = ozc.Handle(0, num_moduli=case["moduli"], mode=case["mode"], algo=case["algo"])
    h.set_verify(case["verify"])
    state["handle"] = h
    if case["entry"] == "batch":
        state["problems"] = [
            {"transa": "N", "transb": "N", "m": m, "n": n, "k": k, "alpha": 1.0, "A": A, "lda": m,
             "B": B, "ldb": k, "beta": 0.0, "C": C, "ldc": m}
            for (m, n, k), (A, B, C) in zip(_batch_shapes(case, seed), state["inputs"])]
    return state


# ---------------------------------------------------------------- one pass

def run(state):
    case = state["case"]
    if case["entry"] == "gemm":
        A, B = state["inputs"]
        return ozc.gemm(A, B, num_moduli=case["moduli"], mode=case["mode"], algo=case["algo"])
    h = state["handle"]
    if case["entry"] == "batch":
        h.gemm_vbatched(state["problems"], single=case["type"] == "c")
        return [C for _, _, C in state["inputs"]]
    A, B, C = state["inputs"]
    if case["beta"]:
        C = C.clone()  # the given C is kept, so that a pass can be repeated
    alpha, beta = _scalars(case)
    call = {"z": h.zgemm, "c": h.cgemm, "d": h.dgemm, "s": h.sgemm}[case["type"]]
    call(case["ta"], case["tb"], case["m"], case["n"], case["k"], alpha, A, A.shape[1], B,
         B.shape[1], beta, C, C.shape[1])
    return C


# ---------------------------------------------------------------- what a pass needs

def _work(case, m, n, k):
    size = {"z": 16, "c": 8, "d": 8, "s": 4}[case["type"]]
    bytes = size * (m * k + k * n + m * n * (2 if case["beta"] else 1))
    # INT8 operations of the residue products (2 per multiply-add): one product of real,
    # three of complex matrices per modulus, and the bound product of accurate scaling
    products = 3 if case["type"] in "zc" else 1
    moduli = case["moduli"] + (1 if case["mode"] == "accurate" else 0)
    return bytes, 2.0 * products * moduli * m * n * k


def work(case):
    shapes = (_batch_shapes(case, 0) if case["entry"] == "batch"
              else [(case["m"], case["n"], case["k"])])
    each = [_work(case, *s) for s in shapes]
    return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}


def _mm(a, b):
    wide = torch.complex128 if a.dtype.is_complex else torch.float64
    return a.to(wide) @ b.to(wide)


def exact(case, seed):
    inputs = _inputs(case, seed)
    if case["entry"] == "batch":
        return [_mm(B, A) for A, B, _ in inputs]  # column-major: C^T = B^T A^T
    if case["entry"] == "gemm":
        return _mm(*inputs)
    A, B, C = inputs
    m, n, k = case["m"], case["n"], case["k"]
    # op(A), op(B) from the column-major buffers
    opA = A[:, :m].T if case["ta"] == "N" else A[:, :k]
    opB = B[:, :k].T if case["tb"] == "N" else B[:, :n]
    if case["ta"] == "C":
        opA = opA.conj()
    if case["tb"] == "C":
        opB = opB.conj()
    alpha, beta = _scalars(case)
    out = C.to(torch.complex128 if C.dtype.is_complex else torch.float64)
    out = out.clone()
    out[:, :m] = alpha * _mm(opA, opB).T + beta * out[:, :m]
    return out
