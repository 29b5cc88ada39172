"""Performance cases: what programs have this library do, through its public entry points.

Every case multiplies matrices with the entries of the paper's experiments,
(rand - 0.5) exp(phi randn).  Kinds:

  "gemm"     one product of row-major torch matrices, A (m x k) times B (k x n), through
             dgemm, sgemm, zgemm or cgemm (by "dtype");
  "batch"    "count" independent DGEMMs of uneven shapes (log-uniform in [64, 2048]) in one
             ozaki2_dgemm_batched call into one caller-owned output buffer, with moduli counts
             that the autotuner chose beforehand (a program that repeats a batch of the same
             shapes on other data);
  "target"   the same kind of batch through dgemm_batched with an error target, so that every
             call estimates the spread of its data and picks the moduli counts itself.
"""
import ctypes
import math
import random

import torch

from paper_2606_29129_amd import ozaki2 as oz

_DTYPES = {"float64": torch.float64, "float32": torch.float32,
           "complex128": torch.complex128, "complex64": torch.complex64}
_GEMMS = {"float64": oz.dgemm, "float32": oz.sgemm, "complex128": oz.zgemm,
          "complex64": oz.cgemm}
_ITEM = {"float64": 8, "float32": 4, "complex128": 16, "complex64": 8}


def _gemm(name, m, n, k, N, dtype="float64", mode="revised", phi=0.5):
    return {"name": name, "kind": "gemm", "m": m, "n": n, "k": k, "N": N, "dtype": dtype,
            "mode": mode, "phi": phi}


def listed():
    return [
        # the smallest product of the benchmark's configurations: a call's latency
        _gemm("dgemm 256", 256, 256, 256, 14),
        # a small product, called many times in a row (blocked factorisations)
        _gemm("dgemm 1024", 1024, 1024, 1024, 14),
        # sizes as they come: nothing a multiple of a tile, uneven sides
        _gemm("dgemm 3001x1777x2503", 3001, 1777, 2503, 16, phi=1.0),
        # an ordinary product
        _gemm("dgemm 4096", 4096, 4096, 4096, 14),
        # the benchmark's own workload: full double accuracy on a large product
        _gemm("dgemm 16384", 16384, 16384, 16384, 17),
        # a tall matrix times a few columns (block vectors, projections), and its transpose
        _gemm("dgemm 65536x64x4096", 65536, 64, 4096, 14, phi=1.0),
        _gemm("dgemm 64x65536x4096", 64, 65536, 4096, 14, phi=1.0),
        # accurate mode: the scaling found by a bound product instead of norms
        _gemm("dgemm accurate 8192x8192x1024", 8192, 8192, 1024, 14, mode="accurate", phi=1.0),
        # binary32 matrices at binary32 accuracy
        _gemm("sgemm 4096", 4096, 4096, 4096, 7, dtype="float32", phi=1.0),
        # complex matrices
        _gemm("zgemm 4096", 4096, 4096, 4096, 14, dtype="complex128"),
        # many independent products at once, repeated with the same shapes on other data
        {"name": "batch of 256", "kind": "batch", "count": 256, "shapes": 0, "target": 1e-15},
        # the same with the moduli counts found anew on every call
        {"name": "batch of 64 by target", "kind": "target", "count": 64, "shapes": 1,
         "target": 1e-15},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "square", "uneven", "uneven", "narrow", "single", "complex",
                       "mode", "batch", "target"])
    if kind in ("batch", "target"):
        return {"kind": kind, "count": _log_int(rng, 16, 256 if kind == "batch" else 64),
                "shapes": rng.randrange(2, 1 << 20), "target": rng.choice([1e-15, 1e-12, 1e-8])}
    case = {"kind": "gemm", "dtype": "float64", "mode": "revised",
            "phi": rng.choice([0.5, 1.0, 2.0]), "N": rng.randint(12, 20)}
    if kind == "square":
        m = n = k = _log_int(rng, 128, 12288)
    elif kind == "narrow":
        # one side of 1 to 64 rows or columns
        m, n, k = _log_int(rng, 2048, 131072), rng.randint(1, 64), _log_int(rng, 256, 8192)
        if rng.random() < 0.5:
            m, n = n, m
    else:
        top = 4096 if kind == "complex" else 10240
        m, n, k = (_log_int(rng, 96, top) for _ in range(3))
    if kind == "single" or (kind == "complex" and rng.random() < 0.5):
        case["N"] = rng.randint(6, 9)
        case["dtype"] = "float32" if kind == "single" else "complex64"
    elif kind == "complex":
        case["dtype"] = "complex128"
    if kind == "mode":
        case["mode"] = rng.choice(["original", "accurate", "exact"])
    case.update(m=m, n=n, k=k)
    return case


def _shapes(case):
    """The (m, n, k, phi) of a batch's problems."""
    rng = random.Random(case["shapes"])
    return [(_log_int(rng, 64, 2048), _log_int(rng, 64, 2048), _log_int(rng, 64, 2048),
             rng.uniform(0.5, 3.0)) for _ in range(case["count"])]


def _moduli(case):
    """The moduli counts of a batch's problems, as the library's autotuner picks them for
    their nominal spread (the counts found on the data are these or a neighbour)."""
    return [oz.ozaki2_autotune_N(k, phi, case["target"]) for _, _, k, phi in _shapes(case)]


def _matrix(gen, rows, cols, phi, dtype):
    real = {"complex128": torch.float64, "complex64": torch.float32}.get(dtype, _DTYPES[dtype])
    shape = (rows, cols, 2) if dtype.startswith("complex") else (rows, cols)
    x = torch.randn(shape, dtype=real, device="cuda", generator=gen).mul_(phi).exp_()
    x.mul_(torch.rand(shape, dtype=real, device="cuda", generator=gen).sub_(0.5))
    return torch.view_as_complex(x) if dtype.startswith("complex") else x


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] == "gemm":
        m, n, k, phi, dtype = (case[x] for x in ("m", "n", "k", "phi", "dtype"))
        return _matrix(gen, m, k, phi, dtype), _matrix(gen, k, n, phi, dtype)
    return [(_matrix(gen, m, k, phi, "float64"), _matrix(gen, k, n, phi, "float64"))
            for m, n, k, phi in _shapes(case)]


def prepare(case, seed):
    inputs = _inputs(case, seed)
    state = {"case": case, "inputs": inputs}
    if case["kind"] == "batch":
        shapes = _shapes(case)
        flat = torch.empty(sum(m * n for m, n, _, _ in shapes), dtype=torch.float64,
                           device="cuda")
        problems = (oz.Oz2Problem * len(shapes))()
        at = 0
        for i, ((m, n, k, _), (A, B), N) in enumerate(zip(shapes, inputs, _moduli(case))):
            C = flat[at:at + m * n]
            at += m * n
            # row-major C = A B is the column-major C^T = B^T A^T
            problems[i] = oz.Oz2Problem(n, m, k, B.data_ptr(), n, A.data_ptr(), k, C.data_ptr(),
                                        n, N, 0)
        state.update(out=flat, problems=problems,
                     bytes=oz.ozaki2_dgemm_batched_workspace_size(list(problems)))
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "gemm":
        A, B = state["inputs"]
        return _GEMMS[case["dtype"]](A, B, N=case["N"], mode=case["mode"])
    if case["kind"] == "target":
        return oz.dgemm_batched(state["inputs"], target=case["target"])
    oz.ozaki2_set_stream(torch.cuda.current_stream())
    oz.ensure_workspace(state["bytes"])
    problems = state["problems"]
    bad = ctypes.c_int(-1)
    rc = oz.lib().ozaki2_dgemm_batched(len(problems), problems, oz.MODE_REVISED, 0.0,
                                       ctypes.byref(bad))
    if rc:
        raise oz.Ozaki2Error("ozaki2_dgemm_batched (problem %d)" % bad.value, rc)
    return state["out"]


def work(case):
    """Inputs read once, outputs written once, and the INT8 operations of the residue products
    (three real products per complex one)."""
    if case["kind"] == "gemm":
        m, n, k, N = (case[x] for x in ("m", "n", "k", "N"))
        comps = 3 if case["dtype"].startswith("complex") else 1
        return {"bytes": _ITEM[case["dtype"]] * (m * k + k * n + m * n),
                "flops": 2.0 * comps * N * m * n * k}
    shapes = _shapes(case)
    return {"bytes": 8 * sum(m * k + k * n + m * n for m, n, k, _ in shapes),
            "flops": sum(2.0 * N * m * n * k
                         for (m, n, k, _), N in zip(shapes, _moduli(case)))}


def exact(case, seed):
    inputs = _inputs(case, seed)

    def product(A, B):
        wide = torch.complex128 if A.is_complex() else torch.float64
        return torch.matmul(A.to(wide), B.to(wide))

    if case["kind"] == "gemm":
        return product(*inputs)
    outs = [product(A, B) for A, B in inputs]
    return torch.cat([C.reshape(-1) for C in outs]) if case["kind"] == "batch" else outs
