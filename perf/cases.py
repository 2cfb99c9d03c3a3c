"""Performance cases of the library: what its users have it do, by entry point.

Five kinds of work, each through the public entry points of the binding:

* ``run``: a resident grid iterated by ``ofl_jacobi_run`` inside a data region,
  the result then fetched by ``ofl_update_host``: a solver that looks at its
  iterate every so many iterations.
* ``residual``: ``ofl_residual`` on a resident grid: a convergence check.
* ``program``: the offloaded program from host arrays to host arrays: handle
  created, inputs uploaded, iterations, result downloaded, handle destroyed.
* ``batch``: many uneven grids in one ``ofl_batch_run``.
* ``gemm``: ``ofl_gemm_f32``, the routine a recognised matrix-product block is
  replaced with.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2011_03602_amd as ofl

OMEGA = np.float32(0.8)
FORMATS = {"f32": ofl.OFL_COEF_F32, "bf16": ofl.OFL_COEF_BF16, "bf16_offset": ofl.OFL_COEF_BF16_OFFSET}
SUMS = {"f64": ofl.OFL_SUM_F64, "compensated": ofl.OFL_SUM_KAHAN_F32}
FUSE_ALL = ofl.OFL_FUSE_RESIDUAL | ofl.OFL_FUSE_COPYBACK_SWAP


def _run(name, I, J, K, iters, fmt="f32", fuse=False, sums="f64"):
    return {"name": name, "kind": "run", "I": I, "J": J, "K": K, "iters": iters, "format": fmt, "fuse": fuse,
            "sum": sums}


def _gemm(name, M, N, K, pad=0):
    return {"name": name, "kind": "gemm", "M": M, "N": N, "K": K, "pad": pad}


def listed():
    return [
        # a convergence check on a small grid: one call, bound by its launches
        {"name": "residual-65", "kind": "residual", "I": 65, "J": 65, "K": 129, "format": "f32"},
        # the smallest grid the project checks end to end, 50 iterations
        _run("run-33x33x65", 33, 33, 65, 50),
        # the middle configuration, as a user calls it without any option
        _run("run-129x129x257", 129, 129, 257, 100),
        # the headline configuration of the benchmark, without any option
        _run("run-257x257x513", 257, 257, 513, 100),
        # the same grid in the precision variant with both fusions asked for
        _run("run-257x257x513-bf16-fused", 257, 257, 513, 100, "bf16_offset", True),
        # a ragged grid with rows of several tiles, plain bfloat16 storage,
        # compensated residual
        _run("run-301x99x143-bf16", 301, 99, 143, 30, "bf16", False, "compensated"),
        # the offloaded program end to end, PCIe and allocation included
        {"name": "program-129x129x257", "kind": "program", "I": 129, "J": 129, "K": 257, "iters": 50,
         "format": "f32"},
        # the batch workload: uneven grids in one graph launch
        {"name": "batch-32", "kind": "batch", "n": 32, "iters": 20, "format": "f32", "fuse": False, "sizes": 1},
        # a smaller batch in the fastest form the library offers
        {"name": "batch-12-bf16-fused", "kind": "batch", "n": 12, "iters": 20, "format": "bf16_offset",
         "fuse": True, "sizes": 2},
        # the last layer of the perceptron program: a tall product 16 columns wide
        _gemm("gemm-8192x16x4096", 8192, 16, 4096),
        # an odd product with odd row strides
        _gemm("gemm-511x333x1001", 511, 333, 1001, 1),
        # the perceptron's hidden layer, square
        _gemm("gemm-4096", 4096, 4096, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes log-uniform, any parity."""
    kind = rng.choice(["run", "run", "run", "gemm", "gemm", "gemm", "batch", "residual", "program"])
    if kind == "gemm":
        while True:
            M, N, K = _log_int(rng, 64, 8192), _log_int(rng, 8, 4096), _log_int(rng, 32, 4096)
            if M * N * K >= 1 << 21:
                return {"kind": "gemm", "M": M, "N": N, "K": K, "pad": rng.choice([0, 0, 0, 1, 4])}
    if kind == "batch":
        return {"kind": "batch", "n": _log_int(rng, 4, 32), "iters": _log_int(rng, 5, 20),
                "format": rng.choice(sorted(FORMATS)), "fuse": rng.random() < 0.5, "sizes": rng.randrange(1 << 20)}
    I, J, K = _log_int(rng, 33, 385), _log_int(rng, 33, 257), _log_int(rng, 33, 385)
    case = {"kind": kind, "I": I, "J": J, "K": K, "format": rng.choice(["f32", "f32", "bf16", "bf16_offset"])}
    if kind != "residual":
        case["iters"] = _log_int(rng, 10, 100)
    if kind == "run":
        case["fuse"] = rng.random() < 0.5
        case["sum"] = "f64" if case["fuse"] else rng.choice(["f64", "compensated"])
    return case


def _batch_shapes(case):
    """Uneven shapes, I and J in 33..161 and K in 65..321."""
    rng = np.random.default_rng(case["sizes"])
    return [(int(rng.integers(33, 162)), int(rng.integers(33, 162)), int(rng.integers(65, 322)))
            for _ in range(case["n"])]


def _fields(shape, seed):
    """The arrays of one grid on the GPU, shape (K, J, I): coefficients near a
    Laplacian's, a small cross term and right-hand side, a random iterate."""
    I, J, K = shape
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def u(lo, hi):
        return torch.empty((K, J, I), device="cuda").uniform_(lo, hi, generator=gen)

    a = {n: u(0.95, 1.05) for n in ("a0", "a1", "a2")}
    a["a3"] = (1.0 / (2.0 * (a["a0"].double() + a["a1"].double() + a["a2"].double()))).float()
    for n in ("b0", "b1", "b2"):
        a[n] = u(-0.01, 0.01)
    for n in ("c0", "c1", "c2"):
        a[n] = torch.ones((K, J, I), device="cuda")
    a["bnd"] = torch.zeros((K, J, I), device="cuda")
    a["bnd"][1:-1, 1:-1, 1:-1] = 1.0
    a["wrk1"] = u(-0.1, 0.1)
    a["p"] = u(0.0, 1.0)
    return a


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


def _grid(shape, seed, case, row_align=0):
    arrays = {n: t.cpu().numpy() for n, t in _fields(shape, seed).items()}
    return ofl.Grid(arrays, coef_format=FORMATS[case["format"]], sum_mode=SUMS[case.get("sum", "f64")],
                    torch_memory=True, pinned=True, row_align=row_align)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        M, N, K, pad = case["M"], case["N"], case["K"], case["pad"]
        a, b = _operands(case, seed)
        return {"kind": kind, "dims": (M, N, K), "a": a, "b": b, "c": torch.zeros((M, N + pad), device="cuda"),
                "ld": (K + pad, N + pad, N + pad)}
    if kind == "batch":
        grids = [_grid(s, seed * 1000 + t, case, row_align=4) for t, s in enumerate(_batch_shapes(case))]
        b = ofl.ofl_batch_create([g.handle for g in grids])
        if case["fuse"]:
            ofl.ofl_batch_set_fusion(b, FUSE_ALL)
        for g in grids:
            ofl.ofl_data_enter(g.handle)
        return {"kind": kind, "batch": _Batch(b, grids), "iters": case["iters"]}
    shape = (case["I"], case["J"], case["K"])
    if kind == "program":
        keep = {n: _pinned(t) for n, t in _fields(shape, seed).items()}
        keep["wrk2"] = torch.zeros(keep["p"].shape, pin_memory=True)
        d = ofl.OflGridDesc()
        d.I, d.J, d.K = shape
        d.coef_format, d.sum_mode, d.device = FORMATS[case["format"]], ofl.OFL_SUM_F64, -1
        d.p, d.wrk2 = (keep[n].numpy().ctypes.data_as(ofl._FP) for n in ("p", "wrk2"))
        for t, n in enumerate(ofl.COEF_NAMES):
            d.coef[t] = keep[n].numpy().ctypes.data_as(ofl._FP)
        return {"kind": kind, "desc": d, "keep": keep, "iters": case["iters"]}
    g = _grid(shape, seed, case)
    if case.get("fuse"):
        ofl.ofl_set_fusion(g.handle, FUSE_ALL)
    ofl.ofl_data_enter(g.handle)
    return {"kind": kind, "grid": g, "iters": case.get("iters")}


class _Batch:
    """A batch and its grids; the batch goes first."""

    def __init__(self, handle, grids):
        self.handle, self.grids = handle, grids

    def __del__(self):
        ofl.ofl_batch_destroy(self.handle)


def run(state):
    kind = state["kind"]
    if kind == "gemm":
        (M, N, K), (lda, ldb, ldc) = state["dims"], state["ld"]
        ofl.ofl_gemm_f32(M, N, K, state["a"].data_ptr(), lda, state["b"].data_ptr(), ldb, state["c"].data_ptr(), ldc,
                         torch.cuda.current_stream().cuda_stream)
        return state["c"]
    if kind == "batch":
        b = state["batch"]
        gosa = ofl.ofl_batch_run(b.handle, state["iters"], OMEGA, len(b.grids))
        for g in b.grids:
            ofl.ofl_update_host(g.handle)
        return {"gosa": np.array(gosa), "p": [g.p for g in b.grids]}
    if kind == "program":
        h = ofl.ofl_grid_create(state["desc"])
        gosa = ofl.ofl_jacobi_run(h, state["iters"], OMEGA)
        ofl.ofl_grid_destroy(h)
        return {"gosa": gosa, "p": state["keep"]["p"].numpy()}
    h = state["grid"].handle
    if kind == "residual":
        return ofl.ofl_residual(h)
    gosa = ofl.ofl_jacobi_run(h, state["iters"], OMEGA)
    ofl.ofl_update_host(h)
    return {"gosa": gosa, "p": state["grid"].p}


def work(case):
    """Inputs read once and outputs written once; the arithmetic of every iteration."""
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 4 * (M * K + K * N + M * N), "flops": 2 * M * N * K}
    celem = 4 if case["format"] == "f32" else 2
    shapes = _batch_shapes(case) if kind == "batch" else [(case["I"], case["J"], case["K"])]
    points = sum((I - 2) * (J - 2) * (K - 2) for I, J, K in shapes)
    p_moves = 1 if kind == "residual" else 2
    # 34 operations of the sweep and 3 of the residual per interior point and iteration
    return {"bytes": (12 * celem + 4 * p_moves) * points, "flops": 37 * points * case.get("iters", 1)}


def _operands(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn((case["M"], case["K"] + case["pad"]), device="cuda", generator=gen)
    b = torch.randn((case["K"], case["N"] + case["pad"]), device="cuda", generator=gen)
    return a, b


def _sweep64(a, p, omega):
    """The new iterate's interior and its scaled step, in 64 bits."""
    mid, lo, hi = slice(1, -1), slice(0, -2), slice(2, None)

    def at(k, j, i):
        return p[k, j, i]

    def c(n):
        return a[n][mid, mid, mid]

    s = c("a0") * at(mid, mid, hi) + c("a1") * at(mid, hi, mid) + c("a2") * at(hi, mid, mid)
    s += c("b0") * (at(mid, hi, hi) - at(mid, lo, hi) - at(mid, hi, lo) + at(mid, lo, lo))
    s += c("b1") * (at(hi, hi, mid) - at(hi, lo, mid) - at(lo, hi, mid) + at(lo, lo, mid))
    s += c("b2") * (at(hi, mid, hi) - at(lo, mid, hi) - at(hi, mid, lo) + at(lo, mid, lo))
    s += c("c0") * at(mid, mid, lo) + c("c1") * at(mid, lo, mid) + c("c2") * at(lo, mid, mid) + c("wrk1")
    ss = (c("a3") * s - at(mid, mid, mid)) * c("bnd")
    return at(mid, mid, mid) + omega * ss, ss


def _solve64(shape, seed, iters, omega):
    a = {n: t.double() for n, t in _fields(shape, seed).items()}
    p = a.pop("p")
    gosa = 0.0
    for _ in range(iters):
        new, ss = _sweep64(a, p, omega)
        gosa = float((ss * ss).sum())
        p[1:-1, 1:-1, 1:-1] = new
    return gosa, p.cpu().numpy()


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        a, b = _operands(case, seed)
        c = torch.zeros((case["M"], case["N"] + case["pad"]), device="cuda", dtype=torch.float64)
        c[:, :case["N"]] = a[:, :case["K"]].double() @ b[:, :case["N"]].double()
        return c
    if kind == "batch":
        out = [_solve64(s, seed * 1000 + t, case["iters"], float(OMEGA)) for t, s in enumerate(_batch_shapes(case))]
        return {"gosa": np.array([g for g, _ in out]), "p": [p for _, p in out]}
    shape = (case["I"], case["J"], case["K"])
    if kind == "residual":
        return _solve64(shape, seed, 1, 1.0)[0]
    gosa, p = _solve64(shape, seed, case["iters"], float(OMEGA))
    return {"gosa": gosa, "p": p}
