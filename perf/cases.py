"""Workloads of the library's public entry points, for timing and comparison.

Every case is one pass of work as a user's program has it done: the R factor
of one matrix (``tsqr.geqr_r``), of many matrices of mixed heights in one
launch (``tsqr.BatchPlan``), A = QR with an explicit Q (``tsqr.geqr_qr``), a
least-squares right-hand side through the stored reflectors
(``tsqr.Factorization``), and the FP64-accurate R of a batch stored in FP32
(``tsqr.MixedPlan``).  Sizes are those of the benchmark, the tests and the
paper (m = 10^6, n = 50), and generic odd ones between them.

Keys of a case:
  kind    r | batch | qr | lsq | mixed
  dtype   f64 | f32 (what A holds; ``mixed`` is always FP32 storage)
  m, n    the matrix; for ``batch`` the heights are ``count`` draws,
          log-uniform in [lo, hi] (fixed by ``sizes_seed``: they belong to the
          plan, not to the data)
  pad     rows of padding in the leading dimension
  decades the singular values fall over this many powers of ten (0: plain
          uniform[-1, 1) entries)
  tuned   whether the program loaded the measured tuning table into its handle
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1002_4250_amd import autotune, inputs, tsqr

_DT = {"f64": torch.float64, "f32": torch.float32}
_BYTES = {"f64": 8, "f32": 4}


def listed():
    return [
        # the smallest call: one small matrix, e.g. a per-block QR inside another
        # solver's loop; launches and the dependent chain are all there is
        {"name": "r_f64_256x50", "kind": "r", "dtype": "f64", "m": 256, "n": 50, "pad": 0, "decades": 0,
         "tuned": False},
        # the paper's experiment (section 4, Table 2)
        {"name": "r_f64_1e6x50", "kind": "r", "dtype": "f64", "m": 1000000, "n": 50, "pad": 0, "decades": 0,
         "tuned": True},
        # the benchmark's instance in both precisions: a long tall-skinny matrix
        {"name": "r_f64_4194304x50", "kind": "r", "dtype": "f64", "m": 1 << 22, "n": 50, "pad": 0, "decades": 0,
         "tuned": True},
        {"name": "r_f32_4194304x50", "kind": "r", "dtype": "f32", "m": 1 << 22, "n": 50, "pad": 0, "decades": 0,
         "tuned": True},
        # an ill-conditioned basis (polynomial or Krylov vectors) with a padded
        # leading dimension and an odd shape
        {"name": "r_f64_200001x37_cond", "kind": "r", "dtype": "f64", "m": 200001, "n": 37, "pad": 7, "decades": 8,
         "tuned": False},
        # a mid-sized FP32 matrix at the largest column count, odd height
        {"name": "r_f32_20001x64", "kind": "r", "dtype": "f32", "m": 20001, "n": 64, "pad": 0, "decades": 0,
         "tuned": False},
        # the ragged batch of the benchmark: many instances of mixed heights in one launch
        {"name": "batch_f32_4096x50", "kind": "batch", "dtype": "f32", "count": 4096, "lo": 64, "hi": 65536, "n": 50,
         "sizes_seed": 2, "tuned": True},
        # a smaller FP64 batch with many short instances (some shorter than n)
        {"name": "batch_f64_512x32", "kind": "batch", "dtype": "f64", "count": 512, "lo": 8, "hi": 20000, "n": 32,
         "sizes_seed": 5, "tuned": False},
        # an explicit orthonormal basis
        {"name": "qr_f64_1048576x50", "kind": "qr", "dtype": "f64", "m": 1 << 20, "n": 50, "pad": 0, "decades": 0,
         "tuned": False},
        {"name": "qr_f32_333333x20", "kind": "qr", "dtype": "f32", "m": 333333, "n": 20, "pad": 3, "decades": 0,
         "tuned": False},
        # least squares with one right-hand side: factor, then c = Q^T b without forming Q
        {"name": "lsq_f64_1e6x50_k1", "kind": "lsq", "dtype": "f64", "m": 1000000, "n": 50, "k": 1, "pad": 0,
         "decades": 0, "tuned": False},
        # a batch stored in FP32 and wanted to FP64 accuracy, condition numbers up to 1e8
        {"name": "mixed_256x65536x50", "kind": "mixed", "batch": 256, "m": 65536, "n": 50, "sample_rows": 4096,
         "decades": 8, "tuned": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["r", "r", "r", "batch", "qr", "lsq", "mixed"])
    n = rng.choice([rng.randint(1, 64), rng.randint(17, 64), 50])
    dtype = rng.choice(["f64", "f32"])
    if kind == "r":
        m = _log_int(rng, 64, min(1 << 22, (1 << 22) * 50 // n))
        decades = rng.choice([0, 0, 0, 6]) if dtype == "f64" and m >= 4 * n and m <= 1 << 20 else 0
        return {"kind": "r", "dtype": dtype, "m": m, "n": n, "pad": rng.choice([0, 0, 1, 13]), "decades": decades,
                "tuned": rng.random() < 0.5}
    if kind == "batch":
        hi = _log_int(rng, 1000, 65536)
        return {"kind": "batch", "dtype": dtype, "count": _log_int(rng, 16, 1024), "lo": rng.choice([16, 64, 500]),
                "hi": hi, "n": n, "sizes_seed": rng.randint(0, 1 << 20), "tuned": rng.random() < 0.5}
    if kind == "qr":
        return {"kind": "qr", "dtype": dtype, "m": _log_int(rng, 256, 1 << 20), "n": n, "pad": rng.choice([0, 5]),
                "decades": 0, "tuned": False}
    if kind == "lsq":
        return {"kind": "lsq", "dtype": dtype, "m": _log_int(rng, 256, 1 << 20), "n": n,
                "k": rng.choice([1, 2, 10, 50, 64]), "pad": 0, "decades": 0, "tuned": False}
    return {"kind": "mixed", "batch": _log_int(rng, 8, 128), "m": _log_int(rng, 2000, 65536), "n": n,
            "sample_rows": rng.choice([0, 1024, 4096]), "decades": rng.choice([2, 6]), "tuned": False}


_TUNED = []


def _handle(case):
    """The handle a program keeps: the library's own for the device, or one with the measured table loaded."""
    if not case.get("tuned"):
        return tsqr.handle(0)
    if not _TUNED:
        _TUNED.append(tsqr.tsqr_create(0))
        autotune.apply_default(_TUNED[0])
    return _TUNED[0]


def _uniform(shape, dtype, gen):
    return torch.empty(shape, dtype=dtype, device="cuda").uniform_(-1.0, 1.0, generator=gen)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _matrix(case, seed):
    """A as the m-by-n view of a column-major buffer with leading dimension m + pad."""
    m, n, dt = case["m"], case["n"], _DT[case["dtype"]]
    buf = _uniform((n, m + case["pad"]), dt, _gen(seed))
    if case["decades"] and n > 1:
        # columns mixed so that the singular values fall over `decades` powers of ten
        gc = torch.Generator(device="cpu")
        gc.manual_seed(int(seed))
        V, _ = torch.linalg.qr(torch.randn((n, n), generator=gc, dtype=torch.float64))
        sigma = 10.0 ** (-case["decades"] * torch.arange(n, dtype=torch.float64) / (n - 1))
        buf = torch.matmul((V * sigma).to(dtype=dt, device="cuda"), buf)
    return buf.t()[:m, :]


def _sizes(case):
    return inputs.batched_sizes(case["count"], case["lo"], case["hi"], case["sizes_seed"])


def _offsets(sizes, n):
    off = np.zeros(len(sizes), dtype=np.int64)
    np.cumsum(sizes[:-1] * n, out=off[1:])
    return off


def prepare(case, seed):
    h = _handle(case)
    n, kind = case["n"], case["kind"]
    if kind == "r":
        A = _matrix(case, seed)
        return {"kind": kind, "A": A, "h": h, "ws": tsqr.workspace(case["m"], n, A.dtype, h=h)}
    if kind == "batch":
        sizes = _sizes(case)
        dt = _DT[case["dtype"]]
        plan = tsqr.BatchPlan(sizes, _offsets(sizes, n), n, dt, h=h)
        return {"kind": kind, "A": _uniform(int(sizes.sum()) * n, dt, _gen(seed)), "plan": plan,
                "R": torch.empty((len(sizes), n, n), dtype=dt, device="cuda")}
    if kind == "qr":
        A = _matrix(case, seed)
        code = tsqr.TSQR_F64 if A.dtype == torch.float64 else tsqr.TSQR_F32
        nbytes = tsqr.tsqr_qr_workspace_bytes(h, case["m"], n, code)
        return {"kind": kind, "A": A, "h": h, "Q": torch.empty((n, case["m"]), dtype=A.dtype, device="cuda").t(),
                "ws": torch.empty(nbytes, dtype=torch.uint8, device="cuda")}
    if kind == "lsq":
        A = _matrix(case, seed)
        return {"kind": kind, "A": A, "h": h, "B": _uniform((case["k"], case["m"]), A.dtype, _gen(seed + 1000003)).t()}
    if kind == "mixed":
        flat, _ = inputs.conditioned_batch_device(torch, case["batch"], case["m"], n, case["decades"], seed)
        plan = tsqr.MixedPlan(case["batch"], case["m"], n, h=h, sample_rows=case["sample_rows"], seed=1)
        return {"kind": kind, "A": flat, "plan": plan,
                "R": torch.empty((case["batch"], n, n), dtype=torch.float64, device="cuda"),
                "flags": torch.empty(case["batch"], dtype=torch.int32, device="cuda")}
    raise ValueError(kind)


def run(state):
    kind = state["kind"]
    if kind == "r":
        return tsqr.geqr_r(state["A"], ws=state["ws"], h=state["h"])
    if kind == "batch":
        return state["plan"].run(state["A"], state["R"])
    if kind == "qr":
        Q, R = tsqr.geqr_qr(state["A"], Q=state["Q"], ws=state["ws"], h=state["h"])
        return {"Q": Q, "R": R}
    if kind == "lsq":
        f = tsqr.Factorization(state["A"], h=state["h"])
        return {"C": f.apply_qt(state["B"]), "R": f.R}
    state["plan"].launch(state["A"], state["R"], state["flags"])
    return {"R": state["R"], "flags": state["flags"]}


def work(case):
    n, kind = case["n"], case["kind"]
    if kind == "batch":
        sizes, w = _sizes(case), _BYTES[case["dtype"]]
        rows = int(sizes.sum())
        return {"bytes": w * (rows * n + case["count"] * n * n), "flops": 2.0 * rows * n * n}
    if kind == "mixed":
        rows = case["batch"] * case["m"]
        return {"bytes": 4 * rows * n + 8 * case["batch"] * n * n, "flops": 2.0 * rows * n * n}
    m, w = case["m"], _BYTES[case["dtype"]]
    b, f = w * (m * n + n * n), 2.0 * m * n * n
    if kind == "qr":        # and Q written, 2 m n^2 more to form it
        b, f = b + w * m * n, 2 * f
    if kind == "lsq":       # and B read, C written, 4 m n k to apply the reflectors
        b, f = b + w * case["k"] * (m + n), f + 4.0 * m * n * case["k"]
    return {"bytes": b, "flops": f}


def _signs(R):
    return torch.where(torch.diagonal(R) < 0, -1.0, 1.0).to(R)


def _r64(A):
    """R with a non-negative diagonal of a float64 device matrix, n x n (zero rows below min(m, n))."""
    m, n = A.shape
    if m * n <= 4000000:
        R = torch.from_numpy(np.linalg.qr(A.cpu().numpy(), mode="r")).cuda()
    else:
        R = torch.linalg.qr(A, mode="r")[1]
    out = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    R = torch.triu(R)
    out[: R.shape[0]] = R * _signs(R)[:, None]
    return out


def _r64_well(A):
    """The same for a well-conditioned matrix (m >= 4 n, uniform entries): Cholesky QR, twice."""
    R = torch.linalg.cholesky(A.t().contiguous() @ A, upper=True)
    Q = torch.linalg.solve_triangular(R, A, upper=True, left=False)
    return torch.linalg.cholesky(Q.t().contiguous() @ Q, upper=True) @ R


def exact(case, seed):
    n, kind = case["n"], case["kind"]
    if kind == "r":
        return _r64(_matrix(case, seed).double()).t().contiguous().t()
    if kind == "batch":
        sizes = _sizes(case)
        flat = _uniform(int(sizes.sum()) * n, _DT[case["dtype"]], _gen(seed))
        out = torch.empty((len(sizes), n, n), dtype=torch.float64, device="cuda")
        for b, (m, o) in enumerate(zip(sizes.tolist(), _offsets(sizes, n).tolist())):
            A = flat[o:o + m * n].view(n, m).t().double()
            well = case["dtype"] == "f32" and m >= 4 * n
            out[b] = (_r64_well(A) if well else _r64(A)).t()
        return out
    if kind == "qr":
        Q, R = torch.linalg.qr(_matrix(case, seed).double())
        if case["m"] < n:
            return None
        s = _signs(R)
        return {"Q": Q * s[None, :], "R": torch.triu(R) * s[:, None]}
    if kind == "lsq":
        if case["m"] < n:
            return None
        Q, R = torch.linalg.qr(_matrix(case, seed).double())
        s = _signs(R)
        B = _uniform((case["k"], case["m"]), _DT[case["dtype"]], _gen(seed + 1000003)).double()
        return {"C": s[:, None] * (Q.t() @ B.t()), "R": torch.triu(R) * s[:, None]}
    flat, _ = inputs.conditioned_batch_device(torch, case["batch"], case["m"], n, case["decades"], seed)
    flat = flat.view(case["batch"], n, case["m"])
    return {"R": torch.stack([_r64(flat[b].t().double()).t() for b in range(case["batch"])]), "flags": None}
