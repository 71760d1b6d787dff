"""The four-column panels of the leaves, merges and Q passes, and the Gram pass
of the mixed-precision correction, at the sizes where they can go wrong: the
edges of the compiled column widths (8, 24, 40 among them), one to seven leaves
(one launch without counters up to four, the last group partly filled, the
first tree level through memory), a ragged last chunk, panels that have to be
done one column at a time, leaves cut shorter so that a batch fills the device, and row counts around
the 16-row tiles of the Gram pass.

Tolerances: the backward-error gates of ``gates`` (they hold at any condition
number), and 900 u for Q R = A, Q^T A = R and the orthogonality of Q, the bound
that the Q tests use in FP64 (1e-13).  Orthogonality is asked for where A has
well-conditioned columns only: the first chunk is stacked under a zero block,
which Q leaves out, so Q's columns for dependent columns of A have rows there
(a zero column of A gives a zero column of Q).
"""
import numpy as np
import pytest

import oracle
from gates import GRAM32, GRAM64
from paper_1002_4250_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1002_4250_amd import tsqr  # noqa: E402

DT = {"f64": (np.float64, GRAM64, 1e-13), "f32": (np.float32, GRAM32, 900 * 2.0 ** -24)}


def relF(X, Y):
    return float(np.linalg.norm(X - Y) / max(np.linalg.norm(Y), 1e-300))


def to_dev(A):
    return torch.from_numpy(np.ascontiguousarray(A.T)).cuda().t()


def check_r_and_q(A, leaf_rows, gram, tol, orthogonal=True):
    """R and Q of A against the oracle's gates, and R the same bit for bit from every entry point."""
    n = A.shape[1]
    h = tsqr.handle(0)
    tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, leaf_rows)
    try:
        Ad = to_dev(A)
        R = tsqr.geqr_r(Ad).cpu().numpy()
        Q, Rq = (x.cpu().numpy() for x in tsqr.geqr_qr(Ad))
        f = tsqr.Factorization(Ad)
        QtA = f.apply_qt(Ad).cpu().numpy().astype(np.float64)
        Rf = f.R.cpu().numpy()
    finally:
        tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, 0)
    assert np.array_equal(R, Rq) and np.array_equal(R, Rf)
    assert np.all(np.tril(R, -1) == 0) and not np.any(np.signbit(np.diag(R)))
    A, Q, R = A.astype(np.float64), Q.astype(np.float64), R.astype(np.float64)
    assert oracle.gram_residual(A, R) < gram
    if orthogonal:
        assert np.linalg.norm(Q.T @ Q - np.eye(n)) / np.sqrt(n) < tol
    assert relF(Q @ R, A) < tol
    assert relF(QtA, R) < tol


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", [4, 5, 9, 12, 13, 17, 20, 21, 28, 33, 36, 37, 44, 45, 48, 51, 52, 57, 60])
def test_panels_past_the_last_column(n, dt):
    """Counts that leave panels of their width without a column, in leaves, merges
    and Q passes; the workspace holds NaN where nothing is written."""
    npdt, gram, tol = DT[dt]
    A = inputs.uniform(900, n, 800 + n, npdt)
    check_r_and_q(A, 128, gram, tol)
    h, Ad = tsqr.handle(0), to_dev(A)
    nbytes = tsqr.tsqr_qr_workspace_bytes(h, 900, n, tsqr.TSQR_F64 if dt == "f64" else tsqr.TSQR_F32)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    Q, R = (x.cpu().numpy().astype(np.float64) for x in tsqr.geqr_qr(Ad, ws=ws))
    assert relF(Q @ R, A.astype(np.float64)) < tol


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,leaves", [(8, 1), (8, 3), (9, 2), (24, 4), (24, 5), (25, 1), (40, 2), (40, 5), (41, 3),
                                      (41, 4), (3, 5), (64, 3), (50, 7)])
def test_widths_and_leaf_counts(n, leaves, dt):
    npdt, gram, tol = DT[dt]
    A = inputs.uniform(128 * leaves - 37, n, 700 + n, npdt)
    check_r_and_q(A, 128, gram, tol)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,m", [(12, 300), (50, 900)])
@pytest.mark.parametrize("kind", ["equal", "close", "closer", "zero", "graded"])
def test_cut_panels(n, m, kind, dt):
    npdt, gram, tol = DT[dt]
    rng = np.random.default_rng(n)
    A = rng.uniform(-1, 1, (m, n))
    eps = float(np.finfo(npdt).eps)
    for j in range(1, n, 3):                         # within panels and across their edges
        noise = rng.uniform(-1, 1, m)
        if kind == "equal":
            A[:, j] = A[:, j - 1]
        elif kind == "close":
            A[:, j] = A[:, j - 1] + eps ** 0.25 * noise
        elif kind == "closer":
            A[:, j] = 2.0 * A[:, j - 1] + eps ** 0.75 * noise
        elif kind == "zero":
            A[:, j] = 0.0
        else:
            A[:, j] *= eps ** (j / n)
    check_r_and_q(np.asfortranarray(A.astype(npdt)), 128, gram, tol, orthogonal=False)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", [4, 8, 15])
@pytest.mark.parametrize("leaf_rows", [256, 128])    # the two blocks as chunks of a leaf, and as leaves that merge
def test_columns_dependent_in_the_lower_block_only(n, leaf_rows, dt):
    """Below, column 4 i + 1 is column 4 i plus e times column 4 i + 2; above, it
    has a large part of its own, so that R's diagonal hides how little is left
    of it below.  What is left has inner products with the later columns."""
    npdt, gram, tol = DT[dt]
    e = 3e-9 if dt == "f64" else 1e-4
    for seed in range(8):
        rng = np.random.default_rng(100 + seed)
        A = rng.uniform(-1, 1, (256, n))
        for j in range(0, n - 2, 4):
            top, u = A[:128, j], A[:128, j + 1]
            A[:128, j + 1] = top + u - top * (top @ u) / (top @ top)
            A[128:, j + 1] = A[128:, j] + e * A[128:, j + 2]
        check_r_and_q(np.asfortranarray(A.astype(npdt)), leaf_rows, gram, tol)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", [8, 23, 50])
def test_zero_column_under_a_diagonal(n, dt):
    """Columns that are zero from the second chunk on keep their rows of R up to
    a reflection, the same in every entry point."""
    npdt, gram, tol = DT[dt]
    A = inputs.uniform(700, n, 60 + n, npdt)
    for j in (0, 2, 5, n - 1):
        A[128:, j] = 0
    for leaf_rows in (1024, 128):
        check_r_and_q(A, leaf_rows, gram, tol)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", [5, 12, 16, 20, 41, 50, 64])
@pytest.mark.parametrize("leaf_rows", [1024, 256, 128])
def test_close_columns_in_some_chunks(n, leaf_rows, dt):
    """Panels done one column at a time, in leaves (where that is kept from chunk
    to chunk until the columns are apart again) and in merges of triangles that
    are both close, or one of them."""
    npdt, gram, tol = DT[dt]
    rng = np.random.default_rng(n)
    V, _ = np.linalg.qr(rng.standard_normal((n, n)))
    close = rng.uniform(-1, 1, (384, n)) * (10.0 ** (-(6 if dt == "f64" else 3) * np.arange(n) / n)) @ V.T
    A = np.concatenate([close, rng.uniform(-1, 1, (391, n)), close[:250]])
    check_r_and_q(np.asfortranarray(A.astype(npdt)), leaf_rows, gram, tol)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,col", [(8, 5), (12, 1), (20, 7), (50, 0), (50, 5), (50, 24), (64, 63)])
@pytest.mark.parametrize("leaf_rows", [1024, 128])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_not_finite_column(n, col, leaf_rows, dt, value):
    """A NaN or an infinity in a column stays out of the rows of R before it,
    but for its own column, wherever in A it is; everything after is not finite,
    the diagonal (of which the contract says nothing) left aside."""
    npdt, _, _ = DT[dt]
    rows, cols = np.triu_indices(n)
    above = (rows < col) & (cols != col)
    for row in (3, 400, 899):
        A = inputs.uniform(900, n, 31, npdt)
        B = A.copy()
        A[:, col] = 0
        B[row, col] = value
        h = tsqr.handle(0)
        tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, leaf_rows)
        try:
            R = tsqr.geqr_r(to_dev(B)).cpu().numpy()[rows, cols]
        finally:
            tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, 0)
        ref = oracle.r_factor(np.asfortranarray(A.astype(np.float64)))[rows, cols]
        assert np.all(np.abs(R[above] - ref[above]) < (1e-10 if dt == "f64" else 1e-3))
        assert not np.any(np.isfinite(R[(rows >= col) & (cols > rows)]))


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("sizes", [(30000,), (8192, 8193, 64, 20000, 1), (70000, 300)])
def test_batch_leaves_fill_the_device(sizes, dt):
    npdt, gram, _ = DT[dt]
    n = 30
    offsets = [int(o) for o in np.concatenate(([0], np.cumsum(sizes)[:-1])) * n]
    A = [inputs.uniform(m, n, 900 + m, npdt) for m in sizes]
    flat = np.concatenate([np.ascontiguousarray(a.T).reshape(-1) for a in A])
    plan = tsqr.BatchPlan(list(sizes), offsets, n, torch.from_numpy(flat).dtype)
    _, _, leaf_rows = plan.info()
    assert 0 < leaf_rows < 8192                      # shorter than on a batch that fills the device by itself
    R = plan.run(torch.from_numpy(flat).cuda()).cpu().numpy()
    h = tsqr.handle(0)
    tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, leaf_rows)
    try:
        single = [tsqr.geqr_r(to_dev(a)).cpu().numpy() for a in A]
    finally:
        tsqr.tsqr_set_option(h, tsqr.TSQR_OPT_LEAF_ROWS, 0)
    for b, a in enumerate(A):
        assert np.array_equal(R[b].T, single[b]), b
        assert oracle.gram_residual(a.astype(np.float64), R[b].T.astype(np.float64)) < gram, b


@pytest.mark.parametrize("n,m", [(8, 1025), (9, 1039), (24, 1024), (33, 1040), (40, 1055), (50, 1056), (50, 1057),
                                 (64, 2049), (64, 2071), (50, 40)])
def test_mixed_gram_tiles(n, m):
    batch = 3
    A = [inputs.uniform(m, n, 40 + b, np.float32) for b in range(batch)]
    if m == 40:                                      # ten rows twice: rank 40, the FP64 path may take over
        A = [np.concatenate([a, a[:10]]) for a in A]
    rows = A[0].shape[0]
    flat = np.concatenate([np.ascontiguousarray(a.T).reshape(-1) for a in A])
    plan = tsqr.MixedPlan(batch, rows, n)
    R, fb = plan.run(torch.from_numpy(flat).cuda())
    R = R.cpu().numpy()
    for b, a in enumerate(A):
        a64 = np.asfortranarray(a.astype(np.float64))
        assert oracle.gram_residual(a64, R[b].T) < GRAM64, b
        if m > 40:
            assert int(fb[b]) == 0, b
            assert relF(R[b].T, oracle.r_factor(a64)) < 1e-12, b
