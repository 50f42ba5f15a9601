"""Generated kernels run on the CPU, every access checked against the ends of its buffers, against the oracle."""
import ctypes

import numpy as np
import pytest

from emu_util import Args, Kernels
from oracle import ops, unfused


@pytest.fixture(scope="module")
def F():
    import paper_1801_00829_amd as F
    from paper_1801_00829_amd import build as B
    if B.needs_build():
        B.build()
    return F


def _ptr(a):
    return a.ctypes.data


# ------------------------------------------------------------------ outer products, row runs --

def _run_row_runs(F, folder, monkeypatch, body, kind, transposed, r, rb, blocks, mask, rp64=False, width=3, last_first=False, row_limit=None):
    """RIGHT_MM over the cells that `mask` (m x n) has, with one side input of that kind: through the preparatory kernel, the main
    one with `blocks` blocks, and the one for long rows.  transposed: the kernels' LEFT_MM build, over the transposed matrix.  Returns
    (result, oracle)."""
    monkeypatch.setenv("FUSE_OUTER_PANELS", "2")
    monkeypatch.setenv("FUSE_OUTER_RUNS", "2")
    monkeypatch.setenv("FUSE_OUTER_RB", str(rb))
    m, n = mask.shape
    rng = np.random.default_rng(17 + m + n + r)
    rp, ci = np.concatenate([[0], np.cumsum(mask.sum(1))]), np.nonzero(mask)[1].astype(np.int32)
    va = rng.uniform(0.1, 1.0, len(ci))
    x = ops.make_csr(rp, ci, va, (m, n))
    u, v = rng.uniform(size=(m, r)), rng.uniform(size=(n, r))
    side = rng.uniform(size={"matrix": (m, n), "colvec": (m, 1), "rowvec": (1, n)}[kind])
    agg = "left_mm" if transposed else "right_mm"
    F.cache_clear()                                 # (the source of the last plan that was compiled is wanted)
    F.prepare_outer(body, (m, n), r, max(len(ci), 1), [(kind, None)], agg, rp64)
    name = F.last_kernel()
    k = Kernels(F.last_source(), folder, [name, "fuse_outer_prep", "fuse_outer_rows"])
    assert k.define("FUSE_PANELS") == 4 and k.define("FUSE_TRANSPOSED") == int(transposed)
    if transposed:                                  # the walked matrix: the columns of X, factors exchanged
        order = np.argsort(ci, kind="stable")
        rows = np.repeat(np.arange(m), np.diff(rp))
        wrp = np.concatenate([[0], np.cumsum(np.bincount(ci, minlength=n))])
        wci, wva, wm, wn, wu, wv = rows[order], va[order], n, m, v, u
    else:
        wrp, wci, wva, wm, wn, wu, wv = rp, ci, va, m, n, u, v
    a = Args()
    keep = dict(x=k.copy(wva, np.float64), colidx=k.copy(wci, np.int32), rowptr=k.copy(wrp, np.int64 if rp64 else np.int32), u=k.copy(wu), v=k.copy(wv),
                out=k.copy(np.full((wm, r), np.nan)), ticket=k.buffer(64, np.uint32), partials=k.buffer(64))
    for f, b in keep.items():
        setattr(a, f, _ptr(b))
    s = k.copy(side)
    a.side[0], a.side_ld[0] = _ptr(s), s.shape[1]
    a.ldu = a.ldv = a.rank = r
    a.m, a.n, a.nnz = wm, wn, len(wci)
    P = (wn + width - 1) // width
    pp = k.buffer((wm, P + 1), np.int64 if rp64 else np.int32)
    a.npanels, a.panel_w, a.panel_ptr, a.block_rows = P, width, _ptr(pp), rb
    a.row_limit = len(wci) if row_limit is None else row_limit
    k.run("fuse_outer_prep", a, (wm * 16 + 255) // 256, 256, last_first)
    k.run(name, a, blocks, k.define("FUSE_BLOCK"), last_first)
    if row_limit is not None:                       # the rows within the limit are complete, and nothing is handed on
        short = np.diff(wrp) <= row_limit
        want = unfused.outer(body, x, u, v, [(kind, side)], agg).reshape(wm, r)
        err = np.abs(keep["out"] - want)[short].max(initial=0.0)
        assert err <= 1e-12 * np.abs(want).max() and not keep["ticket"].any()
    k.run("fuse_outer_rows", a, 3, k.define("FUSE_ROWS_BLOCK"), last_first)
    return keep["out"].copy(), unfused.outer(body, x, u, v, [(kind, side)], agg)


@pytest.mark.parametrize("kind,transposed", [("matrix", False), ("colvec", False), ("matrix", True), ("rowvec", True)])
def test_row_runs_read_side_inputs_of_existing_cells_only(F, tmp_path, monkeypatch, kind, transposed):
    """More blocks than the rows fill: 11 rows, 4 per block, 5 blocks, of which the last two have none."""
    mask = np.random.default_rng(3).uniform(size=(2, 11) if transposed else (11, 9)) < 0.6
    if transposed:
        mask[:, 0] = False, True                    # the walked matrix' first cell lies in the last row of the side
    body = [("uvdot",), ("main",), ("mul",), ("side", 0), ("add",)]
    got, want = _run_row_runs(F, tmp_path, monkeypatch, body, kind, transposed, 33, 4, 5, mask, width=1 if transposed else 3)
    err = np.abs(got - want.reshape(got.shape)).max()
    assert err <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("rp64", [False, True])
def test_row_runs_in_either_order_of_the_lanes(F, tmp_path, monkeypatch, rp64, transposed):
    """Lanes that run from the last one on between two meeting points: what one lane reads from LDS that another one of its wave
    has written needs a barrier of the wave in between (the first panels' books)."""
    rng = np.random.default_rng(4)
    mask = rng.uniform(size=(23, 60)) < 0.4
    if transposed:
        mask = mask.T.copy()
    body = [("uvdot",), ("main",), ("mul",), ("side", 0), ("add",)]
    got, want = _run_row_runs(F, tmp_path, monkeypatch, body, "rowvec" if transposed else "colvec", transposed, 100, 11, 2, mask, rp64, 7, True)
    err = np.abs(got - want.reshape(got.shape)).max()
    assert err <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("r", [33, 100])
def test_row_runs_give_away_the_long_rows_only(F, tmp_path, monkeypatch, r, transposed):
    """Rows beyond the limit -- the first, neighbours, the last, one without a rest for the waves -- are summed by the kernel
    behind the row runs, all others by the row runs."""
    rng = np.random.default_rng(6)
    mask = rng.uniform(size=(31, 70)) < 0.1
    mask[[0, 11, 12, 30]] = rng.uniform(size=(4, 70)) < 0.8
    mask[20] = True
    mask[5] = False
    body = [("uvdot",), ("main",), ("mul",), ("side", 0), ("add",)]
    got, want = _run_row_runs(F, tmp_path, monkeypatch, body, "matrix", transposed, r, 8, 2, mask.T.copy() if transposed else mask, width=9,
                              row_limit=30)
    err = np.abs(got - want.reshape(got.shape)).max()
    assert err <= 1e-12 * np.abs(want).max()


# --------------------------------------------------- matrix units over CSR rows, pipelined form --

_Q = [("side", 1), ("main",), ("side", 0), ("matmult",), ("mul",)]
MLOGREG = [("main",)] + _Q + [("side", 1)] + _Q + [("rowsum",), ("mul",), ("sub",), ("outerk",)]


def _run_csr_tiles(F, folder, monkeypatch, mask, k, pipe=True, expr=MLOGREG, rp64=False, before=0, blocks=2, change=None, last_first=False):
    """t(X) %*% f(X %*% V) over the cells that `mask` has, in CSR arrays that hold `before` cells in front of them, in the
    pipelined or the block form.  change(values): other operands.  Returns (result, oracle)."""
    monkeypatch.setenv("FUSE_MFMA_PIPE", "3" if pipe else "0")
    monkeypatch.setenv("FUSE_MFMA_CSR_DENSITY", "1")
    m, n = mask.shape
    rng = np.random.default_rng(n + k)
    rp = before + np.concatenate([[0], np.cumsum(mask.sum(1))])
    ci = np.nonzero(mask)[1]
    vals = {"x": rng.uniform(0.1, 1.0, len(ci)), "v": rng.normal(size=(n, k)), "p": rng.uniform(size=(m, k))}
    if change:
        change(vals)
    F.cache_clear()
    F.prepare_row(expr, (m, n), [("rhs", (n, k)), ("kvec", (m, k))], "col_t", nnz=len(ci), rowptr64=rp64)
    name = F.last_kernel()
    assert name.startswith("fuse_row_mfma_") and ("_pipe_" in name) == pipe
    kern = Kernels(F.last_source(), folder, [name])
    a = Args()
    side = [kern.copy(vals["v"]), kern.copy(vals["p"])]
    rowptr, part = kern.copy(rp, np.int64 if rp64 else np.int32), kern.buffer((blocks, n, k))
    x, colidx = kern.buffer(before + len(ci)), kern.buffer(before + len(ci), np.int32)
    x[before:], colidx[before:] = vals["x"], ci
    a.x, a.colidx, a.rowptr, a.partials = _ptr(x), _ptr(colidx), _ptr(rowptr), _ptr(part)
    a.m, a.n, a.ld, a.nnz = m, n, n, before + len(ci)
    for q, s in enumerate(side):
        a.side[q], a.side_ld[q] = _ptr(s), k
    kern.run(name, a, blocks, (kern.define("FUSE_NWAVE") + int(pipe)) * 64, last_first)
    with np.errstate(all="ignore"):
        want = unfused.row_csr(expr, ops.make_csr(rp - before, ci, vals["x"], (m, n)), [("rhs", vals["v"]), ("kvec", vals["p"])], "col_t")
        return part.sum(0), want.reshape(n, k)


def test_csr_cells_at_the_end_of_32_bit_offsets(F, tmp_path, monkeypatch):
    """The last cells of a matrix with 2^31 - 1 stored ones and 32-bit row offsets (address space only)."""
    mask = np.random.default_rng(8).uniform(size=(41, 130)) < 0.2
    got, want = _run_csr_tiles(F, tmp_path, monkeypatch, mask, 5, before=2 ** 31 - 1 - int(mask.sum()))
    err = np.abs(got - want).max()
    assert err <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("where", ["v", "v, hidden", "p", "x", "nowhere"])
@pytest.mark.parametrize("pipe", [True, False])
def test_csr_tiles_multiply_stored_cells_only(F, tmp_path, monkeypatch, pipe, where):
    """An infinity in V reaches the rows that store its column, one in P or X the columns that its row stores; tiles that are
    full, and one that is not.  "hidden": a body with a comparison, whose sums are finite whatever V holds."""
    hidden = [("main",), ("main",), ("side", 0), ("matmult",), ("const", 0.0), ("gt",), ("side", 1), ("mul",), ("outerk",)]
    mask = np.random.default_rng(9).uniform(size=(53, 130)) < 0.15
    mask[:, 7] = False
    mask[[3, 50], 7] = True
    mask[40] = False

    def change(vals):
        if where.startswith("v"):
            vals["v"][7, 2] = np.inf
        elif where == "p":
            vals["p"][17, 1], vals["p"][52, 4], vals["p"][40, 0] = np.nan, np.inf, np.inf
        elif where == "x":
            vals["x"][100] = np.nan

    got, want = _run_csr_tiles(F, tmp_path, monkeypatch, mask, 6, pipe, hidden if where == "v, hidden" else MLOGREG, change=change)
    finite = np.isfinite(want)
    assert (where in ("nowhere", "v, hidden")) == finite.all() and finite.any()
    assert np.array_equal(finite, np.isfinite(got)) and np.array_equal(np.isnan(want), np.isnan(got))
    err = np.abs(got - want)[finite].max()
    assert err <= 1e-12 * np.abs(want[finite]).max()
