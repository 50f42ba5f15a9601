"""The calls this library is measured on: fused operators of every template over the sizes they are used at.

Sizes and expressions are those of the benchmark (``workloads/configs.py``), of its timing sweep (``bench.py --sweep``:
the micro-benchmark figures and the dataset shapes of the paper's tables) and of the tests; a drawn case takes one of the
same operators at other sizes of the same ranges, odd ones included.  Everything is fp64, the only type of the library;
CSR matrices have int32 column indices and int32 or int64 row offsets, and row lengths that are binomial (cells stored
independently) or heavy-tailed (``skew``: log-normal, as counts per user or per document are).
"""
import math

import torch

import paper_1801_00829_amd as F

MAIN, MUL, SUB = ("main",), ("mul",), ("sub",)
SIDE0, SIDE1 = ("side", 0), ("side", 1)

XYZ = [MAIN, SIDE0, MUL, SIDE1, MUL]                                        # X * Y * Z per cell
XY_XZ_XX = [[MAIN, SIDE0, MUL], [MAIN, SIDE1, MUL], [MAIN, ("pow2",)]]      # three aggregates over shared inputs
TX_W_XV = [MAIN, SIDE0, ("dot",), SIDE1, MUL, MAIN, MUL]                    # t(X) (w * (X v)) as a column aggregate
TX_XV = [MAIN, SIDE0, ("dot",), MAIN, MUL]                                  # t(X) (X v)
_Q = [SIDE1, MAIN, SIDE0, ("matmult",), MUL]                                # Q = P * (X V)
MLOGREG = [MAIN] + _Q + [SIDE1] + _Q + [("rowsum",), MUL, SUB, ("outerk",)]  # t(X) (Q - P * rowSums(Q))
X_LOG_UV = [MAIN, ("uvdot",), ("const", 1e-15), ("add",), ("log",), MUL]    # X * log(U t(V) + eps)
ALS_UPDATE = [MAIN, ("neq0",), ("uvdot",), MUL]                             # (X != 0) * (U t(V))


def listed():
    return [
        # one Cell operator inside an iterative program on a small matrix: latency counts
        dict(name="cell_sum_small", op="cell_sum", rows=1000, cols=1000),
        # the same template with a matrix result and vector sides (centring / scaling), rows of odd length
        dict(name="cell_map_odd", op="cell_map", rows=99991, cols=1001),
        # several aggregates in one scan of three large matrices
        dict(name="magg_large", op="magg", rows=100000, cols=1000),
        # one step of a linear model's solver on a small matrix: latency counts
        dict(name="row_small", op="row_vec", rows=1000, cols=1000),
        # the same on a tall matrix
        dict(name="row_tall", op="row_vec", rows=1000000, cols=100),
        # the same on a very tall matrix of few, odd columns (the airline shape)
        dict(name="row_narrow_odd", op="row_vec", rows=14000000, cols=29),
        # gradient / Hessian product of multinomial logistic regression, 10 classes, dense digit images
        dict(name="classes_dense", op="classes", rows=1000000, cols=784, classes=10),
        # one solver step over a sparse matrix with short rows
        dict(name="csr_vec", op="csr_vec", rows=10000000, cols=1000, density=0.01, skew=0.0, wide=False),
        # logistic regression over digit images in sparse form: a quarter of the cells stored
        dict(name="csr_classes", op="csr_classes", rows=1000000, cols=784, density=0.25, skew=0.0, wide=False, classes=10),
        # an element-wise aggregate over three sparse matrices
        dict(name="csr_sparse_sides", op="csr_sides", rows=1000000, cols=1000, density=0.1, skew=0.0, wide=False),
        # loss of a factorization over the stored ratings
        dict(name="outer_loss", op="outer_loss", rows=100000, cols=100000, density=0.001, skew=0.0, wide=False, rank=100),
        # both half steps of an alternating-least-squares iteration: the update of the row factors (right_mm) and of the
        # column factors (left_mm over the pattern that the program sorted once)
        dict(name="outer_updates", op="outer_updates", rows=100000, cols=100000, density=0.001, skew=0.0, wide=False, rank=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["cell_sum", "cell_map", "magg", "row_vec", "row_vec", "classes", "csr_vec", "csr_vec", "csr_classes",
                     "csr_sides", "outer_loss", "outer_updates"])
    if op in ("cell_sum", "cell_map", "magg"):
        cells, cols = _log_int(rng, 10000, 100000000), _log_int(rng, 10, 4000)
        return dict(op=op, rows=max(1, cells // cols), cols=cols)
    if op == "row_vec":
        cells, cols = _log_int(rng, 30000, 400000000), _log_int(rng, 8, 2000)
        return dict(op=op, rows=max(1, cells // cols), cols=cols)
    if op == "classes":
        cells, cols = _log_int(rng, 1000000, 600000000), _log_int(rng, 16, 1000)
        return dict(op=op, rows=cells // cols, cols=cols, classes=rng.randint(2, 16))
    skew = rng.choice([0.0, 0.0, 1.0])
    wide = rng.random() < 0.25
    if op == "csr_vec":
        cells, cols, per_row = _log_int(rng, 100000, 100000000), _log_int(rng, 100, 20000), _log_int(rng, 2, 200)
        per_row = min(per_row, cols / 2.0)
        return dict(op=op, rows=max(1, int(cells / per_row)), cols=cols, density=per_row / cols, skew=skew, wide=wide)
    if op == "csr_classes":
        classes, cols, density = rng.randint(2, 16), _log_int(rng, 100, 1000), math.exp(rng.uniform(math.log(0.01), math.log(0.3)))
        cells = _log_int(rng, 500000, 800000000 // classes)
        return dict(op=op, rows=int(cells / (cols * density)), cols=cols, density=density, skew=skew, wide=wide, classes=classes)
    if op == "csr_sides":
        cols, density = _log_int(rng, 100, 2000), math.exp(rng.uniform(math.log(0.02), math.log(0.2)))
        cells = _log_int(rng, 100000, 80000000)
        return dict(op=op, rows=int(cells / (cols * density)), cols=cols, density=density, skew=skew, wide=wide)
    rows, cols, per_row, rank = _log_int(rng, 2000, 120000), _log_int(rng, 2000, 120000), _log_int(rng, 10, 200), rng.randint(10, 110)
    per_row = min(per_row, 8000000 // rows)
    return dict(op=op, rows=rows, cols=cols, density=per_row / cols, skew=skew, wide=wide, rank=rank)


def _uniform(g, lo, hi, *shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda").uniform_(lo, hi, generator=g)


def _normal(g, *shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda").normal_(generator=g)


def _csr(g, case):
    """CSR with ascending distinct columns: row lengths first, then the ordered places of that many cells in a row.
    All sums are over whole numbers, so the matrix depends on the seed alone; values lie in (0, 1]."""
    m, n, d, skew = case["rows"], case["cols"], case["density"], case["skew"]
    if skew:
        lens = n * d * torch.exp(skew * _normal(g, m) - skew * skew / 2)
    else:
        lens = n * d + math.sqrt(n * d * (1.0 - d)) * _normal(g, m)
    lens = lens.round_().clamp_(0, n).to(torch.int64)
    ends = torch.cumsum(lens, 0)
    nnz = int(ends[-1])
    starts = ends - lens
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), lens, output_size=nnz)
    gaps = torch.empty(nnz, dtype=torch.float64, device="cuda").exponential_(generator=g).mul_(1 << 20).to(torch.int64)
    last = torch.empty(m, dtype=torch.float64, device="cuda").exponential_(generator=g).mul_(1 << 20).to(torch.int64) + 1
    place = torch.zeros(nnz + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(gaps, 0, out=place[1:])
    del gaps
    base, total = place[starts], place[ends] - place[starts] + last
    place = place[1:] - base[row]
    colidx = (place.double() / total[row] * (n - lens + 1)[row]).to(torch.int64)
    del place
    colidx += torch.arange(nnz, device="cuda") - starts[row]
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), ends])
    vals = 1.0 - torch.empty(nnz, dtype=torch.float64, device="cuda").uniform_(generator=g)
    return F.Csr(rowptr if case["wide"] else rowptr.to(torch.int32), colidx.to(torch.int32), vals, (m, n))


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op, m, n = case["op"], case["rows"], case["cols"]
    if op == "cell_sum":
        return dict(op=op, x=_uniform(g, 0, 1, m, n), sides=[("matrix", _uniform(g, 0, 1, m, n)), ("matrix", _uniform(g, 0, 1, m, n))])
    if op == "cell_map":
        return dict(op=op, x=_normal(g, m, n), sides=[("colvec", _uniform(g, 0, 1, m)), ("rowvec", _uniform(g, 0, 1, n))])
    if op == "magg":
        return dict(op=op, x=_uniform(g, -1, 1, m, n), sides=[("matrix", _uniform(g, -1, 1, m, n)), ("matrix", _uniform(g, -1, 1, m, n))])
    if op == "row_vec":
        return dict(op=op, x=_normal(g, m, n), sides=[("rowvec", _normal(g, n)), ("colvec", _uniform(g, 0, 1, m))])
    if op in ("classes", "csr_classes"):
        k = case["classes"]
        x = _normal(g, m, n) if op == "classes" else _csr(g, case)
        return dict(op=op, x=x, sides=[("rhs", _normal(g, n, k)), ("kvec", torch.softmax(_normal(g, m, k), 1))])
    if op == "csr_vec":
        return dict(op=op, x=_csr(g, case), sides=[("rowvec", _normal(g, n))])
    if op == "csr_sides":
        return dict(op=op, x=_csr(g, case), sides=[("sparse", _csr(g, case)), ("sparse", _csr(g, case))])
    r = case["rank"]
    if op == "outer_loss":
        return dict(op=op, x=_csr(g, case), u=_uniform(g, 0, 1, m, r), v=_uniform(g, 0, 1, n, r))
    x = _csr(g, case)
    return dict(op=op, x=x, u=_normal(g, m, r), v=_normal(g, n, r), pattern=F.outer_left_prepare(x))


def run(s):
    op = s["op"]
    if op == "cell_sum":
        return F.fuse_cell(XYZ, s["x"], s["sides"], "full")
    if op == "cell_map":
        return F.fuse_cell(XYZ, s["x"], s["sides"], "none")
    if op == "magg":
        return F.fuse_magg(XY_XZ_XX, s["x"], s["sides"])
    if op == "row_vec":
        return F.fuse_row(TX_W_XV, s["x"], s["sides"], "col_t")
    if op in ("classes", "csr_classes"):
        return F.fuse_row(MLOGREG, s["x"], s["sides"], "col_t")
    if op == "csr_vec":
        return F.fuse_row(TX_XV, s["x"], s["sides"], "col_t")
    if op == "csr_sides":
        return F.fuse_cell_csr(XYZ, s["x"], s["sides"], "full")
    if op == "outer_loss":
        return F.fuse_outer(X_LOG_UV, s["x"], s["u"], s["v"], [], "full")
    return (F.fuse_outer(ALS_UPDATE, s["x"], s["u"], s["v"], [], "right_mm"),
            F.fuse_outer_left(ALS_UPDATE, s["x"], s["pattern"], s["u"], s["v"]))


def work(case):
    """Inputs once, outputs once; multiplications and additions of the expression."""
    op, m, n = case["op"], case["rows"], case["cols"]
    if op in ("cell_sum", "magg"):
        return {"bytes": 24 * m * n, "flops": (3 if op == "cell_sum" else 6) * m * n}
    if op == "cell_map":
        return {"bytes": 16 * m * n + 8 * (m + n), "flops": 2 * m * n}
    if op == "row_vec":
        return {"bytes": 8 * m * n + 8 * m + 16 * n, "flops": 4 * m * n + m}
    if op == "classes":
        k = case["classes"]
        return {"bytes": 8 * m * n + 8 * m * k + 16 * n * k, "flops": 4 * m * n * k + 4 * m * k}
    cells, offset = int(m * n * case["density"]), 8 if case["wide"] else 4
    stored = 12 * cells + offset * (m + 1)
    if op == "csr_vec":
        return {"bytes": stored + 16 * n, "flops": 4 * cells}
    if op == "csr_classes":
        k = case["classes"]
        return {"bytes": stored + 8 * m * k + 16 * n * k, "flops": 4 * cells * k + 4 * m * k}
    if op == "csr_sides":
        return {"bytes": 3 * stored, "flops": int(3 * cells * case["density"])}
    r = case["rank"]
    if op == "outer_loss":
        return {"bytes": stored + 8 * r * (m + n), "flops": cells * (2 * r + 3)}
    # two calls: the values and the column offsets of X are read in row order and in column order
    return {"bytes": 2 * stored + 3 * 8 * r * (m + n), "flops": 2 * cells * (4 * r + 1)}


def tolerance(case):
    """Four times the largest difference seen between this path and the same expression evaluated by torch in fp64
    operator by operator, i.e. with its sums in another order (listed cases and fourteen drawn ones): single sums and
    element-wise results 2e-16 (their tolerance leaves room for another order within a thread), products 9e-15
    (largest value 2.5e-14), class gradients 2.7e-14 (1e-13), factor updates 7e-16 (6.3e-15)."""
    op = case["op"]
    if op in ("row_vec", "csr_vec"):
        return {"rel": 4e-14, "max": 1e-13}
    if op in ("classes", "csr_classes"):
        return {"rel": 1e-13, "max": 4e-13}
    if op == "outer_updates":
        return {"rel": 4e-15, "max": 2.5e-14}
    return {"rel": 1e-14}
