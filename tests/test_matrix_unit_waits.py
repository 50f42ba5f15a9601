"""Results of the fp64 matrix instructions are not interlocked: a vector instruction that reads one needs 6 wait states behind a
4x4x4 product (11 behind a 16x16x4 one), a load or store that takes it 9 (18), and the compiler has to put them there.  It has
been seen not to where it merged two branches and copied the results of products behind the jump (2 to 5 wait states, wrong sums
in the last column tile).  So the code objects are looked through, along every path behind a product."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_Q = [("side", 1), ("main",), ("side", 0), ("matmult",), ("mul",)]
MLOGREG = [("main",)] + _Q + [("side", 1)] + _Q + [("rowsum",), ("mul",), ("sub",), ("outerk",)]


def _operands(text):
    return re.split(r",\s*(?![^\[]*\])", text) if text else []


def _regs(operand):
    m = re.match(r"[-|]*v(?:\[(\d+):(\d+)\]|(\d+)\b)", operand.strip())
    if not m:
        return frozenset()
    lo, hi = (m[1], m[2]) if m[1] else (m[3], m[3])
    return frozenset(range(int(lo), int(hi) + 1))


def _instructions(path, tmp):
    data = open(path, "rb").read()
    elf = os.path.join(str(tmp), "code.elf")
    with open(elf, "wb") as f:
        f.write(data[data.index(b"\x7fELF"):])
    out = subprocess.run([OBJDUMP, "-d", elf], capture_output=True, text=True, check=True).stdout
    found = []
    for line in out.splitlines():
        m = re.match(r"^\t(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):", line)
        if m:
            found.append((int(m[3], 16), m[1], m[2]))
    return found


def early_readers(instructions):
    """(wait states, needed, product, reader) for every reader of a product's result that comes too early."""
    at = {a: i for i, (a, _, _) in enumerate(instructions)}

    def behind(i):
        a, op, args = instructions[i]
        if op == "s_endpgm":
            return []
        following = [i + 1] if i + 1 < len(instructions) else []
        if op.startswith(("s_branch", "s_cbranch")):
            off = int(args.split()[0])
            target = at.get(a + 4 + 4 * (off - 65536 if off > 32767 else off))
            return ([] if op == "s_branch" else following) + ([target] if target is not None else [])
        return following

    early = []
    for i, (_, op, args) in enumerate(instructions):
        if not op.startswith("v_mfma_f64"):
            continue
        need_vector, need_memory = (11, 18) if "16x16" in op else (6, 9)
        work, seen = [(j, 0, _regs(_operands(args)[0])) for j in behind(i)], set()
        while work:
            j, states, live = work.pop()
            if states >= need_memory or not live or (j, states, live) in seen:
                continue
            seen.add((j, states, live))
            o, ops = instructions[j][1], _operands(instructions[j][2])
            memory = o.startswith(("ds_", "global_", "buffer_", "flat_", "scratch_"))
            stores = memory and not re.search(r"load|ds_read", o)
            written = _regs(ops[0]) if ops and not stores and (memory or o.startswith("v_")) else frozenset()
            read = frozenset().union(*[_regs(x) for x in (ops if stores else ops[1:])]) if memory or o.startswith("v_") else frozenset()
            if o.startswith("v_fmac"):
                read |= _regs(ops[0])
            need = need_memory if memory else need_vector
            if read & live and not o.startswith("v_mfma"):
                if states < need:
                    early.append((states, need, op + " " + args, o + " " + instructions[j][2]))
                continue
            states += int(ops[0], 0) + 1 if o == "s_nop" else 1
            work += [(s, states, live - written) for s in behind(j)]
    return early


def test_the_search_finds_an_early_reader():
    """The sequence that was seen: products, two jumps, copies of their results."""
    code = [(0, "v_mfma_f64_4x4x4_4b_f64", "v[6:7], v[98:99], v[6:7], v[52:53]"),
            (8, "v_mfma_f64_4x4x4_4b_f64", "v[8:9], v[98:99], v[8:9], v[48:49]"),
            (16, "s_cbranch_execz", "1"), (20, "s_branch", "1"), (24, "s_nop", "5"),
            (28, "v_mov_b64_e32", "v[52:53], v[6:7]"), (32, "v_mov_b64_e32", "v[48:49], v[8:9]"), (36, "s_endpgm", "")]
    assert [(s, n) for s, n, _, _ in early_readers(code)] == [(3, 6), (3, 6)]


@pytest.mark.parametrize("n,k,density", [(500, 14, 0.2), (500, 5, 0.25), (784, 10, 0.25), (640, 8, 0.2), (1050, 16, 0.2), (300, 12, 0.25),
                                         (150, 16, 0.2), (112, 10, 0.3), (40, 16, 0.2), (784, 10, None), (500, 4, None), (128, 12, None),
                                         (100, 9, None)])
def test_results_of_the_matrix_units_are_waited_for(n, k, density, tmp_path, monkeypatch):
    import paper_1801_00829_amd as F
    from paper_1801_00829_amd import build as B
    if B.needs_build():
        B.build()
    monkeypatch.setenv("FUSE_CACHE_DIR", str(tmp_path))
    monkeypatch.setenv("FUSE_MFMA_CSR_DENSITY", "1")
    if density:
        monkeypatch.setenv("FUSE_MFMA_PIPE", "3" if n >= 128 else "1")
    F.cache_clear()
    m = 100000
    F.prepare_row(MLOGREG, (m, n), [("rhs", (n, k)), ("kvec", (m, k))], "col_t", nnz=int(m * n * density) if density else None)
    files = [str(p) for p in tmp_path.iterdir() if p.name.endswith(".co")]
    assert len(files) == 1 and F.last_kernel().startswith("fuse_row_mfma")
    code = _instructions(files[0], tmp_path)
    assert sum(op.startswith("v_mfma_f64") for _, op, _ in code) > 3
    assert not early_readers(code)
