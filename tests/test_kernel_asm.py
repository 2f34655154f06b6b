"""Properties of the compiled kernels that no run can show: what the compiler is told about data
that the lanes of one wavefront exchange through LDS, and which matrix instructions share an
accumulator.

The assembly is made from the sources with the library's own flags (CPU only: hipcc compiles for
gfx950 without a GPU).
"""

import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2609_07816_amd import build

FILES = ("kdn_fwd_bf16", "kdn_bwd")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """File -> kernel name -> its assembly lines, comments included."""
    if not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)):
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("asm")

    def compile_one(name):
        path = out / f"{name}.s"
        subprocess.run([build.HIPCC, *build.CFLAGS, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, f"{name}.hip"), "-o", str(path)],
                       check=True, capture_output=True)
        return split_kernels(path.read_text())

    with ThreadPoolExecutor(len(FILES)) as ex:
        return dict(zip(FILES, ex.map(compile_one, FILES)))


def split_kernels(text):
    found, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = found.setdefault(m.group(1), [])
        elif line.startswith("\t.section"):
            cur = None
        elif cur is not None:
            cur.append(line.strip())
    return {k: v for k, v in found.items() if any(ln.startswith("s_endpgm") for ln in v)}


def fenced_exchanges(lines):
    """Wavefront fences that stand between two LDS accesses with no barrier on either side."""
    n = 0
    for at, line in enumerate(lines):
        if line != "; wave barrier":
            continue
        before = next((x for x in reversed(lines[:at]) if x.startswith(("ds_", "s_barrier"))), "")
        after = next((x for x in lines[at:] if x.startswith(("ds_", "s_barrier"))), "")
        n += before.startswith("ds_") and after.startswith("ds_")
    return n


# forward walk: the V tile (stored in 16-byte pieces, read in the product's layout) and the last
# chunk's output rows; backward prep: the query operands over the key ones and their reads, the key
# operands over those, the substitution's tiles, L^-1 turned from columns to rows
@pytest.mark.parametrize("file,kernel,least", [("kdn_fwd_bf16", "walk_kernel", 2),
                                               ("kdn_bwd", "bw_prep", 5)])
def test_lanes_exchange_through_lds_behind_a_fence(kernels, file, kernel, least):
    found = {k: fenced_exchanges(v) for k, v in kernels[file].items() if kernel in k}
    assert found
    assert not {k: n for k, n in found.items() if n < least}


def _regs(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand)
    if not m:
        return ()
    if m.group(3):
        return (int(m.group(3)),)
    return tuple(range(int(m.group(1)), int(m.group(2)) + 1))


def mixed_accumulations(lines):
    """Matrix instructions that add to a result of another shape: the shapes that may have written
    each vector register last, followed along every path of the kernel."""
    code, labels = [], {}
    for line in lines:
        line = line.split(";")[0].strip()
        m = re.match(r"(\.\w+):", line)
        if m:
            labels[m.group(1)] = len(code)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            if op == line:
                op, _, rest = line.partition("\t")
            code.append((op, [x.strip() for x in rest.split(",")]))
    found, seen, work = set(), {}, [(0, {})]
    while work:
        at, state = work.pop()
        state = dict(state)
        while at < len(code):
            old = seen.get(at)
            if old is not None:  # join with what reached this point before
                joined = {r: old.get(r, frozenset()) | state.get(r, frozenset())
                          for r in old.keys() | state.keys()}
                if joined == old:
                    break
                state = joined
            seen[at] = dict(state)
            op, args = code[at]
            if op.startswith("v_mfma"):
                shape = re.search(r"_(\d+x\d+x\d+)_?", op).group(1)
                for r in _regs(args[3].split()[0]):
                    if any(other != shape for other in state.get(r, ())):
                        found.add((at, op, tuple(args)))
                for r in _regs(args[0]):
                    state[r] = frozenset([shape])
            elif op.startswith(("v_", "ds_read", "buffer_load", "global_load", "scratch_load")):
                for r in _regs(args[0].split()[0]):
                    state.pop(r, None)
            if op == "s_endpgm":
                break
            if op.startswith("s_cbranch"):
                work.append((labels[args[0]], state))
            elif op == "s_branch":
                at = labels[args[0]]
                continue
            at += 1
    return found


def test_an_accumulator_takes_products_of_one_shape(kernels):
    """A 16x16x32 product that adds to a 16x16x16 one's result, or the reverse, can give wrong rows:
    the compiler issues the second without the wait that the first's result needs. (The bf16
    forward alone uses both shapes.)"""
    hits = {k: mixed_accumulations(v) for k, v in kernels["kdn_fwd_bf16"].items()}
    assert not {k: sorted(v)[:2] for k, v in hits.items() if v}
