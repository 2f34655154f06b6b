"""Properties of the compiled kernels that no run can show: what the compiler is told about data
that the lanes of one wavefront exchange through LDS.

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
