"""Barriers of the kernels that order their LDS traffic themselves (block_barrier): no wavefront arrives at one with an LDS access of its own
still under way, since another may write the same bytes behind it.  Read from the assembly of the build's own flags; no GPU."""
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from util import device_assembly

SOURCES = ("streamed.hip", "gemm.hip", "attention.hip")


def outstanding_at_barriers(lines):
    """Largest number of LDS reads and writes issued and not waited for at each s_barrier of one kernel, over all paths to it."""
    label = {m.group(1): i for i, l in enumerate(lines) if (m := re.match(r"(\.L\w+):", l))}
    entry, at_barrier, todo = {}, {}, [(0, 0)]
    while todo:
        i, n = todo.pop()
        while i < len(lines):
            if entry.get(i, -1) >= n:
                break                                             # been here with as many
            entry[i] = n
            op, _, rest = lines[i].strip().partition(" ")
            if op.startswith(("ds_read", "ds_write")):
                n = min(n + 1, 15)                                # the counter's own range
            elif op == "s_waitcnt" and (m := re.search(r"lgkmcnt\((\d+)\)", rest)):
                n = min(n, int(m.group(1)))
            elif op == "s_barrier":
                at_barrier[i] = max(at_barrier.get(i, 0), n)
            elif op.startswith("s_cbranch"):
                todo.append((label[rest.strip()], n))
            elif op == "s_branch":
                i = label[rest.strip()]
                continue
            elif op == "s_endpgm":
                break
            i += 1
    return list(at_barrier.values())


def test_the_walk_itself():
    listing = ["s_cbranch_scc0 .LBB0_2", "ds_read_b128 v[0:3], v4", ".LBB0_1:", "ds_write_b32 v4, v5", "s_waitcnt lgkmcnt(1)", ".LBB0_2:", "s_barrier",
               "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_cbranch_scc1 .LBB0_1", "s_barrier", "s_endpgm"]
    assert outstanding_at_barriers(listing) == [1, 0]
    assert outstanding_at_barriers([l for l in listing if "lgkmcnt(1)" not in l]) == [2, 0]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        return dict(zip(SOURCES, ex.map(lambda src: device_assembly(src, out), SOURCES)))


@pytest.mark.parametrize("src", SOURCES)
def test_no_lds_access_is_under_way_at_a_barrier(assembly, src):
    kernels = re.findall(r"^(_Z\w+):.*?\n(.*?)\n\.Lfunc_end", assembly[src], re.M | re.S)
    found = {name: outstanding_at_barriers(body.split("\n")) for name, body in kernels}
    assert sum(map(len, found.values())) > 0
    assert not {name: n for name, n in found.items() if any(n)}
