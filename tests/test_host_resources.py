"""What the compiler gives the rank search, read from the assembly of the build's own flags; no GPU."""
import re

import pytest

from util import device_assembly


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(workgroup size, one score a thread) -> its resources"""
    found = {}
    for name, body in re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", device_assembly("calib.hip", tmp_path_factory.mktemp("asm")), re.S):
        if m := re.search(r"classify_kernelILi(\d+)ELb(\d)E", name):
            found[int(m.group(1)), m.group(2) == "1"] = {k: int(v) for k, v in re.findall(r"\.amdhsa_(\w+) (\d+)\n", body)}
    return found


def test_rank_search_stays_out_of_scratch_memory(kernels):
    assert set(kernels) == {(256, True), (512, True), (512, False)}
    assert all(k["private_segment_fixed_size"] == 0 for k in kernels.values())


def test_many_scores_fill_a_compute_unit(kernels):
    """Workgroups of 512 threads: four of them, 32 wavefronts, fit in 160 KB of LDS and in the registers (64 a lane at most)."""
    for (threads, _), k in kernels.items():
        assert threads < 512 or k["group_segment_fixed_size"] <= 32768 and k["next_free_vgpr"] <= 64
