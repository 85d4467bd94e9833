"""What the compiler reports of the kernels, read from the assembly that it writes for them: no GPU is needed."""

import os
import re
import subprocess

import pytest

from paper_2510_22556_amd import build


@pytest.fixture(scope="module")
def search_select_kernels(tmp_path_factory):
    asm = str(tmp_path_factory.mktemp("asm") / "search_select.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "search_select.hip"), "-o", asm],
                   check=True, stderr=subprocess.DEVNULL)
    with open(asm) as f:
        text = f.read()
    blocks = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, re.S)
    return {name: {k: int(v) for k, v in re.findall(r"\.amdhsa_(\w+) (\d+)\n", body)} for name, body in blocks}


def test_dynamic_lds_of_the_topb_kernels_begins_on_16_bytes(search_select_kernels):
    # it lies behind the static part and is read and written 16 bytes at a time
    topb = {n: k for n, k in search_select_kernels.items() if "topb_" in n}
    assert len(topb) == 13
    assert all(k["group_segment_fixed_size"] % 16 == 0 for k in topb.values()), topb


def test_topb_and_search_kernels_do_not_spill(search_select_kernels):
    # 64 registers are few for the Top-B kernels of which two share a CU: those may spill a few, the others none
    scratch = {n: k["private_segment_fixed_size"] for n, k in search_select_kernels.items()}
    two = {n for n in scratch if re.search(r"topb_kernelILb[01]ELi\d+ELb1E", n)}
    assert len(two) == 4
    assert all(scratch[n] <= 16 for n in two), scratch
    assert not any(scratch[n] for n in set(scratch) - two), scratch
