"""What the compiler reports of the kernels, read from the assembly that it writes for them: no GPU is needed."""

import os
import re
import subprocess

import pytest

from paper_2510_22556_amd import build


def _assembly(source, folder):
    asm = str(folder / "kernels.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", asm], check=True,
                   stderr=subprocess.DEVNULL)
    with open(asm) as f:
        return f.read()


def _kernels(source, folder):
    text = _assembly(source, folder)
    blocks = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, re.S)
    return {name: {k: int(v) for k, v in re.findall(r"\.amdhsa_(\w+) (\d+)\n", body)} for name, body in blocks}


@pytest.fixture(scope="module")
def search_select_kernels(tmp_path_factory):
    return _kernels("search_select.hip", tmp_path_factory.mktemp("asm"))


def test_dynamic_lds_of_the_topb_kernels_begins_on_16_bytes(search_select_kernels):
    # it lies behind the static part and is read and written 16 bytes at a time
    topb = {n: k for n, k in search_select_kernels.items() if "topb_" in n or "row_rank_" in n}
    assert len(topb) == 13 + 10
    assert all(k["group_segment_fixed_size"] % 16 == 0 for k in topb.values()), topb


def test_topb_and_search_kernels_do_not_spill(search_select_kernels):
    # 64 registers are few for the Top-B kernels of which two share a CU: those may spill a few, the others none
    scratch = {n: k["private_segment_fixed_size"] for n, k in search_select_kernels.items()}
    two = {n for n in scratch if re.search(r"topb_kernelILb[01]ELi\d+ELb1E", n)}
    assert len(two) == 4
    assert all(scratch[n] <= 16 for n in two), scratch
    assert not any(scratch[n] for n in set(scratch) - two), scratch


def test_inline_assembly_of_the_window_attention_reads_no_matrix_result(tmp_path):
    # the compiler puts wait states between a matrix product and an instruction of its own that reads the result, but does not
    # look into inline assembly: there, vector registers hold addresses only
    text = _assembly("window_attn.hip", tmp_path)
    assert "v_mfma_f32_32x32x16_bf16" in text
    inline = set(re.findall(r"^\s+([a-z]\w+)", "\n".join(re.findall(r";;?#ASMSTART\n(.*?);;?#ASMEND", text, re.S)), re.M))
    assert inline == {"s_mov_b32", "s_nop", "s_waitcnt", "s_barrier", "global_load_lds_dwordx4"}


def test_inline_assembly_waits_for_what_it_loads():
    # the compiler takes the registers of a load in inline assembly as written at once: it is waited for in the same statement, or the
    # load is the compiler's own
    loads = 0
    for name in build.SOURCES:
        with open(os.path.join(build.CSRC, name)) as f:
            for statement in re.findall(r"\basm\b[^;]*;", re.sub(r"//.*", "", f.read())):
                for load in re.findall(r"\b(?:ds_read|ds_load|ds_\w*_rtn|(?:global|buffer|flat|scratch|s)_load(?!_lds))\w*", statement):
                    if "_load_lds" not in load:
                        assert "s_waitcnt" in statement.split(load, 1)[1], (name, statement)
                        loads += 1
    assert loads == 1                                          # the addition to a counter in LDS that returns it


def test_any_shape_scoring_plans_as_many_workgroups_as_the_registers_let_reside(tmp_path):
    # the plan's counts per compute unit (the same rule as in the source): 512 registers per lane and SIMD, given out by the
    # eight, and a wavefront of each workgroup on every SIMD
    seen = 0
    for name, k in _kernels("score_generic.hip", tmp_path).items():
        m = re.search(r"score_generic_(stats|columns)I([ft])Li(\d+)ELi(\d+)E", name)
        if not m:
            continue
        dim, window, f32 = 8 * int(m[3]), int(m[4]), m[2] == "f"
        if m[1] == "stats":
            planned = 4 if dim <= 64 else 3 if dim <= 128 and f32 else 2
        else:
            planned = (3 if dim <= 64 else 2) - (window == 64)
        assert 512 // -(-k["next_free_vgpr"] // 8 * 8) >= planned, (name, k)
        assert k["private_segment_fixed_size"] == 0, name
        seen += 1
    assert seen == 48


def test_scoring_kernels_do_not_spill(tmp_path):
    # a reload waits, through the one counter of loads in order, for the keys that are on their way to LDS in front of it.
    # Read from the object as it is built: these are 200 kernels, and take minutes to compile
    os.makedirs(build.OBJ, exist_ok=True)
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code.o")
    llvm = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin")
    subprocess.run([f"{llvm}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", build._compile("score_mfma.hip", False), os.devnull], check=True)
    subprocess.run([f"{llvm}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={bundle}", f"--output={code}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([f"{llvm}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    scratch = dict(re.findall(r"\.name: +(_Z\S*score_mfma_\S+)\n +\.private_segment_fixed_size: (\d+)", notes))
    assert len(scratch) == 88 + 108 + 1, len(scratch)          # statistics, columns and those of all heads of a layer
    assert set(scratch.values()) == {"0"}, {n: x for n, x in scratch.items() if x != "0"}
