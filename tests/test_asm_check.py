"""The checker of the emitted device assembly (paper_2502_02581_amd/asm_check.py): unit cases, and
the assembly of the current build when the build step has left it in place.  CPU only."""
from __future__ import annotations

import os
import re

import pytest

from paper_2502_02581_amd import asm_check, build

LOAD = "\tbuffer_load_dwordx4 v4, s[4:7], 0 offen lds"


def _asm(*body):
    return ["_ZN3moe15row_gemm_kernelIxEEv:", *body, "\ts_endpgm", "; ScratchSize: 0"]


def test_descriptor_written_by_vector_instruction_is_flagged():
    bad = _asm("\tv_readlane_b32 s6, v106, 55", "\tv_add_u32_e32 v13, s3, v12", "\ts_add_i32 s3, s68, 0xc000",
               "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD)
    found = asm_check.check_descriptor_hazards(bad)
    assert len(found) == 1 and "s[6]" in found[0] and "4 wait states" in found[0]
    # v_readfirstlane and a carry-out count as well
    assert asm_check.check_descriptor_hazards(_asm("\tv_readfirstlane_b32 s4, v1", "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD))
    assert asm_check.check_descriptor_hazards(_asm("\tv_add_co_u32_e64 v1, s[4:5], v2, v3", "\ts_nop 0", LOAD))


def test_matrix_operand_written_right_before_is_flagged():
    mfma = "\tv_mfma_f32_32x32x2_f32 a[0:15], v4, v9, a[0:15]"
    assert len(asm_check.check_mfma_sources(_asm("\tv_mov_b32_e32 v9, v1", "\ts_nop 0", mfma))) == 1
    assert asm_check.check_mfma_sources(_asm("\tv_mov_b32_e32 v9, v1", "\ts_nop 1", mfma)) == []
    assert asm_check.check_mfma_sources(_asm("\tds_read_b32 v9, v1", "\ts_waitcnt lgkmcnt(0)", mfma)) == []


def test_enough_wait_states_or_other_registers_pass():
    ok = _asm("\tv_readlane_b32 s6, v106, 55", "\ts_mov_b32 m0, s3", "\ts_nop 4", LOAD)       # 1 + 5 wait states
    assert asm_check.check_descriptor_hazards(ok) == []
    ok = _asm("\tv_readlane_b32 s8, v106, 55", "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD)       # not a descriptor word
    assert asm_check.check_descriptor_hazards(ok) == []
    ok = _asm("\ts_add_u32 s4, s4, s20", "\ts_addc_u32 s5, s5, s21", "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD)  # scalar writes
    assert asm_check.check_descriptor_hazards(ok) == []
    ok = _asm("\tv_readlane_b32 s6, v106, 55", "\tbuffer_load_dwordx4 v[0:3], v4, s[4:7], 0 offen")   # not an LDS-DMA load
    assert asm_check.check_descriptor_hazards(ok) == []


def test_writers_on_other_paths_are_found():
    # the writer sits at the tail of the loop, below the load in the file: it precedes the load through the back edge
    loop = _asm(".LBB0_1:", "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD, "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]",
                "\tv_readfirstlane_b32 s5, v9", "\ts_cbranch_scc1 .LBB0_1")
    found = asm_check.check_descriptor_hazards(loop)
    assert len(found) == 1 and "s[5]" in found[0] and "3 wait states" in found[0]
    # the writer sits in the arm of an `if` that jumps over the other arm to the load
    arm = _asm("\ts_cbranch_scc0 .LBB0_2", "\tv_readfirstlane_b32 s7, v9", "\ts_branch .LBB0_3", ".LBB0_2:",
               "\ts_mov_b32 s7, 0", "\ts_nop 7", ".LBB0_3:", "\ts_mov_b32 m0, s3", "\ts_nop 0", LOAD)
    found = asm_check.check_descriptor_hazards(arm)
    assert len(found) == 1 and "s[7]" in found[0]
    # the same with enough wait states behind the writer on that path
    arm[2:3] = ["\tv_readfirstlane_b32 s7, v9", "\ts_nop 4"]
    assert asm_check.check_descriptor_hazards(arm) == []
    # a path that ends before the load: what stands right above the load in the file but never runs into it is no writer
    dead = _asm("\ts_cbranch_scc1 .LBB0_5", "\tv_readfirstlane_b32 s4, v1", "\ts_endpgm", ".LBB0_5:", "\ts_mov_b32 m0, s3",
                "\ts_nop 0", LOAD)
    assert asm_check.check_descriptor_hazards(dead) == []


def test_scratch_in_a_gemm_kernel_is_flagged():
    lines = ["_ZN3moe15row_gemm_kernelIxEEv:", "\ts_endpgm", "; ScratchSize: 1088",
             "_ZN3moe12route_kernelIxEEv:", "\ts_endpgm", "; ScratchSize: 16"]
    found = asm_check.check_no_scratch(lines)
    assert len(found) == 1 and "row_gemm_kernel" in found[0] and "1088" in found[0]


def test_every_matrix_kernel_of_the_gemm_sources_is_checked_for_scratch():
    """By the names in the sources: a kernel that is renamed or added must not drop out of the check."""
    for src in ("expert.hip", "expert_impl.h", "expert_wide.hip"):
        with open(os.path.join(build.CSRC, src)) as f:
            text = f.read()
        names = re.findall(r"__global__[^;{]*?(\w+)\(", re.sub(r"__launch_bounds__\([^;{]*?\) (?=void)", "", text))
        assert len(names) == text.count("__global__")
        for name in names:
            if name in ("plan_kernel", "recolumn_kernel"):   # no accumulators, no matrix instructions
                continue
            lines = [f"_ZN3moe{len(name)}{name}IxEEv:", "\ts_endpgm", "; ScratchSize: 64"]
            assert len(asm_check.check_no_scratch(lines)) == 1, name


def test_packed_fp32_is_flagged():
    assert asm_check.check_no_packed_fp32(_asm("\tv_pk_fma_f32 v[0:1], v[2:3], v[4:5], v[6:7]"))
    assert asm_check.check_no_packed_fp32(_asm("\tv_fma_f32 v0, v1, v2, v3", "\tv_pk_add_f16 v0, v1, v2")) == []


def test_current_build_passes():
    for src in build.CHECKED:
        path = build.device_asm(src)
        if not os.path.exists(path):
            pytest.skip("the build step has not left its device assembly here")
        assert asm_check.check(path) == []


@pytest.mark.parametrize("src", ["expert_bf16.hip", "expert_tail.hip", "expert_f32.hip"])
def test_launches_of_one_set_have_kernels_of_one_argument_block(src):
    """Every product has a kernel for the routed experts alone and one for the shared ones alone, with half the arguments and
    a part of the code of the kernel that holds both."""
    path = build.device_asm(src)
    if not os.path.exists(path):
        pytest.skip("the build step has not left its device assembly here")
    with open(path) as f:
        text = f.read()
    args = dict(re.findall(r"\.amdhsa_kernel (\S+)[^.]*(?:\.(?!amdhsa_kernarg_size)[^.]*)*\.amdhsa_kernarg_size (\d+)", text))
    both = {n: int(b) for n, b in args.items() if "both_row_gemm_kernel" in n or "both_row_w_gemm_kernel" in n}
    # gate/up gated or not, down; dH gated or not, dX with one product or two
    assert len([n for n in both if "row_gemm" in n]) == 3 and len([n for n in both if "row_w_gemm" in n]) == 4
    for name, size in both.items():
        kernel = re.match(r"_ZN3moe\d+both_(row_\w+?_kernel)(I.*)EEvN", name)
        for plan in (0, 1):   # template parameter PLAN
            one = [n for n in args if n.startswith(f"_ZN3moe{len(kernel[1])}{kernel[1]}{kernel[2]}Lb{plan}EEEv")]
            assert len(one) == 1 and int(args[one[0]]) <= size // 2, name


def test_matrix_probe_issues_the_instruction_of_the_tile_cores():
    """The sustained rate that bench.py divides by is that of the instruction the bf16 products run on."""
    paths = [build.device_asm(src) for src in ("common.hip", "expert_bf16.hip")]
    if not all(os.path.exists(p) for p in paths):
        pytest.skip("the build step has not left its device assembly here")
    probe, cores = (set(re.findall(r"^\s+(v_mfma_\w+)", open(p).read(), re.M)) for p in paths)
    assert probe == cores and len(cores) == 1
