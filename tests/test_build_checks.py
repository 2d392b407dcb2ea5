"""CPU-only checks of what the compiler made of the kernels (hipcc cross-compiles gfx950 here):
no decode kernel variant may use scratch memory, and no vector instruction may read a matrix
instruction's result before the matrix pipeline has delivered it."""
import os
import re
import subprocess

import pytest

from paper_2605_06914_amd.build import CSRC, HIP_FLAGS, ROOT
from tests.asm_hazards import NEED, NEED_SCALAR, scan, scan_scalar_addresses


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """Assembly of the kernels and the compiler's resource-usage remarks, from one device-only compile."""
    out_dir = tmp_path_factory.mktemp("kernels")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIP_FLAGS if f not in ("-shared", "-fPIC")]
    asm = out_dir / "taper_kernels.s"
    cmd = [hipcc, *flags, "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(asm), os.path.join(CSRC, "taper_kernels.hip")]
    run = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert run.returncode == 0, run.stderr[-2000:]
    return asm.read_text(), run.stderr


def test_decode_kernels_use_no_scratch_memory(compiled):
    """Any scratch use makes every launch set up scratch for the whole grid (microseconds per launch);
    the kernels are written to fit the register file, and a change that spills must not go unnoticed."""
    _, remarks = compiled
    name, seen = None, {}
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name:
            seen[name] = int(m.group(1))
    decode = {k: v for k, v in seen.items() if "decode_kernel" in k}
    # head_dim 64 / 128 x 2 partial formats x (1..3 row tiles per wave, and the variant for launches without shared-prefix work)
    assert len(decode) == 16, sorted(seen)
    assert all(v == 0 for v in decode.values()), {k: v for k, v in decode.items() if v}


def test_no_vector_read_of_a_matrix_result_inside_its_latency(compiled):
    """Every control-flow path from every matrix instruction of every decode kernel variant keeps NEED wait
    states before a vector-ALU instruction reads what it wrote."""
    asm, _ = compiled
    findings, kernels = scan(asm)
    assert kernels == 16
    assert not findings, "\n".join(f"{k}: {blk}: `{mfma}` then `{reader}` after {ws} wait states (need {NEED})"
                                   for k, blk, mfma, reader, ws in findings[:10])


def test_the_scanner_sees_a_planted_hazard():
    """The scanner itself: a matrix result copied after two branches and three scalar instructions is
    reported, the same with enough wait states written out is not, and a write in between ends the dependence."""
    def kernel(filler):
        return "\n".join(["_ZN5taper13decode_kernelILi64ELi2ELi0EEEvNS_8StepArgsE:",
                          "\tv_mfma_f32_16x16x32_bf16 v[108:111], v[60:63], v[146:149], v[108:111]",
                          "\ts_cbranch_vccnz .LBB0_2", ".LBB0_1:", "\ts_branch .LBB0_3", ".LBB0_2:", "\ts_mov_b64 s[8:9], 0",
                          *filler, "\tv_mov_b64_e32 v[2:3], v[108:109]", ".LBB0_3:", "\ts_endpgm"])
    bad, n = scan(kernel(["\ts_and_b64 vcc, exec, s[88:89]"]))
    assert n == 1 and len(bad) == 1 and bad[0][4] == 3 and "v_mov_b64" in bad[0][3]
    good, _ = scan(kernel(["\ts_nop 5"]))
    assert good == []
    one_short, _ = scan(kernel(["\ts_nop 4"]))
    assert len(one_short) == 1 and one_short[0][4] == 7
    overwritten, _ = scan(kernel(["\tv_mov_b64_e32 v[108:109], v[4:5]", "\tv_mov_b64_e32 v[110:111], v[6:7]"]))
    assert [f for f in overwritten if f[1] == ".LBB0_2" and "v[2:3]" in f[3]] == []


def test_no_memory_instruction_reads_a_scalar_register_inside_a_vector_writers_latency(compiled):
    asm, _ = compiled
    findings, kernels = scan_scalar_addresses(asm)
    assert kernels == 16
    assert not findings, "\n".join(f"{k}: {blk}: `{w}` then `{r}` after {ws} wait states (need {NEED_SCALAR})"
                                   for k, blk, w, r, ws in findings[:10])


def test_loads_in_inline_assembly_keep_that_distance_by_themselves(compiled):
    """The compiler does not look for hazards inside inline assembly, and what it puts in front of a statement changes from
    build to build: the wait states stand inside the statement."""
    asm, _ = compiled
    statements = [s for s in re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", asm, re.S) if "global_load_lds" in s]
    assert statements
    for s in statements:
        before = s.split("global_load_lds")[0]
        waits = sum(int(n) + 1 for n in re.findall(r"s_nop (\d+)", before))
        assert waits >= NEED_SCALAR, s


def test_the_compiler_has_nothing_to_warn_about(compiled):
    """A warning per use of some statement would hide all others."""
    _, remarks = compiled
    warnings = [l for l in remarks.splitlines() if "warning:" in l]
    assert warnings == [], warnings[:5]


def test_the_scanner_sees_a_planted_scalar_hazard():
    def kernel(*body):
        return "\n".join(["_ZN5taper13decode_kernelILi64ELi2ELi0EEEvNS_8StepArgsE:", *body, ".LBB0_9:", "\ts_endpgm"])
    lane, load = "\tv_readlane_b32 s4, v9, 3", "\tglobal_load_lds_dwordx4 v62, s[4:5] nt"
    bad, n = scan_scalar_addresses(kernel(lane, "\ts_mov_b32 m0, s91", "\ts_nop 0", load))
    assert n == 1 and len(bad) == 1 and bad[0][4] == 2
    assert len(scan_scalar_addresses(kernel(lane, "\ts_cbranch_scc0 .LBB0_1", "\ts_nop 9", ".LBB0_1:", "\ts_nop 2", load))[0]) == 1  # over the branch
    assert scan_scalar_addresses(kernel(lane, "\ts_mov_b32 m0, s91", "\ts_nop 3", load))[0] == []
    assert scan_scalar_addresses(kernel(lane, "\ts_add_u32 s4, s6, s7", load))[0] == []  # the add reads nothing of it and overwrites it
    assert len(scan_scalar_addresses(kernel("\tv_cmp_lt_i32_e64 s[4:5], v1, v2", load))[0]) == 1


def test_every_launch_the_host_code_makes_is_a_strong_symbol(tmp_path):
    """A weak declaration would turn a missing or changed launch function into a call through a null pointer; and the stand-ins of
    the sanitized build are exactly the functions that the host code calls."""
    def symbols(source):
        obj = tmp_path / (os.path.basename(source) + ".o")
        subprocess.check_call(["g++", "-std=c++17", "-fPIC", "-c", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                               "-I", "/opt/rocm/include", "-o", str(obj), source])
        out = subprocess.run(["nm", "-C", str(obj)], capture_output=True, text=True, check=True).stdout
        rows = [re.match(r"\s*[0-9a-f]*\s+(\S)\s+(taper::(?:launch_\w+|static_scratch))\(", l) for l in out.splitlines()]
        return {m.group(2): m.group(1) for m in rows if m}
    calls = symbols(os.path.join(CSRC, "taper_api.cpp"))
    assert len(calls) >= 5 and set(calls.values()) == {"U"}, calls
    stubs = symbols(os.path.join(ROOT, "tests", "sanitize", "kernel_stubs.cpp"))
    assert set(stubs) == set(calls) and set(stubs.values()) == {"T"}, (stubs, calls)


def test_the_merge_kernels_use_no_scratch_memory_and_fit_sixteen_waves(compiled):
    """A workgroup is a wave per query head, up to 16: 128 vector registers each."""
    _, remarks = compiled
    found = re.findall(r"Function Name: (\S*merge_kernel\S*)(?:.|\n)*?VGPRs: (\d+)(?:.|\n)*?ScratchSize \[bytes/lane\]: (\d+)", remarks)
    assert len(found) == 4 and all(int(v) <= 128 and s == "0" for _, v, s in found), found


def test_the_kernels_for_pools_that_start_anywhere_meet_the_same_checks(compiled):
    asm, remarks = compiled
    spilled = re.findall(r"Function Name: (\S*any_start_kernel\S*)(?:.|\n)*?ScratchSize \[bytes/lane\]: (\d+)", remarks)
    assert len(spilled) == 4 and all(n == "0" for _, n in spilled), spilled
    for check in (scan, scan_scalar_addresses):
        findings, kernels = check(asm, name_filter="any_start_kernel")
        assert kernels == 4 and not findings, findings[:5]


def test_the_leading_arguments_arrive_in_registers(compiled):
    """Eight words of arguments are preloaded (a compiler option that is not part of any interface): without it every launch waits for
    a trip to the argument segment before its start record is asked for."""
    asm, _ = compiled
    words = re.findall(r"\.amdhsa_kernel (\S*(?:decode_kernel|any_start_kernel)\S*)(?:.|\n)*?\.amdhsa_user_sgpr_kernarg_preload_length (\d+)", asm)
    assert len(words) == 20 and all(int(n) == 8 for _, n in words), words
