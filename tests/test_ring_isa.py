"""The register-staged load rings of the product kernels, checked in the compiler's output.

`gemm_bf16_pipe_kernel` issues its global loads from inline assembly and waits with explicit
`s_waitcnt vmcnt(n)`.  A build of it once read a load's destination register before the wait
that covered it (a `v_and` of the edge masking, scheduled ahead of a wait that named no
registers): products with a contraction length that is no multiple of 8 came out wrong whenever
the operand was not yet in a near cache.  These tests compile the kernels for gfx950 and prove
on the assembly that no instruction touches a register a load in flight still has to write, on
any path, and that the kernels spill nothing (a spilled ring register would be the same bug).
"""
import os
import re
import subprocess

import pytest

import isa_ring_check as R

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


# ---- the checker itself, on hand-written snippets ---------------------------------------------

def _kernel(body: str) -> str:
    return "_Z4testv:\n" + body + "\n\ts_endpgm\n.Lfunc_end0:\n"


def _asm(line: str) -> str:
    return f"\t;;#ASMSTART\n\t{line}\n\t;;#ASMEND\n"


def _check(body: str):
    ks = R.kernels_with_asm_loads(_kernel(body))
    assert list(ks) == ["_Z4testv"]
    return R.check_kernel(ks["_Z4testv"])


def test_checker_flags_a_read_before_the_wait():
    body = (_asm("global_load_dwordx4 v[4:7], v[0:1], off") +
            "\tv_and_b32_e32 v8, v4, v9\n" +
            _asm("s_waitcnt vmcnt(0)") +
            "\tds_write_b128 v10, v[4:7]\n")
    bad = _check(body)
    assert len(bad) == 1 and bad[0][1].startswith("v_and_b32") and bad[0][2] == (4,)


def test_checker_accepts_use_after_the_wait_and_counts_in_order():
    body = (_asm("global_load_dwordx4 v[4:7], v[0:1], off") +
            _asm("global_load_dwordx4 v[8:11], v[0:1], off") +
            _asm("s_waitcnt vmcnt(1)") +
            "\tv_and_b32_e32 v12, v4, v13\n" +          # the older load has landed
            _asm("s_waitcnt vmcnt(0)") +
            "\tv_and_b32_e32 v12, v8, v13\n")
    assert _check(body) == []
    body_bad = body.replace("v_and_b32_e32 v12, v4, v13", "v_and_b32_e32 v12, v8, v13")
    assert len(_check(body_bad)) == 1                   # the younger one has not


def test_checker_follows_a_ring_around_its_loop():
    ring = (_asm("global_load_dwordx4 v[4:7], v[0:1], off") +
            _asm("global_load_dwordx4 v[8:11], v[0:1], off") +
            ".LBB0_1:\n" +
            _asm("s_waitcnt vmcnt(1)") +
            "\tds_write_b128 v20, v[4:7]\n" +
            _asm("global_load_dwordx4 v[4:7], v[0:1], off") +
            _asm("s_waitcnt vmcnt(1)") +
            "\tds_write_b128 v20, v[8:11]\n" +
            _asm("global_load_dwordx4 v[8:11], v[0:1], off") +
            "\ts_cbranch_scc1 .LBB0_1\n" +
            _asm("s_waitcnt vmcnt(0)"))
    assert _check(ring) == []
    # a compiler-made copy of a register in flight is a violation as well
    moved = ring.replace("\tds_write_b128 v20, v[8:11]\n", "\tv_mov_b32_e32 v30, v5\n\tds_write_b128 v20, v[8:11]\n")
    assert [b[1] for b in _check(moved)] == ["v_mov_b32_e32 v30, v5"]


# ---- the kernels as compiled -------------------------------------------------------------------

@pytest.fixture(scope="module")
def gemm_asm(tmp_path_factory):
    from paper_2009_09523_amd import build as vfbuild
    if not os.path.exists(vfbuild.HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("isa") / "k_gemm_bf16.s"
    src = os.path.join(vfbuild.CSRC, "k_gemm_bf16.hip")
    cmd = [vfbuild.HIPCC, *vfbuild.FLAGS, "-x", "hip", "--cuda-device-only", "-S", src, "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def test_no_instruction_touches_a_register_with_a_load_in_flight(gemm_asm):
    ks = R.kernels_with_asm_loads(gemm_asm)
    assert len(ks) >= 12, sorted(ks)                    # every instantiation of the pipelined kernel
    for name, body in ks.items():
        assert R.check_kernel(body) == [], name


def test_product_kernels_use_no_scratch_memory(gemm_asm):
    sizes = [int(v) for v in re.findall(r"; ScratchSize: (\d+)", gemm_asm)]
    assert sizes and all(v == 0 for v in sizes), sizes


def _stage_loops(asm, kernel):
    """The instructions of the loop bodies with a barrier and matrix instructions, of the kernels named so."""
    loops = []
    for name, body in R.split_kernels(asm).items():
        if kernel not in name:
            continue
        label, ins = None, []
        for _, raw in body:
            line = raw.split(";")[0].strip()
            m = re.match(r"^(\.LBB\w+):", line)
            if m:
                label, ins = m.group(1), []
            elif line and not line.startswith("."):
                ins.append(line)
                if label and re.match(r"s_cbranch\w* " + re.escape(label) + "$", line):
                    if any("s_barrier" in i for i in ins) and any("mfma" in i for i in ins):
                        loops.append((name, ins))
    return loops


def test_stage_loop_of_the_direct_kernel_goes_from_the_wait_to_the_barrier(gemm_asm):
    """Vector arithmetic for the LDS addresses of a stage's loads, and anything between the wait for a stage and the
    barrier behind it, lengthens every stage of a product that is a chain of stages (208 x 112 x 7424: 29.1 us without,
    32.9 with)."""
    loops = _stage_loops(gemm_asm, "gemm_bf16_dl_kernelILi4ELi0E")
    assert len(loops) >= 2, [n for n, _ in loops]       # with and without a masked tail
    for name, ins in loops:
        assert not [i for i in ins if i.startswith("v_readfirstlane")], name
        wait = [k for k, i in enumerate(ins) if i.startswith("s_waitcnt") and "vmcnt" in i][0]
        assert ins[wait + 1].startswith("s_barrier") and "lgkmcnt(0)" in ins[wait], (name, ins[wait:wait + 4])


def test_batchnorm_tiles_wait_for_a_groups_parameters_behind_a_branch(gemm_asm):
    """Eight column groups of the 256 x 256 tile that ends in the BatchNorm backward pass: the rounding of their parameters
    stands behind a branch each.  Without it the compiler orders the groups' requests otherwise, and the launch of
    4096 x 8192 x 8192 takes 615 us instead of 601."""
    bodies = ["\n".join(filter(None, (raw.split(";")[0].strip() for _, raw in body)))
              for name, body in R.split_kernels(gemm_asm).items() if "gemm_bf16_wide_line16_kernelILi1E" in name]
    assert len(bodies) == 1
    waits = re.findall(r"s_cbranch_(?:scc[01]|vccn?z) \S+\n(?:\.LBB\S+\n)?s_waitcnt vmcnt\(\d+\)\nv_cvt_pk_bf16_f32", bodies[0])
    assert len(waits) == 8, len(waits)


def test_a_weight_copy_alone_does_not_carry_a_job_list(tmp_path):
    """An MLP copies its weights layer by layer, one launch each, and its small steps are bound by the launches: with the
    list of sixteen jobs among their arguments (1.1 KB a launch) a step of seven layers took 293 us instead of 287."""
    from paper_2009_09523_amd import build as vfbuild
    if not os.path.exists(vfbuild.HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "k_elem.s"
    cmd = [vfbuild.HIPCC, *vfbuild.FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(vfbuild.CSRC, "k_elem.hip"), "-o", str(out)]
    assert subprocess.run(cmd, capture_output=True).returncode == 0
    sizes = []
    for entry in re.split(r"\n  - \.", out.read_text().split("amdhsa.kernels:")[1]):
        if re.search(r"\.name: +\S*cast_weight_kernel", entry):
            explicit = [(int(o), int(z)) for o, z, kind in
                        re.findall(r"\.offset: +(\d+)\s+\.size: +(\d+)\s+\.value_kind: +(\w+)", entry) if not kind.startswith("hidden")]
            sizes.append(max(o + z for o, z in explicit))
    assert len(sizes) == 2 and min(sizes) <= 128, sizes
