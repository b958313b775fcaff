"""Invariants of the generated code of the MXFP4 GEMM that the source cannot
express: its main-loop global loads are issued from inline asm with explicit
vmcnt waits, so the compiler does not know that their destination registers are
written asynchronously.  That is only safe while (a) nothing in the kernel
spills to scratch and (b) every register of the two W sets has ONE physical
assignment in the whole kernel (2 sets x CB x 4 fragment tuples + 2 x CB scale
registers for the tile shape with CB column blocks per wave, each loaded at the
same number of code sites) -- a second assignment would mean a
register copy that may read a tuple whose load is still in flight.
The test compiles the kernel to gfx950 assembly (no GPU needed) and checks both.
"""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2512_00956_amd", "csrc", "mxfp4_gemm_frag.hip")


@pytest.fixture(scope="module")
def asm_text():
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", os.path.dirname(SRC), "-S",
               "--cuda-device-only", SRC, "-o", out]
        subprocess.run(cmd, check=True, capture_output=True)
        return open(out).read()


def test_gemm_frag_generated_code(asm_text):
    """No scratch, one register assignment per W slot, no compiler-made full drain (vmcnt(0)) inside the
    pipelined loop: the same checks the build runs (paper_2512_00956_amd/build_checks.py)."""
    from paper_2512_00956_amd.build_checks import check_gemm_frag_asm
    check_gemm_frag_asm(asm_text)


def test_the_checks_catch_what_they_are_for(asm_text):
    """Planted faults in the assembly text (not in any kernel): a spill, a second register assignment
    of a W fragment, a full drain in the loop."""
    from paper_2512_00956_amd.build_checks import InvariantError, check_gemm_frag_asm
    import re as _re
    with pytest.raises(InvariantError):
        check_gemm_frag_asm(asm_text.replace("s_barrier", "scratch_store_dword off, v0, s0\n\ts_barrier", 1))
    m = _re.search(r"global_load_dwordx4 v\[(\d+):(\d+)\]", asm_text)
    moved = f"global_load_dwordx4 v[{int(m.group(1)) + 400}:{int(m.group(2)) + 400}]"
    with pytest.raises(InvariantError):
        check_gemm_frag_asm(asm_text[:m.start()] + moved + asm_text[m.end():])
    loop = _re.search(r"Inner Loop Header.*?s_cbranch_scc1", asm_text, flags=_re.S)
    drained = asm_text[:loop.start()] + loop.group(0).replace("s_barrier", "s_waitcnt vmcnt(0)\n\ts_barrier", 1) + asm_text[loop.end():]
    with pytest.raises(InvariantError):
        check_gemm_frag_asm(drained)


@pytest.mark.parametrize("src", ["mxfp4_gemm_frag.hip", "mxfp4_gemm_canon.hip"])
def test_loads_to_lds_wait_for_m0(src):
    """A wait state between every write of m0 and the load to LDS that reads it, and no other use of m0; planted faults in
    the assembly text are caught."""
    from paper_2512_00956_amd.build_checks import InvariantError, check_lds_load_asm
    text = _compile(src)
    check_lds_load_asm(text)
    load = re.search(r"s_mov_b32 m0, s\d+\n\s*s_nop 0\n\s*global_load_lds_dwordx4 v\d+, s\[(\d+):\d+\]", text)
    for planted in (load.group(0).replace("s_nop 0\n", "", 1), "s_mov_b32 m0, 0\n\t" + load.group(0),
                    f"v_readfirstlane_b32 s{load.group(1)}, v0\n\t" + load.group(0)):
        with pytest.raises(InvariantError):
            check_lds_load_asm(text[:load.start()] + planted + text[load.end():])


def test_gemm_canon_generated_code():
    """The canonical GEMM: one step's MFMAs and LDS reads between two barriers, the explicit count of loads in front of the
    barrier, no spill, no drain beside the documented one; planted faults in the assembly text are caught."""
    from paper_2512_00956_amd.build_checks import InvariantError, check_gemm_canon_asm
    text = _compile("mxfp4_gemm_canon.hip")
    check_gemm_canon_asm(text)
    barrier = re.search(r"s_waitcnt vmcnt\(([1-9]\d*)\) lgkmcnt\(0\)\n(?:\s*;[^\n]*\n)*\s*s_barrier\n", text)        # a ring of three or four
    start = text.rindex("v_mfma_scale", 0, barrier.start())
    last = re.search(r"(?s).*(v_mfma_scale[^\n]*\n)", text[:barrier.start()]).end(1)
    read = re.compile(r"\s*ds_read_b128 [^\n]*\n").search(text, barrier.end())
    faults = [
        text.replace("s_barrier", "scratch_store_dword off, v0, s0\n\ts_barrier", 1),
        text[:barrier.start()] + barrier.group(0).replace(barrier.group(1), "0", 1) + text[barrier.end():],
        text[:start] + "s_waitcnt vmcnt(0)\n\t" + text[start:],
        text[:barrier.start()] + read.group(0).strip() + "\n\t" + barrier.group(0) + text[barrier.end():read.start()] + "\n" + text[read.end():],
        text[:last] + read.group(0) + text[last:read.start()] + "\n" + text[read.end():],
    ]
    for planted in faults:
        with pytest.raises(InvariantError):
            check_gemm_canon_asm(planted)


def test_lanes_that_exchange_through_lds_are_fenced():
    """__builtin_amdgcn_wave_barrier touches no memory to the compiler: wherever it orders LDS accesses of one wavefront it stands
    between wavefront fences, that is in wave_lds_sync (wush_device.hpp) and nowhere else."""
    csrc = os.path.dirname(SRC)
    uses = {name: open(os.path.join(csrc, name)).read().count("__builtin_amdgcn_wave_barrier(") for name in os.listdir(csrc)}
    assert {name: n for name, n in uses.items() if n} == {"wush_device.hpp": 1}
    body = re.search(r"void wave_lds_sync\(\) \{(.*?)\n\}", open(os.path.join(csrc, "wush_device.hpp")).read(), flags=re.S).group(1)
    calls = re.findall(r"__builtin_amdgcn_\w+\([^)]*\)", body)
    assert calls == ['__builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local")', "__builtin_amdgcn_wave_barrier()",
                     '__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local")']


# ---------------------------------------------------------------------------
# The FP16-dequantizing GEMM of the NVFP4 / INT4 variants and the three fused quantizers: performance
# invariants of the generated code -- nothing spills to scratch (the GEMM keeps up to 256 accumulator
# registers per lane alive next to its conversion temporaries), and the GEMM's K loop holds exactly the
# MFMAs of one K step and one workgroup barrier.
# ---------------------------------------------------------------------------
def _compile(src_name):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src = os.path.join(ROOT, "paper_2512_00956_amd", "csrc", src_name)
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", os.path.dirname(src), "-S",
               "--cuda-device-only", src, "-o", out]
        subprocess.run(cmd, check=True, capture_output=True)
        return open(out).read()


def _bodies(text, pattern):
    parts = re.split(rf"^(_ZN4wush\S*{pattern}\S*):.*$", text, flags=re.M)
    return {parts[i]: parts[i + 1].split("s_endpgm")[0] for i in range(1, len(parts) - 1, 2)}


def test_f16_gemm_has_no_scratch_and_a_tight_loop():
    text = _compile("nvfp4_gemm.hip")
    kernels = _bodies(text, "w4_f16_gemm_kernel")
    assert len(kernels) == 12, list(kernels)          # {bf16, f32 output} x {4, 3, 2 column blocks} x {NVFP4, INT4}
    for name, body in kernels.items():
        cb = int(re.search(r"ILb[01]ELi(\d+)ELi[01]E", name).group(1))
        assert "scratch_" not in body, f"{name}: spills to scratch"
        # the K loop = the basic blocks the compiler annotates as the loop header or "in Loop"
        blocks = re.split(r"^(\.LBB\d+_\d+:.*)$", body, flags=re.M)
        loop = "".join(blocks[i + 1] for i in range(1, len(blocks) - 1, 2)
                       if "Loop Header" in blocks[i] or "in Loop" in blocks[i])
        assert loop, name
        assert len(re.findall(r"v_mfma_f32_32x32x16_f16", loop)) == 16 * cb, name
        assert len(re.findall(r"s_barrier", loop)) == 1, name
        _assert_loads_cost_no_vector_arithmetic(name, loop, 6)


def _loop_of(body):
    blocks = re.split(r"^(\.LBB\d+_\d+:.*)$", body, flags=re.M)
    return "".join(blocks[i + 1] for i in range(1, len(blocks) - 1, 2)
                   if "Loop Header" in blocks[i] or "in Loop" in blocks[i])


def _assert_loads_cost_no_vector_arithmetic(name, loop, n_loads):
    """Every global load of the K loop takes its base from a scalar register pair and a 32-bit lane
    offset (`global_load_* vdst, voffset, s[base:base+1]`), and no 64-bit address arithmetic runs on the
    vector unit: measured, either costs more than the conversion it sits next to."""
    loads = re.findall(r"^\s*global_load_\S+\s+(.*)$", loop, flags=re.M)
    assert len(loads) == n_loads, (name, len(loads))
    for ops in loads:
        assert re.search(r",\s*v\d+,\s*s\[\d+:\d+\]", ops), (name, ops)
    for insn in ("v_mad_i64_i32", "v_mad_u64_u32", "v_lshl_add_u64", "v_add_co_u32", "v_addc_co_u32"):
        assert insn not in loop, (name, insn)


def test_register_w_gemm_loop():
    """The NVFP4 / INT4 kernel that keeps W in registers: no scratch, two K steps per loop trip (2 x 16 CB MFMAs,
    two barriers), 3 + 2 CB loads per step in scalar-base form, and no register move in the loop (the
    prefetched operand sets swap roles between the two steps instead of being copied)."""
    text = _compile("nvfp4_gemm.hip")
    kernels = _bodies(text, "w4_wreg_gemm_kernel")
    assert len(kernels) == 12, list(kernels)          # {bf16, f32 output} x {4, 3, 2 column blocks} x {NVFP4, INT4}
    for name, body in kernels.items():
        cb = int(re.search(r"ILb[01]ELi(\d+)E", name).group(1))
        assert "scratch_" not in body, f"{name}: spills to scratch"
        loop = _loop_of(body)
        assert loop, name
        assert len(re.findall(r"v_mfma_f32_32x32x16_f16", loop)) == 2 * 16 * cb, name
        assert len(re.findall(r"s_barrier", loop)) == 2, name
        _assert_loads_cost_no_vector_arithmetic(name, loop, 2 * (3 + 2 * cb))
        assert "v_mov_b32" not in loop and "v_accvgpr" not in loop, name


@pytest.mark.parametrize("src,pattern,count", [("nvfp4_quant.hip", "nvfp4_transform_quant_kernel", 8),
                                                ("int4_quant.hip", "int4_transform_quant_kernel", 8),
                                                ("transform_quant.hip", "22transform_quant_kernel", 8)])
def test_quantizers_do_not_spill_and_keep_three_waves_per_simd(src, pattern, count):
    text = _compile(src)
    kernels = _bodies(text, pattern)
    assert len(kernels) == count, list(kernels)
    for name, body in kernels.items():
        assert "scratch_" not in body, f"{name}: spills to scratch"
    # register budget from the kernel descriptors: at most 168 VGPRs = three waves per SIMD of 512 (the
    # instantiations that also write the FP32 transformed values, a test tap, are exempt).  The kernels
    # with two wave groups and two tiles of lookahead run as the only workgroup of their CU, two waves per
    # SIMD: 256.
    for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", text):
        if pattern in m.group(1) and "kernelILb1E" not in m.group(1):
            budget = 256 if "ELi2ELi2EE" in m.group(1) else 176
            assert int(m.group(2)) <= budget, (m.group(1), m.group(2))


@pytest.mark.parametrize("src", ["layer_decode.hip", "mxfp4_gemm_canon_stream.hip"])
def test_results_of_matrix_instructions_are_waited_for(src):
    """The build's check of every kernel, here on streaming ones, whose products end a branch before a store to LDS; a planted fault (no
    s_nop) is caught."""
    from paper_2512_00956_amd.build_checks import InvariantError, check_mfma_result_waits
    text = _compile(src)
    assert check_mfma_result_waits(text) >= text.count("v_mfma_") > 0
    with pytest.raises(InvariantError):
        check_mfma_result_waits(re.sub(r"s_nop \d+\n", "", text))


@pytest.mark.parametrize("src,pattern,count", [("layer_decode.hip", "gemm_skinny(?:16|_short)?_kernel", 18),
                                                ("mxfp4_gemm_canon_stream.hip", "gemm_canon_stream(?:16)?_kernel", 12),
                                                ("w4_gemm_skinny.hip", "w4_(?:skinny|skinny16|shared_x)_kernel", 68)])
def test_streaming_kernels_store_four_outputs_at_a_time(src, pattern, count):
    """The streaming GEMMs write a lane's four outputs in one store at any alignment of the rows: every site of it comes with
    the three element stores of a row's last channels and no others (rows off the alignment stored element by
    element would add a fourth).  None of them spills."""
    parts = re.split(rf"^(_ZN4wush\S*{pattern}\S*):.*$", _compile(src), flags=re.M)
    kernels = {parts[i]: parts[i + 1].split(".Lfunc_end")[0] for i in range(1, len(parts) - 1, 2)}
    assert len(kernels) == count, list(kernels)
    for name, body in kernels.items():
        assert "scratch_" not in body, f"{name}: spills to scratch"
        wide = len(re.findall(r"^\s*global_store_dwordx[24]\b", body, flags=re.M))
        single = len(re.findall(r"^\s*global_store_(?:dword|short\w*)\s", body, flags=re.M))
        assert wide > 0 and single <= 3 * wide, (name, wide, single)


def test_block_kernels_of_wide_layers_share_their_compute_unit():
    """More blocks than compute units go round by round, as many workgroups to a unit as its registers and LDS hold: with the few partial moments
    such layers have in flight, three waves per SIMD of 512 registers for the 32 x 32 blocks (four a workgroup, 54 of 160 KB), five for the 16 x 16."""
    text = _compile("build_transforms.hip")
    for pattern, budget in (("17wush_block_kernelILi4E", 168), ("19wush_block16_kernelILi4E", 96)):
        counts = [int(c) for name, c in re.findall(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", text) if pattern in name]
        assert len(counts) == 1 and counts[0] <= budget, (pattern, counts)


@pytest.mark.parametrize("src,pattern,count", [("layer_decode.hip", r"gemm_skinny_kernelILi\d", 6), ("layer_decode.hip", r"gemm_skinny16_kernelILi\dELi2E", 4),
                                                ("mxfp4_gemm_canon_stream.hip", r"gemm_canon_stream16_kernelILi\dELi[23]E", 6)])
def test_rings_of_tiles_are_never_drained(src, pattern, count):
    """The streaming GEMMs that keep several K tiles in flight: no wait in the K loop for all of them (a first load under a branch, or a scale
    shifted where it is loaded, makes the compiler put one there), and nothing spills."""
    parts = re.split(rf"^(_ZN4wush\S*{pattern}\S*):.*$", _compile(src), flags=re.M)
    kernels = {parts[i]: parts[i + 1].split(".Lfunc_end")[0] for i in range(1, len(parts) - 1, 2)}
    assert len(kernels) == count, list(kernels)
    for name, body in kernels.items():
        assert "scratch_" not in body, f"{name}: spills to scratch"
        loop = _loop_of(body)
        assert "v_mfma_scale" in loop and "global_load" in loop, name
        assert "vmcnt(0)" not in loop, name
