"""The build's static checker for the batched kernel's hand-counted loads: it must accept a
correctly waited load and flag the hazards it exists for (planted here, in text, on the CPU)."""
import os
import re

import pytest

from paper_2407_21082_amd import check_gemm_asm as C

NAME = "_ZN2eh12_GLOBAL__N_117gemm_stats_kernelINS_6DtBf16ELi1ELb0EEEvPKDv4_jS5_iiiPKiiiPNS_5StatsE"


def kernel(body: str) -> str:
    return f"{NAME}:\n{body}\n.Lfunc_end0:\n"


STEP_OK = """
\ts_waitcnt vmcnt(3) lgkmcnt(0) ; step-sync
\ts_barrier
.LBB0_1:
\tglobal_load_lds_dwordx4 v[2:3], off
\tglobal_load_lds_dwordx4 v[4:5], off
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[8:11], a[0:3]
\t;;#ASMSTART
\tglobal_load_dwordx4 v[8:11], v[6:7], off
\t;;#ASMEND
\ts_waitcnt vmcnt(3) lgkmcnt(0) ; step-sync
\ts_barrier
\tglobal_load_lds_dwordx4 v[2:3], off
\tglobal_load_lds_dwordx4 v[4:5], off
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[12:15], a[0:3]
\t;;#ASMSTART
\tglobal_load_dwordx4 v[12:15], v[6:7], off
\t;;#ASMEND
\ts_waitcnt vmcnt(3) lgkmcnt(0) ; step-sync
\ts_barrier
\ts_cbranch_scc1 .LBB0_1
\ts_waitcnt vmcnt(0)
\ts_endpgm
"""


def test_accepts_counted_waits():
    findings, nk, nl = C.check_asm(kernel(STEP_OK))
    assert nk == 1 and nl == 2
    assert findings == []


def test_flags_destination_reused_while_in_flight():
    # the address of a later DMA load is computed into the in-flight destination
    bad = STEP_OK.replace("\ts_cbranch_scc1 .LBB0_1\n",
                          "\ts_cbranch_scc1 .LBB0_1\n\tv_lshl_add_u64 v[12:13], v[30:31], 0, s[0:1]\n")
    findings, _, _ = C.check_asm(kernel(bad))
    assert any("v_lshl_add_u64 v[12:13]" in f for f in findings)


def test_flags_use_before_the_wait():
    # an MFMA hoisted above the wait that covers its operand
    bad = STEP_OK.replace("\tglobal_load_dwordx4 v[12:15], v[6:7], off\n\t;;#ASMEND\n",
                          "\tglobal_load_dwordx4 v[12:15], v[6:7], off\n\t;;#ASMEND\n"
                          "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[12:15], a[0:3]\n")
    findings, _, _ = C.check_asm(kernel(bad))
    assert any("touches its destination" in f for f in findings)


def test_flags_load_in_flight_at_end_and_wrong_step_count():
    bad = STEP_OK.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", "\ts_endpgm")
    findings, _, _ = C.check_asm(kernel(bad))
    assert any("in flight at s_endpgm" in f for f in findings)
    extra = STEP_OK.replace("\tglobal_load_dwordx4 v[12:15], v[6:7], off\n\t;;#ASMEND\n",
                            "\tglobal_load_dwordx4 v[12:15], v[6:7], off\n\t;;#ASMEND\n\tglobal_load_dword v40, v[6:7], off\n")
    findings, _, _ = C.check_asm(kernel(extra))
    assert any("other vector memory" in f for f in findings)


def test_a_store_does_not_count_as_a_younger_load():
    bad = STEP_OK.replace("\tglobal_load_lds_dwordx4 v[4:5], off\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[12:15]",
                          "\tglobal_store_dword v[4:5], v40, off\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[20:23], v[12:15]")
    findings, _, _ = C.check_asm(kernel(bad))
    assert findings


def test_only_inline_asm_loads_are_hand_counted():
    """A 16-byte load the compiler emitted itself is tracked by the compiler's own wait counts: it may
    overwrite a destination whose value is dead while the first load is still on its way (loads return
    in order).  The same two instructions inside inline-asm markers are a hazard."""
    tail_ok = ("\ts_waitcnt vmcnt(0)\n\tglobal_load_dwordx4 v[50:53], v[6:7], off\n\tglobal_load_dwordx2 v[50:51], v[6:7], off\n"
               "\ts_waitcnt vmcnt(0)\n\ts_endpgm")
    ok = STEP_OK.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", tail_ok)
    findings, _, nl = C.check_asm(kernel(ok))
    assert findings == [] and nl == 2
    tail_bad = ("\ts_waitcnt vmcnt(0)\n\t;;#ASMSTART\n\tglobal_load_dwordx4 v[50:53], v[6:7], off\n\t;;#ASMEND\n"
                "\tglobal_load_dwordx2 v[50:51], v[6:7], off\n\ts_waitcnt vmcnt(0)\n\ts_endpgm")
    findings, _, nl = C.check_asm(kernel(STEP_OK.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", tail_bad)))
    assert nl == 3 and any("touches its destination" in f for f in findings)


def _dma(src="s[2:3]"):
    return f"\t;;#ASMSTART\n\ts_add_u32 m0, s8, s9\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v2, {src}\n\t;;#ASMEND\n"


def test_hand_written_loads_to_lds():
    """They have to be drained on every path to the end, own m0, and find their address in scalar registers
    that no vector instruction has just written."""
    step = STEP_OK.replace("\tglobal_load_lds_dwordx4 v[2:3], off\n", _dma())
    assert C.check_asm(kernel(step))[0] == []
    late = step.replace("\ts_endpgm", _dma() + "\ts_endpgm")
    assert any("in flight at s_endpgm" in f for f in C.check_asm(kernel(late))[0])
    m0 = step.replace("\ts_cbranch_scc1 .LBB0_1\n", "\ts_mov_b32 m0, s5\n\ts_cbranch_scc1 .LBB0_1\n")
    assert any("uses m0" in f for f in C.check_asm(kernel(m0))[0])
    near = step.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", "\tv_readlane_b32 s3, v9, 1\n" + _dma() + "\ts_waitcnt vmcnt(0)\n\ts_endpgm")
    assert any("wait states" in f for f in C.check_asm(kernel(near))[0])
    far = near.replace("\tv_readlane_b32 s3, v9, 1\n", "\tv_readlane_b32 s3, v9, 1\n\ts_nop 4\n")
    assert C.check_asm(kernel(far))[0] == []
    # a label in between changes nothing for the path that falls through it
    past = near.replace("\tv_readlane_b32 s3, v9, 1\n", "\tv_readlane_b32 s3, v9, 1\n.LBB0_9:\n")
    assert any("wait states" in f for f in C.check_asm(kernel(past))[0])
    # nor does the way round a loop: the instruction in front of the branch back comes before its first one
    round_ = near.replace("\tv_readlane_b32 s3, v9, 1\n", ".LBB0_9:\n").replace(
        "\ts_endpgm", "\tv_readlane_b32 s3, v9, 1\n\ts_cbranch_scc1 .LBB0_9\n\ts_waitcnt vmcnt(0)\n\ts_endpgm")
    assert any("wait states" in f for f in C.check_asm(kernel(round_))[0])


@pytest.mark.parametrize("writer,asm,states", [
    ("v_cmp_eq_u32_e64 s[4:5], v1, v2", "v_writelane_b32 v3, s5, 7", 2),
    ("v_readlane_b32 s4, v1, 3", "v_writelane_b32 v3, s4, 7", 2),
    ("v_add_co_u32_e64 v5, s[4:5], v1, v2", "v_writelane_b32 v3, s5, 7", 2),
    ("v_mfma_f32_32x32x16_bf16 v[16:31], v[0:3], v[4:7], v[16:31]", "v_max3_f32 v9, v17, v30, v8", 12),
    ("v_mfma_f32_16x16x32_bf16 v[16:19], v[0:3], v[4:7], v[16:19]", "v_max3_f32 v9, v17, v18, v8", 7)])
def test_inline_asm_vector_instructions_keep_their_distance(writer, asm, states):
    """The compiler does not count wait states in front of an instruction that it sees as text."""
    def text(nops):
        gap = f"\ts_nop {nops - 1}\n" if nops else ""
        return f"_ZN2eh19calib_count1_kernelE:\n\t{writer}\n{gap}\t;;#ASMSTART\n\t{asm}\n\t;;#ASMEND\n\ts_endpgm\n.Lfunc_end0:\n"
    assert C.check_asm(text(states)) == ([], 1, 0)
    for nops in (0, states - 1):
        assert any("wait states" in f for f in C.check_asm(text(nops))[0]), nops
    # an instruction the compiler knows is the compiler's business
    own = text(0).replace("\t;;#ASMSTART\n", "").replace("\t;;#ASMEND\n", "")
    assert C.check_asm(own) == ([], 1, 0)


def test_only_checked_sources_have_vector_instructions_in_inline_asm():
    csrc = os.path.join(os.path.dirname(C.__file__), "csrc")
    checked = {"eh_gemm.hip", "eh_gemm32.hip", "eh_calib.hip"}
    for name in sorted(os.listdir(csrc)):
        with open(os.path.join(csrc, name)) as f:
            hit = re.search(r'asm(?: volatile)?\("[^;]*?\bv_\w+', f.read())
        assert not hit or name in checked, (name, hit and hit.group(0))


def test_last_steps_of_a_pass():
    """Behind the last full step (2 DMA + 1 register load, one step in flight: 3) come steps without register
    loads: every wait counts a full step less and the DMA loads in between."""
    full = STEP_OK
    dma2 = "\tglobal_load_lds_dwordx4 v[2:3], off\n\tglobal_load_lds_dwordx4 v[4:5], off\n"
    tail = dma2 + "\ts_waitcnt vmcnt({}) ; end-sync 3\n" + dma2 + "\ts_waitcnt vmcnt({}) ; end-sync 3\n\ts_waitcnt vmcnt(0)\n\ts_endpgm"
    ok = full.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", tail.format(2, 1))
    assert C.check_asm(kernel(ok))[0] == []
    for a, b in ((3, 1), (2, 2)):
        bad = full.replace("\ts_waitcnt vmcnt(0)\n\ts_endpgm", tail.format(a, b))
        assert any("last steps" in f for f in C.check_asm(kernel(bad))[0]), (a, b)


def test_service_waves_keep_nothing_in_scratch_memory():
    """In the persistent cascades the service waves are in the chain that everybody waits for: what the compiler
    spills there comes back from a saturated memory (208 bytes of scratch above 64 rows cost 3 us of a
    head's 25; 36 bytes are of the streaming waves)."""
    path = os.path.join(os.path.dirname(C.__file__), "_build", "eh_gemm32.s")
    if not os.path.exists(path):
        pytest.skip("no build has left the assembly")
    with open(path) as f:
        text = f.read()
    size = {}
    for name, body in re.findall(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", text, re.S):
        size[name] = int(re.search(r"private_segment_fixed_size (\d+)", body).group(1))
    above = [v for k, v in size.items() if "gemm32_stats_kernel_rows" in k]
    upto64 = [v for k, v in size.items() if "rows_ksplit_kernel" in k]
    assert len(above) == 1 and above[0] <= 48, size
    assert len(upto64) == 4 and max(upto64) <= 64, size


def test_calibration_kernels_do_not_ask_for_the_flag_they_raise():
    """A calibration kernel that may find a table too small must not also branch on that finding: its waves
    share barriers, and a store of another workgroup between two waves' reads would send some
    of them home and leave the rest with words of LDS that nobody has written."""
    with open(os.path.join(os.path.dirname(C.__file__), "csrc", "eh_calib.hip")) as f:
        text = re.sub(r"//.*", "", f.read())
    kernels = {re.search(r"(calib_\w+_kernel)", k).group(1): k for k in text.split("__global__")[1:]}
    raising = set()
    for name, body in kernels.items():
        body = body.split("\n}\n")[0]
        raises = re.search(r"\*w\.overflow\s*=[^=]|keep_bin\([^;]*w\.overflow", body)
        asks = re.search(r"\*w\.overflow(?!\s*=[^=])", body)
        if raises:
            raising.add(name)
        assert not (raises and asks), name
    assert raising == {"calib_keep1_kernel", "calib_keep2_kernel"}, raising


def test_waves_of_a_workgroup_do_not_part_over_the_status_word():
    """Any workgroup of a launch may raise the status word of the persistent kernels; waves of another one that each
    looked for themselves could part over it, some leaving before the barriers and the LayerNorm they
    share.  Decode kernel: one wave's answer, in LDS.  Rows kernel: read once, and asked about by the wave that speaks
    for a streaming workgroup and by the service waves, each for itself."""
    text = {}
    for source in ("eh_decode.hip", "eh_gemm32.hip"):
        with open(os.path.join(os.path.dirname(C.__file__), "csrc", source)) as f:
            text[source] = re.sub(r"//.*", "", f.read())
        assert len(re.findall(r"volatile[^;]*p\.status", text[source])) == 1
        assert not re.search(r"if \(\*\(volatile", text[source].replace("*(volatile const int*)p.live", ""))
    assert re.search(r"if \(threadIdx\.x < 2\) \{\s+\*sm\.abort_flag\(threadIdx\.x\) = __builtin_amdgcn_readfirstlane\(\*\(volatile", text["eh_decode.hip"])
    uses = re.findall(r"[^\n]*gave_up != 0[^\n]*", text["eh_gemm32.hip"])
    assert len(uses) == 2 and "? -1 : rows_wait" in uses[0] and uses[1].strip().endswith("return;"), uses
    before_first = text["eh_gemm32.hip"].split(uses[0])[0]
    assert before_first.rstrip().endswith("if (wave == 0) {")


def test_built_library_was_checked():
    """The assembly the in-tree library was built from, if a build left it, is clean."""
    build_dir = os.path.join(os.path.dirname(C.__file__), "_build")
    paths = [os.path.join(build_dir, n) for n in ("eh_gemm.s", "eh_gemm32.s")]
    if not all(os.path.exists(p) for p in paths):
        import pytest
        pytest.skip("no build directory (library built elsewhere)")
    for path in paths:
        findings, nk, nl = C.check_asm(open(path).read())
        assert nk >= 4 and nl > 0 and findings == [], path
