"""The build's own checks on what the compiler made of kernels that wait for their loads by hand, on made-up listings."""
import os
import re
import subprocess

import pytest

from paper_2603_22910_amd import build

READ = ";;#ASMSTART\n\tds_read_b128 v[8:11], v2 offset:16\n\tds_read_b64_tr_b16 v[12:13], v3\n;;#ASMEND\n"


def listing(body, name="_Z6kernelv"):
    return f"{name}:                              ; @{name}\n; %bb.0:\n{body}\ts_endpgm\n.Lfunc_end0:\n"


CLEAN = {
    "waited for": READ + "\ts_waitcnt lgkmcnt(0)\n\tv_mov_b32_e32 v0, v8\n",
    "other registers": READ + "\tv_mov_b32_e32 v0, v7\n\tv_mfma_f32_16x16x32_bf16 a[8:11], v[16:19], v[20:23], a[8:11]\n",
    "one left to come": READ + "\ts_waitcnt vmcnt(2) lgkmcnt(1)\n\tv_mov_b32_e32 v0, v11\n\ts_waitcnt lgkmcnt(0)\n\tv_mov_b32_e32 v0, v12\n",
    "by the compiler": "\tds_read_b128 v[8:11], v2\n\tv_mov_b32_e32 v8, 0\n",      # (its own waits are its own business)
    "waited for in a loop": ".LBB0_1:\n" + READ + "\ts_waitcnt lgkmcnt(0)\n\tv_add_f32_e32 v0, v8, v12\n\ts_cbranch_scc1 .LBB0_1\n",
}
EARLY = {
    "copied": (READ + "\tv_mov_b32_e32 v0, v10\n\ts_waitcnt lgkmcnt(0)\n", "v_mov_b32_e32 v0, v10"),
    "moved to an accumulator": (READ + "\tv_accvgpr_write_b32 a0, v12\n\ts_waitcnt lgkmcnt(0)\n", "v_accvgpr_write_b32 a0, v12"),
    "taken for dead": (READ + "\tv_add_u32_e32 v13, v1, v2\n\tglobal_load_dword v0, v13, s[0:1]\n", "v_add_u32_e32 v13, v1, v2"),
    "part of a range": (READ + "\tv_mfma_f32_16x16x32_bf16 v[20:23], v[4:8], v[16:19], v[20:23]\n", "v_mfma_f32_16x16x32_bf16 v[20:23], v[4:8], v[16:19], v[20:23]"),
    "the wrong wait": (READ + "\ts_waitcnt vmcnt(0)\n\tv_mov_b32_e32 v0, v8\n", "v_mov_b32_e32 v0, v8"),
    "the younger of two": (READ + "\ts_waitcnt lgkmcnt(1)\n\tv_mov_b32_e32 v0, v12\n", "v_mov_b32_e32 v0, v12"),
    "a scalar load in between": (READ + "\ts_load_dwordx2 s[0:1], s[2:3], 0x0\n\ts_waitcnt lgkmcnt(1)\n\tv_mov_b32_e32 v0, v8\n", "v_mov_b32_e32 v0, v8"),
    "on the way back in a loop": (".LBB0_1:\n\tv_mov_b32_e32 v0, v9\n" + READ + "\ts_cbranch_scc1 .LBB0_1\n\ts_waitcnt lgkmcnt(0)\n", "v_mov_b32_e32 v0, v9"),
    "behind a branch around the wait": (READ + "\ts_cbranch_vccnz .LBB0_2\n\ts_waitcnt lgkmcnt(0)\n.LBB0_2:\n\tv_mov_b32_e32 v0, v8\n", "v_mov_b32_e32 v0, v8"),
}


@pytest.mark.parametrize("case", CLEAN)
def test_waits_that_are_kept(case):
    assert build.check_early_uses(listing(CLEAN[case])) == []


@pytest.mark.parametrize("case", EARLY)
def test_early_uses_are_found(case):
    body, text = EARLY[case]
    found = build.check_early_uses(listing("\tv_nop\n", "_Z5otherv") + listing(body))
    assert {k for k, _, _ in found} == {"_Z6kernelv"} and found[0][2] == text


def test_spills_are_found_in_the_kernels_that_count_their_loads():
    remark = "remark: a.h:1:0: Function Name: {}\nremark: a.h:1:0:     ScratchSize [bytes/lane]: {}\nremark: a.h:1:0:     VGPRs Spill: {}\n"
    clean = remark.format("_ZN6echokv5fused19fused_decode_kernelILi128EEEv", 0, 0)
    assert build.check_spills(clean + remark.format("_ZN6echokv12merge_kernelEv", 16, 2)) == []
    bad = remark.format("_ZN6echokv5fused17recon_mfma_kernelILi0EEEv", 8, 1)
    assert [n for _, n in build.check_spills(clean + bad)] == [8, 1]


def compile_header(tmp_path, text):
    """The compiler's run over a source of explicit instances: its result, with the remarks on what each kernel takes."""
    src = tmp_path / "instances.hip"
    src.write_text(text)
    cmd = [build.hipcc_path(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", "-I", build.CSRC, "-I", os.path.join(build.HERE, "..", "include"),
           "-o", str(tmp_path / "instances.s"), str(src)]
    return subprocess.run(cmd, capture_output=True, text=True)


def remarks(res, what):
    """{kernel: value} of one line of the remarks."""
    assert res.returncode == 0, res.stderr
    return {k: int(n) for k, n in re.findall(r"Function Name: (\S+)(?:(?!Function Name)(?:.|\n))*?" + re.escape(what) + r": (\d+)", res.stderr)}


def test_streaming_kernels_keep_three_waves(tmp_path):
    """The kernels that only stream rows hide the memory's latency by other waves: three of a SIMD at least (168 registers), for every
    number of query heads that share a pass."""
    kernels = "".join(f"template __global__ void echokv::attn_split_kernel<{t}, {lpr}, {gt}>(echokv::AttnArgs<{t}>, echokv::SeqMeta);\n"
                      for t, lprs in (("echokv::bf16_t", (8, 16)), ("float", (16, 32))) for lpr in lprs for gt in (1, 2, 4))
    found = remarks(compile_header(tmp_path, '#include "attn_split.h"\n' + kernels +
                                   "template int echokv::launch_streams<echokv::bf16_t>(const echokv::Streams<echokv::bf16_t>&, "
                                   "const echokv::StreamMeta&, hipStream_t);\n"), "Occupancy [waves/SIMD]")
    assert sum("attn_split_kernel" in k for k in found) == 12 and any("13stream_kernel" in k for k in found)
    assert {k: n for k, n in found.items() if n < 3} == {}


@pytest.mark.parametrize("ds,nt,compiles", [(1, 256, True), (4, 1024, True), (1, 1024, False), (1, 512, False)])
def test_merges_with_more_partials_than_lanes_do_not_compile(tmp_path, ds, nt, compiles):
    """The merge of few partials keeps a weight per lane: 64 of them, which 256 threads never pass and more of them would."""
    res = compile_header(tmp_path, f'#include "stream_kernels.h"\ntemplate __global__ void echokv::merge_kernel<float, {ds}, {nt}>'
                         "(echokv::MergeArgs<float>, echokv::SeqMeta);\n")
    assert (res.returncode == 0) == compiles, res.stderr
    assert compiles or "one partial per lane" in res.stderr


def test_merge_of_few_splits_has_no_long_form(tmp_path):
    """The absorbed value pass' merge for up to kYFewSplits splits is one round of registers: no LDS."""
    found = remarks(compile_header(tmp_path, '#include "absorbed_decode.h"\n' + "".join(
        f"template __global__ void echokv::absorbed::y_sum_kernel<{sg}>(echokv::absorbed::Args, echokv::SeqMeta);\n" for sg in (1, 4))), "LDS Size [bytes/block]")
    assert {("ILi1E" in k): n > 0 for k, n in found.items() if "y_sum_kernel" in k} == {True: False, False: True}
