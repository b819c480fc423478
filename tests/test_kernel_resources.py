"""What the compiler reports for the hot kernels (written by the build next to the objects): registers per
lane decide how many waves a SIMD holds, and a source change that looks harmless can cost a kernel a third
of its waves (a struct selected between two address spaces once moved the decode kernel's layer
descriptor from scalar into vector registers: 84 -> 118 VGPRs, 1.2 % slower on every workload) or make it
spill.  The figures asserted here are the ones the measured numbers in the profiles were taken with."""
import collections
import json
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PATH = os.path.join(ROOT, "paper_2404_04793_amd", "_build", "kernel_resources.json")


@pytest.fixture(scope="module")
def res():
    if not os.path.exists(PATH):
        pytest.skip("the library has not been built in this tree (python -m paper_2404_04793_amd.build)")
    with open(PATH) as fh:
        return json.load(fh)


def _one(res, *parts):
    hits = [k for k in res if all(p in k for p in parts)]
    assert len(hits) == 1, (parts, hits)
    return res[hits[0]]


def test_no_decode_kernel_spills(res):
    dec = {k: v for k, v in res.items() if "decode_unit_kernel" in k}
    assert len(dec) == 64                              # 2 types x 2 head sizes x 4 group sizes x with/without H2O x dense/blocked
    for k, v in dec.items():
        assert v["ScratchSize"] == 0 and v["VGPRs Spill"] == 0, k


def test_no_kernel_of_the_other_forms_spills(res):
    """The decode kernels with 8 waves per workgroup and for very large caches, the probe of short rows, and what adds up."""
    for name, n in [("decode_wide_kernel", 52), ("decode_large_kernel", 16), ("importance_short_rows_kernel", 12),
                    ("importance_final_kernel", 2)]:
        hits = {k: v for k, v in res.items() if name in k}
        assert len(hits) == n, (name, len(hits))
        for k, v in hits.items():
            assert v["ScratchSize"] == 0 and v["VGPRs Spill"] == 0, k


def test_decode_kernels_keep_their_waves(res):
    # bf16, D = 128, one query head per KV head: the headline kernel (H2O) and its policy-free sibling
    # (the last template argument: 0 = dense, 1 = K and V in blocks named by a block table)
    for pg in (0, 1):
        h2o = _one(res, "decode_unit_kernel", "bf16_tELi128ELi1ELb1ELb0ELb%dE" % pg)
        assert h2o["VGPRs"] <= 88 and h2o["Occupancy"] >= 5
        plain = _one(res, "decode_unit_kernel", "bf16_tELi128ELi1ELb0ELb0ELb%dE" % pg)
        assert plain["VGPRs"] <= 80 and plain["Occupancy"] >= 6
        # matrix-core variant: compiled for 3 waves per SIMD (its LDS stage buffers allow exactly that)
        for g in (4, 8):
            for h in (0, 1):
                mf = _one(res, "decode_unit_kernel", "bf16_tELi128ELi%dELb%dELb1ELb%dE" % (g, h, pg))
                assert mf["VGPRs"] <= 168 and mf["Occupancy"] >= 3 and mf["AGPRs"] == 0, (g, h, pg, mf)


def test_other_hot_kernels(res):
    for k, v in res.items():
        if any(n in k for n in ("importance_partial_kernel", "prefill_compress_kernel", "score_rowstats", "score_colsum")):
            assert v["ScratchSize"] == 0 and v["VGPRs Spill"] == 0, k
    assert _one(res, "importance_partial_kernel", "bf16_tELb0")["Occupancy"] >= 7
    assert _one(res, "score_colsum_mfma_kernel")["Occupancy"] >= 4
    assert _one(res, "score_rowstats_mfma_kernel")["Occupancy"] >= 4


def test_one_pass_scores_keep_their_registers(res):
    # two waves per SIMD: a stripe's exponentials lie in registers
    stripes = {k: v for k, v in res.items() if "score_stripes_kernel" in k}
    assert len(stripes) == 8                           # 2 types x 2 head sizes x 4 or 8 waves
    for k, v in stripes.items():
        assert v["ScratchSize"] == 0 and v["VGPRs Spill"] == 0 and v["Occupancy"] >= 2, k


LLVM = "/opt/rocm/llvm/bin/"


def _instructions(tmp_path, kernel):
    """The instructions of one decode kernel of this build, by name."""
    obj = os.path.join(os.path.dirname(PATH), "sqa_decode.hip.o")
    if not (os.path.exists(obj) and os.path.exists(LLVM + "llvm-objdump")):
        pytest.skip("no objects of a build, or no LLVM tools to list them")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(LLVM + "llvm-objcopy", "-O", "binary", "--only-section=.hip_fatbin", obj, fat)
    run(LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat,
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + code)
    text = run(LLVM + "llvm-objdump", "-d", "--disassemble-symbols=" + kernel, code)
    names = [l.split()[0] for l in text.splitlines() if l.startswith("\t")]
    assert len(names) > 500, kernel
    return collections.Counter(names)


@pytest.mark.parametrize("g", [4, 8])
@pytest.mark.parametrize("blocked", [0, 1])
def test_streaming_loop_of_grouped_fp32_rows_has_no_lane_swaps(res, tmp_path, g, blocked):
    """fp32 at D = 128: the sums over a row's 32 lanes, one per row and head, end in a shuffle through LDS; a lane swap is a
    vector instruction, which bound this loop (8 heads, rows in blocks: 0.89 of the speed).  4 rows per trip."""
    kernel = "_ZN3sqa18decode_unit_kernelIfLi128ELi%dELb0ELb0ELb%dEEEvNS_10DecodeArgsE" % (g, blocked)
    assert kernel in res
    n = _instructions(tmp_path, kernel)
    assert not any(k.startswith("v_permlane16_swap") for k in n) and n["ds_bpermute_b32"] >= 4 * g
