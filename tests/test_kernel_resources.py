"""CPU: registers and occupancy that kernels were sized for, as the compiler reports them for gfx950."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_17412_amd import build


def resources(source, tmp_path):
    """{mangled kernel name: {quantity: value}} of one source file, compiled with the library's own flags."""
    hipcc = build._hipcc()
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    cmd = [hipcc, *build.FLAGS, *build.EXTRA_FLAGS.get(source, []), "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, source), "-o", str(tmp_path / "o.o")]
    text = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    out, name = {}, None
    for what, value in re.findall(r"remark: [^\n]*?\b(Function Name|VGPRs|VGPRs Spill|LDS Size \[bytes/block\]|Occupancy \[waves/SIMD\]): (\S+)", text):
        if what == "Function Name":
            name = value
            out[name] = {}
        else:
            out[name][what.split(" [")[0]] = int(value)
    return out


def test_convolution_of_128_channels_keeps_two_wavefronts_per_simd(tmp_path):
    conv = {k: v for k, v in resources("cmp_module.hip", tmp_path).items() if "c_conv128" in k}
    assert len(conv) == 4  # both directions, 64 and 128 tokens per workgroup
    for name, r in conv.items():
        assert r["Occupancy"] >= 2 and r["VGPRs Spill"] == 0, (name, r)


def test_one_pass_selection_backward_fits_its_registers(tmp_path):
    kernels = {k: v for k, v in resources("mfma_slc_bwd.hip", tmp_path).items() if re.search(r"m_slc_bwdILi\d+ELi\dELb0", k)}
    assert len(kernels) == 4  # blocks of one segment: head_dim 32 and 64, 4 and 8 wavefronts
    for name, r in kernels.items():
        assert r["Occupancy"] >= 2 and r["VGPRs Spill"] == 0, (name, r)


def test_selection_backward_of_short_blocks_at_head_dim_32(tmp_path):
    """Three workgroups of four wavefronts per compute unit: a fifth of the kernel's time at two."""
    kernels = {k: v for k, v in resources("mfma_slc_bwd.hip", tmp_path).items() if "m_slc_bwdILi32ELi4E" in k}
    assert len(kernels) == 1
    for name, r in kernels.items():
        assert r["Occupancy"] >= 3 and r["VGPRs Spill"] == 0, (name, r)


def test_compression_kernels_keep_their_wavefronts(tmp_path):
    """Three wavefronts per SIMD up to head_dim 64, at 128 two, with no more spilled than was measured."""
    all_ = resources("mfma_fwd.hip", tmp_path)
    kernels = {k: v for k, v in all_.items() if re.search(r"m_cmp_fwdILi|m_walk_fwdILi", k)}
    assert len(kernels) == 3 * (3 + 3)  # head dimensions 32, 64, 128: one kernel for 4, 8, 16 heads, compression walk, window walk of 2, 4 waves
    for name, r in kernels.items():
        assert r["Occupancy"] >= (2 if "ILi128E" in name else 3), (name, r)
        most = {"m_cmp_fwdILi64": 2, "m_cmp_fwdILi128": 30, "m_walk_fwdILi128ELi4ELb1": 6}  # (the last: compression walk)
        assert r["VGPRs Spill"] <= max((v for k, v in most.items() if k in name), default=0), (name, r)
    scores = {k: v for k, v in all_.items() if "m_cmp_scoresILi" in k}
    assert len(scores) == 3 * (5 * 2 + 4)  # 1 to 16 heads per KV head by four and eight wavefronts, 2 to 16 with tiles in LDS
    for name, r in scores.items():
        assert r["Occupancy"] >= (2 if "ILi128ELi1E" in name else 3 if "ILi128E" in name else 4) and r["VGPRs Spill"] == 0, (name, r)


def test_selection_and_dq_kernels_keep_their_wavefronts(tmp_path):
    kernels = {**resources("mfma_slc.hip", tmp_path), **resources("mfma_bwd.hip", tmp_path)}
    want = {"m_slc_fwd_bcILi32E": 4, "m_slc_fwd_bcILi64E": 4, "m_slc_fwd_bcILi128E": 2, "m_bwd_dq_bcILi32E": 4, "m_bwd_dq_bcILi64E": 2,
            "m_bwd_dq_bcILi128E": 2, "m_bwd_dqILi32E": 4, "m_bwd_dqILi64E": 3, "m_bwd_dqILi128E": 2}
    for part, waves in want.items():
        found = [r for name, r in kernels.items() if part in name]
        assert len(found) == 1 and found[0]["Occupancy"] >= waves and found[0]["VGPRs Spill"] == 0, (part, found)


def test_backward_pre_pass_leaves_the_lds_to_its_rows(tmp_path):
    """A token's dO rows may take all LDS there is (81920 elements): alone the kernel has none of its own, beside the count pass of the
    selection index no more than the launch reserves (SEL_COUNT_LDS)."""
    kernels = {k: v for k, v in resources("mfma_bwd.hip", tmp_path).items() if "m_bwd_pre" in k}
    lds = {"Lb1E" in name: r["LDS Size"] for name, r in kernels.items()}
    assert lds[False] == 0 and lds[True] <= 1024, kernels
