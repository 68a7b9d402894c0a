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
    for what, value in re.findall(r"remark: [^\n]*?\b(Function Name|VGPRs|VGPRs Spill|Occupancy \[waves/SIMD\]): (\S+)", text):
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
