"""Compile-time checks of the K-split and LDS-tiled projection GEMMs and the
prefill attention (CPU, needs hipcc): no instance keeps data in scratch memory, none needs more than the 256 registers
per lane that two waves a SIMD leave, and no vector instruction reads an MFMA
result too early (see test_mfma_hazards)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_12422_amd import build as b
from test_mfma_hazards import early_reads

SOURCES = ("pbd_gemm.hip", "pbd_tile.hip", "pbd_attn.hip")


@pytest.mark.slow
def test_gemm_kernels_use_no_scratch_and_wait_for_mfma(tmp_path):
    cc = b.hipcc()
    if not shutil.which(cc) and not os.path.exists(cc):
        pytest.skip("hipcc not available")
    for src in SOURCES:
        out = tmp_path / (src + ".s")
        r = subprocess.run([cc, *b.FLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, src), "-o", str(out),
                            "-Rpass-analysis=kernel-resource-usage"],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-2000:]
        scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
        vgprs = [int(x) for x in re.findall(r" VGPRs: (\d+)", r.stdout)]
        agprs = [int(x) for x in re.findall(r" AGPRs: (\d+)", r.stdout)]
        assert scratch and max(scratch) == 0, (src, scratch)
        assert max(v + a for v, a in zip(vgprs, agprs)) <= 256
        asm = out.read_text()
        assert asm.count("v_mfma") >= 32, src
        assert not early_reads(asm)[:10]
