"""The check of test_asm_hazards_cpu.py (no inline LDS read writes a register
that a recent MFMA still reads as its accumulator input) for the head-dim-64
attention kernels, whose 16x16x32 MFMAs take 4 passes of 4 cycles (the 32x32x16
ones of the other kernels 8): twice that in wait states is scanned."""
import os
import re
import subprocess

import pytest

from paper_2503_03182_amd import build as B

from test_asm_hazards_cpu import scan

WINDOW = 8


@pytest.mark.parametrize("src", ["attention_fwd16.hip", "attention_bwd16.hip"])
def test_inline_lds_reads_never_overwrite_mfma_accumulator_inputs(src, tmp_path):
    dst = str(tmp_path / "a.s")
    cmd = [B.hipcc(), "-x", "hip", *B.COMMON, *B.DEVICE_FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, src),
           "-o", dst]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(dst).read()
    assert len(re.findall(r";;#ASMSTART\s*\n\s*ds_read", text)) > 100
    bad = [h for h in scan(text, WINDOW) if h[1] and h[2] == "C"]
    assert not bad, bad[:5]
