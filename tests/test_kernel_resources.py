"""The one-tile-per-workgroup kernels of lengths with a factor 3 keep their registers: their
occupancy target must not make the compiler spill (they lost up to 1.7 times to spills of
22 to 98 dwords).  Compiles the device code; no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2211_07777_amd._build as B


@pytest.mark.skipif(not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("prec,length,kinds", [("float", 192, (1, 2, 3, 4, 5)), ("double", 384, (1, 2, 3, 4))])
def test_no_spills(prec, length, kinds, tmp_path):
    cmd = [B.HIPCC] + B.FLAGS + [f"-DFM_T={prec}", f"-DFM_MC={length}", "-DFM_NO_BATCHED", "--cuda-device-only", "-S",
                                 "-Rpass-analysis=kernel-resource-usage", os.path.join(B.CSRC, "fm_inst.hip"),
                                 "-o", str(tmp_path / "k.s")]
    out = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    spills = {}
    for block in out.split("Function Name: ")[1:]:
        m = re.match(r"_ZN2fm11pass_kernelI[fd]Li%dELi(\d+)ELi0E" % length, block)
        if m:
            spills[int(m[1])] = int(re.search(r"VGPRs Spill: (\d+)", block)[1])
    for k in kinds:
        assert spills[k] <= 17, (k, spills)
