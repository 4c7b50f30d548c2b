"""The mask kernels' code as the compiler makes it (cross-compiled here, nothing runs): lane masks reach v_writelane by the compiler's own instruction.  On
this chip a vector instruction must not read a scalar register within two wait states of the vector instruction that wrote it; the
compiler keeps them for its own instructions and does not look into inline assembly."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_20470_amd import build as b


def test_no_lane_is_written_by_inline_assembly(tmp_path):
    if not (os.path.exists(b.HIPCC) or shutil.which(b.HIPCC)):
        pytest.skip("no hipcc")
    asm = tmp_path / "mask.s"
    r = subprocess.run([b.HIPCC, *[f for f in b.FLAGS if f != "-fPIC"], "-S", "--cuda-device-only", os.path.join(b.CSRC, "k_mask.hip"), "-o", str(asm)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = asm.read_text()
    assert len(re.findall(r"v_writelane_b32", text)) > 100
    assert not [s for s in re.findall(r"#ASMSTART(.*?)#ASMEND", text, re.S) if "v_writelane" in s]
