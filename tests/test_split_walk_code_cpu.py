"""The fp32-accuracy attention kernel whose softmax stands between the matrix instructions (d = 128, block size 128): the order of
its barriers and matrix instructions in the code that the compiler makes of it (cross-compiled here, nothing runs).  The
four wavefronts read and overwrite the same LDS buffers; a barrier that is missing shows in no result that can be relied on."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_20470_amd import build as b


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not (os.path.exists(b.HIPCC) or shutil.which(b.HIPCC)):
        pytest.skip("no hipcc")
    asm = tmp_path_factory.mktemp("split") / "split.s"
    r = subprocess.run([b.HIPCC, *[f for f in b.FLAGS if f != "-fPIC"], "-S", "--cuda-device-only",
                        os.path.join(b.CSRC, "k_attn_split.hip"), "-o", str(asm)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return asm.read_text()


def test_every_reuse_of_a_buffer_lies_behind_a_barrier(listing):
    body = re.search(r"^_ZN\S*12k_attn_splitILb0ELi128ELi128E\S*:.*?^\.Lfunc_end", listing, re.S | re.M).group(0)
    spans = [dict(reads=0, writes=0, products=0)]      # between one barrier and the next, in the order of the code
    for op in re.findall(r"^\s+(v_mfma|s_barrier|ds_read|ds_write)", body, re.M):
        if op == "s_barrier":
            spans.append(dict(reads=0, writes=0, products=0))
        else:
            spans[-1][{"v_mfma": "products", "ds_read": "reads", "ds_write": "writes"}[op]] += 1
    at = next(i for i, span in enumerate(spans) if span["products"])
    # Before the first span the keys of tiles 0 and 1 and the values of tile 0 are put in place.  The logits of tile 0 then read its
    # keys (8 steps of three parts), which the loop's first pass writes over with those of tile 2; a pass of the loop forms
    # the logits of the next tile and the products with the values of its own (the products of the last step before a barrier
    # need no LDS and may drift behind it).
    assert spans[at]["reads"] == 24 and spans[at]["writes"] == 0, spans
    assert spans[at + 1]["reads"] == 48 and spans[at + 1]["writes"] == 12, spans
    assert spans[at]["products"] + spans[at + 1]["products"] == 48 + 96, spans
    assert not any(span["products"] for span in spans[at + 2:]), spans
