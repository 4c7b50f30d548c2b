"""The second pass over flagged query blocks with more items than workgroups: every flagged item is taken, whichever
workgroup it falls to, with the bits that a launch of its head alone gives."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import dynamicrad_oracle as o
from workloads import tiny_case

from helpers import GpuRun, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,blocks", [(1, [0]), (1, [9]), (40, [0, 9, 300, 301, 302, 303, 1023, 1024, 1025, 1199])])
def test_flagged_items_anywhere_in_the_launch(H, blocks):
    wl = dataclasses.replace(tiny_case("ragged128"), Nf=10, Hg=16, Wg=24 if H > 1 else 8, H=H, index=71)     # 30 or 10 blocks
    run = GpuRun(wl, threads=8)
    Sb = wl.Sb
    assert Sb == (30 if H > 1 else 10)
    for item in blocks:                                     # item = head * Sb + query block
        rows = slice(item % Sb * 128, item % Sb * 128 + 128)
        run.Qc[0, item // Sb, rows] = (run.Qc[0, item // Sb, rows].float() * 12).bfloat16()
    run.Q = run.Qc.cuda()
    rp = np.arange(Sb + 1) * Sb
    ci = np.tile(np.arange(Sb), Sb)
    rowptr = torch.from_numpy(rp.astype(np.int32)).view(1, 1, -1).cuda()
    colidx = torch.from_numpy(ci.astype(np.int32)).view(1, 1, -1).cuda()
    O, lse = run.attention(rowptr, colidx, colidx.shape[2], want_lse=True)
    for item in blocks:
        h, qb = divmod(item, Sb)
        rows = slice(qb * 128, qb * 128 + 128)
        want = o.masked_attention(to_f64(run.Qc[0, h]), to_f64(run.Kc[0, h]), to_f64(run.Vc[0, h]), rp, ci, 128, rows=[qb])
        assert lse[0, h, rows].max() > 44.4                  # beyond the fast pass's range: the item is flagged
        assert np.abs(to_f64(O[0, h, rows]) - want[qb]).max() <= 2e-2, item
        if H > 1:
            alone = GpuRun(dataclasses.replace(wl, H=1))
            alone.Q, alone.K, alone.V = (t[:, h:h + 1].contiguous() for t in (run.Q, run.K, run.V))
            alone.shape.stride_b = alone.Q.stride(0)
            assert torch.equal(alone.attention(rowptr, colidx, colidx.shape[2])[0, 0, rows], O[0, h, rows]), item
