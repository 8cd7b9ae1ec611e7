"""Workgroups that walk several groups, against one workgroup per group: the same
bits for an output on a line, inside one and half a line on, and grids that
really are smaller."""
import numpy as np
import pytest

import paper_1407_6915_amd as fs

from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what,n,batch", [("segments", 1000, 20011), ("segments", 1536, 20011),
                                          ("segments", 4096, 8195), ("segments", 1 << 19, 35),
                                          ("segments", 1 << 20, 19), ("segments", 1 << 21, 19),
                                          ("segments", 1 << 22, 19), ("real", 1024, 40003),
                                          ("real", 4096, 20011), ("real", 16384, 5003)])
@pytest.mark.parametrize("lead", [0, 3, 8])
def test_walking_grids_give_the_same_bits(monkeypatch, what, n, batch, lead):
    import torch
    announce("walking grid %s n=%d lead=%d" % (what, n, lead))
    torch.manual_seed(n)
    x = torch.randn(batch * (n + 2), dtype=torch.complex64, device="cuda")
    for dr in (fs.FORWARD, fs.INVERSE):
        count, dtype, src, make = batch * n, torch.complex64, x[:batch * n], fs.Plan
        if what == "real":
            make = fs.RealPlan
            if dr < 0:
                count, src = batch * (n // 2 + 1), torch.view_as_real(x).view(-1)[:batch * n]
            else:
                dtype, src = torch.float32, x[:batch * (n // 2 + 1)]
        at = lead if dtype.is_complex else 2 * lead
        got, grids = [], []
        for mult in (None, "0"):
            if mult:
                monkeypatch.setenv("FFTSEG_GRID_MULT", mult)
            else:
                monkeypatch.delenv("FFTSEG_GRID_MULT", raising=False)
            y = torch.full((count + 16,), -7.0, dtype=dtype, device="cuda")
            with make(n, batch, dr) as p:
                grids.append(p.describe()["workgroups"])
                p.exec(src, y[at:at + count])
            got.append(y)
        walking, each = (np.atleast_1d(g) for g in grids)
        assert np.all(walking <= each) and np.any(4 * walking <= each + 3), grids
        assert torch.equal(got[0], got[1])
