"""A run-time schedule depends on its length alone: the planner reports it, and a
segment's spectrum is the same bits whatever batch it is in, though few segments
take narrower tiles."""
import numpy as np
import pytest

import paper_1407_6915_amd as fs

from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(360, 3000), (20736, 150), (45000, 150), (80000, 100),
                                     (102400, 100), (253125, 64), (1171875, 16), (1953125, 16),
                                     (3375000, 8), (3 << 20, 8), (1 << 23, 4)])
@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
def test_segment_bits_do_not_depend_on_the_batch(n, batch, direction):
    import torch
    announce("schedule bits n=%d batch=%d dir=%d" % (n, batch, direction))
    torch.manual_seed(n)
    x = torch.randn(batch * n, dtype=torch.complex64, device="cuda")
    with fs.Plan(n, batch, direction) as p:
        assert p.describe()["radices"] == fs.factorize(n)
        want = p.exec(x)
    for few in (1, 3):
        with fs.Plan(n, few, direction) as p:
            assert p.describe()["radices"] == fs.factorize(n)
            for first in (0, batch - few):
                part = slice(first * n, (first + few) * n)
                assert torch.equal(p.exec(x[part].clone()), want[part]), (few, first)


@pytest.mark.parametrize("n,batch", [(90000, 100), (1 << 18, 33), (506250, 33), (2343750, 9),
                                     (3906250, 9), (1 << 21, 9)])
@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
def test_real_segment_bits_do_not_depend_on_the_batch(n, batch, direction):
    import torch
    announce("real schedule bits n=%d batch=%d dir=%d" % (n, batch, direction))
    torch.manual_seed(n)
    if direction < 0:
        row, x = n, torch.randn(batch * n, device="cuda")
    else:
        row = n // 2 + 1
        x = torch.randn(batch * row, dtype=torch.complex64, device="cuda")
    with fs.RealPlan(n, batch, direction) as p:
        radices = p.describe()["radices"]
        want = p.exec(x).view(batch, -1)
    with fs.RealPlan(n, 1, direction) as p:
        assert p.describe()["radices"] == radices
        for s in (0, batch - 1):
            got = p.exec(x[s * row:(s + 1) * row].clone())
            assert torch.equal(got, want[s]), s
