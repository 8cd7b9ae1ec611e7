"""fft_exec_segments_noalloc on run-time schedules of every number of passes:
the tables that a call computes on the device against those of a plan, in
batches of several sub-batches of the padded Y buffer, and a refused length."""
import numpy as np
import pytest

import oracle
import paper_1407_6915_amd as fs

from gpu_helpers import announce, noise
from test_zz_no_alloc import _noalloc

pytestmark = pytest.mark.gpu


# one pass of one stage, of two and three, with every radix from 12 on; two
# passes (two sub-batches of 174 segments and a ragged third; odd lengths, whose Y
# pads the last row tile); three passes
@pytest.mark.parametrize("n,batch", [(3, 1000), (45, 300), (360, 41), (600, 9), (729, 7),
                                     (900, 5), (15625, 3), (19683, 2), (20480, 2), (48000, 400),
                                     (78125, 5), (1953125, 2), (6000000, 2), (7558272, 1)])
@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
def test_noalloc_schedules_match_plan(n, batch, direction):
    import torch
    announce("noalloc schedule n=%d batch=%d dir=%d" % (n, batch, direction))
    x = torch.from_numpy(noise(n, batch, seed=17 + n % 89).reshape(-1)).cuda()
    want = torch.zeros_like(x)
    got = torch.full_like(x, 7)
    with fs.Plan(n, batch, direction) as p:
        assert p.describe()["kind"] == "radix_stages"
        p.exec(x, want)
    _noalloc(n, batch, direction, x.data_ptr(), got.data_ptr(),
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    g = got.cpu().numpy().reshape(batch, n)
    e = oracle.rel_l2(g, want.cpu().numpy().reshape(batch, n).astype(np.complex128))
    assert np.all(e <= oracle.tolerance(n)), float(e.max())
    # a table off by one entry would show: the two differ at most where a sine
    # of the device and one of the host round to different sides
    assert e.max() <= 2.0 ** -24, float(e.max())
