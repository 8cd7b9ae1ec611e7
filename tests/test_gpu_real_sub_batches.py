"""Real plans on run-time schedules of two passes whose batch runs as several
sub-batches through one Y buffer: odd and even row and column pairs, tiles that Y
pads, a ragged last sub-batch."""
import numpy as np
import pytest

import oracle
import paper_1407_6915_amd as fs
import siggen

from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch,sub", [(100000, 5, 2), (156250, 5, 2), (1 << 17, 7, 3),
                                         (1 << 18, 4, 1), (506250, 3, 2)])
def test_real_schedules_across_sub_batches(monkeypatch, n, batch, sub):
    import torch
    announce("real sub-batches n=%d batch=%d sub=%d" % (n, batch, sub))
    monkeypatch.setenv("FFTSEG_SUB_SAMPLES", str(sub * (n // 2)))
    z = siggen.Signal(seed=n % 9973, seg_len=n, sigma=1.0).samples(0, n * batch // 2 + 1)
    x = z.view(np.float32)[:n * batch].copy()
    ref = oracle.real_forward(x, n)
    with fs.RealPlan(n, batch) as p:
        d = p.describe()
        assert d["passes"] == 2 and d["sub_batch"] == sub
        got = p.exec(torch.from_numpy(x).cuda()).cpu().numpy().reshape(batch, n // 2 + 1)
    assert np.all(oracle.rel_l2(got, ref) <= oracle.tolerance(n))
    spec = ref.astype(np.complex64)
    want = oracle.real_inverse(spec, n)
    with fs.RealPlan(n, batch, fs.INVERSE) as p:
        assert p.describe()["sub_batch"] == sub
        back = p.exec(torch.from_numpy(spec.reshape(-1)).cuda()).cpu().numpy().reshape(batch, n)
    err = np.linalg.norm(back - want, axis=1) / np.linalg.norm(want, axis=1)
    assert np.all(err <= oracle.tolerance(n)), err.max()


def test_cap_below_a_segment_is_refused(monkeypatch):
    monkeypatch.setenv("FFTSEG_SUB_SAMPLES", "1000")
    for n in (100000, 31250):
        with pytest.raises(fs.FFTError) as e:
            fs.RealPlan(n, 4)
        assert e.value.name == "FFT_ERR_INVALID_ARG"
