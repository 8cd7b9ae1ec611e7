"""Segments of 3 and 5 points: a thread each, from any hop, and more of them than
a launch has threads."""
import numpy as np
import pytest

import oracle
import paper_1407_6915_amd as fs

from gpu_helpers import announce, check, noise, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 5])
@pytest.mark.parametrize("batch", [1, 255, 256, 257, 70001])
def test_short_segments_match_oracle(n, batch):
    announce("short segments n=%d batch=%d" % (n, batch))
    x = noise(n, batch, seed=batch + n)
    for dr in (fs.FORWARD, fs.INVERSE):
        check(n, run(n, x, dr, inplace=dr > 0), x, dr)


@pytest.mark.parametrize("n", [3, 5])
@pytest.mark.parametrize("hop", [1, 2, 5, 1000])
@pytest.mark.parametrize("windowed", [True, False])
def test_short_frames_match_oracle(n, hop, windowed):
    import torch
    announce("short frames n=%d hop=%d" % (n, hop))
    frames = 3001
    x = noise((frames - 1) * hop + n, 1, seed=n + hop)[0]
    w = np.linspace(0.5, 1.5, n).astype(np.float32) if windowed else None
    with fs.Plan(n, frames) as p:
        y = p.exec_frames(torch.from_numpy(x).cuda(), hop,
                          window=None if w is None else torch.from_numpy(w).cuda())
    ref = np.stack([x[s * hop:s * hop + n] for s in range(frames)]).astype(np.complex128)
    if windowed:
        ref = ref * w.astype(np.float64)
    err = oracle.rel_l2(y.cpu().numpy().reshape(frames, n), oracle.fft_recursive(ref, n))
    assert np.all(err <= oracle.tolerance(n))


def test_more_short_segments_than_a_launch_has_threads():
    """2^32 + 5 segments of 3 points in place (96 GiB): all ones but in the last
    ones, whose spectra are 3, 0, 0."""
    import torch
    n, batch, tail = 3, (1 << 32) + 5, 5
    announce("short segments, 2^32 + 5 of 3 points")
    need = 8 * n * batch
    if torch.cuda.mem_get_info()[0] < need + (12 << 30):
        pytest.skip("needs %d GiB of device memory" % ((need >> 30) + 12))
    last = noise(n, tail, seed=9)
    x = torch.ones(n * batch, dtype=torch.complex64, device="cuda")
    x[-n * tail:] = torch.from_numpy(last.reshape(-1)).cuda()
    with fs.Plan(n, batch) as p:
        p.exec(x, x)
    check(n, x[-n * tail:].cpu().numpy().reshape(tail, n), last)
    want = torch.tensor([3, 0, 0], dtype=torch.complex64, device="cuda")
    rows = x[:-n * tail].view(-1, n)
    step = 1 << 28
    assert all(bool((rows[s:s + step] == want).all()) for s in range(0, len(rows), step))
