"""Lengths without compiled tiles: run-time radix schedules, in one pass
(whole segments in LDS), two (columns, rows) or three, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1407_6915_amd as fs

from gpu_helpers import announce, check, noise, run

pytestmark = pytest.mark.gpu

# (length, batch, passes): the shortest; one stage; copied through LDS (below
# 256 points) and not; ragged last workgroups; the longest in one pass; the
# shortest in two; odd lengths (partial lines everywhere); tiles narrower
# than 16 columns or rows
# (passes None: either, by the planner's cost)
CASES = [(3, 5000, 1), (25, 700, 1), (243, 1000, 1), (250, 1000, 1), (270, 1000, 1),
         (360, 4099, 1), (900, 500, 1), (8000, 301, 1), (2187, 301, 1), (3000, 700, 1), (12288, 5, 1), (15625, 3, 1),
         (19683, 40, 1), (20480, 3, 1), (20736, 3, 2), (78125, 5, 2), (48000, 40, 2),
         (3 << 20, 1, 2), (1953125, 1, None), (15625000, 1, None), (14348907, 2, None),
         (1 << 23, 1, 3), (1 << 24, 2, 3)]


@pytest.mark.parametrize("n,batch,passes", CASES)
def test_schedules_match_oracle(n, batch, passes):
    announce("schedule n=%d batch=%d" % (n, batch))
    with fs.Plan(n, batch) as p:
        d = p.describe()
        assert d["kind"] == "radix_stages" and passes in (None, d["passes"]), d
        assert int(np.prod(d["radices"], dtype=np.int64)) == n
    x = noise(n, batch, seed=n % 9973)
    for dr in (fs.FORWARD, fs.INVERSE):
        check(n, run(n, x, dr, inplace=dr > 0), x, dr)


@pytest.mark.parametrize("n,hop,frames", [(100, 33, 2000), (360, 90, 500), (15000, 7500, 7),
                                          (48000, 60001, 3), (78125, 20000, 5)])
@pytest.mark.parametrize("windowed", [True, False])
def test_schedule_frames_match_oracle(n, hop, frames, windowed):
    """Overlapping (and, for 48000, gapped) frames read in place by the
    schedules' first loads."""
    import torch
    announce("schedule frames n=%d hop=%d frames=%d" % (n, hop, frames))
    x = noise((frames - 1) * hop + n, 1, seed=n + hop)[0]
    w = np.hanning(n).astype(np.float32) if windowed else None
    with fs.Plan(n, frames) as p:
        y = p.exec_frames(torch.from_numpy(x).cuda(), hop,
                          window=None if w is None else torch.from_numpy(w).cuda())
        got = y.cpu().numpy().reshape(frames, n)
    ref = np.stack([x[s * hop:s * hop + n] for s in range(frames)]).astype(np.complex128)
    if windowed:
        ref = ref * w.astype(np.float64)
    assert np.all(oracle.rel_l2(got, oracle.fft_recursive(ref, n)) <= oracle.tolerance(n))


@pytest.mark.parametrize("n,b,sub,passes", [(48000, 7, 2, 2), (1 << 23, 3, 2, 3)])
def test_schedules_across_sub_batches(monkeypatch, n, b, sub, passes):
    """Two- and three-pass schedules whose batch runs as several sub-batches
    through one Y buffer, a ragged last one, with and without frames."""
    import torch
    announce("schedule sub-batches n=%d" % n)
    monkeypatch.setenv("FFTSEG_SUB_SAMPLES", str(sub * n))
    x = noise(n, b, seed=77)
    with fs.Plan(n, b) as p:
        assert p.describe()["sub_batch"] == sub and p.describe()["passes"] == passes
        y = p.exec(torch.from_numpy(x.reshape(-1)).cuda()).cpu().numpy().reshape(b, n)
        z = p.exec_frames(torch.from_numpy(x.reshape(-1)).cuda(), n // 2, n_frames=b)
        z = z.cpu().numpy().reshape(b, n)
    check(n, y, x)
    f = x.reshape(-1)
    check(n, z, np.stack([f[s * n // 2:s * n // 2 + n] for s in range(b)]))


# (real length, batch): half lengths 3 (one stage), 5 x 5, odd and even halves
# in one pass, the longest there; two passes with odd and even n1 and n2,
# paired tiles narrower than 16, one row pair, long compiled halves
@pytest.mark.parametrize("n,batch", [(6, 3000), (50, 1001), (250, 400), (720, 301), (4374, 40),
                                     (38400, 3), (36864, 3), (39366, 3), (100000, 3),
                                     (156250, 2), (1 << 18, 2), (3 << 20, 1), (3906250, 1),
                                     (1 << 24, 1)])
def test_real_schedules_match_oracle(n, batch):
    import siggen
    import torch
    announce("real schedule n=%d batch=%d" % (n, batch))
    z = siggen.Signal(seed=n % 9973, seg_len=n, sigma=1.0).samples(0, n * batch // 2 + 1)
    x = z.view(np.float32)[:n * batch].copy()
    ref = oracle.real_forward(x, n)
    with fs.RealPlan(n, batch) as p:
        got = p.exec(torch.from_numpy(x).cuda()).cpu().numpy().reshape(batch, n // 2 + 1)
    assert np.all(oracle.rel_l2(got, ref) <= oracle.tolerance(n))
    spec = ref.astype(np.complex64)
    want = oracle.real_inverse(spec, n)
    # (imaginary parts of bins 0 and n/2 are ignored)
    spec[:, 0] += 3j
    spec[:, n // 2] -= 5j
    with fs.RealPlan(n, batch, fs.INVERSE) as p:
        back = p.exec(torch.from_numpy(spec.reshape(-1)).cuda()).cpu().numpy().reshape(batch, n)
    err = np.linalg.norm(back - want, axis=1) / np.linalg.norm(want, axis=1)
    assert np.all(err <= oracle.tolerance(n)), err.max()


@pytest.mark.parametrize("n,batch", [(1 << 17, 1), (1 << 17, 5), (1 << 18, 2), (1 << 19, 1),
                                     (1 << 19, 5), (1 << 20, 1), (1 << 20, 3), (1 << 21, 2),
                                     (1 << 22, 1)])
def test_two_pass_row_tiles_by_batch(n, batch):
    """The row tiles that small and mid-size batches of two-pass lengths take,
    on a line and off it, as segments and as frames."""
    import torch
    announce("row tile by batch n=%d batch=%d" % (n, batch))
    x = noise(n, batch, seed=n % 9973 + batch)
    for dr in (fs.FORWARD, fs.INVERSE):
        check(n, run(n, x, dr, inplace=dr > 0), x, dr)
    xd = torch.zeros(n * batch + 16, dtype=torch.complex64, device="cuda")
    xd[3:3 + n * batch] = torch.from_numpy(x.reshape(-1))
    yd = torch.zeros_like(xd)
    with fs.Plan(n, batch) as p:
        p.exec(xd[3:3 + n * batch], yd[5:5 + n * batch])
        check(n, yd[5:5 + n * batch].cpu().numpy().reshape(batch, n), x, what="off a line")
        f = p.exec_frames(xd[3:3 + n * batch], n, n_frames=batch)
    check(n, f.cpu().numpy().reshape(batch, n), x, what="frames")


def test_tiny_batches_of_4096():
    """Fewer than 63 segments of 4096 points (32 workgroups of variant 0) take a kernel with more threads
    a segment; more, and forced variants, take variant 0."""
    announce("tiny batches of 4096")
    for batch, variant in [(1, 5), (62, 5), (63, 0), (64, 0)]:
        with fs.Plan(4096, batch) as p:
            assert p.describe()["variant"] == variant
        x = noise(4096, batch, seed=batch)
        for dr in (fs.FORWARD, fs.INVERSE):
            check(4096, run(4096, x, dr), x, dr)
    with fs.Plan(4096, 1, fs.FORWARD, 0) as p:
        assert p.describe()["variant"] == 0


def test_default_stream_is_the_current_one():
    """Without a stream argument a call goes to torch's current stream of the
    current device, also inside a stream context."""
    import torch
    announce("current stream")
    assert fs._stream_handle(None) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert fs._stream_handle(None) == s.cuda_stream != 0
    assert fs._stream_handle(None) == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("count", [1, 3, 4096, 4097])
def test_two_pass_work_list_route_by_count(count):
    """65536-point work lists: the indexed passes up to 4096 segments, tasks
    above, from unaligned offsets (few distinct segments, repeated, so that
    the largest lists fit); the bits do not depend on the list."""
    import torch
    n, kinds = 1 << 16, 3
    announce("work-list route count=%d" % count)
    src = noise(n, kinds, seed=91)
    in_off = (np.arange(count) % kinds) * (n + 5) + 3
    out_off = np.arange(count, dtype=np.int64) * (n + 7) + 1
    x = torch.zeros(kinds * (n + 5) + 16, dtype=torch.complex64, device="cuda")
    for k in range(kinds):
        x[k * (n + 5) + 3:k * (n + 5) + 3 + n] = torch.from_numpy(src[k])
    y = torch.zeros(count * (n + 7) + 8, dtype=torch.complex64, device="cuda")
    with fs.WorkList([(int(i), int(o), n) for i, o in zip(in_off, out_off)]) as wl:
        d = wl.describe()
        assert d["indexed_two_pass_segments"] == (count if count <= 4096 else 0)
        wl.exec(x, y)
        wl.status()
    with fs.WorkList([(3, 1, n), (n + 8, n + 8, n)]) as wl:
        z = torch.zeros(2 * (n + 8), dtype=torch.complex64, device="cuda")
        wl.exec(x, z)
    for s in {0, 1 % count, count // 2, count - 1}:
        got = y[int(out_off[s]):int(out_off[s]) + n]
        check(n, got.cpu().numpy()[None], src[s % kinds][None])
        if s % kinds < 2:
            o = 1 if s % kinds == 0 else n + 8
            assert torch.equal(got, z[o:o + n])


@pytest.mark.parametrize("what,n", [("segments", 1000), ("segments", 1536), ("segments", 4096),
                                    ("frames", 512), ("frames", 1000), ("frames", 1024),
                                    ("frames", 1536), ("frames", 2048), ("frames", 4096),
                                    ("real", 1024), ("real", 2000), ("real", 2048), ("real", 3072),
                                    ("real", 4096), ("real", 8192), ("real", 16384),
                                    ("segments", 1 << 19), ("segments", 1 << 20),
                                    ("segments", 1 << 21), ("segments", 1 << 22),
                                    ("frames", 1 << 20)])
@pytest.mark.parametrize("log2_total", [20, 22, 24, 25])
def test_walking_grids_give_the_same_bits(monkeypatch, what, n, log2_total):
    """A kernel's own grid (workgroups that walk several groups) against one
    workgroup per group: less than one resident wave, a few, many; ragged last
    groups; an output that starts inside a 64-byte line."""
    import torch
    announce("walking grid %s n=%d 2^%d" % (what, n, log2_total))
    batch = (1 << log2_total) // n + 3

    def both(make, call, count, dtype):
        got = []
        for grid in (None, "0"):
            if grid:
                monkeypatch.setenv("FFTSEG_GRID_MULT", grid)
            else:
                monkeypatch.delenv("FFTSEG_GRID_MULT", raising=False)
            y = torch.full((count + 8,), -7.0, dtype=dtype, device="cuda")
            with make() as p:
                call(p, y[3 if dtype.is_complex else 6:])
            got.append(y)
        torch.cuda.synchronize()
        assert torch.equal(got[0], got[1])

    torch.manual_seed(n)
    x = torch.randn(batch * (n + 2) + 8, dtype=torch.complex64, device="cuda")
    for dr in (fs.FORWARD, fs.INVERSE):
        if what == "real":
            count, dtype = (batch * (n // 2 + 1), torch.complex64) if dr < 0 else (batch * n, torch.float32)
            src = torch.view_as_real(x).view(-1)[:batch * n] if dr < 0 else x[:batch * (n // 2 + 1)]
            both(lambda: fs.RealPlan(n, batch, dr), lambda p, y: p.exec(src, y[:count]), count, dtype)
        elif what == "frames":
            hop = n // 4
            both(lambda: fs.Plan(n, batch, dr),
                 lambda p, y: p.exec_frames(x[:(batch - 1) * hop + n], hop, batch, out=y[:batch * n]),
                 batch * n, torch.complex64)
        else:
            both(lambda: fs.Plan(n, batch, dr), lambda p, y: p.exec(x[:batch * n], y[:batch * n]),
                 batch * n, torch.complex64)
