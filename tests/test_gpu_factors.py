"""Factors that the kernels apply, seen through unit impulses: where every other
factor on an output's way is 1, -1, i or -i, the output is the factor itself,
and one that is rounded once from FP64 is within half a unit in the last
place (2^-25 below 1) of the exact root of unity."""
import numpy as np
import pytest

import paper_1407_6915_amd as fs

from gpu_helpers import announce

pytestmark = pytest.mark.gpu

# half a unit in the last place of a float32 in [0.5, 1), and what FP64
# arithmetic adds (a few 2^-52)
ONCE = 2.0 ** -25 * (1 + 2.0 ** -20)


def roots(m, n, direction):
    """exp(direction 2 pi i m / n) for integer arrays m."""
    m = np.asarray(m, np.int64) % n
    a = 2 * np.pi / n * np.where(2 * m > n, m - n, m)
    return np.cos(a) + 1j * direction * np.sin(a)


def off(got, want):
    d = got.astype(np.complex128) - want
    return max(np.abs(d.real).max(), np.abs(d.imag).max())


def impulse(n, at, direction):
    import torch
    x = torch.zeros(n, dtype=torch.complex64, device="cuda")
    x[at] = 1
    with fs.Plan(n, 1, direction) as p:
        y = p.exec(x)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
@pytest.mark.parametrize("n", [40960, 3 << 20, 1 << 23, 1 << 24])
def test_factors_between_passes_are_rounded_once(n, direction):
    """An impulse half a row into the columns: the columns' transforms and the
    rows' are exact (lengths whose rows are powers of two: a 3-point step has
    factors of its own)."""
    announce("pass factors n=%d dir=%d" % (n, direction))
    with fs.Plan(n, 1) as p:
        d = p.describe()
    assert d["passes"] in (2, 3)
    n1, n2, n3 = d["n1"], d["n2"], d.get("n3", 1)
    k = np.arange(n, dtype=np.int64)
    # column n2 n3 / 2: the first pass's factor
    at = n2 * n3 // 2
    assert off(impulse(n, at, direction), roots(k * at, n, direction)) <= ONCE
    if d["passes"] == 3:
        # column n3 / 2: the second pass's factor in the rows k1 = 0
        at = n3 // 2
        got = impulse(n, at, direction)[::n1]
        assert off(got, roots(k[::n1] * at, n, direction)) <= ONCE


# last radices from 15 to 32 in workgroups of both forms
@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
@pytest.mark.parametrize("n", [225, 360, 625, 900, 8000, 12288, 15625, 20000, 20480])
def test_stage_twiddles_are_rounded_once(n, direction):
    """An impulse at r below the last radix R: the n/R-point transforms before the
    last stage are exact, and output k < n/R, to which only input r of a
    butterfly contributes, undivided, is the twiddle W_n^{r k}."""
    announce("stage twiddles n=%d dir=%d" % (n, direction))
    with fs.Plan(n, 1) as p:
        assert p.describe()["passes"] == 1
    k = np.arange(n // 32)
    for r in (2, 5, 7, 11, 13):
        assert off(impulse(n, r, direction)[:n // 32], roots(k * r, n, direction)) <= ONCE, r


# half lengths in two passes: row and column pairs of odd and even lengths
REAL = [1 << 16, 100000, 156250, 1 << 21, 3906250, 1 << 24]


@pytest.mark.parametrize("n", REAL)
def test_real_split_factors_forward_are_rounded_once(n):
    """A one in sample 1: the even samples' transform is 0 and the odd samples' 1, so
    bin k is the split's factor W_n^k."""
    import torch
    announce("real split factors n=%d" % n)
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    x[1] = 1
    with fs.RealPlan(n, 1) as p:
        assert p.describe()["passes"] == 2
        y = p.exec(x).cpu().numpy()
    assert off(y, roots(np.arange(n // 2 + 1), n, -1)) <= ONCE


@pytest.mark.parametrize("n", REAL)
def test_real_split_factors_inverse_are_rounded_once(n):
    """Bins k and n/2 - k of 1 and -1 (of i and i): the split's sum is 0 and its
    difference 2 (2 i), so the two elements that it makes of them add up to
    4 i cos(2 pi k / n) (-4 i sin), which is samples 0 and 1 by themselves."""
    import torch
    announce("real split factors inverse n=%d" % n)
    m = n // 2
    ks = np.unique(np.random.default_rng(n).integers(1, m, 12))
    ks = ks[2 * ks != m]
    for one, other, want in ((1, -1, np.cos), (1j, 1j, lambda a: -np.sin(a))):
        spec = torch.zeros(len(ks), m + 1, dtype=torch.complex64, device="cuda")
        for s, k in enumerate(ks):
            spec[s, int(k)] = one
            spec[s, m - int(k)] = other
        with fs.RealPlan(n, len(ks), fs.INVERSE) as p:
            assert p.describe()["passes"] == 2
            y = p.exec(spec.reshape(-1)).view(len(ks), n)[:, :2].cpu().numpy()
        assert np.all(y[:, 0] == 0)
        assert np.abs(y[:, 1].astype(np.float64) / 4 - want(2 * np.pi / n * ks)).max() <= ONCE
