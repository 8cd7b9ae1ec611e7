"""Work lists whose route a tuning file sets."""
import json

import numpy as np
import pytest

import paper_1407_6915_amd as fs

from gpu_helpers import announce, check, noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", [fs.FORWARD, fs.INVERSE])
def test_tuned_two_pass_route_has_the_plans_bits(tmp_path, direction):
    """65536-point segments tuned to the indexed passes run the plan's tiles, each
    twiddle a table entry: the same bits as the plan, in any list."""
    import torch
    n, count = 1 << 16, 5
    announce("tuned two-pass route dir=%d" % direction)
    path = str(tmp_path / "tune.json")
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    with open(path, "w") as f:
        json.dump({"arch": arch, "entries": [{"n": n, "variant": -2, "grid_mult": 0,
                                              "wl_route": 1, "wl_grid": 0}]}, f)
    x = torch.from_numpy(noise(n, count, seed=5).reshape(-1)).cuda()
    fs.tune_clear()
    with fs.Plan(n, count, direction) as p:
        want = p.exec(x)
    try:
        assert fs.tune_load(path) == 1
        with fs.WorkList([(s * n, s * n, n) for s in range(count)], direction) as wl:
            assert wl.describe()["indexed_two_pass_segments"] == count
            got = torch.zeros_like(x)
            wl.exec(x, got)
    finally:
        fs.tune_clear()
    assert torch.equal(got, want)
    check(n, got.cpu().numpy().reshape(count, n), x.cpu().numpy().reshape(count, n), direction)
