"""Autotuning where the untuned plan is fastest: later plans stay as without it."""
import json

import numpy as np
import pytest

import paper_1407_6915_amd as fs

from gpu_helpers import announce

pytestmark = pytest.mark.gpu


def entry(n, **kw):
    import torch
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    return {"arch": arch, "entries": [dict({"n": n, "variant": -1, "grid_mult": 0}, **kw)]}


@pytest.mark.parametrize("n,variant,batches", [(4096, 0, (1, 64, 4096)), (1024, 0, (1, 4096)),
                                               (1 << 19, -1, (1, 64)), (1 << 20, -1, (1, 16, 64))])
def test_entry_that_keeps_the_defaults(tmp_path, n, variant, batches):
    """Kernels by batch and walking grids as without the entry (a fixed choice of
    the same tiles and multiple has neither)."""
    announce("kept defaults n=%d" % n)
    fs.tune_clear()

    def plans():
        out = []
        for b in batches:
            with fs.Plan(n, b) as p:
                out.append(p.describe())
        return out

    untuned = plans()
    e = entry(n, variant=variant, grid_mult=untuned[-1]["grid_mult"])
    path = str(tmp_path / "tune.json")
    try:
        for keep in (0, 1):
            e["entries"][0]["keep_defaults"] = keep
            with open(path, "w") as f:
                json.dump(e, f)
            fs.tune_clear()
            assert fs.tune_load(path) == 1
            assert (plans() == untuned) == bool(keep)
    finally:
        fs.tune_clear()


def test_autotune_considers_the_untuned_plan(tmp_path):
    """Whatever wins is what later plans get: its time is not above the untuned
    plan's, and an entry that keeps the defaults survives a reload."""
    n, batch = 1000, 1 << 14
    announce("autotune against the untuned plan")
    path = str(tmp_path / "tune.json")
    fs.tune_clear()
    with fs.Plan(n, batch) as p:
        untuned = p.describe()
    try:
        fs.autotune(n, batch, fs.FORWARD, path)
        ent = json.load(open(path))["entries"][0]
        assert ent["keep_defaults"] in (0, 1)
        for _ in range(2):
            with fs.Plan(n, batch) as p:
                d = p.describe()
            assert (d["variant"], d["grid_mult"]) == (ent["variant"], ent["grid_mult"])
            assert not ent["keep_defaults"] or d == untuned
            fs.tune_clear()
            assert fs.tune_load(path) == 1
        # with the defaults' entry in the table the untuned plan is timed as untuned
        fs.autotune(n, batch, fs.FORWARD, path)
    finally:
        fs.tune_clear()
    assert np.isfinite(ent["us"]) and ent["us"] > 0
