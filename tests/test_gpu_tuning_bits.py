"""Tuning and the bit planes: shapes recorded for windows that a batch runs on
bit planes change nothing there and are kept, whatever the timings say."""

import json

import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_batch_tuning_leaves_bit_plane_windows_alone(tmp_path):
    import paper_2505_22938_amd as mf
    items, shapes = [], []
    for dtype, r in (("u8", 3), ("u8", 5), ("u16", 2), ("u16", 4), ("f32", 1), ("f32", 2)):
        fp = mf.Footprint.ellipse(r + 0.3, r - 0.4, 20)   # used by no other test
        img = torch.from_numpy(workloads.uniform(400, 300, dtype, r)).cuda()
        items.append((img, torch.empty_like(img), fp, "clamp"))
        shapes.append(mf.autotune(img, fp, "clamp", reps=1)[:2])
        p = mf.query_plan(400, 300, {"u8": 0, "u16": 1, "f32": 2}[dtype], fp)
        assert (p["tile_w"], p["tile_h"]) == shapes[-1]
        assert mf.query_call(400, 300, {"u8": 0, "u16": 1, "f32": 2}[dtype], fp)["path"] == "bits"
    before, after, dropped = mf.plan_autotune(items, reps=1)
    assert dropped == 0 and before == after > 0
    mf.tune_cache_save(str(tmp_path / "t.json"))
    kept = {(e["tile_w"], e["tile_h"]) for e in json.load(open(tmp_path / "t.json"))}
    assert set(shapes) <= kept
