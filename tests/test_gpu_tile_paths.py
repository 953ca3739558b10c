"""Tile engine at shapes that calls of these sizes no longer take by themselves:
small windows (which run on bit planes) in the default low tiles, and float
keys whose sort is decided by its stable passes over the high halves, in LDS
and scattered in global scratch, and global-scratch calls queued on two streams
beside a captured one, all against the oracle."""

import numpy as np
import pytest

import workloads
from oracle import footprints as OF

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mf():
    import paper_2505_22938_amd as m
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    m.lib()
    return m


def same(got, exp):
    return np.array_equal(got.cpu().numpy().view(np.uint8), exp.view(np.uint8))


@pytest.mark.parametrize("r", [0, 1, 2, 3, 5, 8, 12, 16])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_small_windows_in_default_tiles(mf, oracle_mod, dtype, r):
    img = workloads.special_floats(201, 133, r) if dtype == "f32" else \
        workloads.uniform(201, 133, dtype, r)
    dev = torch.from_numpy(img).cuda()
    fp, ofp = mf.Footprint.disc(r), OF.disc(r)
    p = mf.query_plan(201, 133, {"u8": 0, "u16": 1, "f32": 2}[dtype], fp)
    mf.set_tile_override(p["tile_w"], p["tile_h"])
    try:
        for boundary, rank in (("clamp", None), ("mirror", fp.taps // 4)):
            assert same(mf.median_filter(dev, fp, boundary, rank=rank),
                        oracle_mod.filter(img, ofp, boundary, rank=rank)), boundary
    finally:
        mf.set_tile_override(0, 0)
    rmap = workloads.random_ranks(201, 133, fp.taps, r)
    got = mf.rank_map_filter(dev, fp, torch.from_numpy(rmap).cuda(), "clamp")
    assert same(got, oracle_mod.filter(img, ofp, "clamp", rank_map=rmap))


@pytest.mark.parametrize("case", ["one_high_half", "few_high_halves"])
# (boxes of 64 x 128 tiles: 160 x 224 sorted in LDS, 192 x 256 scattered)
@pytest.mark.parametrize("r", [48, 64])
def test_stable_passes_decide(mf, oracle_mod, r, case):
    rng = np.random.default_rng(r)
    w, h = 150, 171
    if case == "one_high_half":
        img = (1.0 + rng.random((h, w)) * (2.0 ** -7)).astype(np.float32)
    else:
        hi = rng.choice(np.array([0x3F80, 0x4000, 0x4080, 0xBF80, 0xC000], np.uint32), (h, w))
        img = ((hi << 16) | rng.integers(0, 1 << 16, (h, w), dtype=np.uint32)).view(np.float32)
    fp = mf.Footprint.disc(r)
    mf.set_tile_override(64, 128)
    try:
        p = mf.query_call(w, h, mf.MF_F32, fp)
        assert p["path"] == "scratch", p
        assert (p["scratch_bytes"] > 6 * 4 * p["box_w"] * p["box_h"]) == (r == 64), p
        for boundary in ("clamp", "mirror"):
            assert same(mf.median_filter(torch.from_numpy(img).cuda(), fp, boundary),
                        oracle_mod.filter(img, OF.disc(r), boundary)), boundary
    finally:
        mf.set_tile_override(0, 0)


def test_global_scratch_on_two_streams(mf, oracle_mod):
    a, b = workloads.natural_u16(300, 230, seed=41), workloads.uniform(290, 210, "u16", 42)
    fp = mf.Footprint.disc(110)
    for img in (a, b):
        assert mf.query_call(img.shape[1], img.shape[0], mf.MF_U16, fp)["path"] == "scratch"
    exp_a, exp_b = oracle_mod.filter(a, OF.disc(110), "clamp"), oracle_mod.filter(b, OF.disc(110), "mirror")
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs_a, outs_b = ([torch.empty_like(d) for _ in range(3)] for d in (da, db))
    torch.cuda.synchronize()
    for i in range(3):
        with torch.cuda.stream(s1):
            mf.median_filter(da, fp, "clamp", out=outs_a[i])
        with torch.cuda.stream(s2):
            mf.median_filter(db, fp, "mirror", out=outs_b[i])
    torch.cuda.synchronize()
    assert all(same(o, exp_a) for o in outs_a) and all(same(o, exp_b) for o in outs_b)
    g, out_g = torch.cuda.CUDAGraph(), torch.empty_like(da)
    with torch.cuda.graph(g, stream=s1):
        mf.median_filter(da, fp, "clamp", out=out_g)
    for _ in range(3):
        out_g.copy_(torch.zeros_like(out_g))
        outs_b[0].copy_(torch.zeros_like(outs_b[0]))
        torch.cuda.synchronize()
        g.replay()
        with torch.cuda.stream(s2):
            mf.median_filter(db, fp, "mirror", out=outs_b[0])
        torch.cuda.synchronize()
        assert same(out_g, exp_a) and same(outs_b[0], exp_b)
    del g
    torch.cuda.synchronize()
    mf.release_scratch()
