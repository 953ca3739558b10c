"""Bit planes under batch plans, several ranks and several windows: each plane
equals the oracle's, for calls that mix windows of the bit planes with windows
of the tile engine, strided planes and images smaller than a tile, and for
replays of a captured batch."""

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


def image(dtype, w, h, seed):
    return workloads.special_floats(w, h, seed) if dtype == "f32" else \
        workloads.uniform(w, h, dtype, seed)


def same(got, exp):
    return np.array_equal(np.ascontiguousarray(got.cpu().numpy()).view(np.uint8), exp.view(np.uint8))


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_batch(mf, oracle_mod, dtype):
    """Radii of several variants, an image on each, beside large windows;
    planes with a pitch; eager and captured."""
    items, exp, keep = [], [], []
    for i, (w, h, r) in enumerate([(1, 1, 3), (17, 5, 1), (300, 131, 2), (129, 65, 5), (64, 200, 8),
                                   (200, 64, 10), (90, 90, 30), (257, 33, 16), (40, 41, 1)]):
        img = image(dtype, w, h, i)
        wide = torch.zeros((h, w + 7), dtype=torch.from_numpy(img).dtype, device="cuda")
        wide[:, 3:3 + w].copy_(torch.from_numpy(img).cuda())
        out = torch.empty_like(wide)[:, 3:3 + w]
        keep.append(wide)
        b = "mirror" if i % 2 else "clamp"
        items.append((wide[:, 3:3 + w], out, mf.Footprint.disc(r), b))
        exp.append(oracle_mod.filter(img, OF.disc(r), b))
    plan = mf.BatchPlan(items)
    plan.launch()
    torch.cuda.synchronize()
    for it, e in zip(items, exp):
        assert same(it[1], e), e.shape
    side = torch.cuda.Stream()
    plan.capture(side)
    for _ in range(3):
        for it in items:
            it[1].copy_(torch.zeros_like(it[1]))
        torch.cuda.synchronize()
        plan.replay(side)
        side.synchronize()
        for it, e in zip(items, exp):
            assert same(it[1], e), e.shape
    plan.close()


@pytest.mark.parametrize("r", [0, 1, 4, 8, 12])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_ranks(mf, oracle_mod, dtype, r):
    img = image(dtype, 150, 77, r)
    fp, ofp = mf.Footprint.disc(r), OF.disc(r)
    ranks = sorted({0, (fp.taps - 1) // 4, (fp.taps - 1) // 2, fp.taps - 1})
    got = mf.rank_filter(torch.from_numpy(img).cuda(), fp, ranks, "mirror")
    for k, o in zip(ranks, got):
        assert same(o, oracle_mod.filter(img, ofp, "mirror", rank=k)), k


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_windows(mf, oracle_mod, dtype):
    """In the caller's order, whichever path each takes."""
    img = image(dtype, 140, 95, 3)
    pairs = [(mf.Footprint.disc(30), OF.disc(30)), (mf.Footprint.disc(2), OF.disc(2)),
             (mf.Footprint.ellipse(28, 12, 20), OF.ellipse(28, 12, 20)),
             (mf.Footprint.regular_polygon(6, 7), OF.regular_polygon(6, 7)),
             (mf.Footprint.disc(0), OF.disc(0))]
    got = mf.window_filter(torch.from_numpy(img).cuda(), [p[0] for p in pairs], "clamp")
    for o, (_, ofp) in zip(got, pairs):
        assert same(o, oracle_mod.filter(img, ofp, "clamp"))
