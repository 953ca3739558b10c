"""GPU parity of the bit-plane path (windows of up to a few hundred taps).

The path takes a call by the size of its window and image; set_tile_override
sends the same call to the tile engine.  Each case here compares the two bit
for bit on every pixel, and the smallest ones with the oracle, at the sizes
where the path can go wrong: images narrower than a 16-byte chunk, one pixel
more or less than a tile in either direction, rows starting at any address,
windows that do not contain their centre, every variant's first and last
window, and values at the ends of their type.
"""

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
    if dtype == "f32":
        return workloads.special_floats(w, h, seed)
    if dtype == "u16":
        return workloads.natural_u16(w, h, seed)
    return workloads.uniform(w, h, dtype, seed)


def both(mf, dev, fp, boundary, rank=None):
    """The default route and the tile engine's output as bytes."""
    got = mf.median_filter(dev, fp, boundary, rank=rank)
    mf.set_tile_override(32, 16)
    try:
        exp = mf.median_filter(dev, fp, boundary, rank=rank)
    finally:
        mf.set_tile_override(0, 0)
    torch.cuda.synchronize()
    return (got.contiguous().cpu().numpy().view(np.uint8),
            exp.contiguous().cpu().numpy().view(np.uint8))


# radii around each change of variant (lanes per window, tap pairs per lane)
@pytest.mark.parametrize("r", [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 14, 16, 18, 20])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_radii_against_tile_engine(mf, dtype, r):
    for w, h, boundary in ((300, 129, "clamp"), (131, 67, "mirror")):
        dev = torch.from_numpy(image(dtype, w, h, r)).cuda()
        got, exp = both(mf, dev, mf.Footprint.disc(r), boundary)
        assert np.array_equal(got, exp), (w, h, boundary, int((got != exp).sum()))


@pytest.mark.parametrize("w,h", [(1, 1), (3, 70), (15, 33), (16, 31), (17, 32), (127, 5), (128, 64),
                                 (129, 65), (257, 1), (64, 129)])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_edges_of_tiles_and_chunks(mf, oracle_mod, dtype, w, h):
    img = image(dtype, w, h, 7 * w + h)
    dev = torch.from_numpy(img).cuda()
    for r, boundary in ((2, "mirror"), (5, "clamp")):
        got = mf.median_filter(dev, mf.Footprint.disc(r), boundary).cpu().numpy()
        exp = oracle_mod.filter(img, OF.disc(r), boundary)
        assert np.array_equal(got.view(np.uint8), exp.view(np.uint8)), (r, boundary)


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("offset", [1, 3, 5])
def test_rows_at_any_address(mf, dtype, offset):
    """A view into a larger plane whose rows start at odd elements: outputs
    equal the tile engine's and nothing around the view is written."""
    img = image(dtype, 200, 90, 3)
    base = torch.from_numpy(img).cuda()
    view = base[:, offset:offset + 171]
    fp = mf.Footprint.disc(3)
    out_base = torch.zeros_like(base)
    out = out_base[:, offset:offset + 171]
    mf.median_filter(view, fp, "mirror", out=out)
    mf.set_tile_override(32, 16)
    try:
        exp = mf.median_filter(view, fp, "mirror")
    finally:
        mf.set_tile_override(0, 0)
    torch.cuda.synchronize()
    host = out_base.cpu().numpy()
    assert np.array_equal(np.ascontiguousarray(host[:, offset:offset + 171]).view(np.uint8),
                          exp.contiguous().cpu().numpy().view(np.uint8))
    host[:, offset:offset + 171] = 0
    assert not host.view(np.uint8).any()


SHAPES = {
    "ellipse": (lambda m: m.Footprint.ellipse(11, 2.5, 35), lambda: OF.ellipse(11, 2.5, 35)),
    "hexagon": (lambda m: m.Footprint.regular_polygon(6, 9), lambda: OF.regular_polygon(6, 9)),
}
for _name, _v in (("right", [(3, 3), (9, 3), (9, 8), (3, 8)]),     # without its centre
                  ("left", [(-9, -8), (-3, -8), (-3, -3), (-9, -3)]),
                  ("wide", [(-20, -1), (20, -1), (20, 1), (-20, 1)]),
                  ("tall", [(-1, -20), (1, -20), (1, 20), (-1, 20)])):
    SHAPES[_name] = (lambda m, v=_v: m.Footprint.polygon(v), lambda v=_v: OF.polygon(v))


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_window_shapes_and_ranks(mf, oracle_mod, dtype, shape):
    fp, ofp = SHAPES[shape][0](mf), SHAPES[shape][1]()
    img = image(dtype, 90, 70, 11)
    dev = torch.from_numpy(img).cuda()
    for rank in (0, fp.taps // 3, fp.taps - 1):
        got = mf.median_filter(dev, fp, "clamp", rank=rank).cpu().numpy()
        exp = oracle_mod.filter(img, ofp, "clamp", rank=rank)
        assert np.array_equal(got.view(np.uint8), exp.view(np.uint8)), rank


def test_extreme_values(mf, oracle_mod):
    """Only the smallest and largest values of the type, infinities and NaNs
    of both signs."""
    rng = np.random.default_rng(5)
    fp, ofp = mf.Footprint.disc(4), OF.disc(4)
    bits = np.array([0xffffffff, 0xff800000, 0x80000000, 0, 0x7f800000, 0x7fffffff], dtype=np.uint32)
    for img in (rng.choice(np.array([0, 255], dtype=np.uint8), (70, 90)),
                rng.choice(np.array([0, 65535], dtype=np.uint16), (70, 90)),
                rng.choice(bits, (70, 90)).view(np.float32)):
        got = mf.median_filter(torch.from_numpy(img).cuda(), fp, "clamp").cpu().numpy()
        assert np.array_equal(got.view(np.uint8), oracle_mod.filter(img, ofp, "clamp").view(np.uint8))


def test_graph_capture_and_replay(mf, oracle_mod):
    img = workloads.uniform(333, 150, "u8", 2)
    dev = torch.from_numpy(img).cuda()
    out = torch.empty_like(dev)
    fp = mf.Footprint.disc(3)
    mf.median_filter(dev, fp, "clamp", out=out)   # the span table is on the device
    exp = oracle_mod.filter(img, OF.disc(3), "clamp")
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=s):
        mf.median_filter(dev, fp, "clamp", out=out, stream=s)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), exp)
