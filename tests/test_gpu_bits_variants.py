"""Every bit-plane variant for every key type against the oracle: the variant
is forced and mf_query_call says that it is the one the call runs.  Windows of
as many tap pairs as the variant holds, of odd and even width, and of few (most
lanes' shares empty); ranks at both ends; images that end inside a tile and are
narrower than a chunk; rows at odd addresses; infinities and NaNs of both signs.
Batch plans run kernels of their own, told by the LDS bytes of their one group."""

import math

import numpy as np
import pytest

import workloads
from oracle import footprints as OF

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# lanes per window, tap pairs per lane
VARIANTS = [(1, 4), (1, 9), (1, 18), (1, 29), (1, 46), (2, 32), (2, 41), (2, 50),
            (4, 8), (4, 12), (4, 18), (4, 27), (4, 34), (4, 43), (4, 50),
            (8, 22), (8, 30), (8, 36), (8, 42), (8, 47),
            (16, 22), (16, 27), (16, 33), (16, 41), (16, 50)]
CODE = {"u8": 0, "u16": 1, "f32": 2}


@pytest.fixture(scope="module")
def mf():
    import paper_2505_22938_amd as m
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    m.lib()
    assert len(VARIANTS) == m.BITS_VARIANTS
    return m


@pytest.fixture
def forced(mf):
    yield mf.set_bits_override
    mf.set_bits_override(mf.BITS_AUTO)


def rect(pairs, odd):
    """A rectangle of so many tap pairs, about as wide as tall, off its centre."""
    h = max(d for d in range(1, 65) if pairs % d == 0 and d * d <= 2 * pairs)
    w = 2 * (pairs // h) - odd
    x, y = -(w // 3), -(h // 2)
    return [(x - .25, y - .25), (x + w - .75, y - .25), (x + w - .75, y + h - .75),
            (x - .25, y + h - .75)]


def image(dtype, w, h, seed):
    return workloads.special_floats(w, h, seed) if dtype == "f32" else \
        workloads.uniform(w, h, dtype, seed)


def same(got, exp):
    return np.array_equal(np.ascontiguousarray(got.cpu().numpy()).view(np.uint8), exp.view(np.uint8))


def windows(mf, v):
    pairs = VARIANTS[v][0] * VARIANTS[v][1]
    r = 0
    while sum(math.isqrt((r + 1) ** 2 - d * d) + 1 for d in range(-r - 1, r + 2)) <= pairs:
        r += 1   # (a disc's row of half width x has x + 1 pairs)
    return [(mf.Footprint.polygon(rect(pairs, 0)), OF.polygon(rect(pairs, 0))),
            (mf.Footprint.polygon(rect(pairs, 1)), OF.polygon(rect(pairs, 1))),
            (mf.Footprint.disc(r), OF.disc(r)), (mf.Footprint.disc(1), OF.disc(1))]


@pytest.mark.parametrize("v", range(len(VARIANTS)))
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_plain(mf, forced, oracle_mod, dtype, v):
    forced(v)
    for i, (fp, ofp) in enumerate(windows(mf, v)):
        for w, h, boundary in ((139, 71, "clamp"), (13, 37, "mirror")):
            p = mf.query_call(w, h, CODE[dtype], fp)
            assert (p["path"], p["variant"]) == ("bits", v), (fp, p)
            img = image(dtype, w + 3, h, v + i)
            dev = torch.from_numpy(img).cuda()[:, 3:]
            for rank in (None, 0, fp.taps - 1):
                got = mf.median_filter(dev, fp, boundary, rank=rank)
                exp = oracle_mod.filter(np.ascontiguousarray(img[:, 3:]), ofp, boundary, rank=rank)
                assert same(got, exp), (i, w, h, rank)


@pytest.mark.parametrize("v", range(len(VARIANTS)))
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_batch(mf, forced, oracle_mod, dtype, v):
    forced(v)
    items, exp, lds = [], [], 0
    for i, (fp, ofp) in enumerate(windows(mf, v)):
        w, h, boundary = ((75, 40, "mirror"), (9, 70, "clamp"))[i % 2]
        img = image(dtype, w, h, v + i)
        dev = torch.from_numpy(img).cuda()
        items.append((dev, torch.empty_like(dev), fp, boundary))
        exp.append(oracle_mod.filter(img, ofp, boundary))
        lds = max(lds, mf.query_call(w, h, CODE[dtype], fp)["lds_bytes"])
    plan = mf.BatchPlan(items)
    assert plan.info()["groups"] == 1 and plan.info()["lds_bytes"] == lds
    plan.launch()
    torch.cuda.synchronize()
    for it, e in zip(items, exp):
        assert same(it[1], e)
    plan.close()


@pytest.mark.parametrize("v", [0, 4, 5, 7, 8, 14, 15, 19, 20, 24])
def test_extreme_values(mf, forced, oracle_mod, v):
    """Only the ends of the type, infinities and NaNs."""
    forced(v)
    rng = np.random.default_rng(v)
    bits = np.array([0xffffffff, 0xff800000, 0x80000000, 0, 0x7f800000, 0x7fffffff], dtype=np.uint32)
    fp, ofp = windows(mf, v)[1]
    for img in (rng.choice(np.array([0, 255], dtype=np.uint8), (45, 90)),
                rng.choice(np.array([0, 65535], dtype=np.uint16), (45, 90)),
                rng.choice(bits, (45, 90)).view(np.float32)):
        got = mf.median_filter(torch.from_numpy(img).cuda(), fp, "clamp")
        assert same(got, oracle_mod.filter(img, ofp, "clamp"))


def test_what_the_variant_does_not_hold(mf, forced, oracle_mod):
    img = image("u16", 60, 50, 1)
    dev = torch.from_numpy(img).cuda()
    exp = oracle_mod.filter(img, OF.disc(9), "clamp")
    for v in (0, mf.BITS_OFF):
        forced(v)
        assert mf.query_call(60, 50, 1, mf.Footprint.disc(9))["path"] == "lds"
        assert same(mf.median_filter(dev, mf.Footprint.disc(9), "clamp"), exp)
    forced(mf.BITS_OFF)
    assert mf.query_call(60, 50, 1, mf.Footprint.disc(2))["path"] == "lds"
    for bad in (-3, mf.BITS_VARIANTS):
        with pytest.raises(mf.MedianFilterError):
            mf.set_bits_override(bad)
