"""What a call runs, told by mf_query_call without a GPU: the path of small,
middle and large windows, shapes fitted to the image, and overrides."""

import pytest

import paper_2505_22938_amd as mf

U8, U16, F32 = mf.MF_U8, mf.MF_U16, mf.MF_F32


def test_paths():
    q = lambda w, h, dt, r: mf.query_call(w, h, dt, mf.Footprint.disc(r))  # noqa: E731
    p = q(256, 256, U8, 4)
    assert p["path"] == "bits" and p["variant"] >= 0 and p["scratch_bytes"] == 0
    assert (p["box_w"], p["box_h"]) == (p["tile_w"] + 8, p["tile_h"] + 8)
    p = q(4096, 4096, U16, 32)
    assert p["path"] == "lds" and p["variant"] == -1 and p["scratch_bytes"] == 0
    p = q(4096, 4096, U16, 100)
    assert p["path"] == "scratch" and p["scratch_bytes"] >= 256 * 2 * p["box_w"] * p["box_h"]


def test_fitted_shapes_are_told():
    """Where the default shape (mf_query_plan) is fitted to the image, the call's
    own shape is reported."""
    fp = mf.Footprint.disc(24)
    assert mf.query_plan(641, 479, U16, fp)["tile_h"] == 64
    p = mf.query_call(641, 479, U16, fp)
    tiles = -(-641 // p["tile_w"]) * -(-479 // p["tile_h"])
    assert p["path"] == "lds" and 88 < tiles <= 512
    fp = mf.Footprint.disc(48)
    assert (mf.query_plan(4096, 4096, U16, fp)["tile_w"], mf.query_plan(4096, 4096, U16, fp)["tile_h"]) \
        == (64, 96)
    assert mf.query_call(4096, 4096, U16, fp)["path"] == "scratch"
    big = mf.Footprint.disc(32)
    a, b = mf.query_plan(4096, 4096, U16, big), mf.query_call(4096, 4096, U16, big)
    assert all(a[k] == b[k] for k in a)


def test_tile_override_takes_calls_to_the_tile_engine():
    fp = mf.Footprint.disc(4)
    mf.set_tile_override(32, 16)
    try:
        p = mf.query_call(256, 256, U8, fp)
        assert (p["path"], p["tile_w"], p["tile_h"]) == ("lds", 32, 16)
    finally:
        mf.set_tile_override(0, 0)
    assert mf.query_call(256, 256, U8, fp)["path"] == "bits"


def test_refused_arguments_and_windows():
    L = mf.lib()
    fp = mf.Footprint.disc(4)
    none = [None] * 8
    assert L.mf_query_call(10, 10, 7, fp.handle, *none) == -1
    assert L.mf_query_call(0, 10, U8, fp.handle, *none) == -1
    assert L.mf_query_call(10, 10, U8, None, *none) == -1
    assert L.mf_query_call(10, 10, U8, fp.handle, *none) == 0
    wide = mf.Footprint.polygon([(-150, -1), (149, -1), (149, 0), (-150, 0)])
    for dt in (U8, U16, F32):
        with pytest.raises(mf.MedianFilterError) as e:
            mf.query_call(4096, 4096, dt, wide)
        assert e.value.status == -3


def test_launches_stay_below_two_to_the_32_threads():
    """An 8-bit image of 10 Gpixel: a window that 16 lanes share would take half a
    thread to the pixel on bit planes."""
    fp = mf.Footprint.disc(16)
    p = mf.query_call(4096, 4096, U8, fp)
    assert p["path"] == "bits"
    threads = -(-100000 // p["tile_w"]) * -(-100000 // p["tile_h"]) * 256
    assert threads >= 1 << 32
    assert mf.query_call(100000, 100000, U8, fp)["path"] == "lds"
    assert mf.query_call(100000, 100000, U8, mf.Footprint.disc(3))["path"] == "bits"


def test_scratch_of_float_tiles():
    """Float tiles sorted in LDS take an omnigram of two bytes a box pixel per
    workgroup, others the words of their sort as well (eight bytes)."""
    for w, h, r, each in ((3840, 2160, 48, 2), (4096, 4096, 40, 2), (3840, 2160, 100, 8)):
        p = mf.query_call(w, h, F32, mf.Footprint.disc(r))
        box = p["box_w"] * p["box_h"]
        assert p["path"] == "scratch" and each * box * 256 <= p["scratch_bytes"] <= \
            (each * (box + 24) + 256) * 256, (r, p)


def test_flat_images_keep_the_shorter_tiles():
    """A middle window takes the tall global-scratch tiles only where the image
    gives them fewer box pixels to sort."""
    q = lambda w, h, dt, r: mf.query_call(w, h, dt, mf.Footprint.disc(r))["path"]  # noqa: E731
    for dt, r in ((F32, 42), (U16, 48), (U8, 48)):
        assert q(40000, 32, dt, r) == "lds" and q(40000, 48, dt, r) == "lds"
        assert q(40000, 256, dt, r) == "scratch" and q(4096, 4096, dt, r) == "scratch"


@pytest.mark.gpu
def test_batches_of_small_images_keep_the_shorter_tiles():
    """So do batches of few tiles, which last their longest one."""
    torch = pytest.importorskip("torch")
    fp = mf.Footprint.disc(42)
    for side, n, scratch in ((16, 20000, False), (33, 4500, False), (128, 300, True), (256, 80, True),
                             (128, 20, False), (256, 1, False)):
        img = torch.zeros((n, side, side), dtype=torch.float32, device="cuda")
        out = torch.empty_like(img)
        plan = mf.BatchPlan([(img[i], out[i], fp, "clamp") for i in range(n)])
        assert (plan.info()["scratch_bytes"] > 0) == scratch, (side, n)
        plan.close()


def test_shapes_of_small_windows_on_middle_images():
    """Walks under small windows grow with the box, so few taps keep low tiles:
    float32 radius 2 on 721 x 2197 takes 389 us in 64 x 32 tiles and 738 in one
    round of 64 x 112."""
    mf.set_bits_override(mf.BITS_OFF)
    try:
        for w, h, dt, r in ((721, 2197, F32, 2), (825, 1576, F32, 2), (724, 2170, F32, 3),
                            (2379, 675, F32, 11), (1640, 1124, F32, 13), (2125, 574, U8, 2),
                            (929, 977, U16, 1)):
            fp = mf.Footprint.disc(r)
            p, d = mf.query_call(w, h, dt, fp), mf.query_plan(w, h, dt, fp)
            assert p["tile_h"] <= d["tile_h"], (w, h, dt, r, p, d)
        p = mf.query_call(641, 479, U16, mf.Footprint.disc(24))
        assert p["tile_w"] * p["tile_h"] < 64 * 64
    finally:
        mf.set_bits_override(mf.BITS_AUTO)


def test_line_between_the_paths():
    """The largest disc on bit planes at 4096 x 4096."""
    q = lambda w, h, dt, r: mf.query_call(w, h, dt, mf.Footprint.disc(r))["path"]  # noqa: E731
    for dt, r in ((U8, 16), (U16, 12), (F32, 10)):
        assert q(4096, 4096, dt, r) == "bits" and q(4096, 4096, dt, r + 6) == "lds"
    assert q(641, 479, U8, 16) == "bits" and q(300, 300, U16, 24) == "lds"
