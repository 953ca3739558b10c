"""Vertical slides hold the positions of a window column's entering and leaving
pixels as 16-bit offsets.  Boxes 255 pixels wide under windows of 254 rows and
more come within a row of that limit: the offsets of every plan are checked on
the host (tests/native/slide_check.cpp), and tiles at the limit against the
oracle on the GPU."""

import os
import subprocess

import numpy as np
import pytest

import workloads
from oracle import footprints as OF

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_22938_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_offsets_on_the_host(tmp_path):
    exe = str(tmp_path / "slide_check")
    subprocess.check_call([
        "g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
        "-I", CSRC, os.path.join(ROOT, "tests", "native", "slide_check.cpp"),
        os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "footprint.cpp"),
        "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + os.path.join(ROCM, "lib"),
        "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]


def rect(w, h):
    x, y = -(w // 2), -(h // 2)
    return [(x, y), (x + w - 1, y), (x + w - 1, y + h - 1), (x, y + h - 1)]


# tile, window: (tile box 255 wide) 192 x 254 and 192 x 253 under three and four
# rows, discs of radius 127 and 126 under two and four, and one box of even pitch
@pytest.mark.gpu
@pytest.mark.parametrize("tile,make", [
    ((64, 3), lambda m: m.polygon(rect(192, 254))),
    ((64, 4), lambda m: m.polygon(rect(192, 253))),
    ((1, 2), lambda m: m.disc(127)),
    ((3, 4), lambda m: m.disc(126)),
    ((2, 2), lambda m: m.polygon(rect(254, 255))),
    ((63, 3), lambda m: m.polygon(rect(192, 254))),
])
@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
def test_tiles_at_the_limit(oracle_mod, dtype, tile, make):
    torch = pytest.importorskip("torch")
    import paper_2505_22938_amd as mf
    fp, ofp = make(mf.Footprint), make(OF)
    img = workloads.uniform(12, 9, dtype, 3) if dtype != "f32" else workloads.special_floats(12, 9, 3)
    dev = torch.from_numpy(np.ascontiguousarray(img)).cuda()
    mf.set_tile_override(*tile)
    try:
        for boundary in ("clamp", "mirror"):
            for rank in (None, fp.taps // 5):
                got = mf.median_filter(dev, fp, boundary, rank=rank)
                torch.cuda.synchronize()
                exp = oracle_mod.filter(img, ofp, boundary, rank=rank)
                assert np.array_equal(got.cpu().numpy().view(np.uint8), exp.view(np.uint8)), \
                    (boundary, rank)
    finally:
        mf.set_tile_override(0, 0)
