"""The block pass's patches, checked on the host (no GPU).

The patches of a plan own every body node once, fit the workgroup, list every
boundary node they hold with its record, place and stencils, and hold every
node that the plan's steps of their owned nodes depend on: validity carried
forward step by step from nothing outside the patch reaches all owned nodes
(`patches_harness.cpp`; the library derives the patches backwards).
"""
import hashlib
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from paper_2301_00228_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_2301_00228_amd", "csrc")
SOURCES = [os.path.join(ROOT, "tests", "patches_harness.cpp"),
           os.path.join(ROOT, "tests", "tiles_harness.cpp"),
           os.path.join(ROOT, "include", "lbm.h")]
SOURCES += [os.path.join(CSRC, f) for f in ("lbm_host.cpp", "lbm_types.h", "lbm_kernels.h", "lbm_patches.h")]
# steps, rows per wave, rows of a patch without boundary nodes, reading R2
PLANS = [(4, 4, 32, 0), (2, 2, 16, 0), (1, 2, 8, 0), (3, 4, 28, 0), (5, 3, 24, 0), (5, 4, 28, 0), (5, 5, 40, 0),
         (6, 3, 16, 0), (6, 5, 40, 0), (6, 6, 48, 0), (5, 3, 24, 1), (4, 3, 24, 1)]


@pytest.fixture(scope="module")
def harness():
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    h = hashlib.sha256()
    for f in SOURCES:
        with open(f, "rb") as fh:
            h.update(fh.read())
    exe = os.path.join(tempfile.gettempdir(), f"lbm_patches_harness_{h.hexdigest()[:16]}")
    if not os.path.exists(exe):
        r = subprocess.run([HIPCC, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                            SOURCES[0], "-o", exe + ".tmp"], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        os.replace(exe + ".tmp", exe)
    return exe


def check(exe, plates, plans):
    lines = [str(len(plates))]
    for mask, (px, py) in plates:
        ny, nx = mask.shape
        lines.append(f"{nx} {ny} {int(px)} {int(py)}")
        lines.extend(" ".join(str(int(v)) for v in row) for row in mask)
    lines.append(str(len(plans)))
    lines += [" ".join(str(v) for v in p) for p in plans]
    r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, (r.stdout[-3000:], r.stderr[-2000:])


def full(nx, ny):
    return np.ones((ny, nx), np.uint8)


def test_rectangles_ragged_tiny_and_periodic(harness):
    F = (False, False)
    plates = [(full(3, 3), F), (full(7, 130), F), (full(131, 7), F), (full(259, 37), F), (full(64, 28), F),
              (full(65, 29), F), (full(300, 200), F), (full(96, 96), (True, True)), (full(5, 64), (False, True)),
              (full(3, 3), (True, True)), (full(200, 90), (True, False)), (full(32, 25), F)]
    check(harness, plates, PLANS)


def test_holes_and_curved_outlines(harness):
    rng = np.random.default_rng(7)
    F = (False, False)
    strip = full(260, 90)
    strip[30:52, 100:140] = 0
    plates = [(I.hole_mask(220, 40), F), (strip, (True, False)),
              (I.ellipse_holes_mask(300, 140, 0.05, rng, a_lo=4.0, a_hi=16.0)[0], F),
              (I.shape_mask(180, 150, [(90.3, 74.1, 80.0, 66.0, 0.3, 1), (84.0, 70.0, 20.0, 9.0, 1.1, 0)]), F)]
    check(harness, plates, PLANS)


def test_bodies_that_are_mostly_boundary(harness):
    # a lattice of bars three nodes wide, and bars two wide
    a = np.zeros((90, 110), np.uint8)
    for o in range(0, 90, 9):
        a[o:o + 3, :] = 1
    for o in range(0, 108, 9):
        a[:, o:o + 3] = 1
    b = np.zeros((40, 50), np.uint8)
    for o in range(0, 40, 8):
        b[o:o + 2, :] = 1
    for o in range(0, 48, 8):
        b[:, o:o + 2] = 1
    check(harness, [(a, (False, False)), (b, (False, False))], [(2, 2, 16, 0), (1, 2, 8, 0), (2, 4, 32, 0)])
