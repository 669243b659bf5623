"""The choice of a block pass plan, on the host (no GPU): ordinary plates keep
the steps per pass measured fastest on them; bodies dense in boundary nodes take
fewer, or the tile launches, whatever is predicted to cost less, and no body is
cut into more patches than could pay (`plan_harness.cpp`)."""
import hashlib
import os
import shutil
import subprocess
import tempfile
import time

import numpy as np
import pytest

import test_patches_cpu as patches

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_2301_00228_amd", "csrc")
SOURCES = [os.path.join(ROOT, "tests", f) for f in ("plan_harness.cpp", "tiles_harness.cpp")]
SOURCES += [os.path.join(CSRC, f) for f in ("lbm_host.cpp", "lbm_types.h", "lbm_kernels.h", "lbm_patches.h")]
SOURCES.append(os.path.join(ROOT, "include", "lbm.h"))
F64, F32, F32DEV, F16DEV, BF16DEV = range(5)
DEFAULT_K = {F64: 5, F32: 6, F32DEV: 6, F16DEV: 5, BF16DEV: 5}


@pytest.fixture(scope="module")
def harness():
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    h = hashlib.sha256()
    for f in SOURCES:
        with open(f, "rb") as fh:
            h.update(fh.read())
    exe = os.path.join(tempfile.gettempdir(), f"lbm_plan_harness_{h.hexdigest()[:16]}")
    if not os.path.exists(exe):
        r = subprocess.run([HIPCC, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                            SOURCES[0], "-o", exe + ".tmp"], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        os.replace(exe + ".tmp", exe)
    return exe


def plan(exe, mask, storage, readings=0, periodic=(0, 0)):
    ny, nx = mask.shape
    text = f"1\n{storage} {readings} {nx} {ny} {periodic[0]} {periodic[1]}\n"
    text += "\n".join("".join("1" if v else "0" for v in row) for row in mask) + "\n"
    t0 = time.perf_counter()
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-2000:])
    lines = r.stdout.split("\n")
    use, K, rows, inner_rows, patches, inner = (int(v) for v in lines[0].split()[1:7])
    us, tiles = (float(v) for v in lines[0].split()[7:9])
    by_k = {int(a): float(b) for a, b in (x.split() for x in lines[1:6])}
    print(storage, readings, lines[0], by_k, f"{time.perf_counter() - t0:.2f} s")
    return dict(use=use, K=K, rows=rows, patches=patches, inner=inner, us=us, tiles=tiles, by_k=by_k)


def perforated(n, r, p):
    y, x = np.mgrid[0:n, 0:n]
    cx, cy = (x + p / 2) % p - p / 2, (y + p / 2) % p - p / 2
    m = (cx * cx + cy * cy >= r * r).astype(np.uint8)
    m[:3], m[-3:], m[:, :3], m[:, -3:] = 1, 1, 1, 1
    return m


def bars(n, w, p):
    m = np.zeros((n, n), np.uint8)
    for o in range(0, n - w + 1, p):
        m[o:o + w] = 1
        m[:, o:o + w] = 1
    return m


@pytest.mark.parametrize("storage", range(5))
def test_ordinary_plates_keep_their_steps_per_pass(harness, storage):
    hole = np.ones((1300, 1300), np.uint8)
    y, x = np.mgrid[0:1300, 0:1300]
    hole[(x - 650) ** 2 + (y - 650) ** 2 < 160 ** 2] = 0
    for mask, per in ((hole, (0, 0)), (np.ones((1500, 1200), np.uint8), (0, 0)),
                      (np.ones((1500, 1200), np.uint8), (1, 1)), (perforated(1000, 4.0, 64), (0, 0))):
        p = plan(harness, mask, storage, periodic=per)
        assert p["use"] and p["K"] == DEFAULT_K[storage] and p["inner"] > 0


@pytest.mark.parametrize("storage", range(5))
@pytest.mark.parametrize("body", [(4.0, 12), (6.0, 16), (2.5, 8)])
def test_perforated_bodies_take_the_cheapest_steps_per_pass(harness, storage, body):
    p = plan(harness, perforated(600, *body), storage)
    assert p["use"] and p["us"] < p["tiles"] and p["K"] < DEFAULT_K[storage]
    # (the K tried: from the default down; a K of more patches than pay is not cut)
    cut = [u for K, u in p["by_k"].items() if K <= DEFAULT_K[storage] and u > 0]
    assert p["us"] <= 1.0001 * min(cut) or p["us"] < 0.5 * p["tiles"]


@pytest.mark.parametrize("storage", range(5))
def test_bars_two_nodes_wide_take_the_tile_launches(harness, storage):
    p = plan(harness, bars(600, 2, 8), storage)
    assert not p["use"]
    assert all(u == 0 or u > p["tiles"] for u in p["by_k"].values())


def test_other_readings(harness):
    assert plan(harness, np.ones((300, 300), np.uint8), F64, 3)["K"] == 5
    p = plan(harness, perforated(600, 6.0, 16), F16DEV, 3)
    assert p["use"] and p["K"] < 5
    assert not plan(harness, bars(600, 2, 8), F32, 3)["use"]


patches_harness = patches.harness


def test_patches_of_few_steps_on_dense_bodies(patches_harness):
    # (validity carried forward through every patch, see test_patches_cpu)
    plans = [(K, rows, inner, r) for K in (2, 3) for rows, inner, r in ((4, 28, 0), (5, 40, 0), (5, 36, 0), (6, 48, 0),
                                                                       (3, 24, 0), (3, 24, 1))]
    F = (False, False)
    patches.check(patches_harness, [(perforated(150, 4.0, 12), F), (perforated(90, 2.5, 8), F), (bars(110, 3, 9), F),
                                    (perforated(96, 6.0, 16), (True, False))], plans)
