"""The block pass (several steps of a patch per launch, the default) against
the CPU oracle and, bit for bit, against one step per launch (a tiling with
steps = 1): plates at and around the patch sizes (64 columns, 28 or 32 rows
less the halos), thin and tiny ones, holes, periodic axes, ramped loads, step
counts that are no multiple of the pass, every storage."""
import numpy as np
import pytest

from oracle.oracle import run_case
from paper_2301_00228_amd import experiments as E
from paper_2301_00228_amd import inputs as I
from paper_2301_00228_amd import lbm

pytestmark = pytest.mark.gpu

FIELDS = ("e", "omega", "u", "v")
SINGLE = (128, 8, 0, 2, 0, 1)
STORAGES = ["f64", "f32", "f32dev", "f16dev", "bf16dev"]


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)


def run(cases, storage, calls, tiling=None):
    with lbm.context_for(cases, storage) as ctx:
        if tiling:
            ctx.set_tiling(*tiling)
        for n in calls:
            ctx.step(n)
        return [ctx.fields(p) for p in range(len(cases))]


def same(cases, storage, calls):
    print("case", [(c.name, c.nx, c.ny) for c in cases], storage, calls, flush=True)
    for a, b in zip(run(cases, storage, calls, SINGLE), run(cases, storage, calls)):
        for k in FIELDS:
            assert np.isfinite(a[k]).all() and np.array_equal(a[k], b[k]), (storage, k)


def clamped(nx, ny, **kw):
    return I.clamped_plate(n=nx, ny=ny, sigma=max(1.0, min(nx, ny) / 12), steps=0, **kw)


@pytest.mark.parametrize("sizes", [[(64, 28), (65, 29), (63, 32), (57, 21)], [(3, 3), (3, 90), (130, 3), (25, 25)],
                                   [(112, 50), (113, 75), (240, 100)]])
def test_ragged_plates_bitwise(sizes):
    same([clamped(nx, ny) for nx, ny in sizes], "f64", (1, 2, 3, 4, 5, 50, 23))


@pytest.mark.parametrize("storage", STORAGES)
def test_storages_holes_and_loads_bitwise(storage):
    hole = I.plate_with_hole(n=150, radius=23, sigma=4.0, steps=0)
    ell = I.plate_with_ellipse_hole(nx=140, ny=96, a0_phi=0.99, steps=0)
    same([hole, ell, E.paper_case("shear", 70, 50, t_end=1.0)], storage, (6, 47, 31))


@pytest.mark.parametrize("nx,ny,per", [(3, 5, (True, True)), (60, 40, (True, True)), (129, 33, (True, True)),
                                       (70, 45, (True, False)), (45, 66, (False, True))])
def test_periodic_axes_bitwise(nx, ny, per):
    cases = []
    for integrator in (0, 1):
        c = clamped(nx, ny, a0_phi=0.99)
        c.periodic, c.bcs, c.integrator, c.sync_every = per, [], integrator, 0
        cases.append(c)
    same(cases, "f64", (9, 30))


@pytest.mark.parametrize("storage", STORAGES)
def test_every_shape_of_patches_bitwise(storage):
    # one launch with 3 to 6 rows per wave; two launches, few edges and many;
    # without boundary nodes, small and large
    many = I.plate_batch(count=4, side_lo=500, side_hi=900, steps=0)
    for cases in ([clamped(300, 280)], [clamped(500, 515)], [clamped(645, 600)], [clamped(1031, 517)],
                  [I.plate_with_hole(n=1100, radius=130, sigma=8.0, steps=0)], many):
        same(cases, storage, (7, 52))
    # (single steps of a state past the Infinity Cache: the tile launches)
    same([clamped(2100, 1000), clamped(2000, 900)], storage, (1, 1, 6, 1, 49, 1))
    for nx, ny in ((190, 131), (820, 803)):
        c = clamped(nx, ny, a0_phi=0.99)
        c.periodic, c.bcs, c.sync_every = (True, True), [], 0
        same([c], storage, (7, 52))


@pytest.mark.parametrize("readings", [(1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("storage", STORAGES)
def test_other_readings_bitwise(storage, readings):
    hole = I.plate_with_hole(n=150, radius=23, sigma=4.0, steps=0, a0_phi=0.99)
    shear = E.paper_case("shear", 70, 50, t_end=1.0)
    open_x = clamped(90, 61, a0_phi=0.99)
    open_x.periodic, open_x.bcs = (True, False), []
    for c in (hole, shear, open_x):
        c.readings = readings
    # (with a plate of the default readings, which then runs in the same launch)
    same([hole, shear, open_x, clamped(40, 37, a0_phi=0.99)], storage, (6, 47, 31))


def test_strip_with_holes_matches_the_oracle():
    case = I.strip_with_holes(nx=500, ny=120, sigma=6.0, pulses=3, steps=103, seed_index=7)
    ref, _ = run_case(case)
    (got,) = run([case], "f64", (case.steps,))
    for k in FIELDS:
        assert np.abs(got[k] - ref[k]).max() <= 1e-12 * np.abs(ref[k]).max(), k


def test_switching_between_block_passes_and_tiles_mid_run():
    cases = [I.plate_with_hole(n=130, radius=18, sigma=4.0, steps=0, sync_every=40), clamped(90, 61, sync_every=40)]
    base = run(cases, "f64", (150,), SINGLE)
    with lbm.context_for(cases) as ctx:
        ctx.step(31)
        ctx.set_tiling(*SINGLE)
        ctx.step(10)
        ctx.set_tiling(64, 8, 0, 4, 0, 2, 4)
        ctx.step(33)
        ctx.profile(9)  # (the tile launches of that tiling)
        ctx.step(7)
        ctx.autotune(1)
        ctx.step(150 - ctx.info()["steps_done"])
        got = [ctx.fields(p) for p in range(len(cases))]
    for a, b in zip(base, got):
        for k in FIELDS:
            assert np.array_equal(a[k], b[k]), k


def test_a_body_too_dense_to_cut_takes_the_tile_launches():
    # bars two nodes wide: every node is a boundary node
    m = np.zeros((60, 66), np.uint8)
    for o in range(0, 60, 4):
        m[o:o + 2, :] = 1
    for o in range(0, 64, 4):
        m[:, o:o + 2] = 1
    case = clamped(66, 60)
    case.mask, case.u0 = m, case.u0 * m
    case.bcs = []
    same([case], "f64", (5, 30))
