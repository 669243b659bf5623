"""Which path runs: the tests of ``test_gpu_block`` again, with every context's
``lbm_block_info`` read -- block passes unless a tiling of one step per launch was
set (so that no plan is refused unnoticed), and the patch shapes that the shape
test is there for -- and a body that takes the tile launches."""
import numpy as np
import pytest

import test_gpu_block as block
from paper_2301_00228_amd import inputs as I
from paper_2301_00228_amd import lbm

pytestmark = pytest.mark.gpu

_device = block._device
SHAPES = "test_every_shape_of_patches_bitwise"
_BLOCKS = {k: v for k, v in vars(block).items() if k.startswith("test_") and "switching" not in k}
globals().update(_BLOCKS)


@pytest.fixture(autouse=True)
def _paths(request, monkeypatch):
    """Record the path of every context without a tiling of the caller's."""
    name = request.function.__name__
    if request.function not in _BLOCKS.values():
        yield
        return
    seen, tiled, made, tile = set(), set(), lbm.Context.close, lbm.Context.set_tiling

    def set_tiling(self, *a, **kw):
        tiled.add(id(self))
        tile(self, *a, **kw)

    def close(self):
        if getattr(self, "_h", None):
            b = self.block_info()
            if id(self) in tiled:
                tiled.discard(id(self))
                assert not b["in_use"], b
            else:
                seen.add((b["in_use"], b["steps"], b["rows"], b["inner_rows"], b["patches"] > 0,
                          b["inner_patches"] > 0))
        made(self)

    monkeypatch.setattr(lbm.Context, "set_tiling", set_tiling)
    monkeypatch.setattr(lbm.Context, "close", close)
    yield
    print(name, sorted(seen))
    assert seen
    assert {s[0] for s in seen} == {1}, seen
    if name == SHAPES:
        # one launch of 3 rows per wave and of more, two launches, one without boundary nodes
        assert any(s[2] == 3 and s[4] and not s[5] for s in seen)
        assert any(s[2] > 3 and s[4] and not s[5] for s in seen)
        assert any(s[4] and s[5] for s in seen)
        assert {s[3] for s in seen if not s[4]} >= {16}
        assert len({s[2] for s in seen if s[4]}) >= 2


def test_block_info_follows_the_settings():
    with lbm.context_for(I.plate_with_hole(n=700, radius=60, sigma=6.0, steps=0)) as ctx:
        b = ctx.block_info()
        assert b["in_use"] == 1 and b["steps"] > 1
        assert 0 < b["edge_patches"] <= b["patches"] and b["inner_patches"] > 0
        for call, in_use in ((lambda: ctx.use_blocks(False), 0), (lambda: ctx.use_blocks(True), 1),
                             (lambda: ctx.set_tiling(128, 8, 0, 2, 0, 1), 0), (lambda: ctx.use_blocks(False), 0),
                             (lambda: ctx.use_blocks(True), 0), (lambda: ctx.set_tiling(128, 8, 0, 2, 0, 2), 1)):
            call()
            assert ctx.block_info() == dict(b, in_use=in_use)
            ctx.step(3)


def perforated_everywhere(nx, ny, edge=3):
    """Single-node holes a knight's move apart: every node between them is a
    boundary node, and a patch owns few of the nodes that two steps depend on."""
    y, x = np.mgrid[0:ny, 0:nx]
    m = ((x + 2 * y) % 5 != 0).astype(np.uint8)
    m[:edge], m[-edge:], m[:, :edge], m[:, -edge:] = 1, 1, 1, 1
    return m


@pytest.mark.parametrize("storage", block.STORAGES)
def test_a_body_without_a_plan_takes_the_tile_launches(storage):
    case = block.clamped(400, 300)
    case.mask = perforated_everywhere(400, 300)
    case.u0, case.bcs = case.u0 * case.mask, []
    with lbm.context_for(case, storage) as ctx:
        assert set(ctx.block_info().values()) == {0}
    block.same([case], storage, (5, 30))
    # (pairs of its tiles)
    a, b = (block.run([case], storage, (5, 30), t) for t in (block.SINGLE, (64, 8, 0, 4, 0, 2, 4)))
    for k in block.FIELDS:
        assert np.array_equal(a[0][k], b[0][k]), k


@pytest.mark.parametrize("readings", [(0, 0), (1, 1)])
@pytest.mark.parametrize("storage", block.STORAGES)
def test_bodies_dense_in_boundary_nodes_bitwise(storage, readings):
    # (fewer steps per pass than large plates take)
    y, x = np.mgrid[0:500, 0:530]
    steps = set()
    for r, p in ((4.0, 12), (6.0, 16), (2.5, 8)):
        case = block.clamped(530, 500, a0_phi=0.99)
        cx, cy = (x + p / 2) % p - p / 2, (y + p / 2) % p - p / 2
        m = (cx * cx + cy * cy >= r * r).astype(np.uint8)
        m[:3], m[-3:], m[:, :3], m[:, -3:] = 1, 1, 1, 1
        case.mask, case.u0, case.readings = m, case.u0 * m, readings
        with lbm.context_for(case, storage) as ctx:
            b = ctx.block_info()
        assert b["in_use"], b
        steps.add(b["steps"])
        block.same([case], storage, (1, 6, 52))
    print("steps per pass", steps)
    assert min(steps) <= 3 and max(steps) <= 5


def test_single_steps_and_synchronized_steps_of_large_plates_take_tiles():
    # (a state past the 256 MB of the Infinity Cache, and one within it)
    for n, large in ((1300, True), (700, False)):
        for sync, calls, count, tiles in ((50, 1, 1, large), (1, 3, 3, large), (2, 4, 2, False)):
            case = block.clamped(n, n - 7)
            case.sync_every = sync
            with lbm.context_for(case) as ctx:
                kinds = ctx.profile(calls)
            assert kinds["interior" if tiles else "two_step"][1] == count, (n, sync, kinds)
            assert kinds["two_step" if tiles else "interior"][1] == 0, (n, sync, kinds)
            assert kinds["sync"][1] == (calls // sync), (n, sync, kinds)
            block.same([case], "f64", (4, 1, 7))


@pytest.mark.parametrize("storage", block.STORAGES)
def test_few_steps_of_thin_and_small_plates_take_tiles(storage):
    small = [block.clamped(60 + 3 * k % 41, 60 + 7 * k % 41) for k in range(100)]
    for cases, tiles in (([block.clamped(20000, 4)], 1), (small, 1 if storage == "f64" else None),
                         ([block.clamped(4, 20000)], 0), ([block.clamped(300, 280)], 0)):
        for n in (1, 7):
            with lbm.context_for(cases, storage) as ctx:
                assert ctx.block_info()["in_use"]
                kinds = ctx.profile(n)
            # (near the line in the 4-byte storages)
            assert tiles is None or (kinds["interior"][1] > 0) == (n <= tiles), (cases[0].name, n, kinds)
        print(cases[0].name, len(cases), flush=True)
        block.same(cases, storage, (3, 1, 1, 2, 9, 1))
