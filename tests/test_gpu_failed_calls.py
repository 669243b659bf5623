"""A call that cannot get its memory leaves a context that steps on: the state,
the tiling it had, and no launch on lists or buffers that are not there.  The
context's own allocator refuses from a given allocation on."""
import numpy as np
import pytest

from paper_2301_00228_amd import inputs as I
from paper_2301_00228_amd import lbm

pytestmark = pytest.mark.gpu

FIELDS = ("e", "omega", "u", "v")
SINGLE = (128, 8, 0, 2, 0, 1)
PAIRS = (64, 8, 0, 4, 0, 2, 4)


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)


class Allocator:
    """torch's allocator, which refuses once `left` allocations are done."""

    def __init__(self):
        base = lbm.torch_allocator()
        alloc, free, live = base._keep
        self.left, self.live = None, live

        @lbm.ALLOC_FN
        def limited(nbytes, user):
            if self.left is not None:
                if self.left <= 0:
                    return None
                self.left -= 1
            return alloc(nbytes, user)

        self.struct = lbm.lbm_alloc(limited, free, None)
        self._keep = (base, limited)


def cases():
    return [I.plate_with_hole(n=150, radius=20, sigma=4.0, steps=0, sync_every=40),
            I.clamped_plate(n=110, ny=81, sigma=4.0, steps=0, sync_every=40)]


def reference(total):
    with lbm.context_for(cases()) as ctx:
        ctx.set_tiling(*SINGLE)
        ctx.step(total)
        return [ctx.fields(p) for p in range(2)]


def refused(call):
    try:
        call()
    except lbm.LbmError as e:
        assert e.code == lbm.E_NOMEM, e
        return True
    return False


def check(ctx, total):
    ctx.step(total - ctx.info()["steps_done"])
    for got, ref in zip([ctx.fields(p) for p in range(2)], reference(total)):
        for k in FIELDS:
            assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("left", [0, 1, 3, 5, 6, 12, 25])
@pytest.mark.parametrize("tiling", [None, PAIRS])
def test_autotune_without_memory_leaves_the_tiling_and_the_state(tiling, left):
    print("case autotune", tiling, left, flush=True)
    a = Allocator()
    with lbm.context_for(cases(), allocator=a.struct) as ctx:
        if tiling:
            ctx.set_tiling(*tiling)
        ctx.step(33)
        before, held = ctx.info(), len(a.live)
        a.left = left
        failed = refused(lambda: ctx.autotune(1))
        a.left = None
        if left == 0:
            assert failed
        if failed:
            after = ctx.info()
            assert {k: after[k] for k in after if k.startswith("tile_")} == {
                k: before[k] for k in before if k.startswith("tile_")}
            assert len(a.live) <= held + left
        ctx.step(7)
        ctx.profile(6)
        check(ctx, 101)


@pytest.mark.parametrize("left", [0, 1, 2, 4, 8, 16])
def test_tilings_without_memory(left):
    # (one-row tiles: more of them than any list before has room for)
    print("case set_tiling", left, flush=True)
    a = Allocator()
    with lbm.context_for(cases(), allocator=a.struct) as ctx:
        ctx.step(21)
        for tiling in ((64, 1, 0, 0, 0, 1), (64, 1, 0, 0, 0, 2), SINGLE):
            a.left = left
            refused(lambda: ctx.set_tiling(*tiling))
            refused(lambda: ctx.step(5))
            refused(lambda: ctx.use_overlap(False))
            refused(lambda: ctx.prepare_steps(9))
            refused(lambda: ctx.profile(4))
            a.left = None
            ctx.step(9)
            ctx.use_overlap(True)
        check(ctx, 120)
