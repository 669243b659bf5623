"""The tile launches themselves: one step per launch, two-step pairs, pairs
overlapped on two streams, eager and captured, in the tests of
``test_gpu_parity`` and ``test_gpu_full_size`` written for them, with block
passes turned off in every context (under a two-step tiling they would run
otherwise), and against block passes over longer runs."""
import numpy as np
import pytest

import test_gpu_full_size as full
import test_gpu_parity as parity
from paper_2301_00228_amd import experiments as E
from paper_2301_00228_amd import inputs as I
from paper_2301_00228_amd import lbm

pytestmark = pytest.mark.gpu

FIELDS = ("e", "omega", "u", "v")
PAIRS = (64, 8, 0, 4, 0, 2, 4)

# (the module fixtures that the tests below take)
_device = parity._device
hole8192 = full.hole8192
reference = full.reference

# (the full-size oracle runs, shared by the tests of both modules in one process:
# two minutes of them)
_refs, _oracle = {}, full.run_case


def _run_case(case, steps=None, **kw):
    u0 = case.u0
    key = (case.name, case.nx, case.ny, case.nu, case.steps if steps is None else steps, len(case.bcs),
           float(u0[0].sum()), float(u0[1].sum()), float(abs(u0).max()), tuple(sorted(kw.items())))
    if key not in _refs:
        _refs[key] = _oracle(case, steps=steps, **kw)[0]
    return _refs[key], None


full.run_case = _run_case

_TILED = [parity.test_clamped_plates_ragged_and_tiny, parity.test_two_step_tiles_match_the_oracle,
          parity.test_two_step_batch_and_split_stepping_bitwise,
          parity.test_overlapped_pairs_are_bitwise_identical,
          parity.test_overlapped_pairs_other_storages_and_modes,
          parity.test_overlap_switched_mid_run_and_odd_step_counts,
          parity.test_reduced_storages_bitwise_across_tilings, parity.test_switching_steps_per_pass_mid_run,
          parity.test_autotune_keeps_the_trajectory, parity.test_split_stepping_equals_one_call,
          parity.test_graphs_of_any_step_count_are_bitwise_and_counted,
          parity.test_reading_switches_r2_m2_match_the_oracle, parity.test_blow_up_is_reported]
_TILED += [v for k, v in sorted(vars(full).items()) if k.startswith("test_")]


@pytest.fixture(autouse=True)
def _tile_launches(request, monkeypatch):
    """Contexts without block passes, for the tests taken from other modules."""
    if request.function not in _TILED:
        return
    made = lbm.Context.__init__

    def init(self, *a, **kw):
        made(self, *a, **kw)
        self.use_blocks(False)

    monkeypatch.setattr(lbm.Context, "__init__", init)


for _t in _TILED:
    globals()[_t.__name__] = _t


def _run(cases, storage, calls, tiling=None, overlap=True, graphs=True):
    with lbm.context_for(cases, storage) as ctx:
        if tiling:
            ctx.use_blocks(False)
            ctx.set_tiling(*tiling)
            ctx.use_overlap(overlap)
        ctx.use_graphs(graphs)
        for n in calls:
            ctx.step(n)
        return [ctx.fields(p) for p in range(len(cases))]


@pytest.mark.parametrize("storage", ["f64", "f32", "f32dev", "f16dev", "bf16dev"])
def test_pairs_against_block_passes(storage):
    cases = [I.plate_with_hole(n=260, radius=40, sigma=6.0, steps=0), E.paper_case("shear", 120, 95, t_end=1.0),
             I.clamped_plate(n=301, ny=187, sigma=9.0, steps=0)]
    for c in cases:
        c.sync_every = 50
    base = _run(cases, storage, (400,))
    for overlap, graphs in ((True, True), (True, False), (False, True)):
        got = _run(cases, storage, (151, 2, 47, 200), PAIRS, overlap, graphs)
        for a, b in zip(base, got):
            for k in FIELDS:
                assert np.isfinite(a[k]).all() and np.array_equal(a[k], b[k]), (storage, overlap, graphs, k)


def test_blocks_switched_mid_run():
    cases = [I.plate_with_hole(n=150, radius=20, sigma=4.0, steps=0, sync_every=40)]
    base = _run(cases, "f64", (200,))
    with lbm.context_for(cases) as ctx:
        assert ctx.profile(1)["two_step"][1] == 1  # (a block pass)
        for n, on in ((30, False), (31, True), (7, False), (1, True), (12, True), (9, False)):
            ctx.use_blocks(on)
            ctx.set_tiling(*PAIRS)
            ctx.step(n)
        ctx.use_blocks(False)
        ctx.autotune(1)
        ctx.use_blocks(True)
        ctx.step(200 - ctx.info()["steps_done"])
        got = [ctx.fields(p) for p in range(len(cases))]
    for a, b in zip(base, got):
        for k in FIELDS:
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("storage", ["f64", "f32", "f32dev", "f16dev", "bf16dev"])
def test_long_runs_past_the_rim_and_the_outer_edges(storage):
    """1500 steps of a pulse between a large hole and the outer edges, which it
    reaches both: block passes, pairs and single steps, bit for bit (a
    difference anywhere in the far field would have grown into all of it)."""
    case = I.plate_with_hole(n=1200, radius=500, sigma=4.0, steps=0, a0_phi=0.99)
    print("case", case.name, storage, flush=True)
    calls = (700, 1, 799)
    (base,) = _run([case], storage, calls)
    rim = I.boundary_nodes(case.mask)
    outer = (rim[:, 0] == 0) | (rim[:, 0] == 1199) | (rim[:, 1] == 0) | (rim[:, 1] == 1199)
    for part in (rim[outer], rim[~outer]):  # (the pulse: u up to 1e-3 over 4 nodes)
        assert np.abs(base["e"][part[:, 1], part[:, 0]]).max() > 1e-3 * (1e-3 / 4)
    for tiling in ((128, 8, 0, 2, 0, 1), PAIRS):
        (got,) = _run([case], storage, calls, tiling)
        for k in FIELDS:
            assert np.isfinite(base[k]).all() and np.array_equal(base[k], got[k]), (storage, tiling, k)


def test_profile_times_what_the_autotuner_picked():
    cases = [I.plate_with_hole(n=400, radius=50, sigma=6.0, steps=0)]
    with lbm.context_for(cases) as ctx:
        for blocks in (True, False):
            ctx.use_blocks(blocks)
            ctx.set_tiling(*PAIRS)
            ctx.autotune(1)
            assert ctx.block_info()["in_use"] == int(blocks)  # (0.4 of the best tiling's time)
            prof, steps = ctx.profile(10), ctx.block_info()["steps"]
            assert (prof["interior"][1] == 0) == blocks, prof
            if blocks:
                assert prof["two_step"][1] >= 10 // steps, prof
