"""Nested grids (swe_nest_*) against the nested-grid oracle: coarse-first
subcycling by r, frames from the coarse layers, restriction and reflux
(arXiv 1705.00614 Sec. 2.2 and Sec. 5).  Bars: FP64 <= 1e-10 relative L1 on
the coarse grid and every patch, clocks and time steps to 1e-12; FP32 within
the single-grid FP32 bar; dry-tile skipping of the coarse grid and graph
replay change nothing (bitwise); the volume budget closes on a wet domain.
"""
import sys

import numpy as np
import pytest

from oracle.nest import OracleNest
from paper_1705_00614_amd import scenarios as S
from tests import parity as P

pytestmark = pytest.mark.gpu

swe = pytest.importorskip("paper_1705_00614_amd.swe")


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[gpu] %s" % request.node.nodeid, flush=True)
    sys.stdout.flush()
    yield


def _floodplain_nest(prec, wet=False, seed=4, n=48, r=4):
    sc = S.floodplain(n=n, h=50.0, seed=seed, q_peak=800.0, t_peak=300.0, sigma_t=200.0,
                      inlet_cells=4, precision=prec)
    if wet:
        sc["H0"] = np.maximum(sc["b"].max() + 1.0 - sc["b"], 0.0)
    return S.nest(sc, [(14, 10, 12, 10), (30, 26, 8, 12)], r=r, seed=9)


def _rel(a, b):
    return np.abs(a - b).sum() / max(np.abs(b).sum(), 1e-300)


def _compare(G, O, prec, label=""):
    """The single-grid bars of tests/parity.py (relative L1 of H and of
    (Qx, Qy) together, and per cell) on the coarse grid and every patch."""
    pairs = [(G.coarse_state(), O.coarse_state())]
    pairs += [(G.patch_state(k), O.patch_state(k)) for k in range(len(O.P))]
    for k, (g, o) in enumerate(pairs):
        P.check(g, o, prec, label="%s grid %d" % (label, k))


def _run_held(G, O, steps, prec):
    """Both sides take the oracle nest's coarse step of each layer, rounded
    to the stencil type (substeps: a quarter of it, exact in binary)."""
    for _ in range(steps):
        tc = O.next_taus()[0]
        tc = float(np.float32(tc)) if prec == 32 else tc
        G.hold_dt(tc)
        G.run(1)
        O.step(tc)


@pytest.mark.parametrize("wet", [False, True])
def test_nest_fp64_matches_oracle(wet):
    nest = _floodplain_nest(64, wet=wet)
    O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"])
    G = swe.Nest(nest)
    q0 = G.query()
    assert abs(q0["dt_coarse"] - O.tau_c) <= 1e-12 * O.tau_c
    assert abs(q0["dt_fine"] - O.tau_f) <= 1e-12 * O.tau_f
    for _ in range(3):
        G.run(8)
        O.run(8)
        _compare(G, O, 64)
    for k in range(len(O.P)):                 # the patches carry flow
        Hf, Qxf, Qyf = O.patch_state(k)
        assert (Hf > 1e-4).any() and np.abs(Qxf).max() + np.abs(Qyf).max() > 1e-6
    q = G.query()
    assert q["steps"] == 24
    assert abs(q["time"] - O.time()) <= 1e-12 * O.time()
    assert abs(q["dt_coarse"] - O.tau_c) <= 1e-12 * O.tau_c
    assert abs(q["inflow"] - O.inflow()) <= 1e-11 * O.inflow()
    assert abs(q["volume"] - O.volume()) <= 1e-12 * O.volume()
    assert abs(q["ledger"] - O.total_ledger()) <= 1e-9 * q["volume"]
    if wet:
        assert abs(q["volume"] - q0["volume"] - q["inflow"] - q["ledger"]) <= 1e-12 * q["volume"]


def test_nest_one_way_matches_oracle():
    nest = _floodplain_nest(64)
    O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"], feedback=False)
    G = swe.Nest(nest, feedback=False)
    G.run(16)
    O.run(16)
    _compare(G, O, 64)


def test_nest_fp32_matches_oracle_at_held_steps():
    """FP32 nest over 48 coarse steps at the oracle nest's time steps.  The
    nest's CFL rule takes the minimum over the coarse grid and r times every
    patch, so a film in any grid can set it, and with free steps FP32
    rounding alone parts two oracle runs beyond 1e-4
    (tests/test_oracle_conditioning.py); with the steps held it stays at the
    single-grid level.  The rule itself is checked in FP64 (clock and both
    step lengths to 1e-12 above)."""
    nest = _floodplain_nest(32)
    O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"])
    G = swe.Nest(nest)
    _run_held(G, O, 48, 32)
    _compare(G, O, 32, "held")
    assert G.query()["time"] == O.time()


def test_nest_hold_then_release_follows_the_cfl_rule():
    nest = _floodplain_nest(64)
    O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"])
    G = swe.Nest(nest)
    _run_held(G, O, 5, 64)
    G.hold_dt(0.0)
    q = G.query()
    tc, tf = O.next_taus()
    assert abs(q["dt_coarse"] - tc) <= 1e-12 * tc and abs(q["dt_fine"] - tf) <= 1e-12 * tf
    G.run(11)
    O.run(11)
    _compare(G, O, 64, "released")


@pytest.mark.parametrize("prec", [32, 64])
def test_nest_skip_and_graph_are_exact(prec):
    nest = _floodplain_nest(prec)
    a = swe.Nest(nest)                      # coarse skips dry tiles, graphs of 8 steps
    b = swe.Nest(nest, skip_dry=False)
    c = swe.Nest(nest)
    a.run(19)
    b.run(19)
    c.run_timed(19)                         # one launch sequence per step, no graph
    for other in (b, c):
        for x, y in zip(a.coarse_state(), other.coarse_state()):
            assert np.array_equal(x, y)
        for k in range(2):
            for x, y in zip(a.patch_state(k), other.patch_state(k)):
                assert np.array_equal(x, y)
        assert a.query()["time"] == other.query()["time"]


def test_nest_r2_and_r1():
    for r in (1, 2):
        sc = S.random_state(40, 36, seed=21, wet_frac=0.7, precision=64)
        nest = S.nest(sc, [(9, 8, 14, 12)], r=r, detail=0.0 if r == 1 else 0.3)
        O = OracleNest(nest["coarse"], nest["patches"], r=r)
        G = swe.Nest(nest)
        G.run(12)
        O.run(12)
        _compare(G, O, 64)


def test_nest_rejects_bad_layouts():
    sc = S.floodplain(n=48, h=50.0, seed=4, inlet_cells=4, precision=64)
    nest = S.nest(sc, [(14, 10, 12, 10)], r=4, seed=9)
    bad = dict(nest, patches=[dict(nest["patches"][0], ci0=1)])
    with pytest.raises((swe.SweError, ValueError)):
        swe.Nest(bad)
    two = S.nest(sc, [(14, 10, 6, 6), (20, 10, 6, 6)], r=4, seed=9)
    with pytest.raises(swe.SweError):
        swe.Nest(two)


def test_nest_of_64_patches_matches_oracle_and_65_are_refused():
    """The time-step rule reads one patch per lane of a wave: 64 patches
    (every lane) follow the oracle nest; a 65th is refused at creation."""
    sc = S.random_state(40, 40, seed=23, wet_frac=0.7, precision=64)
    boxes = [(3 + 4 * (k % 8), 3 + 4 * (k // 8), 2, 2) for k in range(64)]
    nest = S.nest(sc, boxes, r=2, seed=11, detail=0.3)
    O = OracleNest(nest["coarse"], nest["patches"], r=2)
    G = swe.Nest(nest)
    G.run(10)
    O.run(10)
    assert abs(G.query()["time"] - O.time()) <= 1e-12 * O.time()
    _compare(G, O, 64, label="64 patches")
    more = S.nest(sc, boxes + [(3, 35, 2, 2)], r=2, seed=11, detail=0.3)
    with pytest.raises(swe.SweError):
        swe.Nest(more)


@pytest.mark.parametrize("prec,vs_oracle,box", [(64, True, (20, 24, 44, 40)), (32, False, (20, 24, 44, 40)),
                                                 (64, True, (22, 26, 46, 38))])
def test_patches_skip_dry_tiles_exactly(prec, vs_oracle, box):
    """Patches skip dry tiles except the ring of tiles holding the frame,
    which the nest rewrites between substeps (also where the frame straddles
    two tile columns and rows): a patch large enough to have dry interior
    tiles while the flood arrives processes fewer fine cells,
    bit for bit the same as without skipping, and (FP64) matches the
    oracle."""
    sc = S.floodplain(n=96, h=50.0, seed=6, q_peak=2500.0, t_peak=600.0, sigma_t=300.0,
                      inlet_cells=4, precision=prec)
    # (46, 38): 194 x 162 fine cells with the frame, so the frame's last
    # columns and rows straddle two tiles.  The boxes are ones where the
    # oracle nest is well conditioned in FP64 (a 1e-15 change of the bed
    # moves it by < 1e-13 after 40 steps, tests/test_oracle_conditioning.py);
    # boxes of 30 x 38 at (20, 22) and 44 x 40 at (24, 24) move by 3e-8, so
    # they cannot pin 1e-10.
    nest = S.nest(sc, [box], r=4, seed=3)
    a = swe.Nest(nest)
    b = swe.Nest(nest, skip_dry=False)
    a.run(40)
    b.run(40)
    for x, y in zip(a.patch_state(0), b.patch_state(0)):
        assert np.array_equal(x, y)
    for x, y in zip(a.coarse_state(), b.coarse_state()):
        assert np.array_equal(x, y)
    assert a.query()["time"] == b.query()["time"]
    wa, wb = a.work(), b.work()
    assert wa["fine_cells"] < wb["fine_cells"]
    assert (a.patch_state(0)[0] > 1e-4).any()
    if vs_oracle:
        O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"])
        O.run(40)
        _compare(a, O, prec, "skip box %s" % (box,))


@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("n,boxes", [
    (24, [(8, 9, 5, 4)]),                                                         # fewer tiles than workgroup groups
    (200, [(4 + 32 * (k % 6), 4 + 32 * (k // 6), 3, 2) for k in range(36)]),      # 169 tiles, 64 workgroups per grid
])
def test_grids_share_a_launch(n, boxes, skip):
    """The grids of a nest step in one launch with the same number of
    workgroups each: more workgroups than a grid has tiles, and fewer than the
    coarse grid has.  FP64 against the oracle, the module's bars."""
    sc = S.random_state(n, n, seed=29, wet_frac=0.7, precision=64)
    nest = S.nest(sc, boxes, r=2, seed=5, detail=0.3)
    O = OracleNest(nest["coarse"], nest["patches"], r=2)
    G = swe.Nest(nest, skip_dry=skip)
    G.run(3)
    O.run(3)
    _compare(G, O, 64, label="n=%d" % n)


@pytest.mark.parametrize("r", [3, 5])
def test_fine_blocks_of_odd_refinement(r):
    """The fine cells of a covered cell and the taps of a face are summed in
    batches (16 cells, 4 taps): 9 and 25 cells, 3 and 5 taps leave ragged
    ones.  FP64 against the oracle, the module's bars."""
    sc = S.random_state(30, 26, seed=37, wet_frac=0.7, precision=64)
    nest = S.nest(sc, [(7, 6, 9, 7)], r=r, detail=0.3)
    O = OracleNest(nest["coarse"], nest["patches"], r=r)
    G = swe.Nest(nest)
    G.run(9)
    O.run(9)
    _compare(G, O, 64, label="r=%d" % r)


def test_full_size_nest_first_coarse_steps_match_oracle():
    """The nested-grid benchmark workload at its full size (2048^2 coarse
    grid at 50 m with two 2048^2 patches at 12.5 m, dry-tile skipping) for
    one 8-step graph replay, as the benchmark runs it, against the FP64
    nested oracle on every cell of the coarse grid and both patches.  The
    stencil runs in FP64 here so that the bar is the FP64 one (1e-10, as for
    the small nests); the FP32 configuration is covered by the small FP32
    nest and the bitwise skip and graph tests.  At this size covered coarse
    cells occur whose block mean is dry (H <= eps) while some fine cells
    carry water: they must store no discharge, like every dry cell."""
    nest = S.nest_floodplain(n=2048, h=50.0, seed=1, r=4, box=512, precision=64)
    G = swe.Nest(nest)
    O = OracleNest(nest["coarse"], nest["patches"], r=nest["r"])
    G.run(8)
    O.run(8)
    _compare(G, O, 64)
    assert abs(G.query()["time"] - O.time()) <= 1e-12 * O.time()
    for k in range(2):
        assert (G.patch_state(k)[0] > 0).any()   # the patches hold water


@pytest.mark.parametrize("skip", [True, False])
def test_grids_of_unequal_shares(skip):
    """Grids of 1 to 30 tiles take one to four groups of a launch's
    workgroups.  FP64 against the oracle, the module's bars."""
    sc = S.random_state(76, 72, seed=41, wet_frac=0.7, precision=64)
    nest = S.nest(sc, [(6, 6, 3, 2), (20, 6, 24, 10), (8, 24, 12, 30), (34, 34, 36, 32)], r=2, seed=5, detail=0.3)
    O = OracleNest(nest["coarse"], nest["patches"], r=2)
    G = swe.Nest(nest, skip_dry=skip)
    G.run(3)
    O.run(3)
    _compare(G, O, 64, label="skip=%s" % skip)
