"""A launch deals its tracks evenly over its waves: histories against the
oracle at the edges of that rule (fewer tracks than waves, one to 64 tracks a
wave with and without remainder, more than the waves hold at once), with few
blocks so that small inputs reach them.  Bars: those of the random-track
history test (energies 1e-11, deposits 5e-11 relative, positions 1e-9 mm)."""
import dataclasses

import numpy as np
import pytest

import ems_inputs as I
from parity_util import compare_logs, ledger_residual
from test_gpu_parity import E, run_gpu  # noqa: F401  (E: the module fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,n", [(1, 1), (1, 4), (1, 5), (1, 4 * 63 + 1), (1, 257), (1, 700), (3, 23), (0, 300)])
def test_histories_at_the_edges_of_the_wave_shares(E, oracle_mod, blocks, n):  # noqa: F811
    print(f"{n} tracks, {blocks} blocks", flush=True)
    geo = I.calorimeter()
    cfg = I.RunConfig(seed=23)
    prim = I.random_tracks(n, n, geo, 1e-3, 50.0, seed=n)
    ref = oracle_mod.Oracle(geo, cfg).run(prim, n_events=n, log_cap=4_000_000)
    got = run_gpu(E, geo, cfg, prim, n, flags=E.F_STEPLOG | E.F_FULL_LEDGER, log_cap=1_000_000, blocks=blocks)
    assert got["n_log"] <= 1_000_000
    dev = compare_logs(got["log"], ref["log"], e_rtol=1e-11, pos_atol=1e-9, dep_rtol=5e-11)
    print(f"steps {dev['n']}: {dev}", flush=True)
    assert ledger_residual(got["edep"], got["ledger"], prim).max() < 1e-9


@pytest.mark.parametrize("n", [256 + 2047, 256 + 2112, 9000, 20001])
def test_index_chunks_by_what_is_left(E, oracle_mod, n):  # noqa: F811
    """One block of four waves takes its queue's indices 64 at a time, by an
    eighth of an even share of what is left, or 256 at a time: every track is
    visited once (tallies of the oracle)."""
    print(f"index chunks, {n} tracks", flush=True)
    geo = I.calorimeter()
    cfg = I.RunConfig(seed=29)
    prim = I.random_tracks(n, 16, geo, 1e-3, 1.0, seed=n)
    ref = oracle_mod.Oracle(geo, cfg).run(prim, n_events=16)
    got = run_gpu(E, geo, cfg, prim, 16, flags=E.F_FULL_LEDGER, blocks=1)
    for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
        assert np.array_equal(got["ledger"][f], ref["ledger"][f]), f
    assert np.allclose(got["edep"], ref["edep"], rtol=1e-9, atol=1e-9)


@pytest.mark.parametrize("n_bins,timing", [(40, False), (200, False), (200, True), (800, False)])
def test_one_launch_for_both_species_or_one_each(E, oracle_mod, n_bins, timing):  # noqa: F811
    """One launch an iteration, two with per-kernel timing, two where the
    tables of both species exceed LDS (800 bins: 154 + 38 KB); 40 bins: range
    tables searched node by node."""
    print(f"{n_bins} bins, timing {timing}", flush=True)
    geo, cfg, prim = I.workload("cal_1GeV_e-_x32")
    cfg = dataclasses.replace(cfg, n_bins=n_bins)
    p = prim[:6]
    ref = oracle_mod.Oracle(geo, cfg).run(p, n_events=6)
    got = run_gpu(E, geo, cfg, p, 6, flags=E.F_FULL_LEDGER | (E.F_KERNEL_TIMING if timing else 0))
    for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
        assert np.array_equal(got["ledger"][f], ref["ledger"][f]), f
    assert np.allclose(got["edep"], ref["edep"], rtol=1e-9, atol=1e-9)
    assert sum(got["stats"]["steps"]) == int(ref["ledger"]["n_steps"].sum())
    assert (got["stats"]["kernel_ms"][0] > 0.0) == timing


@pytest.mark.parametrize("capacity", [224, 256, 1024])
@pytest.mark.parametrize("short", [0.0, 1.0])
def test_nearly_full_queues_keep_moving(E, capacity, short):  # noqa: F811
    """Queues far smaller than the shower (photons wait while less than an
    eighth of the e- queue is free): every run ends, with the results of
    queues that hold everything."""
    print(f"capacity {capacity}, short {short}", flush=True)
    geo, cfg, prim = I.workload("cal_1GeV_e-_x32")
    p = prim[:8]
    ref = run_gpu(E, geo, cfg, p, 8, flags=E.F_FULL_LEDGER, short=short)
    assert ref["stats"]["deferred"] == 0
    for _ in range(4):
        got = run_gpu(E, geo, cfg, p, 8, flags=E.F_FULL_LEDGER, capacity=capacity, short=short)
        assert got["stats"]["deferred"] > 0
        for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
            assert np.array_equal(got["ledger"][f], ref["ledger"][f]), f
        assert np.allclose(got["edep"], ref["edep"], rtol=1e-12, atol=1e-12)
