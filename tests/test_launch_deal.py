"""Late blocks: a launch's blocks may start after the iteration they belong to
was closed (another context's work holds the device, or the grid exceeds it).
On the host, the dealing and closing of a launch with blocks started in any
order; on the GPU, two contexts at work at once and grids far beyond
residency, against each run alone and the default grid."""
import os
import subprocess
import threading

import numpy as np
import pytest

import ems_inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_blocks_started_after_the_close_take_nothing(tmp_path):
    exe = tmp_path / "launch_deal_check"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "launch_deal_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


@pytest.fixture(scope="module")
def E():
    import paper_2209_15445_amd as E
    return E


def context(E, geo, cfg, events, **opt):
    return E.Transport(E.make_config(cfg, events, track_capacity=1 << 18, flags=E.F_FULL_LEDGER, **opt), geo)


def batch(t, prim):
    t.reset()
    t.enqueue(prim)
    t.run()
    return t.edep(), t.ledger(), t.stats()


def assert_same(got, ref):
    """Tolerance: the order of the atomic sums."""
    for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
        assert np.array_equal(got[1][f], ref[1][f]), f
    assert got[2]["steps"] == ref[2]["steps"] and got[2]["created"] == ref[2]["created"]
    assert np.allclose(got[0], ref[0], rtol=1e-12, atol=1e-12)


@pytest.mark.gpu
@pytest.mark.parametrize("precision, short", [(0, 0.0), (1, 0.0), (1, 0.5)])
def test_two_contexts_at_once(E, precision, short):
    """A beam that fills the device beside small batches, each context on a
    stream and a thread of its own."""
    print(f"two contexts, precision {precision}, short {short}", flush=True)
    geo = I.calorimeter()
    opt = dict(precision=precision, short_electron_MeV=short)
    beam = I.mixed_species(300, 1000.0, 4000.0, seed=5)
    small = I.mixed_species(32, 100.0, 1000.0, seed=6)
    a = context(E, geo, I.RunConfig(seed=8), 300, **opt)
    b = context(E, geo, I.RunConfig(seed=9, n_bins=150), 32, **opt)
    alone = batch(a, beam), batch(b, small)
    out, errors = ([], []), []

    def work(t, prim, times, into):
        try:
            for _ in range(times):
                into.append(batch(t, prim))
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=w) for w in ((a, beam, 4, out[0]), (b, small, 12, out[1]))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in (0, 1):
        for got in out[k]:
            assert_same(got, alone[k])
    a.close()
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("opt", [dict(), dict(short_electron_MeV=0.5), dict(precision=1), dict(timing=True),
                                 dict(steps_per_launch=1), dict(steps_per_launch=5)])
def test_more_blocks_than_the_device_holds(E, opt):
    """Grids of 4096 blocks, and chunks of an odd number of iterations, give
    the results of the default grid and chunk."""
    print(f"4096 blocks, {opt}", flush=True)
    geo = I.calorimeter()
    opt = dict(opt)
    flags = E.F_FULL_LEDGER | (E.F_KERNEL_TIMING if opt.pop("timing", False) else 0)
    chunk = opt.pop("steps_per_launch", 0)
    prim = I.mixed_species(24, 100.0, 1500.0, seed=7)
    ref_t = context(E, geo, I.RunConfig(seed=10), 24, **opt)
    ref = batch(ref_t, prim)
    ref_t.close()
    c = E.make_config(I.RunConfig(seed=10), 24, track_capacity=1 << 18, flags=flags, launch_blocks=4096, **opt)
    c.steps_per_launch = chunk
    t = E.Transport(c, geo)
    for _ in range(3):
        assert_same(batch(t, prim), ref)
    t.close()
