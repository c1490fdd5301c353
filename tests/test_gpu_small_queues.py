"""Queues many times smaller than a shower's largest population: scarce room
goes to the lower energies, every run ends, with the results of queues that
hold everything.  Tolerance: the order of the atomic sums."""
import numpy as np
import pytest

import ems_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2209_15445_amd as E
    return E


def run(E, geo, prim, **opt):
    t = E.Transport(E.make_config(I.RunConfig(seed=5), len(prim), flags=E.F_FULL_LEDGER, **opt), geo)
    out = []
    for _ in range(2):  # (the second batch starts without the first one's limits)
        t.reset()
        t.enqueue(prim)
        t.run()
        out.append((t.edep(), t.ledger(), t.stats()))
    t.close()
    return out


@pytest.mark.parametrize("geometry, precision, short, parts", [
    ("cal", 0, 0.0, (2, 8, 16)), ("cal", 1, 0.0, (4, 10, 32)), ("cal", 0, 0.5, (8,)), ("cal", 1, 0.5, (6, 12)),
    ("towers", 0, 0.0, (10,)), ("towers", 1, 0.5, (6,))])
def test_a_fraction_of_the_largest_population(E, geometry, precision, short, parts):
    geo = I.towers() if geometry == "towers" else I.calorimeter()
    prim = I.beam(500, I.ELECTRON, 2e3, smear_rad=1e-3, seed=3)
    opt = dict(precision=precision, short_electron_MeV=short, photon_steps_per_visit=32)
    ref = run(E, geo, prim, track_capacity=1 << 20, **opt)[0]
    assert ref[2]["deferred"] == 0
    for part in parts:
        capacity = max(ref[2]["peak_live"]) // part
        print(f"{geometry}, form {precision}, short {short}, {capacity} slots", flush=True)
        for edep, ledger, stats in run(E, geo, prim, track_capacity=capacity, **opt):
            assert stats["deferred"] > 0 and max(stats["peak_live"]) <= (capacity + 63) // 64 * 64
            for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
                assert np.array_equal(ledger[f], ref[1][f]), f
            assert np.allclose(edep, ref[0], rtol=1e-12, atol=1e-12)
