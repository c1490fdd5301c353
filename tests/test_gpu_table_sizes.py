"""Tables that fill LDS (160 KB) to the last bytes beside a block's tallies:
counts and deposits against the oracle; one slab more is refused."""
import numpy as np
import pytest

import ems_inputs as I
from parity_util import ledger_residual

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


@pytest.fixture(scope="module")
def E():
    import paper_2209_15445_amd as E
    return E


def lds_bytes(geo, n_bins, precision):
    """a block's tallies (17 words, padded), e-/e+ tables, planes, materials (72
    bytes each) and slab materials"""
    slabs, mats = len(geo.material), len(geo.materials)
    tables = (mats * 12 * (n_bins + 1) * (4 if precision else 8) + 7) // 8 * 8
    return 72 + tables + (slabs + 1) * 8 + mats * 72 + slabs * 4


@pytest.mark.parametrize("precision, n_bins, layers, room", [
    (0, 839, 92, 128), (0, 839, 93, 104), (0, 839, 97, 8), (1, 1703, 1, 8)])
@pytest.mark.parametrize("short", [0.0, 0.5])
def test_tables_up_to_the_last_bytes_of_lds(E, oracle_mod, precision, n_bins, layers, room, short):
    print(f"{n_bins} bins, {layers} layers, form {precision}, short {short}", flush=True)
    geo = I.calorimeter(layers)
    assert LDS - lds_bytes(geo, n_bins, precision) == room
    cfg = I.RunConfig(seed=12, n_bins=n_bins)
    prim = I.mixed_species(6, 100.0, 800.0, seed=3)
    ref = oracle_mod.Oracle(geo, cfg).run(prim, n_events=6)
    c = E.make_config(cfg, 6, track_capacity=1 << 16, flags=E.F_FULL_LEDGER, precision=precision,
                      short_electron_MeV=short)
    t = E.Transport(c, geo)
    t.enqueue(prim)
    t.run()
    edep, ledger, stats = t.edep(), t.ledger(), t.stats()
    t.close()
    assert sum(stats["steps"]) == int(ledger["n_steps"].sum()) > 0
    assert list(stats["created"]) == ledger["n_created"].sum(axis=0).tolist()
    if precision == 0:
        for f in ("n_steps", "n_created", "n_null", "n_pair", "n_annih"):
            assert np.array_equal(ledger[f], ref["ledger"][f]), f
        assert np.allclose(edep, ref["edep"], rtol=1e-9, atol=1e-9)
    assert ledger_residual(edep, ledger, prim).max() < 1e-9


def test_tables_beyond_lds_are_refused(E):
    geo = I.calorimeter(98)
    assert lds_bytes(geo, 839, 0) > LDS
    with pytest.raises(E.EmsError, match="LDS"):
        E.Transport(E.make_config(I.RunConfig(n_bins=839), 1, track_capacity=1 << 12), geo)
