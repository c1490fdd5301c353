"""The kernel variants for scattering and fluctuations alone and for compound
materials with or without a field give the results of the kernels with every
part compiled in; configurations one part beyond them (and the short-electron
launch) take the latter.  Tolerance: the order of the atomic sums, as for the
other variants."""
import numpy as np
import pytest

import ems_inputs as I
from test_gpu_device_io import E  # noqa: F401

pytestmark = pytest.mark.gpu


def run(E, geo, cfg, prim, n, **opt):  # noqa: F811
    t = E.Transport(E.make_config(cfg, n, track_capacity=1 << 18, **opt), geo)
    t.enqueue(prim)
    t.run()
    out = t.edep(), t.ledger(), t.stats()
    t.close()
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("absorber, bz, parts, short", [
    ("lead", 0.0, I.P_MSC | I.P_FLUCT, 0.0), ("lead", 0.0, I.P_MSC, 0.0), ("lead", 0.0, I.P_FLUCT, 0.0),
    ("lead", 0.0, I.P_MSC, 0.5), ("lead", 3.8, I.P_MSC, 0.0),
    ("PbWO4", 0.0, 0, 0.0), ("PbWO4", 3.8, 0, 0.0), ("PbWO4", 3.8, 0, 0.5), ("PbWO4", 0.0, I.P_FLUCT, 0.0)])
def test_variant_matches_the_full_kernels(E, precision, absorber, bz, parts, short):  # noqa: F811
    print(f"variant {absorber} bz {bz} parts {parts} short {short} precision {precision}", flush=True)
    geo = I.calorimeter(absorber=I.LEAD_TUNGSTATE) if absorber == "PbWO4" else I.calorimeter()
    cfg = I.RunConfig(seed=6, bz_tesla=bz, process_mask=I.P_ALL | parts)
    prim = I.mixed_species(9, 200.0, 1500.0, seed=2)
    opt = dict(precision=precision, short_electron_MeV=short)
    small = run(E, geo, cfg, prim, 9, **opt)
    full = run(E, geo, cfg, prim, 9, flags=E.F_FULL_KERNELS, **opt)
    assert small[2]["steps"] == full[2]["steps"] and small[2]["created"] == full[2]["created"]
    assert np.allclose(small[0], full[0], rtol=1e-12, atol=1e-12)
    for f in ("escaped", "killed", "n_pair", "n_annih"):
        assert np.allclose(small[1][f], full[1][f], rtol=1e-12, atol=1e-12), f
