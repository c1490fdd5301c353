"""A batch's way in and out around the sizes at which it changes: up to 1024
device primaries go in by one launch (more: check, staging, ids and injection
in turn), ids skip the sort when the rows come in order, up to 128 KB of deposits
and a megabyte of ledgers come back through pinned memory, and ledgers of up
to 256 columns are summed on the device.  The oracle is the host path (same records, bit for
bit) and the sum of the deposits."""
import numpy as np
import pytest

import ems_inputs as I
from test_gpu_device_io import E, assert_identical, on_device, run_both  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2050])
@pytest.mark.parametrize("ordered", [True, False])
def test_device_batches_give_the_host_histories(E, n, ordered):  # noqa: F811
    print(f"device batch of {n}, rows in order: {ordered}", flush=True)
    geo = I.calorimeter()
    rows = 7 if n < 1000 else 200
    p = I.random_tracks(n, rows, geo, 1e-3, 3.0, seed=n)
    if ordered:
        p = p[np.argsort(p["event"], kind="stable")]
    half = n // 3
    parts = [p] if half == 0 else [p[:half], p[half:]]  # (ids go on from the first part)
    h, d = run_both(E, geo, I.RunConfig(seed=3), parts, rows, precision=n % 2)
    assert_identical(h, d)


@pytest.mark.parametrize("layers, events", [(50, 1), (50, 163), (50, 164), (50, 3000), (128, 5), (129, 5)])
def test_restarted_batches_and_read_back_rows(E, layers, events):  # noqa: F811
    """two batches after each other on a context: the second, after a reset,
    gives the deposits of the first; a ledger's deposit is the sum of its row
    column by column"""
    print(f"restart, {layers} layers, {events} events", flush=True)
    geo = I.calorimeter(layers)
    c = E.make_config(I.RunConfig(seed=4), events, track_capacity=1 << 18)
    p = I.random_tracks(events, events, geo, 1.0, 20.0, seed=layers)
    with_device = on_device(p)
    t = E.Transport(c, geo)
    out = []
    for dev in (True, False, True):
        if dev:
            t.enqueue_device(with_device)
        else:
            t.enqueue(p)
        t.run()
        edep, ledger = t.edep(), t.ledger()
        sums = np.zeros(events)
        for k in range(edep.shape[1]):
            sums = sums + edep[:, k]
        assert np.array_equal(ledger["edep"], sums)
        out.append((edep, ledger, t.stats()["steps"]))
        t.reset()
        assert not t.edep().any() and not t.ledger()["edep"].any() and sum(t.stats()["steps"]) == 0
    t.close()
    for edep, ledger, steps in out[1:]:
        assert np.allclose(edep, out[0][0], rtol=1e-12, atol=1e-12)
        assert np.allclose(ledger["escaped"], out[0][1]["escaped"], rtol=1e-12, atol=1e-12)
        assert list(steps) == list(out[0][2])
