"""The work the transport's speed is measured on.

A case is one batch taken through the public entry points the way a
simulation program takes it: a context (or server) made once per
configuration, then for every batch reset, primaries in, run to extinction,
deposits out.  Two ways in and out are used in earnest: primaries and
deposits in device memory (a pipeline that stays on the GPU), and host
arrays with the energy ledger (a host program that offloads a batch).

Fields of a case:
  geometry   "cal" (50 layers Pb / liquid argon), "calPbWO4" (lead tungstate
             absorber), "towers" (9 x 9 towers, 8100 boxes)
  beam       "e-" (one electron per event), "mixed" (e-, e+, gamma by event,
             energy log-uniform), "tracks" (isotropic tracks of all species
             anywhere in the stack), "requests" (offload requests)
  events, energy_MeV (upper end for "mixed" and "tracks"), bz_tesla, fp64,
  msc_fluct (multiple scattering and loss fluctuations), host_io, short_MeV
  (threshold of the short-electron launch, 0: off)
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import ems_inputs as I
import paper_2209_15445_amd as E

COLUMNS = {"cal": 100, "calPbWO4": 100, "towers": 8101}
# track-steps per MeV of primary energy (all species; the showers of these
# stacks take 5 to 6) and the arithmetic a step cannot do without: one
# Philox block (100 integer operations), a logarithm and an exponential, three
# table interpolations, the boundary distance and the move (about 150)
STEPS_PER_MEV = 5.4
OPS_PER_STEP = 250.0


def _case(name, geometry="cal", beam="e-", events=1, energy_MeV=1e3, bz_tesla=0.0, fp64=True, msc_fluct=False,
          host_io=False, short_MeV=0.0):
    return dict(name=name, geometry=geometry, beam=beam, events=events, energy_MeV=energy_MeV, bz_tesla=bz_tesla,
                fp64=fp64, msc_fluct=msc_fluct, host_io=host_io, short_MeV=short_MeV)


def listed():
    return [
        # a hybrid simulation hands over a handful of low-energy tracks:
        # launches, copies and the host decide
        _case("tracks_48_10MeV_field", beam="tracks", events=48, energy_MeV=10.0, bz_tesla=3.8, host_io=True),
        # one small batch: far too few tracks to fill the device
        _case("cal_1GeV_x32", events=32, energy_MeV=1e3),
        # the same size in the mixed form, compound absorber, odd event count
        _case("calPbWO4_1GeV_x37_mixed", geometry="calPbWO4", events=37, energy_MeV=1e3, fp64=False),
        # a middling batch of a host program: host arrays and ledgers
        _case("cal_2GeV_x500_host", events=500, energy_MeV=2e3, host_io=True),
        # a burst of offload requests to the server
        _case("server_requests_x300_field", beam="requests", events=300, energy_MeV=5e3, bz_tesla=3.8, host_io=True),
        # the benchmark beam
        _case("cal_10GeV_x10k", events=10_000, energy_MeV=1e4),
        # the large mixed-form beam, slow electrons in their own launch
        _case("cal_10GeV_x40k_mixed", events=40_000, energy_MeV=1e4, fp64=False, short_MeV=0.5),
        # mixed species over two decades of energy in the solenoid field
        _case("cal_mixed_100GeV_x2500_field", beam="mixed", events=2_500, energy_MeV=1e5, bz_tesla=3.8),
        # the same physics in the mixed form, on the lead tungstate stack
        _case("calPbWO4_mixed_100GeV_x1501_field_mixed", geometry="calPbWO4", beam="mixed", events=1_501,
              energy_MeV=1e5, bz_tesla=3.8, fp64=False),
        # every optional along-step process
        _case("cal_10GeV_x1500_msc_fluct", events=1_500, energy_MeV=1e4, msc_fluct=True),
        # box geometry through the hierarchy, both forms
        _case("towers_10GeV_x1500", geometry="towers", events=1_500, energy_MeV=1e4),
        _case("towers_1GeV_x999_mixed", geometry="towers", events=999, energy_MeV=1e3, fp64=False),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of the same ranges: batches from a few tracks to a few thousand
    showers, every geometry, form and option, odd sizes."""
    kind = rng.choice(["tracks", "small", "beam", "beam", "mixed", "towers", "requests"])
    fp64 = rng.random() < 0.6
    c = _case("drawn", fp64=fp64)
    del c["name"]
    if kind == "tracks":
        c.update(beam="tracks", events=int(_log_uniform(rng, 5, 3000)), energy_MeV=_log_uniform(rng, 5.0, 50.0),
                 bz_tesla=rng.choice([0.0, 3.8]), host_io=True)
    elif kind == "small":
        c.update(geometry=rng.choice(["cal", "calPbWO4"]), events=int(_log_uniform(rng, 1, 200)),
                 energy_MeV=_log_uniform(rng, 300.0, 3000.0), host_io=rng.random() < 0.5)
    elif kind == "beam":
        events = int(_log_uniform(rng, 200, 8000))
        c.update(geometry=rng.choice(["cal", "cal", "calPbWO4"]), events=events,
                 energy_MeV=_log_uniform(rng, 2e3, min(2e4, 8e7 / events)), msc_fluct=rng.random() < 0.3,
                 host_io=rng.random() < 0.3, short_MeV=0.5 if not fp64 and events > 3000 else 0.0)
    elif kind == "mixed":
        c.update(geometry=rng.choice(["cal", "calPbWO4"]), beam="mixed", events=int(_log_uniform(rng, 100, 2000)),
                 energy_MeV=_log_uniform(rng, 1e4, 1e5), bz_tesla=rng.choice([1.0, 3.8]))
    elif kind == "towers":
        c.update(geometry="towers", events=int(_log_uniform(rng, 16, 1500)), energy_MeV=_log_uniform(rng, 500.0, 1e4),
                 bz_tesla=rng.choice([0.0, 0.0, 3.8]))
    else:
        c.update(beam="requests", events=int(_log_uniform(rng, 8, 600)), energy_MeV=_log_uniform(rng, 2e3, 6e3),
                 bz_tesla=3.8, host_io=True)
    c["energy_MeV"] = float(round(c["energy_MeV"], 3))
    return c


def _total_MeV(case):
    n, e = case["events"], case["energy_MeV"]
    if case["beam"] == "mixed":  # log-uniform from 1 GeV
        return n * (e - 1e3) / math.log(e / 1e3)
    if case["beam"] == "requests":  # lognormal, sigma 1
        return n * e * math.exp(0.5)
    if case["beam"] == "tracks":  # log-uniform from 1 MeV
        return n * (e - 1.0) / math.log(e)
    return n * e


def work(case):
    """Primaries read, deposits written, and the arithmetic of the steps."""
    tracks = case["events"] * (100 if case["beam"] == "requests" else 1)
    bytes_ = 64.0 * tracks + 8.0 * case["events"] * COLUMNS[case["geometry"]]
    return {"bytes": bytes_, "flops": OPS_PER_STEP * STEPS_PER_MEV * _total_MeV(case)}


def _geometry(case):
    if case["geometry"] == "towers":
        return I.towers()
    return I.calorimeter(absorber=I.LEAD_TUNGSTATE) if case["geometry"] == "calPbWO4" else I.calorimeter()


def _primaries(case, geo, seed):
    n, e = case["events"], case["energy_MeV"]
    if case["beam"] == "mixed":
        return I.mixed_species(n, 1e3, e, seed=seed)
    if case["beam"] == "tracks":
        p = I.random_tracks(n, n, geo, 1.0, e, seed=seed)
        p["event"] = np.arange(n, dtype=np.uint32)
        return p
    p = I.beam(n, I.ELECTRON, e, smear_rad=1e-3, seed=seed)
    if case["geometry"] == "towers":
        # impact points over the central 3 x 3 towers and their cracks
        rng = np.random.Generator(np.random.Philox(seed + 100))
        p["pos"][:, :2] = rng.uniform(-60.0, 60.0, (n, 2))
    return p


def _config(case, seed, geo):
    form = E.FP64 if case["fp64"] else E.MIXED
    mask = I.P_ALL | (I.P_MSC | I.P_FLUCT if case["msc_fluct"] else 0)
    run = dataclasses.replace(I.RunConfig(), seed=seed % (1 << 31), bz_tesla=case["bz_tesla"], process_mask=mask)
    # queues sized for the whole breadth-first shower (a third of a track
    # per MeV), the launch parameters the benchmark runs with
    need = 0.3 * _total_MeV(case)
    cap = 1 << max(16, min(28, math.ceil(math.log2(max(need, 1.0)))))
    boxes = case["geometry"] == "towers"
    opt = dict(track_capacity=cap, precision=form, steps_per_visit=16 if case["fp64"] else 32,
               photon_steps_per_visit=16 if boxes else 32, photon_refill_below=40 if boxes else 24,
               short_electron_MeV=case["short_MeV"])
    if case["beam"] == "requests":
        opt.update(track_capacity=max(cap, 1 << 20), steps_per_launch=1, steps_per_visit=12)
    return E.make_config(run, case["events"], **opt)


def prepare(case, seed):
    geo = _geometry(case)
    config = _config(case, seed, geo)
    state = {"case": case}
    if case["beam"] == "requests":
        rng = np.random.Generator(np.random.Philox(seed))
        state["requests"] = [I.serving_request(rng, e_median_MeV=case["energy_MeV"]) for _ in range(case["events"])]
        state["server"] = E.Server(config, geo, admit_cap_bytes=8 << 30)
        return state
    prim = _primaries(case, geo, seed)
    state["transport"] = E.Transport(config, geo)
    if case["host_io"]:
        state["primaries"] = prim
    else:
        state["primaries"] = torch.from_numpy(prim.view(np.uint8)).to("cuda")
        state["edep"] = torch.empty((case["events"], geo.n_cols), dtype=torch.float64, device="cuda")
    return state


def _ledger(ledger):
    return {k: np.ascontiguousarray(ledger[k]) for k in ("edep", "escaped", "killed", "n_pair", "n_annih")}


def run(state):
    if "server" in state:
        server = state["server"]
        tickets = [server.submit(tracks, key) for key, tracks in enumerate(state["requests"])]
        results = [server.wait(t) for t in tickets]
        return {"edep": np.stack([r[0] for r in results]), **{"ledger_" + k: v for k, v in _ledger(
            np.array([r[1] for r in results])).items()}}
    t = state["transport"]
    t.reset()
    if state["case"]["host_io"]:
        t.enqueue(state["primaries"])
        t.run()
        return {"edep": t.edep(), **{"ledger_" + k: v for k, v in _ledger(t.ledger()).items()}}
    t.enqueue_device(state["primaries"])
    t.run()
    stats = t.stats()
    return {"edep": t.edep_device(state["edep"]), "steps": stats["steps"], "created": stats["created"]}


def exact(case, seed):
    """None: a deposit is the outcome of some thousand dependent random
    choices per event, and only a second implementation of every model,
    table and random stream could give it in 64 bits; the repository's own
    is the oracle of its tests."""
    return None
