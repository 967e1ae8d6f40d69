"""The work that a user of this library has it do, as cases that can be timed.

A case is one pass of the track-building chain through the public entry
points, from device hits (or pinned host hits) to track candidates on the
host.  `form` names the entry point:

* event:  run_event on one event, with the program's own workspace;
* e2e:    the same from pinned host arrays (host-to-device copies included);
* static: lst_build_event_static, the allocation-free entry;
* batch:  run_batch, several events per launch sequence;
* plan:   Plan.run, the captured batch replayed;
* served: Server, requests submitted to the serving loop and drained.

`detector` and `config` are the generator's (lstgen): `tiny` barrel events,
`cube` displaced muons (impact-parameter bound 3.6 cm), and the pile-up
workloads, whose size `pu` sets (200 pile-up = 8,000 tracks and 40,000 loopers).
Every event number derives from the seed alone.
"""
import numpy as np
import torch

import paper_2207_08207_amd as lst
from lstgen import barrel_geometry, full_geometry, make_event
from lstgen.events import make_tiny_event

CUBE_BOUND = 3.6  # cm, just above the cube sample's largest transverse displacement
DEFAULTS = dict(form="event", config="pu200_seeded", pu=200.0, pu_max=0.0, events=1, requests=0, streams=0,
                max_batch=0, ext=False, stub_bits=32)


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # the smallest call: a barrel test-beam-sized event (about 1,400 hits), one at a time
        _case("event_tiny", config="tiny", pu=0.0),
        # small ragged barrel events processed together
        _case("batch_tiny16", form="batch", config="tiny", pu=0.0, events=16),
        # displaced muons with the widened impact-parameter bound (814 hits on the full detector)
        _case("event_cube", config="cube", pu=0.0),
        # a quiet crossing: the low end of the serving mix (about 133k hits)
        _case("event_pu50", pu=50.0),
        # the allocation-free entry near the largest event that its workspace takes
        _case("static_pu60", form="static", pu=60.0),
        # the benchmark's event: pile-up 200 with pixel seeds, one at a time
        _case("event_pu200", pu=200.0),
        # outer tracker only: no seeds, so no pixel stages
        _case("event_pu200_unseeded", config="pu200", pu=200.0),
        # the extended collection (track extensions switched on)
        _case("event_pu200_ext", pu=200.0, ext=True),
        # mini-doublet stubs in 16 bits
        _case("event_pu140_stub16", pu=140.0, stub_bits=16),
        # a host program's event: pinned host hits in, track candidates on the host
        _case("e2e_pu200", form="e2e", pu=200.0),
        # offline processing: a captured batch over the high pile-up range
        _case("plan_8", form="plan", pu=140.0, pu_max=250.0, events=8),
        # the serving loop at saturation over the serving mix
        _case("served_64", form="served", pu=50.0, pu_max=250.0, events=4, requests=64, streams=4, max_batch=8),
    ]


def _log(rng, lo, hi):
    return float(np.exp(rng.uniform(np.log(lo), np.log(hi))))


def draw(rng):
    form = rng.choice(["event", "event", "event", "e2e", "static", "batch", "batch_tiny", "plan", "served"])
    opts = dict(ext=rng.random() < 0.2, stub_bits=16 if rng.random() < 0.2 else 32)
    if form == "event":
        config = rng.choice(["tiny", "cube", "pu200", "pu200_seeded", "pu200_seeded"])
        pu = 0.0 if config in ("tiny", "cube") else round(_log(rng, 3.0, 250.0), 3)
        return dict(DEFAULTS, config=config, pu=pu, **opts)
    if form == "batch_tiny":
        return dict(DEFAULTS, form="batch", config="tiny", pu=0.0, events=rng.randint(2, 40), **opts)
    if form == "static":
        return dict(DEFAULTS, form=form, pu=round(_log(rng, 2.0, 62.0), 3), stub_bits=opts["stub_bits"])
    if form == "e2e":
        return dict(DEFAULTS, form=form, pu=round(_log(rng, 10.0, 250.0), 3), **opts)
    lo, hi = sorted((round(_log(rng, 3.0, 250.0), 3), round(_log(rng, 3.0, 250.0), 3)))
    if form == "batch":
        return dict(DEFAULTS, form=form, pu=lo, pu_max=hi, events=rng.randint(2, 6), **opts)
    if form == "plan":
        return dict(DEFAULTS, form=form, pu=lo, pu_max=hi, events=rng.randint(1, 8), **opts)
    return dict(DEFAULTS, form=form, pu=lo, pu_max=hi, events=rng.randint(2, 4), requests=rng.randint(8, 48),
                streams=rng.randint(1, 4), max_batch=rng.randint(1, 8), **opts)


# The detectors a program keeps, one handle per set of options, as long as the process runs.
_GEOMETRIES = {}


def _geometry(case):
    barrel, cube = case["config"] == "tiny", case["config"] == "cube"
    key = (barrel, cube, case["ext"], case["stub_bits"])
    if key not in _GEOMETRIES:
        g = lst.Geometry(barrel_geometry() if barrel else full_geometry())
        if cube:
            g.set_impact_bound(CUBE_BOUND)
        g.set_track_extensions(case["ext"])
        g.set_stub_precision(case["stub_bits"])
        _GEOMETRIES[key] = g
    return _GEOMETRIES[key]


def _events(case, seed):
    n, config = case["events"], case["config"]
    rng = np.random.default_rng([int(seed), 11])
    out = []
    for k in range(n):
        number = int(seed) * 64 + k
        if config == "tiny" and n > 1:  # ragged small events
            out.append(make_tiny_event(number, n_tracks=int(rng.integers(5, 200)), n_noise=int(rng.integers(10, 300))))
        elif case["pu"] > 0.0:
            pu = rng.uniform(case["pu"], case["pu_max"]) if case["pu_max"] > case["pu"] else case["pu"]
            out.append(make_event(config, number, pu=float(pu)))
        else:
            out.append(make_event(config, number))
    return out


def _room(case):
    """Candidates and hits that the program's result arrays have room for, over all events of a pass."""
    pu = max(case["pu"], case["pu_max"])
    cand = int(96 * pu) + 1024
    return (case["requests"] or case["events"]) * cand, 18


def prepare(case, seed):
    g = _geometry(case)
    host = _events(case, seed)
    hits, seeds = max(e.n_hits for e in host), max(e.n_seeds for e in host)
    dev = [lst.upload_event(e) for e in host]
    s = dict(case=case, g=g, dev=dev)
    form = case["form"]
    if form in ("event", "e2e"):
        s["ws"] = lst.alloc_workspace(g, hits, seeds)
        if form == "e2e":
            s["pinned"] = {k: v.cpu().pin_memory() for k, v in dev[0].items()}
    elif form == "static":
        i32 = dict(dtype=torch.int32, device="cuda")
        n = 4 * seeds + 4096
        s["out"] = dict(type_out=torch.empty(n, **i32), offsets_out=torch.empty(n + 1, **i32),
                        hits_out=torch.empty(14 * n, **i32), counts_out=torch.zeros(3, **i32))
    elif form == "batch":
        need = lst.lst_batch_workspace_bytes(g.handle, [e.n_hits for e in host], [e.n_seeds for e in host])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    elif form == "plan":
        s["plan"] = lst.Plan(g, len(host), hits, seeds)
    else:
        one = lst.lst_workspace_bytes(g.handle, hits, seeds)
        s["server"] = lst.Server(g, case["streams"], case["max_batch"], one * (case["streams"] * case["max_batch"] + 1))
    # the program's result arrays: what a pass finds goes to their front, -1 stays behind it
    n, w = _room(case)
    s["found"] = [np.full(n, -1, np.int32), np.full(2 * n, -1, np.int32), np.full(w * n, -1, np.int32)]
    if case["ext"]:
        s["found"] += [np.full(n, -1, np.int32), np.full(n, -1, np.int32), np.full((n, 3), -1.0, np.float32)]
    torch.cuda.synchronize()
    return s


def _candidates(case, r):
    return r.extended_track_candidates() if case["ext"] else r.track_candidates()


def _store(s, rows):
    """Events' track candidates one after another in the program's arrays."""
    for dst, col in zip(s["found"], zip(*rows)):
        at = 0
        for x in col:
            dst[at:at + len(x)] = x
            at += len(x)
    return s["found"]


def run(s):
    case, g, form = s["case"], s["g"], s["case"]["form"]
    if form in ("event", "e2e"):
        ev = s["dev"][0]
        if form == "e2e":
            for k, v in s["pinned"].items():
                ev[k].copy_(v, non_blocking=True)
        r = lst.run_event(g, ev, workspace=s["ws"])
        rows = [_candidates(case, r)]
        r.close()
    elif form == "static":
        o = s["out"]
        lst.lst_build_event_static(g.handle, s["dev"][0], **o)
        n, nh, status = o["counts_out"].tolist()
        if status != 0:
            raise RuntimeError(f"status flags {status}")
        rows = [[o["type_out"][:n].cpu().numpy(), o["offsets_out"][:n + 1].cpu().numpy(),
                 o["hits_out"][:nh].cpu().numpy()]]
    elif form in ("batch", "plan"):
        rs = lst.run_batch(g, s["dev"], workspace=s["ws"]) if form == "batch" else s["plan"].run(s["dev"])
        rows = [_candidates(case, r) for r in rs]
        for r in rs:
            r.close()
    else:
        srv, rows = s["server"], [None] * case["requests"]
        for i in range(case["requests"]):
            srv.submit(s["dev"][i % len(s["dev"])], i)

        def take(res):
            if res["status"] != lst.LST_OK:
                raise lst.LSTError(res["status"], f"request {res['id']}")
            h = res["event"]
            rows[res["id"]] = (lst.lst_get_extended_track_candidates(h) if case["ext"]
                               else lst.lst_get_track_candidates(h))
            lst.lst_release_event(h)

        srv.drain(case["requests"], take)
    return _store(s, rows)


def work(case):
    """Bytes of the inputs (20 a hit, 32 a seed) and of the candidates' lists, each once.  The
    arithmetic follows from the hits' combinatorics, which no closed form gives: none is counted."""
    if case["config"] == "tiny":
        hits, seeds, cand = 1400 if case["events"] == 1 else 1250, 0, 90
    elif case["config"] == "cube":
        hits, seeds, cand = 814, 0, 44
    else:
        pu = 0.5 * (case["pu"] + case["pu_max"]) if case["pu_max"] > case["pu"] else case["pu"]
        seeded = case["config"] == "pu200_seeded"
        hits, seeds, cand = 2660.0 * pu if seeded else 2500.0 * pu, 44.5 * pu if seeded else 0.0, 45.0 * pu
    n = case["requests"] or case["events"]
    return {"bytes": n * (20 * hits + 32 * seeds + cand * 4 * (2 + 13)), "flops": 0}


def exact(case, seed):
    """Nothing: the outputs are lists of hit indices, whole numbers that have to stay the same."""
    return None
