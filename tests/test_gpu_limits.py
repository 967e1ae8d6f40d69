"""Calls at the limits of what an event may be -- capacities far below what is found, modules of
unusual shape, hits far out -- object by object against the oracle (needs an MI355X)."""
import numpy as np
import pytest

import oracle
from lstgen import make_event, make_single_track_event
from lstgen.events import make_tiny_event

from dense import dense_event
from parity import compare_event, compare_tc
from wide_modules import merge_event, sector_geometry

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lst():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU is required for the gpu-marked tests")
    import paper_2207_08207_amd as lst
    lst.load_library()
    return lst


# the triplet capacity far below what is found, the quintuplets' duplicates removed over lists
# (capacity above 2,048) and over pairs
@pytest.mark.parametrize("cap_t5", [4096, 2048])
@pytest.mark.parametrize("config", ["dense", "pu200_seeded", "pu200"])
def test_triplet_capacity_overflow_reports_and_recovers(config, cap_t5, lst, barrel, obarrel, full, ofull):
    import torch
    geom, og = (barrel, obarrel) if config == "dense" else (full, ofull)
    ev = dense_event(geom) if config == "dense" else make_event(config, 51, pu=20.0)
    o = oracle.run(og, ev)
    n_t3 = len(o.stage(oracle.ST_T3)[0])
    g = lst.Geometry(geom)
    cap = lst.lst_default_capacity(ev.n_hits, ev.n_seeds)
    cap.t3, cap.t5 = 50, cap_t5
    assert n_t3 > 20 * cap.t3
    dev = lst.upload_event(ev)
    ws = lst.alloc_workspace(g, ev.n_hits, ev.n_seeds, cap)
    print(f"[gpu] {config}: {n_t3} triplets, room for {cap.t3}", flush=True)
    st, h = lst.lst_build_event(g.handle, dev, ws, cap, torch.cuda.current_stream().cuda_stream)
    assert st == lst.LST_E_CAPACITY
    counts, req = lst.lst_get_stage_counts(h)
    assert counts[2] == 50 and req[2] == n_t3
    lst.lst_release_event(h)
    r = lst.run_event(g, dev, cap=cap)  # grows and reruns
    compare_event(r, o)
    compare_tc(r, o)
    r.close()


# every seed past the caches: the fill's tasks counted in one line (fewer than 256 seeds) and in sixteen,
# with lists for all and for a few of them
@pytest.mark.parametrize("lists", [1000, 5])
@pytest.mark.parametrize("n", [1, 17, 255, 256, 257])
def test_seed_tasks_at_the_shard_limit(n, lists, lst, barrel, obarrel):
    import torch
    rng = np.random.default_rng(400 + n)
    ev = make_single_track_event(barrel, np.exp(rng.uniform(np.log(0.9), np.log(20.0), n)), rng.uniform(-0.5, 0.5, n),
                                 rng.uniform(0, 2 * np.pi, n), z0=rng.normal(0, 5, n),
                                 q=np.where(rng.uniform(size=n) < 0.5, -1, 1), seeded=True, seed=n)
    o = oracle.run(obarrel, ev)
    g = lst.Geometry(barrel)
    g.set_tile_config({"pt3_cache": 0, "pt5_cache": 0})
    cap = lst.lst_default_capacity(ev.n_hits, ev.n_seeds)
    cap.t5 = max(len(o.stage(oracle.ST_T5)[0]) + 1, (lists * 1024 + 9) // 10 if n > 200 or lists > 5 else 0)
    ws = lst.alloc_workspace(g, ev.n_hits, ev.n_seeds, cap)
    print(f"[gpu] {ev.n_seeds} seeds, {10 * cap.t5 // 1024} lists", flush=True)
    st, h = lst.lst_build_event(g.handle, lst.upload_event(ev), ws, cap, torch.cuda.current_stream().cuda_stream)
    assert st == lst.LST_OK
    r = lst.EventResult(h, ws, st)
    compare_event(r, o)
    compare_tc(r, o)
    r.close()


# few wide modules: hits outside the range of the bins by u, listed by direction, in LDS and (more than
# 8,192 hits a bucket) in global memory; windows wide enough for lists of partners; all pairs tested
@pytest.mark.parametrize("nphi,nz,n,bound,md_cache", [(1, 1, 60, 0.1, 32), (1, 1, 800, 0.1, 32), (4, 1, 300, 0.1, 32),
                                                      (4, 1, 1500, 0.1, 32), (4, 1, 300, 0.1, 3), (4, 1, 200, 3.6, 32),
                                                      (2, 1, 120, 10.0, 32), (8, 4, 1500, 0.1, 32)])
def test_wide_modules(nphi, nz, n, bound, md_cache, lst, barrel):
    geom, new = sector_geometry(barrel, nphi, nz)
    rng = np.random.default_rng(n)
    ev = make_single_track_event(barrel, np.exp(rng.uniform(np.log(0.8), np.log(50.0), n)), rng.uniform(-0.5, 0.5, n),
                                 rng.uniform(0, 2 * np.pi, n), z0=rng.normal(0, 5, n),
                                 q=np.where(rng.uniform(size=n) < 0.5, -1, 1), smear=True, seed=n, n_noise=50)
    ev = merge_event(ev, new)
    g, og = lst.Geometry(geom), oracle.OracleGeometry(geom, d0_max=bound)
    g.set_tile_config({"md_cache": md_cache})
    g.set_impact_bound(bound)
    o = oracle.run(og, ev)
    print(f"[gpu] {geom.n_modules} modules, {ev.n_hits} hits, {o.count(0)} mini-doublets", flush=True)
    r = lst.run_event(g, lst.upload_event(ev))
    compare_event(r, o)
    compare_tc(r, o)
    r.close()


# a lower hit on the beam line's side of 10 um and one 20 km out: every pair of their modules tested
def test_hits_near_the_beam_line_and_far_out(lst, barrel, obarrel):
    ev = make_tiny_event(4, n_tracks=60, n_noise=40)
    m = [int(k) for k in np.argsort(np.bincount(ev.module[ev.module >= 0]))[-3:]]
    for k, x in zip(m, (1e-5, 2e6, 0.0)):
        i = np.nonzero((ev.module == k) & (ev.sensor == 0))[0][0]
        ev.x[i], ev.y[i] = x, 0.0
    r = lst.run_event(lst.Geometry(barrel), lst.upload_event(ev))
    o = oracle.run(obarrel, ev)
    compare_event(r, o)
    compare_tc(r, o)
    r.close()


# lower hits with more than six partners among many upper hits.  On 5,736 modules all are tested again;
# on 24, crowded (more than 48 hits a module): lists in any order, ranked by the fill, and in order from a
# pass over the module (more partners than twice the root of its upper hits)
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n_upper,spread", [(300, 0.05), (200, 0.001), (64, 0.02), (63, 0.004)])
def test_lists_of_partners(n_upper, spread, wide, lst, barrel):
    geom, new = sector_geometry(barrel, 4, 1) if wide else (barrel, np.arange(barrel.n_modules))
    ev = merge_event(make_tiny_event(6, n_tracks=160, n_noise=30), new)
    og = oracle.OracleGeometry(geom)
    pair = oracle.run(og, ev, last=0).stage(0)[0][0]  # the hits are spread about one mini-doublet's
    m = int(ev.module[pair[0]])
    rng = np.random.default_rng(n_upper)
    add = {k: [getattr(ev, k)] for k in ("x", "y", "z", "module", "sensor", "sim")}
    for sensor, n in ((0, 40), (1, n_upper)):
        i = pair[sensor]
        a = rng.uniform(-spread, spread, n)
        add["x"].append(np.cos(a) * ev.x[i] - np.sin(a) * ev.y[i])
        add["y"].append(np.sin(a) * ev.x[i] + np.cos(a) * ev.y[i])
        add["z"].append(ev.z[i] + rng.uniform(-1e-3, 1e-3, n))
        add["module"].append(np.full(n, m))
        add["sensor"].append(np.full(n, sensor))
        add["sim"].append(np.full(n, -1))
    for k, v in add.items():
        setattr(ev, k, np.concatenate(v).astype(v[0].dtype))
    partners = np.bincount(oracle.run(og, ev, last=0).stage(0)[0][:, 0])
    print(f"[gpu] module {m}: up to {partners.max()} partners of {n_upper}", flush=True)
    assert (partners > 6).sum() > 25
    assert (ev.n_hits > 48 * geom.n_modules) == wide
    cap = lst.lst_default_capacity(ev.n_hits, ev.n_seeds)
    cap.md = cap.ls = cap.t3 = 400000
    r = lst.run_event(lst.Geometry(geom), lst.upload_event(ev), cap=cap)
    o = oracle.run(og, ev)
    compare_event(r, o)
    compare_tc(r, o)
    r.close()
