"""Edges of the kernels' tiles, lists and dispatch rules, object by object against the oracle: sizes
at which a tile, a word of flags, a list or a fixed table is just filled, and the paths taken past
them (needs an MI355X)."""
import copy

import numpy as np
import pytest

import oracle
from lstgen import make_event, make_single_track_event
from lstgen.events import Event, make_tiny_event

from parity import compare_event, compare_tc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lst():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU is required for the gpu-marked tests")
    import paper_2207_08207_amd as lst
    lst.load_library()
    return lst


@pytest.fixture(scope="module")
def gbarrel(lst, barrel):
    return lst.Geometry(barrel)


def _same(r, o):
    compare_event(r, o)
    compare_tc(r, o)
    r.close()


def _tracks(geom, n, seed, seeded=True, n_noise=0):
    rng = np.random.default_rng(seed)
    return make_single_track_event(geom, np.exp(rng.uniform(np.log(0.9), np.log(20.0), n)), rng.uniform(-0.5, 0.5, n),
                                   rng.uniform(0, 2 * np.pi, n), z0=rng.normal(0, 5, n),
                                   q=np.where(rng.uniform(size=n) < 0.5, -1, 1), seeded=seeded, seed=seed,
                                   n_noise=n_noise)


def _add_hits(ev, x, y, z, module, sensor):
    n = len(x)
    cat = lambda a, b, t: np.concatenate([a, np.asarray(b, t)])
    return Event(x=cat(ev.x, x, np.float32), y=cat(ev.y, y, np.float32), z=cat(ev.z, z, np.float32),
                 module=cat(ev.module, np.full(n, module), np.int32), sensor=cat(ev.sensor, sensor, np.int32),
                 sim=cat(ev.sim, np.full(n, -1), np.int32), px=ev.px, py=ev.py, pz=ev.pz, q=ev.q, hits4=ev.hits4,
                 seed_sim=ev.seed_sim, name="dense module")


# one wave of hits, one tile (1,024 hits) and one wave around it, and the first size with two tiles
@pytest.mark.parametrize("n_hits", [1, 63, 64, 65, 1023, 1024, 1025, 2049])
def test_hits_at_tile_edges(n_hits, lst, gbarrel, obarrel):
    ev = make_tiny_event(21, n_tracks=150, n_noise=1200)
    assert ev.n_hits > 2049
    cut = Event(x=ev.x[:n_hits], y=ev.y[:n_hits], z=ev.z[:n_hits], module=ev.module[:n_hits],
                sensor=ev.sensor[:n_hits], sim=ev.sim[:n_hits])
    print(f"[gpu] first {n_hits} hits", flush=True)
    _same(lst.run_event(gbarrel, lst.upload_event(cut)), oracle.run(obarrel, cut))


@pytest.mark.parametrize("n_events", [1, 3])
def test_hits_with_more_modules_than_sixteen_waves_rows(n_events, lst, full, ofull):
    """30,000 modules (the further ones without hits or links): the rows of eight waves fit LDS, those of
    sixteen do not; one small and one large event take 8 x 2 and 8 x 4 rounds, the batch of large ones 8 x 8."""
    geom = copy.copy(full)
    more = 30000 - full.n_modules
    for name in ("subdet", "layer", "side", "type", "pos_lo", "pos_up", "lmin", "lmax"):
        a = getattr(full, name)
        setattr(geom, name, np.concatenate([a, np.repeat(a[-1:], more)]))
    geom.n_modules = 30000
    geom.map_offsets = np.concatenate([full.map_offsets, np.repeat(full.map_offsets[-1:], more)])
    g = lst.Geometry(geom)
    plain = lst.Geometry(full)
    evs = [make_event("pu200_seeded", 40 + k, pu=200.0) for k in range(n_events)]
    if n_events == 1:
        small = make_event("pu200_seeded", 39, pu=20.0)
        _same(lst.run_event(g, lst.upload_event(small)), oracle.run(ofull, small))
    print(f"[gpu] {[e.n_hits for e in evs]} hits on 30,000 modules", flush=True)
    dev = [lst.upload_event(e) for e in evs]
    got = lst.run_batch(g, dev) if n_events > 1 else [lst.run_event(g, dev[0])]
    for r, d in zip(got, dev):
        ref = lst.run_event(plain, d)
        for st in range(7):
            for a, b in zip(r.stage(st), ref.stage(st)):
                assert np.array_equal(a, b), f"stage {st}"
        for a, b in zip(r.track_candidates(), ref.track_candidates()):
            assert np.array_equal(a, b)
        ref.close()
        r.close()


# partners of one lower hit up to and past the six kept; a module of 70 x 70; more hits in a bucket
# than its lists hold (8,192); anchors over 1.2 rad (a disc too wide for azimuth bins, and hits
# outside the range of the MD bins)
@pytest.mark.parametrize("md_cache", [32, 0])
@pytest.mark.parametrize("n_lower,n_upper,spread", [(1, 6, 0.0), (1, 7, 0.0), (70, 70, 0.04), (8200, 40, 0.04),
                                                    (60, 60, 1.2)])
def test_one_dense_module(n_lower, n_upper, spread, md_cache, lst, barrel, obarrel):
    ev = _tracks(barrel, 40, 3)
    m = int(np.bincount(ev.module[ev.module >= 0]).argmax())
    lo, up = (np.nonzero((ev.module == m) & (ev.sensor == s))[0][0] for s in (0, 1))
    rng = np.random.default_rng(n_lower + 7 * n_upper)
    xs, ys, zs, sens = [], [], [], []
    for s, i, n in ((0, lo, n_lower), (1, up, n_upper)):
        a = rng.uniform(-0.5, 0.5, n) * (spread if spread else 1e-5)
        xs += list(np.cos(a) * ev.x[i] - np.sin(a) * ev.y[i])
        ys += list(np.sin(a) * ev.x[i] + np.cos(a) * ev.y[i])
        zs += list(ev.z[i] + rng.uniform(-1e-3, 1e-3, n))
        sens += [s] * n
    ev = _add_hits(ev, xs, ys, zs, m, sens)
    g = lst.Geometry(barrel)
    g.set_tile_config({"md_cache": md_cache})
    print(f"[gpu] module {m}: {n_lower} lower, {n_upper} upper hits over {spread} rad", flush=True)
    _same(lst.run_event(g, lst.upload_event(ev)), oracle.run(obarrel, ev))


# words of 64 flags, bytes of 8, seeds a wave of the fill (4) and a block of it (16)
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 128, 129])
def test_seeds_at_flag_word_edges(n, lst, gbarrel, obarrel, barrel):
    ev = _tracks(barrel, n, 100 + n, n_noise=20)
    print(f"[gpu] {ev.n_seeds} seeds", flush=True)
    _same(lst.run_event(gbarrel, lst.upload_event(ev)), oracle.run(obarrel, ev))


# seeds that share pixel hits: two and three of four, all four; hits with one, few and many more seeds
# than a wave beside the one that owns them
@pytest.mark.parametrize("copies", [1, 2, 63, 64, 65, 200])
def test_seeds_that_share_pixel_hits(copies, lst, gbarrel, obarrel, barrel):
    ev = _tracks(barrel, 12, 8)
    rng = np.random.default_rng(copies)
    px, py, pz, q, h4 = list(ev.px), list(ev.py), list(ev.pz), list(ev.q), [list(r) for r in ev.hits4]
    for k in range(copies):
        a, b = k % 3, 3 + k % 4
        own = list(ev.hits4[a])
        for j in range(k % 5):  # 0 to 4 hits of another seed
            if j < 4:
                own[j] = int(ev.hits4[b][j])
        f = float(np.exp(rng.normal(0, 0.02)))
        px.append(px[a] * f); py.append(py[a] * f); pz.append(pz[a] * f); q.append(q[a]); h4.append(own)
    ev2 = copy.copy(ev)
    ev2.px, ev2.py, ev2.pz = (np.asarray(v, np.float32) for v in (px, py, pz))
    ev2.q, ev2.hits4 = np.asarray(q, np.int32), np.asarray(h4, np.int32).reshape(-1, 4)
    ev2.seed_sim = np.full(len(px), -1, np.int32)
    print(f"[gpu] {ev2.n_seeds} seeds, {copies} of them on others' pixel hits", flush=True)
    _same(lst.run_event(gbarrel, lst.upload_event(ev2)), oracle.run(obarrel, ev2))


# seeds past the per-seed caches: lists for all of them, for the first of them, for none (10 x
# capacity / 1,024 of them); searched bin by bin
@pytest.mark.parametrize("max_slices", [512, 1])
@pytest.mark.parametrize("lists", [64, 3, 0])
def test_seeds_past_the_cache(lists, max_slices, lst, barrel, obarrel):
    import torch
    ev = _tracks(barrel, 60, 12)
    g = lst.Geometry(barrel)
    g.set_tile_config({"pt3_cache": 0, "pt5_cache": 0, "max_slices": max_slices})
    d = lst.upload_event(ev)
    o = oracle.run(obarrel, ev)
    n_t5 = len(o.stage(oracle.ST_T5)[0])
    cap = lst.lst_default_capacity(ev.n_hits, ev.n_seeds)
    cap.t5 = (lists * 1024 + 9) // 10
    if cap.t5 < n_t5:
        ev = _tracks(barrel, max(1, 60 * cap.t5 // (2 * n_t5)), 12)
        d, o = lst.upload_event(ev), oracle.run(obarrel, ev)
        cap.t5 = max(cap.t5, len(o.stage(oracle.ST_T5)[0]))
    print(f"[gpu] {ev.n_seeds} seeds, room for {10 * cap.t5 // 1024} lists", flush=True)
    ws = lst.alloc_workspace(g, ev.n_hits, ev.n_seeds, cap)
    st, h = lst.lst_build_event(g.handle, d, ws, cap, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    _same(lst.EventResult(h, ws, st), o)


# MDs with more segments than the cache, with and without the lists' order: see the rank of the fill
@pytest.mark.parametrize("ls_cache,ls_group", [(32, 16), (32, 5), (3, 1), (0, 16)])
def test_segments_at_cache_and_group_edges(ls_cache, ls_group, lst, full, ofull):
    ev = make_event("pu200_seeded", 17, pu=30.0)
    g = lst.Geometry(full)
    g.set_tile_config({"ls_cache": ls_cache, "ls_group": ls_group})
    print(f"[gpu] ls_cache {ls_cache}, ls_group {ls_group}", flush=True)
    _same(lst.run_event(g, lst.upload_event(ev)), oracle.run(ofull, ev))


# results read from host memory (up to 64 events) and copied from the device (more)
@pytest.mark.parametrize("n", [64, 65])
@pytest.mark.parametrize("ext", [False, True])
def test_results_of_many_events(n, ext, lst, barrel, obarrel):
    g = lst.Geometry(barrel)
    g.set_track_extensions(ext)
    evs = [_tracks(barrel, 1 + k % 9, 300 + k) for k in range(n)]
    print(f"[gpu] batch of {n}", flush=True)
    res = lst.run_batch(g, [lst.upload_event(e) for e in evs])
    alone = {}
    for k, (ev, r) in enumerate(zip(evs, res)):
        if k % 8 == 0 or k >= 63:
            _one = lst.run_event(g, lst.upload_event(ev))
            alone[k] = _one.extended_track_candidates() if ext else _one.track_candidates()
            got = r.extended_track_candidates() if ext else r.track_candidates()
            assert len(got) == len(alone[k]) and all(np.array_equal(a, b) for a, b in zip(got, alone[k]))
            compare_event(r, oracle.run(obarrel, ev))
            compare_tc(r, oracle.run(obarrel, ev))
            _one.close()
        r.close()


def _cut(ev, n):
    return Event(x=ev.x[:n], y=ev.y[:n], z=ev.z[:n], module=ev.module[:n], sensor=ev.sensor[:n], sim=ev.sim[:n])


# sixteen and seventeen hit tiles (the scatter's own sums, and those of a launch before it)
@pytest.mark.parametrize("n_hits", [16384, 16385])
def test_hits_at_the_direct_tile_limit(n_hits, lst, full, ofull):
    ev = make_event("pu200", 31, pu=20.0)
    assert ev.n_hits > 16385
    ev = _cut(ev, n_hits)
    print(f"[gpu] first {n_hits} hits", flush=True)
    _same(lst.run_event(lst.Geometry(full), lst.upload_event(ev)), oracle.run(ofull, ev))


def _with_capacity(lst, g, ev, **caps):
    import torch
    cap = lst.lst_default_capacity(ev.n_hits, ev.n_seeds)
    for k, v in dict(dict(ls=65536, t3=65536, pt3=65536, pt5=65536), **caps).items():  # room in the other stages
        setattr(cap, k, max(v, 1))
    ws = lst.alloc_workspace(g, ev.n_hits, ev.n_seeds, cap)
    st, h = lst.lst_build_event(g.handle, lst.upload_event(ev), ws, cap, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return lst.EventResult(h, ws, st)


# T5 duplicate removal over all pairs (capacities up to 2,048) and over lists, with hundreds of T5s at
# one MD, seeded (the seed search's bins ride in both) and not
@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("cap_t5", [2048, 2049])
@pytest.mark.parametrize("seeded", [True, False])
def test_t5_duplicates_at_the_pair_limit(seeded, cap_t5, block, lst, barrel, obarrel):
    from dense import dense_event
    ev = dense_event(barrel)
    if not seeded:
        ev = _cut(ev, ev.n_hits)
    g = lst.Geometry(barrel)
    g.set_launch_config({"t5_dedup": block})
    o = oracle.run(obarrel, ev)
    assert 500 < len(o.stage(oracle.ST_T5)[0]) <= 2048
    print(f"[gpu] {len(o.stage(oracle.ST_T5)[0])} T5s, room for {cap_t5}", flush=True)
    _same(_with_capacity(lst, g, ev, t5=cap_t5), o)


# segments of unseeded events whose copying blocks sum the counts themselves (MD capacities up to
# 8,192), with MDs past the cache
@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("ls_cache", [32, 2, 0])
@pytest.mark.parametrize("cap_md", [8192, 8193])
def test_segments_at_the_direct_sum_limit(cap_md, ls_cache, block, lst, full, ofull):
    ev = _cut(make_event("pu200", 32, pu=12.0), 22000)
    g = lst.Geometry(full)
    g.set_tile_config({"ls_cache": ls_cache})
    g.set_launch_config({"ls_fill": block})
    o = oracle.run(ofull, ev)
    n_md = len(o.stage(0)[0])
    assert 3000 < n_md <= 8192 and len(o.stage(1)[0]) > n_md / 4
    print(f"[gpu] {n_md} MDs, {len(o.stage(1)[0])} segments", flush=True)
    _same(_with_capacity(lst, g, ev, md=cap_md), o)
