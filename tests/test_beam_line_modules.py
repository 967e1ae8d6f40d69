"""Modules whose anchors' bounding box is centred on the beam line, or lies so far out that its
distance overflows: their disc has no direction, so the segment count's azimuth bins must take the
whole module.  The kernel's own functions run on the host, with the hardware reciprocals exact, 4 ulp
high and 4 ulp low."""
import copy
import ctypes

import numpy as np
import pytest

import oracle
from lstgen import make_single_track_event
from lstgen.events import Event

from kernel_host import build
from test_ls_pretests import SCALES

NAMES = ["anchor_disc", "azimuth_bin", "LsLink", "ls_link", "ls_inner", "ls_azimuth_bins", "ls_window_bound",
         "ls_module_may_pass"]
CODE = """
// (first bin, end) that the count takes of a module with anchors in the box x0..y1 and ranges rng for the
// inner MD (A, st), the bin of its MD B, and whether ls_module_may_pass keeps the module
extern "C" void bins(const float *A, const float *st, int ia, const float *box, const float *rng, int ib, float d0,
                     const float *B, int *out) {
  const float4 a = make_float4(A[0], A[1], A[2], A[3]), b = make_float4(B[0], B[1], B[2], B[3]);
  const float4 disc = anchor_disc(box[0], box[1], box[2], box[3]);
  const ModInfo ma{ia}, mb{ib};
  const float2 s = make_float2(st[0], st[1]);
  const LsLink l = ls_link(disc, make_float4(rng[0], rng[1], rng[2], rng[3]), mb);
  int b0 = 0, b1 = 0;
  if (!ls_azimuth_bins(a, s, ls_inner(a, s, ma, d0), ma, l, mb, d0, &b0, &b1)) b0 = b1 = 0;
  out[0] = b0;
  out[1] = b1;
  out[2] = azimuth_bin(disc.w * frcp(disc.z), (disc.x * b.y - disc.y * b.x) * (frcp(disc.w) * frcp(b.w)));
  out[3] = ls_module_may_pass(a, disc, ls_window_bound(a, ma, disc, mb, d0)) ? 1 : 0;
}
"""


def ring_geometry(geom):
    """The barrel with one module a layer, each linked to the next."""
    g = copy.copy(geom)
    first = np.array([np.nonzero(geom.layer == l + 1)[0][0] for l in range(6)])
    for n in ("subdet", "layer", "side", "type", "pos_lo", "pos_up"):
        setattr(g, n, getattr(geom, n)[first].copy())
    g.lmin, g.lmax = np.full(6, -geom.barrel_zmax), np.full(6, geom.barrel_zmax)
    g.n_modules = 6
    g.map_offsets = np.array([0, 1, 2, 3, 4, 5, 5], np.int32)
    g.map_targets = np.array([1, 2, 3, 4, 5], np.int32)
    return g


def mirrored_event(geom, n=4, seeded=False):
    """n straight-ish tracks, evenly spaced in azimuth, so that each layer's hits mirror each other."""
    ev = make_single_track_event(geom, 40.0, 0.05, 2 * np.pi * np.arange(n) / n + 0.3, q=1, seeded=seeded)
    out = copy.copy(ev)
    out.module = np.where(ev.module >= 0, geom.layer[np.maximum(ev.module, 0)] - 1, -1).astype(np.int32)
    # exactly mirrored: each hit of the second half is the negative of its partner in the first
    x, y = ev.x.copy(), ev.y.copy()
    for m in range(6):
        for s in (0, 1):
            k = np.nonzero((out.module == m) & (ev.sensor == s))[0]
            k = k[np.argsort(np.arctan2(y[k], x[k]))]
            h = len(k) // 2
            x[k[h:2 * h]], y[k[h:2 * h]] = -x[k[:h]], -y[k[:h]]
    out.x, out.y = x, y
    return out


def far_event(geom):
    """The same, with one more lower hit 1e20 cm out in every layer: the disc's distance overflows."""
    ev = mirrored_event(geom)
    cat = lambda a, b: np.concatenate([a, np.asarray(b, a.dtype)])
    return Event(x=cat(ev.x, [1e20] * 6), y=cat(ev.y, [0.0] * 6), z=cat(ev.z, [0.0] * 6),
                 module=cat(ev.module, range(6)), sensor=cat(ev.sensor, [0] * 6), sim=cat(ev.sim, [-1] * 6), name="far")


def event(kind, geom):
    return far_event(geom) if kind == "far" else mirrored_event(geom, 8 if kind == "ring8" else 4)


@pytest.mark.parametrize("sc", SCALES)
@pytest.mark.parametrize("kind", ["ring4", "ring8", "far"])
def test_every_segment_is_in_a_bin_looked_at(kind, sc, barrel, tmp_path):
    geom = ring_geometry(barrel)
    ev = event(kind, barrel)
    r = oracle.run(oracle.OracleGeometry(geom), ev, last=1)
    ls = r.stage(oracle.ST_LS)[0]
    assert len(ls) > 0
    lib = build(tmp_path, NAMES, CODE)
    lib.set_scale(sc)
    f = np.float32
    p = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    with np.errstate(over="ignore"):
        rr = np.sqrt(ev.x.astype(f) * ev.x + ev.y * ev.y)
    anchor = lambda i: np.array([ev.x[i], ev.y[i], ev.z[i], rr[i]], f)
    md = r.stage(oracle.ST_MD)[0]
    lost = 0
    for lo_a, up_a, lo_b, _ in ls:
        A, B = anchor(lo_a), anchor(lo_b)
        st = np.array([(ev.x[lo_a] * ev.y[up_a] - ev.y[lo_a] * ev.x[up_a]) / rr[lo_a], rr[up_a] - rr[lo_a]], f)
        ma, mb = int(ev.module[lo_a]), int(ev.module[lo_b])
        hits = np.nonzero((ev.module == mb) & (ev.sensor == 0))[0]
        box = np.array([ev.x[hits].min(), ev.x[hits].max(), ev.y[hits].min(), ev.y[hits].max()], f)
        if kind != "far":
            assert box[0] == -box[1] and box[2] == -box[3]
        anc = md[ev.module[md[:, 0]] == mb, 0]  # the module's MDs
        rng = np.array([rr[anc].min(), rr[anc].max(), ev.z[anc].min(), ev.z[anc].max()], f)
        out = (ctypes.c_int * 4)()
        lib.bins(p(A), p(st), int(geom.type[ma] == 1), p(box), p(rng), int(geom.type[mb] == 1), ctypes.c_float(0.1), p(B), out)
        b0, b1, own, reached = out
        assert reached
        lost += not b0 <= own < b1
    assert lost == 0, f"{lost} of {len(ls)} segments outside the bins"


@pytest.mark.gpu
@pytest.mark.parametrize("ls_cache", [32, 0])
@pytest.mark.parametrize("kind", ["ring4", "ring8", "far"])
def test_segments_of_a_ring(kind, ls_cache, barrel):
    import paper_2207_08207_amd as lst
    from parity import compare_event, compare_tc
    geom = ring_geometry(barrel)
    ev = event(kind, barrel)
    g = lst.Geometry(geom)
    g.set_tile_config({"ls_cache": ls_cache})
    print(f"[gpu] {kind}: {ev.n_hits} hits on {geom.n_modules} modules", flush=True)
    r = lst.run_event(g, lst.upload_event(ev))
    o = oracle.run(oracle.OracleGeometry(geom), ev)
    assert len(o.stage(oracle.ST_LS)[0]) > 0
    compare_event(r, o)
    compare_tc(r, o)
    r.close()
