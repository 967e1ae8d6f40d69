"""The segment count's azimuth bins at wider impact-parameter bounds (each of their margins has the
bound in it), and for layers close to each other: every segment of the oracle lies in a bin looked at.
The kernel's own functions run on the host; the MDs' own bins and the bins looked at are computed by
separate kernels, so the hardware reciprocals are exact, 4 ulp high and 4 ulp low for each apart."""
import copy
import ctypes

import numpy as np
import pytest

import oracle
from lstgen.events import geometry_for, make_event

from kernel_host import build
from test_ls_pretests import SCALES

NAMES = ["anchor_disc", "azimuth_bin", "LsLink", "ls_link", "ls_inner", "ls_azimuth_bins"]
CODE = """
extern "C" void looked_at(int n, const float4 *A, const float2 *st, const int *ia, const float4 *disc, const float4 *rng,
                          const int *ib, float d0, int *out) {
  for (int i = 0; i < n; ++i) {
    const LsLink l = ls_link(disc[i], rng[i], ModInfo{ib[i]});
    int *b = out + 2 * i;
    if (!ls_azimuth_bins(A[i], st[i], ls_inner(A[i], st[i], ModInfo{ia[i]}, d0), ModInfo{ia[i]}, l, ModInfo{ib[i]}, d0,
                         b, b + 1))
      b[0] = b[1] = 0;
  }
}
extern "C" void own(int n, const float4 *B, const float4 *disc, int *out) {
  for (int i = 0; i < n; ++i)
    out[i] = azimuth_bin(disc[i].w * frcp(disc[i].z),
                         (disc[i].x * B[i].y - disc[i].y * B[i].x) * (frcp(disc[i].w) * frcp(B[i].w)));
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return build(tmp_path_factory.mktemp("k"), NAMES, CODE)


def _segments(config, pu, bound, squeeze):
    """Per segment: inner and outer anchors, inner stub, module infos, the outer module's disc and ranges."""
    geom, ev = geometry_for(config), make_event(config, 7, pu=pu)
    x, y, z = (v.astype(np.float32) for v in (ev.x, ev.y, ev.z))
    if squeeze:  # every barrel layer's sensors brought to within `squeeze` of the first layer's
        geom, r0 = copy.copy(geom), float(geom.pos_lo[0])
        f = lambda p: r0 + (p - r0) * squeeze
        rad = np.hypot(x.astype(np.float64), y)
        x, y = ((v * f(rad) / rad).astype(np.float32) for v in (x, y))
        geom.pos_lo, geom.pos_up = f(geom.pos_lo), f(geom.pos_up)
        ev.x, ev.y = x, y
    r = oracle.run(oracle.OracleGeometry(geom, d0_max=bound), ev, last=1)
    md, ls = r.stage(0)[0], r.stage(1)[0]
    rr = np.sqrt(x * x + y * y)
    pos = np.stack([x, y, z, rr], 1)
    m = np.maximum(ev.module, 0).astype(np.int64)
    M = geom.n_modules

    def ext(op, v, idx, start):
        out = np.full(M, start, np.float32)
        op.at(out, m[idx], v[idx])
        return out

    low = np.nonzero((ev.module >= 0) & (ev.sensor == 0))[0]
    x0, x1 = ext(np.minimum, x, low, np.inf), ext(np.maximum, x, low, -np.inf)
    y0, y1 = ext(np.minimum, y, low, np.inf), ext(np.maximum, y, low, -np.inf)
    anc = np.unique(md[:, 0])
    rng = np.stack([ext(np.minimum, rr, anc, np.inf), ext(np.maximum, rr, anc, -np.inf),
                    ext(np.minimum, z, anc, np.inf), ext(np.maximum, z, anc, -np.inf)], 1)
    f32 = np.float32
    with np.errstate(invalid="ignore", over="ignore"):
        cx, cy, hx, hy = f32(0.5) * (x0 + x1), f32(0.5) * (y0 + y1), f32(0.5) * (x1 - x0), f32(0.5) * (y1 - y0)
        disc = np.stack([cx, cy, np.sqrt(hx * hx + hy * hy) * f32(1.0001) + f32(1e-3), np.sqrt(cx * cx + cy * cy)], 1)
    la, ua, lb = ls[:, 0], ls[:, 1], ls[:, 2]
    info = ((geom.type == 1) | ((geom.subdet == 1).astype(int) << 1)).astype(np.int32)
    tau = (x[la] * y[ua] - y[la] * x[ua]) / rr[la]
    dl = np.where(geom.subdet[m[la]] == 1, np.abs(z[ua]) - np.abs(z[la]), rr[ua] - rr[la])
    c = np.ascontiguousarray
    return (c(pos[la], f32), c(pos[lb], f32), c(np.stack([tau, dl], 1), f32), c(info[m[la]]), c(info[m[lb]]),
            c(disc[m[lb]], f32), c(rng[m[lb]], f32))


@pytest.mark.parametrize("config,pu,bound,squeeze,least", [("pu200_seeded", 20.0, 3.6, 0, 15000), ("cube", None, 3.6, 0, 100),
                                                           ("pu200_seeded", 20.0, 1.0, 0, 8000), ("pu200_seeded", 10.0, 10.0, 0, 9000),
                                                           ("tiny", None, 0.1, 0.2, 100), ("tiny", None, 0.1, 0.05, 50),
                                                           ("tiny", None, 3.6, 0.05, 100)])
def test_every_segment_is_in_a_bin_looked_at(lib, config, pu, bound, squeeze, least):
    A, B, st, ia, ib, disc, rng = _segments(config, pu, bound, squeeze)
    n = len(A)
    assert n > least
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    looked, own = np.zeros((n, 2), np.int32), np.zeros(n, np.int32)
    for sc in SCALES:
        lib.set_scale(sc)
        lib.looked_at(n, p(A), p(st), p(ia), p(disc), p(rng), p(ib), ctypes.c_float(bound), p(looked))
        for sc_hit in SCALES:
            lib.set_scale(sc_hit)
            lib.own(n, p(B), p(disc), p(own))
            bad = ~((own >= looked[:, 0]) & (own < looked[:, 1]))
            assert not bad.any(), f"{bad.sum()} of {n} segments outside the bins ({sc}, {sc_hit})"
