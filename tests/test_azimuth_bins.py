"""The two searches over azimuth bins replayed in IEEE float32 on the host: every mini-doublet
and every segment of the oracle, which searches without bins, must lie in a bin that the kernels
look at.  The hardware reciprocal, reciprocal square root and square root (within 1 ulp) are taken
exact, 4 ulp high and 4 ulp low; the bins of the hits (or MDs) and the bins looked at are computed
by separate kernels, so each combination of the two is checked.
"""
import numpy as np
import pytest

import oracle
from lstgen.events import make_event, geometry_for

from test_ls_pretests import D0, K_EPS, K_HALF_KMAX, K_MARGIN, SCALES, _info, module_may_pass, rcp, rsq, seg, \
    window_bound  # noqa: F401 (seg is a fixture)

f32 = np.float32
N_BINS = 32


# ------------------------------------------------------------- segments
def azimuth_bin(scale, s):
    u = (s * scale + f32(1)) * f32(0.5 * N_BINS)
    return np.minimum(np.maximum(u, f32(0)), f32(N_BINS - 1)).astype(np.int64)


def bins_looked_at(A, st, ma, disc, rng, mb, s, sc):
    """First bin and end of the bins of module mb that the count pass takes for the inner MD A
    (end 0: none)."""
    ec_a, hphi_a, hlong_a, er_a = _info(s, ma)
    ec_b, hphi_b, hlong_b, er_b = _info(s, mb)
    sqrt = lambda x: np.sqrt(x) * sc
    r = A[:, 3]
    ia = rcp(r, sc)
    ic = rcp(disc[:, 3], sc)
    nx, ny, c, rho = disc[:, 0] * ic, disc[:, 1] * ic, disc[:, 3], disc[:, 2]
    ub = K_HALF_KMAX * ((c + rho) + er_b)
    with np.errstate(invalid="ignore", divide="ignore", over="ignore"):
        w = (ub - K_HALF_KMAX * (r - er_a)) * rsq(f32(1) - ub * ub, sc) + (D0 + hphi_a + f32(0.005)) * ia
        wmax = np.where(ub < f32(0.99), (w * K_MARGIN + K_EPS) * f32(1.01) + f32(1e-6), f32(3e38)).astype(f32)
        sd = (nx * A[:, 1] - ny * A[:, 0]) * ia
        cd = (nx * A[:, 0] + ny * A[:, 1]) * ia
        some = c * np.abs(sd) - rho <= (wmax * (c + rho)) * f32(1.001) + f32(1e-4)
        scale = np.where(rho < f32(0.5) * c, c * rcp(rho, sc), f32(-1)).astype(f32)
        whole = ~((scale > 0) & (wmax < f32(0.69)) & (cd > f32(0.5)))
        sw = wmax * f32(1.0001) + f32(1e-6)
        cw = f32(0.9999) * sqrt(f32(1) - sw * sw)
        e2 = np.where(ec_a, hlong_a, hphi_a) + np.where(ec_b, hlong_b, hphi_b)
        x, y = st[:, 0], st[:, 1]
        near_b, far_b = rng[:, 0] - r, rng[:, 1] - r * cw
        bound_b = (rng[:, 0] * cw > r * f32(1.0001)) & (r * sw <= f32(0.9) * near_b)
        err_b = (f32(2) * hphi_a + (f32(2) * y) * (e2 * rcp(near_b, sc) + D0 * ia)) * (K_MARGIN * f32(1.0005)) + K_EPS \
            + f32(2e-4) * np.abs(x)
        z0, z1 = rng[:, 2] - A[:, 2], rng[:, 3] - A[:, 2]
        near_e, far_e = np.minimum(np.abs(z0), np.abs(z1)), np.maximum(np.abs(z0), np.abs(z1))
        chord = np.maximum(np.abs(rng[:, 0] - r), np.abs(rng[:, 1] - r)) + f32(1.1) * r * sw
        err_e = (f32(2) * hphi_a + y * (e2 + chord * D0 * ia) * rcp(near_e, sc)) * (K_MARGIN * f32(1.033)) + K_EPS \
            + f32(0.0313) * np.abs(x)
        near, far, err = np.where(ec_a, near_e, near_b), np.where(ec_a, far_e, far_b), np.where(ec_a, err_e, err_b)
        bound = np.where(ec_a, (z0 > 0) | (z1 < 0), bound_b) & (y > 0)
        f = ia * rcp(y, sc)
        x0, x1 = x - err, x + err
        p = x0 * np.where(x0 >= 0, near, far) * f
        q = x1 * np.where(x1 >= 0, far, near) * f
        lo = np.where(bound, np.fmax(-sw, p - (f32(1e-4) * np.abs(p) + f32(1e-5))), -sw)
        hi = np.where(bound, np.fmin(sw, q + (f32(1e-4) * np.abs(q) + f32(1e-5))), sw)
        none = ~some | (~whole & bound & ~(lo <= hi))
        cl, ch = sqrt(f32(1) - lo * lo), sqrt(f32(1) - hi * hi)
        b0 = np.where(~whole & (cl * cd - lo * sd > 0), azimuth_bin(scale, lo * cd + cl * sd - f32(1e-5)), 0)
        b1 = np.where(~whole & (ch * cd - hi * sd > 0), azimuth_bin(scale, hi * cd + ch * sd + f32(1e-5)) + 1, N_BINS)
    return b0, np.where(none, 0, b1)


def own_bin(B, disc, sc):
    with np.errstate(invalid="ignore"):
        s = (disc[:, 0] * B[:, 1] - disc[:, 1] * B[:, 0]) * (rcp(disc[:, 3], sc) * rcp(B[:, 3], sc))
        return azimuth_bin(disc[:, 3] * rcp(disc[:, 2], sc), s)


def module_ranges(s):
    M = s["geom"].n_modules
    rng = np.zeros((M, 4), f32)
    for k, (col, red, start) in enumerate(((3, np.minimum, np.inf), (3, np.maximum, -np.inf),
                                           (2, np.minimum, np.inf), (2, np.maximum, -np.inf))):
        v = np.full(M, start, f32)
        red.at(v, s["mod"], s["A"][:, col])
        rng[:, k] = v
    return rng


@pytest.mark.parametrize("sc_hit", SCALES)
@pytest.mark.parametrize("sc", SCALES)
def test_every_segment_is_in_a_bin_looked_at(seg, sc, sc_hit):  # noqa: F811
    s = seg
    a, b = s["la"], s["lb"]
    mb = s["mod"][b]
    disc, rng = s["disc"][mb], module_ranges(s)[mb]
    b0, b1 = bins_looked_at(s["A"][a], s["st"][a], s["mod"][a], disc, rng, mb, s, sc)
    at = own_bin(s["A"][b], disc, sc_hit)
    ok = (at >= b0) & (at < b1)
    assert len(a) > 400000
    assert ok.all(), f"{np.count_nonzero(~ok)} of {len(ok)} segments outside the bins"


def test_bins_prune(seg):  # noqa: F811
    """Of the MDs of the modules that the window reaches, the bins leave less than a third."""
    s = seg
    g = s["geom"]
    mo, mt = g.map_offsets.astype(np.int64), g.map_targets.astype(np.int64)
    md_off = np.searchsorted(s["mod"], np.arange(g.n_modules + 1))
    inner = np.sort(np.random.default_rng(5).choice(s["n_md"], 3000, replace=False))
    ne = mo[s["mod"][inner] + 1] - mo[s["mod"][inner]]
    pa = np.repeat(inner, ne)
    mb = mt[np.repeat(mo[s["mod"][inner]], ne) + np.arange(ne.sum()) - np.repeat(np.cumsum(ne) - ne, ne)]
    has = md_off[mb + 1] > md_off[mb]
    pa, mb = pa[has], mb[has]
    disc = s["disc"][mb]
    ma = s["mod"][pa]
    reach = module_may_pass(s["A"][pa], disc, window_bound(s["A"][pa], ma, disc, mb, s))
    b0, b1 = bins_looked_at(s["A"][pa], s["st"][pa], ma, disc, module_ranges(s)[mb], mb, s, f32(1))
    bins = own_bin(s["A"], s["disc"][s["mod"]], f32(1))
    seen = sum(int(np.count_nonzero((bins[md_off[m]:md_off[m + 1]] >= l) & (bins[md_off[m]:md_off[m + 1]] < h)))
               for m, l, h in zip(mb, b0, b1))
    assert seen < (md_off[mb + 1] - md_off[mb])[reach].sum() / 3


# ------------------------------------------------------------- mini-doublets
@pytest.mark.parametrize("config", ["pu200_seeded", "tiny"])
@pytest.mark.parametrize("sc", SCALES)
def test_every_md_is_in_a_bin_looked_at(config, sc):
    """An upper hit joins its module's bin floor(0.47 u / d) (mod 64) of u = tan(azimuth from one of the
    module's lower hits); a lower hit looks at the bins of u - d and u + d, d = 1.27 W + 4e-6."""
    geom = geometry_for(config)
    ev = make_event(config, 3)
    og = oracle.OracleGeometry(geom)
    md, _, _ = oracle.run(og, ev, last=0).stage(0)
    win = og.module_consts()[:, 0].astype(f32)
    lo, up = md[:, 0], md[:, 1]
    x, y = ev.x.astype(f32), ev.y.astype(f32)
    mod = ev.module[lo].astype(np.int64)
    ref = np.full(geom.n_modules, -1, np.int64)
    low = np.nonzero((ev.module >= 0) & (ev.sensor == 0))[0]
    for pick in (low, low[::-1]):  # any of the module's lower hits
        ref[ev.module[pick]] = pick
        d = win[mod] * f32(1.27) + f32(4e-6)
        inv = f32(0.47) / d

        def u_of(h):
            r = ref[mod]
            dot, cr = x[r] * x[h] + y[r] * y[h], x[r] * y[h] - y[r] * x[h]
            return cr * rcp(dot, sc), (dot > 0) & (np.abs(cr) <= f32(0.5) * dot)

        ul, in_l = u_of(lo)
        uu, in_u = u_of(up)
        bin_of = lambda u: np.floor(u * inv).astype(np.int64) & 63
        seen = (bin_of(uu) == bin_of(ul - d)) | (bin_of(uu) == bin_of(ul + d))
        # (a module with a hit outside the bins' range, or with a wide window, tests every pair)
        binned = in_l & in_u & (d < f32(0.25))
        assert binned.mean() > 0.99
        assert seen[binned].all(), f"{np.count_nonzero(~seen & binned)} of {binned.sum()} MDs outside the bins"
