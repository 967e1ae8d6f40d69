"""The barrel with few, wide modules: its modules merged into `nphi` sectors of `nz` rings a layer."""
import copy

import numpy as np


def sector_geometry(geom, nphi, nz):
    """The merged barrel, each module linked to the three nearest sectors of the next layer, and the
    merged module of each module."""
    phi, z = 0.5 * (geom.phimin + geom.phimax), 0.5 * (geom.lmin + geom.lmax)
    sec = np.minimum((phi / (2 * np.pi) * nphi).astype(int), nphi - 1)
    ring = np.minimum(((z + geom.barrel_zmax) / (2 * geom.barrel_zmax) * nz).astype(int), nz - 1)
    new = ((geom.layer - 1) * nz + ring) * nphi + sec
    n = 6 * nphi * nz
    first = np.array([np.nonzero(new == m)[0][0] for m in range(n)])
    g = copy.copy(geom)
    for a in ("subdet", "layer", "side", "type", "pos_lo", "pos_up"):
        setattr(g, a, getattr(geom, a)[first].copy())
    zi = (np.arange(n) // nphi) % nz
    step = 2 * geom.barrel_zmax / nz
    g.lmin, g.lmax = -geom.barrel_zmax + step * zi, -geom.barrel_zmax + step * (zi + 1)
    g.n_modules = n
    links = []
    for m in range(n):
        l, k = m // (nphi * nz), m % nphi
        links.append([] if l == 5 else sorted(((l + 1) * nz + q) * nphi + s for q in range(nz)
                                              for s in {(k + d) % nphi for d in (-1, 0, 1)}))
    g.map_offsets = np.cumsum([0] + [len(t) for t in links]).astype(np.int32)
    g.map_targets = np.concatenate(links).astype(np.int32)
    return g, new


def merge_event(ev, new):
    out = copy.copy(ev)
    out.module = np.where(ev.module >= 0, new[np.maximum(ev.module, 0)], -1).astype(np.int32)
    return out
