"""The mini-doublet search of modules that are listed by direction: whatever pair of hits the selection
accepts, anywhere round the beam line and for any window, the upper hit's bin is one of the two that the
lower hit looks at.  The kernel's own functions run on the host; the bins of the two hits are computed
in one kernel, so the hardware reciprocals are exact, 4 ulp high or 4 ulp low for both."""
import ctypes

import numpy as np
import pytest

from kernel_host import build
from test_ls_pretests import SCALES

CODE = """
// 1: not accepted, 2: all pairs tested, 3: in a bin looked at, 0: outside them
extern "C" void pairs(int n, const float *lo, const float *up, const float *W, int *out) {
  for (int i = 0; i < n; ++i) {
    const float *a = lo + 2 * i, *b = up + 2 * i;
    const float4 hi = make_float4(a[0], a[1], 0.f, sqrtf(a[0] * a[0] + a[1] * a[1]));
    const float4 hj = make_float4(b[0], b[1], 0.f, sqrtf(b[0] * b[0] + b[1] * b[1]));
    const float3 k = md_bins(W[i]);
    out[i] = 1;
    if (!md_pass(hi, hj, make_float4(W[i], 0.f, 0.f, 0.f), ModInfo{1})) continue;  // (2S: azimuth alone)
    out[i] = 2;
    if (k.z == 0.0f) continue;
    const float p = direction(hi.x, hi.y);
    const int at = md_bin(direction(hj.x, hj.y), k), b0 = md_bin(p - k.x, k), b1 = md_bin(p + k.x, k);
    out[i] = at >= 0 && at < (int)k.z && (at == b0 || at == b1) ? 3 : 0;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return build(tmp_path_factory.mktemp("k"), ["direction", "md_bins", "md_bin"], CODE)


@pytest.mark.parametrize("sc", SCALES)
def test_every_accepted_pair_is_in_a_bin_looked_at(lib, sc):
    lib.set_scale(sc)
    rng = np.random.default_rng(12)
    f, n = np.float32, 400000
    W = np.exp(rng.uniform(np.log(1e-7), np.log(2.0), n)).astype(f)
    W[:1000] = 0.0
    W[1000:2000] = rng.choice([0.3, 0.45, 0.9486, 0.95, 1.0, np.inf], 1000)
    phi = rng.uniform(-np.pi, np.pi, n)
    # about the directions where the pieces of `direction` meet, and where it wraps round
    phi[::3] = rng.choice([-np.pi, -np.pi / 2, 0, np.pi / 2, np.pi], n)[::3] + rng.normal(0, 1e-3, n)[::3] * rng.choice([0, 1, 1e-4], n)[::3]
    edge = np.arcsin(np.minimum(W.astype(np.float64), 1.0))  # at the window's edge, inside and outside
    dphi = edge * np.where(rng.uniform(size=n) < 0.5, 1 + rng.normal(0, 1e-6, n), rng.uniform(0, 1, n)) * rng.choice([-1, 1], n)
    ra, rb = np.exp(rng.uniform(np.log(1.1e-3), np.log(9e5), n)), np.exp(rng.uniform(np.log(1.1e-3), np.log(9e5), n))
    lo = np.stack([ra * np.cos(phi), ra * np.sin(phi)], 1).astype(f)
    up = np.stack([rb * np.cos(phi + dphi), rb * np.sin(phi + dphi)], 1).astype(f)
    lo[5000:6000, 1] = -0.0
    out = np.zeros(n, np.int32)
    p = lambda a: np.ascontiguousarray(a).ctypes.data_as(ctypes.c_void_p)
    lo, up = np.ascontiguousarray(lo), np.ascontiguousarray(up)
    lib.pairs(n, p(lo), p(up), p(W), p(out))
    assert (out == 3).sum() > 0.5 * n and (out == 2).sum() > 1000
    bad = np.nonzero(out == 0)[0]
    assert bad.size == 0, f"{bad.size} pairs outside the bins, first W {W[bad[0]]}, {lo[bad[0]]}, {up[bad[0]]}"
