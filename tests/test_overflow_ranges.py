"""Ranges of objects taken from offsets that run on past a stage's capacity (the event is then
refused, and rebuilt with more room): every index read stays inside the arrays."""
import ctypes

import numpy as np
import pytest

from kernel_host import build

CODE = """
extern "C" void ranges(int n_md, int *ls_off, int *t3_off, int *t5_off, int n_ls, int n_t3, int n_t5, int *out) {
  Ws w{};
  w.ls_off = ls_off;
  w.t3_off = t3_off;
  w.t5_off = t5_off;
  for (int m = 0; m < n_md; ++m) {
    const int2 r = md_triplets(w, m, n_ls, n_t3);
    out[4 * m] = r.x;
    out[4 * m + 1] = r.y;
    if (r.x < 0 || r.x > n_t3 || r.y < 0 || r.y > n_t3) continue;  // (t5_off has n_t3 + 1 entries)
    const int2 v = triplets_t5(w, r, n_t5);
    out[4 * m + 2] = v.x;
    out[4 * m + 3] = v.y;
  }
}
"""


# capacities over what is found (none past), just at it, and far below it, stage by stage
@pytest.mark.parametrize("cap_ls,cap_t3,cap_t5", [(1.5, 1.5, 1.5), (1, 1, 1), (1, 0.3, 1), (1, 0.01, 1), (1, 0, 1),
                                                  (0.4, 1, 1), (0.4, 0.2, 0.1)])
def test_ranges_of_an_md_stay_inside(cap_ls, cap_t3, cap_t5, tmp_path):
    lib = build(tmp_path, ["md_triplets", "triplets_t5"], CODE)
    rng = np.random.default_rng(3)
    n_md = 500
    off = lambda counts: np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ls_off = off(rng.integers(0, 12, n_md))
    n_ls = min(int(ls_off[-1]), int(cap_ls * ls_off[-1]))
    t3_off = off(rng.integers(0, 5, n_ls))       # offsets as the fills write them: not clamped
    n_t3 = min(int(t3_off[-1]), int(cap_t3 * t3_off[-1]))
    t5_off = off(rng.integers(0, 4, n_t3))
    n_t5 = min(int(t5_off[-1]), int(cap_t5 * t5_off[-1]))
    out = np.full((n_md, 4), -1, np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int))
    lib.ranges(n_md, p(ls_off), p(t3_off), p(t5_off), n_ls, n_t3, n_t5, p(out))
    bad = np.nonzero((out[:, :2] < 0).any(1) | (out[:, :2] > n_t3).any(1))[0]
    assert bad.size == 0, f"{bad.size} of {n_md} MDs read t5_off up to entry {out[bad, :2].max()} of {n_t3 + 1}"
    assert (out[:, 0] <= out[:, 1]).all() and (out[:, 2] <= out[:, 3]).all() and (out[:, 2:] <= n_t5).all()
    # the built triplets and quintuplets, each in one MD's range
    assert (out[:, 1] - out[:, 0]).sum() == n_t3 and (out[:, 3] - out[:, 2]).sum() == n_t5
