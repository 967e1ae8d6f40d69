"""The triplet search's pre-test as the kernel evaluates it now: the azimuth-z test alone, with the
parent segment's terms (its sine as a product of two reciprocals) computed apart from the pair's.
Replayed in IEEE float32 as in test_t3_t5_pretests, the reciprocals exact, 4 ulp high and 4 ulp low,
for the parent's terms and the pair's independently: every triplet of the oracle passes, and few of
the other segment pairs do (the curvature cut, no longer tested first, would take 2% of them).
"""
import numpy as np
import pytest

from test_t3_t5_pretests import D0, K_EPS, K_MARGIN, K_THIRD, SCALES, curvature_may_pass, objs, rcp  # noqa: F401

f32 = np.float32


def parent(A, B, mA, mB, sc):
    iP, iQ = rcp(A[:, 3], sc), rcp(B[:, 3], sc)
    return ((A[:, 0] * B[:, 1] - A[:, 1] * B[:, 0]) * (iP * iQ), B[:, 2] - A[:, 2],
            (mA["hphi"] * iP + mB["hphi"] * iQ) + D0 * np.abs(iP - iQ), iQ)


def may_pass(p, B, C, mA, mB, mC, sc):
    su, dzpq, ePQ, iQ = p
    iR = rcp(C[:, 3], sc)
    sv = (B[:, 0] * C[:, 1] - B[:, 1] * C[:, 0]) * (iQ * iR)
    dzqr = C[:, 2] - B[:, 2]
    t1, t2 = su * dzqr, sv * dzpq
    eQR = (mB["hphi"] * iQ + mC["hphi"] * iR) + D0 * np.abs(iQ - iR)
    au, av, adpq, adqr = np.abs(su), np.abs(sv), np.abs(dzpq), np.abs(dzqr)
    nl = (au * au + av * av) * K_THIRD
    tol = ((adqr * ePQ + adpq * eQR) + (au * (mB["ez"] + mC["ez"]) + av * (mA["ez"] + mB["ez"]))) + \
        nl * (au * adqr + av * adpq)
    return np.abs(t1 - t2) <= (tol * K_MARGIN + K_EPS) * f32(1.00001) + f32(1e-5) * (np.abs(t1) + np.abs(t2))


def _split(anchors):
    P, m = anchors
    return [P[:, k] for k in range(3)], [{n: v[:, k] for n, v in m.items()} for k in range(3)]


@pytest.mark.parametrize("sc_pair", SCALES)
@pytest.mark.parametrize("sc", SCALES)
def test_every_triplet_passes(objs, sc, sc_pair):  # noqa: F811
    (A, B, C), (mA, mB, mC) = _split(objs[0])
    ok = may_pass(parent(A, B, mA, mB, sc), B, C, mA, mB, mC, sc_pair)
    assert len(ok) > 50000
    assert ok.all(), f"{np.count_nonzero(~ok)} of {len(ok)} triplets rejected"


def test_it_prunes(objs):  # noqa: F811
    cands, n_t3 = objs[2]["t3"]
    (A, B, C), (mA, mB, mC) = _split(cands)
    ok = may_pass(parent(A, B, mA, mB, f32(1)), B, C, mA, mB, mC, f32(1))
    both = ok & curvature_may_pass(A, B, C, mA, mB, mC)
    assert n_t3 <= both.sum() <= ok.sum() < 0.05 * len(ok)
    assert ok.sum() < 1.05 * both.sum()
