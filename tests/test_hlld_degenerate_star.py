"""The Riemann solver where an outer star state is degenerate (host only).

rho (S - u)(S - S_M) - B_n^2 can vanish with a tangential field present, when
the fast speed of the other side bounds the fan.  The star state then keeps v_t
and B_t (Miyoshi & Kusano 2005), so the flux of B_t across the outer wave is that
of the outer state, B_t u - B_n v, and not the star state's B_t S_M - B_n v.  Such
states are found by bisection between random ones on either side of the
degeneracy and compared with the oracle, which says that it took that branch.
Tolerance: the denominator is within 1e-12 of the total pressure of zero, and
what is formed from values of order 1 to 40 without it agrees to 1e-11."""

import numpy as np
import pytest

import oracle as O
from test_hlld_range import GAMMA, hlld


def fast(r, p, b2, bn):
    a = (GAMMA * p + b2) / r
    return np.sqrt(0.5 * (a + np.sqrt(max(a * a - 4.0 * GAMMA * p * bn * bn / (r * r), 0.0))))


def fan(x, right):
    """The degeneracy's denominator and the speeds S (of that side) and S_M."""
    ql, qr, bn = x[:8], x[8:16], x[16]
    bl, br = (bn * bn + q[6] ** 2 + q[7] ** 2 for q in (ql, qr))
    c = max(fast(ql[0], ql[4], bl, bn), fast(qr[0], qr[4], br, bn))
    sl, sr = min(ql[1], qr[1]) - c, max(ql[1], qr[1]) + c
    rl, rr = ql[0] * (sl - ql[1]), qr[0] * (sr - qr[1])
    sm = (rr * qr[1] - rl * ql[1] - qr[4] - 0.5 * br + ql[4] + 0.5 * bl) / (rr - rl)
    return ((rr * (sr - sm), sr) if right else (rl * (sl - sm), sl)) + (sm, bn * bn)


def denominator(x, right):
    d, _, _, bn2 = fan(x, right)
    return d - bn2


def degenerate_states(right, count, seed):
    rng = np.random.default_rng(seed)
    below, above, out = [], [], []
    while len(out) < count:
        x = np.zeros(17)
        for o in (0, 8):
            x[o], x[o + 4] = 10.0 ** rng.uniform(-1.5, 1.5, 2)
            x[o + 1:o + 4] = rng.normal(0.0, 1.0, 3)
            x[o + 6:o + 8] = rng.normal(0.0, 0.7, 2)
        x[16] = rng.normal(0.0, 2.0)
        (below if denominator(x, right) < 0.0 else above).append(x)
        if not below or not above:
            continue
        a, b = below.pop(), above[-1]  # a: negative, b: positive
        for _ in range(200):
            m = 0.5 * (a + b)
            if denominator(m, right) < 0.0:
                a = m
            else:
                b = m
        _, s, sm, _ = fan(b, right)
        b[[1, 9]] -= 0.5 * (s + sm)  # the frame where x/t = 0 lies between S and S_M
        o = 8 if right else 0
        if abs(b[16]) < 0.2 or np.hypot(b[o + 6], b[o + 7]) < 0.1 or abs(sm - 0.5 * (s + sm) - b[o + 1]) < 0.02:
            continue
        L, R = b[:8].copy(), b[8:16].copy()
        L[5] = R[5] = b[16]
        F, info = O.hlld(L, R, GAMMA)
        if info[2 if right else 1] and info[0] not in (0, 5):
            out.append((b, F))
    return out


@pytest.mark.parametrize("right", [False, True])
def test_degenerate_star_keeps_the_outer_field_flux(right):
    cases = degenerate_states(right, 12, 7 + right)
    got = hlld(8, np.array([x for x, _ in cases]))
    for (_, want), g in zip(cases, got):
        assert np.max(np.abs(g - want)) <= 1e-11 * max(1.0, np.max(np.abs(want))), (g, want)
