"""The reverse of the HLLD flux follows the flux's own branches (host only).

Where the two sides are equal, or equal to a few roundings, the flux still picks
one fast speed to bound the fan, one velocity for each outermost wave and one
region; its derivative jumps between those choices.  The exact directional
derivative of the flux (forward-mode) and the hand-written reverse have to agree
there too.  Both sum some hundred products of order up to 1e2: 1e-9 of their
scale."""

import ctypes as C

import numpy as np
import pytest

from paper_1110_1616_amd import amr as A

GAMMA = 5.0 / 3.0


def dots(states, d, a):
    fn = A.lib().amr_selfcheck_hlld_adjoint
    fn.restype = C.c_int32
    fn.argtypes = [C.c_int64] + [C.c_void_p] * 3 + [C.c_double] + [C.c_void_p] * 2
    s, d, a = (np.ascontiguousarray(v, dtype=np.float64) for v in (states, d, a))
    f, r = np.empty(len(s)), np.empty(len(s))
    assert fn(len(s), s.ctypes.data, d.ctypes.data, a.ctypes.data, GAMMA, f.ctypes.data, r.ctypes.data) == A.AMR_OK
    return f, r


def base(n, r, drift):
    s = np.zeros((n, 8))
    s[:, 0] = r.uniform(0.5, 2.0, n)
    s[:, 1:4] = r.normal(0.0, 0.4, (n, 3))
    s[:, 1] += drift
    s[:, 4] = r.uniform(0.3, 2.0, n)
    s[:, 6:8] = r.normal(0.0, 0.6, (n, 2))
    return s


def jitter(x, r, roundings):
    return x * (1.0 + 2.0 ** -52 * r.integers(-roundings, roundings + 1, x.shape))


def fast2(q, bn):
    b2, gp = bn * bn + q[:, 6] ** 2 + q[:, 7] ** 2, GAMMA * q[:, 4]
    a = (gp + b2) / q[:, 0]
    return 0.5 * (a + np.sqrt(np.maximum(a * a - 4.0 * gp * (bn / q[:, 0]) ** 2, 0.0)))


def alfven(ql, qr, bn, right):
    """Speed of one side's Alfven wave."""
    c = np.sqrt(np.maximum(fast2(ql, bn), fast2(qr, bn)))
    sl, sr = np.minimum(ql[:, 1], qr[:, 1]) - c, np.maximum(ql[:, 1], qr[:, 1]) + c
    rl, rr = ql[:, 0] * (sl - ql[:, 1]), qr[:, 0] * (sr - qr[:, 1])
    pl, pr = (q[:, 4] + 0.5 * (bn * bn + q[:, 6] ** 2 + q[:, 7] ** 2) for q in (ql, qr))
    sm = (rr * qr[:, 1] - rl * ql[:, 1] - pr + pl) / (rr - rl)
    return sm + np.abs(bn) / np.sqrt(rr / (sr - sm)) if right else sm - np.abs(bn) / np.sqrt(rl / (sl - sm))


@pytest.mark.parametrize("roundings", [0, 1, 4])
@pytest.mark.parametrize("kind", ["state", "velocity", "fast speed", "left Alfven", "right Alfven"])
@pytest.mark.parametrize("drift", [0.0, 1.5])
def test_reverse_follows_the_flux_at_ties(drift, kind, roundings):
    n = 4000
    r = np.random.default_rng(int(10 * drift) + roundings)
    left, right, bn = base(n, r, drift), base(n, r, drift), r.normal(0.0, 0.6, n)
    if kind == "state":
        right = jitter(left, r, roundings)
    elif kind == "velocity":
        right[:, 1] = jitter(left[:, 1], r, roundings)
    elif kind == "fast speed":  # the same density, pressure and |B_t|, another direction of B_t
        right[:, [0, 4]] = jitter(left[:, [0, 4]], r, roundings)
        right[:, 6], right[:, 7] = jitter(left[:, 7], r, roundings), -left[:, 6]
    else:  # x/t = 0 on an Alfven wave
        for _ in range(3):
            sa = alfven(left, right, bn, kind.startswith("right"))
            left[:, 1] -= sa
            right[:, 1] -= sa
        left[:, 1] = jitter(left[:, 1], r, roundings)
    s = np.concatenate([left, right, bn[:, None]], axis=1)
    d, a = r.normal(0.0, 1.0, (n, 17)), r.normal(0.0, 1.0, (n, 7))
    f, rev = dots(s, d, a)
    err = np.abs(f - rev) / (1.0 + np.abs(f))
    assert np.all(np.isfinite(err)) and np.max(err) <= 1e-9, (np.max(err), np.count_nonzero(err > 1e-9))
