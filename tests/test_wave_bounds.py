"""The bracket algebra of the wave kernel (`wave_level`, `draw_bound` of
da_wave.hip) restated in numpy and checked on the CPU against its definition
d < T (-ln U_u), over every draw: both forms of the bound, temperatures from
10^-3 to 10^8 and zero, every number of fraction bits a level may get, a device
log2 off by its largest measured error in either direction, costs at and around
the threshold, at zero and below, both values of x.  z >= 0 must mean accepted,
z < -wt rejected."""
import numpy as np
import pytest

LN2 = np.log(2.0)
U = np.arange(65536)
G = -np.log((U + 0.5) / 65536.0)
LOG2_ERR = 2.0 ** -19          # above any fp32 log2's rounding at 16


def _level(T, qcap, gerr, clamp):
    e = np.frexp(T)[1] if T > 0 else 0
    q = min(max(17 - e, 0), qcap)
    Tq = np.ldexp(T, q)
    m = np.float32(np.float32(np.float32(Tq) * np.float32(gerr)) + np.float32(0.01))
    c0 = (min(q, 1) if T > 0 else -1) if clamp else 0
    wt = int(2 * m) + (2 if clamp else 3) if T > 0 else 1 - min(q, 1)
    mid = Tq * 16.0 * LN2
    ga = np.float32(-Tq * LN2)
    gb = np.float32(mid - float(m) - c0) if clamp else np.float32(12582912.0 + np.floor(mid - float(m) - 0.5))
    return q, Tq, c0, wt, ga, gb


def _bound(lg, ga, gb, clamp):
    # the product of two fp32 numbers is exact in double; one rounding of the sum
    t = (lg.astype(np.float64) * float(ga) + float(gb)).astype(np.float32)
    if clamp:
        return np.trunc(np.maximum(t, 0)).astype(np.int64)
    assert (t >= 2.0**23).all() and (t < 2.0**24).all()
    return t.view(np.int32).astype(np.int64) - 0x4B400000


@pytest.mark.parametrize("T", [0.0, 1e-3, 0.05, 1.0, 3.2, 96.0, 3277.0, 65536.0, 131071.9, 131072.0,
                               196608.0, 262143.0, 262144.0, 3.4e6, 1e8])
@pytest.mark.parametrize("off", [-1.0, 0.0, 1.0])
def test_bracket(T, off):
    exact = 16.0 - G / LN2
    lg = (exact + off * LOG2_ERR).astype(np.float32)
    gerr = 0.6932 * float(np.abs(lg - exact).max()) + 2.2e-6
    for qcap in (0, 1, 5, 17):
        for clamp in (True, False):
            q, Tq, c0, wt, ga, gb = _level(T, qcap, gerr, clamp)
            if not clamp and Tq >= 2.0**18:
                continue      # that form is not used there
            L = _bound(lg, ga, gb, clamp)
            y = Tq * G if T > 0 else np.zeros(65536)
            near = np.floor(np.minimum(y, 2.0**40) / 2.0**q).astype(np.int64)
            for d in [near + k for k in range(-3, 5)] + [np.full(65536, v) for v in (-(2**20), -1, 0, 1)]:
                dq = d << q
                accepted = dq < y
                for short in (0, 1):                    # x = 1, x = 0
                    z = L + c0 - dq - short
                    assert accepted[z >= 0].all(), (qcap, clamp)
                    assert not accepted[z < -wt].any(), (qcap, clamp)
            if T > 0 and clamp and q >= 1:              # costs of zero never need the definition
                assert (L + c0 - 1 >= 0).all()
