"""The encoder's row quantizer at the edges of fp32: denormal rows, infinities, NaN, ties; against the definition step by step."""
import numpy as np
import pytest

import paper_2509_22951_amd as tq
from oracle import oracle as O


def _by_definition(row, qmax):
    amax = np.float32(0)
    for v in np.abs(row):
        if amax < v:          # (a NaN compares false: it counts for nothing)
            amax = v
    with np.errstate(all="ignore"):
        s = np.float32(amax / np.float32(qmax))
        if not s > 0:
            return np.zeros(row.size, np.int8), s
        t = np.rint(row / s)
        t = np.where(-qmax < t, t, np.float32(-qmax))
        t = np.where(t < qmax, t, np.float32(qmax))
    return t.astype(np.int8), s


@pytest.mark.parametrize("bits", [8, 4, 2])
def test_rows_at_the_edges_of_fp32(bits):
    rng = np.random.default_rng(3)
    qmax = 2 ** (bits - 1) - 1
    w = (rng.standard_normal((9, 67)) * 0.02).astype(np.float32)
    w[0] = 0
    w[1] = np.float32(1e-45) * rng.integers(-100, 101, 67).astype(np.float32)   # a few denormal steps: the scale rounds
    w[2, 5] = np.nan
    w[3, 7] = np.inf
    w[4] = np.nan
    w[5] = np.arange(67, dtype=np.float32) - 33.0
    w[5, 0] = 2 * qmax                                                       # scale 2: odd values are ties
    w[6] *= np.float32(1e38)
    w[7, 3] = -np.nan
    w[8, 1], w[8, 2] = np.inf, np.nan
    blob = tq.tq_encode(w, bits=bits)
    Q, s = O.decode_blob(blob)[:2]
    for r in range(w.shape[0]):
        want_q, want_s = _by_definition(w[r], qmax)
        assert np.array_equal(Q[r], want_q), r
        assert s[r] == want_s or (np.isnan(s[r]) and np.isnan(want_s)), r
