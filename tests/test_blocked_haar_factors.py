"""The blocked form of the 1-D Haar transform of any length: its factors on the CPU."""
import numpy as np

from oracle import stamp_oracle as so


def test_factors_give_the_inverse_transform():
    """The factors that make up for a short block (host copy of the device formulas): plain a +- d with them equals the
    orthonormal inverse with carried nodes, for every level count and block length."""
    C = np.sqrt(0.5)

    def carries(m, l, i, r):
        c = 0
        for k in range(l, r):
            nk = -(-m // (1 << k))
            c += i == nk - 1 and nk & 1
            i >>= 1
        return c

    rng = np.random.default_rng(0)
    for r in range(3, 7):
        for m in range(1, (1 << r) + 1):
            t = rng.standard_normal((m, 1))
            ref = so.haar1d_ragged_inverse(t, r, np.float64)[:, 0] if m > 1 else t[:, 0]
            sizes = [-(-m // (1 << l)) for l in range(r + 1)]
            v = np.array([t[0, 0] * C ** (r + carries(m, r, 0, r))])
            for l in range(r, 0, -1):
                d = np.zeros(1 << (r - l))
                for i in range(sizes[l - 1] // 2):
                    d[i] = t[sizes[l] + i, 0] * C ** (l + carries(m, l, i, r))
                v = np.stack([v + d, v - d], 1).reshape(-1)
            y = np.array([v[i] * np.sqrt(2.0) ** carries(m, 0, i, r) for i in range(m)])
            assert np.allclose(y, ref, rtol=0, atol=1e-12), (r, m)
