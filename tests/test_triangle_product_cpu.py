"""The squared side of a triangle from |p|^2 - 2 p.q + |q|^2 in FP32, for p and q
the FP32 displacements of two neighbours within r' of the primary: within 80 u
r'^2 of the FP64 square in any order of the sum, products rounded or fused."""
import itertools

import numpy as np
import pytest

U32 = 2.0 ** -24


@pytest.mark.parametrize("r", [1e-3, 10.0, 30.0, 977.0])
def test_error_of_the_product_form(r):
    rng = np.random.default_rng(int(r) + 1)
    n = 40000

    def ball():
        v = rng.normal(size=(n, 3))
        v *= (r * np.where(rng.random(n) < 0.5, 1.0, rng.random(n)) / np.linalg.norm(v, axis=1))[:, None]
        return v.astype(np.float32)

    p, q = ball(), ball()
    q[: n // 4] = -p[: n // 4]                                        # the longest sides
    q[n // 4: n // 2] = p[n // 4: n // 2] * np.float32(1 + 2 ** -12)  # close pairs
    V = ((q.astype(np.float64) - p) ** 2).sum(axis=1)

    def sq(a):
        return (a[:, 0] * a[:, 0] + a[:, 1] * a[:, 1]) + a[:, 2] * a[:, 2]

    terms = [sq(q), np.float32(-2) * p[:, 0] * q[:, 0], np.float32(-2) * p[:, 1] * q[:, 1],
             np.float32(-2) * p[:, 2] * q[:, 2], sq(p)]
    worst = 0.0
    for order in itertools.permutations(range(5)):
        s = terms[order[0]]
        for k in order[1:]:
            s = (s + terms[k]).astype(np.float32)
        worst = max(worst, float(np.max(np.abs(s.astype(np.float64) - V))))
    assert worst <= 80.0 * U32 * r * r
    assert worst > 2.0 * U32 * r * r  # (the bound is not loose by orders of magnitude)
