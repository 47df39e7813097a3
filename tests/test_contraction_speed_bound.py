"""The bound that lets the march skip along contracted rays (Sec. 4, the
L-infinity contraction).  At a point u of a straight ray with velocity v,
m = |u|inf > 1 on axis i, m' = sign(u_i) v_i, w = v - (u / m) m', and ml = m
for an outward ray (m' >= 0), (m + 1) / 2 for an inward one, the image C(u)
moves no faster than |m'| / ml^2 along axis i and |m'| / ml^2 + (2 - 1/ml) / ml
|w_j| m / ml along any axis j, until axis j may dominate, (m - |u_j|) /
(|v_j| - m') later, or the inward ray reaches ml.  Checked in FP64 on densely
sampled curves of seeded rays; CPU only."""
import numpy as np
import pytest


def contract(u):
    m = np.max(np.abs(u), axis=-1, keepdims=True)
    return np.where(m <= 1.0, u, (2.0 - 1.0 / m) * u / m)


@pytest.mark.parametrize("inward", [False, True])
def test_speed_bound_holds_and_is_useful(inward):
    rng = np.random.default_rng(5 + inward)
    checked, ratio = 0, []
    while checked < 2000:
        u = rng.normal(size=3) * np.exp(rng.uniform(0.0, 4.0))
        v = rng.normal(size=3)
        v /= np.linalg.norm(v)
        i = int(np.argmax(np.abs(u)))
        m, dm = np.abs(u[i]), np.sign(u[i]) * v[i]
        if m <= 1.0 or (dm < 0) != inward:
            continue
        checked += 1
        ml = 0.5 * (m + 1.0) if inward else m
        speed = np.abs(dm) / ml ** 2 + (2.0 - 1.0 / ml) / ml * np.abs(v - u / m * dm) * (m / ml)
        reach = (m - ml) / -dm if inward else 8.0 * m
        for j in range(3):
            if j != i and np.abs(v[j]) > dm:
                reach = min(reach, (m - np.abs(u[j])) / (np.abs(v[j]) - dm))
        s = np.linspace(0.0, reach, 400)[1:]
        moved = np.abs(contract(u + s[:, None] * v) - contract(u))
        assert np.all(moved <= speed * s[:, None] * (1 + 1e-9) + 1e-12), (u, v)
        k = max(0, len(s) // 16 - 1)
        ratio.append(float(np.max(moved[k] / (speed * s[k] + 1e-300))))
    assert np.median(ratio) > (0.2 if inward else 0.5)
