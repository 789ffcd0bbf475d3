"""The bound by which the collapse z pass leaves out points: F > 0 implies F <= delta/2 + 0.6915 |T|
(applied there with 0.7).  Checked with the oracle's model over the eigenvalue directions."""

import numpy as np

from oracle import collapse


def _ratio(lam):
    lam = lam / np.linalg.norm(lam, axis=1)[:, None]
    z = np.zeros(len(lam))
    f = collapse.inverse_collapse_time([lam[:, 0], z, z, lam[:, 1], z, lam[:, 2]])
    return np.where(f > 0, f - 0.5 * lam.sum(axis=1), -np.inf)


def test_collapse_time_bound():
    th, ph = np.meshgrid(np.linspace(0, np.pi, 701), np.linspace(0, 2 * np.pi, 1401))
    lam = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], -1).reshape(-1, 3)
    r = _ratio(lam)
    worst = lam[np.argmax(r)]
    # and densely around the worst direction of the grid
    near = worst + 2e-2 * np.random.default_rng(0).standard_normal((200000, 3))
    top = max(r.max(), _ratio(near).max())
    assert 0.68 < top < 0.692, top
