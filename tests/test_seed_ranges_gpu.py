"""GPU: the seed's residual features over turning angles up to a full turn and
residuals of every size, against the fp64 oracle: both sides of the lines where the
kernel's arc length and asinh change their method (turning angle pi / 4 and
argument 1/2), batches on both sides of the rows that a wave keeps on chip, and
track counts around a wave's 32.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# A float32 feature may differ by the rounding of the result (half an ulp, 6e-8)
# and by the fp64 rounding of the residual: the two circle formulas differ by
# about 1e-8 mm on these circles (R up to 3 m, first chords of 50 mm and more).
REL, ABS = 1.5e-7, 2e-8


def _circle_tracks(n, n_hits, max_angle, moved, seed):
    """Hits on helices whose circles pass near the axis, at increasing turning
    angles up to max_angle; hits from the fourth on moved by N(0, moved) mm."""
    g = np.random.default_rng(seed)
    R, phi, k = g.uniform(300, 3000, (n, 1)), g.uniform(-np.pi, np.pi, (n, 1)), np.sign(g.uniform(-1, 1, (n, 1)))
    a = np.cumsum(g.uniform(0.5, 1.5, (n, n_hits)), axis=1)
    a = a / a[:, -1:] * max_angle
    cx, cy = -k * R * np.sin(phi), k * R * np.cos(phi)
    x = cx + R * np.sin(phi + k * a) * k
    y = cy - R * np.cos(phi + k * a) * k
    z = g.normal(0, 1, (n, 1)) + R * a * g.uniform(-2, 2, (n, 1))
    h = np.stack([x, y, z], axis=2)
    h[:, 3:] += g.normal(0, 1, h[:, 3:].shape) * moved
    return np.ascontiguousarray(h.reshape(-1, 3), dtype=np.float32), np.arange(0, n * n_hits + 1, n_hits, dtype=np.int32)


@pytest.mark.parametrize("n,n_hits", [(1, 3), (31, 12), (33, 16), (200, 17), (65, 40)])
@pytest.mark.parametrize("max_angle", [0.3, 0.8, 1.57, 3.1])
@pytest.mark.parametrize("moved", [0.0, 0.3, 30.0])
def test_features_over_angles_and_residuals(n, n_hits, max_angle, moved):
    import paper_2609_32479_amd as tf
    hits, offs = _circle_tracks(n, n_hits, max_angle, moved, 7)
    seeds, feats = tf.seed_tracks(torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda(), 2.0)
    r_seed, r_feat, bad = oracle.seed_tracks(hits, offs, 2.0)
    g = feats.cpu().numpy().astype(np.float64)
    assert bad == 0 and np.isfinite(g).all()
    assert np.all(np.abs(g - r_feat) <= ABS + REL * np.abs(r_feat)), np.max(np.abs(g - r_feat) - REL * np.abs(r_feat))
    alone, _ = tf.seed_tracks(torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda(), 2.0, features=False)
    assert torch.equal(alone, seeds)  # the same seeds without the features
