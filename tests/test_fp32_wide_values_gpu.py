"""GPU: fp32 models whose weights or operands are infinite, or so large that the bf16
parts of a product would overflow apart.  The sums must be what fp32 arithmetic gives,
infinite with the right sign or finite to fp32 precision, never the NaN of parts that
cancel; and the other tracks of the tile keep their bits."""
import dataclasses

import numpy as np
import pytest

import oracle
import tracksynth as ts
from tests.parity import TOL
from tests.test_fp32_sparse_rows_gpu import _params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BIG = 3.4e38
# normal, around the limit of the operands, close to and (times the embedding's 4) beyond fp32
X = np.array([100.0, 2.0 ** 87, 2.0 ** 88, 2.0 ** 89, 1e30, BIG / 4, 1.9922 * 2.0 ** 125, BIG, 777.0], np.float32)


def _one_hit(x):
    h = np.zeros((len(x), 3), np.float32)
    h[:, 0] = x
    return torch.from_numpy(h).cuda(), torch.arange(len(x) + 1, dtype=torch.int32, device="cuda")


def _embed(p):
    """Channel 0 of the embedding is 4 times the hit's x, exactly; the others are 0."""
    p["embed.W"][0, 0], p["embed.b"][0] = 8000.0, -4000.0


def _close(got, ref, rel):
    """fp32's infinities of ref (64 bits), else ref to rel."""
    with np.errstate(over="ignore"):
        r32 = ref.astype(np.float32)
    inf = np.isinf(r32)
    assert np.array_equal(got[inf], r32[inf]), (got, r32)
    assert (np.abs(got[~inf] - ref[~inf]) <= rel * np.abs(ref[~inf])).all(), (got, ref)


@pytest.mark.parametrize("w", [1.5, 1.25e-20, -1.5, 3e20, np.inf])
@pytest.mark.parametrize("d,max_hits", [(32, 32), (64, 32), (128, 32), (32, 64), (128, 64)])
def test_head_of_large_values(d, max_hits, w):
    """A model without layers: every unit of the hidden layer takes channel 0 with weight w,
    every output all units with weight 1."""
    import paper_2609_32479_amd as tf
    blob = np.zeros(tf.blob_size(0, d), np.float32)
    p = _params(blob, ts.blob_layout(0, d))
    _embed(p)
    p["head.W1"][:, 0], p["head.W2"][:] = w, 1.0
    W = tf.Weights(blob, 0, d, "fp32", max_hits=max_hits)
    with np.errstate(over="ignore"):
        pooled = (4 * X.astype(np.float64)).astype(np.float32)
        hidden = (pooled * np.float64(np.float32(w))).astype(np.float32).astype(np.float64)
    # SiLU; its exponent is clamped to 80, which matters for large negative arguments
    ref = d * hidden / (1.0 + np.exp(-np.clip(hidden, -80.0, 80.0)))
    use = hidden != 0.0
    got = tf.fit_tracks(*_one_hit(X), W).cpu().numpy()
    for c in range(5):
        _close(got[use, c], ref[use], 1e-5)
    for i in range(len(X)):  # every track alone
        assert np.array_equal(tf.fit_tracks(*_one_hit(X[i:i + 1]), W).cpu().numpy()[0], got[i])


@pytest.mark.parametrize("w,gate", [(1.5, 1.0), (1.25e-20, 1.0), (-1.5, 1.0), (3e20, 1.0), (1.5, np.inf)])
@pytest.mark.parametrize("d,H,layers", [(32, 64, 1), (128, 192, 1), (32, 64, 2), (128, 192, 2)])
def test_mingru_of_large_values(d, H, layers, w, gate):
    """Tracks of one hit: the last layer's candidates take channel 0 (or the first layer's
    state 0, which is channel 0) with weight w, its gates are open (80 + gate times channel 0)."""
    import paper_2609_32479_amd as tf
    blob = np.zeros(tf.MinGRU.blob_size(layers, d, H), np.float32)
    p = _params(blob, ts.mingru_layout(layers, d, H, 0))
    _embed(p)
    for l in range(layers):
        p[f"mg{l}.b"][H:2 * H] = p[f"mg{l}.b"][3 * H:] = 80.0
        p[f"mg{l}.W"][H:2 * H, 0] = p[f"mg{l}.W"][3 * H:, 0] = gate
    if layers == 2:
        p["mg0.W"][0, 0] = 1.0
    p[f"mg{layers - 1}.W"][:H, 0] = p[f"mg{layers - 1}.W"][2 * H:3 * H, 0] = w
    M = tf.MinGRU(blob, layers, d, H, "fp32")
    # (an infinite state would be multiplied by the 0 of the next track's start, and infinite
    # first-layer inputs by zero weights: those only alone, and through one layer)
    with np.errstate(over="ignore"):
        first = (4 * X.astype(np.float64)).astype(np.float32)
        ref = first * np.float64(np.float32(w))
        inf = np.isinf(first) | np.isinf(ref.astype(np.float32))
    alone = np.stack([M.states(*_one_hit(X[i:i + 1])).cpu().numpy()[0] for i in range(len(X))])
    for i in range(len(X)):
        if not (layers == 2 and np.isinf(first[i])):
            _close(alone[i], np.full(2 * H, ref[i]), 1e-6)
    fin = X[~inf]
    if len(fin):
        many = np.resize(fin, 5000)  # tiles of wide and other tracks
        assert np.array_equal(M.states(*_one_hit(many)).cpu().numpy(), np.resize(alone[~inf], (5000, 2 * H)))


@pytest.mark.parametrize("d,max_hits", [(32, 32), (64, 32), (128, 32), (64, 64), (128, 64)])
def test_encoder_with_infinite_gate_weights(d, max_hits):
    """Some gates always open or shut, against the oracle."""
    import paper_2609_32479_amd as tf
    w = dataclasses.replace(ts.workload("d128x4_fp32_65k"), n_layers=2, d_model=d, len_min=1,
                            len_max=20 if max_hits == 32 else 64, n_det_layers=64)
    hits, offs = ts.make_tracks(w, n_tracks=200)
    blob = ts.make_weights(n_layers=2, d=d, dtype="fp32", seed=5)
    p = _params(blob, ts.blob_layout(2, d))
    p["layer0.in.W"][d + 3, 7], p["layer0.in.W"][2 * d - 1, 0], p["layer1.in.W"][d, d - 1] = np.inf, -np.inf, np.inf
    W = tf.Weights(blob, 2, d, "fp32", max_hits=max_hits)
    h, o = torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda()
    g = tf.fit_tracks(h, o, W).cpu().numpy().astype(np.float64)
    r = oracle.fit_tracks(hits, offs, blob, 2, d)
    assert np.isfinite(r).all()
    rms = np.sqrt(np.mean(r ** 2, axis=0))
    assert np.max(np.abs(g - r) / np.maximum(np.abs(r), rms)) <= TOL["fp32"]
    assert torch.isfinite(tf.fit_tracks_states(h, o, W)).all()


@pytest.mark.parametrize("max_hits", [32, 64])
@pytest.mark.parametrize("d", [32, 128])
def test_fourier_projection_of_large_weights(d, max_hits):
    """The front end's weights 2^40 times as large, the head's first layer 2^-40: the
    outputs of the model as it was (the layers' norm takes the factor out), against the
    oracle."""
    import paper_2609_32479_amd as tf
    w = dataclasses.replace(ts.workload("d128x4_fp32_65k"), n_layers=1, d_model=d, len_min=1, len_max=20)
    _, offs = ts.make_tracks(w, n_tracks=200)
    nf, rng = 5, np.random.default_rng(8)
    feats = rng.uniform(0, 1, (int(offs[-1]), nf)).astype(np.float32)
    layout = ts.fourier_layout(1, d, nf)
    blob = np.concatenate([rng.normal(0, s[-1] ** -0.5, int(np.prod(s))) if len(s) > 1 else rng.uniform(0.5, 1, s)
                           for _, s, _, _ in layout]).astype(np.float32)
    p = _params(blob, layout)
    p["fe.lo"][:], p["fe.hi"][:] = 0.0, 1.0
    for k in ("fe.W", "fe.b", "layer0.out.W", "layer0.out.b"):
        p[k] *= np.float32(2.0 ** 40)
    p["head.W1"] *= np.float32(2.0 ** -40)
    W = tf.Weights(blob, 1, d, "fp32", max_hits=max_hits, n_features=nf)
    g = tf.fit_tracks(torch.from_numpy(feats).cuda(), torch.from_numpy(offs).cuda(), W).cpu().numpy().astype(np.float64)
    r = oracle.fit_tracks(feats, offs, blob, 1, d, n_features=nf)
    rms = np.sqrt(np.mean(r ** 2, axis=0))
    assert np.max(np.abs(g - r) / np.maximum(np.abs(r), rms)) <= TOL["fp32"]
