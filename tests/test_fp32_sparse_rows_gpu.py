"""GPU: fp32 sums of few terms, read out through models that pass their operands
through exactly, against 64 bits.  Such rows (pruned or sparse weights) show what a product
and an addition lose, which dense rows average away.

Each is compared with a chain of fp32 fused multiply-adds over the same terms
(emulated here: each step rounded to fp32 from 64 bits), the error in units of 2^-24 of
the sum of magnitudes.  An fp32 product is taken as bf16 parts without m l + l m, where
|m| <= 2^-8 and |l| <= 2^-17 of a significand: at most 1 unit, and for a given weight
with l and m of the other operand spread evenly at most sqrt(2 / 3) / 2 = 0.41 units in
the root mean square.  A row of one term may exceed the chain's rounding by that (its
largest error: 1 + 1 units and the rounding of the small products); rows of more terms
have fewer roundings at full size than the chain, so their root mean square error is no
larger (2 % for the sampling)."""
import numpy as np
import pytest

import tracksynth as ts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 4000


def _params(blob, layout):
    p, o = {}, 0
    for name, shape, _, _ in layout:
        p[name] = blob[o:o + int(np.prod(shape))].reshape(shape)
        o += p[name].size
    assert o == blob.size
    return p


def _pass_through(p, d):
    """Embedding weights that make channel c the hit's coordinate c % 3 over 2^(c % 5):
    the normalisation's spans and offsets are undone exactly."""
    span, lo = np.array([2000.0, 2000.0, 6000.0]), np.array([-1000.0, -1000.0, -3000.0])
    for c in range(d):
        s = 2.0 ** -(c % 5)
        p["embed.W"][c, c % 3] = span[c % 3] * s
        p["embed.b"][c] = lo[c % 3] * s
    return lambda h: h[:, np.arange(d) % 3] * (2.0 ** -(np.arange(d) % 5)).astype(np.float32)


def _sparse(rng, rows, cols, terms, positive=False):
    W = np.zeros((rows, cols), np.float32)
    for r in range(rows):
        v = rng.normal(0, 1, terms).astype(np.float32)
        W[r, rng.choice(cols, terms, replace=False)] = np.abs(v) + np.float32(0.5) if positive else v
    return W


def _check(got, X, W, terms, what):
    """got [N, rows] against X [N, cols] W^T."""
    ref, mag = np.zeros(got.shape), np.zeros(got.shape)
    chain = np.zeros(got.shape, np.float32)
    for r in range(W.shape[0]):
        for c in np.nonzero(W[r])[0]:
            t = X[:, c].astype(np.float64) * np.float64(W[r, c])
            ref[:, r] += t
            mag[:, r] += np.abs(t)
            chain[:, r] = (t + chain[:, r]).astype(np.float32)
    e, ec = np.abs(got - ref) / mag * 2.0 ** 24, np.abs(chain - ref) / mag * 2.0 ** 24
    rms, rms_c = np.sqrt((e ** 2).mean()), np.sqrt((ec ** 2).mean())
    print(f"[sparse] {what}, {terms} terms: rms {rms:.3f} (chain {rms_c:.3f}), max {e.max():.2f} ({ec.max():.2f})", flush=True)
    assert rms <= (np.hypot(rms_c, 0.41) if terms == 1 else 1.02 * rms_c)
    assert e.max() <= max(ec.max() + 0.5, 2.1)


def _hits(rng):
    h = rng.uniform(100, 1000, (N, 3)).astype(np.float32)
    return h, torch.from_numpy(h).cuda(), torch.arange(N + 1, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("terms", [1, 2, 3, 8, 16])
@pytest.mark.parametrize("d,H,layers", [(32, 64, 1), (128, 192, 1), (32, 64, 2), (128, 192, 2)])
def test_mingru_rows(d, H, layers, terms):
    """Tracks of one hit with the gates at 80 (sigmoid 1): a state is its candidate.  With
    two layers the first one passes the channels on, so that the second one's rows are seen."""
    import paper_2609_32479_amd as tf
    rng = np.random.default_rng([d, layers, terms])
    blob = np.zeros(tf.MinGRU.blob_size(layers, d, H), np.float32)
    p = _params(blob, ts.mingru_layout(layers, d, H, 0))
    emb = _pass_through(p, d)
    for l in range(layers):
        p[f"mg{l}.b"][H:2 * H] = p[f"mg{l}.b"][3 * H:] = 80.0
    W = _sparse(rng, 2 * H, d if layers == 1 else 2 * H, terms)
    p[f"mg{layers - 1}.W"][:H], p[f"mg{layers - 1}.W"][2 * H:3 * H] = W[:H], W[H:]
    h, hg, og = _hits(rng)
    X = emb(h)
    if layers == 2:
        for j in range(2 * H):
            p["mg0.W"][j if j < H else j + H, j % d] = 1.0
        X = X[:, np.arange(2 * H) % d]
    got = tf.MinGRU(blob, layers, d, H, "fp32").states(hg, og).cpu().numpy()
    _check(got, X, W, terms, f"minGRU d={d} layers={layers}")


@pytest.mark.parametrize("terms", [1, 2, 3, 8, 16])
@pytest.mark.parametrize("which", ["W1", "W2"])
@pytest.mark.parametrize("d,max_hits", [(32, 32), (64, 32), (128, 32), (128, 64)])
def test_head_rows(d, max_hits, which, terms):
    """A model without layers and tracks of one hit: out = W2 SiLU(W1 p), with arguments
    above 90, where SiLU is its argument; the other matrix passes its input on."""
    import paper_2609_32479_amd as tf
    rng = np.random.default_rng([d, max_hits, terms])
    blob = np.zeros(tf.blob_size(0, d), np.float32)
    p = _params(blob, ts.blob_layout(0, d))
    emb = _pass_through(p, d)
    h, hg, og = _hits(rng)
    h *= 32
    hg *= 32
    if which == "W1":
        W = _sparse(rng, 5, d, terms, positive=True)
        p["head.W1"][:5] = W
        p["head.W2"][np.arange(5), np.arange(5)] = 1.0
    else:
        W = _sparse(rng, 5, d, terms)
        p["head.W1"][np.arange(d), np.arange(d)] = 1.0
        p["head.W2"][:] = W
    out = tf.fit_tracks(hg, og, tf.Weights(blob, 0, d, "fp32", max_hits=max_hits)).cpu().numpy()
    _check(out, emb(h), W, terms, f"head {which} d={d} max_hits={max_hits}")
