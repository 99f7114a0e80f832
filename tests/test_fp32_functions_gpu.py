"""GPU: the fp32 gate's sigmoid and the head's SiLU, read out through models whose
weights pass their argument through exactly, against 64 bits: no further from it than the
library's exp and a division are.

Both are compared with the same form in the library's functions (torch's exp and
quotient on the GPU): the root mean square error over 60 000 arguments may exceed its by
one per cent (the sampling error of that figure), the largest by a tenth of an ulp (the
hardware's exp2 sees arguments that differ in their last bit)."""
import numpy as np
import pytest

import tracksynth as ts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _ulp_error(got, ref):
    return np.abs(got.astype(np.float64) - ref) / np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)


def _check(got, lib, ref):
    g, l = _ulp_error(got, ref), _ulp_error(lib, ref)
    print(f"max {g.max():.4f} (library {l.max():.4f}), rms {np.sqrt((g ** 2).mean()):.4f} "
          f"({np.sqrt((l ** 2).mean()):.4f}) ulp", flush=True)
    assert np.sqrt((g ** 2).mean()) <= 1.01 * np.sqrt((l ** 2).mean())
    assert g.max() <= l.max() + 0.1


@pytest.mark.parametrize("span", [80.0, 10.0, 1.0])
def test_gate_sigmoid(span):
    """A one-hit track's state is sigmoid(gate) * candidate: channel 0 of the
    embedding is the hit's x (weights 2000, bias -1000 undo the normalisation exactly), the
    gate rows take it with weight 1 and the candidate is 1."""
    import paper_2609_32479_amd as tf
    d, H, n = 32, 64, 60000
    blob, p, o = np.zeros(tf.MinGRU.blob_size(1, d, H), np.float32), {}, 0
    for name, shape, _, _ in ts.mingru_layout(1, d, H, 0):
        p[name] = blob[o:o + int(np.prod(shape))].reshape(shape)
        o += p[name].size
    eW, eb, W, b = p["embed.W"], p["embed.b"], p["mg0.W"], p["mg0.b"]
    eW[0, 0], eb[0] = 2000.0, -1000.0
    W[H:2 * H, 0] = W[3 * H:, 0] = 1.0
    b[:H] = b[2 * H:3 * H] = 1.0
    M = tf.MinGRU(blob, 1, d, H, "fp32")
    hits = np.zeros((n, 3), np.float32)
    hits[:, 0] = np.random.default_rng(1).uniform(-span, span, n)
    st = M.states(torch.from_numpy(hits).cuda(), torch.arange(n + 1, dtype=torch.int32, device="cuda")).cpu().numpy()
    x = hits[:, 0]
    xg = torch.from_numpy(x).cuda()
    lib = (1.0 / (1.0 + torch.exp(-xg))).cpu().numpy()
    for c in (0, 2 * H - 1):
        _check(st[:, c], lib, 1.0 / (1.0 + np.exp(-x.astype(np.float64))))


@pytest.mark.parametrize("span", [80.0, 10.0, 1.0])
def test_head_silu(span):
    """A model without layers and tracks of one hit: out = W2 SiLU(W1 p), p the embedded
    hit; unit 0 takes channel 0 (the hit's x, as above) and output 0 takes unit 0."""
    import paper_2609_32479_amd as tf
    d, n = 32, 60000
    blob = np.zeros(tf.blob_size(0, d), np.float32)
    blob[0], blob[3 * d] = 2000.0, -1000.0  # embed.W[0][0], embed.b[0]
    blob[4 * d] = 1.0                       # head.W1[0][0]
    blob[4 * d + d * d + d] = 1.0           # head.W2[0][0]
    W = tf.Weights(blob, 0, d, "fp32", max_hits=32)
    hits = np.zeros((n, 3), np.float32)
    hits[:, 0] = np.random.default_rng(2).uniform(-span, span, n)
    out = tf.fit_tracks(torch.from_numpy(hits).cuda(), torch.arange(n + 1, dtype=torch.int32, device="cuda"), W).cpu().numpy()
    x = hits[:, 0]
    xg = torch.from_numpy(x).cuda()
    lib = (xg / (1.0 + torch.exp(-xg))).cpu().numpy()
    _check(out[:, 0], lib, x.astype(np.float64) / (1.0 + np.exp(-x.astype(np.float64))))


def test_head_silu_of_infinity():
    """An infinite argument of the readout head's SiLU (a bias) stays infinite, with its sign."""
    import paper_2609_32479_amd as tf
    st, sd = torch.ones((40, 64), device="cuda"), torch.zeros((40, 5), dtype=torch.float64, device="cuda")
    for s in (np.inf, -np.inf):
        blob = np.zeros(tf.readout_blob_size(32, 32), np.float32)
        o = 64 + 32 * 64
        blob[o] = s                             # b1[0]
        blob[o + 32:o + 32 + 35 * 32:32] = 1.0  # W2[:, 0]
        _, q = tf.decode_tracks(st, sd, tf.Readout(blob, 32, 32, "fp32"), quantiles=True)
        assert (q == s).all()
