"""GPU: the fp32 models, whose operands run as three bf16 parts, on every width and
tile shape, and with weights whose parts span the exponent range (a gain of 2^40
undone by weights of 2^-40, so that no sum leaves fp32's range), against the fp64
oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
import tracksynth as ts
from tests.parity import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _err(g, r):
    rms = np.sqrt(np.mean(r ** 2, axis=0))
    return float(np.max(np.abs(g - r) / np.maximum(np.abs(r), rms)))


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 40, 2.0 ** -40])
@pytest.mark.parametrize("max_hits", [32, 64])
@pytest.mark.parametrize("d,layers", [(32, 1), (32, 3), (64, 2), (128, 1), (128, 2)])
def test_fp32_widths_match_oracle(d, layers, max_hits, scale):
    import paper_2609_32479_amd as tf
    w = dataclasses.replace(ts.workload("d128x4_fp32_65k"), n_layers=layers, d_model=d, len_min=1,
                            len_max=20 if max_hits == 32 else 64, n_det_layers=64)
    hits, offs = ts.make_tracks(w, n_tracks=300)
    blob = ts.make_weights(n_layers=layers, d=d, dtype="fp32", seed=11)
    o = 0
    for name, shape, _, _ in ts.blob_layout(layers, d):
        n = int(np.prod(shape))
        if name.endswith("norm.g"):
            blob[o:o + n] *= np.float32(scale)
        elif name.endswith("in.W"):
            blob[o:o + n] /= np.float32(scale)
        o += n
    W = tf.Weights(blob, layers, d, "fp32", max_hits=max_hits)
    h, f = torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda()
    g = tf.fit_tracks(h, f, W).cpu().numpy().astype(np.float64)
    r = oracle.fit_tracks(hits, offs, blob, layers, d)
    assert _err(g, r) <= TOL["fp32"]
    assert tf.device_error(W) == 0
