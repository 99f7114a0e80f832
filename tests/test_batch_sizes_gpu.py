"""GPU: batch sizes around the launch rules (one workgroup per track up to one per
compute unit, tiles packed from the workgroup's tracks).  A track's result does not depend on
the batch it comes in, bit for bit, so every batch is compared with the same
tracks in one large call, which the parity tests hold to the oracle."""
import numpy as np
import pytest
import torch

import paper_2609_32479_amd as tf
import tracksynth as ts

pytestmark = pytest.mark.gpu


def _call(w):
    """(tracks -> outputs) of a workload: pooled head, or the minGRU's end states."""
    mode = tf.MODE_FOR_WEIGHTS[w.dtype]
    if w.arch == "mingru":
        M = tf.MinGRU(ts.make_mingru_weights(w), w.n_layers, w.d_model, w.hidden, mode, w.n_features)
        return lambda h, o: M.states(h, o)
    W = tf.Weights(ts.make_weights(w), w.n_layers, w.d_model, mode, max_hits=w.len_max)
    return lambda h, o: tf.fit_tracks(h, o, W)


@pytest.mark.parametrize("name", ["tiny_d32_fp32", "deploy_d128x4_bf16_8m", "long64_d128x4_bf16_200k",
                                  "d256x6_bf16_1m", "mingru2_h192_fourier15_deploy_bf16_8m"])
def test_batch_sizes_match_one_large_call(name):
    w = ts.workload(name)
    n = 3000
    hits, offs = ts.make_tracks(w, n_tracks=n)
    if w.n_features:
        g = np.random.default_rng(5)
        lo, hi = ts.feature_bounds(w)
        hits = g.uniform(lo, hi, (len(hits), w.n_features)).astype(np.float32)
    h, o = torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda()
    call = _call(w)
    whole = call(h, o).cpu()
    assert torch.isfinite(whole).all()
    for first, m in ((0, 1), (7, 2), (0, 13), (100, 255), (3, 256), (11, 257), (500, 1025)):
        part = call(h, o[first:first + m + 1].contiguous()).cpu()
        assert torch.equal(part, whole[first:first + m]), (name, first, m)
