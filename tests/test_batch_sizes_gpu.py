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
    W = tf.Weights(ts.make_weights(w), w.n_layers, w.d_model, mode, max_hits=64 if w.len_max > 32 else 32)
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


@pytest.mark.parametrize("lens", [(1, 1), (1, 3), (16, 16), (17, 17), (32, 32), (1, 34), (0, 40)])
@pytest.mark.parametrize("name", ["deploy_d128x4_bf16_8m", "mingru2_h64_tiny_d32_fp32"])
def test_tiles_of_any_lengths_match_single_tracks(name, lens):
    """Tiles packed from windows of 64 tracks: one full track a tile, 16 one-hit
    tracks a tile (windows used up within a round), tracks that never share a
    tile, refused tracks in between.  Sampled tracks must give the bits of a call
    of their own; every refused track gives NaN and no other does."""
    w = ts.workload(name)
    n = 9000 if lens[1] <= 3 else 3000
    rng = np.random.default_rng(17)
    lengths = rng.integers(lens[0], lens[1] + 1, n)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    hits = (rng.uniform(-1, 1, (offs[-1], 3)) * [1000, 1000, 3000]).astype(np.float32)
    h, o = torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda()
    call = _call(w)
    whole = call(h, o).cpu()
    good = torch.from_numpy((lengths > 0) & (lengths <= 32))
    assert torch.equal(torch.isfinite(whole).all(dim=1), good)
    assert torch.isnan(whole[~good]).all()
    for i in rng.choice(n, 40, replace=False):
        one = call(h, o[i:i + 2].contiguous()).cpu()
        assert torch.equal(one.isnan(), whole[i:i + 1].isnan()) and torch.equal(one.nan_to_num(), whole[i:i + 1].nan_to_num())
