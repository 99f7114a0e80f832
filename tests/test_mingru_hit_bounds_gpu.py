"""GPU: minGRU offsets that run past the hit array while the workspace has room for
them.  The front end writes no rows for such a track, so every later launch must refuse
it too: NaN end states whatever the workspace holds (NaN bytes, or an earlier call's
rows), and the other tracks' bits unchanged, also where they would have shared a tile."""
import dataclasses

import numpy as np
import pytest

import tracksynth as ts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PAPER16 = "mingru2_h192_fourier15_deploy_bf16_8m"


@pytest.mark.parametrize("name,fused", [("mingru2_h64_tiny_d32_fp32", None), ("mingru2_h192_fourier15_d128_fp32_65k", None),
                                        (PAPER16, False), (PAPER16, True)])
@pytest.mark.parametrize("cut", [0, 2])  # the hits end with a track, or inside one
def test_tracks_past_the_hits_are_refused(name, fused, cut):
    import paper_2609_32479_amd as tf
    print(f"[bounds] {name} fused={fused} cut={cut}", flush=True)
    w = dataclasses.replace(ts.workload(name), len_min=3, len_max=9)
    M = tf.MinGRU(ts.make_mingru_weights(w), w.n_layers, w.d_model, w.hidden, tf.MODE_FOR_WEIGHTS[w.dtype], w.n_features)
    if fused is not None:
        M.set_fused(fused)
    n, good = 6000, 4731
    hits, offs = ts.make_tracks(w, n_tracks=n)
    if w.n_features:
        lo, hi = ts.feature_bounds(w)
        hits = np.random.default_rng(3).uniform(lo, hi, (len(hits), w.n_features)).astype(np.float32)
    h, o = torch.from_numpy(hits).cuda(), torch.from_numpy(offs).cuda()
    ref = M.states(h, o).cpu()
    assert torch.isfinite(ref).all() and M.device_error() == 0
    short = h[:int(offs[good]) + cut].contiguous()

    def check(st, what):
        st = st.cpu()
        assert M.device_error() == tf.DEVERR_BAD_OFFSETS, what
        assert torch.equal(st[:good], ref[:good]), what
        assert torch.isnan(st[good:]).all(), what

    ws = torch.full((M.workspace_bytes(int(offs[-1])),), 0xff, dtype=torch.uint8, device="cuda")
    check(M.states(short, o, workspace=ws), "workspace of NaN")
    out = torch.empty((n, 2 * w.hidden), device="cuda")
    M.states_noalloc(h, o, out)  # rows of an earlier call in the library's array
    assert torch.equal(out.cpu(), ref)
    check(M.states_noalloc(short, o, out), "rows of an earlier call")
