"""The 16-bit head's workgroups go on from tile to tile (2048 waves on 256 compute
units: from 65 536 tracks on a second tile, from 131 072 a third, from 196 608 a fourth):
a batch of one to four tiles per wave, ragged at its end, gives each track the bits that a
call of few tiles gives it, and the fp64 oracle's values; also with the weights read
from memory (a head that does not fit in LDS, one tile per wave) and with quantile rows
that are not 16-byte aligned."""
import numpy as np
import pytest

import oracle
from tests.parity import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hidden,n,shift", [(192, 128, 66001, 0), (192, 128, 2017, 1), (32, 32, 70001, 0),
                                              (32, 32, 200003, 1), (192, 128, 200003, 0), (192, 192, 8193, 0),
                                              (64, 224, 8193, 3), (256, 256, 2017, 0), (256, 128, 66001, 2)])
def test_many_tiles_match_few(d, hidden, n, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32479_amd as tf
    print(f"[tiles] d={d} hidden={hidden} n={n} shift={shift}", flush=True)
    rng = np.random.default_rng([d, hidden, n])
    s = 2 * d
    blob = np.concatenate([rng.uniform(0.5, 1.5, s), rng.normal(0, s ** -0.5, hidden * s), rng.uniform(-0.1, 0.1, hidden),
                           rng.normal(0, hidden ** -0.5, 35 * hidden), rng.uniform(-0.1, 0.1, 35)]).astype(np.float32)
    blob = torch.from_numpy(blob).bfloat16().float().numpy()
    R = tf.Readout(blob, d, hidden, "bf16_f16act")
    st = torch.from_numpy(rng.standard_normal((n, s), dtype=np.float32)).cuda()
    sd = torch.from_numpy(rng.uniform(-0.5, 0.5, (n, 5))).cuda()
    qbuf = torch.full((n * 35 + shift + 8,), 7.0, device="cuda")
    q = qbuf[shift:shift + n * 35].view(n, 35)
    out, _ = tf.decode_tracks(st, sd, R, quantiles=True, q=q)
    torch.cuda.synchronize()
    assert (qbuf[:shift] == 7).all() and (qbuf[shift + n * 35:] == 7).all()
    for a, b in ((0, 33), (n // 2 + 5, n // 2 + 300), (3 * n // 4, 3 * n // 4 + 100), (n - 70, n)):
        o1, q1 = tf.decode_tracks(st[a:b].contiguous(), sd[a:b].contiguous(), R, quantiles=True)
        assert torch.equal(o1, out[a:b]) and torch.equal(q1, q[a:b])
    pick = np.unique(np.concatenate([np.arange(40), rng.integers(0, n, 200), np.arange(n - 40, n)]))
    r_q, r_out = oracle.readout_tracks(st.cpu().numpy()[pick].astype(np.float64), sd.cpu().numpy()[pick], blob, d, hidden)
    for g, r in ((q.cpu().numpy()[pick], r_q), (out.cpu().numpy()[pick], r_out)):
        rms = np.sqrt(np.mean(r ** 2, axis=0))
        assert np.max(np.abs(g - r) / np.maximum(np.abs(r), rms)) <= TOL["bf16"]
