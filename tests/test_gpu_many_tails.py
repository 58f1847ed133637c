"""The routing tail over more than 64 rows: block products with softmax statistics, against the oracle, at row counts and vocabularies that fill
no block exactly, with and without the router's rows behind the vocabulary."""
import numpy as np
import pytest
import torch

from paper_2504_07878_amd import synth
from parity import assert_rows_close

pytestmark = pytest.mark.gpu
SEED = 7878


@pytest.mark.parametrize("d,vocab,hidden,n", [
    (208, 1000, 40, 65),       # one 128-row block; a ragged last tile of the vocabulary, router tiles in the same block
    (896, 33, 40, 129),        # three 64-row blocks; one feature block
    (64, 4096, 0, 200),        # no router; 4 k-steps (fewer than the ring holds)
    (96, 2049, 64, 256),
])
def test_many_tail_rows(d, vocab, hidden, n):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="tails", n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=1, d_ffn=64, vocab=vocab, router_hidden=hidden,
                         dtype=synth.BF16, kv_dtype=synth.BF16)
    w = synth.make_weights(s, SEED + 13, std=0.05, bias_std=0.05, gain_std=0.1)
    g = tr.Model(s.asdict(), w, n, 32)
    x = synth.hidden_rows(SEED, "tails.x", n, d, True)
    go = g.tail(torch.from_numpy(x).cuda(), want_logits=True).cpu()
    exempt = 0
    for i in range(n):
        hn = tro.rmsnorm(x[i], w["final_norm"], s.dtype, s.rms_eps)
        z = tro.linear(w["tok_emb"], None, s.dtype, hn)
        tok, conf = tro.softmax_stats(z)
        assert_rows_close(go.logits[i], z, 2e-2, f"row {i} logits")
        assert go.conf[i] == pytest.approx(conf, rel=2e-2)
        if go.token[i] != tok:
            assert z[tok] - z[go.token[i]] < 1e-3
            exempt += 1
        assert go.token[i] == np.argmax(go.logits[i])       # the lowest index that attains the maximum
        if hidden:
            assert go.score[i] == pytest.approx(tro.router_score(hn, w["r_w1"], w["r_b1"], w["r_w2"], w["r_b2"], s.dtype), abs=2e-3)
            assert go.flag[i] == int(go.score[i] < np.float32(s.threshold))
        else:
            assert go.score[i] == 1.0 and go.flag[i] == 0
    assert exempt <= 2
    g2 = g.tail(torch.from_numpy(x).cuda()).cpu()           # without the logits: the same bits
    assert np.array_equal(g2.token, go.token) and np.array_equal(g2.conf, go.conf) and np.array_equal(g2.score, go.score)
