"""Attention of many (row, kv head) pairs over contexts that take a wavefront several trips: the blocks requested ahead, around the ends of
blocks, trips and parts, for both head widths and both cache forms."""
import numpy as np
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878
LENS = [1, 255, 256, 511, 544, 767, 768, 1055]   # a step reads one key more


@pytest.mark.parametrize("head_dim,kv_page", [(64, 0), (64, 32), (128, 0), (128, 64)])
def test_long_rows(head_dim, kv_page):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="long", n_layers=2, d_model=128, n_q_heads=8, n_kv_heads=8, head_dim=head_dim, d_ffn=96, vocab=500, router_hidden=40,
                         dtype=synth.BF16, kv_dtype=synth.BF16)
    w = synth.make_weights(s, SEED + 9, std=0.08, bias_std=0.05, gain_std=0.1)
    B = len(LENS)
    g = tr.Model(s.asdict(), w, B, 1100, kv_page=kv_page)
    o = tro.Model(s.asdict(), w, B, 1100)
    prompts = [synth.prompt_tokens(SEED, f"long.{i}", n, s.vocab) for i, n in enumerate(LENS)]
    toks = o.prefill(list(range(B)), prompts).token.copy()
    g.prefill(list(range(B)), prompts)
    exempt = 0
    for slots in (list(range(B)), list(range(B - 1, -1, -1))):      # 64 pairs: one workgroup each
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"rows {slots}")
        np.put(toks, slots, oo.token)
    # catch-up segments: rows of one sequence side by side
    segs = [synth.prompt_tokens(SEED, f"long.seg.{i}", n, s.vocab) for i, n in enumerate([3, 5])]
    go, oo = g.extend([4, 7], segs, want_logits=True).cpu(), o.extend([4, 7], segs, want_logits=True)
    exempt += compare_outputs(go, oo, s.dtype, s.threshold, "segments")
    assert exempt <= 2
