"""Passes of several groups of 64 rows against the oracle: ranges of one to many weight tiles, 1 to 14 k-steps of a wavefront, FFN widths that leave a tile pair
partly empty, row counts around the groups, and work that does not divide by the 8 parts it is dealt in."""
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878


@pytest.mark.parametrize("d_model,d_ffn,lens", [
    (32, 48, [65]),                 # one k-step of two wavefronts; one and a half tile pairs
    (144, 1040, [63, 66]),          # 9 k-steps for four wavefronts; 33 pairs
    (256, 704, [100, 1, 92]),       # 4 of a wavefront
    (256, 704, [448]),              # FFN output: one tile a range, 6 k-steps of a wavefront in two splits
    (256, 704, [200, 440]),         # the same in one split, 11
    (512, 2048, [129, 128]),        # 8; 5 groups
    (896, 4864, [70, 300]),         # 14; 6 groups
    (896, 4880, [831]),             # the most rows that come this way; 13 groups
])
def test_prompts(d_model, d_ffn, lens):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="groups", n_layers=2, d_model=d_model, d_ffn=d_ffn, n_q_heads=7, n_kv_heads=1, vocab=512, router_hidden=40, dtype=synth.BF16,
                         kv_dtype=synth.BF16)
    w = synth.make_weights(s, SEED + 9, std=0.05, bias_std=0.05, gain_std=0.1)
    n = len(lens)
    prompts = [synth.prompt_tokens(SEED, f"groups.{i}", m, s.vocab) for i, m in enumerate(lens)]
    g, o = tr.Model(s.asdict(), w, n, max(lens) + 1), tro.Model(s.asdict(), w, n, max(lens) + 1)
    go, oo = g.prefill(list(range(n)), prompts, want_logits=True).cpu(), o.prefill(list(range(n)), prompts, want_logits=True)
    assert compare_outputs(go, oo, s.dtype, s.threshold, f"{d_model} {d_ffn} {lens}") <= 1
