"""Prompts and catch-up segments whose rows share the keys they read: each number of wavefronts a block of rows can be given, at contexts that leave
some of them without keys, that end inside a block of keys, and for last blocks of one to three rows."""
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878


@pytest.mark.parametrize("head_dim,kv_page", [(64, 0), (64, 32), (128, 0), (128, 64)])
@pytest.mark.parametrize("lens,segs", [
    ([45, 1], [47, 3]),         # 104 workgroups: four wavefronts (short contexts)
    ([299, 31], [49, 45]),      # 664, then 200 over contexts to 348: four, then eight (64-wide heads)
    ([301, 160], [1, 50]),      # 928, then 112: two, then eight
])
def test_prompt_blocks(head_dim, kv_page, lens, segs):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="blocks", n_layers=2, d_model=128, n_q_heads=16, n_kv_heads=8, head_dim=head_dim, d_ffn=96, vocab=500, router_hidden=40,
                         dtype=synth.BF16, kv_dtype=synth.BF16)
    w = synth.make_weights(s, SEED + 5, std=0.08, bias_std=0.05, gain_std=0.1)
    g = tr.Model(s.asdict(), w, 4, 400, kv_page=kv_page)
    o = tro.Model(s.asdict(), w, 4, 400)
    slots, exempt = [3, 1], 0
    prompts = [synth.prompt_tokens(SEED, f"blocks.{i}", n, s.vocab) for i, n in enumerate(lens)]
    go, oo = g.prefill(slots, prompts, want_logits=True).cpu(), o.prefill(slots, prompts, want_logits=True)
    exempt += compare_outputs(go, oo, s.dtype, s.threshold, "prompts")
    more = [synth.prompt_tokens(SEED, f"blocks.seg.{i}", n, s.vocab) for i, n in enumerate(segs)]
    go, oo = g.extend(slots, more, want_logits=True).cpu(), o.extend(slots, more, want_logits=True)
    exempt += compare_outputs(go, oo, s.dtype, s.threshold, "segments")
    assert exempt <= 1
