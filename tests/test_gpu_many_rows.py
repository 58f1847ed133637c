"""Passes over many rows (prompts of many requests at once) against the oracle, at row counts and widths that fill no block exactly, for both kinds of
model (fused and split-K) and both cache forms: narrow fused models on the few-row kernels, wide ones on block products, deep fused ones on both."""
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878

# fused layers: 208 columns (13 k-steps), FFN 336 (a ragged last tile pair), 7 heads in one group; wide: 928 columns, K split in two and more
FUSED = dict(n_layers=2, d_model=208, n_q_heads=7, n_kv_heads=1, head_dim=64, d_ffn=336, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16)
LONG_K = dict(FUSED, d_ffn=1296)     # an FFN output in uneven parts
DEEP = dict(FUSED, n_layers=1, d_model=208, d_ffn=3824)
WIDE = dict(n_layers=2, d_model=928, n_q_heads=5, n_kv_heads=1, head_dim=128, d_ffn=1184, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16)


@pytest.mark.parametrize("name,shape,lens,kv_page", [
    ("long_k", LONG_K, [97] * 8 + [56], 0),         # 832 rows
    ("long_k", LONG_K, [128] * 7 + [127], 32),      # 1023 rows
    ("long_k", LONG_K, [120] * 19 + [24], 0),       # 2304 rows: gate/up as blocks
    ("long_k", LONG_K, [128] * 24, 0),              # 3072 rows
    ("deep", DEEP, [97] * 8 + [56], 0),             # 832 rows: the smallest pass of blocks (FFN output in parts; output projection and gate/up on the others)
    ("deep", DEEP, [127] * 18 + [18], 32),          # 2304 rows: gate/up as blocks
    ("deep", DEEP, [127] * 28 + [28], 0),           # 3584 rows: 112 blocks, the output projection too
    ("deep", DEEP, [127] * 41, 0),                  # 5207 rows: 164 blocks, the FFN output in one piece
    ("fused", FUSED, [97] * 15 + [81], 0),
    ("fused", FUSED, [130] * 15 + [1, 64], 32),     # 2015 rows, paged
    ("fused_f32kv", dict(FUSED, kv_dtype=synth.F32), [111] * 14, 0),
    ("wide", WIDE, [33, 63], 0),
    ("wide", WIDE, [79, 81], 0),                    # 160 rows: 24 blocks of the FFN output, the smallest pass of blocks, parts of K kept apart
    ("wide", WIDE, [100, 1, 120], 32),
    ("wide", WIDE, [127] * 20, 0),                  # whole projections
])
def test_many_rows_in_one_pass(name, shape, lens, kv_page):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **shape)
    w = synth.make_weights(s, SEED + 17, std=0.05, bias_std=0.05, gain_std=0.1)
    B = len(lens)
    g = tr.Model(s.asdict(), w, B, 160, kv_page=kv_page)
    o = tro.Model(s.asdict(), w, B, 160)
    slots = list(range(B))
    prompts = [synth.prompt_tokens(SEED, f"many.{name}.{i}", n, s.vocab) for i, n in enumerate(lens)]
    go, oo = g.prefill(slots, prompts, want_logits=True).cpu(), o.prefill(slots, prompts, want_logits=True)
    exempt = compare_outputs(go, oo, s.dtype, s.threshold, f"{name} prefill")
    toks = oo.token.copy()      # a step over what the pass left in the cache
    go, oo = g.decode_step(slots, toks, want_logits=True).cpu(), o.decode_step(slots, toks, want_logits=True)
    exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{name} step")
    assert exempt <= 2
    assert all(g.seq_len(b) == n + 1 for b, n in enumerate(lens))
