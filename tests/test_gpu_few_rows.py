"""Decode steps of 3 to 8 rows: the kernels that take and leave fp32 rows (fp32 caches, wide models) and, where model and cache allow it, the launch over all
layers, against the oracle, at widths that leave wavefronts with unequal
shares of the reduction dimension or none, for both kinds of model and both cache forms."""
import numpy as np
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878
BASE = dict(n_layers=2, n_q_heads=7, n_kv_heads=1, head_dim=64, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16)


@pytest.mark.parametrize("name,shape,kv_page", [
    ("fused", dict(d_model=224, d_ffn=352), 0),                             # 7 steps of 32 columns: one wavefront without any
    ("fused_paged", dict(d_model=896, n_q_heads=14, n_kv_heads=2, d_ffn=5152), 32),   # FFN columns past one round of steps in flight
    ("fused_224_f32kv", dict(d_model=224, d_ffn=352, kv_dtype=synth.F32), 0),
    ("fused_896_f32kv", dict(d_model=896, n_q_heads=14, n_kv_heads=2, d_ffn=5152, kv_dtype=synth.F32), 0),
    ("fused_f32kv", dict(d_model=480, d_ffn=96, kv_dtype=synth.F32), 0),    # fewer FFN pairs than wavefronts
    ("wide", dict(d_model=1120, n_q_heads=6, head_dim=128, d_ffn=1184), 0),     # 5 steps a wavefront
    ("wide_paged", dict(d_model=2208, n_q_heads=5, head_dim=128, d_ffn=9248), 32),   # 9 steps a wavefront; two units of FFN rows for some workgroups
    ("widest", dict(n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=4, head_dim=128, d_ffn=2080), 0),
])
def test_few_rows(name, shape, kv_page):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **{**BASE, **shape})
    w = synth.make_weights(s, SEED + 5, std=0.04, bias_std=0.05, gain_std=0.1)
    lens = [1, 31, 32, 33, 64, 5, 70, 17]
    g = tr.Model(s.asdict(), w, 8, 96, kv_page=kv_page)
    o = tro.Model(s.asdict(), w, 8, 96)
    prompts = [synth.prompt_tokens(SEED, f"few.{i}", n, s.vocab) for i, n in enumerate(lens)]
    toks = o.prefill(list(range(8)), prompts).token.copy()
    g.prefill(list(range(8)), prompts)
    exempt = 0
    for slots in ([0, 3, 6], [7, 1, 2, 4], [5, 0, 2, 6, 1], list(range(7)), list(range(7, -1, -1))):
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{name} rows {slots}")
        np.put(toks, slots, oo.token)
    assert exempt <= 2
