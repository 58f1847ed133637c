"""Small fp32 and bf16 models: the streaming kernels (a head that normalises its own rows, attention that finishes a row in one workgroup) and, up to 4 rows of
fp32 models of up to 32768 words, the launch over all layers, against the oracle at widths, vocabularies and contexts around their limits."""
import numpy as np
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878


@pytest.mark.parametrize("d,vocab,heads,kv_heads,dtype", [
    (64, 17, 1, 1, synth.F32),         # one slice and a wavefront without rows; one head
    (520, 4097, 6, 2, synth.F32),      # a second half of columns of one lane; a slice of one row; three heads a group
    (1024, 20000, 5, 1, synth.F32),    # the widest row; slices of 80 rows; five heads a group
    (1032, 4100, 8, 1, synth.F32),     # one column block too wide: a norm of its own
    (72, 32769, 3, 3, synth.F32),      # one word too many for the launch over all layers: 1 to 4 rows on the streaming kernels
    (256, 28700, 4, 2, synth.BF16),    # slices of the full 128 rows: a norm of its own
    (248, 4099, 4, 2, synth.BF16),
])
def test_small_model_steps(d, vocab, heads, kv_heads, dtype):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="small", d_model=d, vocab=vocab, n_q_heads=heads, n_kv_heads=kv_heads, d_ffn=136, router_hidden=40, dtype=dtype)
    w = synth.make_weights(s, SEED + 3, std=0.05, bias_std=0.05, gain_std=0.1)
    lens = [1, 63, 64, 127, 190, 254, 9, 70, 128]
    g = tr.Model(s.asdict(), w, len(lens), 320)
    o = tro.Model(s.asdict(), w, len(lens), 320)
    prompts = [synth.prompt_tokens(SEED, f"small.{i}", n, vocab) for i, n in enumerate(lens)]
    toks = o.prefill(list(range(9)), prompts).token.copy()
    g.prefill(list(range(9)), prompts)
    # 1 to 4 rows, two groups of rows, more rows than the head normalises itself; the last step passes the four chunks of a workgroup
    for slots in ([0], [1, 5], [2, 3, 4], [6, 7, 8, 0, 1], list(range(9)), [5]):
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        assert compare_outputs(go, oo, s.dtype, s.threshold, f"rows {slots}") <= 1
        np.put(toks, slots, oo.token)
