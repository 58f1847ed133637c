"""A pass over many rows leaves the bits that the same rows leave in passes over few: the block products add the k-steps of a sum in the order of the kernels
they stand in for, however K is dealt to workgroups. (A bf16 cache turns another order into other roundings, and the layers amplify those.)"""
import numpy as np
import pytest
import torch

from paper_2504_07878_amd import synth

pytestmark = pytest.mark.gpu
SEED = 7878
# 928 columns: two splits of K and few blocks, a workgroup a split; the 7B-class width: 4 and 22 splits, several to a workgroup
WIDE = dict(n_layers=2, d_model=928, n_q_heads=5, n_kv_heads=1, head_dim=128, d_ffn=1184, vocab=1000, router_hidden=0, tie_lm_head=0, dtype=synth.BF16, kv_dtype=synth.BF16)
WIDE_7B = dict(WIDE, n_layers=1, d_model=3584, n_q_heads=28, n_kv_heads=4, d_ffn=18944)
WIDE_2048 = dict(WIDE, d_model=2048, n_q_heads=16, n_kv_heads=4, d_ffn=8192)
LONG_K = dict(n_layers=2, d_model=256, n_q_heads=7, n_kv_heads=1, head_dim=64, d_ffn=3104, vocab=1000, router_hidden=0, dtype=synth.BF16, kv_dtype=synth.BF16)


def _weights(s, gen):
    """Drawn on the device: a layer of the 7B-class width takes seconds on the host."""
    def t(*shape, std=0.03, mean=0.0):
        return torch.empty(shape, device="cuda", dtype=torch.bfloat16).normal_(mean, std, generator=gen)

    d, qw, kvw, F = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_ffn
    w = {"tok_emb": t(s.vocab, d), "lm_head": t(s.vocab, d), "final_norm": t(d, std=0.1, mean=1.0)}
    for i in range(s.n_layers):
        w.update({f"l{i}.{k}": v for k, v in dict(
            ln1=t(d, std=0.1, mean=1.0), wq=t(qw, d), wk=t(kvw, d), wv=t(kvw, d), bq=t(qw), bk=t(kvw), bv=t(kvw), wo=t(d, qw), ln2=t(d, std=0.1, mean=1.0),
            wg=t(F, d), wu=t(F, d), wd=t(d, F)).items()})
    return w


def _filled(tr, s, rows, seed):
    """A model whose slots hold contexts of 1 to 31 positions (one block of keys: no attention kernel splits them)."""
    gen = torch.Generator("cuda").manual_seed(seed)
    g = tr.Model(s.asdict(), _weights(s, gen), rows, 40)
    for b in range(rows):
        k, v = (torch.empty((s.n_layers, s.n_kv_heads, 1 + b % 31, s.head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2))
        g.load_kv(b, k, v)
    return g


@pytest.mark.parametrize("name,shape,rows", [("wide", WIDE, 161), ("wide", WIDE, 250), ("wide_2048", WIDE_2048, 97), ("wide_7b", WIDE_7B, 165), ("wide_7b", WIDE_7B, 250)])
def test_wide_step_has_the_bits_of_the_few_row_kernels(name, shape, rows):
    # a step whose rows are selected on the device stays on the few-row kernels for any number of rows
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **shape)
    g = _filled(tr, s, rows, SEED + 3)
    toks = synth.prompt_tokens(SEED, f"order.{name}", rows, s.vocab)
    a = g.decode_step(list(range(rows)), toks, want_logits=True).cpu()
    for b in range(rows):
        g.seq_truncate(b, 1 + b % 31)
    i32 = lambda v: torch.as_tensor(v, dtype=torch.int32, device="cuda")   # noqa: E731
    out = g.outputs(rows, want_logits=True)
    g.decode_step_active(list(range(rows)), i32(np.ones(rows)), i32(toks), rows, i32(np.zeros(2 + rows)), None, out)
    b = out.cpu()
    for f in ("hidden", "logits", "token"):
        assert np.array_equal(getattr(a, f), getattr(b, f)), (f, float(np.abs(getattr(a, f) - getattr(b, f)).max()))


@pytest.mark.parametrize("rows", [832, 1023])
def test_fused_step_has_the_bits_of_smaller_steps(rows):
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="long_k", **LONG_K)
    g = _filled(tr, s, rows, SEED + 4)
    toks = synth.prompt_tokens(SEED, "order.long_k", rows, s.vocab)
    a = g.decode_step(list(range(rows)), toks).cpu()
    for b in range(rows):
        g.seq_truncate(b, 1 + b % 31)
    half = rows // 2
    for lo, hi in ((0, half), (half, rows)):
        b = g.decode_step(list(range(lo, hi)), toks[lo:hi]).cpu()
        assert np.array_equal(a.hidden[lo:hi], b.hidden), float(np.abs(a.hidden[lo:hi] - b.hidden).max())
