"""Decode steps of 9 to 64 rows of a bf16 model in one launch over all layers, against the oracle: groups of 16 rows that are full, short and missing, contexts around the
blocks of 32 keys and the parts of a context, both head widths, widths that fill no task, FFN columns of several rounds, a paged cache; NaNs must end the step; two steps at once."""
import numpy as np
import pytest

import exact
from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878
BASE = dict(n_layers=2, n_q_heads=7, n_kv_heads=1, head_dim=64, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16, d_model=256, d_ffn=704)


def bf16(rng, shape):
    bits = synth.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    return synth.bf16_bits_to_f32(bits), bits


@pytest.mark.parametrize("name,shape,rows,lens,page", [
    ("nine", {}, 9, [0, 1, 31, 32, 33, 255, 256, 257, 767, 768, 769], 0),
    ("sixteen", dict(d_model=896, d_ffn=4864, n_q_heads=14, n_kv_heads=2), 16, [255, 256, 257, 511, 40] * 4, 0),
    ("seventeen", dict(d_ffn=32, n_q_heads=8, n_kv_heads=8), 17, [0, 31, 256, 64, 3] * 4, 32),            # one FFN step; heads of their own keys
    ("narrow", dict(d_model=32, n_q_heads=2, d_ffn=5408), 32, [0, 31, 32, 255] * 8, 0),                    # FFN columns past one round; one step of columns
    ("odd_groups", dict(d_model=896, d_ffn=4864, n_q_heads=14, n_kv_heads=2), 37, [64, 100, 1, 513] * 10, 64),
    ("wide_heads", dict(head_dim=128, n_q_heads=4, n_kv_heads=2, d_ffn=96), 41, [0, 1, 32, 255, 256, 257, 600, 1000] * 6, 0),
    ("heads_of_16_keys", dict(n_q_heads=16, n_kv_heads=16), 20, [769, 1537, 768, 2310, 31] * 5, 0),       # a merge of all 16 heads; of all 8
    ("wide_heads_of_8_keys", dict(head_dim=128, n_q_heads=8, n_kv_heads=8), 49, [257, 256, 769, 1000, 3] * 10, 32),
    ("one_part", {}, 10, [768, 767, 513, 512, 1] * 3, 0),                                                  # the longest contexts of one part, ..
    ("one_part_wide", dict(head_dim=128, n_q_heads=4, n_kv_heads=2), 50, [256, 255, 0, 33] * 13, 64),      # .. of 128-wide heads
    ("all", dict(d_model=480, d_ffn=1120), 64, [1537, 2300] + [5 * i for i in range(62)], 0),
])
def test_steps(name, shape, rows, lens, page):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **{**BASE, **shape})
    w = synth.make_weights(s, SEED + 9, std=0.05, bias_std=0.05, gain_std=0.1)
    n, max_seq = len(lens), max(lens) + 4
    g = tr.Model(s.asdict(), w, n, max_seq, kv_page=page)
    o = tro.Model(s.asdict(), w, n, max_seq)
    rng = synth.rng(SEED, name)
    first = synth.prompt_tokens(SEED, "rows.first", n, s.vocab)
    g.prefill(list(range(n)), [first[i:i + 1] for i in range(n)])
    o.prefill(list(range(n)), [first[i:i + 1] for i in range(n)])
    for i, m in enumerate(lens):
        if m == 0:
            g.seq_truncate(i, 0); o.seq_truncate(i, 0)
            continue
        (kf, kb), (vf, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, m, s.head_dim)) for _ in range(2))
        g.load_kv(i, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype)); o.load_kv(i, kf, vf)
    toks = synth.prompt_tokens(SEED, "rows.tok", n, s.vocab).copy()
    exempt = 0
    for at in (0, 1):
        slots = [(7 * at + i) % n for i in range(rows)]
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{name} rows {slots}")
        np.put(toks, slots, oo.token)   # (the second step attends to what the first has appended)
    assert exempt <= 2


def in_one_launch(model, step):
    """Whether a call ran its layers in one launch; its result."""
    from paper_2504_07878_amd import tokroute as tr
    model.profile_select(tr.KERNEL_FAMILIES.index("layers"))
    model.profile_enable(True)
    out = step()
    n = model.profile_read()[2]
    model.profile_enable(False)
    return n == 1, out


@pytest.mark.parametrize("rows,one", [(2, False), (3, True), (4, True), (8, False), (9, False), (64, False)])
def test_steps_beside_other_streams_keep_a_launch_per_link(rows, one):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="shared", **BASE)
    w = synth.make_weights(s, SEED + 9, std=0.05)
    g, o = tr.Model(s.asdict(), w, 64, 8), tro.Model(s.asdict(), w, 64, 8)
    slots, toks = list(range(rows)), synth.prompt_tokens(SEED, "shared", rows, s.vocab)
    for m in (g, o):
        m.prefill(slots, [toks[i:i + 1] for i in range(rows)])
    exempt = 0
    for shared in (False, True, False):
        g.set_shared(shared)
        assert g.lib.tr_set_shared(g._h, 2) == tr.ERR_INVALID_ARG
        was, go = in_one_launch(g, lambda: g.decode_step(slots, toks, want_logits=True).cpu())
        assert was == (one or not shared)
        exempt += compare_outputs(go, o.decode_step(slots, toks, want_logits=True), s.dtype, s.threshold, f"{rows} rows, shared {shared}")
    assert exempt <= 1


@pytest.mark.parametrize("shape,rows,longest,page", [({}, 64, 3072, 0), (dict(head_dim=128, n_q_heads=4, n_kv_heads=2), 64, 1024, 32), ({}, 16, 12288, 64), ({}, 9, 21504, 0)])
def test_limit_of_parts(shape, rows, longest, page):
    """256 parts of contexts in one launch at most (rows x parts of the longest): a step at the limit, 28 parts of 9 rows among them, and the next one, a launch per link."""
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="limit", **{**BASE, **shape})
    w = synth.make_weights(s, SEED + 9, std=0.05)
    lens = [longest, longest - 1, longest // 2 + 1] + [1 + 37 * i for i in range(rows - 3)]
    g, o = tr.Model(s.asdict(), w, rows, longest + 2, kv_page=page), tro.Model(s.asdict(), w, rows, longest + 2)
    rng = synth.rng(SEED, "limit")
    (kf, kb), (vf, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, longest, s.head_dim)) for _ in range(2))
    for b, m in enumerate(lens):
        g.load_kv(b, *(tr.to_device(np.ascontiguousarray(c[:, :, :m]), s.kv_dtype) for c in (kb, vb)))
        o.load_kv(b, *(np.ascontiguousarray(c[:, :, :m]) for c in (kf, vf)))
    slots, toks = list(range(rows)), synth.prompt_tokens(SEED, "limit", rows, s.vocab)
    exempt = 0
    for one in (True, False):
        was, go = in_one_launch(g, lambda: g.decode_step(slots, toks, want_logits=True).cpu())
        oo = o.decode_step(slots, toks, want_logits=True)
        assert was == one
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{rows} rows after {longest} keys, in one launch: {one}")
        toks = oo.token.copy()
    assert exempt <= 2


@pytest.mark.parametrize("d_model,d_ffn,rows,one", [(256, 10240, 17, True), (256, 10272, 17, False), (512, 10272, 32, True), (512, 10272, 33, False), (512, 15392, 32, False),
                                                    (256, 15360, 16, True), (256, 15392, 16, False), (512, 20480, 9, True), (512, 20512, 9, False)])
def test_wide_ffns_keep_a_launch_per_link(d_model, d_ffn, rows, one):
    """Past two rounds of 5120 FFN columns (one more up to 16 rows, one more up to 32 rows of 512 columns) the FFN output of one launch is slower than a launch per link."""
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="ffn", **{**BASE, **dict(d_model=d_model, d_ffn=d_ffn, n_layers=1)})
    w = synth.make_weights(s, SEED + 9, std=0.05)
    g, o = tr.Model(s.asdict(), w, rows, 8), tro.Model(s.asdict(), w, rows, 8)
    slots, toks = list(range(rows)), synth.prompt_tokens(SEED, "ffn", rows, s.vocab)
    for m in (g, o):
        m.prefill(slots, [toks[i:i + 1] for i in range(rows)])
    was, go = in_one_launch(g, lambda: g.decode_step(slots, toks, want_logits=True).cpu())
    assert was == one
    assert compare_outputs(go, o.decode_step(slots, toks, want_logits=True), s.dtype, s.threshold, f"FFN of {d_ffn}") <= 1


@pytest.mark.parametrize("rows", [9, 64])
def test_nans_end_the_step(rows):
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="nan", **BASE)
    for key in ("tok_emb", "l0.wk", "l0.wo", "l1.wg", "l1.wd", "l0.ln1"):
        w = {k: v.copy() for k, v in synth.make_weights(s, SEED + 9, std=0.05).items()}
        w[key].reshape(-1)[:] = 0xffff   # a negative NaN with every bit set
        m = tr.Model(s.asdict(), w, 64, 64)
        rng = synth.rng(SEED, "nan")
        for b in range(rows):
            (_, kb), (_, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, 33, s.head_dim)) for _ in range(2))
            m.load_kv(b, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype))
        out = m.decode_step(list(range(rows)), np.arange(rows, dtype=np.int32))
        torch.cuda.synchronize()
        assert torch.isnan(out.hidden).all(), key
        m.counters()   # (an error if a wait was given up)


def test_steps_of_two_models_at_the_same_time():
    """Each launch wants every compute unit; neither may depend on having them all."""
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="pair", **{**BASE, **dict(d_model=896, d_ffn=4864, n_q_heads=14, n_kv_heads=2)})
    rng = synth.rng(SEED, "pair")
    (_, kb), (_, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, 900, s.head_dim)) for _ in range(2))
    models = [tr.Model(s.asdict(), synth.make_weights(s, SEED + i, std=0.05), 64, 1000) for i in range(2)]
    for m in models:
        for b in range(64):
            m.load_kv(b, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype))
            m.seq_truncate(b, 900 - 13 * b)
    toks = [np.arange(64, dtype=np.int32), np.arange(20, dtype=np.int32)]
    want, outs = [], [m.outputs(len(t)) for m, t in zip(models, toks)]
    for m, t, o in zip(models, toks, outs):
        m.decode_step(list(range(len(t))), t, o)
        torch.cuda.synchronize()
        want.append(o.hidden.clone())
    streams = [torch.cuda.Stream() for _ in models]
    for _ in range(20):
        for m, t, o, st in zip(models, toks, outs, streams):
            for b in range(len(t)):
                m.seq_truncate(b, 900 - 13 * b)
            with torch.cuda.stream(st):
                m.decode_step(list(range(len(t))), t, o)
    torch.cuda.synchronize()
    for o, h in zip(outs, want):
        assert torch.equal(o.hidden, h)


@pytest.mark.parametrize("rows", [9, 16, 31, 48, 64])
@pytest.mark.parametrize("shape", [dict(d_model=896, n_q_heads=14, n_kv_heads=2, d_ffn=4864), dict(d_model=128, n_q_heads=8, n_kv_heads=8, d_ffn=96, head_dim=128)])
def test_steps_against_64_bits(shape, rows):
    """One layer over given keys. hi + lo activations (exact.REL, exact.WORST); a new key or value that the cache's type rounds the other way weighs at most 1/60 of a row."""
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="exact", **{**BASE, **dict(n_layers=1, vocab=500, router_hidden=0), **shape})
    w = exact.weights(s, SEED)
    lens = [60 + 41 * i % 700 for i in range(rows)]
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, 64, 800)
    gen = torch.Generator().manual_seed(SEED)
    caches = [tuple(torch.empty((1, s.n_kv_heads, n, s.head_dim)).normal_(generator=gen).bfloat16() for _ in range(2)) for n in lens]
    for b, (k, v) in enumerate(caches):
        g.load_kv(b, k.cuda(), v.cuda())
    toks = synth.prompt_tokens(SEED, "rows.exact", rows, s.vocab)
    ref = exact.forward(s, w, [[t] for t in toks], [(k.double(), v.double()) for k, v in caches])
    out = g.decode_step(list(range(rows)), toks, want_logits=True).cpu()
    d, worst = exact.distance(out.hidden, ref[0])
    print(f"{shape['d_model']} columns {rows} rows: {d:.2e} of the norm, largest {worst:.2e} of the rms")
    assert d < exact.REL and worst < exact.WORST


def test_catch_up_rows_over_contexts_in_parts():
    """Segments of two tokens keep the launch of attention by rows whose contexts are split over workgroups: every repetition has the same bits."""
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="parts", **BASE)
    w = synth.make_weights(s, SEED + 9, std=0.05)
    lens = [1990, 800, 1500, 33] + [769 + i for i in range(20)]
    n = len(lens)
    g, o = tr.Model(s.asdict(), w, 64, 2000), tro.Model(s.asdict(), w, n, 2000)
    rng = synth.rng(SEED, "parts")
    (kf, kb), (vf, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, 1990, s.head_dim)) for _ in range(2))
    for b, m in enumerate(lens):
        g.load_kv(b, *(tr.to_device(np.ascontiguousarray(c[:, :, :m]), s.kv_dtype) for c in (kb, vb)))
        o.load_kv(b, *(np.ascontiguousarray(c[:, :, :m]) for c in (kf, vf)))
    segs = [synth.prompt_tokens(SEED, f"parts.{b}", 2, s.vocab) for b in range(n)]
    want, first = o.extend(list(range(n)), segs, want_logits=True), None
    for _ in range(100):
        out = g.extend(list(range(n)), segs, want_logits=True)
        got = out.logits.clone()
        for b, m in enumerate(lens):
            g.seq_truncate(b, m)
        if first is None:
            assert compare_outputs(out.cpu(), want, s.dtype, s.threshold, "parts") <= 1
            first = got
        assert torch.equal(got, first)
