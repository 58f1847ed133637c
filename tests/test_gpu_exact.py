"""What the kernels compute against 64 bits, one layer deep, with the bound that hi + lo activations and fp32 sums give: a kernel that lost the low parts of
one product would pass the parity tolerance and fails here (the first test shows it, on the reference)."""
import numpy as np
import pytest
import torch

import exact
from paper_2504_07878_amd import synth

SEED = 7878
FUSED = dict(n_layers=1, d_model=224, n_q_heads=7, n_kv_heads=1, head_dim=64, d_ffn=3824, vocab=997, router_hidden=0, rope_theta=1e4, dtype=synth.BF16, kv_dtype=synth.F32)
WIDE = dict(FUSED, d_model=928, n_q_heads=5, n_kv_heads=1, head_dim=128, d_ffn=1184, vocab=1000, tie_lm_head=0)
DEEP = dict(WIDE, d_model=1104, d_ffn=6016)       # 7 splits of the FFN output, the last one shorter
HEADS = dict(FUSED, d_model=128, n_q_heads=16, n_kv_heads=8, d_ffn=96, vocab=500, kv_dtype=synth.BF16)

# contexts given, rows of the pass: 208 blocks of rows and kv heads over contexts to 360 (eight wavefronts a block; 128-wide heads four), contexts to 160 (four),
# 928 blocks (two)
SEGMENTS = [(64, [300, 150], [60, 41]), (64, [100, 31], [60, 41]), (64, [200, 33], [290, 171]), (128, [300, 150], [60, 41]), (128, [200, 33], [290, 171])]
# decode steps in one launch: the smallest and the widest rows, both head widths, contexts that leave the keys of a step their weight
ONE_LAUNCH = [("one", HEADS), ("one_896", dict(HEADS, d_model=896, n_q_heads=14, n_kv_heads=2, d_ffn=4864)), ("one_128", dict(HEADS, head_dim=128, n_q_heads=8, n_kv_heads=1))]
ONE_LAUNCH_LENS = [5, 9, 2, 12, 3, 7]
SEGMENTS_REL = 4e-5   # between REL and REL_BF16_CACHE: most keys are given, those of the pass are rounded


def shape(name, kw):
    return synth.TINY.with_(name=name, **kw)


def tokens(s, lens, name):
    return [synth.prompt_tokens(SEED, f"exact.{name}.{i}", n, s.vocab) for i, n in enumerate(lens)]


def step_tokens(s, name, n):
    return [[t] for t in synth.prompt_tokens(SEED, f"exact.step.{name}", n, s.vocab)]


def check(out, ref, what, rel=exact.REL, worst=exact.WORST):
    for field, r in (("hidden", ref[0]), ("logits", ref[1])):
        d, e = exact.distance(getattr(out, field), r)
        print(f"{what} {field}: {d:.2e} of the norm, largest {e:.2e} of the rms")
        assert d < rel and e < worst, (what, field, d, e)


def caches_of(s, lens):
    """Random (k, v) of each length in the cache's type."""
    gen, dt = torch.Generator().manual_seed(SEED), torch.float32 if s.kv_dtype == synth.F32 else torch.bfloat16
    return [tuple(torch.empty((s.n_layers, s.n_kv_heads, n, s.head_dim)).normal_(generator=gen).to(dt) for _ in range(2)) for n in lens]


def given_caches(g, s, lens):
    """Random caches loaded into slots 0, 1, ...; as the reference takes them."""
    caches = caches_of(s, lens)
    for slot, (k, v) in enumerate(caches):
        g.load_kv(slot, k.cuda(), v.cuda())
    return [(k.double(), v.double()) for k, v in caches]


@pytest.mark.parametrize("name,kw", [("fused", FUSED), ("wide", WIDE), ("heads", HEADS)])
def test_the_bound_sees_a_product_without_its_low_parts(name, kw):
    s = shape(name, kw)
    w, segs = exact.weights(s, SEED), tokens(s, [1, 9, 33], name)
    hidden, logits = exact.forward(s, w, segs)
    bound = 2 * exact.REL if s.kv_dtype == synth.F32 else exact.REL_BF16_CACHE
    for p in ("qkv", "o", "gate_up", "down", "head"):
        h, z = exact.forward(s, w, segs, coarse=p)
        assert exact.distance(z, logits)[0] > bound, (p, exact.distance(z, logits))
        assert p == "head" or exact.distance(h, hidden)[0] > bound, (p, exact.distance(h, hidden))


@pytest.mark.parametrize("head_dim,lens,segs", SEGMENTS)
def test_the_bound_sees_attention_without_its_low_parts(head_dim, lens, segs):
    s = shape("heads", dict(HEADS, head_dim=head_dim))
    w, toks, caches = exact.weights(s, SEED), tokens(s, segs, "segments"), [(k.double(), v.double()) for k, v in caches_of(s, lens)]
    hidden, _ = exact.forward(s, w, toks, caches)
    for p in ("q", "p"):
        h, _ = exact.forward(s, w, toks, caches, coarse=p)
        print(p, exact.distance(h, hidden))
        assert exact.distance(h, hidden)[0] > SEGMENTS_REL, (p, exact.distance(h, hidden))


@pytest.mark.parametrize("name,kw", ONE_LAUNCH)
def test_the_bound_sees_a_product_without_its_third_part(name, kw):
    s = shape(name, kw)
    w, toks, caches = exact.weights(s, SEED), step_tokens(s, name, 4), [(k.double(), v.double()) for k, v in caches_of(s, ONE_LAUNCH_LENS[:4])]
    hidden, _ = exact.forward(s, w, toks, caches)
    for p in ("qkv", "q", "p", "o", "gate_up", "down"):
        h, _ = exact.forward(s, w, toks, caches, coarse=p, parts=2)
        print(p, exact.distance(h, hidden))
        assert exact.distance(h, hidden)[0] > 2 * exact.REL_24, (p, exact.distance(h, hidden))
        assert exact.distance(exact.forward(s, w, toks, caches, coarse=p, parts=3)[0], hidden)[0] < exact.REL_24 / 50


@pytest.mark.gpu
@pytest.mark.parametrize("name,kw,lens", [
    ("fused", FUSED, [13] * 64),                    # 832 rows: FFN output in parts
    ("fused", FUSED, [16] * 48 + [31] * 50),        # 2318 rows: gate and up as blocks
    ("fused", FUSED, [40] * 96 + [1] * 4),          # 3844 rows: output projection as blocks
    ("fused", FUSED, [54] * 100),                   # 5400 rows: everything in one piece
    ("wide", WIDE, [11] * 15),                      # 165 rows: two workgroups a sum
    ("wide", WIDE, [27] * 55),                      # 1485 rows: everything in one piece
    ("deep", DEEP, [33] * 5),
    ("deep", DEEP, [50] * 10),
    ("fused_bf16", dict(FUSED, kv_dtype=synth.BF16), [13] * 64),
    ("wide_bf16", dict(WIDE, kv_dtype=synth.BF16), [11] * 15),
    ("heads", HEADS, [45, 1]),                      # attention of blocks of rows: four wavefronts a block
    ("heads", HEADS, [299, 31]),
    ("heads", HEADS, [301, 160]),                   # two
    ("heads_128", dict(HEADS, head_dim=128), [301, 160]),
])
def test_prompts(name, kw, lens):
    from paper_2504_07878_amd import tokroute as tr
    s = shape(name, kw)
    w, segs = exact.weights(s, SEED), tokens(s, lens, name)
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, len(lens), max(320, max(lens)))
    bound = (exact.REL, exact.WORST) if s.kv_dtype == synth.F32 else (exact.REL_BF16_CACHE, exact.WORST_BF16_CACHE)
    check(g.prefill(list(range(len(lens))), segs, want_logits=True).cpu(), exact.forward(s, w, segs), f"{name} {sum(lens)} rows", *bound)


@pytest.mark.gpu
@pytest.mark.parametrize("name,kw,lens", [
    ("fused", FUSED, [1, 40, 33]),                          # kernels of 3 to 8 rows
    ("fused", FUSED, [5, 70, 2, 31, 32, 64, 9, 17]),
    ("wide", WIDE, [1, 40, 33, 8, 64]),
    ("deep", DEEP, [5, 70, 2, 31, 32, 64, 9, 17]),
    ("heads", HEADS, [5, 700, 2, 310, 32, 64, 9, 170]),     # a workgroup a row and kv head
    ("heads_128", dict(HEADS, head_dim=128), [255, 256, 511, 544, 767, 768, 1055, 31]),
    ("fused", FUSED, [1 + 7 * i % 90 for i in range(40)]),  # few-row matrix-core kernels
    ("wide", WIDE, [1 + 7 * i % 90 for i in range(40)]),
    ("wide", WIDE, [7, 50]),                                # streaming kernels
])
def test_steps_over_given_caches(name, kw, lens):
    from paper_2504_07878_amd import tokroute as tr
    s = shape(name, kw)
    w, toks = exact.weights(s, SEED), synth.prompt_tokens(SEED, f"exact.step.{name}", len(lens), s.vocab)
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, max(8, len(lens)), 1100)
    ref = exact.forward(s, w, [[t] for t in toks], given_caches(g, s, lens))
    check(g.decode_step(list(range(len(lens))), toks, want_logits=True).cpu(), ref, f"{name} {len(lens)} rows")


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("name,kw", ONE_LAUNCH)
def test_one_launch_steps(name, kw, rows):
    """All 24 bits of up to 4 rows' activations, 16 of more. (Slots and tokens for which no key or value of the step comes so near the middle between two bf16 values
    that fp32 decides how the cache rounds it: one that goes the other way is 5e-6 and more.)"""
    from paper_2504_07878_amd import tokroute as tr
    s = shape(name, kw)
    w, lens, toks = exact.weights(s, SEED), ONE_LAUNCH_LENS[:rows], step_tokens(s, name, rows)
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, 8, 64)
    ref = exact.forward(s, w, toks, given_caches(g, s, lens))
    out = g.decode_step(list(range(rows)), np.concatenate(toks), want_logits=True).cpu()
    check(out, ref, f"{name} {rows} rows")
    if rows <= 4:
        assert exact.distance(out.hidden, ref[0])[0] < exact.REL_24


@pytest.mark.gpu
@pytest.mark.parametrize("head_dim,kv_page,lens,in_one", [
    # 64-wide heads: up to 12288 cached keys go through one launch (16 parts of a context, three blocks a wavefront; from 4609 on more than 6), 128-wide up to 4096;
    # past that 1 and 2 rows of 64-wide heads take the projection with the attention in it, others the chunked attention
    (64, 0, [12288], True), (64, 0, [12289], False), (64, 64, [12288, 40], True), (64, 64, [4609, 12289], False), (64, 0, [9000, 4609, 12288, 6145], True),
    (64, 64, [9000, 4609, 12289], False), (64, 0, [4609, 12288, 1, 31, 7000, 12000, 8000, 513], True),
    (128, 0, [4096], True), (128, 0, [4097, 1537], False), (128, 64, [1537, 4096], True), (128, 0, [2049, 1537, 33, 4096], True), (128, 0, [2049, 4097, 33], False),
    (128, 64, [1537, 4096, 1, 31, 2500, 4000, 3000, 300], True),
])
def test_steps_over_the_longest_contexts(head_dim, kv_page, lens, in_one):
    from paper_2504_07878_amd import tokroute as tr
    s = shape("longest", dict(HEADS, head_dim=head_dim, n_q_heads=7, n_kv_heads=1))
    w = exact.weights(s, SEED)
    w["l0.wq"] = (w["l0.wq"].float() * 3).bfloat16()   # (few keys have most of the weight, wherever they are)
    toks = step_tokens(s, "longest", len(lens))
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, len(lens), 12352 if head_dim == 64 else 4160, kv_page=kv_page)
    ref = exact.forward(s, w, toks, given_caches(g, s, lens))
    out = g.decode_step(list(range(len(lens))), np.concatenate(toks), want_logits=True).cpu()
    check(out, ref, f"{head_dim} {lens}")
    if in_one and len(lens) <= 4:
        assert exact.distance(out.hidden, ref[0])[0] < 2 * exact.REL_24   # (scores three times as large)


@pytest.mark.gpu
@pytest.mark.parametrize("kv_page", [0, 64])
@pytest.mark.parametrize("head_dim,lens,segs", SEGMENTS)
def test_segments_over_given_caches(head_dim, lens, segs, kv_page):
    """Blocks of rows that share their keys; most keys are given, few of the pass's own are rounded."""
    from paper_2504_07878_amd import tokroute as tr
    s = shape("heads", dict(HEADS, head_dim=head_dim))
    w, toks = exact.weights(s, SEED), tokens(s, segs, "segments")
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, 4, 500, kv_page=kv_page)
    ref = exact.forward(s, w, toks, given_caches(g, s, lens))
    check(g.extend([0, 1], toks, want_logits=True).cpu(), ref, f"segments {head_dim} {segs}", SEGMENTS_REL, 3 * exact.WORST)


@pytest.mark.gpu
@pytest.mark.parametrize("d,vocab,n", [(224, 997, 3), (224, 997, 64), (896, 1031, 65), (96, 2049, 256), (1104, 1000, 40)])
def test_tails(d, vocab, n):
    from paper_2504_07878_amd import tokroute as tr
    s = shape("tail", dict(FUSED, d_model=d, d_ffn=64, vocab=vocab))
    w = exact.weights(s, SEED)
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, n, 32)
    x = torch.from_numpy(synth.hidden_rows(SEED, "exact.tail", n, d, True))
    out = g.tail(x.cuda(), want_logits=True).cpu()
    hn = x.double() / torch.sqrt((x.double() ** 2).mean(-1, keepdim=True) + s.rms_eps) * w["final_norm"].double()
    check(out, (hn.numpy(), (hn @ w["tok_emb"].double().T).numpy()), f"{n} rows")
    conf = torch.softmax(hn @ w["tok_emb"].double().T, -1).max(-1).values.numpy()
    assert np.allclose(out.conf, conf, rtol=1e-3)
