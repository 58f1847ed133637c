"""Decode steps of 1 to 8 rows of a bf16 model and 1 to 4 rows of an fp32 model in one launch over all layers, against the oracle: contexts around the blocks of 32 keys, the wavefronts of a
workgroup and the parts of a context, both head widths, FFN widths of unequal shares and of several rounds; NaNs that must end the step, not stall it; two models'
steps at the same time on two streams."""
import numpy as np
import pytest

from paper_2504_07878_amd import synth
from parity import compare_outputs

pytestmark = pytest.mark.gpu
SEED = 7878
BASE = dict(n_layers=2, n_q_heads=7, n_kv_heads=1, head_dim=64, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16, d_model=256, d_ffn=704)


def bf16(rng, shape):
    """Values N(0, 1) rounded to bf16, as fp32 and as the bit patterns."""
    bits = synth.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    return synth.bf16_bits_to_f32(bits), bits


@pytest.mark.parametrize("name,shape,lens", [
    # one row class each (1, 2, 3-4, 5-8 rows); cached keys: none, one short of, exactly and one more than a block, a block for every wavefront, a part of 512, 768
    ("one", {}, [0, 1, 31, 32, 33, 255, 256, 257, 767, 768, 769]),
    ("two", dict(d_model=896, d_ffn=4864, n_q_heads=14, n_kv_heads=2), [255, 256, 257, 511, 512, 513, 768, 769]),
    ("four", dict(d_ffn=32, n_q_heads=8, n_kv_heads=8), [0, 31, 256, 769, 1537, 64]),          # one FFN step; more wavefronts than steps; heads of their own keys
    ("eight", dict(d_model=32, n_q_heads=2, d_ffn=5152), [0, 31, 32, 255, 512, 513, 1025, 1100]),   # FFN columns past one round; one step of columns
    ("wide_heads", dict(head_dim=128, n_q_heads=4, n_kv_heads=2, d_ffn=96), [0, 1, 32, 255, 256, 257, 1000, 300]),
])
def test_steps(name, shape, lens):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **{**BASE, **shape})
    w = synth.make_weights(s, SEED + 9, std=0.05, bias_std=0.05, gain_std=0.1)
    rows = {"one": 1, "two": 2, "four": 3, "eight": 7, "wide_heads": 5}[name]
    n, max_seq = len(lens), max(lens) + 4
    g = tr.Model(s.asdict(), w, n, max_seq)
    o = tro.Model(s.asdict(), w, n, max_seq)
    rng = synth.rng(SEED, name)
    first = synth.prompt_tokens(SEED, "flow.first", n, s.vocab)
    g.prefill(list(range(n)), [first[i:i + 1] for i in range(n)])
    o.prefill(list(range(n)), [first[i:i + 1] for i in range(n)])
    for i, m in enumerate(lens):
        if m == 0:
            g.seq_truncate(i, 0); o.seq_truncate(i, 0)
            continue
        (kf, kb), (vf, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, m, s.head_dim)) for _ in range(2))
        g.load_kv(i, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype)); o.load_kv(i, kf, vf)
    toks = synth.prompt_tokens(SEED, "flow.tok", n, s.vocab).copy()
    exempt = 0
    for at in range(n):
        slots = [(at + i) % n for i in range(rows)]
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{name} rows {slots}")
        np.put(toks, slots, oo.token)
        for b in slots:   # the contexts stay where they are
            g.seq_truncate(b, lens[b]); o.seq_truncate(b, lens[b])
    assert exempt <= 2


@pytest.mark.parametrize("rows", [1, 2, 4, 8])
def test_nans_end_the_step(rows):
    """A NaN of any bit pattern in the weights reaches the outputs; words that stand for "not there yet" are never handed on."""
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="nan", **BASE)
    for key in ("l0.wk", "l0.wo", "l1.wg", "l1.wd", "l0.ln1"):
        w = {k: v.copy() for k, v in synth.make_weights(s, SEED + 9, std=0.05).items()}
        w[key].reshape(-1)[:] = 0xffff   # a negative NaN with every bit set
        m = tr.Model(s.asdict(), w, 8, 64)
        rng = synth.rng(SEED, "nan")
        for b in range(rows):
            (_, kb), (_, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, 33, s.head_dim)) for _ in range(2))
            m.load_kv(b, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype))
        out = m.decode_step(list(range(rows)), np.arange(rows, dtype=np.int32))
        torch.cuda.synchronize()
        assert torch.isnan(out.hidden).all(), key
        m.counters()   # (an error if a wait was given up: the words of a step that was are NaNs too)


def test_steps_of_two_models_at_the_same_time():
    """Each launch wants every compute unit; neither may depend on having them all."""
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="pair", **{**BASE, **dict(d_model=896, d_ffn=4864, n_q_heads=14, n_kv_heads=2)})
    rng = synth.rng(SEED, "pair")
    (_, kb), (_, vb) = (bf16(rng, (s.n_layers, s.n_kv_heads, 600, s.head_dim)) for _ in range(2))
    models = [tr.Model(s.asdict(), synth.make_weights(s, SEED + i, std=0.05), 8, 700) for i in range(2)]
    for m in models:
        for b in range(8):
            m.load_kv(b, tr.to_device(kb, s.kv_dtype), tr.to_device(vb, s.kv_dtype))
    toks = [np.arange(8, dtype=np.int32), np.arange(2, dtype=np.int32)]
    want, outs = [], [m.outputs(len(t)) for m, t in zip(models, toks)]
    for m, t, o in zip(models, toks, outs):
        m.decode_step(list(range(len(t))), t, o)
        torch.cuda.synchronize()
        want.append(o.hidden.clone())
    streams = [torch.cuda.Stream() for _ in models]
    for _ in range(20):
        for m, t, o, st in zip(models, toks, outs, streams):
            for b in range(len(t)):
                m.seq_truncate(b, 600)
            with torch.cuda.stream(st):
                m.decode_step(list(range(len(t))), t, o)
    torch.cuda.synchronize()
    for o, h in zip(outs, want):
        assert torch.equal(o.hidden, h)


F32 = dict(n_layers=2, n_q_heads=4, n_kv_heads=2, head_dim=64, vocab=1000, router_hidden=40, dtype=synth.F32, kv_dtype=synth.F32, d_model=256, d_ffn=1024)


@pytest.mark.parametrize("name,shape,rows,lens,options", [
    # both widths of a row, 1 to 8 wavefronts that share the FFN's columns, columns and vocabularies that fill no task; cached keys around a step of all wavefronts (32
    # keys, 16 of wide heads), a round (256, 128) and the longest (2047, 1023 and the new one)
    ("narrow", {}, 2, [0, 1, 31, 32, 33, 255, 256, 257], {}),
    ("one", dict(d_model=200, d_ffn=24, vocab=33, router_hidden=0), 1, [3, 600, 64], {}),
    ("short", dict(d_model=40, d_ffn=2048, n_q_heads=1, n_kv_heads=1, vocab=31), 3, [0, 63, 511, 2047, 2048], {}),
    ("wide", dict(d_model=1024, d_ffn=8192, n_q_heads=8, n_kv_heads=8, head_dim=128, vocab=4100), 4, [0, 127, 128, 129, 1023, 1024], {}),
    ("tapped", dict(d_model=264, d_ffn=4104, head_dim=128, vocab=65), 2, [15, 17, 1022], dict(hidden_tap=1)),
])
def test_steps_of_fp32_models(name, shape, rows, lens, options):
    from oracle import tro
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name=name, **{**F32, **shape})
    w = synth.make_weights(s, SEED + 9, std=0.05, bias_std=0.05, gain_std=0.1)
    n, max_seq = len(lens), (max(lens) + 4 + 63) // 64 * 64
    g = tr.Model(s.asdict(), w, n, max_seq, **options)
    o = tro.Model(s.asdict(), w, n, max_seq, hidden_tap=options.get("hidden_tap", 0))
    rng = synth.rng(SEED, name)
    first = synth.prompt_tokens(SEED, "flow.first", n, s.vocab)
    for m in (g, o):
        m.prefill(list(range(n)), [first[i:i + 1] for i in range(n)])
    for i, m in enumerate(lens):
        if m == 0:
            g.seq_truncate(i, 0); o.seq_truncate(i, 0)
            continue
        k, v = (rng.standard_normal((s.n_layers, s.n_kv_heads, m, s.head_dim), dtype=np.float32) for _ in range(2))
        g.load_kv(i, tr.to_device(k, s.kv_dtype), tr.to_device(v, s.kv_dtype)); o.load_kv(i, k, v)
    toks = synth.prompt_tokens(SEED, "flow.tok", n, s.vocab).copy()
    exempt = 0
    for at in range(n):
        slots = [(at + i) % n for i in range(rows)]
        go = g.decode_step(slots, toks[slots], want_logits=True).cpu()
        oo = o.decode_step(slots, toks[slots], want_logits=True)
        exempt += compare_outputs(go, oo, s.dtype, s.threshold, f"{name} rows {slots}")
        np.put(toks, slots, oo.token)
        for b in slots:
            g.seq_truncate(b, lens[b]); o.seq_truncate(b, lens[b])
    assert exempt <= 2


def test_nans_end_the_step_of_an_fp32_model():
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="nan32", **F32)
    for key in ("tok_emb", "l0.wk", "l0.wo", "l1.wg", "l1.wd", "l0.ln1"):
        w = {k: v.copy() for k, v in synth.make_weights(s, SEED + 9, std=0.05).items()}
        w[key].view(np.uint32).reshape(-1)[:] = 0xffffffff
        m = tr.Model(s.asdict(), w, 8, 64)
        rng = synth.rng(SEED, "nan")
        for b in range(2):
            k, v = (rng.standard_normal((s.n_layers, s.n_kv_heads, 33, s.head_dim), dtype=np.float32) for _ in range(2))
            m.load_kv(b, tr.to_device(k, s.kv_dtype), tr.to_device(v, s.kv_dtype))
        out = m.decode_step([0, 1], np.arange(2, dtype=np.int32))
        torch.cuda.synchronize()
        assert torch.isnan(out.hidden).all(), key
        m.counters()   # (an error if a wait was given up: the words of a step that was are NaNs too)


def given_up_word(m):
    """The word behind the counters, as the header describes it."""
    import ctypes
    p = ctypes.c_void_p()
    m._check(m.lib.tr_counters_ptr(m._h, ctypes.byref(p)), "tr_counters_ptr")
    off = p.value - m.workspace.data_ptr() + m.cfg.max_batch * 16
    return m.workspace[off:off + 4]


@pytest.mark.parametrize("shape", [BASE, F32], ids=["bf16", "fp32"])
def test_a_step_that_was_given_up_is_reported(shape):
    """The word is set from the host, as a wait that ends without its input would: the steps and prompts from then on say so, whatever kernels they take."""
    from paper_2504_07878_amd import tokroute as tr
    import torch
    s = synth.TINY.with_(name="given-up", **shape)
    m = tr.Model(s.asdict(), synth.make_weights(s, SEED + 9, std=0.05), 16, 64)
    prompts = [[1, 2, 3]] * 12
    m.prefill(list(range(12)), prompts)
    out = m.decode_step([0, 1], [4, 5]).cpu()
    assert (out.token >= 0).all() and (out.conf > 0).all() and m.counters()[0, 0] == 2
    assert int(given_up_word(m).view(torch.int32)) == 0
    given_up_word(m).view(torch.int32).fill_(1)
    for out in (m.decode_step([0, 1], [4, 5]), m.decode_step(list(range(9)), [4] * 9), m.decode_step_dev([3], torch.full((1,), 4, dtype=torch.int32, device="cuda")),
                m.extend([0, 1], [[1], [2]]), m.extend([0, 1], [[1], [2, 3]]), m.prefill([0], prompts[:1])):
        o = out.cpu()
        assert (o.token == -1).all() and not o.conf.any() and not o.score.any() and not o.flag.any()
    x = torch.randn((2, s.d_model), device="cuda")
    assert (m.tail(x).cpu().token >= 0).all()   # touches no cache
    with pytest.raises(tr.TokrouteError) as e:
        m.counters()
    assert e.value.code == tr.ERR_HIP
    if s.dtype == synth.BF16:   # lengths that only the device knows
        n, one = 3, torch.ones(3, dtype=torch.int32, device="cuda")
        o = m.decode_step_active([4, 5, 6], one, one, n, torch.zeros(2 + n, dtype=torch.int32, device="cuda")).cpu()
        assert (o.token == -1).all()
        with pytest.raises(tr.TokrouteError) as e:
            m.seq_len(4)
        assert e.value.code == tr.ERR_HIP
    given_up_word(m).view(torch.int32).fill_(0)   # (nothing was counted meanwhile)
    assert m.counters()[1, 0] == 2 and m.counters()[3, 0] == 1
