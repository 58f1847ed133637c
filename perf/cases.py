"""The work that programs built on this library have it do, as measured cases.

A case names a model shape of `paper_2504_07878_amd.synth` (tiny fp32; 0.5B-class bf16 small model with its router;
7B-class bf16 large model), one of the library's calls, and sizes. `prepare` makes what a serving program holds before the
call (weights, context, filled caches, the tokens of the call), `run` makes the call.

Sequence lengths and segment lengths are spread evenly over [lo, hi] and dealt to the slots in an order drawn from the
seed, so that a case's work does not depend on the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_07878_amd import synth, tokroute

DEVICE = "cuda:0"
MAX_BATCH = {"tiny": 4, "slm-0.5b": 64, "llm-7b": 32}   # sequence slots a server keeps
MAX_SEQ = {"tiny": 192, "slm-0.5b": 2048, "llm-7b": 2112}
SPARE = 32          # steps an active-subset loop takes between two looks at the lengths


def listed():
    return [
        # the smallest call: two sequences of the tiny fp32 model, nothing but launches and latency
        dict(name="tiny_decode_2", model="tiny", op="decode", rows=2, lo=33, hi=37, page=0, feed="host"),
        # one user on a device: batch-1 decode after a 256-token prompt
        dict(name="slm_decode_1", model="slm-0.5b", op="decode", rows=1, lo=256, hi=256, page=0, feed="host"),
        # a handful of users, long and short contexts, cache in pages
        dict(name="slm_decode_7_paged", model="slm-0.5b", op="decode", rows=7, lo=100, hi=1900, page=64, feed="host"),
        # a full decode batch with ragged prompts
        dict(name="slm_decode_64", model="slm-0.5b", op="decode", rows=64, lo=128, hi=1024, page=0, feed="host"),
        # time to first token of one request
        dict(name="slm_prefill_1", model="slm-0.5b", op="prefill", rows=1, lo=256, hi=256),
        # a batch of requests arriving together
        dict(name="slm_prefill_64", model="slm-0.5b", op="prefill", rows=64, lo=128, hi=1024),
        # every sequence takes in what the large model produced for it
        dict(name="slm_extend_64", model="slm-0.5b", op="extend", rows=64, lo=128, hi=640, seg_lo=14, seg_hi=14),
        # the routing tail alone on rows from elsewhere
        dict(name="slm_tail_256", model="slm-0.5b", op="tail", rows=256),
        # the large model produces the tokens of the few routed sequences (7 % of 32)
        dict(name="llm_decode_2", model="llm-7b", op="decode", rows=2, lo=2048, hi=2048, page=0, feed="host"),
        # the same with the subset read from flags on the device
        dict(name="llm_active_8", model="llm-7b", op="active", rows=32, flagged=2, n_max=8, lo=2048, hi=2048),
        # sequences routed for the first time: the large model reads their whole prefixes
        dict(name="llm_prefill_4", model="llm-7b", op="prefill", rows=4, lo=64, hi=512),
        # sequences routed again: the large model catches up on the tokens since
        dict(name="llm_extend_3", model="llm-7b", op="extend", rows=3, lo=100, hi=900, seg_lo=5, seg_hi=37),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny_decode", "slm_decode", "slm_decode", "slm_prefill", "slm_extend", "slm_tail", "llm_decode", "llm_active", "llm_prefill", "llm_extend"])
    if kind == "tiny_decode":
        hi = _log(rng, 8, 190)
        return dict(model="tiny", op="decode", rows=rng.randint(1, 4), lo=rng.randint(1, hi), hi=hi, page=0, feed=rng.choice(["host", "device"]))
    if kind == "slm_decode":
        hi = _log(rng, 32, 2000)
        return dict(model="slm-0.5b", op="decode", rows=_log(rng, 1, 64), lo=rng.randint(1, hi), hi=hi, page=rng.choice([0, 0, 64]), feed=rng.choice(["host", "device"]))
    if kind == "slm_prefill":
        hi = _log(rng, 16, 1024)
        return dict(model="slm-0.5b", op="prefill", rows=_log(rng, 1, min(64, 36000 // hi)), lo=rng.randint(max(1, hi // 8), hi), hi=hi)
    if kind == "slm_extend":
        hi, seg = _log(rng, 32, 1500), _log(rng, 1, 32)
        return dict(model="slm-0.5b", op="extend", rows=_log(rng, 1, 64), lo=rng.randint(1, hi), hi=hi, seg_lo=rng.randint(1, seg), seg_hi=seg)
    if kind == "slm_tail":
        return dict(model="slm-0.5b", op="tail", rows=_log(rng, 1, 256))
    if kind == "llm_decode":
        hi = _log(rng, 128, 2048)
        return dict(model="llm-7b", op="decode", rows=rng.randint(1, 8), lo=rng.randint(64, hi), hi=hi, page=0, feed="host")
    if kind == "llm_active":
        hi, n_max = _log(rng, 128, 2048), rng.randint(3, 8)
        return dict(model="llm-7b", op="active", rows=rng.randint(n_max, 32), flagged=rng.randint(1, n_max), n_max=n_max, lo=rng.randint(64, hi), hi=hi)
    if kind == "llm_prefill":
        hi = _log(rng, 32, 512)
        return dict(model="llm-7b", op="prefill", rows=rng.randint(1, 4), lo=rng.randint(hi // 4, hi), hi=hi)
    hi, seg = _log(rng, 64, 1500), _log(rng, 2, 48)
    return dict(model="llm-7b", op="extend", rows=rng.randint(1, 6), lo=rng.randint(32, hi), hi=hi, seg_lo=rng.randint(1, seg), seg_hi=seg)


# ------------------------------------------------------------------ inputs

def _spread(n, lo, hi):
    return [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in range(n)]


def _lengths(case):
    return _spread(case["rows"], case["lo"], case["hi"])


def _segments(case):
    return _spread(case["rows"], case["seg_lo"], case["seg_hi"])


def _weights(s, gen):
    """All weight tensors of a model of shape s as views of one draw: matrices N(0, 0.02^2), gains 1 + N(0, 0.1^2), biases
    N(0, 0.02^2)."""
    d, qw, kvw, F = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_ffn
    shapes = {"tok_emb": (s.vocab, d), "final_norm": (d,)}
    if not s.tie_lm_head:
        shapes["lm_head"] = (s.vocab, d)
    for i in range(s.n_layers):
        shapes.update({f"l{i}.{k}": v for k, v in dict(
            ln1=(d,), wq=(qw, d), wk=(kvw, d), wv=(kvw, d), bq=(qw,), bk=(kvw,), bv=(kvw,), wo=(d, qw), ln2=(d,), wg=(F, d), wu=(F, d), wd=(d, F)).items()})
    if s.router_hidden:
        shapes.update(r_w1=(s.router_hidden, d), r_b1=(s.router_hidden,), r_w2=(s.router_hidden,), r_b2=(1,))
    room = {k: (math.prod(v) + 127) // 128 * 128 for k, v in shapes.items()}
    flat = torch.empty(sum(room.values()), dtype=torch.float32 if s.dtype == tokroute.F32 else torch.bfloat16, device=DEVICE)
    flat.normal_(0.0, 0.02, generator=gen)
    w, at = {}, 0
    for k, shape in shapes.items():
        w[k] = flat[at:at + math.prod(shape)].view(shape)
        at += room[k]
        if k.endswith(("ln1", "ln2", "final_norm")):
            w[k].mul_(5.0).add_(1.0)
    return w


def _fill(model, s, slots, lens, gen):
    """Caches of the given lengths, N(0, 1), as left by earlier calls."""
    dt = torch.float32 if s.kv_dtype == tokroute.F32 else torch.bfloat16
    for slot, n in zip(slots, lens):
        k, v = (torch.empty((s.n_layers, s.n_kv_heads, int(n), s.head_dim), dtype=dt, device=DEVICE).normal_(generator=gen) for _ in range(2))
        model.load_kv(int(slot), k, v)


def prepare(case, seed):
    s = synth.SHAPES[case["model"]].with_(threshold=0.47)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(DEVICE).manual_seed(int(seed))
    op, n = case["op"], case["rows"]
    max_batch, max_seq = (256, 8) if op == "tail" else (MAX_BATCH[s.name], MAX_SEQ[s.name])
    model = tokroute.Model(s.asdict(), _weights(s, gen), max_batch, max_seq, kv_page=case.get("page", 0), device=DEVICE)
    st = {"op": op, "model": model}
    if op == "tail":
        st["x"] = torch.randn((n, s.d_model), dtype=torch.float32, device=DEVICE, generator=gen)
        st["out"] = model.outputs(n)
        return st
    slots = rng.permutation(max_batch)[:n].astype(np.int32)
    lens = rng.permutation(_lengths(case))
    tokens = lambda m: rng.integers(0, s.vocab, size=int(m), dtype=np.int32)   # noqa: E731
    st["slots"] = slots
    st["out"] = model.outputs(case["n_max"] if op == "active" else n)
    if op == "prefill":
        st["prompts"] = [tokens(m) for m in lens]
        return st
    st["back"] = [(int(b), int(m)) for b, m in zip(slots, lens)]   # where a pass starts from
    _fill(model, s, slots, lens, gen)
    if op == "decode":
        st["tokens"] = tokens(n)
        if case["feed"] == "device":
            st["tokens"] = torch.from_numpy(st["tokens"]).to(DEVICE)
            st["op"] = "decode_dev"
    elif op == "extend":
        st["segments"] = [tokens(m) for m in rng.permutation(_segments(case))]
    else:
        flags = np.zeros(n, np.int32)
        flags[rng.permutation(n)[:case["flagged"]]] = 1
        st["flags"], st["tokens"] = torch.from_numpy(flags).to(DEVICE), torch.from_numpy(tokens(n)).to(DEVICE)
        st["active"] = torch.zeros(2 + case["n_max"], dtype=torch.int32, device=DEVICE)
        st["next"] = st["tokens"].clone()
        st["taken"], st["n_max"], st["passes"] = min(case["flagged"], case["n_max"]), case["n_max"], 0
    return st


# ------------------------------------------------------------------ one pass

def _roll_back(st):
    for slot, n in st["back"]:
        st["model"].seq_truncate(slot, n)


def run(st):
    m, op, out = st["model"], st["op"], st["out"]
    if op == "tail":
        m.tail(st["x"], out)
    elif op == "prefill":
        m.prefill(st["slots"], st["prompts"], out)
    elif op == "decode":
        m.decode_step(st["slots"], st["tokens"], out)
        _roll_back(st)      # host bookkeeping only: the next pass decodes at the same contexts
    elif op == "decode_dev":
        m.decode_step_dev(st["slots"], st["tokens"], out)
        _roll_back(st)
    elif op == "extend":
        m.extend(st["slots"], st["segments"], out)
        _roll_back(st)
    else:
        if st["passes"] == SPARE:   # reading the lengths back waits for the steps so far: only now and then
            _roll_back(st)
            st["passes"] = 0
        m.decode_step_active(st["slots"], st["flags"], st["tokens"], st["n_max"], st["active"], st["next"], out)
        st["passes"] += 1
        k = st["taken"]             # rows past the taken ones are padding
        return {"active": st["active"], "next": st["next"], "token": out.token, "conf": out.conf, "score": out.score, "flag": out.flag, "hidden": out.hidden[:k]}
    return {"token": out.token, "conf": out.conf, "score": out.score, "flag": out.flag, "hidden": out.hidden}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    s = synth.SHAPES[case["model"]]
    size, kv_size = (4 if dt == tokroute.F32 else 2 for dt in (s.dtype, s.kv_dtype))
    qw, kvw = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layers = s.n_layers * (2 * qw * s.d_model + 2 * kvw * s.d_model + 3 * s.d_model * s.d_ffn)
    tail = s.vocab * s.d_model + s.router_hidden * (s.d_model + 1)
    op, n = case["op"], case["rows"]
    if op == "tail":
        rows, outs, seen, kept, layers = n, n, 0, 0, 0
    elif op == "prefill":
        lens = _lengths(case)
        rows, outs, kept = sum(lens), n, 0
        seen = sum(m * (m + 1) // 2 for m in lens)
    elif op == "extend":
        lens, segs = _lengths(case), _segments(case)
        rows, outs, kept = sum(segs), n, sum(lens)
        seen = sum(t * a + t * (t + 1) // 2 for a, t in zip(lens, segs))
    else:
        lens = _lengths(case)
        if op == "active":      # the flagged sequences' share of the contexts
            k = min(case["flagged"], case["n_max"])
            kept = sum(lens) * k // n
            rows = outs = k
        else:
            kept, rows, outs = sum(lens), n, n
        seen = kept + rows
    kv_token = 2 * s.n_layers * kvw * kv_size
    nbytes = (layers + tail) * size + (kept + (0 if op == "tail" else rows)) * kv_token + rows * s.d_model * size + outs * (16 + 4 * s.d_model)
    if op == "tail":
        nbytes += n * s.d_model * (4 - size)    # the rows come as fp32
    flops = 2 * (rows * layers + outs * tail) + 4 * s.n_layers * qw * seen
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["model"] == "tiny":     # fp32 throughout
        return {"rel": 2e-5, "differ": 0.01}
    if case["op"] == "tail":        # bf16 weights, fp32 rows carried to about 16 bits
        return {"rel": 1e-4, "differ": 0.01}
    return {"rel": 1e-3, "differ": 0.01}    # the same over all layers, keys and values rounded to bf16 in the cache
