"""A model's forward pass in 64 bits, from its definition alone (plain torch on the CPU), for tests whose bound is the precision that the kernels keep rather
than the parity tolerance: bf16 weights times activations carried as a high and a low bf16 part (16 bits), sums in fp32.

`coarse` names a product (or attention's queries q, weights p) whose activations are cut to their first `parts` bf16 parts (one: rounded to bf16), as if the others
were lost: the distance a test has to be able to see.
"""
import numpy as np
import torch

from paper_2504_07878_amd import synth

# An activation as hi + lo is off by at most 2^-17 of itself, evenly spread: 4.4e-6 rms a product at most (2.5e-6 is what tails show). A layer is four products
# deep on two branches of a residual row, the head one more; sums in fp32, exponentials and roots add 1e-6 or less each. With its low parts gone a product's
# activations are off by 2^-9 at most, 1.1e-3 rms. WORST: the same for the largest of some 1e5 elements, 5 to 6 times the rms.
REL, WORST = 1.5e-5, 9e-5
# Keys and values that the pass itself rounds to a bf16 cache: where an fp32 value lies within its error (4e-6 of itself) of the middle between two bf16 values it
# may go the other way: up to 2^-17 / 2^-9 = 4e-3 of the values by 2^-8, 2.5e-4 rms where a row sees one key, less with every key more.
REL_BF16_CACHE, WORST_BF16_CACHE = 1.5e-4, 1.5e-3
# Three bf16 parts hold an activation's 24 bits: what is left is fp32 arithmetic, about ten roundings of 2^-24 / sqrt(3) = 3.4e-8 rms between a row and its hidden
# row, an exponential and a root, 1.0e-7 to 1.5e-7 as measured. Without its third part a product is off by 2^-17 at most, 7e-7 of the hidden row and more.
REL_24 = 3e-7


def weights(s, seed):
    """name -> bf16 tensor (CPU), drawn as wide as keeps activations of every layer near 1"""
    gen = torch.Generator().manual_seed(seed)
    t = lambda *shape, std, mean=0.0: torch.empty(shape).normal_(mean, std, generator=gen).bfloat16()   # noqa: E731
    d, qw, kvw, F = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_ffn
    w = {"tok_emb": t(s.vocab, d, std=1.0), "final_norm": t(d, std=0.1, mean=1.0)}
    if not s.tie_lm_head:
        w["lm_head"] = t(s.vocab, d, std=d ** -0.5)
    for i in range(s.n_layers):
        w.update({f"l{i}.{k}": v for k, v in dict(
            ln1=t(d, std=0.1, mean=1.0), wq=t(qw, d, std=d ** -0.5), wk=t(kvw, d, std=d ** -0.5), wv=t(kvw, d, std=d ** -0.5), bq=t(qw, std=0.1), bk=t(kvw, std=0.1),
            bv=t(kvw, std=0.1), wo=t(d, qw, std=qw ** -0.5), ln2=t(d, std=0.1, mean=1.0), wg=t(F, d, std=d ** -0.5), wu=t(F, d, std=d ** -0.5),
            wd=t(d, F, std=F ** -0.5)).items()})
    return w


def forward(s, w, segments, caches=None, coarse=None, parts=1):
    """hidden rows (after the final norm) and logits of the last token of each segment, float64 arrays. caches[i] = (k, v) of segment i, float64
    [layer][kv head][position][head_dim], or None."""
    d, Hq, Hkv, dh = s.d_model, s.n_q_heads, s.n_kv_heads, s.head_dim
    lens = [len(t) for t in segments]
    base = [0 if caches is None else c[0].shape[2] for c in (caches or [None] * len(lens))]
    pos = torch.cat([torch.arange(b, b + n) for b, n in zip(base, lens)]).double()
    angle = pos[:, None] * s.rope_theta ** (-2.0 * torch.arange(dh // 2).double() / dh)
    cos, sin = torch.cos(angle)[:, None], torch.sin(angle)[:, None]

    def norm(x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * gain.double()

    def low_lost(name, x):
        if coarse != name:
            return x
        kept, rest = 0, x
        for _ in range(parts):
            p = rest.bfloat16().double()
            kept, rest = kept + p, rest - p
        return kept

    def product(name, x, m):
        return low_lost(name, x) @ m.double().T

    def rotate(u):
        a, b = u[..., :dh // 2], u[..., dh // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def cached(u):
        return u.bfloat16().double() if s.kv_dtype == synth.BF16 else u

    x = w["tok_emb"][torch.from_numpy(np.concatenate(segments)).long()].double()
    for l in range(s.n_layers):
        W = lambda k: w[f"l{l}.{k}"]   # noqa: E731
        n = norm(x, W("ln1"))
        q, k, v = (product("qkv", n, W("w" + c)) + W("b" + c).double() for c in "qkv")
        q, k, v = rotate(q.view(-1, Hq, dh)), cached(rotate(k.view(-1, Hkv, dh))), cached(v.view(-1, Hkv, dh))
        att, at = torch.empty_like(q), 0
        for i, (T, b0) in enumerate(zip(lens, base)):
            r = slice(at, at + T)
            at += T
            K, V = k[r].transpose(0, 1), v[r].transpose(0, 1)
            if b0:
                K, V = torch.cat([caches[i][0][l], K], 1), torch.cat([caches[i][1][l], V], 1)
            past = torch.arange(b0 + T)[None] > (b0 + torch.arange(T))[:, None]
            K, V = K.repeat_interleave(Hq // Hkv, 0), V.repeat_interleave(Hq // Hkv, 0)
            score = (low_lost("q", q[r].transpose(0, 1)) @ K.transpose(1, 2) / dh ** 0.5).masked_fill(past, -float("inf"))
            att[r] = (low_lost("p", torch.softmax(score, -1)) @ V).transpose(0, 1)
        x = x + product("o", att.reshape(-1, Hq * dh), W("wo"))
        n = norm(x, W("ln2"))
        g = product("gate_up", n, W("wg"))
        x = x + product("down", g * torch.sigmoid(g) * product("gate_up", n, W("wu")), W("wd"))
    hidden = norm(x[torch.tensor(np.cumsum(lens) - 1)], w["final_norm"])
    return hidden.numpy(), product("head", hidden, w["tok_emb"] if s.tie_lm_head else w["lm_head"]).numpy()


def distance(a, ref):
    """2-norm of the difference over that of the reference, and the largest difference over the reference's root mean square"""
    e = np.asarray(a, np.float64) - ref
    return float(np.linalg.norm(e) / np.linalg.norm(ref)), float(np.abs(e).max() / np.sqrt((ref * ref).mean()))
