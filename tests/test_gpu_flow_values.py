"""What a decode step of few rows of a bf16 model (one launch over all layers) makes of values at the ends of their range, against the definition in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2504_07878_amd import synth

pytestmark = pytest.mark.gpu
SEED = 7878
# One layer. Its attention adds nothing (wo = 0), so the FFN sees the embedding: 16 in column 0, zeros elsewhere, whose root mean square over 256 columns is 1 (rms_eps
# = 0). Gate f is 16 wg[f][0], up 16 wu[f][0] = 1, and column 1 + f of the residual row takes h[f]: every SwiGLU value comes out of the call by itself.
GATED = synth.TINY.with_(name="gated", n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=64, d_ffn=256, vocab=64, router_hidden=0, rms_eps=0.0,
                         dtype=synth.BF16, kv_dtype=synth.BF16)


def gated_step(gates, rows, x0=16.0, gain=1.0):
    """rows of hidden (before the final norm) of a decode step whose 255 gates (at a gain of 1) are given (bf16 values)"""
    from paper_2504_07878_amd import tokroute as tr
    s, bf = GATED, lambda *shape: torch.zeros(shape, dtype=torch.bfloat16)   # noqa: E731
    w = {"tok_emb": bf(s.vocab, s.d_model), "final_norm": bf(s.d_model) + 1, "l0.ln1": bf(s.d_model) + gain, "l0.ln2": bf(s.d_model) + gain, "l0.wq": bf(128, s.d_model),
         "l0.wk": bf(64, s.d_model), "l0.wv": bf(64, s.d_model), "l0.wo": bf(s.d_model, 128), "l0.wg": bf(s.d_ffn, s.d_model), "l0.wu": bf(s.d_ffn, s.d_model),
         "l0.wd": bf(s.d_model, s.d_ffn)}
    w["tok_emb"][:, 0] = x0
    w["l0.wg"][:255, 0] = torch.tensor(gates, dtype=torch.float64).bfloat16() / 16
    w["l0.wu"][:, 0] = 1 / 16
    w["l0.wd"][1 + torch.arange(255), torch.arange(255)] = 1
    g = tr.Model(s.asdict(), {k: v.cuda() for k, v in w.items()}, max(rows, 8), 64, hidden_tap=tr.PRE_FINAL_NORM)
    g.prefill(list(range(rows)), [[3, 4]] * rows)
    out = g.decode_step(list(range(rows)), np.arange(rows, dtype=np.int32)).cpu()
    return out.hidden.astype(np.float64)


def bf16_values(lo, hi, n):
    return np.unique(torch.linspace(lo, hi, n, dtype=torch.float64).bfloat16().double().numpy())


def silu(t):
    return t / (1 + np.exp(-t))


@pytest.mark.parametrize("rows", [1, 2, 4, 8, 9, 17, 64])
def test_saturated_gates(rows):
    """exp(-t) of a gate t below -88.7 is infinite in fp32: SwiGLU is -0 there, as in passes of more rows."""
    t = np.resize(np.concatenate([bf16_values(-120, -80, 60), bf16_values(-20, 20, 60), bf16_values(80, 300, 20), [-300, -1e4, -2.0 ** 100, 1e4, 88.5, 0.0]]), 255)
    t = torch.tensor(t).bfloat16().double().numpy()
    with np.errstate(over="ignore"):
        want = silu(t)
    got = gated_step(t, rows)[:, 1:]
    assert np.isfinite(got).all()
    # activations of 8 rows and more are carried to 2^-17; below 1e-30 parts of them may vanish
    assert (np.abs(got - want) <= 1e-5 * np.abs(want) + 1e-30).all(), np.abs(got - want).max()


@pytest.mark.parametrize("lo,hi", [(-20, 0), (-60, -20), (0, 79.75), (79, 90)])   # (from 80 on another form)
@pytest.mark.parametrize("rows", [1, 2, 4])
def test_gates_to_24_bits(rows, lo, hi):
    """Exponential 1 ulp, the sum below the fraction, the division, the product with up and the sum of the parts half a one each: 3 ulp of 1.2e-7."""
    t = np.resize(bf16_values(lo, hi, 400)[:255], 255)
    got, want = gated_step(t, rows)[:, 1:], silu(t)
    off = np.abs(got - want)[:, want != 0] / np.abs(want[want != 0])
    print(f"{rows} rows, gates {lo} to {hi}: mean {off.mean():.1e} largest {off.max():.1e}")
    assert off.max() < 3.6e-7


@pytest.mark.parametrize("rows", [1, 2, 4, 8, 9, 17, 64])
def test_rows_whose_sum_of_squares_overflows(rows):
    """1/rms is 0 then, as in passes of more rows: the row goes through unchanged."""
    got = gated_step(np.linspace(-4, 4, 255), rows, x0=2.0 ** 70)
    want = np.zeros_like(got)
    want[:, 0] = 2.0 ** 70
    assert np.array_equal(got, want), got


@pytest.mark.parametrize("rows", [9, 17, 64])
@pytest.mark.parametrize("x0,gain", [(2.0 ** 64, 1.0), (2.0 ** 70, 2.0 ** 60), (2.0 ** 120, 2.0 ** 8), (-255 * 2.0 ** 120, 3.0)])
def test_rows_whose_values_leave_the_range_with_their_gain(rows, x0, gain):
    """1/rms is 0: neither a value's product with its gain nor a sum of such products may make a NaN of the row."""
    got = gated_step(np.linspace(-400, 400, 255), rows, x0=x0, gain=gain)
    want = np.zeros_like(got)
    want[:, 0] = x0
    assert np.array_equal(got, want), got


@pytest.mark.parametrize("rows", [9, 17, 64])
def test_rows_whose_sum_of_squares_just_fits(rows):
    """The largest value whose square is finite: its row's 1/rms is 2^-60 and the gates are what they always are."""
    t = torch.tensor(np.linspace(-6, 6, 255)).bfloat16().double().numpy()
    got, want = gated_step(t, rows, x0=255 * 2.0 ** 56)[:, 1:], silu(t)
    assert (np.abs(got - want) <= 1e-5 * np.abs(want)).all(), np.abs(got - want).max()


@pytest.mark.parametrize("rows", [1, 2, 4, 8, 9, 17, 64])
def test_values_past_the_context_count_for_nothing(rows):
    """A cache block's places past the row's context hold what an earlier sequence left there, a NaN too."""
    from paper_2504_07878_amd import tokroute as tr
    s = synth.TINY.with_(name="past", n_layers=2, n_q_heads=7, n_kv_heads=1, vocab=1000, router_hidden=40, dtype=synth.BF16, kv_dtype=synth.BF16, d_ffn=704)
    w = synth.make_weights(s, SEED + 9, std=0.05)
    gen = torch.Generator().manual_seed(SEED)
    k, v = (torch.empty((s.n_layers, s.n_kv_heads, 64, s.head_dim)).normal_(generator=gen).bfloat16() for _ in range(2))
    outs = []
    for left in (0.0, float("nan")):
        g = tr.Model(s.asdict(), w, max(rows, 8), 64)
        for b in range(rows):
            n = 33 + 3 * b % 30
            vb = v.clone()
            vb[:, :, n:] = left
            g.load_kv(b, k.cuda(), vb.cuda())
            g.seq_truncate(b, n)
        outs.append(g.decode_step(list(range(rows)), np.arange(rows, dtype=np.int32)).cpu().hidden)
    assert np.isfinite(outs[0]).all() and np.array_equal(*outs)
