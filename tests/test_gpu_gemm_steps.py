"""The matrix-core GEMMs at the edges of their steps over K, of their tables of partial sums and of the rules that choose them."""
import numpy as np
import pytest

import workloads as W
import paper_2601_19139_amd as dk
from workloads.blocktable import build_block_tables
from workloads.quant import quantize_weights
from gpu_common import run_both, run_sampled, check_parity, check_pool, check_pool_sampled

pytestmark = pytest.mark.gpu


def variant(base, **kw):
    return W.ModelConfig(**{**W.CONFIGS[base].as_dict(), **kw})


@pytest.mark.parametrize("hidden,ffn,batch", [
    (136, 120, 5),       # two steps of K for eight waves; 9 sum-of-squares partials
    (136, 120, 16),
    (1288, 1032, 5),     # a last step of 8 columns; 81 partials
    (1288, 1032, 16),
    (1152, 2176, 16),    # 9 and 17 whole steps
    (4104, 512, 16),     # 257 partials
    (8192, 256, 5),      # four waves hold 256 partials in registers: 512, with packed terms
    (8200, 256, 5),      # 513, terms apart; 65 steps, the last of 8 columns
    (8192, 256, 16),     # eight waves (terms apart, K a multiple of 2048) hold 512: all of them ...
    (10240, 256, 16),    # ... and 640, the rest one by one
])
def test_rotated_steps_and_partials(orc, hidden, ffn, batch):
    """Up to 16 rows a block starts at its own step of K and wraps around where the steps are whole: steps that do not
    divide among the waves, fewer steps than waves, a last step that is not whole.  Bound: that of the other dense parity tests."""
    # No short contexts: with an empty one the attention output is the new token's v, and one of its 128 elements
    # rounded to the other bf16 neighbour (2^-8 of it) is 2^-8 / sqrt(128) = 3.5e-4 of the row, above the bound,
    # whatever the order of the sums; among 30 tokens it is a thirtieth of that.
    shape = variant("tiny", n_layers=1, hidden=hidden, ffn=ffn, vocab=1003, qk_norm=True)
    lay = build_block_tables([30 + (29 * i) % 70 for i in range(batch)], 16, 2, seed=11)
    pool = W.fill_kv_pool(shape, lay, 12)
    out = run_both(orc, shape, W.make_weights(shape, 13), lay, pool, W.initial_tokens(shape, batch, 14), 2)
    worst, agree = check_parity(out)
    check_pool(out, pool, shape, lay, 2)
    assert worst < 2e-4 and agree == 1.0


@pytest.mark.parametrize("batch", [3, 4, 5, 8, 9])
@pytest.mark.parametrize("model,hidden,ffn,q4", [
    ("dense", 4096, 4096, False),     # three and four rows: three terms of an activation in one operand; 5..8: two
    ("dense", 1024, 2048, False),     # 4 MB a matrix: the smallest that four rows take so, three stay on the vector kernel
    ("dense", 1024, 1920, False),     # below: four rows stay there too
    ("dense", 384, 8192, False),      # the down projection in K slices across blocks
    ("dense", 256, 9728, False),      # gate/up of 608 row tiles: the shared-activation kernel, one slice of two steps
    ("dense", 2560, 9728, False),     # ... three, of seven and six steps
    ("dense", 392, 1032, False),      # sizes off the 128 grid: terms stay apart
    ("dense", 392, 1024, False),      # ... of the normed rows alone
    ("dense", 1024, 1032, False),     # ... of the MLP's inner rows alone
    ("dense", 1024, 2048, True),
    ("moe", 1024, 768, False),
])
def test_packed_terms(orc, model, hidden, ffn, q4, batch):
    """Up to eight rows the terms of an activation lie side by side in one matrix-core operand: both sides of the row
    counts and sizes at which that begins and ends.  Bound: that of the other parity tests."""
    kw = dict(n_experts=8, top_k=2, expert_ffn=ffn, ffn=0) if model == "moe" else dict(ffn=ffn)
    if ffn == 9728 and batch >= 5:
        assert dk.gemm_plan_query(2, ffn, hidden, batch)[:2] == (4, {256: 1, 2560: 3}[hidden])
    shape = variant("tiny_moe" if model == "moe" else "tiny", n_layers=1, hidden=hidden, vocab=2003, n_q_heads=8,
                    n_kv_heads=4, head_dim=64 if hidden != 4096 else 128, qk_norm=True, **kw)
    lay = build_block_tables([30 + (29 * i) % 70 for i in range(batch)], 16, 2, seed=21)
    weights = W.make_weights(shape, 22)
    if q4:
        weights = quantize_weights(weights)
    pool = W.fill_kv_pool(shape, lay, 23)
    out = run_both(orc, shape, weights, lay, pool, W.initial_tokens(shape, batch, 24), 2)
    worst, agree = check_parity(out)
    check_pool(out, pool, shape, lay, 2)
    assert worst < 2e-4 and agree == 1.0


@pytest.mark.parametrize("hidden,ffn,batch,q4", [
    (1024, 12288, 17, False),    # 768 row tiles in two slices: blocks of six waves, all whole
    (1024, 12288, 64, False),
    (1152, 12160, 48, False),    # 760: a last block of four row tiles, slices of four and five steps
    (1152, 12160, 64, False),
    (4096, 10368, 64, True),     # 648 row tiles
])
def test_gate_up_in_blocks_of_six_waves(orc, hidden, ffn, batch, q4):
    """Six waves share an activation tile that does not divide among them, and sum the partials of eight.  Bound: that
    of the other dense parity tests."""
    assert dk.gemm_plan_query(2, ffn, hidden, batch, q4)[0] == 6
    shape = variant("tiny", n_layers=1, hidden=hidden, ffn=ffn, vocab=1003, qk_norm=True)
    lay = build_block_tables([30 + (29 * i) % 70 for i in range(batch)], 16, 1, seed=31)
    weights, pool = W.make_weights(shape, 32), W.fill_kv_pool(shape, lay, 33)
    if q4:
        weights = quantize_weights(weights)
    rows = sorted({0, batch // 2, batch - 1})
    out = run_sampled(orc, shape, weights, lay, pool, W.initial_tokens(shape, batch, 34), 1, rows)
    worst, agree = check_parity(out)
    check_pool_sampled(out, pool, shape, lay, 1, rows)
    assert worst < 2e-4 and agree == 1.0


@pytest.mark.parametrize("batch", [4, 5, 9, 16])
@pytest.mark.parametrize("hidden,ffn,vocab,q4", [
    (1024, 2048, 4112, False),    # lm_head of 257 row tiles: two per wave, the last block has one
    (1024, 2048, 4112, True),
    (1536, 2048, 8200, False),    # 513: blocks of eight waves in three slices of four steps; terms packed: two per wave
    (2048, 2048, 10007, False),   # 626: three slices of five and six steps
    (2048, 2048, 16381, False),   # 1024: the smallest without slices
])
def test_rules_of_plain_stores(orc, hidden, ffn, vocab, q4, batch):
    """Plain stores up to 16 rows at both ends of their rules on row tiles.  Bound: that of the other dense parity tests.
    (Weights without ties: in the oracle the two largest logits of any row lie 3e-4 of the row's rms apart or more, thirty
    times what the sides differ by; with the seed before, two of them lay 6e-6 apart.)"""
    if batch > 8 and not q4 and vocab > 8192:
        assert dk.gemm_plan_query(0, vocab, hidden, batch)[:2] == (8, 1 if vocab == 16381 else 3)
    shape = variant("tiny", n_layers=1, hidden=hidden, ffn=ffn, vocab=vocab, n_q_heads=8, n_kv_heads=4, head_dim=64, qk_norm=True)
    lay = build_block_tables([30 + (29 * i) % 70 for i in range(batch)], 16, 2, seed=41)
    weights = W.make_weights(shape, 43)
    if q4:
        weights = quantize_weights(weights)
    pool = W.fill_kv_pool(shape, lay, 43)
    out = run_both(orc, shape, weights, lay, pool, W.initial_tokens(shape, batch, 44), 2)
    worst, agree = check_parity(out)
    check_pool(out, pool, shape, lay, 2)
    assert worst < 2e-4 and agree == 1.0


def bf16_terms(x, n):
    """x as the sum of n bf16 numbers, each rounding what the ones before it leave."""
    out = np.zeros_like(x)
    for _ in range(n):
        out += W.f32_from_bf16_bits(W.bf16_bits_from_f32((x - out).astype(np.float32))).astype(np.float64)
    return out


@pytest.mark.parametrize("hidden,ffn,batch", [(1024, 2048, 4), (2048, 8192, 3)])
def test_three_terms_keep_float32(orc, hidden, ffn, batch):
    """Three and four rows on the matrix cores keep every activation as three bf16 terms.  Every matrix selects: the
    output projection, the down projection and the lm_head pass their input on, gate and up rows pick one element each,
    so the logits are the residual stream itself behind attention (a mean of cached v, as the embeddings are zero), the
    output projection, SwiGLU and the down projection, in turn, and an element that lost its third term anywhere shows.

    Bound: the third term of x is what two leave of it, 2^-17 of its binade at most and 2.2e-6 of x in the mean square;
    float32 itself rounds to 2^-24 = 6e-8 some ten times on the way (mean, norm twice, silu, the terms' sums).  8e-7 lies
    between, and the two-term value of each of the four activations alone is checked to lie beyond it."""
    one = W.bf16_bits_from_f32(np.float32(1.0))
    shape = variant("tiny", n_layers=1, hidden=hidden, ffn=ffn, vocab=hidden, n_q_heads=hidden // 128, n_kv_heads=hidden // 256,
                    head_dim=128, qk_norm=False)
    rows = np.arange(ffn)
    pick_a, pick_b = rows % hidden, (7 * rows + 3) % hidden

    def selector(n, k, cols):
        m = np.zeros((n, k), np.uint16)
        m[np.arange(len(cols)), cols] = one
        return m

    eye = selector(hidden, hidden, np.arange(hidden))
    gain = np.full(hidden, one, np.uint16)
    zero = lambda n: np.zeros((n, hidden), np.uint16)
    layer = dict(g_attn=gain, g_mlp=gain, wq=zero(shape.q_dim), wk=zero(shape.kv_dim), wv=zero(shape.kv_dim), wo=eye,
                 w_gate=selector(ffn, hidden, pick_a), w_up=selector(ffn, hidden, pick_b), w_down=selector(hidden, ffn, np.arange(hidden)))
    weights = dict(embed=zero(shape.vocab), lm_head=eye, g_final=gain, layers=[layer])
    lay = build_block_tables([37 + 11 * i for i in range(batch)], 16, 1, seed=51)
    pool = W.fill_kv_pool(shape, lay, 52)

    def reference(**terms):
        t = lambda name, x: bf16_terms(x, 2) if name in terms else x
        norm = lambda x, stored: stored / np.sqrt((x * x).mean(-1, keepdims=True) + shape.rms_eps)
        att = np.empty((batch, shape.n_q_heads, 128))
        for b, n in enumerate(lay.contexts):
            v = np.stack([pool[0, lay.tables[b, p // 16], 1, :, p % 16] for p in range(n)])
            att[b] = np.repeat(W.f32_from_bf16_bits(v).astype(np.float64).sum(0) / (n + 1), 2, axis=0)
        x = t("attention", att.reshape(batch, hidden))
        h = norm(x, t("o", x))
        g, u = h[:, pick_a], h[:, pick_b]
        f = t("swiglu", g / (1 + np.exp(-g)) * u)
        x = x + f[:, :hidden]
        return norm(x, t("down", x))

    want = reference()
    err = lambda got: float((np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)).max())
    for name in ("attention", "o", "swiglu", "down"):
        assert err(reference(**{name: True})) > 8e-7, name
    dm = dk.DeviceModel(shape, weights)
    dkv = dk.DeviceKV(dm, lay, pool)
    dec = dk.Decoder(dm, dkv, lay.contexts.copy().astype(np.int32), np.zeros(batch, np.int32))
    dec.ws.fill_(0x3f)      # a term that nobody writes is 0.75, not the zero that fresh memory may hold
    dec.step()
    got = dec.logits.cpu().numpy().astype(np.float64)
    dkv.close()
    dm.close()
    print(f"hidden {hidden}, {batch} rows: {err(got):.2e}")
    assert err(got) < 8e-7


@pytest.mark.parametrize("hidden,ffn", [(1024, 2048), (4096, 512), (12288, 256)])
def test_sums_of_three_terms(orc, hidden, ffn):
    """A long sum of four rows against float64, the matrix cores (three terms) and the vector kernel (two rows of the same):
    one layer that adds nothing, so the logits are the lm_head's products with normalised embeddings.

    Bound: the matrix cores add a K-step of 128 on their own and the steps in float32, K / 512 of them per wave; with every
    partial sum rounded to 2^-24 of its size a walk of n steps is off by 2^-24 * sqrt(n / 3) of the result in the mean
    square, 1.7e-7 for the 24 of K = 12288.  2.5e-7 leaves the norm's own rounding its share; a single chain through the
    matrix cores measured 3.3e-7 there."""
    shape = variant("tiny", n_layers=1, hidden=hidden, ffn=ffn, vocab=2003, n_q_heads=8, n_kv_heads=4, head_dim=64)
    weights = W.make_weights(shape, 61)
    layer = weights["layers"][0]
    layer["wo"], layer["w_down"] = np.zeros_like(layer["wo"]), np.zeros_like(layer["w_down"])
    f64 = lambda bits: W.f32_from_bf16_bits(bits).astype(np.float64)
    for batch in (4, 2):
        lay = build_block_tables([20 + i for i in range(batch)], 16, 1, seed=62)
        tokens = W.initial_tokens(shape, 4, 63)[:batch]
        x = f64(weights["embed"][tokens])
        want = (x / np.sqrt((x * x).mean(-1, keepdims=True) + shape.rms_eps) * f64(weights["g_final"])) @ f64(weights["lm_head"]).T
        dm = dk.DeviceModel(shape, weights)
        dkv = dk.DeviceKV(dm, lay, W.fill_kv_pool(shape, lay, 64))
        dec = dk.Decoder(dm, dkv, lay.contexts.copy().astype(np.int32), tokens)
        dec.step()
        got = dec.logits.cpu().numpy().astype(np.float64)
        dkv.close()
        dm.close()
        err = float((np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)).max())
        print(f"K {hidden}, {batch} rows: {err:.2e}")
        assert err < 2.5e-7
