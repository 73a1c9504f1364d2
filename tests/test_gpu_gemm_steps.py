"""The matrix-core GEMMs at the edges of their steps over K, of their tables of partial sums and of the rules that choose them."""
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
