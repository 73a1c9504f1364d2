"""Decode attention whose contexts are split on the device, from the rows' lengths: every kernel that takes such a
split, rows without a token, at the ends of blocks and chunks, one long row among short ones, equal rows, a row that
fills its table.  Bound: that of the other decode parity tests."""
import numpy as np
import pytest

import workloads as W
from workloads.blocktable import build_block_tables
from gpu_common import run_sampled, check_parity, check_pool_sampled

pytestmark = pytest.mark.gpu


def variant(base, **kw):
    return W.ModelConfig(**{**W.CONFIGS[base].as_dict(), **kw})


EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300]


@pytest.mark.parametrize("lengths", ["ragged", "equal", "one_long"])
@pytest.mark.parametrize("heads,d,longest", [
    ((4, 4), 64, 1100),      # vector-ALU kernel, a head of its own per kv head
    ((8, 4), 64, 1700),      # ... groups of two, chunks too long for the lighter matrix-core variant
    ((8, 4), 128, 1100),     # the lighter variant
    ((12, 4), 128, 1700),    # the matrix-core kernel that requests ahead
    ((16, 2), 64, 1100),     # ... groups of eight
])
def test_split_from_lengths(orc, heads, d, longest, lengths):
    batch, steps = 64, 2
    if lengths == "ragged":
        rng = np.random.default_rng(longest + heads[0])
        ctx = [EDGES[i % len(EDGES)] if i % 2 else int(rng.integers(30, longest)) for i in range(batch)]
    else:
        ctx = [longest - 8] * batch if lengths == "equal" else [40 + i for i in range(batch)]
    ctx[21] = longest
    shape = variant("tiny", n_layers=1, hidden=256, ffn=512, vocab=1003, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d,
                    qk_norm=True)
    lay = build_block_tables(ctx, 16, steps, seed=51)
    pool = W.fill_kv_pool(shape, lay, 52)
    rows = [0, 1, 3, 5, 13, 20, 21, 22, 42, 63]
    out = run_sampled(orc, shape, W.make_weights(shape, 53), lay, pool, W.initial_tokens(shape, batch, 54), steps, rows)
    worst, agree = check_parity(out)
    check_pool_sampled(out, pool, shape, lay, steps, rows)
    # (a row of few tokens whose new v lies on a rounding boundary moves by 2^-8 / sqrt(d) of itself)
    assert worst < 5e-4 and agree == 1.0, worst
