"""Decode attention whose chunks are ordered on the device, from the rows' lengths: every kernel that takes such a
plan, rows without a token, at the ends of blocks and chunks, one long row among short ones, equal rows, a row that
fills its table.  Bound: that of the other decode parity tests, 2e-4, where no row is short; 5e-4 with rows of few tokens
among them."""
import numpy as np
import pytest

import workloads as W
from workloads.blocktable import build_block_tables
from workloads.quant import quantize_weights
from gpu_common import TIE_TOL, run_sampled, check_parity, check_pool_sampled

pytestmark = pytest.mark.gpu


def variant(base, **kw):
    return W.ModelConfig(**{**W.CONFIGS[base].as_dict(), **kw})


def weights_of(shape, base, seed):
    w = W.make_weights(shape, seed)
    return quantize_weights(w) if base == "tiny_q4" else w


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


@pytest.mark.parametrize("lengths", ["equal", "one_long"])
@pytest.mark.parametrize("heads,d,longest", [
    ((4, 4), 64, 1100),
    ((8, 8), 64, 1100),      # two chunks a row, next to each other in the grid's order
    ((8, 4), 64, 1700),
    ((8, 4), 128, 1100),
    ((12, 4), 128, 1700),
    ((16, 2), 64, 1100),
])
def test_order_without_rows_of_few_tokens(orc, heads, d, longest, lengths):
    """The same kernels where no row is short: the bound of the other decode parity tests."""
    batch, steps = 64, 2
    ctx = [longest - 8] * batch if lengths == "equal" else [40 + i for i in range(batch)]
    ctx[21] = longest
    shape = variant("tiny", n_layers=1, hidden=256, ffn=512, vocab=1003, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d,
                    qk_norm=True)
    lay = build_block_tables(ctx, 16, steps, seed=51)
    pool = W.fill_kv_pool(shape, lay, 52)
    rows = [0, 1, 20, 21, 22, 63]
    out = run_sampled(orc, shape, W.make_weights(shape, 53), lay, pool, W.initial_tokens(shape, batch, 54), steps, rows)
    worst, agree = check_parity(out)
    check_pool_sampled(out, pool, shape, lay, steps, rows)
    assert worst < 2e-4 and agree == 1.0, worst


# (base, batch, other sizes, longest): what else takes a plan
OTHERS = [
    ("tiny", 3, dict(hidden=2048, ffn=8192, n_q_heads=32, n_kv_heads=32, head_dim=64), 3000),   # three terms, vector-ALU kernel
    ("tiny", 4, dict(hidden=1024, ffn=2048, n_q_heads=32, n_kv_heads=32, head_dim=64), 2200),
    ("tiny_q4", 16, dict(n_q_heads=16, n_kv_heads=8), 2000),      # 4-bit weights
    ("tiny_moe", 16, dict(n_q_heads=16, n_kv_heads=8), 2000),     # experts
]


@pytest.mark.parametrize("lengths", ["ragged", "one_long"])
@pytest.mark.parametrize("base,batch,sizes,longest", OTHERS)
def test_models_that_take_a_plan(orc, base, batch, sizes, longest, lengths):
    steps = 2
    ctx = [int(x) for x in np.random.default_rng(batch).integers(30, longest, size=batch)] if lengths == "ragged" else [40 + i for i in range(batch)]
    ctx[1] = longest
    shape = variant(base, n_layers=1, qk_norm=True, **sizes)
    lay = build_block_tables(ctx, 16, steps, seed=61)
    pool = W.fill_kv_pool(shape, lay, 62)
    rows = list(range(batch)) if batch < 5 else [0, 1, 2, 7, 15]
    out = run_sampled(orc, shape, weights_of(shape, base, 63), lay, pool, W.initial_tokens(shape, batch, 64), steps, rows,
                      tie_tol=TIE_TOL if base == "tiny_moe" else 0.0)
    worst, agree = check_parity(out)
    check_pool_sampled(out, pool, shape, lay, steps, rows)
    assert worst < 2e-4 and agree == 1.0 and not out["tie_refused"], worst


def plan_words(dec):
    """The plan's word and the first word of its first record: they lie in the float32 attention output, the third
    buffer of the workspace, which a batched step does not write otherwise."""
    import torch
    c = dec.m.shape
    at = dec._ws_ptr - dec.ws.data_ptr()
    for width in (c.hidden, (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim):
        at += (dec.B * width * 4 + 255) // 256 * 256
    return dec.ws[at:at + 4].view(torch.int32).item(), dec.ws[at + 64:at + 68].view(torch.int32).item()


@pytest.mark.parametrize("base,batch,sizes,longest", [
    ("tiny", 64, dict(n_q_heads=4, n_kv_heads=4, head_dim=64), 1100),
    ("tiny", 64, dict(n_q_heads=8, n_kv_heads=4, head_dim=128), 1100),
    ("tiny", 64, dict(n_q_heads=12, n_kv_heads=4, head_dim=128), 1700),
    *OTHERS,
    ("tiny_moe", 16, dict(hidden=512, expert_ffn=768, n_q_heads=16, n_kv_heads=8), 2000),
    ("qwen3_0p6b", 2, dict(n_layers=2, vocab=1000, tie_lm_head=False), 700),     # no plan: the persistent kernel
    ("tiny", 4, {}, 700),                                                        # ... and the vector kernels
    ("tiny", 16, {}, 300),                                                       # ... and short chunks
])
def test_rows_do_not_interact(base, batch, sizes, longest):
    """A row's logits and its appended K/V are the same bits whatever the lengths and tokens of the other rows: long ones,
    short ones, a mixture, all equal (same batch, same table width)."""
    import torch
    import paper_2601_19139_amd as dk
    shape = variant(base, **{"n_layers": 2, "qk_norm": True, **sizes})
    lay = build_block_tables([longest] * batch, 16, 1, seed=71)
    pool = W.fill_kv_pool(shape, lay, 72)
    dm = dk.DeviceModel(shape, weights_of(shape, base, 73))
    takes_plan = longest > 1000
    kept = {0: longest * 5 // 8} if batch < 5 else {0: longest, 1: longest * 5 // 8, 2: 100, batch - 1: longest // 2 + 1}
    rng = np.random.default_rng(75)
    seen = []
    for others in (lambda: longest, lambda: 20, lambda: int(rng.integers(0, longest)), lambda: int(rng.integers(longest // 2, longest))):
        lens = np.array([kept.get(b, others()) for b in range(batch)], dtype=np.int32)
        dkv = dk.DeviceKV(dm, lay, pool)
        tokens = rng.integers(0, shape.vocab, size=batch, dtype=np.int32)
        for b in kept:
            tokens[b] = 7 + b
        dec = dk.Decoder(dm, dkv, lens, tokens)
        dec.step()
        torch.cuda.synchronize()
        assert not takes_plan or plan_words(dec)[0] == 1
        bits = dkv.bits().reshape(pool.shape)
        seen.append([(dec.logits[b].cpu().numpy(), bits[:, lay.tables[b, T // 16], :, :, T % 16]) for b, T in kept.items()])
        dkv.close()
    dm.close()
    for other in seen[1:]:
        for (l0, kv0), (l1, kv1) in zip(seen[0], other):
            assert np.array_equal(l0, l1) and np.array_equal(kv0, kv1)


@pytest.mark.parametrize("heads,length,width,word", [
    (4, 1100, 1104, 0),     # four chunks of 320, the last one short: the grid's order
    (4, 500, 1104, 1),      # two of four
    (4, 1100, 4400, 1),     # one chunk of 1152 in a table of four
    (8, 1100, 1104, 0),     # two chunks of 576, the second nearly whole
    (8, 900, 1104, 1),      # ... and not
])
def test_equal_rows_take_a_plan_only_where_it_orders_something(heads, length, width, word):
    """A plan that is not wanted is not written either: behind its word the workspace is left as it was."""
    import torch
    import paper_2601_19139_amd as dk
    batch = 64
    shape = variant("tiny", n_layers=1, qk_norm=True, n_q_heads=heads, n_kv_heads=heads, head_dim=64)
    lay = build_block_tables([length] * batch, 16, 1, seed=81)
    wide = np.full((batch, width // 16), -1, dtype=np.int32)
    wide[:, :lay.tables.shape[1]] = lay.tables
    lay.tables = wide
    dm = dk.DeviceModel(shape, W.make_weights(shape, 83))
    dkv = dk.DeviceKV(dm, lay, W.fill_kv_pool(shape, lay, 82))
    dec = dk.Decoder(dm, dkv, lay.contexts, W.initial_tokens(shape, batch, 84))
    dec.ws.fill_(0xab)
    dec.step()
    torch.cuda.synchronize()
    got, record = plan_words(dec)
    assert got == word and (record == int(np.uint32(0xabababab).view(np.int32))) == (word == 0), (got, hex(record))
    dkv.close()
    dm.close()


def test_plan_is_made_anew_by_every_replay_of_a_graph():
    """Equal rows that reach their last chunk while a captured step is replayed: the plan of the first replays gives way to
    the grid's order, and tokens and logits are those of eager steps bit for bit."""
    import torch
    import paper_2601_19139_amd as dk
    batch, length, steps = 64, 955, 8                          # chunks of 320: the fourth begins at 960
    shape = variant("tiny", n_layers=2, qk_norm=True, n_q_heads=4, n_kv_heads=4, head_dim=64)
    lay = build_block_tables([length] * batch, 16, 149, seed=91)       # tables of 1104 tokens
    dm = dk.DeviceModel(shape, W.make_weights(shape, 93))
    pool = W.fill_kv_pool(shape, lay, 92)
    flags = dk.STEP_ADVANCE | dk.STEP_NO_FUSED
    seen = []
    for replayed in (False, True):
        dkv = dk.DeviceKV(dm, lay, pool)
        dec = dk.Decoder(dm, dkv, lay.contexts, W.initial_tokens(shape, batch, 94))
        stream, graph, got = torch.cuda.Stream(), torch.cuda.CUDAGraph(), []
        with torch.cuda.stream(stream):
            for step in range(steps):
                if replayed and step == 1:
                    graph.capture_begin()
                    dec.step(flags=flags, stream=stream.cuda_stream)
                    graph.capture_end()
                if replayed and step:
                    graph.replay()
                else:
                    dec.step(flags=flags, stream=stream.cuda_stream)
                stream.synchronize()
                got.append((plan_words(dec)[0], dec.next.cpu().numpy(), dec.logits.cpu().numpy()))
        assert [w for w, _, _ in got] == [1] * 5 + [0] * 3     # lengths 955 to 962
        seen.append(got)
        dkv.close()
    for (_, n0, l0), (_, n1, l1) in zip(*seen):
        assert np.array_equal(n0, n1) and np.array_equal(l0, l1)
    dm.close()
