"""The branches that choose between wide and narrow accesses, at the sizes where they can go wrong."""
import numpy as np
import pytest

import workloads as W
from workloads.blocktable import build_block_tables
from gpu_common import run_both, check_parity, check_pool

pytestmark = pytest.mark.gpu


def variant(base, **kw):
    return W.ModelConfig(**{**W.CONFIGS[base].as_dict(), **kw})


@pytest.fixture(scope="module")
def dk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2601_19139_amd as dk
    dk.lib()
    return dk


@pytest.fixture(scope="module")
def orc():
    from oracle import oracle_f64
    return oracle_f64()


@pytest.mark.parametrize("batch", [5, 17, 64])
@pytest.mark.parametrize("vocab", [1000, 1001])
@pytest.mark.parametrize("shift", [1, 2])
def test_logits_at_any_float_address(dk, batch, vocab, shift):
    """A matrix-core GEMM writes four logits of a row per store where the vocabulary and the address allow it:
    the same bits come out at an address that allows it and at one that does not, and nothing beside them changes."""
    import torch
    shape = variant("tiny", vocab=vocab)
    lay = build_block_tables([(13 * i) % 40 for i in range(batch)], 16, 1, seed=3)
    dm = dk.DeviceModel(shape, W.make_weights(shape, 4))
    dkv = dk.DeviceKV(dm, lay, W.fill_kv_pool(shape, lay, 5))
    dec = dk.Decoder(dm, dkv, lay.contexts.copy().astype(np.int32), W.initial_tokens(shape, batch, 6))
    dec.step()
    torch.cuda.synchronize()
    want = dec.logits.clone()
    flat = torch.full((batch * vocab + 8,), 7.5, device="cuda")
    assert flat.data_ptr() % 16 == 0
    dec.logits = flat[shift:shift + batch * vocab].view(batch, vocab)
    dec.step()
    torch.cuda.synchronize()
    assert torch.equal(dec.logits, want)
    assert bool((flat[:shift] == 7.5).all()) and bool((flat[shift + batch * vocab:] == 7.5).all())
    dkv.close()
    dm.close()


# One layer of 24 query and 8 kv heads of 128: q/k/v [5120][hidden], output projection [hidden][3072], gate and up
# [ffn][hidden], down [hidden][ffn], lm_head [vocab][hidden].
FEW_ROWS = [
    # hidden, ffn, vocab
    (2048, 4088, 2003),      # gate, up and down 32 KB below 16 MB ...
    (2048, 4096, 2003),      # ... exactly 16 MB ...
    (2048, 4104, 2003),      # ... and 32 KB above
    (3072, 3072, 2003),      # 18 MB each: K is three strides of 128 threads
    (3000, 2800, 2003),      # K ends inside a stride
    (2040, 4120, 2003),      # more than 16 MB, K just below the 2048 ...
    (4104, 2048, 2003),      # ... and just above the 4096 between which a block has 128 threads
    (2456, 512, 2003),       # q/k/v just below the 24 MB of four weight rows per block ...
    (2464, 512, 2003),       # ... and just above
    (3400, 2552, 2003),      # gate/up just below the 2560 weight rows from which three batch rows take four of them ...
    (3400, 2560, 2003),      # ... and on the line
    (2048, 6144, 2003),      # gate/up at four batch rows: the most weight rows that take four per block at 128 threads ...
    (2048, 6152, 2003),      # ... and more
    (5120, 3072, 2003),      # the same at 256 threads ...
    (5120, 3080, 2003),      # ... and more
    (1592, 8192, 2003),      # the down projection, K above 4096, just below its 1600 weight rows ...
    (1600, 8192, 2003),      # ... and on them
    (3072, 512, 4003),       # lm_head of 23 MB: two weight rows per block, two waves in the argmax
    (3072, 512, 12003),      # 70 MB: eight; 128 threads at three and four batch rows
    (4096, 512, 10235),      # 80 MB at K = 4096: four batch rows, below the 10240 weight rows of 128 threads ...
    (4096, 512, 10243),      # ... and above
    (3072, 10928, 2003),     # gate/up and down just above 64 MB; gate/up with 128 threads at three and four batch rows
    (4096, 10240, 2003),     # gate/up at four batch rows with 128 threads, K = 4096
]


@pytest.mark.parametrize("batch", [2, 3, 4])
@pytest.mark.parametrize("hidden,ffn,vocab", FEW_ROWS)
def test_few_rows_on_matrices_around_the_line(dk, orc, batch, hidden, ffn, vocab):
    """Two to four rows: both sides of every line at which the vector kernel's rows per block or threads change, K a
    multiple of a block's stride or not, a last block with fewer weight rows than the others (the odd vocabularies).
    Bound: that of the other dense parity tests."""
    shape = variant("tiny", n_layers=1, hidden=hidden, n_q_heads=24, n_kv_heads=8, head_dim=128, ffn=ffn, vocab=vocab,
                    rope_theta=1e6)
    lay = build_block_tables([40 + 31 * i for i in range(batch)], 16, 2, seed=7)
    pool = W.fill_kv_pool(shape, lay, 8)
    out = run_both(orc, shape, W.make_weights(shape, 9), lay, pool, W.initial_tokens(shape, batch, 10), 2,
                   gpu_flags=dk.STEP_NO_FUSED)
    worst, agree = check_parity(out)
    check_pool(out, pool, shape, lay, 2)
    assert worst < 2e-4 and agree == 1.0
