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


@pytest.mark.parametrize("batch", [2, 3, 4])
@pytest.mark.parametrize("hidden,ffn", [(3072, 3072), (3000, 2800), (2048, 4104)])
def test_few_rows_on_matrices_around_the_line(dk, orc, batch, hidden, ffn):
    """Two to four rows of matrices just above and just below 16 MB, K a multiple of the 128 threads' stride or not:
    four weight rows per block above the line, two below.  Bound: that of the other dense parity tests."""
    shape = variant("tiny", n_layers=1, hidden=hidden, n_q_heads=24, n_kv_heads=8, head_dim=128, ffn=ffn, vocab=2003,
                    rope_theta=1e6)
    lay = build_block_tables([40 + 31 * i for i in range(batch)], 16, 2, seed=7)
    pool = W.fill_kv_pool(shape, lay, 8)
    out = run_both(orc, shape, W.make_weights(shape, 9), lay, pool, W.initial_tokens(shape, batch, 10), 2,
                   gpu_flags=dk.STEP_NO_FUSED)
    worst, agree = check_parity(out)
    check_pool(out, pool, shape, lay, 2)
    assert worst < 2e-4 and agree == 1.0
