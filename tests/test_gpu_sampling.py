"""GPU parity of dk_sample_tokens against the oracle's sampler.

The sampled token is an integer decided by float arithmetic (weights, masses,
a running sum against u * total).  The kernel computes in float32 with its own
summation order, the oracle in float64, so the two can differ only where a
decision sits on a boundary up to rounding: a case is compared exactly unless
the oracle's own margins are that small, in which case the kernel's token must
be one that the same rounding of u * total would select."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2601_19139_amd as dk
    dk.lib()
    return dk


def oracle_margins(l, T, top_k, top_p, u):
    """Relative distance of u*total from the nearest running-sum boundary of the kept set, and of
    the top-p requirement from the nearest sorted running mass (float64, sorted formulation)."""
    s = l.astype(np.float64) / T
    p = np.exp(s - s.max())
    ps = np.sort(p)[::-1]
    n = len(p)
    ncand = n if not (0 < top_k < n) else int(np.searchsorted(-ps, -ps[top_k - 1], side="right"))
    tau = ps[ncand - 1] if ncand < n else 0.0
    m_p = 1.0
    if top_p < 1.0:
        cum = np.cumsum(ps[:ncand])
        m_p = float(np.min(np.abs(cum - top_p * cum[-1])) / cum[-1])
        tau = ps[int(np.argmax(cum >= top_p * cum[-1]))]
    kept = np.flatnonzero(p >= tau)
    cum = np.cumsum(p[kept])
    m_u = float(np.min(np.abs(cum - u * cum[-1])) / cum[-1])
    return m_u, m_p, kept


CASES = [
    # V, B, temperature, top_k, top_p
    (1003, 3, 1.0, 0, 1.0),
    (1003, 4, 0.7, 40, 1.0),
    (1003, 4, 1.3, 0, 0.9),
    (5000, 2, 0.9, 50, 0.8),
    (151936, 2, 0.8, 0, 0.95),       # the vocabulary of the 0.6B / 8B shapes
    (151936, 1, 1.0, 20, 1.0),
    (64, 5, 1.0, 1, 1.0),            # top_k = 1: the argmax
    (70, 64, 1.0, 5, 0.8),           # slices of one or two entries, the engine's largest batch
    (151936, 16, 0.8, 50, 0.9),      # a serving batch: few candidates out of a large vocabulary
    (5000, 3, 1.0, 64, 0.5),         # the largest top_k that is found by selection
    (5000, 2, 1.0, 65, 0.9),         # ... and the smallest that is not
    (5000, 2, 1.2, 10, 1.0),         # the 10th largest weight is one of 20 equal ones in two slices
    (5000, 2, 1.2, 10, 0.57),
    (300001, 1, 1.0, 40, 0.9),       # slices too long for the selection path and for the draw's registers
    (300001, 1, 0.9, 0, 1.0),
    (5000, 2, 1.0, 64, 0.5001),      # 63 copies of the largest weight in every 1/64 of the row: ~4000 candidates
    (300, 3, 1e-3, 0, 1.0),          # tiny temperature: the argmax
    (70, 64, 1.0, 0, 0.9),           # the general chain where most slices are empty, at the largest batch
    (5000, 64, 1.0, 100, 0.9),       # both of its searches there
    (16449, 3, 1.1, 0, 0.7),         # a slice one weight longer than the block has threads, the last ones short
]


@pytest.mark.parametrize("V,B,T,top_k,top_p", CASES)
def test_sampler_matches_oracle(dk, orc, V, B, T, top_k, top_p):
    import torch
    rng = np.random.default_rng(V + B + top_k)
    logits = (rng.normal(size=(B, V)) * 2.5).astype(np.float32)
    if V == 1003:
        logits[0, 10:40] = logits[0, 10]                      # a run of equal values
    if V == 5000 and top_p == 0.5001:
        for start in range(0, V, -(-V // 64)):
            logits[1, start:start + 63] = 9.0
    if V == 5000 and top_k == 10:
        logits[0, 70:90] = logits[0].max() + 0.5              # 20 equal largest values: all of them stay
    d_logits = torch.from_numpy(logits).cuda()
    scratch = torch.empty(dk.sample_scratch_bytes(B, V), dtype=torch.uint8, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    seed = 0x1234567890abcdef
    exact = same = 0
    for step in range(12):
        dk.sample_tokens(d_logits, T, top_k, top_p, seed, step, scratch, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        again = torch.empty_like(out)
        dk.sample_tokens(d_logits, T, top_k, top_p, seed, step, scratch, again)
        torch.cuda.synchronize()
        assert np.array_equal(got, again.cpu().numpy())      # repeatable bit for bit
        for b in range(B):
            u = orc.sample_uniform(seed, step, b)
            want = orc.sample(logits[b], T, top_k, top_p, u)
            m_u, m_p, kept = oracle_margins(logits[b], T, top_k, top_p, u)
            same += int(got[b] == want)
            if m_u > 1e-5 and m_p > 1e-5:
                assert got[b] == want, (step, b, got[b], want, m_u, m_p)
                exact += 1
            elif m_p > 1e-5:
                # u * total within rounding of a running-sum boundary: the token must be one that a shift of
                # u * total by that rounding (1e-5 of the total: the worst case of ~340 float32 additions in a
                # row, which is what the kernel's three-level sums amount to) would select.  Between two
                # such tokens there may be any number of candidates of negligible weight.
                assert got[b] in kept, (step, b, got[b], want)
                s64 = logits[b].astype(np.float64) / T
                cum = np.cumsum(np.exp(s64 - s64.max())[kept])
                g = int(np.searchsorted(kept, got[b]))
                r, slack = u * cum[-1], 1e-5 * cum[-1]
                assert (cum[g - 1] if g else 0.0) <= r + slack and cum[g] >= r - slack, (step, b, got[b], want, m_u)
    # With a few thousand candidates the running-sum steps are far wider than float32 rounding and
    # nearly every draw must be decided exactly; with 150 000 candidates a step is ~7e-6 of the
    # total, the size of the rounding itself, so there only "the same or the neighbour" holds.
    if V <= 5000:
        assert exact >= 8 * B
    assert same >= 6 * B, f"only {same} of {12 * B} draws equal the oracle's"


@pytest.mark.parametrize("row,V,top_k,top_p", [
    ("flat", 4096, 0, 0.37),          # every weight the same: all of them in one digit, all tied at the threshold
    ("flat", 1, 0, 0.5),
    ("two_levels", 5000, 0, 0.9),     # the threshold on the upper of two values, the lower ones negligible or not
    ("two_levels", 5000, 700, 0.9),
    ("half_excluded", 3001, 0, 0.8),  # logits of minus infinity: weight zero
    ("half_excluded", 3001, 2000, 0.8),   # ... and fewer others than top_k
    ("ties", 5000, 300, 1.0),         # the 300th largest is one of 500 equal ones
    ("wide", 20000, 0, 0.999),        # weights down to 1e-30: most of them negligible
])
def test_threshold_searches(dk, orc, row, V, top_k, top_p):
    """The searches over whole rows (no small top_k) where digits, ties and negligible weights meet: the kept set must
    be the oracle's, seen through draws at many u."""
    import torch
    rng = np.random.default_rng(V)
    l = rng.normal(size=V).astype(np.float32)
    if row == "flat":
        l[:] = 1.5
    elif row == "two_levels":
        l[:] = np.where(np.arange(V) % 50 == 3, 9.0, -4.0)
    elif row == "half_excluded":
        l[::2] = -np.inf
    elif row == "ties":
        l[100:600] = 2.0
    else:
        l *= 20.0
    B = 16
    d_logits = torch.from_numpy(np.tile(l, (B, 1))).cuda()
    scratch = torch.full((dk.sample_scratch_bytes(B, V),), 255, dtype=torch.uint8, device="cuda")   # nothing cleared before
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    exact = 0
    for step in range(6):
        dk.sample_tokens(d_logits, 1.0, top_k, top_p, 77, step, scratch, out)
        got = out.cpu().numpy()
        for b in range(B):
            u = orc.sample_uniform(77, step, b)
            m_u, m_p, kept = oracle_margins(l, 1.0, top_k, top_p, u)
            assert m_p < 1e-6 or got[b] in kept, (step, b, got[b])
            if m_u > 1e-5 and m_p > 1e-6:
                assert got[b] == orc.sample(l, 1.0, top_k, top_p, u), (step, b, got[b])
                exact += 1
    assert exact >= 4 * B


def test_negligible_weights_that_move_the_nucleus(dk, orc):
    """The largest weight 1, 2000 of 3e-4 to 6e-4, and 18000 just below what counts as negligible: 1, 0.9 and 0.17 in all.
    Without the last ones the nucleus would end more than 100 tokens earlier."""
    import torch
    V, B, top_p = 20000, 16, 0.6
    rng = np.random.default_rng(V)
    w = np.full(V, 0.95 * (1.0 - top_p) / (2 * V))
    w[rng.permutation(V)[:2000]] = np.linspace(3e-4, 6e-4, 2000)
    w[V // 2] = 1.0
    l = np.log(w).astype(np.float32)
    few = np.where(w < (1.0 - top_p) / (2 * V), 0.0, w)
    ends = [int((np.cumsum(np.sort(w)[::-1]) < top_p * x.sum()).sum()) for x in (w, few)]
    assert ends[0] > ends[1] + 100, ends
    d_logits = torch.from_numpy(np.tile(l, (B, 1))).cuda()
    scratch = torch.full((dk.sample_scratch_bytes(B, V),), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    exact = 0
    for step in range(6):
        dk.sample_tokens(d_logits, 1.0, 0, top_p, 77, step, scratch, out)
        got = out.cpu().numpy()
        for b in range(B):
            u = orc.sample_uniform(77, step, b)
            m_u, m_p, kept = oracle_margins(l, 1.0, 0, top_p, u)
            assert m_p < 1e-6 or got[b] in kept, (step, b, got[b])
            if m_u > 1e-5 and m_p > 1e-6:
                assert got[b] == orc.sample(l, 1.0, 0, top_p, u), (step, b, got[b])
                exact += 1
    assert exact >= 4 * B


def test_nan_among_the_logits(dk, orc):
    """A NaN makes the total that the nucleus is a share of a NaN: no threshold reaches it, and every other token stays
    a candidate (the oracle's sums come to the same)."""
    import torch
    V, B, top_p = 5000, 16, 0.3
    l = (np.random.default_rng(8).normal(size=V) * 2.0).astype(np.float32)
    l[[17, 1234, V - 1]] = np.nan
    d_logits = torch.from_numpy(np.tile(l, (B, 1))).cuda()
    scratch = torch.empty(dk.sample_scratch_bytes(B, V), dtype=torch.uint8, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    cum = np.cumsum(np.where(np.isnan(l), 0.0, np.exp(l.astype(np.float64) - np.nanmax(l))))
    exact = 0
    for step in range(6):
        dk.sample_tokens(d_logits, 1.0, 0, top_p, 9, step, scratch, out)
        got = out.cpu().numpy()
        for b in range(B):
            u = orc.sample_uniform(9, step, b)
            if np.min(np.abs(cum - u * cum[-1])) > 1e-5 * cum[-1]:
                assert got[b] == orc.sample(l, 1.0, 0, top_p, u), (step, b, got[b])
                exact += 1
    assert exact >= 4 * B


def test_sampled_distribution_on_device(dk):
    """Many independent draws (one per row and step) follow the softmax probabilities."""
    import torch
    l = np.array([0.0, 1.0, 2.0, -1.0, 0.5, -3.0], dtype=np.float32)
    p = np.exp(l.astype(np.float64))
    p /= p.sum()
    B = 64
    d_logits = torch.from_numpy(np.tile(l, (B, 1))).cuda()
    scratch = torch.empty(dk.sample_scratch_bytes(B, len(l)), dtype=torch.uint8, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    counts = np.zeros(len(l))
    steps = 300
    for step in range(steps):
        dk.sample_tokens(d_logits, 1.0, 0, 1.0, 7, step, scratch, out)
        counts += np.bincount(out.cpu().numpy(), minlength=len(l))
    n = B * steps
    assert np.abs(counts / n - p).max() < 4 * np.sqrt(0.25 / n)


def test_sampler_argument_checks(dk):
    import torch
    d_logits = torch.zeros((2, 100), dtype=torch.float32, device="cuda")
    scratch = torch.empty(dk.sample_scratch_bytes(2, 100), dtype=torch.uint8, device="cuda")
    out = torch.empty(2, dtype=torch.int32, device="cuda")
    for T, k, p in ((0.0, 0, 1.0), (-1.0, 0, 1.0), (1.0, -1, 1.0), (1.0, 0, 0.0), (1.0, 0, 1.5)):
        with pytest.raises(dk.DecodeKitError) as e:
            dk.sample_tokens(d_logits, T, k, p, 1, 0, scratch, out)
        assert e.value.status == "DK_E_INVALID_ARG"
    with pytest.raises(dk.DecodeKitError) as e:
        dk.sample_tokens(d_logits, 1.0, 0, 1.0, 1, 0, scratch[:512], out)
    assert e.value.status == "DK_E_WORKSPACE_TOO_SMALL"
