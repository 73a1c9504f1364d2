"""Workloads of the decode-step library, for measuring it: what a serving program has it do, from a single
sampled row to 16 long sequences of the 8B shape.

A case is a dict of plain values; `kind` says which path it takes:

  decode   one batched decode step (dk_decode_step) over ragged sequences that may share a cached prefix
  prefill  one prompt turned into KV state in chunks (dk_prefill_chunk), behind `start` cached tokens
  sample   one token drawn per row from given logits (dk_sample_tokens)
  serve    a whole run of the scheduler with its prefix cache (dk_engine_*): requests submitted, run to the end

Model shapes are those of `workloads.configs`; weights, caches and tokens are seeded random numbers of the
distributions `workloads.generate` uses (matrices N(0, 0.02), gains around 1, cached K/V N(0, 1)), made on the GPU.
"""
import math
import random

import numpy as np
import torch

import paper_2601_19139_amd as dk
from workloads.configs import CONFIGS

BLOCK = 16        # tokens per KV block
CHUNK = 64        # prompt tokens per prefill call: the largest the library takes
DENSE = ("qwen3_0p6b", "llama32_3b", "qwen3_8b")
MOE = "qwen3_30b_a3b_l4"


def listed():
    return [
        # one chat user's next token: 0.6B shape alone (the benchmark's default workload)
        dict(name="decode_0p6b_b1", kind="decode", model="qwen3_0p6b", bits=16, batch=1, ctx_lo=512, ctx_hi=512, shared=0, sharers=0),
        # 16 and 64 concurrent short conversations on the small model
        dict(name="decode_0p6b_b16", kind="decode", model="qwen3_0p6b", bits=16, batch=16, ctx_lo=384, ctx_hi=640, shared=0, sharers=0),
        dict(name="decode_0p6b_b64", kind="decode", model="qwen3_0p6b", bits=16, batch=64, ctx_lo=37, ctx_hi=900, shared=0, sharers=0),
        # a handful of requests on the mid-size model
        dict(name="decode_3b_b4", kind="decode", model="llama32_3b", bits=16, batch=4, ctx_lo=200, ctx_hi=1500, shared=0, sharers=0),
        # 4-bit weights (the precision of the paper's checkpoints), half of the requests behind one cached system prompt
        dict(name="decode_3b_q4_b16", kind="decode", model="llama32_3b", bits=4, batch=16, ctx_lo=128, ctx_hi=2048, shared=1024, sharers=8),
        # long documents on the large dense model
        dict(name="decode_8b_b16_long", kind="decode", model="qwen3_8b", bits=16, batch=16, ctx_lo=4096, ctx_hi=4096, shared=0, sharers=0),
        # mixture of experts, ragged, half of the requests behind a long cached prefix
        dict(name="decode_moe_b16", kind="decode", model=MOE, bits=16, batch=16, ctx_lo=256, ctx_hi=4096, shared=2048, sharers=8),
        # an ordinary prompt on the large model; its length is no multiple of anything
        dict(name="prefill_8b_501", kind="prefill", model="qwen3_8b", bits=16, start=0, tokens=501),
        # a longer prompt behind a cached prefix, 4-bit weights
        dict(name="prefill_3b_q4_700", kind="prefill", model="llama32_3b", bits=4, start=256, tokens=700),
        # the sampler alone: one row with the usual thresholds; a batch with a nucleus threshold only
        dict(name="sample_b1", kind="sample", vocab=151936, batch=1, top_k=50, top_p=0.9),
        dict(name="sample_b16_top_p", kind="sample", vocab=151936, batch=16, top_k=0, top_p=0.9),
        # eight requests submitted together, sharing a stem, more than there are rows: queueing, prefix reuse, retirement
        dict(name="serve_0p6b", kind="serve", model="qwen3_0p6b", bits=16, requests=8, rows=6, stem=128, prompt_lo=140, prompt_hi=420, new=12),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("decode", "prefill", "sample", "serve"), (9, 4, 2, 1))[0]
    if kind == "decode":
        model = rng.choice(DENSE + (MOE,))
        batch = _log_int(rng, 1, 64)
        hi = _log_int(rng, 16, min(4096, 65536 // batch))
        lo = rng.randint(max(0, hi // 8), hi)
        shared = rng.choice((0, 0, 1)) * (hi // 2 // BLOCK * BLOCK) if batch > 1 else 0
        sharers = rng.randint(2, batch) if shared else 0
        return dict(kind=kind, model=model, bits=rng.choice((16, 4)), batch=batch, ctx_lo=lo, ctx_hi=hi, shared=shared, sharers=sharers)
    if kind == "prefill":
        model = rng.choice(DENSE + (MOE,))
        most = {"qwen3_0p6b": 2048, "llama32_3b": 1000, "qwen3_8b": 500, MOE: 1500}[model]
        return dict(kind=kind, model=model, bits=rng.choice((16, 4)), start=rng.choice((0, 0, BLOCK * rng.randint(1, 64))),
                    tokens=_log_int(rng, 5, most))
    if kind == "sample":
        top_k, top_p = rng.choice(((0, 1.0), (_log_int(rng, 1, 64), 1.0), (0, rng.uniform(0.3, 0.99)),
                                   (_log_int(rng, 2, 64), rng.uniform(0.3, 0.99))))
        return dict(kind=kind, vocab=rng.choice((128256, 151936)), batch=_log_int(rng, 1, 64), top_k=top_k, top_p=top_p)
    requests = rng.randint(2, 8)
    lo = rng.randint(20, 200)
    return dict(kind=kind, model="qwen3_0p6b", bits=rng.choice((16, 4)), requests=requests, rows=rng.randint(1, requests),
                stem=min(lo - 1, rng.choice((0, 64, 128))), prompt_lo=lo, prompt_hi=rng.randint(lo, 420), new=rng.randint(2, 12))


# ---- inputs --------------------------------------------------------------------------------------------------

class _Model:
    """Weights on the GPU and the library's handle for them."""

    def __init__(self, name, bits, gen):
        self.shape, self.bits, self.gen, self.keep = CONFIGS[name], bits, gen, []
        s = self.shape
        self.cfg = dk.DkModelConfig.from_shape(s)
        embed = self._matrix(s.vocab, s.hidden)
        lm_head = embed if s.tie_lm_head and bits == 16 else self._weights(s.vocab, s.hidden)
        g_final = self._gain(s.hidden)
        self.layers = (dk.LayerWeights * s.n_layers)()
        E = s.n_experts
        for L in self.layers:
            L.g_attn, L.g_mlp = self._gain(s.hidden), self._gain(s.hidden)
            L.g_q = self._gain(s.head_dim) if s.qk_norm else None
            L.g_k = self._gain(s.head_dim) if s.qk_norm else None
            L.w_qkv = self._weights(s.q_dim + 2 * s.kv_dim, s.hidden)
            L.w_o = self._weights(s.hidden, s.q_dim)
            L.w_router = self._matrix(E, s.hidden) if E else None
            L.w_gate = self._weights(E * s.expert_ffn if E else s.ffn, s.hidden)
            L.w_up = self._weights(E * s.expert_ffn if E else s.ffn, s.hidden)
            L.w_down = self._weights(E * s.hidden, s.expert_ffn) if E else self._weights(s.hidden, s.ffn)
        self.ptrs = dk.WeightPtrs(embed, lm_head, g_final, self.layers)
        self.handle = (dk.create_model if bits == 16 else dk.create_model_q4)(self.cfg, self.ptrs)

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            dk.destroy_model(self.handle)

    def _keep(self, t):
        self.keep.append(t)
        return t.data_ptr()

    def _gain(self, n):
        return self._keep(torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(1.0, 0.02, generator=self.gen))

    def _matrix(self, n, k):
        return self._keep(torch.empty(n, k, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=self.gen))

    def _weights(self, n, k):
        if self.bits == 16:
            return self._matrix(n, k)
        # the packed 4-bit format: codes as min/max quantisation of 64 normal numbers gives them, two to a byte,
        # then (scale, bias) pairs per row and 64 columns
        codes, groups = n * k // 2, (n + 15) // 16 * 16 * (k // 64)
        buf = torch.empty(codes + groups * 4, dtype=torch.uint8, device="cuda")
        for o in range(0, codes, 1 << 28):
            m = min(1 << 28, codes - o)
            z = torch.empty(2, m, dtype=torch.bfloat16, device="cuda").normal_(7.5, 3.1, generator=self.gen)
            z = z.round_().clamp_(0, 15).to(torch.uint8)
            torch.add(z[0], z[1], alpha=16, out=buf[o:o + m])
        pairs = buf[codes:].view(torch.bfloat16).view(groups, 2)
        scale = torch.empty(groups, device="cuda").normal_(0.0064, 0.0008, generator=self.gen).clamp_(0.003)
        pairs[:, 0] = scale
        pairs[:, 1] = scale * torch.empty(groups, device="cuda").normal_(-7.5, 0.6, generator=self.gen)
        return self._keep(buf)


class _State:
    pass


def _aligned(nbytes, s):
    """256-byte aligned device scratch, kept by the state."""
    s.raw = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    return (s.raw.data_ptr() + 255) // 256 * 256


def _pool(s, n_blocks, gen):
    nbytes = dk.kv_pool_bytes(s.model.cfg, n_blocks, BLOCK)
    s.kv = torch.empty(nbytes // 2, dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=gen)
    s.pool = dk.create_kv_pool(s.model.cfg, n_blocks, BLOCK, s.kv, nbytes)


def _contexts(case, rng):
    """Cached tokens of every row; the sharers' are longer than the shared prefix."""
    ctx = [rng.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["batch"])]
    for i in range(case["sharers"]):
        ctx[i] = max(ctx[i], rng.randint(case["shared"], case["ctx_hi"]))
    return ctx


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    s = _State()
    s.kind = case["kind"]
    if s.kind == "sample":
        B, V = case["batch"], case["vocab"]
        # logits as a trained model gives them: a wide bulk and a few tokens that stand out
        s.logits = torch.empty(B, V, device="cuda").normal_(0.0, 2.0, generator=gen)
        hot = torch.randint(0, V, (B, 40), device="cuda", generator=gen)
        s.logits.scatter_(1, hot, torch.empty(B, 40, device="cuda").normal_(14.0, 2.0, generator=gen))
        s.scratch = torch.empty(dk.sample_scratch_bytes(B, V), dtype=torch.uint8, device="cuda")
        s.out = torch.empty(B, dtype=torch.int32, device="cuda")
        s.args = (0.8, case["top_k"], case["top_p"], rng.getrandbits(32), rng.getrandbits(16))
        return s
    s.model = _Model(case["model"], case["bits"], gen)
    shape, h = s.model.shape, s.model.handle
    if s.kind == "serve":
        stem = [rng.randrange(shape.vocab) for _ in range(case["stem"])]
        s.prompts = [np.array(stem + [rng.randrange(shape.vocab) for _ in range(rng.randint(case["prompt_lo"], case["prompt_hi"]) - len(stem))],
                              dtype=np.int32) for _ in range(case["requests"])]
        s.new, width = case["new"], (case["prompt_hi"] + case["new"]) // BLOCK + 2
        _pool(s, case["requests"] * width, gen)
        s.cfg = dk.EngineConfig(case["rows"], width, CHUNK, 1)
        s.arena_bytes = dk.engine_device_bytes(h, s.cfg)
        s.arena = _aligned(s.arena_bytes, s)
        return s
    if s.kind == "prefill":
        s.start, width, rows = case["start"], (case["start"] + case["tokens"]) // BLOCK + 4, 1
        ids = list(range(width))
        rng.shuffle(ids)
        tables = [ids]
        s.chunks = torch.randint(0, shape.vocab, (case["tokens"],), dtype=torch.int32, device="cuda", generator=gen).split(CHUNK)
        rows = min(CHUNK, case["tokens"])
    else:
        ctx = _contexts(case, rng)
        rows, width = case["batch"], case["ctx_hi"] // BLOCK + 8
        shared = case["shared"] // BLOCK
        ids = list(range(shared + rows * (case["ctx_hi"] // BLOCK + 1)))
        n_ids = len(ids)
        rng.shuffle(ids)
        prefix, ids = ids[:shared], ids[shared:]
        tables = []
        for i, t in enumerate(ctx):
            head = prefix if i < case["sharers"] else []
            own = t // BLOCK + 1 - len(head)
            tables.append(head + ids[:own] + [-1] * (width - len(head) - own))
            ids = ids[own:]
        s.seq_lens = torch.tensor(ctx, dtype=torch.int32, device="cuda")
        s.tokens = torch.randint(0, shape.vocab, (rows,), dtype=torch.int32, device="cuda", generator=gen)
    _pool(s, width if s.kind == "prefill" else n_ids, gen)
    s.tables = torch.tensor(tables, dtype=torch.int32, device="cuda")
    s.ws_bytes = dk.workspace_bytes(h, rows, width)
    s.ws = _aligned(s.ws_bytes, s)
    last = s.chunks[-1].numel() if s.kind == "prefill" else rows
    s.logits = torch.empty(last, shape.vocab, device="cuda")
    s.next = torch.empty(last, dtype=torch.int32, device="cuda")
    return s


# ---- one pass ------------------------------------------------------------------------------------------------

def run(s):
    if s.kind == "sample":
        temperature, top_k, top_p, seed, step = s.args
        dk.sample_tokens(s.logits, temperature, top_k, top_p, seed, step, s.scratch, s.out)
        return s.out
    h = s.model.handle
    if s.kind == "decode":
        dk.decode_step(h, s.pool, s.tables, s.seq_lens, s.tokens, s.ws, s.logits, s.next, workspace_bytes_=s.ws_bytes)
        return {"logits": s.logits, "next": s.next, "kv": s.kv}
    if s.kind == "prefill":
        at, table = s.start, s.tables[0]
        for part in s.chunks[:-1]:      # predictions are wanted for the last chunk only
            dk.prefill_chunk(h, s.pool, table, at, part, s.ws, s.ws_bytes, None, None)
            at += CHUNK
        dk.prefill_chunk(h, s.pool, table, at, s.chunks[-1], s.ws, s.ws_bytes, s.logits, s.next)
        return {"logits": s.logits, "next": s.next, "kv": s.kv}
    engine = dk.engine_create(h, s.pool, s.cfg, s.arena, s.arena_bytes)
    ids = [dk.engine_submit(engine, p, s.new) for p in s.prompts]
    while dk.engine_step(engine):
        pass
    tokens = [dk.engine_poll(engine, i, s.new)[0] for i in ids]
    dk.engine_destroy(engine)
    return {"tokens": np.stack(tokens), "kv": s.kv}


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def _params(c):
    """(dense weights of all layers, weights of one expert of one layer, lm_head weights)"""
    attn = 2 * c.hidden * c.q_dim + 2 * c.hidden * c.kv_dim
    if c.n_experts:
        return c.n_layers * (attn + c.n_experts * c.hidden), 3 * c.hidden * c.expert_ffn, c.vocab * c.hidden
    return c.n_layers * (attn + 3 * c.hidden * c.ffn), 0, c.vocab * c.hidden


def _forward(case, n_tokens, attended, kv_tokens, n_logits):
    """Bytes and flops of n_tokens positions that attend to `attended` positions in all, `kv_tokens` distinct cached
    tokens read or written, logits for n_logits positions."""
    c = CONFIGS[case["model"]]
    dense, expert, head = _params(c)
    size = 2.0 if case["bits"] == 16 else 0.5 + 4.0 / 64
    weights = dense + head
    active = dense + c.n_layers * c.top_k * expert
    if c.n_experts:   # distinct experts of n_tokens routings, expected
        weights += c.n_layers * expert * c.n_experts * (1 - (1 - c.top_k / c.n_experts) ** n_tokens)
    return {"bytes": weights * size + kv_tokens * c.kv_bytes_per_token() + n_tokens * c.hidden * 2 + n_logits * c.vocab * 4,
            "flops": 2.0 * active * n_tokens + 2.0 * head * n_logits + 4.0 * c.n_layers * c.q_dim * attended}


def work(case):
    if case["kind"] == "sample":
        n = case["batch"] * case["vocab"]
        return {"bytes": n * 4 + case["batch"] * 4, "flops": n * 2}
    if case["kind"] == "decode":
        B, mean = case["batch"], (case["ctx_lo"] + case["ctx_hi"]) / 2
        if case["sharers"]:   # a sharer's context lies above the prefix, of which one copy is read
            sharer = max(mean, (case["shared"] + case["ctx_hi"]) / 2)
            total = (B - case["sharers"]) * mean + case["sharers"] * sharer
            distinct = total - (case["sharers"] - 1) * case["shared"]
        else:
            total = distinct = B * mean
        return _forward(case, B, total + B, distinct + B, B)
    if case["kind"] == "prefill":
        P, at = case["tokens"], case["start"]
        return _forward(case, P, P * at + P * (P + 1) / 2, at + P, (P - 1) % CHUNK + 1)
    # serve: every prompt token behind the reused stem once, then a step per new token and group of rows
    R, mean = case["requests"], (case["prompt_lo"] + case["prompt_hi"]) / 2
    reused = (R - 1) * (case["stem"] // BLOCK * BLOCK)
    steps = (case["new"] - 1) * -(-R // case["rows"])
    p = _forward(case, R * mean - reused, R * mean * mean / 2, R * mean - reused, R)
    d = _forward(case, R / max(1, -(-R // case["rows"])), mean * R, mean * min(R, case["rows"]), case["rows"])
    return {k: p[k] + steps * d[k] for k in p}


def tolerance(case):
    """float32 sums over bf16 weights and 16-bit activations; new K/V are rounded to bf16, so values on a rounding
    boundary move by one bf16 step (at most 2^-7 of the value), and what follows from them a little.  Seen between
    a decode step and the same rows one by one on the vector kernels: logits 4e-5; between a prompt in chunks of 64
    and in chunks of 48 or 13: logits 3e-4, K/V 1e-3 (largest 0.014)."""
    if case["kind"] == "sample":
        return {"differ": 0.01}
    if case["kind"] == "decode":
        return {"rel": 2e-4, "max": 0.016, "differ": 0.01}
    return {"rel": 4e-3, "max": 0.05, "differ": 0.01}
