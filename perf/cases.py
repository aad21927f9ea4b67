"""The work that programs ask of this library, as cases that can be timed and compared.

Three kinds of work, all through the public entry points of `paper_2512_19206_amd`:

  step      one mixkvq_decode_step over a filled cache: a generated token enters the fp16 window and the step's
            queries attend over the whole context.  The pass rewinds the token counts first (mixkvq_cache_set_state,
            host-only), as a program does that takes a rejected token back, so every pass sees the same context.
  generate  a run of decode steps from a prompt's snapshot (a further continuation of one prompt): the window
            fills, blocks are scored and packed on the way.  The sequences of the batch have equal or different
            lengths, their blocks live in the contiguous or in the paged layout.
  prefill   a prompt into an empty cache: scoring, channel selection, quantize-and-pack; whole or in chunks, for
            the batch or for one request in a slot of it, with one selection per prompt or per block.

Inputs follow synth_inputs.py's structure (heavy-tailed token magnitudes, a few outlier channels in the keys and in
the queries), drawn on the GPU from the seed alone.
"""
import math

import torch

import paper_2512_19206_amd as M

D = 128
PROMPT_QUERIES = 64        # queries a cache is scored with while it is filled (decode cases; not part of a pass)


def _cfg(hq, hkv, R=128, G=128, k4=16, k16=0, thresholds=False, dtype="f16"):
    return dict(hq=hq, hkv=hkv, R=R, G=G, k4=k4, k16=k16, thresholds=thresholds, dtype=dtype)


def listed():
    return [
        # The first answers of a chat: one short prompt that still sits in the fp16 window, nothing packed yet.
        dict(name="step_b1_window", kind="step", B=1, T=90, **_cfg(28, 4)),
        # The smallest quantized cache: one head, 1024 tokens, groups and residual window of 32 (parity configuration).
        dict(name="step_b1_1k", kind="step", B=1, T=1027, **_cfg(1, 1, R=32, G=32, k4=8)),
        # The benchmark's headline: a 7B-shaped layer, 8 sequences at 32K.
        dict(name="step_b8_32k", kind="step", B=8, T=32805, **_cfg(28, 4)),
        # A 32B-shaped layer serving a large batch at 32K, salient channels kept in fp16.
        dict(name="step_b64_32k", kind="step", B=64, T=32790, **_cfg(40, 8, k4=0, k16=12)),
        # Long reasoning: few sequences, 128K tokens each.
        dict(name="step_b4_128k", kind="step", B=4, T=131091, **_cfg(40, 8)),
        # The accuracy setting: thresholds instead of budgets, groups of 32, both side tiers, bfloat16 tensors.
        dict(name="step_b6_9k_thresholds", kind="step", B=6, T=9001,
             **_cfg(28, 4, G=32, k4=16, k16=8, thresholds=True, dtype="bf16")),
        # Continuous batching: sequences of very different lengths, paged blocks, a few tokens for all of them.
        dict(name="generate_b24_ragged_paged", kind="generate", B=24, T_min=60, T=12003, steps=24, ragged=True,
             paged=True, **_cfg(28, 4, dtype="bf16")),
        # The throughput setting with the short residual window: a block is packed every 32 tokens.
        dict(name="generate_b4_4k_r32", kind="generate", B=4, T_min=4100, T=4100, steps=48, ragged=False, paged=False,
             **_cfg(40, 8, R=32, G=32)),
        # A whole batch of long prompts (offline work).
        dict(name="prefill_b16_32k", kind="prefill", B=16, T=32768, chunk=32768, slot=False, per_block=False,
             **_cfg(40, 8)),
        # One request of ordinary length admitted into a slot of a running batch.
        dict(name="prefill_slot_1531", kind="prefill", B=8, T=1531, chunk=1531, slot=True, per_block=False,
             **_cfg(28, 4, dtype="bf16")),
        # A prompt that arrives in chunks; every block is scored on its own tokens under the thresholds.
        dict(name="prefill_b2_chunks_thresholds", kind="prefill", B=2, T=8190, chunk=1000, slot=False, per_block=True,
             **_cfg(28, 4, G=32, k4=16, k16=8, thresholds=True)),
        # A small batch of medium prompts, fp16 tier.
        dict(name="prefill_b4_5k", kind="prefill", B=4, T=5000, chunk=5000, slot=False, per_block=False,
             **_cfg(40, 8, k4=0, k16=12)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    hq, hkv = rng.choice([(1, 1), (14, 2), (28, 4), (40, 8), (40, 8), (28, 4), (8, 8)])
    R, G = rng.choice([(128, 128), (128, 128), (128, 128), (128, 32), (128, 64), (64, 64), (32, 32), (256, 128)])
    k4, k16, thr = rng.choice([(16, 0, False), (16, 0, False), (0, 12, False), (8, 0, False), (16, 8, True)])
    base = _cfg(hq, hkv, R=R, G=G, k4=k4, k16=k16, thresholds=thr, dtype=rng.choice(["f16", "bf16"]))
    kind = rng.choice(["step", "step", "step", "generate", "prefill", "prefill"])
    if kind == "step":
        B = _log_int(rng, 1, 64)
        most = min(131072, 64 * 8 * 32768 // (B * hkv))
        return dict(kind=kind, B=B, T=_log_int(rng, 40, most), **base)
    if kind == "generate":
        ragged = rng.random() < 0.6
        B = _log_int(rng, 2 if ragged else 1, 32)
        T = _log_int(rng, 200, 16000)
        return dict(kind=kind, B=B, T_min=_log_int(rng, 30, T) if ragged else T, T=T, steps=rng.randint(8, 48),
                    ragged=ragged, paged=rng.random() < 0.5, **base)
    B = _log_int(rng, 1, 16)
    T = _log_int(rng, 100, 32768)
    slot = rng.random() < 0.4
    per_block = thr or rng.random() < 0.25
    chunk = T if rng.random() < 0.6 else _log_int(rng, max(50, T // 12), T)
    return dict(kind=kind, B=B, T=T, chunk=chunk, slot=slot, per_block=per_block, **base)


# ---------------------------------------------------------------------------- inputs

def _lengths(case):
    """Context length of every sequence of a decode case (spread over the logarithm when they differ)."""
    B, T = case["B"], case["T"]
    if not case.get("ragged"):
        return [T] * B
    lo = case["T_min"]
    return [int(round(lo * (T / lo) ** ((0.618034 * (b + 1)) % 1.0))) for b in range(B)]


def _heavy_tail(shape, gen):
    """|t| with 3 degrees of freedom, unit mean."""
    z = torch.randn((4,) + shape, generator=gen, device="cuda")
    return z[0].abs_() / (z[1:].square().sum(0) / 3.0).sqrt_() / 1.1027


def _outliers(heads, gen):
    """[heads, 1, D] channel scales: 1, except 4 channels at 10 to 20."""
    c = torch.ones((heads, D), device="cuda")
    at = torch.rand((heads, D), generator=gen, device="cuda").topk(4, dim=1).indices
    c.scatter_(1, at, 10.0 + 10.0 * torch.rand((heads, 4), generator=gen, device="cuda"))
    return c[:, None, :]


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float16


def _fill(out, scale, gen, heavy):
    """out [heads, L, D] <- scale * token magnitude * N(0, 1), in pieces that bound the temporaries."""
    H, L = out.shape[0], out.shape[1]
    step = max(1, (1 << 25) // (H * D))
    for t in range(0, L, step):
        n = min(step, L - t)
        x = torch.randn((H, n, D), generator=gen, device="cuda")
        if heavy:
            x *= _heavy_tail((H, n, 1), gen)
        if scale is not None:
            x *= scale
        out[:, t:t + n] = x.clamp_(-32768.0, 32768.0)


class _Source:
    """Keys, values and queries of one sequence: fixed outlier channels, tokens drawn as they are asked for."""

    def __init__(self, case, gen):
        self.case, self.gen = case, gen
        self.kc, self.qc = _outliers(case["hkv"], gen), _outliers(case["hq"], gen)

    def kv(self, n):
        k = torch.empty((self.case["hkv"], n, D), dtype=_dtype(self.case), device="cuda")
        v = torch.empty_like(k)
        _fill(k, self.kc, self.gen, True)
        _fill(v, None, self.gen, True)
        return k, v

    def q(self, n):
        q = torch.empty((self.case["hq"], n, D), dtype=_dtype(self.case), device="cuda")
        _fill(q, self.qc, self.gen, False)
        return q


def _make_cache(case, T_max):
    R = case["R"]
    kw = dict(B=case["B"], Hq=case["hq"], Hkv=case["hkv"], D=D, T_max=-(-T_max // R) * R, Gk=min(case["G"], R),
              Gv=case["G"], R=R, k4=case["k4"], k16=case["k16"], in_dtype=1 if case["dtype"] == "bf16" else 0)
    if case["thresholds"]:
        kw.update(policy=1, tau16=20.0, tau4=4.0)
    return M.Cache(M.make_config(**kw))


def _rewind(state):
    """Token counts back to the snapshot's."""
    gc = state["cache"]
    if state["ragged"]:
        for b, (nq, r, ns) in enumerate(state["counts"]):
            gc.lib.mixkvq_cache_set_state_seq(gc.handle, b, nq, r, ns)
    else:
        gc.lib.mixkvq_cache_set_state(gc.handle, *state["counts"][0])


def _prepare_decode(case, gen):
    B, lens, R = case["B"], _lengths(case), case["R"]
    n_steps = case.get("steps", 1)
    gc = _make_cache(case, max(lens) + n_steps + R)
    table = None
    if case.get("paged"):
        slots = B * (gc.cfg.T_max // gc.rec_tokens)
        table = torch.randperm(slots, generator=gen, device="cuda").to(torch.int32).view(B, -1).contiguous()
        gc.set_block_table(table)
    # the new tokens of every step, and their queries
    new_k = torch.empty((n_steps, B, case["hkv"], 1, D), dtype=_dtype(case), device="cuda")
    new_v, new_q = torch.empty_like(new_k), torch.empty((n_steps, B, case["hq"], D), dtype=_dtype(case), device="cuda")
    for b in range(B):
        src = _Source(case, gen)
        k, v = src.kv(lens[b] + n_steps)
        n = lens[b]
        if case["kind"] == "step":       # the pass's token must find room in the window (no block is packed by it)
            n = max(1, n - 1) if n % R == 0 else n
        sel = gc.select_channels_seq(b, src.q(PROMPT_QUERIES), k[:, :n])
        gc.quantize_append_seq(b, k[:, :n], v[:, :n], sel=None if case["thresholds"] else sel)
        new_k[:, b] = k[:, lens[b]:].permute(1, 0, 2)[:, :, None]
        new_v[:, b] = v[:, lens[b]:].permute(1, 0, 2)[:, :, None]
        new_q[:, b] = src.q(n_steps).permute(1, 0, 2)
    out = torch.empty((n_steps, B, case["hq"], D), dtype=_dtype(case), device="cuda")
    lse = torch.empty((n_steps, B, case["hq"]), dtype=torch.float32, device="cuda")
    counts = [gc.state_seq(b) for b in range(B)]
    state = dict(case=case, cache=gc, counts=counts, ragged=any(c != counts[0] for c in counts), out=out, lse=lse)
    state["steps"] = [dict(k=new_k[i], v=new_v[i], q=new_q[i], out=out[i], lse=lse[i]) for i in range(n_steps)]
    # the parts of the cache a pass writes, as views: the accumulator, and after it the fp16 rows in use
    acc, cnt = gc.query_accumulator()
    state["qacc"] = [acc, cnt]
    if case["kind"] == "step":
        rk, rv = gc.fp16_rows()
        n = counts[0][1] + 1
        state["rows"] = [rk[:, :n], rv[:, :n]]
    else:
        # rows no token has reached yet hold nothing: give them a value once, so that they can be returned whole
        _settle_rows(gc, counts, case)
        state["saved"] = [t.clone() for t in (gc.res_k, gc.res_v, gc.qacc)]
        state["rows"] = list(gc.fp16_rows())
        state["packed"] = _packed_views(gc, case, table, counts, n_steps)
    torch.cuda.synchronize()
    return state


def _settle_rows(gc, counts, case):
    rk, rv = gc.fp16_rows()
    for b, (_, r, ns) in enumerate(counts):
        p = slice(b * case["hkv"], (b + 1) * case["hkv"])
        rk[p, ns + r:] = 0
        rv[p, ns + r:] = 0


def _packed_views(gc, case, table, counts, n_steps):
    """Views of the block records a pass packs (at most 24 of them are returned)."""
    R, per = case["R"], case["R"] // gc.rec_tokens
    got = []
    for b, (nq, r, _) in enumerate(counts):
        flushed = max(0, -(-(r + n_steps) // R) - 1)
        for i in range(nq // gc.rec_tokens, nq // gc.rec_tokens + flushed * per):
            if len(got) == 24:
                return got
            if table is not None:
                got.append(gc.pool_records()[int(table[b, i])])
            else:
                got.append(gc.block_records()[b * case["hkv"]:(b + 1) * case["hkv"], i])
    return got


def _prepare_prefill(case, gen):
    B, T = case["B"], case["T"]
    gc = _make_cache(case, T)
    n_seq = 1 if case["slot"] else B
    k = torch.empty((n_seq, case["hkv"], T, D), dtype=_dtype(case), device="cuda")
    v = torch.empty_like(k)
    q = torch.empty((n_seq, case["hq"], T, D), dtype=_dtype(case), device="cuda")
    for b in range(n_seq):
        src = _Source(case, gen)
        _fill(k[b], src.kc, gen, True)
        _fill(v[b], None, gen, True)
        _fill(q[b], src.qc, gen, False)
    state = dict(case=case, cache=gc, slot=B // 2, k=k, v=v, q=q)
    shape = (case["hkv"], gc.ks) if case["slot"] else (B, case["hkv"], gc.ks)
    chunks = []
    for t in range(0, T, case["chunk"]):
        part = [x[:, :, t:t + case["chunk"]] for x in (q, k, v)]
        if case["slot"]:
            part = [x[0] for x in part]
        chunks.append((*part, torch.zeros(shape, dtype=torch.uint8, device="cuda")))
    state["chunks"] = chunks
    # views of what a pass writes: the records, the fp16 rows in use, the accumulator
    R, nb = case["R"], max(0, -(-T // case["R"]) - 1) * (case["R"] // gc.rec_tokens)
    p = slice(state["slot"] * case["hkv"], (state["slot"] + 1) * case["hkv"]) if case["slot"] else slice(0, B * case["hkv"])
    rk, rv = gc.fp16_rows()
    r = T - (nb * gc.rec_tokens)
    acc, cnt = gc.query_accumulator()
    state["written"] = [gc.block_records()[p, :nb], rk[p, :r], rv[p, :r], acc[p], cnt[p]]
    torch.cuda.synchronize()
    return state


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return _prepare_prefill(case, gen) if case["kind"] == "prefill" else _prepare_decode(case, gen)


# ---------------------------------------------------------------------------- one pass

def _run_step(state):
    s = state["steps"][0]
    _rewind(state)
    M.mixkvq_decode_step(state["cache"], s["k"], s["v"], s["q"], out=s["out"], lse=s["lse"], accumulate_q=True)
    return [s["out"], s["lse"]] + state["rows"] + state["qacc"]


def _run_generate(state):
    gc = state["cache"]
    for dst, src in zip((gc.res_k, gc.res_v, gc.qacc), state["saved"]):
        dst.copy_(src)
    _rewind(state)
    for s in state["steps"]:
        M.mixkvq_decode_step(gc, s["k"], s["v"], s["q"], out=s["out"], lse=s["lse"], accumulate_q=True)
    return [state["out"], state["lse"]] + state["rows"] + state["qacc"] + state["packed"]


def _run_prefill(state):
    case, gc, b = state["case"], state["cache"], state["slot"]
    if case["slot"]:
        gc.reset_seq(b)
        for q, k, v, sel in state["chunks"]:
            gc.select_channels_seq(b, q, k, sel=sel)
            gc.quantize_append_seq(b, k, v, sel=None if case["per_block"] else sel)
    else:
        gc.reset()
        for q, k, v, sel in state["chunks"]:
            if case["per_block"]:
                M.mixkvq_select_channels(gc, q, k, sel=sel)
                M.mixkvq_quantize_append(gc, k, v)
            else:
                M.mixkvq_prefill(gc, q, k, v, sel=sel)
    return [c[3] for c in state["chunks"]] + state["written"]


def run(state):
    return {"step": _run_step, "generate": _run_generate, "prefill": _run_prefill}[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------- what a pass cannot do without

def _packed_bytes(case, n):
    """Minimal representation of n quantized tokens of one KV head (thresholds: at the capacities)."""
    k4, k16, G, R = case["k4"], case["k16"], case["G"], case["R"]
    ks, gk = k4 + k16, min(case["G"], case["R"], 128)
    return (n * (D - ks) / 4 + n / gk * (D - ks) * 4 + n * k4 / 2 + n / gk * k4 * 4 + n * k16 * 2 + n / R * ks
            + n * D / 4 + n * (D // G) * 4)


def _split(case, n):
    """(quantized, window) tokens of a sequence of n tokens (a full window is flushed when the next token enters)."""
    nq = max(0, -(-n // case["R"]) - 1) * case["R"]
    return nq, n - nq


def work(case):
    g, hkv = case["hq"] // case["hkv"], case["hkv"]
    row = 2 * D
    if case["kind"] == "prefill":
        n_seq = 1 if case["slot"] else case["B"]
        nq, r = _split(case, case["T"])
        nbytes = n_seq * hkv * (case["T"] * (2 + g) * row + _packed_bytes(case, nq) + r * 2 * row + D * 8)
        return {"bytes": nbytes, "flops": 0.0}
    nbytes = flops = 0.0
    for n0 in _lengths(case):
        for i in range(case.get("steps", 1)):
            nq, r = _split(case, n0 + i + 1)
            nbytes += hkv * (_packed_bytes(case, nq) + r * 2 * row + g * 2 * row + 2 * 2 * row + 2 * D * 8)
            flops += 4.0 * (n0 + i + 1) * D * case["hq"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Selections, records, fp16 rows and |q| sums are whole numbers and bit patterns: the same.  Attention outputs
    differ by the rounding of the softmax weights to fp16 and of the output: against binary64 attention over the same
    cache 1.3e-4 to 2.3e-4 (largest single difference 4.6e-4) with fp16 tensors, 1.4e-3 (3.8e-3; 7.8e-3 between two
    orders of the sums) with bfloat16; four times that."""
    if case["kind"] == "prefill":
        return "exact"
    return {"rel": 6e-3, "max": 0.03} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 4e-3}
