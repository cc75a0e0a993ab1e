"""Performance cases of the D^3 decode path: what a serving or evaluation program has the library do.

Each case is one call sequence through the public entry points (`binding.Decoder`): the prompt pass, a continuation prompt
on a filled cache, or a decode step with the missing-state fill that follows it.  Models are the shapes of the benchmark
configurations (a tiny fp32 one; the 7B, 13B and 70B widths in bf16), with every block holding weights of its own; apart from the one
whole 7B model the depth is cut so that a case is a few blocks and the head, i.e. the layers of the path.

    listed(), draw(rng)   the cases, and more of the same ranges
    prepare(case, seed)   weights, caches, prompt and plan on the GPU, as a program keeps them between calls
    run(state)            one pass; returns the logits and the cache rows that the pass wrote
    work(case)            bytes and flops a pass cannot do without
    tolerance(case)       how far another correct implementation at this precision may be off
    exact(case, seed)     the same outputs in float64 by plain torch, rows of the cache unrounded

Tokens are given, not fed back, so that one near-tie between two logits does not change what the rest of a pass computes.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2503_08524_amd import binding

DEVICE = "cuda:0"

# Widths of the benchmark configurations.
WIDTHS = {
    "tiny": dict(d=256, H=4, H_kv=4, hd=64, F=688, V=1024, dtype="f32", kv="f32"),
    "7b": dict(d=4096, H=32, H_kv=32, hd=128, F=11008, V=32000, dtype="bf16", kv="f16"),
    "13b": dict(d=5120, H=40, H_kv=40, hd=128, F=13824, V=32000, dtype="bf16", kv="f16"),
    # the 70B model has 80 blocks, whose cache the library keeps in fp32 (binding.default_kv_dtype)
    "70b": dict(d=8192, H=64, H_kv=8, hd=128, F=28672, V=32000, dtype="bf16", kv="f32"),
}
START_FRACTION = 0.6      # first dropped block, as a fraction of the depth (the benchmark's)
SPARE_ROWS = 64           # cache rows a program leaves for the tokens to come


def _decode(name, model, L, keep, B, P, fill="copy"):
    return {"name": name, "kind": "decode", "model": model, "L": L, "keep": keep, "B": B, "P": P, "fill": fill}


def _prompt(name, model, L, B, P, past=0, ragged=False):
    return {"name": name, "kind": "prompt", "model": model, "L": L, "B": B, "P": P, "past": past, "ragged": ragged}


def listed():
    return [
        # one step of the smallest model: nothing but latencies and launches
        _decode("decode_tiny_b1", "tiny", 4, 3, 1, 16),
        # the headline workload: a whole 7B model, one user, a step at the request's average depth (alpha 0.995: 17.5 blocks)
        _decode("decode_7b_b1", "7b", 32, 17, 1, 512),
        # few users on the 13B model, every block of the cut model kept, as early in a request
        _decode("decode_13b_b4", "13b", 8, 8, 4, 1024),
        # the full batch with long contexts: as many cache bytes as weight bytes
        _decode("decode_7b_b32", "7b", 6, 4, 32, 2048),
        # grouped-query attention on an fp32 cache
        _decode("decode_70b_b8", "70b", 4, 3, 8, 1024),
        # one few-shot prompt
        _prompt("prompt_7b_b1", "7b", 8, 1, 512),
        # an evaluation harness's batch of equal prompts
        _prompt("prompt_13b_b4", "13b", 4, 4, 1024),
        # the largest: 65 536 prompt tokens
        _prompt("prompt_7b_b32", "7b", 2, 32, 2048),
        # grouped-query prompt on an fp32 cache
        _prompt("prompt_70b_b8", "70b", 2, 8, 1024),
        # unequal few-shot prompts padded on the left: 512, 384, 256, 128 tokens
        _prompt("prompt_7b_ragged_b4", "7b", 8, 4, 512, ragged=True),
        # a batch of short questions of odd length
        _prompt("prompt_7b_short_b8", "7b", 8, 8, 77),
        # the next turn of four conversations: 203 new tokens on 1024 cached ones
        _prompt("prompt_7b_next_turn_b4", "7b", 8, 4, 203, past=1024),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    model = rng.choice(["tiny", "7b", "7b", "13b", "70b"])
    B = _log_uniform(rng, 1, 32)
    if rng.random() < 0.5:
        L = 4 if model == "tiny" else rng.randint(2, 6)
        P = min(_log_uniform(rng, 16, 128 if model == "tiny" else 3000), 65536 // B)
        case = _decode(None, model, L, rng.randint(max(1, L // 2), L), B, P, rng.choice(["copy", "copy", "recompute", "none"]))
    else:
        most = {"tiny": 4096, "7b": 49152, "13b": 16384, "70b": 8192}[model]      # tokens: no dearer than the largest listed case
        P = min(_log_uniform(rng, 16, 128 if model == "tiny" else 2048), most // B)
        L = 4 if model == "tiny" else 2 if B * P > most // 2 else rng.randint(2, 4)
        form = rng.choice(["equal", "ragged", "next_turn"])
        past = _log_uniform(rng, 16, 64 if model == "tiny" else 1024) if form == "next_turn" else 0
        case = _prompt(None, model, L, B, P, past, form == "ragged" and B > 1)
    del case["name"]
    return case


# ---------------- what a case stands for ----------------

def _shape(case):
    w = WIDTHS[case["model"]]
    return SimpleNamespace(name=case["model"], L=case["L"], eps=1e-6, rope_base=10000.0, **w)


def _lengths(case):
    """Tokens of each sequence: equal, or falling in equal steps from P to P / 4."""
    B, P = case["B"], case["P"]
    if not case.get("ragged"):
        return [P] * B
    return [int(round(P - 0.75 * P * b / (B - 1))) for b in range(B)]


def _window(case):
    """(first dropped block, dropped blocks) of the decode step."""
    L, n = case["L"], case["L"] - case["keep"]
    return min(int(START_FRACTION * L + 1e-9), L - n), n


def _weights(s, seed):
    """N(0, 0.02) linears and embedding, norm gains near one: drawn on the GPU from the seed alone."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000003 * seed + 17)
    wt = torch.float32 if s.dtype == "f32" else torch.bfloat16

    def normal(rows, cols):
        return torch.empty(rows, cols, dtype=torch.float32, device=DEVICE).normal_(0.0, 0.02, generator=g).to(wt)

    def gain():
        return torch.empty(s.d, dtype=torch.float32, device=DEVICE).normal_(1.0, 0.1, generator=g)

    q, kv = s.H * s.hd, s.H_kv * s.hd
    layers = [{"attn_norm": gain(), "wq": normal(q, s.d), "wk": normal(kv, s.d), "wv": normal(kv, s.d), "wo": normal(s.d, q),
               "mlp_norm": gain(), "w_gate": normal(s.F, s.d), "w_up": normal(s.F, s.d), "w_down": normal(s.d, s.F)} for _ in range(s.L)]
    return {"tok_emb": normal(s.V, s.d), "lm_head": normal(s.V, s.d), "final_norm": gain(), "layers": layers}


def _tokens(case, s, seed):
    """(tokens already in the cache or None, tokens of the pass): int32 arrays."""
    r = np.random.default_rng([seed, 5])
    B, P = case["B"], case["P"]
    if case["kind"] == "decode":
        return r.integers(0, s.V, (B, P), dtype=np.int32), r.integers(0, s.V, (B,), dtype=np.int32)
    past = r.integers(0, s.V, (B, case["past"]), dtype=np.int32) if case["past"] else None
    return past, r.integers(0, s.V, (B, P), dtype=np.int32)


# ---------------- prepare and run ----------------

def prepare(case, seed):
    s = _shape(case)
    B, past = case["B"], (case["P"] if case["kind"] == "decode" else case["past"])
    rows = past + (1 if case["kind"] == "decode" else case["P"])
    dec = binding.Decoder(s, _weights(s, seed), B, rows + SPARE_ROWS, kv_dtype=s.kv, device=DEVICE)
    before, now = _tokens(case, s, seed)
    st = SimpleNamespace(case=case, dec=dec, past=past, rows=rows, lengths=_lengths(case), tokens=torch.from_numpy(now).to(DEVICE),
                         next_tok=torch.empty(B, dtype=torch.int32, device=DEVICE),
                         logits=torch.empty(B, s.V, dtype=torch.float32, device=DEVICE),
                         fill=binding.D3_FILL_RECOMPUTE if case.get("fill") == "recompute" else binding.D3_FILL_COPY)
    if before is not None:
        dec.prefill(torch.from_numpy(before).to(DEVICE))
    if case["kind"] == "decode":
        begin, _ = _window(case)
        dec.set_plan_table([case["L"], case["keep"]], [0, begin])
        dec.set_fill_mode(st.fill)
    torch.cuda.synchronize()
    return st


def run(state):
    st, dec, case = state, state.dec, state.case
    if case["kind"] == "decode":
        dec.truncate(st.past)                       # back to the prompt: every pass is the first step after it
        dec.decode_step(st.tokens, 1, st.next_tok, logits=st.logits)
        if case["fill"] != "none":
            dec.fill_missing_kv(st.past, st.past + 1, st.fill)
    elif case["ragged"]:
        dec.prefill_ragged(st.tokens, st.lengths, next_tok=st.next_tok, logits=st.logits)
    else:
        if st.past:
            dec.truncate(st.past)
        dec.prefill(st.tokens, pos_begin=st.past, next_tok=st.next_tok, logits=st.logits)
    new = slice(st.past, st.rows)                   # the rows that the pass wrote, of every block and sequence
    return {"logits": st.logits, "k": dec.k_cache[:, :, :, new], "v": dec.v_cache[:, :, :, new]}


# ---------------- what a pass cannot do without ----------------

def work(case):
    s = _shape(case)
    B, wb, eb = case["B"], 4 if s.dtype == "f32" else 2, 4 if s.kv == "f32" else 2
    q, kv = s.H * s.hd, s.H_kv * s.hd
    block = (q + 2 * kv) * s.d + q * s.d + 3 * s.F * s.d
    row = 2 * kv * eb                               # K and V of one token in one block
    head_b, head_f = s.V * s.d * wb + B * s.V * 4, 2 * s.V * s.d * B
    if case["kind"] == "decode":
        keep, n, ctx = case["keep"], case["L"] - case["keep"], case["P"] + 1
        by = keep * (block * wb + B * ctx * row) + head_b + B * s.d * wb
        fl = keep * B * (2 * block + 4 * q * ctx) + head_f
        if case["fill"] == "copy":
            by += n * B * row
        elif case["fill"] == "recompute":
            by += n * (2 * kv * s.d * wb + B * row)
            fl += n * B * 4 * kv * s.d
        return {"bytes": by, "flops": fl}
    lens, past = _lengths(case), case["past"]
    tokens = sum(lens)
    pairs = sum(n * past + n * (n + 1) // 2 for n in lens)      # (query, visible row)
    return {"bytes": s.L * (block * wb + tokens * row + B * past * row) + head_b + tokens * s.d * wb,
            "flops": s.L * (2 * block * tokens + 4 * q * pairs) + head_f}


def tolerance(case):
    """About four times what the path is off from float64 (relative 2-norm, measured over these ranges): 2e-7 for the fp32
    model, 3e-5 with an fp32 cache (activations go into the matrix cores as two bf16 halves, 16 bits in all), 2e-3 with an
    fp16 cache (the rounding of its rows)."""
    if case["model"] == "tiny":
        return {"rel": 2e-6}
    return {"rel": 1.2e-4} if WIDTHS[case["model"]]["kv"] == "f32" else {"rel": 8e-3}


# ---------------- the same outputs in 64 bits ----------------

def exact(case, seed):
    s = _shape(case)
    w = _weights(s, seed)
    before, now = _tokens(case, s, seed)
    dt, B, past = torch.float64, case["B"], (case["P"] if case["kind"] == "decode" else case["past"])
    lens = [1] * B if case["kind"] == "decode" else _lengths(case)
    new = max(lens)
    freq = torch.tensor([s.rope_base ** (-2.0 * j / s.hd) for j in range(s.hd // 2)], dtype=dt, device=DEVICE)
    k_out = torch.zeros(s.L, B, s.H_kv, new, s.hd, dtype=dt, device=DEVICE)
    v_out = torch.zeros_like(k_out)

    def norm(x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.eps) * gain.to(dt)

    def rope(x, pos):                               # x [n, heads, hd]: dims j and j + hd/2 turn by pos * freq[j]
        a = pos.to(dt)[:, None] * freq
        c, n = torch.cos(a)[:, None], torch.sin(a)[:, None]
        lo, hi = x[..., :s.hd // 2], x[..., s.hd // 2:]
        return torch.cat([lo * c - hi * n, lo * n + hi * c], -1)

    def keys_values(wl, a, pos):                    # normalised rows -> [H_kv, n, hd]
        k = rope((a @ wl["wk"].T).view(-1, s.H_kv, s.hd), pos)
        return k.transpose(0, 1), (a @ wl["wv"].T).view(-1, s.H_kv, s.hd).transpose(0, 1)

    def block(wl, x, pos, k_past, v_past):          # one sequence: x [n, d]
        a = norm(x, wl["attn_norm"])
        k, v = keys_values(wl, a, pos)
        k = k if k_past is None else torch.cat([k_past, k], 1)
        v = v if v_past is None else torch.cat([v_past, v], 1)
        qh = rope((a @ wl["wq"].T).view(-1, s.H, s.hd), pos).transpose(0, 1)
        first = k.shape[1] - x.shape[0]
        seen = torch.arange(k.shape[1], device=DEVICE)[None, :] <= first + torch.arange(x.shape[0], device=DEVICE)[:, None]
        out, grp = torch.empty(s.H, x.shape[0], s.hd, dtype=dt, device=DEVICE), s.H // s.H_kv
        for h in range(s.H):
            sc = (qh[h] @ k[h // grp].T) / math.sqrt(s.hd)
            out[h] = torch.softmax(sc.masked_fill(~seen, -math.inf), -1) @ v[h // grp]
        x = x + out.transpose(0, 1).reshape(x.shape[0], -1) @ wl["wo"].T
        m = norm(x, wl["mlp_norm"])
        return x + (torch.nn.functional.silu(m @ wl["w_gate"].T) * (m @ wl["w_up"].T)) @ wl["w_down"].T, k, v

    emb = w["tok_emb"]
    old = None if before is None else [emb[torch.from_numpy(before[b]).to(DEVICE).long()].to(dt) for b in range(B)]
    cur = []
    for b in range(B):
        t = now[b:b + 1] if case["kind"] == "decode" else now[b, case["P"] - lens[b]:]
        cur.append(emb[torch.from_numpy(np.ascontiguousarray(t)).to(DEVICE).long()].to(dt))
    begin, dropped = _window(case) if case["kind"] == "decode" else (0, 0)
    entered = None                                  # the residual that entered the drop window
    for l in range(s.L):
        wl = {n: t.to(dt) for n, t in w["layers"][l].items()}
        skip = begin <= l < begin + dropped
        if l == begin:
            entered = [c.clone() for c in cur]
        for b in range(B):
            kp = vp = None
            if old is not None:
                old[b], kp, vp = block(wl, old[b], torch.arange(past, device=DEVICE), None, None)
            pos = torch.arange(past, past + lens[b], device=DEVICE)
            if not skip:
                cur[b], k, v = block(wl, cur[b], pos, kp, vp)
                k_out[l, b, :, new - lens[b]:], v_out[l, b, :, new - lens[b]:] = k[:, past:], v[:, past:]
            elif case["fill"] == "recompute":
                k_out[l, b], v_out[l, b] = keys_values(wl, norm(entered[b], wl["attn_norm"]), pos)
    if case["kind"] == "decode" and case["fill"] == "copy" and case["keep"]:
        src = begin - 1 if begin > 0 else dropped
        for l in range(begin, begin + dropped):
            k_out[l], v_out[l] = k_out[src], v_out[src]
    last = norm(torch.stack([c[-1] for c in cur]), w["final_norm"])
    return {"logits": last @ w["lm_head"].to(dt).T, "k": k_out, "v": v_out}
