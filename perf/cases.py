"""Performance cases of the mixed continuous-batching iteration.

Each case is one pass through the public entry points a serving program calls
for a layer (or a few layers) of one iteration: the one-launch append +
attention, the attention launch alone, the paged KV append, the dense
projections, and a whole iteration from its metadata to its completion time.
Shapes are the attention layers of Qwen3-0.6B / 8B / 32B (head_dim 128, 8 KV
heads, 16 / 32 / 64 query heads) and the projections of a Qwen3-0.6B layer
(hidden 1024, MLP 3072).  Queries, keys, values and activations are N(0, 1) in
bf16, weights N(0, 1 / fan_in); physical pages are a random permutation of the
pool.  The lengths of a case are fixed by the case, so its work is too; the
seed decides their order, the pages and every value.

Fields of a case (kind "attention"): hq / hkv heads; `decoders` sequences of
one new token with contexts spread over [ctx_lo, ctx_hi]; `chunk` prompt tokens
over a cached prefix of `prefix` tokens (0: no prompt); `out` the output type;
`append` whether the launch also writes the new keys and values.  Kind
"append": `tokens` new tokens of one prompt from position `prefix` on.  Kind
"linear": out[m][n] = x[m][k] w[n][k]^T with x rows `ldx` apart.  Kind
"iteration": `layers` layers, each with its projections around the attention,
with the sequences of an attention case.
"""
import math

import numpy as np
import torch

from paper_2609_38386_amd import dlfp
from paper_2609_38386_amd import runtime

HEAD_DIM = 128
PAGE = 16
SCALE = 1.0 / math.sqrt(HEAD_DIM)
HIDDEN, MLP = 1024, 3072          # a Qwen3-0.6B layer
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
# Position of token slot t inside a value page row (slots 4-7 and 8-11 trade places).
VALUE_POS = [(t & 3) | ((t & 4) << 1) | ((t & 8) >> 1) for t in range(PAGE)]


def _attention(hq, decoders, ctx_lo, ctx_hi, chunk, prefix, out="bf16", append=True, hkv=8):
    return {"kind": "attention", "hq": hq, "hkv": hkv, "decoders": decoders, "ctx_lo": ctx_lo,
            "ctx_hi": ctx_hi, "chunk": chunk, "prefix": prefix, "out": out, "append": append}


def _linear(m, n, k, ldx=0, out="bf16"):
    return {"kind": "linear", "m": m, "n": n, "k": k, "ldx": ldx or k, "out": out}


def listed():
    return [
        # The smallest mixed iteration: a nearly idle server, bound by launch and round trips.
        {"name": "tiny-mixed", **_attention(16, 4, 64, 256, 128, 384)},
        # Qwen3-0.6B serving between prompts: 32 decoders, no prompt in the batch.
        {"name": "0.6b-decode", **_attention(16, 32, 512, 2048, 0, 0)},
        # Qwen3-0.6B, a capped chunk in the middle of an 8192-token prompt beside its decoders.
        {"name": "0.6b-mixed", **_attention(16, 32, 512, 2048, 256, 3840)},
        # Qwen3-0.6B, the last uncapped chunk of a prompt with no decoder active.
        {"name": "0.6b-prefill", **_attention(16, 0, 0, 0, 2048, 6144)},
        # Qwen3-8B at its operating point, a prompt whose chunk is no multiple of anything.
        {"name": "8b-mixed", **_attention(32, 128, 1024, 8192, 1999, 7777)},
        # Qwen3-32B long-context serving, the largest chunk beside 256 decoders.
        {"name": "32b-mixed", **_attention(64, 256, 2048, 32768, 8192, 16384)},
        # Qwen3-32B prompt alone, attention launch after a separate append, fp32 output.
        {"name": "32b-prefill", **_attention(64, 0, 0, 0, 4096, 8192, out="fp32", append=False)},
        # The cache write of the two-launch form: an uncapped Qwen3-0.6B chunk.
        {"name": "append", "kind": "append", "hkv": 8, "tokens": 2048, "prefix": 4096},
        # Projections of a decode-only iteration: the query projection of 32 tokens.
        {"name": "linear-decode", **_linear(32, 2048, 1024)},
        # A mid-size iteration's down projection, which reads half of the gate/up rows.
        {"name": "linear-down", **_linear(545, 1024, 3072, ldx=6144)},
        # Gate/up projection at the batch budget of 8192 tokens.
        {"name": "linear-gate-up", **_linear(8192, 6144, 1024)},
        # A whole iteration with its projections, metadata and completion time.
        {"name": "0.6b-iteration", **dict(_attention(16, 32, 512, 2048, 512, 2048),
                                          kind="iteration", layers=4)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention"] * 6 + ["linear"] * 3 + ["append", "iteration"])
    if kind == "linear":
        n, k = rng.choice([(2048, 1024), (1024, 1024), (1024, 2048), (6144, 1024), (1024, 3072)])
        return _linear(_log_int(rng, 1, 8192), n, k, ldx=6144 if k == 3072 else 0,
                       out=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "append":
        return {"kind": "append", "hkv": 8, "tokens": _log_int(rng, 1, 8192),
                "prefix": rng.randint(0, 8192)}
    share = rng.choice(["mixed", "mixed", "decode", "prefill"])
    hq = rng.choice([16, 16, 32, 64]) if kind == "attention" else 16
    hkv = 8 if kind == "iteration" or rng.random() < 0.85 else hq
    lo = _log_int(rng, 16, 4096)
    decoders = 0 if share == "prefill" else _log_int(rng, 1, 256)
    # At most about 500k decode keys and 2 TFLOP, below the largest listed case.
    lo = min(lo, 400000 // max(decoders, 1))
    hi = max(lo + 1, min(8 * lo, 1000000 // max(decoders, 1) - lo))
    chunk = 0 if share == "decode" else _log_int(rng, 2, 8192)
    prefix = rng.randint(0, min(16384, 2 * 10 ** 12 // (512 * hq * max(chunk, 1))))
    case = _attention(hq, decoders, lo if decoders else 0, hi if decoders else 0, chunk,
                      prefix if chunk else 0, hkv=hkv, out=rng.choice(["bf16", "bf16", "fp32"]),
                      append=rng.random() < 0.75)
    if kind == "iteration":
        case.update(kind="iteration", layers=4, out="bf16", append=True)
        case["chunk"] = min(case["chunk"], 4096)
    return case


# ----------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _generator(seed, salt=0):
    return torch.Generator(device=_device()).manual_seed(1000003 * int(seed) + salt)


def _normal(shape, gen, scale=1.0):
    if scale == 1.0:
        return torch.empty(shape, dtype=torch.bfloat16, device=_device()).normal_(generator=gen)
    x = torch.empty(shape, dtype=torch.float32, device=_device()).normal_(generator=gen)
    return (x * scale).to(torch.bfloat16)


def _contexts(case):
    """Decoder contexts spread over the range, the new token included."""
    n, lo, hi = case["decoders"], case["ctx_lo"], case["ctx_hi"]
    return [max(1, int(lo + (hi - lo) * (i + 0.5) / n)) for i in range(n)]


def _sequences(case, seed):
    """(q_len, kv_len) of the packed batch (the prompt first) and its block table."""
    rng = np.random.default_rng(int(seed))
    q_len, kv_len = [], []
    if case["chunk"]:
        q_len.append(case["chunk"])
        kv_len.append(case["prefix"] + case["chunk"])
    contexts = _contexts(case)
    rng.shuffle(contexts)
    q_len += [1] * len(contexts)
    kv_len += contexts
    return np.array(q_len, np.int32), np.array(kv_len, np.int32), _block_table(kv_len, rng)


def _block_table(kv_len, rng):
    pages = [(n + PAGE - 1) // PAGE for n in kv_len]
    order = rng.permutation(sum(pages)).astype(np.int32)
    table = np.full((len(pages), max(pages)), -1, np.int32)
    at = 0
    for s, n in enumerate(pages):
        table[s, :n] = order[at:at + n]
        at += n
    return table


def _new_pool(blocks, hkv):
    return runtime.KVPool(blocks, hkv, _device())


class _PlainPool:
    """The same two tensors without the framework's class."""

    def __init__(self, blocks, hkv):
        self.k = torch.empty((blocks, hkv, PAGE, HEAD_DIM), dtype=torch.bfloat16, device=_device())
        self.v = torch.empty((blocks, hkv, HEAD_DIM, PAGE), dtype=torch.bfloat16, device=_device())


def _fill(pool, seed, layer=0):
    gen = _generator(seed, 7919 + layer)
    pool.k.normal_(generator=gen)
    pool.v.normal_(generator=gen)
    return pool


def _new_tokens(case, seed, tokens):
    gen = _generator(seed)
    q = _normal((tokens, case["hq"], HEAD_DIM), gen)
    k = _normal((tokens, case["hkv"], HEAD_DIM), gen)
    v = _normal((tokens, case["hkv"], HEAD_DIM), gen)
    return q, k, v


def _layer_weights(case, seed, layer, tokens):
    """A layer's input rows and its weights: query, key, value, output, gate/up, down."""
    gen = _generator(seed, 104729 + layer)
    hq, hkv = case["hq"] * HEAD_DIM, case["hkv"] * HEAD_DIM
    x = _normal((tokens, HIDDEN), gen)
    shapes = [(hq, HIDDEN), (hkv, HIDDEN), (hkv, HIDDEN), (HIDDEN, hq), (2 * MLP, HIDDEN),
              (HIDDEN, MLP)]
    return x, [_normal((n, k), gen, 1.0 / math.sqrt(k)) for n, k in shapes]


def _linear_inputs(case, seed):
    gen = _generator(seed)
    x = _normal((case["m"], case["ldx"]), gen)
    w = _normal((case["n"], case["k"]), gen, 1.0 / math.sqrt(case["k"]))
    return x[:, :case["k"]], w


# ----------------------------------------------------------------- the framework

def prepare(case, seed):
    dev = _device()
    s = {"kind": case["kind"]}
    if case["kind"] == "linear":
        s["x"], s["w"] = _linear_inputs(case, seed)
        s["y"] = torch.empty((case["m"], case["n"]), dtype=DTYPES[case["out"]], device=dev)
        return s
    if case["kind"] == "append":
        tokens, hkv = case["tokens"], case["hkv"]
        q_len = np.array([tokens], np.int32)
        kv_len = np.array([case["prefix"] + tokens], np.int32)
        table = _block_table(kv_len, np.random.default_rng(int(seed)))
        s["pool"] = _fill(_new_pool(table.shape[1], hkv), seed)
        s["batch"] = runtime.Batch(dlfp.make_dims(2 * hkv, hkv), q_len, kv_len, table,
                                   table.shape[1], dev)
        gen = _generator(seed)
        s["k_new"], s["v_new"] = (_normal((tokens, hkv, HEAD_DIM), gen) for _ in range(2))
        return s
    q_len, kv_len, table = _sequences(case, seed)
    blocks, tokens = int(table.max()) + 1, int(q_len.sum())
    dims = dlfp.make_dims(case["hq"], case["hkv"])
    s["workspace"] = runtime.Workspace(dev, 64 << 20)
    if case["kind"] == "attention":
        s["append"] = case["append"]
        s["pool"] = _fill(_new_pool(blocks, case["hkv"]), seed)
        s["batch"] = runtime.Batch(dims, q_len, kv_len, table, blocks, dev)
        s["q"], s["k_new"], s["v_new"] = _new_tokens(case, seed, tokens)
        s["y"] = torch.empty((tokens, case["hq"], HEAD_DIM), dtype=DTYPES[case["out"]], device=dev)
        return s
    # A serving loop's buffers: staging for the metadata, activations, a pool a layer.
    s.update(dims=dims, q_len=q_len, kv_len=kv_len, table=table, blocks=blocks)
    s["d_table"] = torch.from_numpy(table).to(dev)
    probe = dlfp.dlfp_build_varlen_meta(dims, q_len, kv_len, table, blocks)
    s["stage"] = runtime.StagedBatch(dims, len(q_len), tokens,
                                     probe.num_units + probe.num_append, dev)
    s["timer"] = dlfp.Timer()
    s["controller"] = dlfp.dlfp_controller_init(80.0, 3072, 1024, 6144)
    hq, hkv = case["hq"], case["hkv"]
    s["layers"] = []
    for layer in range(case["layers"]):
        x, weights = _layer_weights(case, seed, layer, tokens)

        def buf(*shape):
            return torch.empty(shape, dtype=torch.bfloat16, device=dev)

        s["layers"].append({
            "x": x, "w": weights, "pool": _fill(_new_pool(blocks, hkv), seed, layer),
            "q": buf(tokens, hq, HEAD_DIM), "k": buf(tokens, hkv, HEAD_DIM),
            "v": buf(tokens, hkv, HEAD_DIM), "attn": buf(tokens, hq, HEAD_DIM),
            "o": buf(tokens, HIDDEN), "gate_up": buf(tokens, 2 * MLP), "y": buf(tokens, HIDDEN)})
    return s


def run(state):
    s = state
    if s["kind"] == "linear":
        dlfp.dlfp_linear_bf16(s["x"], s["w"], s["y"])
        return s["y"]
    if s["kind"] == "append":
        s["batch"].append(s["pool"], s["k_new"], s["v_new"])
        return [s["pool"].k.view(torch.int16), s["pool"].v.view(torch.int16)]
    if s["kind"] == "attention":
        if s["append"]:
            s["batch"].append_attention(s["pool"], s["q"], s["k_new"], s["v_new"], SCALE, s["y"],
                                        s["workspace"])
            return [s["y"], s["pool"].k.view(torch.int16), s["pool"].v.view(torch.int16)]
        s["batch"].attention(s["pool"], s["q"], SCALE, s["y"], s["workspace"])
        return [s["y"]]
    # One iteration: metadata, the layers, the completion time, the next cap.
    st = s["stage"].build(s["q_len"], s["kv_len"], s["table"], s["blocks"])
    ws = s["workspace"].ensure(st.meta.workspace_bytes)
    s["timer"].start()
    for l in s["layers"]:
        rows = l["x"].shape[0]
        w_q, w_k, w_v, w_o, w_gu, w_d = l["w"]
        dlfp.dlfp_linear_bf16(l["x"], w_q, l["q"].view(rows, -1))
        dlfp.dlfp_linear_bf16(l["x"], w_k, l["k"].view(rows, -1))
        dlfp.dlfp_linear_bf16(l["x"], w_v, l["v"].view(rows, -1))
        dlfp.dlfp_append_attention_mixed(s["dims"], st.meta, st.d_work, s["d_table"], l["q"],
                                         l["k"], l["v"], l["pool"].k, l["pool"].v, SCALE,
                                         l["attn"], ws)
        dlfp.dlfp_linear_bf16(l["attn"].view(rows, -1), w_o, l["o"])
        dlfp.dlfp_linear_bf16(l["o"], w_gu, l["gate_up"])
        dlfp.dlfp_linear_bf16(l["gate_up"][:, :MLP], w_d, l["y"])
    s["timer"].stop()
    dlfp.dlfp_controller_step(s["controller"], 1, True, s["timer"].elapsed_ms())
    return [[l["attn"], l["y"], l["k"], l["v"]] for l in s["layers"]]


# ----------------------------------------------------------------- work and accuracy

def _attention_work(case):
    g_row = case["hq"] * HEAD_DIM
    kv_row = 2 * 2 * case["hkv"] * HEAD_DIM          # bytes of a token's key and value
    contexts, p, prefix = _contexts(case), case["chunk"], case["prefix"]
    tokens = p + len(contexts)
    keys = sum(contexts) + (prefix + p if p else 0)
    pairs = sum(contexts) + p * prefix + p * (p + 1) // 2
    out_bytes = 4 if case["out"] == "fp32" else 2
    data = keys * kv_row + tokens * g_row * (2 + out_bytes)
    if case["append"]:
        # The new keys and values come from their own buffers and go to the cache.
        data += tokens * kv_row
    return data, 4 * g_row * pairs


def _linear_work(m, n, k, out_bytes=2):
    return 2 * (m * k + n * k) + out_bytes * m * n, 2 * m * n * k


def work(case):
    if case["kind"] == "linear":
        data, flops = _linear_work(case["m"], case["n"], case["k"],
                                   4 if case["out"] == "fp32" else 2)
        return {"bytes": data, "flops": flops}
    if case["kind"] == "append":
        return {"bytes": 2 * case["tokens"] * 4 * case["hkv"] * HEAD_DIM, "flops": 0}
    data, flops = _attention_work(case)
    if case["kind"] == "iteration":
        tokens = case["chunk"] + case["decoders"]
        hq, hkv = case["hq"] * HEAD_DIM, case["hkv"] * HEAD_DIM
        for n, k in [(hq, HIDDEN), (hkv, HIDDEN), (hkv, HIDDEN), (HIDDEN, hq), (2 * MLP, HIDDEN),
                     (HIDDEN, MLP)]:
            d, f = _linear_work(tokens, n, k)
            data, flops = data + d, flops + f
        data, flops = case["layers"] * data, case["layers"] * flops
    return {"bytes": data, "flops": flops}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"
    # About four times the error measured against 64 bits: 1.7e-3 for a product
    # rounded to bf16, 2.3e-3 / 1.6e-3 for attention with bf16 / fp32 output
    # (probabilities are rounded to bf16), 4.2e-3 after a layer's chained products.
    if case["kind"] == "linear":
        return {"rel": 1e-5 if case["out"] == "fp32" else 7e-3}
    if case["kind"] == "iteration":
        return {"rel": 1.7e-2}
    return {"rel": 6.5e-3 if case["out"] == "fp32" else 1e-2}


def _gather(pool, blocks, n):
    """Logical keys and values [hkv][n][128] in 64 bits of one sequence."""
    at = torch.from_numpy(np.ascontiguousarray(blocks)).to(pool.k.device).long()
    k = pool.k[at].double()                                # [pages][hkv][16][128]
    v = pool.v[at].double()[..., VALUE_POS]                # [pages][hkv][128][16]
    hkv = k.shape[1]
    k = k.permute(1, 0, 2, 3).reshape(hkv, -1, HEAD_DIM)[:, :n].contiguous()
    v = v.permute(1, 0, 3, 2).reshape(hkv, -1, HEAD_DIM)[:, :n].contiguous()
    return k, v


def _exact_attention(case, seed, pool, q, k_new, v_new):
    """Masked softmax attention in 64 bits; k_new None: the cache holds every key."""
    q_len, kv_len, table = _sequences(case, seed)
    hq, hkv = case["hq"], case["hkv"]
    g = hq // hkv
    out = torch.empty((q.shape[0], hq, HEAD_DIM), dtype=torch.float64, device=q.device)
    row = 0
    for s in range(len(q_len)):
        p, n = int(q_len[s]), int(kv_len[s])
        k, v = _gather(pool, table[s, :(n + PAGE - 1) // PAGE], n)
        if k_new is not None:
            k[:, n - p:] = k_new[row:row + p].double().permute(1, 0, 2)
            v[:, n - p:] = v_new[row:row + p].double().permute(1, 0, 2)
        keys = torch.arange(n, device=q.device)
        for h in range(hkv):
            kt = k[h].t().contiguous()
            for t0 in range(0, p, 512):
                t1 = min(p, t0 + 512)
                end = n - p + t1
                qs = q[row + t0:row + t1, h * g:(h + 1) * g].double().reshape(-1, HEAD_DIM)
                sc = (qs @ kt[:, :end].contiguous()) * SCALE
                last = torch.arange(n - p + t0, end, device=q.device).repeat_interleave(g)
                sc.masked_fill_(keys[None, :end] > last[:, None], -math.inf)
                o = torch.softmax(sc, -1) @ v[h, :end]
                out[row + t0:row + t1, h * g:(h + 1) * g] = o.reshape(t1 - t0, g, HEAD_DIM)
        row += p
    return out


def exact(case, seed):
    if case["kind"] == "append":
        return None                                       # a bit copy
    if case["kind"] == "linear":
        x, w = _linear_inputs(case, seed)
        return x.double() @ w.double().t().contiguous()
    q_len, kv_len, table = _sequences(case, seed)
    blocks, tokens = int(table.max()) + 1, int(q_len.sum())
    if case["kind"] == "attention":
        pool = _fill(_PlainPool(blocks, case["hkv"]), seed)
        q, k, v = _new_tokens(case, seed, tokens)
        if not case["append"]:
            return [_exact_attention(case, seed, pool, q, None, None)]
        return [_exact_attention(case, seed, pool, q, k, v), None, None]
    got = []
    for layer in range(case["layers"]):
        pool = _fill(_PlainPool(blocks, case["hkv"]), seed, layer)
        x, (w_q, w_k, w_v, w_o, w_gu, w_d) = _layer_weights(case, seed, layer, tokens)

        def times(a, w):
            return a.double() @ w.double().t().contiguous()

        q = times(x, w_q).reshape(tokens, case["hq"], HEAD_DIM)
        k = times(x, w_k).reshape(tokens, case["hkv"], HEAD_DIM)
        v = times(x, w_v).reshape(tokens, case["hkv"], HEAD_DIM)
        attn = _exact_attention(case, seed, pool, q, k, v)
        y = times(times(times(attn.reshape(tokens, -1), w_o), w_gu)[:, :MLP], w_d)
        got.append([attn, y, k, v])
    return got
