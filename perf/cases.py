"""The work a rollout engine has this library do, as cases to be timed.

A case is one call path of the package's public interface with the sizes of
one step.  Sizes are those of the configurations in `workloads` and of the
benchmark, or generic ones in between.  Context lengths are evenly spread
quantiles of the case's distribution (so that a case costs the same whatever
the seed) in an order drawn from the seed; blocks are scattered over the pool.

Operations (`op`):
  decode     attention of `n` new tokens per sequence over the paged cache,
             through a bound call (n = 1: a decode step, a few: verification
             of drafted tokens, tens to hundreds: chunked prefill)
  append     the new token's K/V rows stored and the decode step, one call
  prefill    new prompts: the K/V rows of all their tokens appended, then
             causal attention over them (prompts are aligned to their end, so
             the first of the `n` rows of a shorter prompt see nothing)
  prefix     the decode step of parallel samples that share a prompt's blocks
  model      `layers` layers of append + decode replayed as one HIP graph
  logprob    token log-probabilities (and entropies) of LM-head logits
"""
import math

import numpy as np
import torch

import paper_2405_11143_amd as pda

BLOCK = 16


def listed():
    return [
        # The smallest step: a handful of short sequences, where the call itself is the cost.
        dict(name="decode_tiny", op="decode", batch=4, q_heads=8, kv_heads=2, head_dim=64, n=1,
             dist="uniform", lo=1, hi=257),
        # The end of a rollout: a few long samples are left in the batch.
        dict(name="append_few_long", op="append", batch=8, q_heads=32, kv_heads=8, head_dim=128, n=1,
             dist="loguniform", lo=512, hi=16384),
        # The headline decode step (Llama-3-8B shape).
        dict(name="decode_8b", op="decode", batch=256, q_heads=32, kv_heads=8, head_dim=128, n=1,
             dist="uniform", lo=512, hi=4096),
        # One GPU's share of a TP=8 Llama-3-70B layer: one KV head, split contexts.
        dict(name="decode_70b_tp8", op="decode", batch=512, q_heads=8, kv_heads=1, head_dim=128, n=1,
             dist="uniform", lo=1024, hi=8192),
        # Verification of four drafted tokens and the one after them.
        dict(name="verify_8b", op="decode", batch=256, q_heads=32, kv_heads=8, head_dim=128, n=5,
             dist="uniform", lo=512, hi=4096),
        # Small chunks of prompts or of long drafts over long contexts.
        dict(name="chunk64_long_cot", op="decode", batch=64, q_heads=32, kv_heads=8, head_dim=128, n=64,
             dist="loguniform", lo=1024, hi=16384),
        # Chunked prefill: 512 tokens of each prompt over what is cached.
        dict(name="chunked_prefill", op="decode", batch=32, q_heads=32, kv_heads=8, head_dim=128, n=512,
             dist="uniform", lo=1024, hi=8192),
        # New prompts of up to 1024 tokens (the paper's input limit), seven query heads per KV head.
        dict(name="prefill_prompts", op="prefill", batch=48, q_heads=28, kv_heads=4, head_dim=128, n=1024,
             dist="uniform", lo=64, hi=1024),
        # Parallel sampling: 32 prompts x 8 samples over shared prompt blocks.
        dict(name="shared_prefix", op="prefix", prompts=32, samples=8, prefix=1024, q_heads=32, kv_heads=8,
             head_dim=128, n=1, dist="uniform", lo=256, hi=8192),
        # A small batch's whole decode step as one graph.
        dict(name="model_step", op="model", batch=6, layers=16, q_heads=32, kv_heads=8, head_dim=128, n=1,
             dist="uniform", lo=64, hi=640),
        # Rollout: log-probabilities of the sampled tokens from fp32 logits.
        dict(name="logprob_rollout", op="logprob", rows=64, vocab=128256, dtype="f32", entropy=False,
             inv_temperature=1.0),
        # Training: log-probabilities and entropies of a micro-batch's tokens, bf16 logits.
        dict(name="logprob_train", op="logprob", rows=1500, vocab=151936, dtype="bf16", entropy=True,
             inv_temperature=1.0),
    ]


HEADS = [(8, 2, 64), (32, 8, 128), (8, 1, 128), (28, 4, 128), (40, 8, 128), (12, 2, 128), (16, 16, 64), (16, 1, 128)]
MOST_BYTES, MOST_FLOPS = 4.0e9, 1.1e12


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: operations in the shares they have above, sizes spread
    over the logarithm of their ranges, no more work than the largest listed."""
    op = rng.choice(["decode"] * 6 + ["append", "prefill", "prefix", "model"] + ["logprob"] * 2)
    if op == "logprob":
        return dict(op=op, rows=_log(rng, 1, 1600), vocab=_log(rng, 1000, 160000), dtype=rng.choice(["bf16", "f32"]),
                    entropy=rng.random() < 0.5, inv_temperature=round(rng.uniform(0.6, 1.6), 2))
    hq, hkv, d = rng.choice(HEADS)
    case = dict(op=op, q_heads=hq, kv_heads=hkv, head_dim=d, dist=rng.choice(["uniform", "loguniform"]))
    hi = _log(rng, 64, 16384)
    case["n"] = _log(rng, 1, 1024) if op == "decode" and rng.random() < 0.7 else 1
    if op == "prefill":
        hi = _log(rng, 64, 2048)
        case["n"] = hi
    hi = max(hi, case["n"])
    case["lo"], case["hi"] = max(1, min(hi, _log(rng, max(1, hi // 32), hi))), hi
    if op == "prefix":
        case["prompts"], case["samples"] = _log(rng, 1, 48), rng.randint(2, 20)
        case["prefix"] = BLOCK * _log(rng, 4, 128)
    else:
        case["batch"] = _log(rng, 1, 512)
    if op == "model":
        case["layers"], case["batch"] = rng.randint(2, 20), _log(rng, 1, 16)
        case["hi"] = min(case["hi"], 2048)
        case["lo"] = min(case["lo"], case["hi"])
    key = "prompts" if op == "prefix" else "batch"
    while case[key] > 1 and _too_much(case):
        case[key] = case[key] * 2 // 3
    while _too_much(case):
        case["hi"] = case["hi"] * 2 // 3
        case["n"] = min(case["n"], case["hi"])
        case["lo"] = min(case["lo"], case["hi"])
    return case


def _too_much(case):
    w = work(case)
    return w["bytes"] > MOST_BYTES or w["flops"] > MOST_FLOPS


# ------------------------------------------------------------------ sizes --

def _spread(case, count):
    """`count` evenly spread quantiles of the case's length distribution."""
    u = (np.arange(count) + 0.5) / count
    lo, hi = case["lo"], case["hi"]
    x = lo + u * (hi - lo) if case["dist"] == "uniform" else lo * (hi / lo) ** u
    return np.clip(np.rint(x), lo, hi).astype(np.int64)


def _batch(case):
    return case["prompts"] * case["samples"] if case["op"] == "prefix" else case["batch"]


def _lens(case, seed=None):
    """Context lengths: the case's quantiles, shuffled by the seed."""
    x = _spread(case, _batch(case)) + case.get("prefix", 0)
    return x if seed is None else np.random.RandomState(seed % (1 << 31)).permutation(x)


def work(case):
    if case["op"] == "logprob":
        size = 2 if case["dtype"] == "bf16" else 4
        r = case["rows"]
        return dict(bytes=r * case["vocab"] * size + r * (4 + 4 + (4 if case["entropy"] else 0)),
                    flops=4 * r * case["vocab"])
    lens = _lens(case)
    B, n, hq, hkv, d = len(lens), case["n"], case["q_heads"], case["kv_heads"], case["head_dim"]
    i = np.arange(n)
    visible = np.clip(lens[:, None] - n + 1 + i[None, :], 0, None).sum()
    tokens = lens.sum() - (case["prompts"] * (case["samples"] - 1) * case["prefix"] if case["op"] == "prefix" else 0)
    nbytes = 4 * tokens * hkv * d + 6 * B * n * hq * d + 4 * (-(-lens // BLOCK)).sum() + 4 * B
    if case["op"] in ("append", "prefill", "model"):  # new rows read and stored
        nbytes += 8 * np.minimum(lens, n).sum() * hkv * d
    layers = case.get("layers", 1)
    return dict(bytes=float(layers * nbytes), flops=float(layers * 4 * d * hq * visible))


# ----------------------------------------------------------------- inputs --

def _inputs(case, seed):
    """Everything on the GPU that the call reads, from the seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape, dtype=torch.bfloat16):
        return torch.randn(shape, generator=gen, device=dev, dtype=dtype)

    if case["op"] == "logprob":
        # A language model's logits: noise and a few tens of likely tokens, one of which is usually the sampled one.
        R, V = case["rows"], case["vocab"]
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        stride = -(-V // 8) * 8  # 16-byte rows
        logits = torch.empty(R, stride, dtype=dtype, device=dev)
        for r in range(0, R, 256):
            m = min(R, r + 256) - r
            x = normal(m, stride, dtype=torch.float32) * 2
            likely = torch.randint(V, (m, 32), generator=gen, device=dev)
            boost = 6 + 8 * torch.rand((m, 32), generator=gen, device=dev)
            logits[r:r + m] = x.scatter_add(1, likely, boost).to(dtype)
            pick = torch.where(torch.rand(m, generator=gen, device=dev) < 0.7, likely[:, 0],
                               torch.randint(V, (m,), generator=gen, device=dev))
            tokens = pick if r == 0 else torch.cat([tokens, pick])
        return dict(logits=logits, tokens=tokens.to(torch.int32))

    hq, hkv, d, n = case["q_heads"], case["kv_heads"], case["head_dim"], case["n"]
    lens = _lens(case, seed)
    B, layers = len(lens), case.get("layers", 1)
    blocks = -(-lens // BLOCK)
    shared = case.get("prefix", 0) // BLOCK
    total = int(blocks.sum()) - (case["prompts"] * (case["samples"] - 1) * shared if shared else 0)
    NB, width = int(math.ceil(1.1 * total)), int(blocks.max())
    perm = np.random.RandomState((seed + 1) % (1 << 31)).permutation(NB).astype(np.int32)
    table, used, prefix = np.full((B, width), -1, np.int32), 0, None
    for b in range(B):
        if shared and b % case["samples"] == 0:
            prefix, used = perm[used:used + shared], used + shared
        if shared:
            table[b, :shared] = prefix
        own = int(blocks[b]) - shared
        table[b, shared:blocks[b]] = perm[used:used + own]
        used += own
    # Keys carry an offset per head and channel, queries are sharper than unit normal: rows whose largest
    # weights stand out and whose running maximum moves, as trained attention has.
    k = normal(layers, NB, hkv, d // 8, BLOCK, 8)
    offset = (normal(layers, 1, hkv, d // 8, 1, 8) * 0.5)
    k += offset
    v = normal(layers, NB, hkv, BLOCK, d)
    q = normal(layers, B, n, hq, d) * 1.5
    out = dict(q=q, k=k, v=v, table=torch.from_numpy(table).to(dev), lens=torch.from_numpy(lens.astype(np.int32)).to(dev),
               host_lens=lens, host_table=table)
    if case["op"] in ("append", "prefill", "model"):
        out["k_new"] = normal(layers, B, n, hkv, d) + offset.permute(0, 1, 4, 2, 3, 5).reshape(layers, 1, 1, hkv, d)
        out["v_new"] = normal(layers, B, n, hkv, d)
    return out


def prepare(case, seed):
    x = _inputs(case, seed)
    dev = torch.device("cuda")
    if case["op"] == "logprob":
        call = pda.bind_token_logprobs(x["logits"], x["tokens"], case["inv_temperature"], case["entropy"], case["vocab"])
        return dict(op="logprob", call=call)
    scale, longest = 1.0 / math.sqrt(case["head_dim"]), int(x["host_lens"].max())
    q, k, v = x["q"], x["k"], x["v"]
    out = torch.empty(q.shape, dtype=torch.float32, device=dev)
    state = dict(op=case["op"], out=out, k=k, v=v)
    if case["op"] in ("decode", "append") and case["n"] == 1:
        q1, out1 = q[0, :, 0], out[0, :, 0]
    else:
        q1, out1 = q[0], out[0]
    step = (k[0], v[0], x["table"], x["lens"], scale)
    if case["op"] == "decode":
        state["call"] = pda.bind_decode(q1, *step, out1, max_context_len=longest)
    elif case["op"] == "append":
        state["call"] = pda.bind_decode_append(q1, x["k_new"][0], x["v_new"][0], *step, out1, max_context_len=longest)
    elif case["op"] == "prefill":
        state["store"] = pda.bind_append_kv(x["k_new"][0], x["v_new"][0], x["table"], x["lens"], k[0], v[0],
                                            max_context_len=longest, num_q_heads=case["q_heads"])
        state["call"] = pda.bind_decode(q1, *step, out1, max_context_len=longest)
    elif case["op"] == "prefix":
        P, S = case["prompts"], case["samples"]
        start = torch.arange(P + 1, dtype=torch.int32, device=dev) * S
        plen = torch.full((P,), case["prefix"], dtype=torch.int32, device=dev)
        B, width = x["table"].shape
        prob = pda.make_problem(B, case["q_heads"], case["kv_heads"], case["head_dim"], k.shape[1], width, longest)
        plan = pda.pda_plan_shared_prefix(prob, pda.make_prefix_groups(P, S, case["prefix"]))
        space = torch.empty(plan["workspace_bytes"], dtype=torch.uint8, device=dev)
        state["args"] = (q[0, :, 0], *step, start, plen, out[0, :, 0])
        state["more"] = dict(max_context_len=longest, max_group_size=S, max_prefix_len=case["prefix"], workspace=space)
    else:
        rows = [dict(q=q[i, :, 0], k_new=x["k_new"][i], v_new=x["v_new"][i], k_cache=k[i], v_cache=v[i],
                     out=out[i, :, 0]) for i in range(case["layers"])]
        state["graph"] = pda.ModelStepGraph(rows, x["table"], x["lens"], scale, max_context_len=longest)
    return state


def run(state):
    op = state["op"]
    if op == "logprob":
        logprobs, entropies = state["call"]()
        return dict(logprobs=logprobs, entropies=entropies)
    if op == "prefix":
        pda.pda_decode_shared_prefix(*state["args"], **state["more"])
    elif op == "model":
        state["graph"].launch()
    else:
        if op == "prefill":
            state["store"]()
        state["call"]()
    if op in ("decode", "prefix"):
        return dict(out=state["out"])
    return dict(out=state["out"], k=state["k"], v=state["v"])


# -------------------------------------------------------------- reference --

def tolerance(case):
    # Measured against exact(): the attention outputs (fp32, from bf16 inputs) are 2e-6 to 5e-6 off, the
    # log-probabilities up to 1e-7 and the entropies 2e-6 (fp32 sums over the vocabulary).
    if case["op"] == "logprob":
        return dict(rel=8e-6, max=8e-5)
    return dict(rel=2e-5, max=1e-3)


def exact(case, seed):
    x = _inputs(case, seed)
    f64 = torch.float64
    if case["op"] == "logprob":
        lp, ent = [], []
        for r in range(0, case["rows"], 128):
            z = x["logits"][r:r + 128, :case["vocab"]].to(f64) * float(np.float32(case["inv_temperature"]))
            logp = torch.log_softmax(z, dim=1)
            lp.append(logp.gather(1, x["tokens"][r:r + 128, None].long())[:, 0])
            ent.append(-(logp.exp() * logp).sum(1))
        return dict(logprobs=torch.cat(lp), entropies=torch.cat(ent) if case["entropy"] else None)
    hq, hkv, d, n = case["q_heads"], case["kv_heads"], case["head_dim"], case["n"]
    G, B, layers = hq // hkv, len(x["host_lens"]), case.get("layers", 1)
    scale = float(np.float32(1.0 / math.sqrt(d)))
    q, k, v = x["q"], x["k"], x["v"]
    dev = q.device
    if "k_new" in x:
        for b in range(B):
            L = int(x["host_lens"][b])
            t = torch.arange(max(0, L - n), L, device=dev)
            p, o = x["table"][b][t // BLOCK].long(), t % BLOCK
            kn = x["k_new"][:, b, n - len(t):]  # [layers][t][hkv][d]
            k[:, p, :, :, o] = kn.reshape(layers, len(t), hkv, d // 8, 8).permute(1, 0, 2, 3, 4)
            v[:, p, :, o] = x["v_new"][:, b, n - len(t):].permute(1, 0, 2, 3)
    out = torch.zeros(q.shape, dtype=f64, device=dev)
    for layer in range(layers):
        for b in range(B):
            L = int(x["host_lens"][b])
            ids = x["table"][b, :-(-L // BLOCK)].long()
            kb = k[layer, ids].permute(1, 0, 3, 2, 4).reshape(hkv, -1, d)[:, :L].to(f64)
            vb = v[layer, ids].permute(1, 0, 2, 3).reshape(hkv, -1, d)[:, :L].to(f64)
            first = max(0, n - L)  # rows before it see nothing
            limit = torch.arange(L - n + first, L, device=dev)[:, None, None]  # a row's own position
            hidden = torch.arange(L, device=dev)[None, None, :] > limit
            for g in range(hkv):
                qb = q[layer, b, first:, g * G:(g + 1) * G].to(f64)
                s = (qb.reshape(-1, d) @ kb[g].T).reshape(n - first, G, L) * scale
                s = torch.softmax(s.masked_fill(hidden, -math.inf), dim=2)
                out[layer, b, first:, g * G:(g + 1) * G] = (s.reshape(-1, L) @ vb[g]).reshape(n - first, G, d)
    if case["op"] in ("decode", "prefix"):
        return dict(out=out)
    return dict(out=out, k=k.to(f64), v=v.to(f64))
