"""What a user of this framework has it do, as cases that can be timed.

A case is one call sequence through the public entry points of the package on one batch of synthetic inputs:

  score    arb_score_steps with a router head: the drafted steps of a batch against their cached prefixes
  append   arb_score_steps without a head: the target's pass over an appended step
  decode   one token position of Algorithm 1's generation loop: the batch description of this position
           (DeviceBatch), arb_prefill with one new token per sequence, arb_next_token on the hidden states
  prefill  arb_prefill of whole prompts into an empty cache

Models are the repository's three shapes (workloads/configs.py) with random-init weights, bf16 or 4-bit.  Every layer
of a model does the same work, so the deep shapes are cut to a few layers: with N(0, 0.02) random weights a
perturbation grows with the square root of the depth, and at full depth (28 and 32 layers) two correct bf16
implementations already differ by 3 to 5 % in the final hidden states, which would hide a mistake.
"""
import math

import numpy as np
import torch

import paper_2512_05033_amd as A

# layers, d, query heads, kv heads, head dim, ffn, vocab, std of synthetic prefix keys and values
SHAPES = {
    "tiny": (2, 256, 4, 2, 64, 1024, 32000, 0.8),
    "router": (8, 1536, 12, 2, 128, 8960, 151936, 0.8),          # 8 of the 1.5B shape's 28 layers
    "target": (4, 4096, 32, 8, 128, 14336, 128256, 1.28),        # 4 of the 8B shape's 32 layers
}
BLOCK = 16


def _case(name, kind, shape, batch, prefix, step, **more):
    c = {"name": name, "kind": kind, "shape": shape, "bits": 16, "batch": batch, "prefix_lo": prefix[0],
         "prefix_hi": prefix[1], "step_lo": step[0], "step_hi": step[1], "alternate": False, "shuffled": True,
         "two_class": False, "last_token": False, "lengths_seed": 1}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: the tiny router of the parity workload, bound by launches
        _case("score-tiny-b4-s32", "score", "tiny", 4, (512, 512), (32, 32)),
        # one question at a time, the paper's own setting (batch size 1), with its head: two classes on the last token
        _case("score-router-b1-s37", "score", "router", 1, (1531, 1531), (37, 37), two_class=True, last_token=True),
        # the router over a serving batch: bench.py's headline workload
        _case("score-router-b16-s64", "score", "router", 16, (2048, 2048), (64, 64)),
        # long, ragged chains of thought at a large batch
        _case("score-router-b64-ragged", "score", "router", 64, (1024, 16384), (16, 128)),
        # drafting token by token with the 1.5B shape
        _case("decode-router-b16", "decode", "router", 16, (2048, 2048), (1, 1)),
        # the target regenerates the few escalated steps, token by token
        _case("decode-target-b5", "decode", "target", 5, (700, 3100), (1, 1)),
        # the weight-quantized 8B draft, token by token
        _case("decode-target-4bit-b16", "decode", "target", 16, (512, 1024), (1, 1), bits=4),
        # the same draft catching up with steps that the target wrote
        _case("append-target-4bit-b12", "append", "target", 12, (512, 2048), (16, 64), bits=4),
        # the target's pass over appended steps, contiguous cache
        _case("append-target-b8-s64", "append", "target", 8, (4096, 4096), (64, 64), shuffled=False),
        # long contexts, decode rows and appended steps mixed 1:1
        _case("append-target-b32-mix", "append", "target", 32, (4096, 32768), (1, 64), alternate=True),
        # the prompts of a batch of questions enter the router's cache
        _case("prefill-router-b16", "prefill", "router", 16, (0, 0), (100, 900)),
        # one long prompt enters the target's cache
        _case("prefill-target-b1-s3001", "prefill", "target", 1, (0, 0), (3001, 3001)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _span(rng, lo, hi):
    """An inclusive range of lengths inside [lo, hi]; one draw in three is a single length."""
    a, b = sorted((_log(rng, lo, hi), _log(rng, lo, hi)))
    return (b, b) if rng.random() < 1 / 3 else (a, b)


def _cost(c):
    w = work(c)
    return w["flops"] / 8e14 + w["bytes"] / 4e12


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        seed = rng.randrange(1, 1 << 30)
        k = rng.randrange(8)
        if k == 0:
            c = _case("", "score", "tiny", _log(rng, 1, 64), _span(rng, 64, 4096), _span(rng, 8, 128))
        elif k <= 2:
            c = _case("", "score", "router", _log(rng, 1, 64), _span(rng, 256, 16384), _span(rng, 8, 128),
                      two_class=rng.random() < 0.5, last_token=rng.random() < 0.5)
        elif k == 3:
            c = _case("", "decode", "router", _log(rng, 1, 64), _span(rng, 256, 8192), (1, 1))
        elif k == 4:
            c = _case("", "decode", "target", _log(rng, 1, 32), _span(rng, 256, 8192), (1, 1),
                      bits=rng.choice((4, 16)))
        elif k == 5:
            c = _case("", "append", "target", _log(rng, 1, 32), _span(rng, 512, 16384), _span(rng, 8, 96),
                      bits=rng.choice((4, 16, 16)), shuffled=rng.random() < 0.8)
        elif k == 6:
            c = _case("", "append", "target", _log(rng, 2, 32), _span(rng, 1024, 32768), (1, _log(rng, 8, 96)),
                      alternate=True)
        else:
            shape = rng.choice(("router", "target"))
            c = _case("", "prefill", shape, _log(rng, 1, 16 if shape == "router" else 4), (0, 0),
                      _span(rng, 64, 2048))
        c["lengths_seed"] = seed
        del c["name"]
        if _cost(c) <= most:
            return c


def _lengths(c):
    """Prefix and step lengths of the batch: part of the case, the same for every seed of the inputs."""
    r = np.random.default_rng(c["lengths_seed"])
    n = c["batch"]
    prefix = r.integers(c["prefix_lo"], c["prefix_hi"] + 1, size=n).astype(np.int32)
    if c["alternate"]:
        step = np.where(np.arange(n) % 2 == 0, c["step_lo"], c["step_hi"]).astype(np.int32)
    else:
        step = r.integers(c["step_lo"], c["step_hi"] + 1, size=n).astype(np.int32)
    return prefix, step


class _Weights:
    pass


def _make_weights(c, normal):
    L, d, hq, hkv, hd, f, vocab, _ = SHAPES[c["shape"]]
    w = _Weights()
    w.embed = normal((vocab, d), 0.02)
    w.wqkv = [normal(((hq + 2 * hkv) * hd, d), 0.02) for _ in range(L)]
    w.wo = [normal((d, hq * hd), 0.02) for _ in range(L)]
    w.wgu = [normal((2 * f, d), 0.02) for _ in range(L)]
    w.wd = [normal((d, f), 0.02) for _ in range(L)]
    gain = lambda: 1.0 + normal((d,), 0.1).float()
    w.g_attn, w.g_mlp, w.g_final = [gain() for _ in range(L)], [gain() for _ in range(L)], gain()
    w.w_head = normal((2, d) if c["two_class"] else (d,), 0.02).float()
    w.b_head = -0.5         # the log odds of the paper's label balance (38 % of the steps have class 1)
    return A.QuantizedWeights(w, c["bits"]) if c["bits"] < 16 else w


def prepare(case, seed):
    L, d, hq, hkv, hd, f, vocab, sigma = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    prefix, step = _lengths(case)
    cu = np.concatenate([[0], np.cumsum(step)]).astype(np.int32)
    need = (prefix + step + BLOCK - 1) // BLOCK
    n_blocks = int(need.sum())
    ids = np.random.default_rng(seed).permutation(n_blocks) if case["shuffled"] else np.arange(n_blocks)
    tables = np.zeros((case["batch"], int(need.max())), np.int32)
    at = 0
    for b in range(case["batch"]):
        tables[b, :need[b]] = ids[at:at + need[b]]
        at += need[b]
    tokens = torch.randint(0, vocab, (int(cu[-1]),), generator=gen, device="cuda", dtype=torch.int32)

    model = A.Model(n_layers=L, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=f, vocab=vocab,
                    weights=_make_weights(case, normal), has_router_head=case["kind"] == "score",
                    pool=A.ARB_POOL_LAST if case["last_token"] else A.ARB_POOL_MEAN)
    pool = (n_blocks, hkv, BLOCK, hd)
    kv = A.KVCache([normal(pool, sigma) for _ in range(L)], [normal(pool, sigma) for _ in range(L)])
    max_ctx = int((prefix + step).max())
    # Thresholds that a budget of few escalations gives.  They lie in the tail of these random scores, so that hardly
    # ever a score is within the bf16 results' distance of its threshold.
    tau = 0.95 if case["two_class"] else 2.0 if case["last_token"] else 0.5
    state = {"kind": case["kind"], "model": model, "kv": kv, "tau": tau,
             "ws": torch.empty(model.workspace_bytes(case["batch"], int(cu[-1]), max_ctx), dtype=torch.uint8,
                               device="cuda")}
    if case["kind"] == "decode":
        state.update(prefix=prefix, cu=cu, tables=tables, tokens=tokens, w_lm=normal((vocab, d), 0.02),
                     rows=torch.arange(case["batch"], dtype=torch.int32, device="cuda"))
    else:
        state["batch"] = A.DeviceBatch(prefix, cu, tables, tokens)
    return state


def run(state):
    model, kv, ws, kind = state["model"], state["kv"], state["ws"], state["kind"]
    out = {"k_pools": kv.k_pools, "v_pools": kv.v_pools}
    if kind == "score":
        out["scores"], out["escalate"], out["hidden"] = A.arb_score_steps(model, kv, state["batch"], state["tau"],
                                                                          want_hidden=True, ws=ws)
    elif kind == "append":
        _, _, out["hidden"] = A.arb_score_steps(model, kv, state["batch"], 0.0, want_hidden=True, ws=ws)
    elif kind == "prefill":
        out["hidden"] = A.arb_prefill(model, kv, state["batch"], want_hidden=True, ws=ws)
    else:
        batch = A.DeviceBatch(state["prefix"], state["cu"], state["tables"], state["tokens"])
        out["hidden"] = A.arb_prefill(model, kv, batch, want_hidden=True, ws=ws)
        # The greedy token's logit stands for the token: over random-init logits the largest two are often closer
        # than bf16 results of two correct implementations, so the index may differ where the logit does not.
        _, out["logit"] = A.arb_next_token(out["hidden"], state["rows"], state["w_lm"])
    return out


def work(case):
    L, d, hq, hkv, hd, f, vocab, _ = SHAPES[case["shape"]]
    prefix, step = (x.astype(np.float64) for x in _lengths(case))
    T = float(step.sum())
    per_layer = ((hq + 2 * hkv) * hd + hq * hd + 3 * f) * d
    weight_bytes = 2.0 if case["bits"] == 16 else 0.5 + 2.0 / 128
    kv_token = 2 * hkv * hd * 2                                     # bytes of one cached position and layer
    read = L * (per_layer * weight_bytes + float(prefix.sum()) * kv_token) + min(T, vocab) * d * 2
    written = L * T * kv_token + T * d * 2
    flops = L * (2.0 * T * per_layer + float((4 * hq * hd * (step * prefix + step * (step + 1) / 2)).sum()))
    if case["kind"] == "decode":
        read += vocab * d * 2
        flops += 2.0 * T * vocab * d
    return {"bytes": read + written, "flops": flops}


def tolerance(case):
    # Measured on the final hidden states by computing the same sequences as part of another batch, which changes the
    # tiles, the K splits and the key splits, i.e. the order of every sum and the roundings to bf16 behind it:
    # 2-norm 1.5 % at 8 layers of the 1.5B shape, 1.6 % at 4 layers of the 8B shape, 1.2 % at 2; largest difference
    # 0.08 of the root mean square.
    return {"rel": 0.03, "max": 0.4}
