"""Glue between the seeded workloads and the oracle's plain-array interface."""
from __future__ import annotations

import ctypes as C

import numpy as np

import workloads as W
from oracle import arb_oracle as O


# Hidden-state bars (max|got - ref| / max|ref| over the output tensor).  2e-2 is the stated bar.  A deep model
# with random weights amplifies perturbations: rounding nothing but the operands of the matrix products to bf16
# (inside otherwise exact fp64 arithmetic: forward_bf16_operands below, built from the oracle's own functions)
# already moves the output of the 28-layer 1.5B-class shape by 2e-2 to 2.7e-2, depending on the sample.  So an
# end-to-end run at full depth measures that floor on its own sample and is held to
# max(2e-2, FLOOR_FACTOR x floor); every layer is also checked on its own, from the oracle's residual stream,
# against the stated 2e-2.
HIDDEN_TOL, SCORE_TOL, FLOOR_FACTOR = 2e-2, 1e-2, 1.3


def round_bf16(x: np.ndarray) -> np.ndarray:
    return O.bf16_to_float(O.float_to_bf16(x))


def forward_bf16_operands(m: O.Model, p: O.Params, kp, vp, token_ids, prefix_lens, cu_step_lens, block_tables,
                          rnd, depths, progress=None):
    """The oracle's forward, stage by stage, with `rnd` applied to the inputs of the matrix products
    (normed activations, rotated queries, attention output, SwiGLU output).  Returns the final-normed
    hidden states after each depth in `depths`.  With rnd = identity it is O.forward (tested)."""
    blk, Hq, Hkv, hd = m.kv_block, m.n_q_heads, m.n_kv_heads, m.head_dim
    pl, cu, bt = prefix_lens, cu_step_lens, block_tables
    pos, slots = O.positions(pl, cu), O.slot_mapping(pl, cu, bt, blk)
    h = O.embed(p.embed, token_ids)
    T, out = h.shape[0], {}
    for l in range(m.n_layers):
        x = rnd(O.rmsnorm(h, p.g_attn[l], m.rms_eps))
        qkv = (x @ O.as_float(p.wqkv[l]).T).reshape(T, Hq + 2 * Hkv, hd)
        q = rnd(O.rope(qkv[:, :Hq], pos, m.rope_base))
        O.kv_append(kp[l], vp[l], slots, O.rope(qkv[:, Hq:Hq + Hkv], pos, m.rope_base), qkv[:, Hq + Hkv:], blk)
        o = rnd(O.append_attention(q, kp[l], vp[l], pl, cu, bt, blk))
        h = h + o.reshape(T, Hq * hd) @ O.as_float(p.wo[l]).T
        gu = rnd(O.rmsnorm(h, p.g_mlp[l], m.rms_eps)) @ O.as_float(p.wgu[l]).T
        F = gu.shape[1] // 2
        h = h + rnd(O.silu(gu[:, :F]) * gu[:, F:]) @ O.as_float(p.wd[l]).T
        if l + 1 in depths:
            out[l + 1] = O.rmsnorm(h, p.g_final, m.rms_eps)
        if progress:
            progress(l + 1)
    return out


def oracle_model(m: W.ModelShape) -> O.Model:
    return O.Model(m.n_layers, m.d_model, m.n_q_heads, m.n_kv_heads, m.head_dim, m.d_ffn, m.vocab,
                   m.rms_eps, m.rope_base, m.kv_block)


def oracle_params(w: W.Weights) -> O.Params:
    bits = W.bf16_bits
    f32 = lambda t: t.detach().cpu().numpy().astype(np.float64)
    return O.Params(embed=bits(w.embed), wqkv=[bits(t) for t in w.wqkv], wo=[bits(t) for t in w.wo],
                    wgu=[bits(t) for t in w.wgu], wd=[bits(t) for t in w.wd],
                    g_attn=[f32(t) for t in w.g_attn], g_mlp=[f32(t) for t in w.g_mlp],
                    g_final=f32(w.g_final), w_head=f32(w.w_head), b_head=w.b_head)


def oracle_pools(ks, vs):
    return [W.bf16_bits(k).copy() for k in ks], [W.bf16_bits(v).copy() for v in vs]


def rel_err(got: np.ndarray, ref: np.ndarray) -> float:
    """max|got - ref| / max|ref| over the tensor."""
    return float(np.max(np.abs(got.astype(np.float64) - ref)) / np.max(np.abs(ref)))


def rms_err(got: np.ndarray, ref: np.ndarray) -> float:
    """sqrt(mean (got - ref)^2 / mean ref^2)."""
    return float(np.sqrt(np.mean((got.astype(np.float64) - ref) ** 2) / np.mean(ref ** 2)))


class AttentionPlan(C.Structure):
    _fields_ = [("kv_chunk", C.c_int), ("max_splits", C.c_int), ("max_qtiles", C.c_int), ("n_items", C.c_int)]


def attention_plan(lib, m: W.ModelShape, prefix, steps) -> AttentionPlan:
    """What the library plans for an attention launch over this batch (a host function that the header does not declare)."""
    f = lib._Z14plan_attentioniPKiS0_iii
    f.restype, f.argtypes = AttentionPlan, [C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int]
    p, cu = np.asarray(prefix, np.int32), np.concatenate([[0], np.cumsum(steps)]).astype(np.int32)
    return f(len(p), p.ctypes.data, cu.ctypes.data, m.group, m.n_kv_heads, m.head_dim)


def first_attention_chunk(m: W.ModelShape, prefix, steps) -> int:
    """Keys per split before any estimate: about 512 workgroups, between 256 keys and 4096 (6144 where every step is one wave)."""
    keys = sum(-(-s * m.group // 128) * m.n_kv_heads * (p + s) for p, s in zip(prefix, steps))
    chunk = -(-(keys // 512) // 64) * 64
    chunk = max(256, min(chunk, 6144 if max(steps) * m.group <= 32 else 4096))
    longest = max(p + s for p, s in zip(prefix, steps))
    while longest > 64 * chunk:
        chunk += 64
    return chunk


# Batches for which the planner leaves that choice.
REPLANNED = [
    (W.ROUTER_1P5B, [16384], [64]),                          # one long context
    (W.TARGET_8B, [2048] * 16, [1] * 16),                    # one token each: a full round instead of a round and a quarter
    (W.ROUTER_1P5B, [2048] * 16, [1] * 16),
    (W.ROUTER_1P5B, [3119, 4555, 5707, 305, 950, 4955], [94, 25, 31, 87, 42, 28]),       # ragged
    (W.TARGET_8B, [5002, 3954, 2229], [9, 70, 35]),
    (W.TINY, [3060, 1467, 3282, 4631, 901, 1897, 1907, 4806, 3517, 2456, 4768], [97, 15, 89, 23, 64, 94, 40, 66, 36, 76, 49])]
