"""The entry point that allocates nothing (arb_score_steps_noalloc: workspace in a static device
array) against arb_score_steps with a caller workspace: same kernels, so the same bits; two calls
in a row, the second on a smaller batch, so that the array still holds the first call's contents."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05033_amd as A
    A.load_library()
    return A


def _both(A, sess, dbatch, B, T):
    """One call of each entry point on the same inputs -> ((scores, escalate, hidden), (same)), all on the host."""
    import harness  # noqa: F401
    d = sess.workload.model.d_model
    out = []
    for noalloc in (False, True):
        scores = torch.full((B,), float("nan"), device="cuda")
        esc = torch.full((B,), 7, dtype=torch.uint8, device="cuda")
        hidden = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
        if noalloc:
            A.arb_score_steps_noalloc(sess.model, sess.kv, dbatch, sess.batch.tau, scores=scores, escalate=esc, hidden=hidden)
        else:
            A.arb_score_steps(sess.model, sess.kv, dbatch, sess.batch.tau, ws=sess.ws, scores=scores, escalate=esc, hidden=hidden)
        torch.cuda.synchronize()
        out.append((scores.cpu().numpy(), esc.cpu().numpy(), W.bf16_bits(hidden)))
    return out


@pytest.mark.parametrize("w", [W.scaled(W.C1, batch=4), W.scaled(W.C2, n_layers=2, batch=2)], ids=["tiny", "router-shape"])
def test_noalloc_matches_the_workspace_entry_point_twice_in_a_row(A, w):
    import harness
    sess = harness.setup(w, "cuda", gain_jitter=0.1)
    batch = sess.batch
    ref, got = _both(A, sess, sess.dbatch, batch.batch, batch.total_tokens)
    assert np.isfinite(ref[0]).all() and set(np.unique(ref[1])) <= {0, 1}
    for r, g in zip(ref, got):
        assert np.array_equal(r, g)
    # a smaller batch next: the last sequence alone, then the first two with shorter steps
    for rows in ([batch.batch - 1], [0, 1]):
        sub = batch.select(rows)
        if len(rows) == 2:
            keep = np.maximum(sub.step_lens // 2, 1)
            tok = np.concatenate([sub.token_ids[sub.cu_step_lens[i]:sub.cu_step_lens[i] + keep[i]] for i in range(2)])
            sub = W.Batch(sub.prefix_lens, np.concatenate([[0], np.cumsum(keep)]).astype(np.int32), sub.block_tables,
                          tok.astype(np.int32), sub.n_blocks, sub.kv_block, sub.tau, sub.spare_blocks)
        ref, got = _both(A, sess, harness.device_batch(sub), sub.batch, sub.total_tokens)
        for r, g in zip(ref, got):
            assert np.array_equal(r, g)


def test_noalloc_rejects_what_does_not_fit(A):
    """The full 1.5B-router batch (1024 step tokens) needs more than the static array holds."""
    import harness
    w = W.scaled(W.C2, n_layers=1)
    sess = harness.setup(w, "cuda")
    need = sess.model.workspace_bytes(sess.batch.batch, sess.batch.total_tokens, sess.dbatch.max_ctx)
    assert need > A.NOALLOC_SCRATCH_BYTES
    B, T = sess.batch.batch, sess.batch.total_tokens
    scores = torch.zeros(B, device="cuda"); esc = torch.zeros(B, dtype=torch.uint8, device="cuda")
    with pytest.raises(A.ArbError) as e:
        A.arb_score_steps_noalloc(sess.model, sess.kv, sess.dbatch, 0.0, scores=scores, escalate=esc)
    assert e.value.status == A.ARB_ECAPACITY and "ARB_NOALLOC_SCRATCH_BYTES" in str(e.value)
    torch.cuda.synchronize()


def test_noalloc_without_room_for_the_work_list_is_bit_identical(A):
    """Several hundred one-token steps against 100000 cached tokens each (the sequences share one prefix's blocks): as
    many as fit the array without the attention work list, which then does not (one sequence more is refused, so less
    than a token's share is free, and the list is larger than that).  The same splits of the keys, so the same bits."""
    import harness
    w = W.scaled(W.C2, n_layers=1, batch=1)
    m, ctx, blk = w.model, 100000, 16
    hq, splits = m.n_q_heads * m.head_dim, -(-ctx // 6144)         # decode steps: 6144 keys per split
    # h, x, q, attn, act, position, slot, rotary row, head dot, eight partial products; splits of the token, partial results
    token = (4 * m.d_model + 2 * m.d_model + 2 * hq + 2 * hq + 2 * m.d_ffn + 4 + 4 + 4 * m.head_dim + 4 + 32 * m.d_model +
             4 + splits * m.n_q_heads * (2 * m.head_dim + 8))
    most = A.NOALLOC_SCRATCH_BYTES // token                        # the areas' alignment (256 bytes) may cost one more
    n_shared = (ctx - 1) // blk
    gen = torch.Generator(device="cuda").manual_seed(5)
    pool = lambda: [torch.empty(n_shared + most + 1, m.n_kv_heads, blk, m.head_dim, dtype=torch.bfloat16, device="cuda").normal_(0, 0.8, generator=gen)]
    kv = A.KVCache(pool(), pool())
    model = harness.make_model(m, W.make_weights(m, 3, "cuda"))

    def noalloc(B):
        tables = np.empty((B, n_shared + 1), np.int32)
        tables[:, :n_shared] = np.arange(n_shared)
        tables[:, n_shared] = n_shared + np.arange(B)
        db = A.DeviceBatch(np.full(B, ctx - 1, np.int32), np.arange(B + 1, dtype=np.int32), tables,
                           np.arange(B, dtype=np.int32) * 7)
        out = (torch.empty(B, device="cuda"), torch.empty(B, dtype=torch.uint8, device="cuda"),
               torch.empty(B, m.d_model, dtype=torch.bfloat16, device="cuda"))
        A.arb_score_steps_noalloc(model, kv, db, 0.0, scores=out[0], escalate=out[1], hidden=out[2])
        return db, out

    B = most
    try:
        db, got = noalloc(B)
    except A.ArbError as e:
        assert e.status == A.ARB_ECAPACITY
        B -= 1
        db, got = noalloc(B)
    with pytest.raises(A.ArbError) as e:
        noalloc(B + 1)
    assert e.value.status == A.ARB_ECAPACITY
    assert 32 * B * splits * m.n_kv_heads > token + 16 * 256       # bytes of the list against what is free
    for g, r in zip(got, A.arb_score_steps(model, kv, db, 0.0, want_hidden=True)):
        assert torch.equal(g, r)
