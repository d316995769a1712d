"""The C ABI on a machine without a GPU: the library loads, exports every
function include/arb.h declares, and its host-side validation returns the
documented status codes before anything is launched."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import workloads as W
from helpers import REPLANNED, attention_plan, first_attention_chunk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2512_05033_amd import binding, build
    if not os.path.exists(build.LIB):
        build.build_library(verbose=False)
    return binding.load_library()


def declared_functions():
    text = open(os.path.join(ROOT, "include", "arb.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(arb_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    from paper_2512_05033_amd import binding
    names = declared_functions()
    assert "arb_prefill" in names and "arb_score_steps" in names and "arb_route" in names
    for n in names:
        assert getattr(lib, n) is not None
    assert sorted(binding.EXPORTS) == names


def _cfg(**over):
    from paper_2512_05033_amd.binding import _Cfg
    v = dict(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ffn=1024, vocab=32000,
             rms_eps=1e-6, rope_base=10000.0, kv_block=16, pool=0, has_router_head=1)
    v.update(over)
    return _Cfg(*[v[k] for k, _ in _Cfg._fields_])


def _weights(n_layers=2, head=True):
    from paper_2512_05033_amd.binding import _Weights
    arr = (C.c_void_p * n_layers)(*([0x1000] * n_layers))      # never dereferenced by arb_model_create
    return _Weights(0x1000, arr, arr, arr, arr, arr, arr, 0x1000, 0x1000 if head else None, 0.0), arr


def _create(lib, cfg, w):
    h = C.c_void_p()
    st = lib.arb_model_create(C.byref(cfg), C.byref(w), C.byref(h))
    return st, h


def test_model_create_validation(lib):
    from paper_2512_05033_amd import binding as B
    w, _keep = _weights()
    st, h = _create(lib, _cfg(), w)
    assert st == B.ARB_OK and h.value
    assert lib.arb_workspace_bytes(h, 4, 128, 544) > 128 * 256 * 4
    assert lib.arb_workspace_bytes(h, 4, -1, 544) == 0
    lib.arb_model_destroy(h)
    assert _create(lib, _cfg(n_q_heads=5), w)[0] == B.ARB_ESHAPE
    assert _create(lib, _cfg(head_dim=63), w)[0] == B.ARB_ESHAPE
    assert _create(lib, _cfg(n_layers=0), w)[0] == B.ARB_ESHAPE
    assert _create(lib, _cfg(head_dim=32, n_q_heads=8, n_kv_heads=4), w)[0] == B.ARB_EUNSUPPORTED
    assert _create(lib, _cfg(kv_block=32), w)[0] == B.ARB_EUNSUPPORTED
    assert _create(lib, _cfg(d_model=200), w)[0] == B.ARB_EUNSUPPORTED
    assert b"d_model" in lib.arb_last_error()
    assert _create(lib, _cfg(pool=7), w)[0] == B.ARB_EINVAL
    assert _create(lib, _cfg(has_router_head=3), w)[0] == B.ARB_EINVAL
    assert _create(lib, _cfg(has_router_head=B.ARB_HEAD_TWO_CLASS), w)[0] == B.ARB_OK
    wn, _k2 = _weights(head=False)
    assert _create(lib, _cfg(), wn)[0] == B.ARB_EINVAL
    assert _create(lib, _cfg(has_router_head=0), wn)[0] == B.ARB_OK
    assert lib.arb_model_create(None, None, None) == B.ARB_EINVAL
    # optional K-blocked gate/up copies: one pointer per layer or none at all
    wb, keep_b = _weights()
    wb.wgu_blocked = keep_b
    assert _create(lib, _cfg(), wb)[0] == B.ARB_OK
    holes = (C.c_void_p * 2)(0x1000, None)
    wb.wgu_blocked = holes
    assert _create(lib, _cfg(), wb)[0] == B.ARB_EINVAL and b"wgu_blocked" in lib.arb_last_error()
    assert lib.arb_pack_k_blocked(0x1000, 4, 48, 0x1000, None) == B.ARB_EUNSUPPORTED       # K % 32
    assert lib.arb_pack_k_blocked(None, 4, 64, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_pack_k_blocked(None, 0, 64, None, None) == B.ARB_OK


def test_batch_validation_happens_on_the_host(lib):
    """Bad descriptors are refused from the host copies of the lengths, before
    any device pointer is touched (all device pointers here are fake)."""
    from paper_2512_05033_amd import binding as B
    w, _keep = _weights()
    st, h = _create(lib, _cfg(), w)
    pools = (C.c_void_p * 2)(0x1000, 0x1000)
    kv = B._KV(pools, pools, 8)

    def call(prefix, cu, max_blocks, total=None, ws_bytes=1 << 30, scores=0x1000):
        p, c = np.asarray(prefix, np.int32), np.asarray(cu, np.int32)
        bt = B._Batch(len(p), int(c[-1]) if total is None else total, max_blocks, 0x1000, 0x1000, 0x1000, 0x1000,
                      p.ctypes.data, c.ctypes.data)
        return lib.arb_score_steps(h, C.byref(kv), C.byref(bt), 0.0, scores, None, None, 0x1000, ws_bytes, None)

    assert call([10, 10], [0, 4, 4], 4) == B.ARB_EINVAL            # empty step
    assert b"step" in lib.arb_last_error()
    assert call([10, 10], [1, 4, 8], 4) == B.ARB_EINVAL            # cu[0] != 0
    assert call([10, -1], [0, 4, 8], 4) == B.ARB_EINVAL            # negative prefix
    assert call([10, 10], [0, 4, 8], 4, total=9) == B.ARB_EINVAL   # total mismatch
    assert call([60, 10], [0, 5, 8], 4) == B.ARB_ECAPACITY         # 65 tokens need 5 blocks
    assert call([59, 10], [0, 5, 8], 4, ws_bytes=16) == B.ARB_ECAPACITY   # workspace too small
    assert call([10, 10], [0, 4, 8], 4, scores=None) == B.ARB_EINVAL      # head but no scores buffer
    assert lib.arb_route(None, -1, 0.0, 0, None, None) == B.ARB_EINVAL
    assert lib.arb_route(None, 0, 0.0, 0, None, None) == B.ARB_OK
    assert lib.arb_route(0x1000, 4, 0.0, 9, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_advantage_route(None, None, 0, 0.0, None, None, None, None, None) == B.ARB_OK
    assert lib.arb_advantage_route(None, 0x1000, 4, 0.0, None, 0x1000, None, None, None) == B.ARB_EINVAL
    assert lib.arb_advantage_route(0x1000, 0x1000, 4, 0.0, None, None, None, None, None) == B.ARB_EINVAL   # no output
    assert lib.arb_budget_threshold(0x1000, -1, 0, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_budget_threshold(0x1000, 4, 1, None, None) == B.ARB_EINVAL
    assert lib.arb_stage_layers(None, None, None, 0, 1, None, None, None, 0, None) == B.ARB_EINVAL
    # step bookkeeping of the decode loop
    assert lib.arb_step_advance(None, None, 0, 4, 8, 1, 2, None, None, None, None, None, None, None) == B.ARB_EINVAL   # no n_next
    assert lib.arb_step_advance(0x1000, 0x1000, 5, 4, 8, 1, 2, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_step_advance(0x1000, 0x1000, 2, 4, 0, 1, 2, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_step_advance(0x1000, None, 2, 4, 8, 1, 2, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_pack_steps(None, 8, None, None, 0, None, None) == B.ARB_OK
    assert lib.arb_pack_steps(0x1000, 0, 0x1000, 0x1000, 2, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_pack_steps(0x1000, 8, None, 0x1000, 2, 0x1000, None) == B.ARB_EINVAL
    assert lib.arb_stage_gemm(0x1000, 0x1000, None, 0x1000, 8, 128, 96, 0, None) == B.ARB_EUNSUPPORTED
    assert lib.arb_stage_gemm(0x1000, 0x1000, None, 0x1000, 8, 100, 128, 0, None) == B.ARB_EUNSUPPORTED
    lib.arb_model_destroy(h)


def test_launch_plan_of_the_projection_gemm_is_host_arithmetic(lib):
    """arb_gemm_large_tile_columns: whole rounds of 256 large tiles go to the large-tile kernel, the rest
    (or everything, when there is less than a round) to small tiles."""
    from paper_2512_05033_amd import binding as B
    cols = lambda M, N, K, e: lib.arb_gemm_large_tile_columns(M, N, K, e)
    # C2 gate/up: 4 x 70 large tiles -> one round of 4 x 64, 6 columns (768 features) left to small tiles
    assert cols(1024, 8960, 1536, B.ARB_EPI_SWIGLU_BF16) == 64
    # less than 205 large tiles: small tiles only
    assert cols(130, 64, 128, B.ARB_EPI_SWIGLU_BF16) == 0
    assert cols(1024, 2048, 1536, B.ARB_EPI_STORE_BF16) == 0
    # 13 x 16 = 208 large tiles: one round, at least 80 % full -> all 16 columns
    assert cols(3300, 4096, 256, B.ARB_EPI_STORE_BF16) == 16
    # 16 x 35 = 560: two rounds = 32 columns, the other 3 columns in small tiles
    assert cols(4000, 8960, 128, B.ARB_EPI_STORE_BF16) == 32
    # a width that is not a multiple of the large tile never uses it; bad sizes give 0
    assert cols(4000, 8960 + 128, 128, B.ARB_EPI_STORE_BF16) == 0
    assert cols(0, 4096, 256, B.ARB_EPI_STORE_BF16) == 0 and cols(-5, 4096, 256, B.ARB_EPI_STORE_BF16) == 0


def test_workspace_size_grows_with_every_argument(lib):
    w, _keep = _weights()
    st, h = _create(lib, _cfg(), w)
    base = lib.arb_workspace_bytes(h, 4, 128, 544)
    assert base > 0 and base % 256 == 0
    assert lib.arb_workspace_bytes(h, 4, 256, 544) > base
    assert lib.arb_workspace_bytes(h, 4, 128, 40000) > base            # more key splits to merge
    assert lib.arb_workspace_bytes(h, 4, 0, 0) >= 0
    lib.arb_model_destroy(h)


@pytest.mark.parametrize("d,hq,hkv,hd,F", [(1536, 12, 2, 128, 8960), (4096, 32, 8, 128, 14336),
                                           (128, 16, 4, 128, 256), (128, 64, 64, 64, 128)])      # QKV rows 24 and 96 times d_model wide
def test_scratch_of_a_call_per_token(lib, d, hq, hkv, hd, F):
    """What a call needs per step token does not grow with the width of the QKV projection beyond its bf16 row: h, x, q, k and
    v, attention output, SwiGLU output, position, slot, rotary row, head dot, splits, eight fp32 partial products."""
    from paper_2512_05033_amd import binding as B
    w, _keep = _weights()
    st, h = _create(lib, _cfg(d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=F), w)
    assert st == B.ARB_OK
    pools = (C.c_void_p * 2)(0x1000, 0x1000)
    kv = B._KV(pools, pools, 8)

    def need(T):                        # one sequence, nothing cached: a single key split; refused on the host
        p, c = np.zeros(1, np.int32), np.array([0, T], np.int32)
        bt = B._Batch(1, T, 16, 0x1000, 0x1000, 0x1000, 0x1000, p.ctypes.data, c.ctypes.data)
        assert lib.arb_score_steps(h, C.byref(kv), C.byref(bt), 0.0, 0x1000, None, None, 0x1000, 16, None) == B.ARB_ECAPACITY
        return int(re.search(rb"workspace 16 < (\d+) bytes", lib.arb_last_error()).group(1))

    token = 4 * d + 2 * d + 2 * (hq + 2 * hkv) * hd + 2 * hq * hd + 2 * F + 4 + 4 + 4 * hd + 4 + 4 + 32 * d
    for T in (200, 256):
        assert need(T) <= T * token + 12 * 256
    lib.arb_model_destroy(h)


def test_binding_refuses_to_run_without_the_library(tmp_path):
    from paper_2512_05033_amd import binding
    with pytest.raises(RuntimeError, match="no fallback"):
        binding.load_library(str(tmp_path / "libarb.so"))


def test_product_path_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2512_05033_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), f


def test_few_token_kernel_names_no_register_before_its_load_has_landed():
    """The compiler takes the outputs of an asm statement as written when it ends.  A load that is still in flight then can fill a
    register that has been copied, spilled or given to something else: each asm load of this kernel waits in its own statement."""
    text = open(os.path.join(ROOT, "paper_2512_05033_amd", "csrc", "gemm_few.hip")).read()
    loads = [a for a in re.findall(r"asm volatile\((.*?)\);", text, flags=re.S)
             if re.search(r"(ds_read|ds_load|global_load|buffer_load|flat_load)", a)]
    assert loads
    for a in loads:
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', a.split(": \"=")[0]))
        assert re.search(r"s_waitcnt [a-z]+cnt\(0\)$", code), a


def _internal(lib, mangled, argtypes, restype=C.c_bool):
    """A host function of the library that the header does not declare."""
    f = getattr(lib, mangled)
    f.argtypes, f.restype = argtypes, restype
    return f


@pytest.mark.parametrize("tokens", [1, 8, 16])
@pytest.mark.parametrize("d,hq,fused", [(1024, 1024, True), (1024, 3072, True), (1024, 4096, False), (1024, 8192, False),      # 64 workgroups
                                        (1280, 4096, True), (1408, 8192, False), (1536, 4096, True), (2048, 8192, True),       # 80, 88, 96, 128
                                        (4096, 4096, True), (4096, 8192, True),                    # one full round
                                        (4224, 4224, False), (5120, 2560, True), (5120, 5120, False), (6144, 1024, True),
                                        (6144, 6144, False), (7168, 4096, True), (8192, 8192, True)])
def test_fused_o_projection_only_where_it_is_the_faster_one(lib, tokens, d, hq, fused):
    """One workgroup per 16 features and CU, each over the whole K: not where idle CUs cost more than a norm kernel."""
    assert _internal(lib, "_Z14gemm_few_normsiiii", [C.c_int] * 4)(tokens, d, hq, 2048) == fused


@pytest.mark.parametrize("tokens", [1, 8, 16])
@pytest.mark.parametrize("d,rows,fused", [(1024, 1280, True), (1024, 10240, True), (1536, 2048, True), (4096, 6144, True), (4096, 10240, True),
                                          (6144, 8192, True), (6144, 5120, False), (6656, 7680, True), (7168, 2560, True),
                                          (7168, 9216, False), (8192, 2560, True), (8192, 1280, False), (8192, 10240, False)])
def test_fused_qkv_projection_only_where_it_is_the_faster_one(lib, tokens, d, rows, fused):
    """K is not split there: not where the workgroups' uneven shares of the rows cost more than a rotary kernel."""
    assert _internal(lib, "_Z16gemm_few_rotatesiii", [C.c_int] * 3)(tokens, rows, d) == fused


def _items(m, plan, prefix, steps):
    """(sequence, split, kv head, query tile) with at least one visible key, as the work list counts them."""
    n = 0
    for p, s in zip(prefix, steps):
        parts = -(-(p + s) // plan.kv_chunk)
        part = -(-(-(-(p + s) // parts)) // 64) * 64
        tiles = -(-s * m.group // 128)
        for begin in range(0, p + s, part):
            n += (tiles - (max(0, begin - p) * m.group) // 128) * m.n_kv_heads
    return n


@pytest.mark.parametrize("m,prefix,steps", REPLANNED)
def test_the_attention_planner_leaves_its_first_choice(lib, m, prefix, steps):
    """Each of these batches is cut otherwise than the number of places alone would have it."""
    plan, first = attention_plan(lib, m, prefix, steps), first_attention_chunk(m, prefix, steps)
    assert plan.kv_chunk != first


def test_the_attention_planner_never_needs_more_scratch_than_its_first_choice(lib):
    """Whatever the estimates say: whole tiles of keys, no more splits than the first choice needs (a caller's scratch is sized by them),
    and the items that belong to the chunk."""
    r = np.random.default_rng(17)
    moved = 0
    for m in (W.TINY, W.ROUTER_1P5B, W.TARGET_8B):
        for _ in range(150):
            n = int(r.integers(1, 40))
            prefix = [int(v) for v in r.integers(0, int(np.exp(r.uniform(3, 10.5))), n)]
            steps = [int(v) for v in r.integers(1, int(r.choice([2, 9, 129])), n)]
            plan, first = attention_plan(lib, m, prefix, steps), first_attention_chunk(m, prefix, steps)
            longest = max(p + s for p, s in zip(prefix, steps))
            moved += plan.kv_chunk != first
            assert plan.kv_chunk % 64 == 0 and plan.max_splits == -(-longest // plan.kv_chunk) <= -(-longest // first)
            assert plan.max_splits <= _internal(lib, "_Z20attention_splits_capi", [C.c_int], C.c_int)(longest)
            assert plan.n_items == _items(m, plan, prefix, steps)
    assert moved >= 20
