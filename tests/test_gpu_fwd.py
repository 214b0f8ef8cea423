"""GPU parity: sfa_attn_fwd (fed by sfa_topk_encode) against the oracle.

The GPU path codes dense Q and K with its own encoder; the oracle codes the
same dense inputs with its own Top-k and evaluates the plain definition in
float64.  Tolerances: helpers.TOL_* (O 1e-5 float32 path, 5e-3 bf16-V path,
LSE 1e-4)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2603_22300_amd as sfa
import sfa_inputs as si
from helpers import (TOL_LSE, TOL_O_BF16V, TOL_O_F32, check_lse, check_o, np_vals,
                     sample_rows)

pytestmark = pytest.mark.gpu
DEV = "cuda"
_MAXF = float(np.finfo(np.float32).max)
_LN2 = math.log(2.0)


def _gpu_codes(x, k, idx_dtype=torch.int32, val_dtype=torch.float32):
    return sfa.sfa_topk_encode(x, k, idx_dtype=idx_dtype, val_dtype=val_dtype)


def _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed, idx_dtype=torch.int32,
              val_dtype=torch.float32, zipf_s=0.0, fwd=None, scale=None):
    fwd = fwd or sfa.sfa_attn_fwd
    q, kk, v = si.dense_qkv(B, Hq, Hkv, n, d, seed,
                            v_dtype=torch.bfloat16 if v_bf16 else torch.float32, device=DEV)
    if zipf_s:
        for b in range(B):
            for h in range(Hq):
                perm = si.zipf_feature_perm(d, seed, h // (Hq // Hkv))
                i_, v_ = si.zipf_codes(n, d, k, zipf_s, perm, seed, "q", b, h, device=DEV)
                q[b, h] = si.dense_from_codes(i_, v_, d)
            for h in range(Hkv):
                perm = si.zipf_feature_perm(d, seed, h)
                i_, v_ = si.zipf_codes(n, d, k, zipf_s, perm, seed, "k", b, h, device=DEV)
                kk[b, h] = si.dense_from_codes(i_, v_, d)
    qi, qv = _gpu_codes(q, k, idx_dtype, val_dtype)
    ki, kv = _gpu_codes(kk, k, idx_dtype, val_dtype)
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    o32, lse = fwd(qi, qv, ki, kv, v, causal=causal, scale=scale, o_dtype=torch.float32)
    ob16 = None
    if v_bf16:
        ob16, _ = fwd(qi, qv, ki, kv, v, causal=causal, scale=scale, o_dtype=torch.bfloat16,
                      want_lse=False)
    torch.cuda.synchronize()
    # oracle: its own codes of the same dense inputs
    qn, kn, vn = q.cpu().numpy(), kk.cpu().numpy(), np_vals(v)
    if val_dtype == torch.bfloat16:
        oqi, oqv = oracle.topk_encode_bf16(qn, k)
        oki, okv = oracle.topk_encode_bf16(kn, k)
    else:
        oqi, oqv = oracle.topk_encode(qn, k)
        oki, okv = oracle.topk_encode(kn, k)
    O, L = oracle.attn_fwd(oqi, oqv, oki, okv, vn, d, scale, causal)
    tol = TOL_O_BF16V if v_bf16 else TOL_O_F32
    eo = check_o(o32, O, tol, "O (float32 output)")
    el = check_lse(lse, L, "LSE")
    if ob16 is not None:
        check_o(ob16, O, tol, "O (bf16 output)")
    return eo, el


def test_tiny_workload_fp32():
    w = si.workload("tiny")
    _run_case(w.B, w.Hq, w.Hkv, w.n, w.d, w.k, w.causal, w.v_bf16, w.seed)


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,v_bf16",
    [
        (1, 1, 1, 1, 64, 8, True, False),      # n = 1
        (1, 1, 1, 37, 64, 8, True, False),     # one ragged tile
        (2, 2, 2, 130, 64, 16, True, True),    # ragged tail past two tiles
        (1, 4, 1, 200, 128, 16, True, True),   # GQA 4:1, d = 128
        (1, 8, 1, 100, 128, 16, True, True),   # GQA 8:1 (two heads per wave)
        (1, 2, 1, 257, 128, 8, False, True),   # non-causal
        (1, 1, 1, 300, 64, 1, True, True),     # k = 1
        (1, 2, 2, 150, 64, 64, True, False),   # k = d: dense attention
        (1, 2, 1, 129, 128, 64, True, True),   # largest supported k at d = 128
        (2, 4, 2, 96, 128, 16, False, False),  # float32 V, GQA 2:1
        (1, 16, 1, 70, 64, 8, True, True),     # 16 heads per KV head
        (1, 2, 2, 140, 128, 128, True, True),  # k = d = 128
        (1, 8, 2, 700, 128, 16, True, True),   # GQA 4:1 over eleven key tiles
        (1, 2, 2, 333, 128, 16, True, False),  # float32 V, causal, ragged
    ])
def test_shapes(B, Hq, Hkv, n, d, k, causal, v_bf16):
    _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed=B * 1000 + Hq * 100 + n)


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,v_bf16",
    [
        (1, 1, 1, 37, 64, 8, True, False),
        (2, 2, 2, 130, 64, 16, True, True),
        (1, 4, 1, 200, 128, 16, True, True),
        (1, 2, 1, 257, 128, 8, False, True),
        (1, 2, 2, 150, 64, 64, True, False),
        (1, 16, 1, 70, 64, 8, True, True),
        (1, 2, 1, 300, 128, 32, True, True),   # d = 128, 16 < k <= 64 (the k <= 64 tables)
        (1, 2, 2, 200, 128, 64, True, True),   # d = 128, k = 64, the largest supported
        (1, 32, 1, 150, 128, 16, True, True),  # 32 heads per KV head (4 rows per head and block)
        (1, 128, 1, 70, 128, 8, True, True),   # 128 heads per KV head (1 row per head and block)
        (1, 4, 2, 1000, 128, 4, True, True),   # small k over 16 key tiles
    ])
def test_index_variant(B, Hq, Hkv, n, d, k, causal, v_bf16):
    _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed=B * 1000 + Hq * 100 + n + 7,
              fwd=sfa.sfa_attn_fwd_index)


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,v_bf16",
    [
        (1, 2, 1, 150, 32, 4, True, False),    # d = 32
        (1, 3, 1, 97, 80, 8, True, True),      # d = 80, three query heads per KV head
        (2, 2, 2, 70, 96, 12, False, False),   # d = 96, non-causal
        (1, 2, 2, 65, 256, 16, True, True),    # d = 256, the largest
        (1, 1, 1, 40, 200, 200, True, False),  # k = d = 200
        (1, 2, 1, 35, 16, 1, True, True),      # d = 16, k = 1
        (1, 6, 2, 300, 192, 24, True, True),   # d = 192, ten key tiles
    ])
def test_other_head_dims(B, Hq, Hkv, n, d, k, causal, v_bf16):
    """Head dimensions other than 64 and 128 run on the forward of float32
    accuracy; any group size."""
    _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed=d * 10 + n)


@pytest.mark.parametrize("scale,v_bf16", [(1.0, True), (-0.5, True), (0.0, True), (1.0, False),
                                           (-1.0 / 128, True), (2.0, True), (-1.0, True)])
def test_scales(scale, v_bf16):
    """Scales other than 1/sqrt(d), of either sign and zero.  At |scale| = 1
    the exponents reach ~50 (base 2), far above the first tiles' maxima: the
    lazily raised maximum and its rescaling run on most rows.  The score
    error is ~3 * 2^-22 of |scale| * sum |q_u k_u| (float16 pieces), so the
    LSE stays within 1e-4 at these scales too."""
    d = 128
    _run_case(1, 4, 1, 1100, d, 16, True, v_bf16, seed=31 + int(8 * abs(scale)), scale=scale)


@pytest.mark.parametrize("side", ["key", "query"])
def test_codes_beyond_float16_pieces(side):
    """Code values too large for the float16 score pieces (|x| >= 65504; for
    queries x includes scale * log2(e)) hand their workgroups to the rerun,
    which splits them into three bf16 pieces.  The scale keeps the scores
    moderate (an LSE in the thousands is not representable to 1e-4 in
    float32), so the ordinary tolerances apply."""
    B, Hq, Hkv, n, d, k = 1, 8, 2, 700, 128, 16
    q, kk, v = si.dense_qkv(B, Hq, Hkv, n, d, 95, v_dtype=torch.bfloat16, device=DEV)
    if side == "key":
        kk[0, 0, 70, 5] = 70000.0      # KV head 0, second tile
        kk[0, 1, 650, 100] = -3.0e5    # KV head 1, last tile
        scale = 1e-4
    else:
        kk *= 1e-5
        q[0, 2, 300, 7] = 70000.0      # x = 70000 * log2(e) > 65504
        q[0, 7, 5, 9] = -1.0e5
        scale = 1.0
    qi, qv = _gpu_codes(q, k)
    ki, kv = _gpu_codes(kk, k)
    o32, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=True, scale=scale, o_dtype=torch.float32)
    torch.cuda.synchronize()
    oqi, oqv = oracle.topk_encode(q.cpu().numpy(), k)
    oki, okv = oracle.topk_encode(kk.cpu().numpy(), k)
    O, L = oracle.attn_fwd(oqi, oqv, oki, okv, np_vals(v), d, scale, True)
    check_o(o32, O, TOL_O_BF16V, f"O with large {side} codes")
    check_lse(lse, L, f"LSE with large {side} codes")


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,v_bf16",
    [
        (1, 6, 2, 300, 128, 16, True, True),   # groups of 3 query heads
        (1, 5, 1, 200, 128, 16, True, True),   # a group of 5
        (2, 10, 2, 130, 64, 16, False, True),  # groups of 5 at d = 64, non-causal
        (1, 3, 1, 150, 128, 8, True, False),   # group of 3, float32 V
    ])
def test_group_not_power_of_two(B, Hq, Hkv, n, d, k, causal, v_bf16):
    """Group sizes that are not a power of two run the float32 kernel at any
    head dim."""
    _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed=Hq * 10 + n)


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,v_bf16",
    [
        (1, 4, 1, 700, 128, 2, True, True),    # k = 2, eleven key tiles
        (1, 8, 2, 300, 128, 1, True, True),    # k = 1, GQA 4:1
        (2, 2, 2, 257, 128, 2, False, True),   # non-causal, ragged
        (1, 1, 1, 200, 64, 1, True, True),     # d = 64: the dense product (faster there)
        (1, 16, 1, 130, 128, 2, True, True),   # 16 heads per KV head
        (1, 128, 1, 40, 128, 2, True, True),   # 128 heads per KV head (one row per head)
        (1, 2, 1, 1, 128, 2, True, True),      # n = 1
        (1, 6, 2, 300, 128, 2, True, True),    # groups of 3: the float32 kernel
    ])
def test_index_scores_small_k(B, Hq, Hkv, n, d, k, causal, v_bf16):
    """k <= 2 at d = 128 with bf16 V and near-uniform supports: sfa_attn_fwd
    scores through the per-tile inverted indexes (bucket walks) instead of the
    dense product."""
    _run_case(B, Hq, Hkv, n, d, k, causal, v_bf16, seed=k * 100 + n + Hq)


def test_index_scores_skewed_supports():
    """Zipf-skewed supports at k = 2 make long buckets: the data-dependent
    choice may take either mode; the result must match either way."""
    _run_case(1, 4, 2, 1500, 128, 2, True, True, seed=14, zipf_s=1.1)


def test_index_scores_deterministic():
    q, kk, v = si.dense_qkv(1, 4, 1, 2100, 128, 19, device=DEV)
    qi, qv = _gpu_codes(q, 2)
    ki, kv = _gpu_codes(kk, 2)
    o1, l1 = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, o_dtype=torch.float32)
    o2, l2 = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, o_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


def test_index_scores_v_beyond_float16_range():
    """The index mode hands workgroups whose keys reach a V value outside the
    float16 range to the bf16 rerun, like the dense mode."""
    B, Hq, Hkv, n, d, k = 1, 8, 2, 700, 128, 2
    q, kk, v = si.dense_qkv(B, Hq, Hkv, n, d, 97, v_dtype=torch.bfloat16, device=DEV)
    v[0, 0, 70, 5] = 65536.0
    v[0, 1, 650, 100] = -3.0e5
    qi, qv = _gpu_codes(q, k)
    ki, kv = _gpu_codes(kk, k)
    scale = 1.0 / math.sqrt(d)
    o32, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=True, scale=scale, o_dtype=torch.float32)
    torch.cuda.synchronize()
    oqi, oqv = oracle.topk_encode(q.cpu().numpy(), k)
    oki, okv = oracle.topk_encode(kk.cpu().numpy(), k)
    vn = np_vals(v)
    O, L = oracle.attn_fwd(oqi, oqv, oki, okv, vn, d, scale, True)
    tol = TOL_O_BF16V + 2.0 ** -16 * float(np.abs(oracle.widen(vn)).max())
    got = o32.double().cpu().numpy()
    err = np.abs(got - O).max()
    print(f"[parity] index mode, large V: max|O-O_oracle| = {err:.3e} (bound {tol:.3e})", flush=True)
    assert np.isfinite(got).all() and err <= tol
    check_lse(lse, L, "LSE (index mode, large V)")


def test_int16_indices_bf16_values():
    _run_case(1, 4, 2, 190, 128, 16, True, True, seed=77, idx_dtype=torch.int16,
              val_dtype=torch.bfloat16)


def test_zipf_small():
    _run_case(1, 2, 2, 260, 128, 8, True, True, seed=4, zipf_s=1.1)


@pytest.mark.parametrize("where", ["some_tiles", "every_tile"])
def test_v_beyond_float16_range(where):
    """bf16 V values of magnitude >= 65536 do not fit the float16 P.V path;
    the workgroups whose keys reach them are recomputed with bf16 V (P split
    hi + lo).  Some workgroups keep the float16 path, the others are redone:
    every output must match the oracle, to an error bound that scales with
    max|V| (2^-17 per weight, plus the bf16-output half-ulp)."""
    B, Hq, Hkv, n, d, k = 1, 8, 2, 700, 128, 16
    q, kk, v = si.dense_qkv(B, Hq, Hkv, n, d, 91, v_dtype=torch.bfloat16, device=DEV)
    big = [65536.0, -1.0e6, 3.0e5, 2.0e30]
    if where == "some_tiles":
        # KV head 0: key 70 (second tile); KV head 1: key 650 (last tile)
        v[0, 0, 70, 5] = big[0]
        v[0, 0, 70, 77] = big[1]
        v[0, 1, 650, 100] = big[2]
    else:
        for j in range(0, n, 64):
            v[0, j // 64 % Hkv, j, (7 * j) % d] = big[(j // 64) % len(big)]
    qi, qv = _gpu_codes(q, k)
    ki, kv = _gpu_codes(kk, k)
    scale = 1.0 / math.sqrt(d)
    o32, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=True, scale=scale, o_dtype=torch.float32)
    ob16, _ = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=True, scale=scale, o_dtype=torch.bfloat16,
                               want_lse=False)
    torch.cuda.synchronize()
    oqi, oqv = oracle.topk_encode(q.cpu().numpy(), k)
    oki, okv = oracle.topk_encode(kk.cpu().numpy(), k)
    vn = np_vals(v)
    O, L = oracle.attn_fwd(oqi, oqv, oki, okv, vn, d, scale, True)
    vmax = float(np.abs(oracle.widen(vn)).max())
    tol = TOL_O_BF16V + 2.0 ** -16 * vmax
    got = o32.double().cpu().numpy()
    assert np.isfinite(got).all()
    err = np.abs(got - O).max()
    print(f"[parity] O with max|V| = {vmax:.3g}: max|O-O_oracle| = {err:.3e} (bound {tol:.3e})", flush=True)
    assert err <= tol
    check_o(ob16, O, tol, "O (bf16 output, large V)")
    check_lse(lse, L, "LSE (large V)")
    # rows whose keys hold no large value are held to the ordinary tolerance
    if where == "some_tiles":
        small = np.abs(O).max(axis=-1) < 100.0
        e_small = np.abs(got - O)[small].max()
        print(f"[parity] rows away from the large values: max|O-O_oracle| = {e_small:.3e}", flush=True)
        assert e_small <= TOL_O_BF16V


def test_gpt2s_workload_full():
    # every output of the GPT-2-small-shaped workload, against the oracle
    w = si.workload("gpt2s")
    _run_case(w.B, w.Hq, w.Hkv, w.n, w.d, w.k, w.causal, w.v_bf16, w.seed)


def _big_case_sampled(w, heads, zipf=False):
    """Full-size workload on the GPU (encode + forward), oracle on sampled rows."""
    G = w.G
    q = torch.empty((1, w.Hq, w.n, w.d), device=DEV)
    kk = torch.empty((1, w.Hkv, w.n, w.d), device=DEV)
    v = torch.empty((1, w.Hkv, w.n, w.d), device=DEV, dtype=torch.bfloat16)
    for h in range(w.Hq):
        if zipf:
            perm = si.zipf_feature_perm(w.d, w.seed, h // G)
            i_, v_ = si.zipf_codes(w.n, w.d, w.k, w.zipf_s, perm, w.seed, "q", 0, h, device=DEV)
            q[0, h] = si.dense_from_codes(i_, v_, w.d)
        else:
            q[0, h] = si.normal((w.n, w.d), w.seed, "q", 0, h, device=DEV)
    for h in range(w.Hkv):
        if zipf:
            perm = si.zipf_feature_perm(w.d, w.seed, h)
            i_, v_ = si.zipf_codes(w.n, w.d, w.k, w.zipf_s, perm, w.seed, "k", 0, h, device=DEV)
            kk[0, h] = si.dense_from_codes(i_, v_, w.d)
        else:
            kk[0, h] = si.normal((w.n, w.d), w.seed, "k", 0, h, device=DEV)
        v[0, h] = si.normal((w.n, w.d), w.seed, "v", 0, h, device=DEV).to(torch.bfloat16)
    qi, qv = _gpu_codes(q, w.k)
    ki, kv = _gpu_codes(kk, w.k)
    o32, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=w.causal, scale=w.scale,
                                o_dtype=torch.float32)
    torch.cuda.synchronize()
    rows = sample_rows(w.n, extra=(127, 128, 4095, 4096, w.n // 2), count=16, seed=w.seed)
    for h in heads:
        g = h // G
        kn = kk[0, g, : rows.max() + 1].cpu().numpy()
        oki, okv = oracle.topk_encode(kn, w.k)
        oqi, oqv = oracle.topk_encode(q[0, h, torch.from_numpy(rows).to(DEV)].cpu().numpy(), w.k)
        qi_full = np.zeros((w.n, w.k), np.int64); qv_full = np.zeros((w.n, w.k), np.float32)
        qi_full[rows], qv_full[rows] = oqi, oqv
        O, L = oracle.attn_fwd_rows(qi_full, qv_full, oki, okv,
                                    np_vals(v[0, g, : rows.max() + 1]), w.d, w.scale, w.causal, rows)
        sel = torch.from_numpy(rows).to(DEV)
        check_o(o32[0, h, sel], O, TOL_O_BF16V, f"O head {h}")
        check_lse(lse[0, h, sel], L, f"LSE head {h}")


def test_qwen3_32k_full_size_sampled():
    _big_case_sampled(si.workload("qwen3_32k"), heads=(0, 5, 31))


def test_zipf_128k_full_size_sampled():
    _big_case_sampled(si.workload("zipf_128k"), heads=(0, 7), zipf=True)


def test_deterministic():
    # the matrix-core forward has a fixed summation order: bitwise repeatable
    q, kk, v = si.dense_qkv(1, 4, 1, 500, 128, 9, device=DEV)
    qi, qv = _gpu_codes(q, 16)
    ki, kv = _gpu_codes(kk, 16)
    o1, l1 = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, o_dtype=torch.float32)
    o2, l2 = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, o_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


def test_index_variant_repeatable():
    # the inverted-index variant: the order of keys inside a bucket may vary
    # between runs (the counting sort takes slots with atomics), but every
    # score entry has one owner that adds its overlaps in the row's code
    # order, so the results are bitwise repeatable
    q, kk, v = si.dense_qkv(1, 4, 1, 2100, 128, 9, device=DEV)
    qi, qv = _gpu_codes(q, 16)
    ki, kv = _gpu_codes(kk, 16)
    o1, l1 = sfa.sfa_attn_fwd_index(qi, qv, ki, kv, v, o_dtype=torch.float32)
    o2, l2 = sfa.sfa_attn_fwd_index(qi, qv, ki, kv, v, o_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


@pytest.mark.parametrize(
    "B,Hq,Hkv,n,d,k,causal,codes,v_bf16,window,n_global,mag",
    [
        (1, 6, 1, 129, 128, 16, True, "f32", True, 0, 0, 1.0),      # one row past a block, groups of 2 of 6
        (1, 12, 1, 65, 128, 17, True, "f32", True, 0, 0, 1.0),      # groups of 4 of 12, k just past 16
        (2, 7, 1, 64, 64, 8, False, "i16bf16", True, 0, 0, 1.0),    # 16-bit codes, one whole tile
        (1, 5, 1, 300, 96, 16, True, "u8f16", True, 70, 5, 1.0),    # fp16 codes, a window and global tokens
        (1, 2, 2, 333, 96, 12, False, "f32", True, 40, 70, 1.0),    # global tokens past a tile
        (1, 2, 1, 131, 77, 77, True, "f32", True, 0, 0, 1.0),       # odd d: element loads, k = d
        (1, 3, 1, 1, 33, 3, True, "f32", False, 0, 0, 1.0),         # n = 1
        (1, 1, 1, 100, 129, 9, True, "f32", False, 0, 0, 1.0),      # just past the d = 128 kernel, float32 V
        (1, 3, 3, 200, 256, 256, False, "i16bf16", True, 0, 0, 1.0),  # the largest d and k
        (1, 6, 2, 200, 128, 16, True, "f32", True, 0, 0, 2.0 ** -30),  # V far below the float16 range
        (1, 2, 2, 200, 96, 16, True, "f32", True, 0, 0, 2.0 ** 40),    # V far above it
        (1, 8, 8, 300, 96, 16, True, "f32", True, 0, 0, 1.0),        # head groups a multiple of 8: placed by XCD
        (2, 48, 4, 150, 128, 16, True, "u8f16", True, 50, 3, 1.0),   # 24 of them, groups of 4 of 12, a window
    ])
def test_generic_forward_float32_accuracy(B, Hq, Hkv, n, d, k, causal, codes, v_bf16, window,
                                          n_global, mag):
    """The forward for other head dims and groups, at the edges of its tiles and
    formats, to float32 accuracy with a float32 output (1e-5 of the values'
    scale, the bound of the float32 path) and rounded once with a bf16 one;
    from arrays 16-byte aligned and not."""
    it, vt = {"f32": (torch.int32, torch.float32), "i16bf16": (torch.int16, torch.bfloat16),
              "u8f16": (torch.uint8, torch.float16)}[codes]
    q, kk, v = si.dense_qkv(B, Hq, Hkv, n, d, 7 * d + n, v_dtype=torch.float32, device=DEV)
    v = (v * mag).to(torch.bfloat16 if v_bf16 else torch.float32)
    qi, qv = sfa.sfa_topk_encode(q, k, idx_dtype=it, val_dtype=vt)
    ki, kv = sfa.sfa_topk_encode(kk, k, idx_dtype=it, val_dtype=vt)
    scale = 1.0 / math.sqrt(d)

    def wide(x):
        return x.float().cpu().numpy()
    O, L = oracle.attn_fwd(qi.cpu().numpy(), wide(qv), ki.cpu().numpy(), wide(kv), np_vals(v), d, scale,
                           causal, window=window, n_global=n_global)
    base = torch.zeros(v.numel() + 1, dtype=v.dtype, device=DEV)
    base[1:] = v.reshape(-1)
    for vin in (v, base[1:].view(v.shape)):  # the second one element off the allocation
        o, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, vin, causal=causal, scale=scale, window=window,
                                  n_global=n_global, o_dtype=torch.float32)
        torch.cuda.synchronize()
        check_o(o / mag, O / mag, TOL_O_F32, "generic O")
        check_lse(lse, L, "generic LSE", tol=1e-5)
    o16, _ = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, causal=causal, scale=scale, window=window,
                              n_global=n_global, o_dtype=torch.bfloat16)
    # the same values, rounded once
    check_o((o16.float() / mag).to(torch.bfloat16), O / mag, TOL_O_F32, "generic bf16 O")


@pytest.mark.parametrize("Hq,Hkv,n,d,k,codes,v_bf16", [
    (6, 1, 700, 128, 16, "f32", True),
    (2, 2, 1000, 192, 16, "f32", False),
    (2, 2, 1000, 192, 16, "u8f16", True),
    (3, 3, 777, 80, 8, "i16bf16", True),
])
def test_generic_forward_error_against_64_bits(Hq, Hkv, n, d, k, codes, v_bf16):
    """The general forward loses no more than float32 arithmetic does: its
    relative error (2-norm) against the float64 oracle, with peaked softmax rows
    (codes of three times the usual size), is at most 1.25 times that of the same
    formulas in plain float32: base-2 exponents, a score the sum of a key's k
    products in turn, the softmax sum and O added up by tiles of 32 keys."""
    it, vt = {"f32": (torch.int32, torch.float32), "i16bf16": (torch.int16, torch.bfloat16),
              "u8f16": (torch.uint8, torch.float16)}[codes]
    q, kk, v = si.dense_qkv(1, Hq, Hkv, n, d, n + d, v_dtype=torch.bfloat16 if v_bf16 else torch.float32,
                            device=DEV)
    qi, qv = sfa.sfa_topk_encode(3 * q, k, idx_dtype=it, val_dtype=vt)
    ki, kv = sfa.sfa_topk_encode(3 * kk, k, idx_dtype=it, val_dtype=vt)
    scale = 1.0 / math.sqrt(d)
    o, lse = sfa.sfa_attn_fwd(qi, qv, ki, kv, v, scale=scale, o_dtype=torch.float32)
    torch.cuda.synchronize()
    qi, qv, ki, kv = (x.float().cpu().numpy() for x in (qi, qv, ki, kv))
    O, L = oracle.attn_fwd(qi.astype(np.int64), qv, ki.astype(np.int64), kv, np_vals(v), d, scale, True)
    # plain float32, head by head
    vf = v.float().cpu().numpy()
    f32 = np.float32
    o_p, l_p = np.empty((Hq, n, d), f32), np.empty((Hq, n), f32)
    for h in range(Hq):
        g = h // (Hq // Hkv)
        qd = np.zeros((n, d), f32)
        np.put_along_axis(qd, qi[0, h].astype(np.int64), qv[0, h] * f32(scale / _LN2), 1)
        s = np.zeros((n, n), f32)
        for t in range(k):
            s += qd[:, ki[0, g, :, t].astype(np.int64)] * kv[0, g, :, t]
        s[np.triu_indices(n, 1)] = -np.inf
        m = s.max(1, keepdims=True)
        p = np.exp2(s - m)
        acc, l = np.zeros((n, d), f32), np.zeros((n, 1), f32)
        for j in range(0, n, 32):
            acc += p[:, j:j + 32] @ vf[0, g, j:j + 32]
            l += p[:, j:j + 32].sum(1, keepdims=True)
        o_p[h], l_p[h] = acc / l, (m + np.log2(l))[:, 0] * f32(_LN2)

    def rel(x, y):
        return np.linalg.norm(x.astype(np.float64) - y) / np.linalg.norm(y)
    for got, plain, want, nm in ((o[0].cpu().numpy(), o_p, O[0], "O"), (lse[0].cpu().numpy(), l_p, L[0], "LSE")):
        e, b = rel(got, want), rel(plain, want)
        print(f"[parity] general forward {nm}: {e:.2e} against 64 bits, plain float32 {b:.2e}", flush=True)
        assert e <= 1.25 * b, nm


@pytest.mark.parametrize("what", ["v", "keys", "queries", "raised maximum", "bf16 product", "scale 0",
                                  "negative scale"])
@pytest.mark.parametrize("d", [96, 200])
def test_generic_forward_extreme_magnitudes(what, d):
    """Values and products at the ends of the float32 range, where float32 arithmetic
    stays finite: the largest float32 as V or a code value (past the largest bf16), a
    running maximum raised by less than 2^8 under V of 2^121, products of bf16 codes
    that only the scale brings back into range."""
    n, k, scale, causal, vdt, cdt = 96, 4, _LN2, True, torch.float32, torch.float32
    rng = np.random.default_rng(d)
    qi = np.tile(np.arange(k), (1, 1, n, 1)); ki = qi.copy()
    qv = rng.standard_normal((1, 1, n, k)).astype(np.float32); kv = qv[:, :, ::-1].copy()
    v = rng.standard_normal((1, 1, n, d)).astype(np.float32)
    if what == "v":  # one such key, in every row's softmax
        v[0, 0, 0] = np.where(np.arange(d) % 2, _MAXF, -_MAXF)
    elif what in ("keys", "queries"):  # score of about 4 with its counterpart 2^-126
        big, small = (kv, qv) if what == "keys" else (qv, kv)
        small[...] = 0
        small[..., 0] = 2.0 ** -126
        big[0, 0, ::3, 0] = _MAXF
        big[0, 0, 1::3, 0] = -_MAXF
    elif what == "raised maximum":  # 64 keys of score 0, then one of 7 (base 2)
        causal = False
        qv[...] = 0; kv[...] = 0
        qv[..., 0] = 1.0
        kv[0, 0, 64, 0] = 7.0
        v[...] = 1.5 * 2.0 ** 121
    else:
        cdt, vdt = torch.bfloat16, torch.bfloat16
        qv[...] = 0; kv[...] = 0
        qv[..., 0] = 2.0 ** 65
        kv[0, 0, :, 0] = np.where(np.arange(n) % 7, -1.0, 1.0) * 2.0 ** 65
        kv[0, 0, ::7, 0] *= 1.0 + np.arange(len(kv[0, 0, ::7, 0]))[::-1] / 16  # key 0 the largest
        scale = {"bf16 product": 2.0 ** -6, "scale 0": 0.0, "negative scale": -2.0 ** -6}[what]
        if what == "negative scale":
            qv = -qv
    ti, tv = torch.from_numpy(qi).int().to(DEV), torch.from_numpy(qv).to(cdt).to(DEV)
    tki, tkv = torch.from_numpy(ki).int().to(DEV), torch.from_numpy(kv).to(cdt).to(DEV)
    tvv = torch.from_numpy(v).to(vdt).to(DEV)
    o, lse = sfa.sfa_attn_fwd(ti, tv, tki, tkv, tvv, causal=causal, scale=scale, o_dtype=torch.float32)
    torch.cuda.synchronize()

    def wide(x):
        return x.double().cpu().numpy()
    S = wide(tv)[0, 0] @ wide(tkv)[0, 0].T * np.float32(scale).astype(np.float64)
    if causal:
        S[np.triu_indices(n, 1)] = -np.inf
    m = S.max(1, keepdims=True)
    P = np.exp(S - m)
    O = P / P.sum(1, keepdims=True) @ wide(tvv)[0, 0]
    L = (m + np.log(P.sum(1, keepdims=True)))[:, 0]
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()
    mag = np.abs(O).max(1, keepdims=True)
    assert (np.abs(wide(o)[0, 0] - O) <= TOL_O_F32 * mag).all()
    # float32 scores: 2^-23 of their size beside the bound of ordinary ones
    assert (np.abs(wide(lse)[0, 0] - L) <= 1e-5 + 2.0 ** -22 * np.abs(L)).all()


@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs two GPUs in one process")
def test_generic_forward_on_a_second_device():
    """The general kernel's LDS limit is set on every device that it runs on."""
    q, kk, v = si.dense_qkv(1, 3, 1, 200, 128, 5, v_dtype=torch.bfloat16, device=DEV)
    (qi, qv), (ki, kv) = _gpu_codes(q, 16), _gpu_codes(kk, 16)
    o = []
    for dev in range(2):
        with torch.cuda.device(dev):
            o.append(sfa.sfa_attn_fwd(*(x.to(f"cuda:{dev}") for x in (qi, qv, ki, kv, v)))[0].cpu())
    assert torch.equal(o[0], o[1])
