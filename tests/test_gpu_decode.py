"""GPU parity: sfa_attn_decode over a sparse-code KV cache against the
oracle.  The cache codes are written by sfa_topk_encode (int16 indices, bf16
values); the oracle codes the same dense keys with its own Top-k and bf16
rounding."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2603_22300_amd as sfa
import sfa_inputs as si
from helpers import TOL_O_BF16V, TOL_O_F32, check_lse, check_o, np_vals

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(B, Hq, Hkv, Lmax, d, k, v_bf16, seq, seed, cache_bf16=True):
    kd = torch.empty((B, Hkv, Lmax, d), device=DEV)
    vdt = torch.bfloat16 if v_bf16 else torch.float32
    vc = torch.empty((B, Hkv, Lmax, d), device=DEV, dtype=vdt)
    for b in range(B):
        for h in range(Hkv):
            kd[b, h] = si.normal((Lmax, d), seed, "k", b, h, device=DEV)
            vv = si.normal((Lmax, d), seed, "v", b, h, device=DEV)
            vc[b, h] = vv.to(vdt)
    qd = si.normal((B, Hq, d), seed, "q", device=DEV)
    ci, cv = sfa.sfa_topk_encode(kd, k, idx_dtype=torch.int16,
                                 val_dtype=torch.bfloat16 if cache_bf16 else torch.float32)
    qi, qv = sfa.sfa_topk_encode(qd, k)
    seq_t = None if seq is None else torch.tensor(seq, dtype=torch.int32, device=DEV)
    scale = 1.0 / math.sqrt(d)
    o, lse = sfa.sfa_attn_decode(qi, qv, ci, cv, vc, seq_len=seq_t, scale=scale,
                                 o_dtype=torch.float32)
    torch.cuda.synchronize()
    kn = kd.cpu().numpy()
    oci, ocv = (oracle.topk_encode_bf16 if cache_bf16 else oracle.topk_encode)(kn, k)
    oqi, oqv = oracle.topk_encode(qd.cpu().numpy(), k)
    O, L = oracle.attn_decode(oqi, oqv, oci, ocv, np_vals(vc), d, scale, seq_len=seq)
    check_o(o, O, TOL_O_BF16V if v_bf16 else TOL_O_F32, "decode O")
    check_lse(lse, L, "decode LSE")


@pytest.mark.parametrize(
    "B,Hq,Hkv,Lmax,d,k,v_bf16,seq",
    [
        (3, 8, 2, 300, 128, 16, True, [300, 1, 157]),
        (2, 4, 4, 5000, 64, 8, False, None),         # several context chunks, float32 V
        (2, 8, 1, 4097, 128, 16, True, [4097, 2049]),  # chunk boundaries, 8:1 groups
        (1, 2, 1, 64, 64, 64, False, None),           # k = d
        (2, 2, 2, 100, 128, 1, True, [100, 63]),      # k = 1
        (2, 4, 1, 3000, 128, 8, True, [3000, 1]),     # vectorized codes, k = 8
        (1, 8, 4, 2500, 64, 32, True, [2500]),        # vectorized codes, k = 32, d = 64
        (3, 2, 2, 777, 128, 16, True, [5, 777, 64]),  # vectorized codes, short sequences
    ])
def test_shapes(B, Hq, Hkv, Lmax, d, k, v_bf16, seq):
    _case(B, Hq, Hkv, Lmax, d, k, v_bf16, seq, seed=Lmax + k)


@pytest.mark.parametrize(
    "B,Hq,Hkv,Lmax,d,k,v_bf16,seq",
    [
        (2, 3, 1, 300, 80, 8, True, [300, 37]),          # three query heads per KV head
        (2, 8, 1, 4500, 96, 12, False, [4500, 2049]),    # chunks, 8:1 groups, float32 V
        (1, 2, 2, 100, 256, 16, True, None),             # d = 256
        (2, 4, 2, 129, 32, 32, True, [129, 1]),          # k = d = 32
        (1, 6, 2, 2100, 200, 10, True, [2100]),          # d = 200, group of 3
    ])
def test_other_head_dims(B, Hq, Hkv, Lmax, d, k, v_bf16, seq):
    """Head dimensions other than 64 and 128 run the float32 decode."""
    _case(B, Hq, Hkv, Lmax, d, k, v_bf16, seq, seed=d + Lmax)


@pytest.mark.parametrize(
    "B,Hq,Hkv,Lmax,d,k,v_bf16,seq",
    [
        (2, 6, 2, 5000, 128, 16, True, [5000, 77]),   # groups of 3, two chunks
        (1, 5, 1, 300, 128, 16, True, None),          # a group of 5
        (2, 10, 2, 700, 64, 8, False, [700, 1]),      # groups of 5 at d = 64
    ])
def test_group_not_power_of_two(B, Hq, Hkv, Lmax, d, k, v_bf16, seq):
    """Group sizes that are not a power of two run the next power of two's kernel."""
    _case(B, Hq, Hkv, Lmax, d, k, v_bf16, seq, seed=Hq + Lmax)


@pytest.mark.parametrize("d,k,v_bf16", [(128, 16, True), (64, 8, False)])
def test_group_of_three_unaligned_cache(d, k, v_bf16):
    """A group that is not a power of two over cache arrays off a 16-byte boundary runs
    the float32 decode, contiguous and paged: float32 results as from aligned arrays."""
    B, Hq, Hkv, L, P = 2, 6, 2, 4500, 16
    pages = -(-L // P)
    shape = (B * pages, Hkv, P)
    ci, cv = sfa.sfa_topk_encode(si.normal(shape + (d,), d, "k", device=DEV), k, idx_dtype=torch.int16,
                                 val_dtype=torch.bfloat16)
    vc = si.normal(shape + (d,), d, "v", device=DEV).to(torch.bfloat16 if v_bf16 else torch.float32)
    q = si.normal((B, Hq, d), d, "q", device=DEV)
    table = torch.arange(B * pages, dtype=torch.int32, device=DEV).reshape(B, pages)
    lens = torch.tensor([L, 77], dtype=torch.int32, device=DEV)

    def off(x):
        base = torch.zeros(x.numel() + 1, dtype=x.dtype, device=DEV)
        base[1:] = x.reshape(-1)
        return base[1:].view(x.shape)

    def flat(x):
        return x.reshape((B, pages) + x.shape[1:]).transpose(1, 2).reshape(B, Hkv, pages * P, x.shape[-1]).contiguous()
    kw = dict(seq_len=lens, o_dtype=torch.float32)
    want = sfa.sfa_attn_decode_paged(ci, cv, vc, table, q=q, **kw)
    qc = sfa.sfa_topk_encode(q, k)
    got = [sfa.sfa_attn_decode_paged(*(off(x) for x in (ci, cv, vc)), table, q=q, **kw),
           sfa.sfa_attn_decode(*qc, *(off(flat(x)) for x in (ci, cv, vc)), **kw)]
    torch.cuda.synchronize()
    for o, lse in got:
        assert (o - want[0]).abs().max() <= TOL_O_F32 and (lse - want[1]).abs().max() <= 1e-5


def test_float32_cache_values():
    _case(2, 4, 1, 700, 128, 16, True, [700, 333], seed=3, cache_bf16=False)


def test_decode_64k_full_size_sampled():
    """The full 64-sequence x 64K-token cache (int16 indices, bf16 values, bf16
    V), all outputs computed on the GPU; the oracle rebuilds 6 sampled
    (sequence, head) outputs from regenerated dense keys."""
    w = si.workload("decode_64k")
    B, Hq, Hkv, L, d, k = w.B, w.Hq, w.Hkv, w.n, w.d, w.k
    ci = torch.empty((B, Hkv, L, k), dtype=torch.int16, device=DEV)
    cv = torch.empty((B, Hkv, L, k), dtype=torch.bfloat16, device=DEV)
    vc = torch.empty((B, Hkv, L, d), dtype=torch.bfloat16, device=DEV)
    for b in range(B):
        for h in range(Hkv):
            kd = si.normal((L, d), w.seed, "k", b, h, device=DEV)
            sfa.sfa_topk_encode(kd, k, idx=ci[b, h], val=cv[b, h])
            vc[b, h] = si.normal((L, d), w.seed, "v", b, h, device=DEV).to(torch.bfloat16)
    qd = si.normal((B, Hq, d), w.seed, "q", device=DEV)
    qi, qv = sfa.sfa_topk_encode(qd, k)
    o, lse = sfa.sfa_attn_decode(qi, qv, ci, cv, vc, scale=w.scale, o_dtype=torch.float32)
    torch.cuda.synchronize()
    oqi, oqv = oracle.topk_encode(qd.cpu().numpy(), k)
    for (b, h) in [(0, 0), (0, 31), (17, 5), (33, 12), (63, 30), (63, 7)]:
        g = h // w.G
        kd = si.normal((L, d), w.seed, "k", b, g, device=DEV).cpu().numpy()
        oci, ocv = oracle.topk_encode_bf16(kd, k)
        qd1 = oracle.densify(oqi[b, h][None], oqv[b, h][None], d)
        kdd = oracle.densify(oci, ocv, d)
        O, Lse = oracle.softmax_attention(qd1, kdd, oracle.widen(np_vals(vc[b, g])), w.scale, False)
        check_o(o[b, h][None], O, TOL_O_BF16V, f"decode O ({b},{h})")
        check_lse(lse[b, h].reshape(1), Lse, f"decode LSE ({b},{h})")


@pytest.mark.parametrize(
    "B,Hq,Hkv,Lmax,d,k,seq,window,n_global",
    [
        (1, 8, 2, 1025, 128, 16, [1025], 0, 0),             # 256-key chunks, one key over
        (3, 4, 1, 1024, 64, 8, [1024, 256, 257], 0, 0),     # at chunk edges
        (2, 7, 1, 4500, 128, 16, [4500, 0], 0, 0),          # a group of 7, an empty sequence
        (1, 12, 2, 9000, 64, 16, [8193], 0, 0),             # a group of 6, capacity beyond the length
        (2, 8, 1, 6000, 128, 16, [6000, 513], 700, 5),      # a window, both sides of its gap
        (2, 3, 1, 3000, 128, 12, [3000, 301], 256, 300),    # generic codes; a query just past the global tokens
        (40, 8, 8, 600, 64, 8, None, 0, 0),                 # B * Hkv above the aim: whole chunks
    ])
def test_context_split(B, Hq, Hkv, Lmax, d, k, seq, window, n_global):
    """Sequences cut into chunks below 4096 keys: against the oracle, with the
    smallest workspace the call takes (4096-key chunks), and bit for bit against
    the allocation-free entry point."""
    seed = Lmax + Hq
    kd = torch.stack([si.normal((Hkv, Lmax, d), seed, "k", b, device=DEV) for b in range(B)])
    vc = torch.stack([si.normal((Hkv, Lmax, d), seed, "v", b, device=DEV) for b in range(B)]).to(torch.bfloat16)
    qd = si.normal((B, Hq, d), seed, "q", device=DEV)
    ci, cv = sfa.sfa_topk_encode(kd, k, idx_dtype=torch.int16, val_dtype=torch.bfloat16)
    qi, qv = sfa.sfa_topk_encode(qd, k)
    seq_t = None if seq is None else torch.tensor(seq, dtype=torch.int32, device=DEV)
    least = B * Hq * -(-Lmax // 4096) * (d + 2) * 4
    assert least <= sfa.sfa_attn_decode_workspace(B, Hq, Lmax, d)
    oci, ocv = oracle.topk_encode_bf16(kd.cpu().numpy(), k)
    oqi, oqv = oracle.topk_encode(qd.cpu().numpy(), k)
    lens = np.full(B, Lmax) if seq is None else np.array(seq)
    live = lens > 0
    O, L = oracle.attn_decode(oqi, oqv, oci, ocv, np_vals(vc), d, 1.0 / math.sqrt(d),
                              seq_len=np.maximum(lens, 1), window=window, n_global=n_global)
    O[~live] = 0  # an empty sequence: O = 0, LSE = -inf
    outs = []
    for ws in (None, torch.empty(least, dtype=torch.uint8, device=DEV)):
        o, lse = sfa.sfa_attn_decode(qi, qv, ci, cv, vc, seq_len=seq_t, o_dtype=torch.float32, ws=ws,
                                     window=window, n_global=n_global)
        torch.cuda.synchronize()
        # float32 throughout: 1e-5 as for float32 V, far inside the bf16-V bound
        check_o(o, O, TOL_O_F32, "split decode O")
        check_lse(lse[torch.from_numpy(live).to(DEV)], L[live], "split decode LSE")
        assert torch.isneginf(lse[torch.from_numpy(~live).to(DEV)]).all()
        outs.append((o, lse))
    o, lse = torch.empty_like(outs[0][0]), torch.empty_like(outs[0][1])
    sfa.sfa_attn_decode_noalloc(qi, qv, ci, cv, vc, o, lse=lse, seq_len=seq_t, window=window,
                                n_global=n_global)
    assert torch.equal(o, outs[0][0]) and torch.equal(lse, outs[0][1])
