"""Jumps of the softmax reference, masks and segments folded in on the pipelined kernel: the same 64 query heads in groups of
1, 2, 4 and 8 per KV head, with enough rows that every call has a work item for each compute unit
(tests/test_kernel_choice.py makes sure of that)."""
import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth
from test_gpu_underfilled import DEV, assert_close

pytestmark = pytest.mark.gpu
HQ = 64
KV_HEADS = (64, 32, 16, 8)
# (sq, sk, q_off, causal) and keys 16 ... 130 log2 units above the bulk, as (key, query row, gain): in the first tile, in the
# second one, in late tiles with and without a mask, in the last key and in the ragged last tile
JUMPS = [
    ((1024, 1024, 0, True), [(5, 130, 4), (70, 950, 1), (300, 400, 2), (301, 1000, 4), (640, 700, 8), (900, 901, 8), (1023, 1023, 2)]),
    ((1024, 1024, 4096, True), [(5, 3, 2), (70, 31, 8), (300, 32, 2), (511, 1000, 4), (515, 33, 8), (700, 600, 1), (1020, 1, 8)]),
    ((1000, 1001, 0, False), [(64, 999, 8), (500, 17, 8), (961, 0, 4), (1000, 250, 2)]),
]
BATCH_Q, BATCH_K = [200, 1024, 1, 77], [200, 1024, 9000, 77]
MASKS = [(0, 0, 1000, 1000), (1000, 937, 1001, 1400), (5, 200, 1000, 300), (0, 64, 1000, 960), (255, 0, 1003, 1300)]


def some_groups(hkv, *tensors):
    """The first, a middle and the last KV head with their query heads: the oracle takes a head at a time."""
    g = HQ // hkv
    for h in (0, hkv // 2 + 1, hkv - 1):
        yield (slice(h * g, (h + 1) * g), *[t[:, h * g:(h + 1) * g] if t.shape[1] == HQ else t[:, h:h + 1] for t in tensors])


@pytest.mark.parametrize("hkv", KV_HEADS)
@pytest.mark.parametrize("sizes,outliers", JUMPS)
def test_jumps_of_the_row_maximum(sizes, outliers, hkv):
    sq, sk, q_off, causal = sizes
    q, k, v = synth.qkv_with_outlier_keys(5100 + hkv, sq, sk, HQ, hkv, outliers)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    out = torch.full((sq, HQ, 128), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((HQ, sq), float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_chunk(qd, kd, vd, q_off, 0, causal, out_dtype=torch.float32, out=out, lse=lse)
    cut = sk // 2                # and the running state carried across the jumps of both halves, in both orders
    folded = []
    for first, second in ((slice(0, cut), slice(cut, sk)), (slice(cut, sk), slice(0, cut))):
        o_acc, l_acc = pec.pec_attn_chunk(qd, kd[first], vd[first], q_off, first.start, causal, out_dtype=torch.float32)
        pec.pec_attn_chunk_merge(qd, kd[second], vd[second], q_off, second.start, o_acc, l_acc, causal)
        folded.append((o_acc, l_acc))
    for heads, qh, kh, vh in some_groups(hkv, q, k, v):
        o_ref, l_ref = oracle.attention(qh, kh, vh, q_off=q_off, kv_off=0, causal=causal)
        assert_close(out[:, heads], lse[heads], o_ref, l_ref, "whole")
        for o_acc, l_acc in folded:
            assert_close(o_acc[:, heads], l_acc[heads], o_ref, l_ref, "two segments")


@pytest.mark.parametrize("times", [1, 2])      # one head and several heads per work item
@pytest.mark.parametrize("hkv", KV_HEADS)
def test_jumps_of_the_row_maximum_in_batches(hkv, times):
    len_q = BATCH_Q * times
    for len_k in (len_q, BATCH_K * times):
        cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
        tq, tk = int(cq[-1]), int(ck[-1])
        q1, k1, q2, k2 = int(cq[1]), int(ck[1]), int(cq[2]), int(ck[2])
        outliers = [(10, 150, 8), (k1 + 70, q1 + 950, 2), (k1 + 640, q1 + 700, 8), (k1 + 900, q1 + 901, 4), (k1 + 1023, q1 + 1023, 8)]
        if len_k is not len_q:   # the decode step: in the first key range, around its end and in the last, short one
            outliers += [(k2 + 100, q2, 1), (k2 + 4095, q2, 1), (k2 + 4100, q2, 2), (k2 + 8999, q2, 1)]
        q, k, v = synth.qkv_with_outlier_keys(5200 + hkv, tq, tk, HQ, hkv, outliers)
        cqd, ckd = torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV)
        out = torch.full((tq, HQ, 128), float("nan"), dtype=torch.float32, device=DEV)
        lse = torch.full((HQ, tq), float("nan"), dtype=torch.float32, device=DEV)
        if len_k is len_q:
            pec.pec_attn_varlen(q.to(DEV), k.to(DEV), v.to(DEV), cqd, max(len_q), True, out_dtype=torch.float32, out=out, lse=lse)
        else:
            pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), cqd, ckd, True, out_dtype=torch.float32, out=out, lse=lse)
        for heads, qh, kh, vh in some_groups(hkv, q, k, v):
            o_ref, l_ref = oracle.colocated(qh, kh, vh, cq, ck, causal=True)
            assert_close(out[:, heads], lse[heads], o_ref, l_ref, "batch of %d keys" % tk)


@pytest.mark.parametrize("hkv", KV_HEADS)
@pytest.mark.parametrize("q_off,kv_off,sq,sk", MASKS)
def test_visible_keys_are_counted_exactly(q_off, kv_off, sq, sk, hkv):
    """Q = 0 gives LSE_i = ln n_i with n_i the visible keys; V = 1 in one key gives 1 / n_i or exactly 0."""
    _, k, _ = synth.qkv(5300, 1, sk, HQ, hkv)
    q = torch.zeros(sq, HQ, 128, dtype=torch.bfloat16, device=DEV)
    v = torch.zeros(sk, hkv, 128, dtype=torch.bfloat16, device=DEV)
    one = sk // 2
    v[one] = 1.0
    out = torch.full((sq, HQ, 128), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((HQ, sq), float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_chunk(q, k.to(DEV), v, q_off, kv_off, True, out_dtype=torch.float32, out=out, lse=lse)
    out, lse = out.cpu().numpy(), lse.cpu().numpy().astype(np.float64)
    n = np.clip(q_off + np.arange(sq) - kv_off + 1, 0, sk)
    assert np.all(lse[:, n == 0] == -np.inf)
    assert np.array_equal(np.rint(np.exp(lse[:, n > 0])).astype(np.int64), np.tile(n[n > 0], (HQ, 1)))
    sees = n > one
    assert np.all(out[~sees] == 0.0)
    # every weight is exactly 1, so 1 / n is rounded in fp32 alone: far inside 2e-3
    np.testing.assert_allclose(out[sees], np.broadcast_to((1.0 / n[sees])[:, None, None], out[sees].shape), rtol=2e-3, atol=0)
