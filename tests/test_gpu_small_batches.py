"""Batches of up to 64 sequences, whose workgroups find their items in the offsets, and the next larger ones, which get a list."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth
from test_gpu_underfilled import DEV, assert_close

pytestmark = pytest.mark.gpu

# row-tile edges, equal lengths, nothing, keys without queries, chunks behind prefixes, caches of one and of several ranges
SEQ_Q = [33, 1, 0, 64, 1, 65, 0, 1, 5, 33, 1, 32]
SEQ_K = [33, 1, 0, 64, 4097, 65, 9, 12300, 300, 33, 4096, 40]
CASES = [  # sequences, heads, where in the cycle of lengths they start; without a list up to the last four
    (1, 8, 8, 5), (1, 4, 1, 7), (3, 8, 2, 3), (12, 6, 3, 0), (2, 40, 1, 11), (63, 2, 2, 0), (64, 2, 1, 0),
    (65, 2, 1, 0), (64, 8, 1, 0), (64, 40, 1, 0), (130, 2, 1, 0)]


def lengths(n, first):
    i = [(first + j) % len(SEQ_Q) if j < len(SEQ_Q) or j >= n - 2 else 6 + 3 * (j % 2) for j in range(n)]
    return [SEQ_Q[j] for j in i], [SEQ_K[j] for j in i]


@pytest.mark.parametrize("n,hq,hkv,first", CASES)
def test_small_batches_match_oracle(n, hq, hkv, first):
    len_q, len_k = lengths(n, first)
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    tq, tk = int(cq[-1]), int(ck[-1])
    q, _, _ = synth.qkv(9600 + n, tq, 1, hq, hkv)
    _, k, v = synth.qkv(9700 + n, 1, max(tk, tq), hq, hkv)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    cqd, ckd = torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV)
    for causal in (True, False):
        o_ref, l_ref = oracle.colocated(q, k[:tk], v[:tk], cq, ck, causal=causal)
        for dt in (torch.float32, torch.bfloat16):
            out = torch.full((tq, hq, 128), float("nan"), dtype=dt, device=DEV)
            lse = torch.full((hq, tq), float("nan"), dtype=torch.float32, device=DEV)
            pec.pec_attn_colocated(qd, kd[:tk], vd[:tk], cqd, ckd, causal, out_dtype=dt, out=out, lse=lse)
            assert_close(out, lse, o_ref, l_ref, "mixed batch of %d sequences" % n)
        o_ref, l_ref = oracle.varlen(q, k[:tq], v[:tq], cq, causal=causal)
        out, lse = pec.pec_attn_varlen(qd, kd[:tq], vd[:tq], cqd, max(len_q), causal, out_dtype=torch.float32)
        assert_close(out, lse, o_ref, l_ref, "packed batch of %d sequences" % n)


# one range more or less than a whole number, none, and ranges of all four lengths (the last argument)
RANGES = [
    (8, 2, [5, 1, 1, 1, 1, 1], [5, 511, 512, 513, 1, 4097], 512), (4, 1, [1, 32], [20481, 32], 512),
    (4, 1, [1, 1, 40], [61441, 1024, 40], 1024), (8, 2, [1, 200, 1, 1], [150016, 200, 2047, 2049], 2048),
    (4, 1, [1, 1], [900001, 4096], 4096), (8, 8, [1, 1], [8193, 1023], 512), (16, 1, [1] * 70, [600 + 13 * i for i in range(70)], 2048)]


@pytest.mark.parametrize("hq,hkv,len_q,len_k,keys", RANGES)
def test_key_ranges_of_every_length(hq, hkv, len_q, len_k, keys):
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    q, _, _ = synth.qkv(9960, int(cq[-1]), 1, hq, hkv)
    _, k, v = synth.qkv(9961, 1, int(ck[-1]), hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full(o_ref.shape, float("nan"), dtype=dt, device=DEV)
        lse = torch.full(l_ref.shape, float("nan"), dtype=torch.float32, device=DEV)
        pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV), True,
                               out_dtype=dt, out=out, lse=lse)
        assert_close(out, lse, o_ref, l_ref, "ranges of %d keys" % keys)


def test_list_with_an_item_heavier_than_its_buckets():
    len_q, len_k = [3] + [1] * 65 + [70], [2048 * 256 + 1] + [1] * 65 + [70]
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    q, _, _ = synth.qkv(9800, int(cq[-1]), 1, 2, 1)
    _, k, v = synth.qkv(9900, 1, int(ck[-1]), 2, 1)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    out, lse = pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV), True,
                                      out_dtype=torch.float32)
    assert_close(out, lse, o_ref, l_ref, "list of %d sequences" % len(len_q))


def test_offsets_that_are_not_monotone_stay_inside_the_arrays():
    """Clamped bounds: lengths that add up to more than there is, offsets below zero and beyond the end; out, lse and the
    workspace each between bytes that stay as they are."""
    hq, hkv, tq, tk = 4, 2, 64, 20000
    q, _, _ = synth.qkv(9950, tq, 1, hq, hkv)
    _, k, v = synth.qkv(9951, 1, tk, hq, hkv)
    cq = torch.tensor([0, 1, 40, 39, 40, 41, -5, 900, 64], dtype=torch.int32, device=DEV)
    ck = torch.tensor([0, 20000, 100, 20000, 0, 19999, 50000, -7, 20000], dtype=torch.int32, device=DEV)
    shape = pec.PecShape(hq, hkv, 128, pec.PEC_F32, 0.0, 0)
    need = pec.lib().pec_colocated_workspace_bytes(ctypes.byref(shape), cq.numel() - 1, tq, tk)
    out = torch.zeros((tq + 2, hq, 128), dtype=torch.float32, device=DEV)
    lse = torch.zeros((3, hq, tq), dtype=torch.float32, device=DEV)
    ws = torch.full((need + 8192,), 0xA5, dtype=torch.uint8, device=DEV)
    pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), cq, ck, True, out_dtype=torch.float32, out=out[1:-1], lse=lse[1],
                           workspace=ws[4096:-4096])
    torch.cuda.synchronize()
    assert not out[0].any() and not out[-1].any() and not lse[0].any() and not lse[2].any()
    assert bool((ws[:4096] == 0xA5).all()) and bool((ws[-4096:] == 0xA5).all())
    o_ref, _ = oracle.attention(q[:1], k, v, q_off=tk - 1, kv_off=0, causal=True)      # the one sequence with proper bounds
    assert np.abs(out[1:2].cpu().numpy() - o_ref).max() <= 2e-2


@pytest.mark.parametrize("hq,hkv,len_q,len_k,keys", RANGES)
def test_workspace_of_a_larger_batch(hq, hkv, len_q, len_k, keys):
    """One that was sized for more sequences, queries and keys is taken, and nothing behind what this batch needs is written."""
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    tq, tk = int(cq[-1]), int(ck[-1])
    q, _, _ = synth.qkv(9980, tq, 1, hq, hkv)
    _, k, v = synth.qkv(9981, 1, tk, hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    shape = pec.PecShape(hq, hkv, 128, pec.PEC_F32, 0.0, 0)
    need = [pec.lib().pec_colocated_workspace_bytes(ctypes.byref(shape), len(len_q) + n, tq + 40 * n, tk + 700 * n) for n in (0, 1, 9)]
    buffer = torch.full((need[-1],), 0xA5, dtype=torch.uint8, device=DEV)
    for size in need:
        out, lse = torch.full(o_ref.shape, float("nan"), device=DEV), torch.full(l_ref.shape, float("nan"), device=DEV)
        pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV), True,
                               out_dtype=torch.float32, out=out, lse=lse, workspace=buffer[:size])
        assert_close(out, lse, o_ref, l_ref, "workspace of %d bytes" % size)
        assert bool((buffer[need[0]:] == 0xA5).all())
