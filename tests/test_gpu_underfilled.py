"""Calls with fewer query tiles than compute units, which share the keys of a tile out among the wavefronts of a
workgroup, at the edges of their tiles (32 or 64 rows, 32 keys, 8 key streams), and calls just large enough for the
pipelined kernel at the same edges."""
import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL_O, TOL_LSE = 2e-2, 1e-3


def assert_close(out, lse, o_ref, l_ref, what):
    o, l = out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    fin = np.isfinite(l_ref)
    assert np.array_equal(np.isfinite(l), fin), what
    assert np.abs(o - o_ref).max() <= TOL_O, what
    if fin.any():
        assert (np.abs(l[fin] - l_ref[fin]) / np.maximum(1.0, np.abs(l_ref[fin]))).max() <= TOL_LSE, what


@pytest.mark.parametrize("sq,sk,q_off,kv_off,causal,hq,hkv", [
    (1, 1, 0, 0, True, 8, 8),
    (31, 33, 2, 0, True, 8, 2),            # one row tile, second key tile with one key
    (33, 255, 222, 0, True, 4, 1),         # second row tile with one row, last stream one key short
    (32, 257, 225, 0, True, 8, 8),         # ninth key tile (second step of the first stream) with one key
    (65, 512, 447, 0, True, 3, 3),         # three KV heads: contiguous ranges of the work order
    (100, 700, 90, 0, True, 8, 2),         # later key tiles wholly in the future
    (96, 64, 0, 500, True, 8, 2),          # segment wholly in the future
    (80, 300, 0, 40, True, 8, 2),          # the first rows see nothing
    (50, 90, 0, 0, False, 16, 4),          # no mask, ragged keys
    (70, 0, 0, 0, True, 8, 8),             # no keys
    (256, 300, 44, 0, True, 64, 4),        # 64-row workgroups, one per compute unit
    (193, 543, 350, 0, True, 64, 8),       # 64-row workgroups, the last one with a single row
    (224, 256, 0, 0, False, 64, 64),       # 64-row workgroups, half a row tile at the end, no mask
    (40, 100, 0, 0, False, 256, 1),        # 64-row workgroups on one KV head, no mask
    (130, 200, 70, 0, True, 256, 64),      # enough heads for the pipelined kernel: ragged last row tile
    (257, 321, 64, 0, True, 128, 128),     # the same, second row tile with one row
    (300, 100, 0, 0, False, 256, 1),       # the same on one KV head, no mask
])
def test_underfilled_calls_match_oracle_alone_and_merged(sq, sk, q_off, kv_off, causal, hq, hkv):
    q, k, v = synth.qkv(6000 + 7 * sq + sk, sq, max(sk, 1), hq, hkv)
    k, v = k[:sk], v[:sk]
    o_ref, l_ref = oracle.attention(q, k, v, q_off=q_off, kv_off=kv_off, causal=causal)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((sq, hq, 128), float("nan"), dtype=dt, device=DEV)       # every row must be written
        lse = torch.full((hq, sq), float("nan"), dtype=torch.float32, device=DEV)
        pec.pec_attn_chunk(qd, kd, vd, q_off, kv_off, causal, out_dtype=dt, out=out, lse=lse)
        assert_close(out, lse, o_ref, l_ref, "whole, %s" % dt)
    cut = sk // 3                                                                   # folded in as two segments
    o_acc, l_acc = pec.pec_attn_chunk(qd, kd[:cut], vd[:cut], q_off, kv_off, causal, out_dtype=torch.float32)
    final = torch.full((sq, hq, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    pec.pec_attn_chunk_merge(qd, kd[cut:], vd[cut:], q_off, kv_off + cut, o_acc, l_acc, causal, out_final=final)
    assert_close(o_acc, l_acc, o_ref, l_ref, "two segments, running state")
    assert_close(final, l_acc, o_ref, l_ref, "two segments, final")


def test_late_jumps_of_the_row_maximum_in_single_key_streams():
    """Keys 16 ... 130 log2 units above the bulk: the softmax reference of single key streams jumps, early and late, and
    the merge of the streams has to weigh them against each other."""
    sq, sk, hq, hkv = 64, 1500, 8, 2
    outliers = [(5, 3, 2), (300, 40, 8), (700, 40, 4), (1023, 10, 8), (1024, 11, 1), (1300, 60, 8), (1440, 63, 2)]
    q, k, v = synth.qkv_with_outlier_keys(6100, sq, sk, hq, hkv, outliers)
    o_ref, l_ref = oracle.attention(q, k, v, q_off=sk - sq, kv_off=0, causal=True)
    out, lse = pec.pec_attn_chunk(q.to(DEV), k.to(DEV), v.to(DEV), sk - sq, 0, True, out_dtype=torch.float32)
    assert_close(out, lse, o_ref, l_ref, "outlier keys")


@pytest.mark.parametrize("hq,hkv", [(8, 1), (8, 2), (4, 4), (6, 3), (80, 2), (40, 1)])
def test_small_mixed_batches_for_every_deal_of_kv_heads_to_xcds(hq, hkv):
    """Prompts at row-tile edges, a chunk behind a prefix, decode steps with whole and cut caches; groups wider than 32
    and than 64 heads leave the 32- and 64-row workgroups out."""
    len_q = [32, 1, 33, 1, 0, 64, 1, 65, 5]
    len_k = [32, 4096, 33, 4097, 7, 64, 9000, 65, 300]
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    tq, tk = int(cq[-1]), int(ck[-1])
    q, _, _ = synth.qkv(6200 + hq, tq, 1, hq, hkv)
    _, k, v = synth.qkv(6300 + hq, 1, tk, hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    out = torch.full((tq, hq, 128), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((hq, tq), float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV),
                           True, out_dtype=torch.float32, out=out, lse=lse)
    assert_close(out, lse, o_ref, l_ref, "mixed batch %d / %d" % (hq, hkv))
