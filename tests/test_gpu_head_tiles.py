"""Work items of the pipelined kernel that hold 1, 2, 4 or 8 query heads of a KV group, at the edges of their 256, 128, 64
or 32 query positions.  Enough heads that every call has a work item for each compute unit."""
import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth
from test_gpu_underfilled import DEV, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,sq,sk,q_off,causal", [
    (512, 64, 127, 260, 133, True),      # 8 heads x 32 positions: last tile one position short
    (512, 64, 97, 65, 0, True),          # ... last tile with one position, rows past the last key
    (512, 128, 129, 190, 61, True),      # 4 heads x 64 positions: last tile with one position
    (512, 128, 63, 100, 0, False),       # ... no mask; so few items and keys that a head has an item of its own
    (512, 128, 127, 100, 0, False),      # ... no mask, last tile one position short
    (384, 32, 130, 130, 0, True),        # 12 heads per KV head: three work units of 4
    (256, 128, 257, 257, 0, True),       # 2 heads x 128 positions: last tile with one position
    (192, 32, 200, 70, 200, True),       # 6 heads per KV head, every key visible; a head has an item of its own
    (192, 32, 300, 70, 300, True),       # ... three work units of 2
    (512, 64, 130, 100, 0, False),       # a little more than one item of 8 heads per compute unit: one head each
    (264, 88, 90, 150, 20, True),        # 3 heads per KV head: one head x 256 positions, KV heads not a power of two
])
def test_items_of_several_heads_match_oracle(hq, hkv, sq, sk, q_off, causal):
    q, k, v = synth.qkv(7000 + sq, sq, sk, hq, hkv)
    o_ref, l_ref = oracle.attention(q, k, v, q_off=q_off, kv_off=0, causal=causal)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((sq, hq, 128), float("nan"), dtype=dt, device=DEV)       # every row must be written
        lse = torch.full((hq, sq), float("nan"), dtype=torch.float32, device=DEV)
        pec.pec_attn_chunk(qd, kd, vd, q_off, 0, causal, out_dtype=dt, out=out, lse=lse)
        assert_close(out, lse, o_ref, l_ref, "%s" % dt)
    cut = sk // 2                                                                   # folded in as two segments
    o_acc, l_acc = pec.pec_attn_chunk(qd, kd[:cut], vd[:cut], q_off, 0, causal, out_dtype=torch.float32)
    pec.pec_attn_chunk_merge(qd, kd[cut:], vd[cut:], q_off, cut, o_acc, l_acc, causal)
    assert_close(o_acc, l_acc, o_ref, l_ref, "two segments")


# prompts at the edges of 32, 64, 128 and 256 positions, a chunk behind a prefix, whole and cut caches
LEN_Q = [32, 1, 33, 64, 0, 65, 127, 1, 128, 129, 255, 1, 256, 257, 31, 63, 5, 700, 40]
LEN_K = [32, 5000, 33, 64, 7, 65, 127, 4097, 128, 129, 255, 9, 256, 257, 31, 63, 300, 700, 1000]


@pytest.mark.parametrize("hq,hkv,times", [(64, 8, 1), (32, 8, 1), (24, 2, 2), (16, 8, 2), (36, 6, 1), (8, 8, 2),   # one head
                                         (64, 8, 2), (32, 8, 3), (24, 2, 3), (16, 8, 5), (36, 6, 2)])
def test_mixed_batches_with_items_of_several_heads(hq, hkv, times):
    """The batch above, as often as it takes for an item per compute unit, and for 2.5 of them (tests/test_kernel_choice.py)."""
    len_q, len_k = LEN_Q * times, LEN_K * times
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    tq, tk = int(cq[-1]), int(ck[-1])
    q, _, _ = synth.qkv(7200 + hq, tq, 1, hq, hkv)
    _, k, v = synth.qkv(7300 + hq, 1, tk, hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    out = torch.full((tq, hq, 128), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((hq, tq), float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV),
                           True, out_dtype=torch.float32, out=out, lse=lse)
    assert_close(out, lse, o_ref, l_ref, "mixed batch %d / %d" % (hq, hkv))
