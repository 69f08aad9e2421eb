"""Work lists beyond what the builder keeps in LDS: more sequences than it holds at once, with cut caches among them, and an
item heavier than its buckets."""
import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth
from test_gpu_underfilled import DEV, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("len_q,len_k", [
    # 1,024 and more sequences: cut caches before, on and behind the 1,024th
    ([1 if i in (3, 1023, 1024, 1099) else i % 5 for i in range(1100)],
     [5000 + i if i in (3, 1023, 1024, 1099) else i % 5 + i % 3 for i in range(1100)]),
    # 2,047, 2,048 and 2,049 blocks of 256 keys
    ([2, 300], [2047 * 256, 300]), ([2, 1], [2048 * 256 - 3, 4097]), ([3, 0, 70], [2048 * 256 + 1, 0, 70]),
])
def test_large_work_lists(len_q, len_k):
    hq, hkv = 2, 1
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    tq, tk = int(cq[-1]), int(ck[-1])
    q, _, _ = synth.qkv(9100, tq, 1, hq, hkv)
    _, k, v = synth.qkv(9200, 1, tk, hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    out = torch.full((tq, hq, 128), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((hq, tq), float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV),
                           True, out_dtype=torch.float32, out=out, lse=lse)
    assert_close(out, lse, o_ref, l_ref, "mixed batch of %d sequences" % len(len_q))


# one, two and three items of a sequence, a whole number of tiles, none; caches of one range and of several items of ranges;
# keys without queries, a chunk behind a prefix
SEQ_Q = [257, 1, 0, 512, 1, 600, 1, 3, 256, 64]
SEQ_K = [257, 1, 40, 512, 4097, 600, 20000, 300, 256, 500]


@pytest.mark.parametrize("hq,hkv,n", [(16, 4, 520), (8, 8, 1030), (16, 2, 1024)])
def test_lists_by_sequence(hq, hkv, n):
    """Short sequences around a few long ones (also the 1,024th), so that the list is long and the oracle has little to do."""
    long = {n * i // len(SEQ_Q): i for i in range(len(SEQ_Q))} | {1023: 0, 1024: 6}
    len_q = [SEQ_Q[long[i]] if i in long else i % 4 for i in range(n)]
    len_k = [SEQ_K[long[i]] if i in long else i % 4 + i % 3 for i in range(n)]
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    q, _, _ = synth.qkv(9300, int(cq[-1]), 1, hq, hkv)
    _, k, v = synth.qkv(9400, 1, int(ck[-1]), hq, hkv)
    o_ref, l_ref = oracle.colocated(q, k, v, cq, ck, causal=True)
    out = torch.full(o_ref.shape, float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full(l_ref.shape, float("nan"), dtype=torch.float32, device=DEV)
    pec.pec_attn_colocated(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV),
                           True, out_dtype=torch.float32, out=out, lse=lse)
    assert_close(out, lse, o_ref, l_ref, "mixed batch of %d sequences" % n)
    _, k, v = synth.qkv(9500, 1, int(cq[-1]), hq, hkv)
    o_ref, l_ref = oracle.varlen(q, k, v, cq, causal=True)
    out, lse = pec.pec_attn_varlen(q.to(DEV), k.to(DEV), v.to(DEV), torch.from_numpy(cq).to(DEV), max(len_q), True,
                                   out_dtype=torch.float32)
    assert_close(out, lse, o_ref, l_ref, "packed batch of %d sequences" % n)
