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
