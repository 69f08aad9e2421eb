"""Decode steps whose key ranges are shared out among the wavefronts of a workgroup, and their neighbours on the kernel with
one range per wavefront, at the edges: the last key range short, of one key or empty, one tile per wavefront and one more."""
import numpy as np
import pytest
import torch

from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth
from test_gpu_underfilled import DEV, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sk,hq,hkv,n_splits", [
    (65, 8, 8, 1), (64, 8, 8, 1),          # just over and just at the range length that changes kernels
    (255, 32, 8, 0), (257, 32, 8, 1),      # a tile per wavefront, the last one key short; the ninth tile with one key
    (4097, 32, 8, 0), (1000, 64, 2, 7),    # last range short
    (9 * 128 + 1, 16, 4, 10),              # last range with one key
    (500, 6, 3, 4),                        # last range empty
    (8192, 32, 8, 32), (8192, 32, 8, 33),  # as many workgroups as compute units, and one round more
    (300, 32, 1, 0), (300, 33, 1, 0),      # widest group of either kernel; the next one runs on the prefill kernel
    (700, 100, 100, 0),                    # 200 workgroups of one range and KV head
    (1500, 90, 90, 0), (1100, 150, 150, 0),    # 180 and 150 of them
    (2500, 90, 90, 0), (1400, 150, 150, 0),    # more than 768 keys per compute unit in all: a wavefront each
    (6145, 64, 32, 0), (6144, 64, 32, 0),      # on either side of that line
    (1100, 300, 300, 0), (600, 600, 300, 1),   # more KV heads than compute units
    (24 * 96, 6, 2, 24), (25 * 96, 6, 2, 25),   # as many ranges as one wavefront merges per head, and one more
    (96 * 23 - 95, 4, 4, 24),              # ... the last but one with one key, the last empty
    (40000, 8, 1, 1100),                   # more ranges than the merge has threads, many of them empty
])
def test_decode_ranges_match_oracle(sk, hq, hkv, n_splits):
    q, k, v = synth.qkv(8000 + sk + hq, 1, sk, hq, hkv)
    o_ref, l_ref = oracle.attention(q, k, v, causal=False)
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((1, hq, 128), float("nan"), dtype=dt, device=DEV)
        lse = torch.full((hq,), float("nan"), dtype=torch.float32, device=DEV)
        pec.pec_decode_splitkv(q.to(DEV), k.to(DEV), v.to(DEV), n_splits=n_splits, out_dtype=dt, out=out, lse=lse)
        assert_close(out, lse.reshape(hq, 1), o_ref, l_ref, "%s" % dt)
