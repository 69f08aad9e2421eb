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


@pytest.mark.parametrize("hq,hkv,n", [(8, 8, 2), (8, 8, 32), (8, 8, 33), (64, 32, 8), (64, 2, 2), (66, 2, 2), (6, 2, 21), (6, 2, 22), (33, 33, 7)])
def test_merge_in_the_launch(hq, hkv, n):
    """Ranges merged by the workgroup that is there last, on either side of its limits, against the merge by a second launch
    (a workspace without room for its words): the same bits for up to 24 ranges, which that one sums in the same order.  One
    workspace, filled with different bytes and used by steps of other shapes in between, and a graph replayed over it."""
    sk = n * 96 - 37
    q, k, v = [t.to(DEV) for t in synth.qkv(8500 + hq + n, 1, sk, hq, hkv)]
    o_ref, l_ref = oracle.attention(q.cpu(), k.cpu(), v.cpu(), causal=False)
    q2, k2, v2 = [t.to(DEV) for t in synth.qkv(8600, 1, 700, 8, 4)]
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    partials = n * hq * 129 * 4
    two = pec.pec_decode_splitkv(q, k, v, n_splits=n, workspace=ws[:partials])
    out, lse = torch.empty_like(two[0]), torch.empty_like(two[1])

    def check(what):
        torch.cuda.synchronize()
        assert_close(out, lse.reshape(hq, 1), o_ref, l_ref, what)
        assert n > 24 or (torch.equal(out, two[0]) and torch.equal(lse, two[1])), what
        out.fill_(float("nan"))
        lse.fill_(float("nan"))

    for fill in (0, 255, 90):
        ws.fill_(fill)
        for again in range(3):
            pec.pec_decode_splitkv(q, k, v, n_splits=n, out=out, lse=lse, workspace=ws)
            check((fill, again))
            pec.pec_decode_splitkv(q2, k2, v2, n_splits=2 + again, workspace=ws)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pec.pec_decode_splitkv(q, k, v, n_splits=n, out=out, lse=lse, workspace=ws)
    for again in range(3):
        graph.replay()
        check(again)
        pec.pec_decode_splitkv(q2, k2, v2, n_splits=3, workspace=ws)
