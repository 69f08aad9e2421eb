"""Resumable sweeps around the line between those that a stop word can interrupt and those that run as a plain call."""
import pytest
import torch

import test_gpu_parity as parity
from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("sq,sk,hq,hkv,q_off,chunk,causal,calls", [
    (256, 1152, 2, 1, 896, 1024, True, 1),     # the 256 rows see 14 whole tiles, the boundary lies behind tile 16
    (256, 1408, 2, 1, 1216, 1024, True, 2),    # 19 whole tiles: the boundary can be cut at
    (255, 4096, 8, 2, 3841, 1024, True, 1),    # no whole query tile
    (256, 3000, 4, 4, 0, 1024, False, 3),
    (700, 2900, 4, 1, 2200, 960, True, 1),     # segments of 15 tiles
    (448, 448, 8, 1, 0, 448, True, 1),
    (1, 100, 3, 3, 99, 64, True, 1),
    (256, 16384, 8, 1, 16128, 512, True, 1),   # would be cut into spans if there were something to stop at
    (513, 900, 64, 8, 0, 1024, False, 1),      # more rows and heads, one segment
    (2048, 1000, 40, 8, 0, 128, True, 2),      # more items than compute units: the second of a workgroup is left out
])
def test_sweeps_around_the_line_of_those_that_can_stop(sq, sk, hq, hkv, q_off, chunk, causal, calls):
    q, k, v = synth.qkv(900 + sq + sk, sq, sk, hq, hkv)
    o_ref, l_ref = oracle.attention(q, k, v, q_off=q_off, kv_off=0, causal=causal)
    qd, kd, vd = parity.gpu(q, k, v)
    for raised in (0, 1):
        stop = torch.full((1,), raised, dtype=torch.int32, device=DEV)
        for dt in (torch.bfloat16, torch.float32):
            out, lse, n, hist = parity._resumable_run(qd, kd, vd, q_off, chunk, causal, stop, out_dtype=dt)
            assert n == (calls if raised else 1), hist
            parity.assert_close(out, lse, o_ref, l_ref, "stop %d, %s" % (raised, dt))
    # a call that resumes a finished sweep does nothing
    ws = torch.empty(pec.pec_sp_resumable_workspace_bytes(qd, kd), dtype=torch.uint8, device=DEV)
    pending = torch.full((1,), -7, dtype=torch.int32, device=DEV)
    clear = torch.zeros(1, dtype=torch.int32, device=DEV)
    pec.pec_sp_prefill_resumable(qd, kd, vd, q_off, chunk, out, lse, ws, pending, stop=clear, causal=causal)
    out.fill_(7), lse.fill_(7)
    pec.pec_sp_prefill_resumable(qd, kd, vd, q_off, chunk, out, lse, ws, pending, stop=clear, resume=True, causal=causal)
    assert int(pending.item()) == 0 and bool((out == 7).all()) and bool((lse == 7).all())
