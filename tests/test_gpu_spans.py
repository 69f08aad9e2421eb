"""Sweeps with few query tiles and many keys, which are cut into one span of tile steps per workgroup: pieces that start and end
inside items, whole items between them, items of several KV heads, ragged ends, and every one of them stopped and continued."""
import numpy as np
import pytest
import torch

import test_gpu_parity as parity
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # s_q, s_kv, hq, hkv, q_off, chunk, causal
    (256, 20000, 4, 1, 19744, 4096, True),       # one query tile per head, several spans each, ragged key total
    (300, 16384, 4, 2, 16084, 1024, True),       # the second tile has 44 rows and is left between tiles only
    (520, 9000, 6, 3, 8400, 2048, True),         # three KV heads, keys end behind the last row's
    (256, 12345, 8, 8, 0, 4096, False),          # no mask
    (256, 16384, 40, 1, 16128, 1024, True),      # wide group on one KV head
    (1280, 6000, 64, 8, 4720, 1280, True),       # more items than compute units: whole items inside spans
    (257, 20000, 16, 2, 9000, 2048, True),       # half of the keys in the future
    (16700, 30000, 1, 1, 13300, 4096, True),     # 66 query tiles of a head: a workgroup finds its place in two rounds
    (16641, 9000, 2, 1, 0, 2048, False),         # the same without a mask, the last tile has one row
]


@pytest.mark.parametrize("case", CASES)
def test_spans_match_oracle_whole_and_stopped(case):
    s_q, s_kv, hq, hkv, q_off, chunk, causal = case
    # keys 20 log2 units and more above the bulk, around the ends of pieces and segments as anywhere else
    keys = np.random.default_rng(s_kv).integers(0, min(s_kv, q_off + 1) if causal else s_kv, size=24)
    outliers = [(int(j), int(r), int(a)) for j, r, a in zip(keys, np.linspace(0, s_q - 1, 24), np.tile([2, 4, 8], 8))]
    q, k, v = synth.qkv_with_outlier_keys(50 + s_q + s_kv, s_q, s_kv, hq, hkv, outliers)
    qd, kd, vd = parity.gpu(q, k, v)
    rows = np.unique(np.clip([0, 1, 31, 32, 255, 256, 511, 512, 16383, 16384, s_q // 2, s_q - 2, s_q - 1, *[o[1] for o in outliers[::3]]], 0, s_q - 1))
    runs = []
    for raised in (0, 1):
        stop = torch.full((1,), raised, dtype=torch.int32, device=DEV)
        for dt in (torch.bfloat16, torch.float32):
            out, lse, calls, hist = parity._resumable_run(qd, kd, vd, q_off, chunk, causal, stop, out_dtype=dt)
            assert bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(lse).all())
            assert calls == 1 if not raised else calls > 1 or chunk < 1024, hist
            assert hist[0] <= (s_q + 255) // 256 * hq and all(a >= b for a, b in zip(hist, hist[1:])), hist
            runs.append((out, lse))
    for heads in {0, hkv - 1}:
        for out, lse in runs:
            parity._sampled_check(qd, kd, vd, out, lse, q_off if causal else s_kv, rows, heads=heads, what=str(case))


@pytest.mark.parametrize("case", CASES)
def test_spans_keep_every_bit_when_stopped(case):
    s_q, s_kv, hq, hkv, q_off, chunk, causal = case
    q, k, v = synth.qkv(60 + s_q + s_kv, s_q, s_kv, hq, hkv)
    qd, kd, vd = parity.gpu(q, k, v)

    def other_work(call, ws):     # the workspace is the only thing that lives on
        saved = ws.clone()
        ws.fill_(0x5A)
        ws.copy_(saved)

    got = [parity._resumable_run(qd, kd, vd, q_off, chunk, causal, torch.full((1,), raised, dtype=torch.int32, device=DEV),
                                 out_dtype=torch.float32, between=other_work) for raised in (0, 1)]
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("case", CASES)
def test_sweeps_without_room_for_spans(case):
    """The least workspace inside a larger buffer: taken, whole and stopped, with the same bits; only its bytes are written, and
    they and lse are all the state there is.  A byte less is refused."""
    s_q, s_kv, hq, hkv, q_off, chunk, causal = case
    q, k, v = synth.qkv(70 + s_q + s_kv, s_q, s_kv, hq, hkv)
    qd, kd, vd = parity.gpu(q, k, v)
    least, best = [pec.pec_sp_resumable_workspace_bytes(qd, kd, least) for least in (True, False)]
    buffer = torch.full((best,), 0xA5, dtype=torch.uint8, device=DEV)
    pending = torch.zeros(1, dtype=torch.int32, device=DEV)
    got = []
    for raised in (0, 1):
        stop = torch.full((1,), raised, dtype=torch.int32, device=DEV)
        out, lse = torch.full((s_q, hq, 128), float("nan"), device=DEV), torch.full((hq, s_q), float("nan"), device=DEV)
        for call in range(400):
            pec.pec_sp_prefill_resumable(qd, kd, vd, q_off, chunk, out, lse, buffer[:least], pending, stop=stop, resume=call > 0,
                                         causal=causal)
            assert bool((buffer[least:] == 0xA5).all())
            if int(pending.item()) == 0:
                break
            saved = buffer[:least].clone(), lse.clone()
            buffer[:least].fill_(0x5A), lse.fill_(7)
            buffer[:least].copy_(saved[0]), lse.copy_(saved[1])
        assert int(pending.item()) == 0
        got.append((out, lse))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    rows = np.unique(np.clip([0, 31, 255, 256, s_q // 2, s_q - 1], 0, s_q - 1))
    parity._sampled_check(qd, kd, vd, *got[0], q_off if causal else s_kv, rows, heads=hkv - 1, what=str(case))
    with pytest.raises(pec.PecError) as refused:
        pec.pec_sp_prefill_resumable(qd, kd, vd, q_off, chunk, out, lse, buffer[:least - 1], pending, causal=causal)
    assert refused.value.status == -4
