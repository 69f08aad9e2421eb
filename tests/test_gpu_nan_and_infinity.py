"""NaN and infinity in the operands come out alike whichever way a call is cut: rows whose weights are NaN are NaN, the others
are as if nothing were there."""
import pytest
import torch

from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAN, INF = float("nan"), float("inf")

PLANTS = ["a query row", "a key", "an infinite key", "a value", "a whole head's queries"]


def plant(what, q, k, v, group, key):
    """`key`: one that every row sees."""
    if what == "a query row":
        q[q.shape[0] // 2, 0, 5] = NAN
        q[-1, -1] = NAN
    elif what == "a key":
        k[key, -1, 77] = NAN
    elif what == "an infinite key":      # scores of +inf (weights NaN) and -inf (weight 0), by the sign of the query's element
        k[key, 0, 3] = INF
    elif what == "a value":
        v[key, 0, 9] = NAN
    else:
        q[:, :group] = NAN


def same_kind(got, want, what):
    """NaN and infinities at the same places, numbers within the rounding of the weights to bf16 (2**-9 each, fp32 results)."""
    got, want = got.double(), want.double()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf()), what
    fin = want.isfinite()
    assert bool(((got - want).abs() <= 2e-2)[fin].all()), what


@pytest.mark.parametrize("what", PLANTS)
@pytest.mark.parametrize("s_q,s_kv,hq,hkv,q_off,chunk", [(256, 20000, 4, 1, 19744, 4096), (520, 9000, 6, 3, 8400, 2048),
                                                         (448, 448, 8, 1, 0, 448)])
def test_sweeps_cut_and_uncut(s_q, s_kv, hq, hkv, q_off, chunk, what):
    """The sweep (cut into spans, or without anything to stop at), whole and stopped after every segment, and the plain call."""
    q, k, v = [t.to(DEV) for t in synth.qkv(700 + s_kv, s_q, s_kv, hq, hkv)]
    plant(what, q, k, v, hq // hkv, 0)
    o_ref, l_ref = pec.pec_sp_prefill(q, k, v, q_off, chunk, out_dtype=torch.float32)
    assert o_ref.isnan().any()
    ws = torch.empty(pec.pec_sp_resumable_workspace_bytes(q, k), dtype=torch.uint8, device=DEV)
    pending = torch.zeros(1, dtype=torch.int32, device=DEV)
    for raised in (0, 1):
        stop = torch.full((1,), raised, dtype=torch.int32, device=DEV)
        out, lse = torch.zeros_like(o_ref), torch.zeros_like(l_ref)
        for call in range(400):
            pec.pec_sp_prefill_resumable(q, k, v, q_off, chunk, out, lse, ws, pending, stop=stop, resume=call > 0)
            if int(pending.item()) == 0:
                break
        same_kind(out, o_ref, "out, stop %d" % raised)
        same_kind(lse, l_ref, "lse, stop %d" % raised)


# caches around the lengths at which they are cut into ranges, of 512, 1024, 2048 and 4096 keys (the last: more rows per workgroup)
@pytest.mark.parametrize("what", PLANTS)
@pytest.mark.parametrize("hq,hkv,len_q,len_k", [
    (8, 2, [5, 1, 1], [5, 600, 4000]), (4, 1, [1, 1, 40], [61441, 1025, 40]), (8, 2, [1, 200, 1], [150016, 200, 2049]),
    (32, 8, [1000] * 40 + [1, 1], [1000] * 40 + [50000, 4097])])
def test_decode_steps_of_a_mixed_batch_cut_and_uncut(hq, hkv, len_q, len_k, what):
    """Every one-token sequence, cut into ranges or not, against the same decode step in one range."""
    cq, ck = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
    q, _, _ = [t.to(DEV) for t in synth.qkv(9970, int(cq[-1]), 1, hq, hkv)]
    _, k, v = [t.to(DEV) for t in synth.qkv(9971, 1, int(ck[-1]), hq, hkv)]
    steps = [i for i, n in enumerate(len_q) if n == 1]
    for i in steps:
        plant(what, q[int(cq[i]):int(cq[i + 1])], k[int(ck[i]):int(ck[i + 1])], v[int(ck[i]):int(ck[i + 1])], hq // hkv, len_k[i] // 3)
    out, lse = pec.pec_attn_colocated(q, k, v, torch.from_numpy(cq).to(DEV), torch.from_numpy(ck).to(DEV), out_dtype=torch.float32)
    for i in steps:
        row = slice(int(cq[i]), int(cq[i + 1]))
        keys = slice(int(ck[i]), int(ck[i + 1]))
        o_ref, l_ref = pec.pec_decode_splitkv(q[row], k[keys], v[keys], n_splits=1)
        assert o_ref.isnan().any()
        same_kind(out[row], o_ref, (i, len_k[i]))
        if len_k[i] <= 4096:
            same_kind(lse[:, row].reshape(-1), l_ref, (i, len_k[i]))
