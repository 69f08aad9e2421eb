"""The words by which a decode step's workgroups learn that all key ranges of a KV head are there, in a workspace that other
steps and other writers use in between: what an earlier step left never counts for a later one."""
import numpy as np
import pytest
import torch

import kernel_choice as choice
from oracle import reference as oracle
from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

DEV = "cuda:0"
# a step whose launch merges its ranges, and one whose partial results end inside the first one's words; on the same inputs it
# always leaves the same bytes there (LSEs, those of its last, empty ranges -inf)
HEADS, RANGES, KEYS = 8, 32, 9000
HEADS2, KV_HEADS2, RANGES2, KEYS2 = 2, 1, 129, 1000
WORDS = RANGES * HEADS * 129 * 4           # byte offset of the first step's words
END2 = RANGES2 * HEADS2 * 129 * 4          # end of the second step's partial results


def test_the_second_step_ends_inside_the_first_ones_words():
    assert choice.merged_in_launch(HEADS, HEADS, KEYS, RANGES) and choice.decode_kernel_of(HEADS, HEADS, KEYS, 0)[0] == RANGES
    assert not choice.merged_in_launch(HEADS2, KV_HEADS2, KEYS2, RANGES2)
    assert WORDS % 8 == 0 and WORDS + 8 < END2 < WORDS + 8 * RANGES * HEADS - 8


@pytest.mark.parametrize("seed", [1, 2**63, 2**64 - 1, 0x123456789abcdef0])
def test_no_word_of_an_earlier_step_holds_a_later_ones_mark(seed):
    marks = [choice.merge_mark(seed, n) for n in range(20000)]
    assert len(set(marks)) == len(marks)
    words, lse2 = np.zeros(RANGES * HEADS, dtype=np.uint64), np.full(2, -np.inf, np.float32).view(np.uint64)[0]
    for mark in marks[:50]:
        assert not (words == np.uint64(mark)).any()      # before the first workgroup of the step has run
        words[:] = mark
        words[:(END2 - WORDS) // 8] = lse2               # the step in between


@pytest.mark.gpu
def test_steps_that_share_a_workspace_and_overwrite_part_of_the_words():
    steps = []
    for seed, hq, hkv, sk, n in ((8700, HEADS, HEADS, KEYS, RANGES), (8701, HEADS2, KV_HEADS2, KEYS2, RANGES2)):
        q, k, v = [t.to(DEV) for t in synth.qkv(seed, 1, sk, hq, hkv)]
        two = pec.pec_decode_splitkv(q, k, v, n_splits=n, workspace=torch.empty(n * hq * 129 * 4, dtype=torch.uint8, device=DEV))
        o_ref, _ = oracle.attention(q.cpu(), k.cpu(), v.cpu(), causal=False)
        assert np.abs(two[0].cpu().numpy() - o_ref).max() <= 2e-2
        steps.append((q, k, v, n, two))
    ws = torch.zeros(1 << 18, dtype=torch.uint8, device=DEV)
    words = ws[WORDS:WORDS + 8 * RANGES * HEADS].view(torch.int64)
    seen = set()

    def run(which, what):
        q, k, v, n, two = steps[which]
        out, lse = torch.full_like(two[0], float("nan")), torch.full_like(two[1], float("nan"))
        pec.pec_decode_splitkv(q, k, v, n_splits=n, out=out, lse=lse, workspace=ws)
        assert torch.equal(out, two[0]) and torch.equal(lse, two[1]), what
        if which == 0:       # one number in all words, and no step's twice
            now = set(words.tolist())
            assert len(now) == 1 and not now & seen, what
            seen.update(now)

    for again in range(4):
        run(0, again)
        run(1, again)
    for head in range(HEADS):         # the same bytes up to any word of a KV head before each of two steps
        for first in range(0, RANGES, 5):
            for again in range(2):
                ws[:WORDS + 8 * (RANGES * head + first)].zero_()
                run(0, (head, first, again))
    saved = ws.clone()
    for again in range(3):            # a workspace put back to what it was
        run(0, again)
        ws.copy_(saved)


@pytest.mark.gpu
def test_captured_steps_have_the_same_bits_and_leave_the_words_alone():
    """A replay brings the arguments of the capture again; it merges by a second launch."""
    q, k, v = [t.to(DEV) for t in synth.qkv(8702, 1, KEYS, HEADS, HEADS)]
    want = pec.pec_decode_splitkv(q, k, v, n_splits=RANGES)
    ws = torch.zeros(1 << 18, dtype=torch.uint8, device=DEV)
    out, lse = torch.empty_like(want[0]), torch.empty_like(want[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pec.pec_decode_splitkv(q, k, v, n_splits=RANGES, out=out, lse=lse, workspace=ws)
    for again in range(3):
        out.fill_(float("nan")), lse.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(lse, want[1]), again
        assert not ws[WORDS:].any()
        pec.pec_decode_splitkv(q, k, v, n_splits=RANGES, out=out, lse=lse, workspace=ws)
        assert torch.equal(out, want[0]) and bool(ws[WORDS:WORDS + 8 * RANGES * HEADS].any())
        ws.zero_()
