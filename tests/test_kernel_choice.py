"""The GPU tests that are about one kernel run on it: the library's own choice, asked for the sizes that they use."""
import ctypes
import random

import pytest

import kernel_choice as choice
from paper_2409_15104_amd import binding
import test_gpu_decode_ranges as decode
import test_gpu_head_tiles as head_tiles
import test_gpu_pipelined_kernel as pipelined
import test_gpu_small_batches as small_batches
import test_gpu_small_sweeps as small_sweeps
import test_gpu_spans as spans
import test_gpu_underfilled as underfilled
import test_gpu_work_list as work_list


@pytest.fixture(scope="module")
def lib():
    return binding.lib()


def cases(test):
    (mark,) = [m for m in test.pytestmark if m.name == "parametrize"]
    return [tuple(c) for c in mark.args[1]]


@pytest.mark.parametrize("hkv", pipelined.KV_HEADS)
def test_pipelined_kernel_cases(hkv):
    hq = pipelined.HQ
    for (sq, sk, q_off, causal), _ in pipelined.JUMPS:
        cut = sk // 2
        for n, kv_off in ((sk, 0), (cut, 0), (sk - cut, cut)):
            assert choice.dense_rows(hq, hkv, sq, n, q_off, kv_off, causal) == 256
            assert choice.dense_heads(hq, hkv, sq, n, q_off, kv_off, causal) == hq // hkv
    for q_off, kv_off, sq, sk in pipelined.MASKS:
        assert choice.dense_rows(hq, hkv, sq, sk, q_off, kv_off) == 256
        assert choice.dense_heads(hq, hkv, sq, sk, q_off, kv_off) == hq // hkv
    for times, heads in ((1, 1), (2, hq // hkv)):
        assert choice.packed_rows(hq, hkv, pipelined.BATCH_Q * times) == 256
        assert choice.mixed_rows(hq, hkv, pipelined.BATCH_Q * times, pipelined.BATCH_K * times) == 256
        assert choice.batch_heads(hq, hkv, pipelined.BATCH_Q * times) == heads


def test_head_tile_cases_run_on_the_pipelined_kernel():
    heads = []
    for hq, hkv, sq, sk, q_off, causal in cases(head_tiles.test_items_of_several_heads_match_oracle):
        assert choice.dense_rows(hq, hkv, sq, sk, q_off, 0, causal) == 256
        heads.append(choice.dense_heads(hq, hkv, sq, sk, q_off, 0, causal))
    assert heads == [8, 8, 4, 1, 4, 4, 2, 1, 2, 1, 1]
    heads = []
    for hq, hkv, times in cases(head_tiles.test_mixed_batches_with_items_of_several_heads):
        assert choice.mixed_rows(hq, hkv, head_tiles.LEN_Q * times, head_tiles.LEN_K * times) == 256
        heads.append(choice.batch_heads(hq, hkv, head_tiles.LEN_Q * times))
    assert heads == [1] * 6 + [8, 4, 4, 2, 2]


@pytest.mark.parametrize("case,heads", [
    # fewer items than compute units: by the keys
    ((64, 8, 322, 767), 1), ((64, 8, 322, 768, 446), 8), ((64, 8, 322, 768, 445), 1), ((16, 4, 700, 700, 0, 0, False), 1),
    # a little more than a whole number of items per compute unit and nearly equal lengths
    ((64, 8, 1047, 11729, 0, 0, False), 1), ((64, 8, 2073, 7188, 5115), 1), ((128, 8, 1560, 16985, 15425), 1),
    # ... exactly a whole number; more than 0.35 above it
    ((64, 8, 1024, 11729, 0, 0, False), 8), ((64, 8, 1409, 11729, 0, 0, False), 8), ((64, 8, 1400, 11729, 0, 0, False), 8),
    # ... lengths from one to all keys, a short call with a mask
    ((64, 8, 2118, 2118), 8), ((128, 8, 598, 1680, 1082), 8), ((128, 8, 598, 2048, 1450), 1),
    ((40, 8, 1047, 11729, 0, 0, False), 1),   # groups of five
])
def test_heads_per_work_item_of_dense_calls(case, heads):
    assert choice.dense_heads(*case) == heads


def test_underfilled_cases_cover_all_three_workgroups():
    rows = [choice.dense_rows(hq, hkv, sq, sk, q_off, kv_off, causal) for sq, sk, q_off, kv_off, causal, hq, hkv in
            cases(underfilled.test_underfilled_calls_match_oracle_alone_and_merged)]
    assert rows == [32] * 10 + [64] * 4 + [256] * 3
    batch = ([32, 1, 33, 1, 0, 64, 1, 65, 5], [32, 4096, 33, 4097, 7, 64, 9000, 65, 300])
    assert {hq // hkv: choice.mixed_rows(hq, hkv, *batch) for hq, hkv in
            cases(underfilled.test_small_mixed_batches_for_every_deal_of_kv_heads_to_xcds)} == {8: 32, 4: 32, 1: 32, 2: 32, 40: 64}


def test_decode_cases_run_on_all_kernels():
    kernels = {c: choice.decode_kernel_of(c[1], c[2], c[0], c[3])[1] for c in cases(decode.test_decode_ranges_match_oracle)}
    others = {(64, 8, 8, 1), (8192, 32, 8, 33), (2500, 90, 90, 0), (1400, 150, 150, 0), (6145, 64, 32, 0), (1100, 300, 300, 0),
              (600, 600, 300, 1), (40000, 8, 1, 1100)}
    for c, kernel in kernels.items():
        assert kernel == ("fwd_il_kernel" if c == (300, 33, 1, 0) else "decode_kernel" if c in others else "fwd_split_kernel"), c


@pytest.mark.parametrize("hq,hkv", [(8, 8), (32, 8), (64, 8), (8, 2), (8, 1), (4, 1), (256, 2)])
def test_workspace_of_a_mixed_batch_does_for_all_smaller_ones(lib, hq, hkv):
    shape = binding.PecShape(hq, hkv, 128, binding.PEC_F32, 0.0, 0)
    need = lambda *totals: lib.pec_colocated_workspace_bytes(ctypes.byref(shape), *totals)  # noqa: E731
    assert (hq, hkv) != (8, 2) or need(7, 5387, 43041) >= need(7, 125, 40367)
    rng = random.Random(23)
    for _ in range(5000):
        large = [int(2 ** rng.uniform(0, top)) for top in (9, 18, 21)]
        small = [rng.choice((n, n - 1, rng.randint(0, n))) for n in large]
        assert need(*large) >= need(*small), (large, small)
        for rows in (32, 64, 256):       # what the smaller one's ranges need has room too
            keys = choice._lib().range_keys_of(choice.COMPUTE_UNITS, rows, hq, hkv, *small)
            slots = small[2] // keys + small[0]
            assert need(*large) >= slots * hq * 129 * 4 + (small[1] // rows + small[0] + slots + 1) * 32, (large, small)


def test_a_dominating_prompt_counts_by_its_own_length():
    lengths = [9622] + [6] * 10 + [3]      # 32-row workgroups took 243 us, these take 197
    assert choice.packed_rows(5, 5, lengths) == 64


def test_lists_by_sequence_cases():
    for hq, hkv, n in cases(work_list.test_lists_by_sequence):
        len_q = [1] * n + work_list.SEQ_Q       # at least as few queries as the test has
        assert choice.mixed_rows(hq, hkv, len_q, len_q) == choice.packed_rows(hq, hkv, len_q) == 256
        assert choice.by_sequence(hq, 256, [1] * n) and not choice.by_sequence(hq, 64, [1] * n)
    assert not choice.by_sequence(32, 256, [1000] * 29) and choice.by_sequence(32, 256, [1000] * 30)


def test_merge_in_the_launch_cases():
    got = [choice.merged_in_launch(hq, hkv, n * 96 - 37, n) for hq, hkv, n in cases(decode.test_merge_in_the_launch)]
    assert got == [True, True, False, True, True, False, True, False, True]


def test_sweeps_that_cannot_stop_are_those_whose_tiles_have_no_boundary_to_stop_at():
    """Against a restatement of where fwd_il_kernel lets a tile be left (its stop_limit), tile by tile: this holds the rule for a
    whole call to it, not to the kernel, whose own limits test_gpu_small_sweeps.py sees in the number of calls."""
    rng, left = random.Random(17), 0
    for _ in range(20000):
        hq, sq, sk = rng.choice((1, 4, 8, 64)), rng.randint(1, 1500), rng.randint(0, 4000)
        q_off, causal = rng.randint(0, 4000), rng.random() < 0.8
        chunk = 64 * rng.choice((4, 15, 16, 17, 20, rng.randint(1, 40)))
        delta, seg = max(-sq - 1, min(q_off, sk)), chunk // 64
        stops = (-(-sq // 256) * hq + 7) // 8 > 32
        for row0 in range(0, sq - 255, 256):
            n_tiles = -(-(max(0, min(sk, row0 + 255 + delta + 1)) if causal else sk) // 64)
            whole = min(sk // 64, max(0, row0 + delta + 1) // 64) if causal else sk // 64
            seen = min(n_tiles, max(0, row0 + 31 + delta + 64) // 64) if causal else n_tiles
            stops |= seg >= 16 and seg <= min(max(0, min(whole - 1, seen - 1)) & ~1, n_tiles - 1)
        assert choice.sweep_can_stop(hq, sq, sk, q_off, chunk, causal) == stops
        left += not stops
    assert 2000 < left < 18000


def test_small_sweep_cases():
    got = [choice.sweep_can_stop(hq, sq, sk, q_off, chunk, causal) for sq, sk, hq, hkv, q_off, chunk, causal, _ in
           cases(small_sweeps.test_sweeps_around_the_line_of_those_that_can_stop)]
    assert got == [False, True, False, True, False, False, False, False, False, True]
    assert choice.sweep_spans(8, 1, 256, 16384, 16128) > 0


def test_span_cases():
    got = [(choice.sweep_spans(hq, hkv, sq, sk, q_off, causal), choice.sweep_can_stop(hq, sq, sk, q_off, chunk, causal))
           for sq, sk, hq, hkv, q_off, chunk, causal in spans.CASES]
    assert all(groups >= 16 and can_stop for groups, can_stop in got)
    assert {causal for sq, *_, causal in spans.CASES if sq > 64 * 256} == {True, False}     # a wavefront's lanes, one tile each


def test_workspaces_of_sweeps_with_and_without_room_for_spans(lib):
    """The least one is the running state and a word per tile; the other one has room for the pieces of any number of spans."""
    rng = random.Random(29)
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    for _ in range(2000):
        hq, s_q = rng.choice((1, 4, 8, 32, 64)), int(2 ** rng.uniform(0, 18))
        shape = binding.PecShape(hq, 1, 128, binding.PEC_BF16, 0.0, 0)
        least, best = [f(ctypes.byref(shape), s_q) for f in (lib.pec_sp_resumable_workspace_bytes, lib.pec_sp_resumable_best_workspace_bytes)]
        assert least == 512 * s_q * hq + up(8 * s_q * hq) + up(4 * -(-s_q // 256) * hq)
        spans = choice.sweep_spans(hq, 1, s_q, 1 << 20, 0, False)
        assert best >= max(least, spans * (2 * 256 * 131 * 4 + 36))
        assert best <= max(least, 70_000_000) and best >= lib.pec_sp_resumable_best_workspace_bytes(ctypes.byref(shape), s_q - 1)


def test_small_batch_cases_run_with_and_without_a_list():
    got = []
    for n, hq, hkv, first in cases(small_batches.test_small_batches_match_oracle):
        len_q, len_k = small_batches.lengths(n, first)
        rows = choice.packed_rows(hq, hkv, len_q), choice.mixed_rows(hq, hkv, len_q, len_k)
        got.append((rows, *[choice.without_list(r, hq, len_q) for r in rows]))
    assert [g[1:] for g in got] == [(True, True)] * 7 + [(False, False)] * 4
    assert {r for g in got[:7] for r in g[0]} == {32, 64}
    assert not choice.without_list(256, 1, [8] * 8)


def test_key_range_cases_have_ranges_of_every_length():
    assert [choice.mixed_range(*c[:4]) for c in small_batches.RANGES] == [c[4] for c in small_batches.RANGES]
    assert choice.mixed_range(32, 8, [1000] * 100 + [1], [1000] * 100 + [50000]) == 4096      # on fwd_il_kernel


@pytest.mark.parametrize("hq,hkv,batch,tq,tk", [(8, 2, 6, 10, 5635), (64, 8, 3, 80, 400000), (8, 1, 40, 3000, 90000), (32, 8, 300, 200000, 900000)])
def test_workspace_of_a_mixed_batch_holds_the_slots_of_every_choice(lib, hq, hkv, batch, tq, tk):
    need = lib.pec_colocated_workspace_bytes(ctypes.byref(binding.PecShape(hq, hkv, 128, binding.PEC_F32, 0.0, 0)), batch, tq, tk)
    for rows in (32, 64, 256):
        keys = choice._lib().range_keys_of(choice.COMPUTE_UNITS, rows, hq, hkv, batch, tq, tk)
        slots = tk // keys + batch
        assert need >= slots * hq * 129 * 4 + (tq // rows + batch + slots + 1) * 32
