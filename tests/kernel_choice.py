"""The library's own choice of kernel (csrc/kernel_choice.hpp, plain C++) for a call of given sizes, so that a test can make
sure that its cases run on the kernel that they are about."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_15104_amd", "csrc")
COMPUTE_UNITS = 256
COLOC_RANGE = 4096
SOURCE = """
#include "kernel_choice.hpp"
extern "C" int dense(int cu, int hq, int hkv, int64_t sq, int64_t sk, int64_t delta, int causal) {
    return pec::rows_of_dense_call(cu, hq, hkv, sq, sk, delta, causal);
}
extern "C" int list(int cu, int hq, int hkv, int64_t batch, int64_t tq, int64_t tk, int64_t longest, int causal, int range) {
    return pec::rows_of_list_call(cu, hq, hkv, batch, tq, tk, longest, causal, range);
}
extern "C" int dense_heads(int cu, int hq, int hkv, int64_t sq, int64_t sk, int64_t delta, int causal) {
    return 1 << pec::log_heads_of_dense_call(cu, hq, hkv, sq, sk, delta, causal);
}
extern "C" int list_heads(int cu, int hq, int hkv, int64_t batch, int64_t tq) {
    return 1 << pec::log_heads_of_list_call(cu, hq, hkv, batch, tq);
}
extern "C" int by_sequence(int cu, int hq, int rows, int64_t batch, int64_t tq) {
    return pec::list_by_sequence(cu, hq, rows, batch, tq);
}
extern "C" int can_stop(int cu, int hq, int64_t sq, int64_t sk, int64_t delta, int causal, int64_t seg_tiles) {
    return pec::sweep_can_stop(cu, hq, sq, sk, delta, causal, seg_tiles);
}
extern "C" int spans(int cu, int hq, int hkv, int64_t sq, int64_t sk, int64_t delta, int causal) {
    return pec::spans_of_sweep(cu, hq, hkv, sq, sk, delta, causal).groups;
}
extern "C" int without_list(int cu, int rows, int hq, int64_t batch, int64_t tq) { return pec::batch_without_list(cu, rows, hq, batch, tq); }
extern "C" int range_keys_of(int cu, int rows, int hq, int hkv, int64_t batch, int64_t tq, int64_t tk) {
    return pec::range_of_mixed_call(cu, rows, hq, hkv, batch, tq, tk);
}
extern "C" int merged(int g, int64_t n) { return pec::merge_in_launch(g, n); }
extern "C" uint64_t mark(uint64_t seed, uint64_t n) { return pec::merge_mark(seed, n); }
extern "C" int64_t ranges(int cu, int hq, int hkv, int64_t sk) { return pec::decode_default_ranges(cu, hq, hkv, sk); }
extern "C" int split(int cu, int hq, int hkv, int64_t sk, int64_t n) { return pec::decode_on_split_kernel(cu, hq, hkv, sk, n); }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "choice.cpp"), os.path.join(d, "choice.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src], check=True)
        L = ctypes.CDLL(lib)
    i64 = ctypes.c_int64
    L.dense.argtypes = [ctypes.c_int] * 3 + [i64] * 3 + [ctypes.c_int]
    L.dense_heads.argtypes = L.dense.argtypes
    L.list_heads.argtypes = [ctypes.c_int] * 3 + [i64] * 2
    L.list.argtypes = [ctypes.c_int] * 3 + [i64] * 4 + [ctypes.c_int] * 2
    L.by_sequence.argtypes = [ctypes.c_int] * 3 + [i64] * 2
    L.can_stop.argtypes = [ctypes.c_int] * 2 + [i64] * 3 + [ctypes.c_int, i64]
    L.spans.argtypes = L.dense.argtypes
    L.without_list.argtypes = [ctypes.c_int] * 3 + [i64] * 2
    L.range_keys_of.argtypes = [ctypes.c_int] * 4 + [i64] * 3
    L.merged.argtypes = [ctypes.c_int, i64]
    L.mark.argtypes, L.mark.restype = [ctypes.c_uint64] * 2, ctypes.c_uint64
    L.ranges.argtypes, L.ranges.restype = [ctypes.c_int] * 3 + [i64], i64
    L.split.argtypes = [ctypes.c_int] * 3 + [i64] * 2
    return L


def dense_rows(hq, hkv, sq, sk, q_off=0, kv_off=0, causal=True):
    """Query rows per workgroup: 256 is fwd_il_kernel, 64 and 32 are fwd_split_kernel<2> and <1>."""
    delta = max(-sq - 1, min(q_off - kv_off, sk))
    return _lib().dense(COMPUTE_UNITS, hq, hkv, sq, sk, delta, int(causal))


def dense_heads(hq, hkv, sq, sk, q_off=0, kv_off=0, causal=True):
    """Query heads per work item of a call that runs on fwd_il_kernel."""
    return _lib().dense_heads(COMPUTE_UNITS, hq, hkv, sq, sk, max(-sq - 1, min(q_off - kv_off, sk)), int(causal))


def sweep_can_stop(hq, sq, sk, q_off, chunk, causal=True):
    """Whether a stop word can change what the resumable sweep does; if not it runs as a plain call."""
    return bool(_lib().can_stop(COMPUTE_UNITS, hq, sq, sk, max(-sq - 1, min(q_off, sk)), int(causal), chunk // 64))


def sweep_spans(hq, hkv, sq, sk, q_off, causal=True):
    """Workgroups of a resumable sweep that is cut into spans, 0 if it is not."""
    return _lib().spans(COMPUTE_UNITS, hq, hkv, sq, sk, max(-sq - 1, min(q_off, sk)), int(causal))


def batch_heads(hq, hkv, len_q):
    """The same for a packed or mixed batch."""
    return _lib().list_heads(COMPUTE_UNITS, hq, hkv, len(len_q), int(sum(len_q)))


def by_sequence(hq, rows, len_q):
    """Whether the work list of a batch keeps the items of a sequence together."""
    return bool(_lib().by_sequence(COMPUTE_UNITS, hq, rows, len(len_q), int(sum(len_q))))


def mixed_range(hq, hkv, len_q, len_k, causal=True):
    """Keys per range of the one-token sequences of a mixed batch."""
    return _lib().range_keys_of(COMPUTE_UNITS, mixed_rows(hq, hkv, len_q, len_k, causal), hq, hkv, len(len_q), int(sum(len_q)), int(sum(len_k)))


def without_list(rows, hq, len_q):
    """Whether the workgroups of a batch find their items in the offsets."""
    return bool(_lib().without_list(COMPUTE_UNITS, rows, hq, len(len_q), int(sum(len_q))))


def packed_rows(hq, hkv, lengths, hint=None, causal=True):
    total = int(sum(lengths))
    return _lib().list(COMPUTE_UNITS, hq, hkv, len(lengths), total, total, min(hint or max(lengths), total), int(causal), 0)


def mixed_rows(hq, hkv, len_q, len_k, causal=True):
    return _lib().list(COMPUTE_UNITS, hq, hkv, len(len_q), int(sum(len_q)), int(sum(len_k)), 0, int(causal), COLOC_RANGE)


def merged_in_launch(hq, hkv, sk, n_splits):
    """Whether a decode step of so many ranges is one launch."""
    return bool(decode_kernel_of(hq, hkv, sk, n_splits)[1] == "fwd_split_kernel" and n_splits <= 32 and _lib().merged(hq // hkv, n_splits))


def merge_mark(seed, n):
    """What the words of call number n of a process hold where the launch merges its own key ranges."""
    return _lib().mark(seed, n)


def decode_kernel_of(hq, hkv, sk, n_splits):
    """(key ranges, kernel) of a decode step; n_splits 0 is the library's choice."""
    n = n_splits or _lib().ranges(COMPUTE_UNITS, hq, hkv, sk)
    if _lib().split(COMPUTE_UNITS, hq, hkv, sk, n):
        return n, "fwd_split_kernel"
    return n, "decode_kernel" if hq // hkv <= 32 else "fwd_il_kernel"
