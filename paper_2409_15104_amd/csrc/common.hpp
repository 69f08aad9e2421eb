// Types, constants, launch parameters and LDS layouts shared by the attention kernels (gfx950).
//
// MFMA 32x32x16 operand layout (lane l, l32 = l % 32, hl = l / 32):
//   A[M=32][K=16]: lane holds row l32, k-slots 8*hl .. 8*hl+7
//   B[K=16][N=32]: lane holds column l32, k-slots 8*hl .. 8*hl+7
//   C[M=32][N=32]: lane holds column l32, rows 8*(r/4) + 4*hl + r%4 for register r
// Scores are computed TRANSPOSED, S^T = K Q^T (keys along M, queries along N), so each lane owns one
// query column: row max / row sum are in-lane reductions plus one exchange between the two lane
// halves, and the running rescale of O is a per-lane scalar.  The contraction O^T += V^T P^T only
// needs A and B to agree on which key sits in which k-slot, so P (taken straight from the score
// registers) fixes the key order of the V^T operand: slots 0..3 <- keys 16*t2 + 4*hl + 0..3,
// slots 4..7 <- +8.
//
// LDS layout: a tile is 64 rows (keys) of 256 B (128 bf16).  K rows are XOR-swizzled at 16 B
// granularity (chunk c -> c ^ (key & 15)) for conflict-free b128 operand reads; V rows at 64 B
// granularity (segment s -> s ^ (key & 3)) for the transposing ds_read_b64_tr_b16 reads that
// deliver 4 consecutive keys of one head-dim column.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pec {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kHeadDim = 128;
constexpr int kBN = 64;               // keys per LDS tile
constexpr int kRowBytes = 256;        // one key row of 128 bf16
constexpr int kTileBytes = kBN * kRowBytes;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct WorkItem {        // one (sequence, query tile) of a packed or colocated batch, with all an attention kernel needs
    int32_t q0, len_q;   // query rows of the sequence, in the packed arrays
    int32_t k0, len_k;   // its keys; query i sits at position len_k - len_q + i
    int32_t qtile;       // query tile; negative: keys k0 ... of a one-token (decode) sequence, one range for each of the
                         // item's work units (as many per KV head as it has query heads)
    int32_t slot;        // where the first range's partial result goes
    int32_t pad[2];
};
static_assert(sizeof(WorkItem) == 32, "fwd_il_kernel fetches work items as eight words");

constexpr int32_t kSweepDone = 0x7fffffff;

struct FwdParams {
    const __bf16* q;
    const __bf16* k;
    const __bf16* v;
    void* out;              // [tokens, Hq, 128] bf16 or fp32 (may be null when only acc_out is wanted)
    float* lse;             // [Hq, lse_stride]
    const float* acc_in;    // running O (fp32, normalised) to continue from, or null
    const float* lse_in;    // running LSE matching acc_in
    float* acc_out;         // fp32 copy of the result (running state), or null
    int64_t lse_stride;     // tokens per head row in lse arrays
    int32_t sq, sk;         // dense mode: rows / keys of this call
    int32_t delta;          // q_off - kv_off, clamped to [-sq-1, sk]
    int32_t causal;
    int32_t n_q_heads, n_kv_heads, group;
    int32_t log_heads;      // fwd_il_kernel: 2^log_heads query heads of a KV group share a work item, (256 >> log_heads)
                            // query positions of each; group is a multiple of 2^log_heads
    int32_t n_items;        // query tiles (dense) or work-list capacity (varlen)
    int32_t out_f32;
    float scale_log2;       // scale * log2(e)
    // packed or colocated batch (work != null): work list built on the device
    const WorkItem* work;
    const int32_t* n_work;  // number of valid work items
    int32_t* sched;         // eight zeroed counters (fwd_il_kernel only): work items are drawn from them, one
                            // counter per XCD's share of the work order, instead of being dealt in fixed rounds
    // split-KV mode (kv_split_len > 0; not in fwd_simple_kernel): work item = key range
    // [item * kv_split_len, ...), partial results go to out / lse + item * split_*_stride
    int32_t kv_split_len;
    int64_t split_out_stride, split_lse_stride;   // elements
    // key ranges of a decode step whose last workgroup per KV head merges them (fwd_split_kernel; null: a kernel of its own
    // does): one word per KV head and range (last_workgroup()) and where the results go; `mark`: what this call writes there
    uint64_t* arrived;
    void* merged_out;
    float* merged_lse;
    int32_t merged_f32;
    // element strides of q / out / acc between rows and between heads (0 = the packed
    // [tokens, n_q_heads, 128] layout; not in fwd_simple_kernel, and fwd_split_kernel reads them for decode steps only)
    int64_t q_row_stride, q_head_stride;
    // colocated batch: partial results of the key ranges that one-token sequences with long caches are cut into
    float* part_out;            // [slots][n_q_heads][128] fp32
    float* part_lse;            // [slots][n_q_heads]
    int32_t range_len;          // keys per range, a multiple of 64
    // resumable sweep (dense mode, progress != null; fwd_il_kernel only): work item i has finished its first
    // progress[i] key segments of seg_tiles tiles each (kSweepDone: all of them) and continues from there, its
    // running state in acc_in / lse_in / l_part.  A nonzero *stop makes a workgroup end the item in hand at the next
    // segment boundary (state to acc_out / lse / l_part, progress updated) and take no further item; an item that
    // gets through its last key writes out / lse and takes one off *pending.  The state of a stopped item is kept
    // as the registers hold it -- un-normalised O, the softmax reference (log2 units) in the LSE slot, and the two
    // lane halves' partial denominators in l_part [n_q_heads][lse_stride][2] -- so a stop adds no rounding step.
    float* l_part;
    int32_t* progress;
    int32_t* pending;
    const int32_t* stop;
    int32_t seg_tiles;
    // resumable sweep cut into one span of tile steps per workgroup (fwd_il_kernel<kFwdSpan>): the first span_extra workgroups
    // take span_len + 1 steps, the others span_len; span_kvh steps per KV head.  A piece of an item leaves its fp32 result, or
    // its state, in one of its workgroup's two slots, slot_out [2 x workgroups][256][128] and slot_lse [2 x workgroups][256].
    // progress[w] steps of span w are done; words behind them say which items span_merge_kernel has merged.
    float* slot_out;
    float* slot_lse;
    int32_t span_len, span_extra, span_kvh;
    // a batch of up to 64 sequences without a work list (fwd_split_kernel<kSplitBatch>): its offsets, and, for the merge of split
    // sequences' key ranges, how many slots there are and where block 0 lists those sequences
    const int32_t* cu_q;
    const int32_t* cu_k;
    int32_t batch, total_q, total_k, slot_capacity;
    struct SplitSeq* split_seqs;
    int32_t* n_split;
    uint64_t mark;
};
struct SplitSeq {        // a one-token sequence whose keys are cut into ranges
    int32_t seq, slot0, n_ranges, pad;
};

// Tile steps of a query tile (in work order, number `item`) of a sweep cut into spans, at least one.
__device__ __forceinline__ int span_steps_of(const FwdParams& p, int item) {
    const int qt = p.causal ? p.n_items - 1 - item : item;
    const int keys = p.causal ? max(0, min(p.sk, min(p.sq, (qt + 1) * 256) + p.delta)) : p.sk;
    return max(1, (keys + kBN - 1) / kBN);
}
__device__ __forceinline__ int span_start(const FwdParams& p, int w) { return w * p.span_len + min(w, p.span_extra); }

// Where step `pos` of the whole call lies: work unit (KV head, query tile, head within its group, in this order) and tile step
// inside it.  Called by whole wavefronts; both results are uniform.
struct SpanPos {
    int unit, tile;
};
__device__ __forceinline__ SpanPos span_locate(const FwdParams& p, int pos) {
    const int lane = threadIdx.x & 63;
    const int kvh = pos / p.span_kvh;
    int left = pos - kvh * p.span_kvh;
    for (int item0 = 0;; item0 += 64) {
        const int own = item0 + lane < p.n_items ? span_steps_of(p, item0 + lane) * p.group : 0;
        int upto = own;                       // steps of the query tiles up to this lane's
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(upto, d);
            if (lane >= d) upto += y;
        }
        const uint64_t behind = __ballot(upto > left);
        if (behind != 0 || item0 + 64 >= p.n_items) {
            const int l = behind != 0 ? __builtin_ctzll(behind) : 63;
            const int in_tile = left - (__shfl(upto, l) - __shfl(own, l)), steps = __shfl(own, l) / p.group;
            const int head = in_tile / max(1, steps);
            return SpanPos{__builtin_amdgcn_readfirstlane((kvh * p.n_items + item0 + l) * p.group + head),
                           __builtin_amdgcn_readfirstlane(in_tile - head * steps)};
        }
        left -= __shfl(upto, 63);
    }
}

// Work order of the attention kernels.  The units of a launch are numbered KV-head-major, the heaviest items of a KV
// head first; consecutive block ids go round-robin over the 8 XCDs, each with an L2 of its own.  XCD x takes units
// unit(x, 0), unit(x, 1), ... unit(x, count - 1):
//  * 1, 2 or 4 KV heads: 8 / n XCDs per KV head, its units dealt to them in turn, each turn starting somewhere else (the
//    multiplicative hash: with a fixed start the one real unit per KV group of a decode key range, whose distance is the
//    group size, would always fall to the same XCDs).  (One contiguous range per XCD would
//    give the first XCD the heaviest items of the head and the last one the lightest: a causal 3072-row prefill of 4
//    query heads on one KV head spent 2x as long on the first XCD as on average.)
//  * otherwise one contiguous range per XCD: with 8 KV heads every L2 then holds one of them.
struct WorkOrder {
    int log_shares;       // log2 of the XCDs per KV head, -1: contiguous ranges
    int per_kvh;          // units per KV head
    int64_t total, count;
    __device__ __forceinline__ WorkOrder(int n_items, int group, int n_kv_heads) {
        per_kvh = n_items * group;
        total = (int64_t)per_kvh * n_kv_heads;
        log_shares = n_kv_heads == 1 ? 3 : n_kv_heads == 2 ? 2 : n_kv_heads == 4 ? 1 : -1;
        count = (total + 7) >> 3;     // with shares: ceil(per_kvh / shares), the same number
    }
    // unit number `i` < count of XCD x, or -1 if there is none
    __device__ __forceinline__ int64_t unit(int x, int64_t i) const {
        if (log_shares > 0) {
            const uint32_t turn = ((uint32_t)i * 2654435761u >> 29) + x;
            const int64_t j = (i << log_shares) + (turn & ((1u << log_shares) - 1));
            return j < per_kvh ? (int64_t)(x >> log_shares) * per_kvh + j : -1;
        }
        const int64_t u = x * count + i;
        return u < total ? u : -1;
    }
};

// One tile-load instruction: 16 bytes per lane from sbase + voff to LDS, lane i at lds_addr + 16 i (M0 holds the address,
// and needs one wait state before the load).
// A load may read its scalar base five wait states after a vector instruction (v_readlane, v_readfirstlane) wrote it at the
// earliest, and the compiler does not look inside asm.  In the tile loops (IN_LOOP) the base is the sum that a scalar add
// has just made.  Everywhere else it may have come out of a spill or a readfirstlane the instruction before: s_mov_b64 is
// interlocked and leaves it written by a scalar instruction.  (In the loops as well it costs 0.3 % of long calls and 1.2 %
// of a 512 x 2048 one; tests/test_sgpr_wait_states.py looks every load of the built library over.)
template <bool IN_LOOP>
__device__ __forceinline__ void dma16(const unsigned char* sbase, uint32_t voff, uint32_t lds_addr) {
    if constexpr (IN_LOOP)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                     :
                     : "s"(sbase), "v"(voff), "s"(lds_addr)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 %0, %0\n\tglobal_load_lds_dwordx4 %1, %0"
                     : "+s"(sbase)
                     : "v"(voff), "s"(lds_addr)
                     : "memory", "m0");
}

// Results that one workgroup writes and another one of the same launch reads, maybe on another XCD: accesses at device scope
// go past the L2 that would keep them, so that no cache needs to be written back or invalidated (a __threadfence on
// either side does that to the whole L2: a decode step of 4,096 keys took 28 instead of 10 us with them).  Stores are in
// place when the wavefront's vmcnt is zero.
__device__ __forceinline__ void store_shared(float* p, f32x4 x) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
        __hip_atomic_store(reinterpret_cast<uint64_t*>(p) + i, __builtin_bit_cast(uint64_t, f32x2{x[2 * i], x[2 * i + 1]}),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 load_shared(const float* p) {
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x2 y = __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        x[2 * i] = y[0];
        x[2 * i + 1] = y[1];
    }
    return x;
}

__device__ __forceinline__ uint32_t k_lds_off(int key, int chunk16) {
    return (uint32_t)(key * kRowBytes + ((chunk16 ^ (key & 15)) << 4));
}
__device__ __forceinline__ uint32_t v_lds_off(int key, int byte_in_row) {
    const int seg = byte_in_row >> 6;
    return (uint32_t)(key * kRowBytes + (((seg ^ (key & 3)) << 6) | (byte_in_row & 63)));
}

}  // namespace pec
