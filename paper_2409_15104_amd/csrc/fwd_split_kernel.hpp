// Blockwise attention forward kernel for calls that leave most of the chip idle (gfx950).
//
// The pipelined kernel (fwd_kernel_il.hpp) gives one workgroup 256 query rows and the whole key range: a call with
// few rows and heads has fewer such work items than there are compute units, and its time is the serial walk of one
// workgroup over all keys.  Here a workgroup takes only 32 * NT query rows (NT = 1 or 2) and its 8 wavefronts share
// the KEYS out among themselves: wavefront w works on the 32-key tiles w, w + 8, w + 16, ... for all of the
// workgroup's rows, with an online softmax of its own; the eight partial results of a row are merged by log-sum-exp
// in LDS at the end, so nothing but the result leaves the workgroup and no workspace is needed.
//
// Every wavefront has a private 8 KiB LDS stage for K and one for V and there is no barrier in the loop: K(j+1) is
// requested as soon as the scores of tile j have read K(j), V(j+1) as soon as O += P(j) V(j) has read V(j), and the loop's
// own waits are counted so that the other of the two may still be on its way.  That holds in the build only for NT = 2 on
// batches.  Elsewhere registers loaded ahead of the loop -- Q with NT = 1, the running O of a dense call with NT = 2 -- are
// first used in it, and the compiler, which does not see the waits in inline asm, takes those loads for outstanding in every
// iteration and adds waits down to vmcnt(0) of its own: with NT = 1 ahead of the scores, where V(j), requested at the end
// of the step before, is waited for too, with NT = 2 within O += P(j) V(j), where K(j+1) is.  So with NT = 1 nothing is on
// its way under the scores and every step holds one whole trip to memory; from then on it is 64 KiB per compute unit, K(j+1).
// The two wavefronts of a SIMD drift apart until one does its softmax under the other's MFMAs.
//
// A decode step is the same thing with the query heads of a KV group as the rows and a key range as the work item.  At
// 524,288 keys and 8 KV heads 256 workgroups read 2147 MB in 355 us, 6.0 TB/s, what a kernel that only reads gets.
//
// Measured (microseconds, 256-row pipelined kernel -> this one): 512 rows x 2048 keys, 8 heads: 47.1 -> 14.8 (NT = 1,
// 128 workgroups; the host needs 10 of them); 1024 x 8192, 8 heads: 157 -> 49 (NT = 1, 256 workgroups); 2048 x 8192, 8
// heads: 158 -> 80 (NT = 2, 256 workgroups).  A step of 256 keys takes 1.17 us with NT = 1 -- 128 KiB at 112 GB/s per
// compute unit, the trip to memory that nothing covers included; how much of the step that trip is has not been measured --
// and 1.68 us with NT = 2, where MFMAs and softmax of the two wavefronts of a SIMD add up.  Tried and dropped: NT = 2 with Q
// in registers (spills in the loop); 64 rows as two wavefronts sharing each of four key streams (two barriers per step:
// 2.7 us per 256 keys); four-wavefront workgroups of the pipelined kernel, two per compute unit (twice the tile loads:
// packed batches 11 ... 14 % slower).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "aux_kernels.hpp"
#include "common.hpp"

namespace pec {

constexpr int kSplitWaves = 8;                              // key streams
constexpr int kSplitTile = 32;                              // keys per tile
constexpr int kSplitTileBytes = kSplitTile * kRowBytes;     // 8 KiB for K, 8 KiB for V

// Merge of a decode step's key ranges in the launch that makes them, by whichever workgroup of a KV head finds that all of
// its ranges are there: every workgroup writes its partial results, then its word, then reads the words of all ranges; of
// the workgroups that do so last, at least one sees them all (several may: they write the same results).  A word says
// "there" by holding the mark of this call, which the host makes anew for every launch (merge_mark(); a launch that a graph
// replays would bring the same one again, so captured steps are merged by a launch of their own).  Words stay behind a call,
// and any of them may be overwritten or put back between calls: no call has the mark of another.

// Called by all wavefronts of a workgroup behind its stores; `range`: its key range, `words`: the words of its KV head.
__device__ __forceinline__ bool last_workgroup(uint64_t* words, uint64_t mark, int range, int n_ranges, int wave) {
    __shared__ int all_there;
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt 0: this wavefront's results (store_shared()) are in place
    asm volatile("" ::: "memory");
    __syncthreads();
    if (wave == 0) {
        const int lane = threadIdx.x & 63;
        if (lane == 0) __hip_atomic_store(words + range, mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0x0F70);    // the word is in place before the others are read
        asm volatile("" ::: "memory");
        const bool there = lane >= n_ranges || __hip_atomic_load(words + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark;
        const bool all = __all(there);
        if (lane == 0) all_there = all;
    }
    __syncthreads();
    return all_there;
}

// What a launch works on: the query tiles of one call, the items of a packed or colocated batch (a device-built list of
// bm = 32 * NT rows per item), or the key ranges of a decode step; kSplitBatch: the items of a batch of up to 64 sequences,
// which every wavefront finds in the offsets by itself.
enum { kSplitDense = 0, kSplitList = 1, kSplitDecode = 2, kSplitBatch = 3 };

// Items of a batch of up to 64 sequences in the order of a work list (build_worklist_kernel) that keeps the items of a
// sequence together: a lane per sequence, sequences by the keys of their heaviest item, a sequence's longest item first.
// Building the list would be a launch of its own, 3 us of the host's time and 6 of the GPU's; here it is one trip to memory
// and a few instructions per sequence at the start of every workgroup.
struct BatchItems {
    int q0, len_q, k0, len_k, first, count, slot0;     // of this lane's sequence; slot0 -1: not split
    int total;                                         // items of the batch
    __device__ __forceinline__ BatchItems(const FwdParams& p, int bm) {
        const int b = threadIdx.x & 63;
        q0 = len_q = k0 = len_k = first = count = 0;
        slot0 = -1;
        if (b < p.batch) {      // bounds clamped as in build_worklist_kernel
            q0 = min(max(p.cu_q[b], 0), p.total_q);
            len_q = min(max(p.cu_q[b + 1], q0), p.total_q) - q0;
            k0 = min(max(p.cu_k[b], 0), p.total_k);
            len_k = min(max(p.cu_k[b + 1], k0), p.total_k) - k0;
        }
        const bool split = p.range_len > 0 && len_q == 1 && len_k > p.range_len;
        const int ranges = split ? (len_k + p.range_len - 1) / p.range_len : 0;
        count = split ? (ranges + p.group - 1) / p.group : (len_q + bm - 1) / bm;
        if (p.range_len > 0) {
            int upto = ranges;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(upto, d);
                if (b >= d) upto += y;
            }
            if (split) slot0 = upto - ranges;
            if (split && upto > p.slot_capacity) {      // offsets that are not monotone: left out
                count = 0;
                slot0 = -1;
            }
            const uint64_t listed = __ballot(slot0 >= 0);
            if (blockIdx.x == 0 && threadIdx.x < 64) {
                if (slot0 >= 0) p.split_seqs[__popcll(listed & ((1ull << b) - 1))] = SplitSeq{b, slot0, ranges, 0};
                if (b == 0) *p.n_split = __popcll(listed);
            }
        }
        const int keys = split ? min(p.range_len, len_k) : len_k;
        total = 0;
        for (int i = 0; i < p.batch; ++i) {
            const int n = __builtin_amdgcn_readlane(count, i), other = __builtin_amdgcn_readlane(keys, i);
            total += n;
            if (other > keys || (other == keys && i < b)) first += n;
        }
    }
    __device__ __forceinline__ WorkItem item(const FwdParams& p, int n) const {     // n < total, uniform
        const int b = __builtin_ctzll(__ballot((uint32_t)(n - first) < (uint32_t)count));
        const int i = n - __builtin_amdgcn_readlane(first, b), s = __builtin_amdgcn_readlane(slot0, b);
        const int sq0 = __builtin_amdgcn_readlane(q0, b), sk0 = __builtin_amdgcn_readlane(k0, b), lk = __builtin_amdgcn_readlane(len_k, b);
        const int r0 = i * p.group;      // first key range of a split sequence's item
        if (s >= 0) return WorkItem{sq0, 1, sk0 + r0 * p.range_len, lk - r0 * p.range_len, -1, s + r0, {0, 0}};
        return WorkItem{sq0, __builtin_amdgcn_readlane(len_q, b), sk0, lk, __builtin_amdgcn_readlane(count, b) - 1 - i, 0, {0, 0}};
    }
};
template <int NT, int MODE>
__global__ __launch_bounds__(kSplitWaves * 64, 2) void fwd_split_kernel(const FwdParams p) {
    constexpr bool BATCH = MODE == kSplitBatch;
    constexpr bool LIST = MODE == kSplitList || BATCH;
    constexpr bool DECODE = MODE == kSplitDecode;
    constexpr int KS = kSplitWaves;
    constexpr int BM = 32 * NT;
    constexpr int LOADS = 8;                 // load instructions (1 KiB each) per matrix and tile
    // NT = 2 keeps Q in LDS (the registers hold two 32-row accumulators instead)
    constexpr bool kQLds = NT == 2;
    // K and V stages (128 KiB), reused for the partial O of the merge; then Q; then the merge's scalars
    constexpr int kQBytes = kQLds ? BM * kRowBytes : 0;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[16 * kSplitTileBytes + kQBytes + 3 * KS * 32 * 4];
    unsigned char* const lds_q = lds + 16 * kSplitTileBytes;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, hl = lane >> 5;

    using Items = std::conditional_t<BATCH, BatchItems, int>;
    const Items items = [&]() -> Items {
        if constexpr (BATCH) return BatchItems(p, BM);
        else return 0;
    }();
    int n_items = p.n_items;
    if constexpr (BATCH) n_items = min(items.total, n_items);
    else if constexpr (LIST) n_items = min(*p.n_work, n_items);
    const WorkOrder order(n_items, p.group, p.n_kv_heads);
    if ((blockIdx.x >> 3) >= order.count) return;
    const int64_t logical = order.unit(blockIdx.x & 7, blockIdx.x >> 3);
    if (logical < 0) return;
    const int per_kvh = order.per_kvh;
    const int kvh = (int)(logical / per_kvh);
    const int rem = (int)(logical % per_kvh);
    const int item = rem / p.group;
    const int head = kvh * p.group + rem % p.group;

    // rows sq x keys sk with diagonal offset delta; element offsets of row 0 in q, in out / acc and in lse
    int sq, sk, delta, qt;
    int64_t kv_tok0 = 0, q_stride = (int64_t)p.n_q_heads * kHeadDim, q_off0, o_off0, lse_off0;
    void* out_ptr = p.out;
    float* lse_ptr = p.lse;
    int out_f32 = p.out_f32;
    if constexpr (DECODE) {   // the item is a key range, all of it visible; the heads of a KV group are the rows
        qt = 0;
        sq = p.sq;
        q_stride = p.q_row_stride;
        q_off0 = o_off0 = (int64_t)head * p.q_head_stride;
        lse_off0 = (int64_t)head * p.lse_stride;
        kv_tok0 = (int64_t)item * p.kv_split_len;
        sk = delta = (int)max((int64_t)0, min((int64_t)p.kv_split_len, (int64_t)p.sk - kv_tok0));
        o_off0 += item * p.split_out_stride;
        lse_off0 += item * p.split_lse_stride;
    } else if constexpr (LIST) {
        WorkItem w;
        if constexpr (BATCH) w = items.item(p, item);
        else w = p.work[item];
        sk = w.len_k;
        kv_tok0 = w.k0;
        if (w.qtile >= 0) {
            sq = w.len_q;
            delta = sk - sq;
            qt = w.qtile;
            q_off0 = w.q0 * q_stride + (int64_t)head * kHeadDim;
            o_off0 = q_off0;
            lse_off0 = (int64_t)head * p.lse_stride + w.q0;
        } else {              // a key range of a one-token sequence: the heads of a KV group are the rows
            const int r = rem % p.group;
            const int64_t slot_no = (int64_t)w.slot + r;
            sq = p.group;
            sk = min(p.range_len, w.len_k - r * p.range_len);
            if (sk <= 0) return;
            kv_tok0 += (int64_t)r * p.range_len;
            delta = sk;       // every key of the range is visible
            qt = 0;
            q_off0 = w.q0 * q_stride + (int64_t)kvh * p.group * kHeadDim;
            q_stride = kHeadDim;
            o_off0 = (slot_no * p.n_q_heads + (int64_t)kvh * p.group) * kHeadDim;
            lse_off0 = slot_no * p.n_q_heads + (int64_t)kvh * p.group;
            out_ptr = p.part_out;
            lse_ptr = p.part_lse;
            out_f32 = 1;
        }
    } else {
        sq = p.sq;
        sk = p.sk;
        delta = p.delta;
        qt = p.causal ? (n_items - 1 - item) : item;
        q_off0 = o_off0 = (int64_t)head * kHeadDim;
        lse_off0 = (int64_t)head * p.lse_stride;
    }
    const int causal = DECODE ? 0 : p.causal;
    const int row0 = qt * BM;
    int kv_end = sk;
    if (causal) kv_end = max(0, min(sk, min(sq, row0 + BM) + delta));
    const int n_tiles = (kv_end + kSplitTile - 1) / kSplitTile;

    const uint32_t kv_stride_b = (uint32_t)p.n_kv_heads * kHeadDim * 2;
    const unsigned char* kbase =
        reinterpret_cast<const unsigned char*>(p.k) + (kv_tok0 * p.n_kv_heads + kvh) * (int64_t)(kHeadDim * 2);
    const unsigned char* vbase =
        reinterpret_cast<const unsigned char*>(p.v) + (kv_tok0 * p.n_kv_heads + kvh) * (int64_t)(kHeadDim * 2);

    // ---- Q fragments
    bf16x8 qf[NT][8];
    if constexpr (!kQLds) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int row = row0 + nt * 32 + l32;
            const __bf16* qrow = p.q + q_off0 + row * q_stride + 8 * hl;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                u32x4 raw = {0u, 0u, 0u, 0u};
                if (row < sq) raw = *reinterpret_cast<const u32x4*>(qrow + 16 * t);
                qf[nt][t] = __builtin_bit_cast(bf16x8, raw);
            }
        }
    }
    // ---- running state; what is carried in belongs to the first key stream
    f32x16 o[NT][4];
    float m_run[NT], l_run[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_run[nt] = -INFINITY;
        l_run[nt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[nt][dt][r] = 0.f;
        const int row = row0 + nt * 32 + l32;
        if (MODE == kSplitDense && p.acc_in && wave == 0 && row < sq) {
            const float lin = p.lse_in[lse_off0 + row];
            if (lin != -INFINITY) {
                m_run[nt] = lin * kLog2e;
                l_run[nt] = hl == 0 ? 1.f : 0.f;
                const float* arow = p.acc_in + o_off0 + row * q_stride + 4 * hl;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const f32x4 x = *reinterpret_cast<const f32x4*>(arow + 32 * dt + 8 * b);
#pragma unroll
                        for (int i = 0; i < 4; ++i) o[nt][dt][4 * b + i] = x[i];
                    }
            }
        }
    }

    // ---- tile loads: one instruction moves four key rows (M0 = LDS address, SGPR base + 32-bit lane offset).  In a
    // whole tile the lane offset of K block i is the first block's with the swizzle's row bits 2..3 flipped in.
    const int ld_row = lane >> 4, ld_pos = lane & 15;
    const uint32_t ldk_off = (uint32_t)ld_row * kv_stride_b + (uint32_t)(ld_pos ^ ld_row) * 16u;
    const uint32_t ldv_off = (uint32_t)ld_row * kv_stride_b + (uint32_t)((((ld_pos >> 2) ^ ld_row) << 2) | (ld_pos & 3)) * 16u;
    auto issue = [&](auto in_loop, const unsigned char* base, bool is_v, int tile, unsigned char* stage) {
        const int key0 = tile * kSplitTile;
        const unsigned char* tb = base + (int64_t)key0 * kv_stride_b;
        const uint32_t l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)stage;
        if (key0 + kSplitTile <= sk) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                dma16<decltype(in_loop)::value>(tb + (uint32_t)(4 * i) * kv_stride_b, is_v ? ldv_off : ldk_off ^ ((i & 3) << 6), l0 + i * 1024);
        } else {   // rows past the end re-read the last valid one: finite data, weight zero
            int ln;     // rebuilt from the lane id: the loop carries no register for this path
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
            const int r_row = ln >> 4, r_pos = ln & 15;
            const int last = sk - 1 - key0;      // >= 0 for every tile that is asked for
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int key = 4 * i + r_row;
                const uint32_t col = is_v ? (uint32_t)((((r_pos >> 2) ^ (key & 3)) << 2) | (r_pos & 3)) * 16u
                                          : (uint32_t)(r_pos ^ (key & 15)) * 16u;
                dma16<decltype(in_loop)::value>(tb, (uint32_t)min(key, last) * kv_stride_b + col, l0 + i * 1024);
            }
        }
    };

    // ---- LDS operand offsets: K chunk 2t + hl of row l32 is k_lds_off(l32, hl) with t at bits 5..7 flipped in
    const uint32_t k_off0 = k_lds_off(l32, hl);
    uint32_t v_off[4];
    {
        const int gi = l32 & 15, gg = l32 >> 4;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) v_off[dt] = v_lds_off(4 * hl + (gi >> 2), dt * 64 + gg * 32 + (gi & 3) * 8);
    }
    const float sl2 = p.scale_log2;

    if constexpr (kQLds) {   // rows past the end re-read the last valid one; their results are not stored
        const unsigned char* qb = reinterpret_cast<const unsigned char*>(p.q + q_off0 + row0 * q_stride);
        const uint32_t l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_q;
#pragma unroll
        for (int i = 0; i < BM / 4 / KS; ++i) {
            const int blk = wave + i * KS, row = 4 * blk + ld_row;
            dma16<false>(qb, (uint32_t)min(row, sq - 1 - row0) * (uint32_t)(q_stride * 2) + (uint32_t)(ld_pos ^ (row & 15)) * 16u, l0 + blk * 1024);
        }
    }
    unsigned char* const kst = lds + wave * 2 * kSplitTileBytes;
    unsigned char* const vst = kst + kSplitTileBytes;
    if (wave < n_tiles) {
        issue(std::false_type{}, kbase, false, wave, kst);
        issue(std::false_type{}, vbase, true, wave, vst);
    }
    static_assert(LOADS == 8, "the vmcnt immediates below assume eight loads per matrix and tile");
    if constexpr (kQLds) {
        if (wave < n_tiles) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");   // this wavefront's share of Q
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    for (int tile = wave; tile < n_tiles; tile += KS) {
        const bool more = tile + KS < n_tiles;
        const int key0 = tile * kSplitTile;
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");       // K(j); V(j) may be on its way (but see the top for NT = 1)
        f32x16 s[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[nt][r] = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bf16x8 kf = *reinterpret_cast<const bf16x8*>(kst + (k_off0 ^ (t << 5)));
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if constexpr (kQLds) qf[nt][t] = *reinterpret_cast<const bf16x8*>(lds_q + nt * 32 * kRowBytes + (k_off0 ^ (t << 5)));
                s[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[nt][t], s[nt], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the K stage has been read
        if (more) issue(std::true_type{}, kbase, false, tile + KS, kst);

        // mask, softmax reference (kept lazily: it moves only for a score more than 2^8 ahead of it), weights
        const bool need_mask = key0 + kSplitTile > sk || (causal && key0 + kSplitTile - 1 > row0 + delta);
        bf16x8 pp[NT][2];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (need_mask) {
                int last_vis = sk - 1;
                if (causal) last_vis = min(last_vis, row0 + nt * 32 + l32 + delta);
                const int lim = last_vis - key0 - 4 * hl;   // compare against 8*(r/4) + r%4
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + (r & 3) > lim) s[nt][r] = -INFINITY;
            }
            float mx = s[nt][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[nt][r]);
            {
                const uint32_t u = __builtin_bit_cast(uint32_t, mx);
                const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
                mx = fmaxf(__builtin_bit_cast(float, (uint32_t)sw[0]), __builtin_bit_cast(float, (uint32_t)sw[1]));
            }
            const float mx2 = mx * sl2;
            const float m_new = (mx2 > m_run[nt] + 8.f) ? mx2 : m_run[nt];
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;   // a row that has seen no key yet
            const float alpha = __builtin_amdgcn_exp2f(m_run[nt] - m_use);
            m_run[nt] = m_new;
            float rs = 0.f;
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                u32x4 packed;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x2 x = {__builtin_amdgcn_exp2f(fmaf(s[nt][8 * t2 + 2 * e], sl2, -m_use)),
                                     __builtin_amdgcn_exp2f(fmaf(s[nt][8 * t2 + 2 * e + 1], sl2, -m_use))};
                    rs += x[0] + x[1];   // denominator from the unrounded weights
                    packed[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
                }
                pp[nt][t2] = __builtin_bit_cast(bf16x8, packed);
            }
            l_run[nt] = l_run[nt] * alpha + rs;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[nt][dt][r] *= alpha;
            }
        }

        if (more) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");   // V(j); K(j+1) may still be on its way (NT = 2, dense: see the top)
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const unsigned char* src = vst + v_off[dt] + k2 * 16 * kRowBytes;
                const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(src));
                const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (__attribute__((address_space(3))) bf16x4*)(src + 8 * kRowBytes));
                const bf16x8 vf = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    o[nt][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pp[nt][k2], o[nt][dt], 0, 0, 0);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the V stage has been read
        if (more) issue(std::true_type{}, vbase, true, tile + KS, vst);
    }

    // ---- merge of the eight partial results of every row, 32 rows at a time.  O goes to LDS in 16-byte chunks of 4
    // head-dim values, chunk c of row r at slot c * 32 + (r ^ c): the writers (fixed c, one row per lane) and the
    // readers (fixed row, one chunk per lane, so that a row leaves as one 256- or 512-byte run) touch all banks evenly.
    float* const lds_m = reinterpret_cast<float*>(lds_q + kQBytes);
    float* const lds_l = lds_m + KS * 32;
    float* const lds_w = lds_l + KS * 32;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        __syncthreads();
        {
            const float l_tot = l_run[nt] + __shfl_xor(l_run[nt], 32);
            if (hl == 0) {
                lds_m[wave * 32 + l32] = m_run[nt];
                lds_l[wave * 32 + l32] = l_tot;
            }
            f32x4* const po = reinterpret_cast<f32x4*>(lds) + wave * 1024;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int c = 8 * dt + 2 * b + hl;
                    f32x4 x;
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = o[nt][dt][4 * b + i];
                    po[c * 32 + (l32 ^ c)] = x;
                }
        }
        __syncthreads();
        if (threadIdx.x < KS * 32) {   // one thread per (row, key stream): the stream's weight
            const int r = threadIdx.x & 31, k = threadIdx.x >> 5;
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < KS; ++i) mx = fmaxf(mx, lds_m[i * 32 + r]);
            const float m_use = mx == -INFINITY ? 0.f : mx;
            float den = 0.f;
#pragma unroll
            for (int i = 0; i < KS; ++i) den += lds_l[i * 32 + r] * __builtin_amdgcn_exp2f(lds_m[i * 32 + r] - m_use);
            const float inv = den > 0.f ? 1.f / den : 0.f;
            lds_w[k * 32 + r] = __builtin_amdgcn_exp2f(lds_m[k * 32 + r] - m_use) * inv;
            const int row = row0 + nt * 32 + r;
            if (k == 0 && row < sq) {
                // (a key range of a batch whose weights are NaN says so in its LSE, which makes the merged row's what it is uncut)
                const float none = LIST && out_ptr == p.part_out && den != den ? den : -INFINITY;
                const float lse = den > 0.f ? (mx + __builtin_amdgcn_logf(den)) * kLn2 : none;
                if (DECODE) __hip_atomic_store(lse_ptr + lse_off0 + row, lse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else lse_ptr[lse_off0 + row] = lse;
            }
        }
        __syncthreads();
        const int c = threadIdx.x & 31;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int r = pass * 16 + (threadIdx.x >> 5);
            const int row = row0 + nt * 32 + r;
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const float w = lds_w[k * 32 + r];
                const f32x4 x = reinterpret_cast<const f32x4*>(lds)[k * 1024 + c * 32 + (r ^ c)];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = fmaf(w, x[i], a[i]);
            }
            if (row < sq) {
                const int64_t idx = o_off0 + row * q_stride + 4 * c;
                if (MODE == kSplitDense && p.acc_out) *reinterpret_cast<f32x4*>(p.acc_out + idx) = a;
                if (out_ptr) {
                    if (DECODE && p.arrived)
                        store_shared(reinterpret_cast<float*>(out_ptr) + idx, a);
                    else if (out_f32)
                        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out_ptr) + idx) = a;
                    else
                        *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(out_ptr) + idx) = __builtin_convertvector(a, bf16x4);
                }
            }
        }
    }
    if constexpr (DECODE) {
        if (!p.arrived || !last_workgroup(p.arrived + (int64_t)kvh * n_items, p.mark, item, n_items, wave))
            return;
        const int n_heads = p.n_kv_heads * sq;
        for (int h = wave; h < sq; h += KS)
            combine_few<kMergeRanges, true>(static_cast<const float*>(p.out), p.lse, n_items, n_heads, kvh * sq + h, p.merged_out,
                                      p.merged_f32, p.merged_lse);
    }
}

}  // namespace pec
