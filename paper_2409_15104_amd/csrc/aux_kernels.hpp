// HBM-bound helpers around the attention kernel: the log-sum-exp merge of two
// partial results, the fp32 -> bf16 finalisation, and the device-side work list for
// packed variable-length batches.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace pec {

// o_acc <- o_acc * exp(la - L) + o_part * exp(lb - L),  L = ln(exp(la) + exp(lb)).
// One thread per 4 consecutive head-dim values; the 32 threads of one (row, head)
// sit in one wavefront, so all of them read lse_acc before thread 0 overwrites it.
template <bool F32>
__global__ __launch_bounds__(256) void merge_kernel(void* __restrict__ o_acc_v, float* __restrict__ lse_acc,
                                                    const void* __restrict__ o_part_v,
                                                    const float* __restrict__ lse_part, int64_t sq, int n_q_heads) {
    const int64_t n_groups = sq * n_q_heads * 32;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_groups;
         g += (int64_t)gridDim.x * blockDim.x) {
        const int64_t rh = g >> 5;
        const int64_t row = rh / n_q_heads;
        const int h = (int)(rh % n_q_heads);
        const int64_t li = (int64_t)h * sq + row;
        const float la = lse_acc[li], lb = lse_part[li];
        const float mx = fmaxf(la, lb);
        float wa = 0.f, wb = 0.f, L = -INFINITY;
        if (mx != -INFINITY) {
            const float ea = expf(la - mx), eb = expf(lb - mx);
            const float den = ea + eb;
            wa = ea / den;
            wb = eb / den;
            L = mx + logf(den);
        }
        f32x4 a, b;
        if constexpr (F32) {
            a = reinterpret_cast<const f32x4*>(o_acc_v)[g];
            b = reinterpret_cast<const f32x4*>(o_part_v)[g];
        } else {
            a = __builtin_convertvector(reinterpret_cast<const bf16x4*>(o_acc_v)[g], f32x4);
            b = __builtin_convertvector(reinterpret_cast<const bf16x4*>(o_part_v)[g], f32x4);
        }
        f32x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = a[i] * wa + b[i] * wb;
        if constexpr (F32)
            reinterpret_cast<f32x4*>(o_acc_v)[g] = r;
        else
            reinterpret_cast<bf16x4*>(o_acc_v)[g] = __builtin_convertvector(r, bf16x4);
        if ((g & 31) == 0) lse_acc[li] = L;
    }
}

__global__ __launch_bounds__(256) void finalize_kernel(const float* __restrict__ src, __bf16* __restrict__ dst,
                                                       int64_t n_groups) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_groups;
         g += (int64_t)gridDim.x * blockDim.x)
        reinterpret_cast<bf16x4*>(dst)[g] = __builtin_convertvector(reinterpret_cast<const f32x4*>(src)[g], bf16x4);
}

// Combines the partial results of a split-KV decode: for one head, L = ln sum_s exp(lse_s) and
// O = sum_s O_s exp(lse_s - L) over the n_splits disjoint key ranges (the two-set merge applied to
// all ranges at once), by one workgroup of kCombineThreads.  Thread (grp, c) sums dimensions 4c .. 4c + 3 of the ranges
// grp, grp + kCombineGroups, ...; every range's weight is taken once and handed round through LDS.  Partials are fp32
// [n_splits][n_heads][128] and [n_splits][n_heads]; out_row points at the 128 outputs.
// A few KB per head: latency is all there is to it, so the first kCombineAhead ranges of every thread are requested
// together with the LSEs.  128 ranges of 64 heads: 9.0 -> 5.1 us.
constexpr int kCombineThreads = 1024, kCombineGroups = kCombineThreads / 32, kCombineAhead = 4;
template <bool OUT_F32>
__device__ __forceinline__ void combine_one_head(const float* __restrict__ o_part, const float* __restrict__ lse_part,
                                                 int n_splits, int n_heads, int h, void* __restrict__ out_row,
                                                 float* __restrict__ lse_dst) {
    constexpr int kWaves = kCombineThreads / 64;
    __shared__ float weight[kCombineThreads];
    __shared__ __attribute__((aligned(16))) float red[kWaves][kHeadDim];
    __shared__ float red_mx[kWaves], red_den[kWaves];
    const int tid = threadIdx.x, wave = tid >> 6, grp = tid >> 5, c = tid & 31;
    auto lse_of = [&](int s) { return lse_part[(int64_t)s * n_heads + h]; };
    auto o_of = [&](int s) {
        return *reinterpret_cast<const f32x4*>(o_part + ((int64_t)s * n_heads + h) * kHeadDim + 4 * c);
    };
    float l = tid < n_splits ? lse_of(tid) : -INFINITY;
    f32x4 ahead[kCombineAhead];
#pragma unroll
    for (int i = 0; i < kCombineAhead; ++i) {
        ahead[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (grp + i * kCombineGroups < n_splits) ahead[i] = o_of(grp + i * kCombineGroups);
    }
    float mx = l;
    for (int s = tid + kCombineThreads; s < n_splits; s += kCombineThreads) mx = fmaxf(mx, lse_of(s));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    __syncthreads();                 // a previous call's readers are done with the shared arrays
    if ((tid & 63) == 0) red_mx[wave] = mx;
    __syncthreads();
    mx = red_mx[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, red_mx[w]);
    float den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // (nothing is skipped where no range has a key: O is 0 then, or NaN from NaN weights, and stays that)
    const float ref = mx == -INFINITY ? 0.f : mx;
    for (int s0 = 0; s0 < n_splits; s0 += kCombineThreads) {   // as many ranges as there are weights in LDS
        const int n = min(n_splits - s0, kCombineThreads);
        if (s0 > 0) {
            l = tid < n ? lse_of(s0 + tid) : -INFINITY;
            __syncthreads();     // the weights of the round before have been read
        }
        const float w = expf(l - ref);
        den += w;
        weight[tid] = w;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kCombineAhead; ++i) {
            const int s = grp + i * kCombineGroups;
            if (s < n) {
                const f32x4 x = s0 == 0 ? ahead[i] : o_of(s0 + s);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += weight[s] * x[e];
            }
        }
#pragma unroll 4
        for (int s = grp + kCombineAhead * kCombineGroups; s < n; s += kCombineGroups) {
            const f32x4 x = o_of(s0 + s);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += weight[s] * x[e];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], 32);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off);
    if ((tid & 63) < 32) *reinterpret_cast<f32x4*>(&red[wave][4 * c]) = acc;
    if ((tid & 63) == 0) red_den[wave] = den;
    __syncthreads();
    if (tid < kHeadDim) {
        float a = 0.f, dn = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            a += red[w][tid];
            dn += red_den[w];
        }
        if (dn > 0.f) a /= dn;
        if constexpr (OUT_F32)
            reinterpret_cast<float*>(out_row)[tid] = a;
        else
            reinterpret_cast<__bf16*>(out_row)[tid] = (__bf16)a;
        if (tid == 0) *lse_dst = dn > 0.f ? ref + logf(dn) : -INFINITY;
    }
}

template <bool OUT_F32>
__global__ __launch_bounds__(kCombineThreads) void combine_splits_kernel(const float* __restrict__ o_part,
                                                                              const float* __restrict__ lse_part,
                                                                              int n_splits, int n_heads,
                                                                              void* __restrict__ out,
                                                                              float* __restrict__ lse) {
    const int h = blockIdx.x;
    void* out_row = OUT_F32 ? static_cast<void*>(reinterpret_cast<float*>(out) + (int64_t)h * kHeadDim)
                            : static_cast<void*>(reinterpret_cast<__bf16*>(out) + (int64_t)h * kHeadDim);
    combine_one_head<OUT_F32>(o_part, lse_part, n_splits, n_heads, h, out_row, lse + h);
}

// The same for up to N ranges by one wavefront, without LDS or barriers: lane i holds the weight of range i, each half of the
// wavefront sums every second range, all loads in flight at once.  SHARED: the ranges come from this launch (load_shared()).
constexpr int kMergeRanges = 32;       // most ranges that one wavefront merges
template <int N, bool SHARED>
__device__ __forceinline__ void combine_few(const float* o_part, const float* lse_part, int n_splits, int n_heads, int h,
                                            void* out, bool out_f32, float* lse) {
    static_assert(N <= 32, "the ranges' weights sit in the lower half of the wavefront");
    const int lane = threadIdx.x & 63, half = lane >> 5, c = lane & 31;
    float l = -INFINITY;
    if (lane < n_splits) {
        const float* const src = lse_part + (int64_t)lane * n_heads + h;
        l = SHARED ? __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *src;
    }
    f32x4 x[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int s = 2 * i + half;
        if (s < n_splits) {
            const float* const src = o_part + ((int64_t)s * n_heads + h) * kHeadDim + 4 * c;
            x[i] = SHARED ? load_shared(src) : *reinterpret_cast<const f32x4*>(src);
        }
    }
    float mx = l;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    mx = __shfl(mx, 0);                 // ranges sit in the lower half
    const float w = mx != -INFINITY ? expf(l - mx) : 0.f;
    float den = w;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) den += __shfl_xor(den, off);
    den = __shfl(den, 0);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        if (2 * i >= n_splits) break;
        const float ws = __shfl(w, 2 * i + half);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += ws * x[i][e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        acc[e] += __shfl_xor(acc[e], 32);
        if (mx != -INFINITY) acc[e] /= den;
    }
    if (half == 0) {
        if (out_f32)
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + (int64_t)h * kHeadDim + 4 * c) = acc;
        else
            *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(out) + (int64_t)h * kHeadDim + 4 * c) = __builtin_convertvector(acc, bf16x4);
        if (c == 0) lse[h] = mx != -INFINITY ? mx + logf(den) : -INFINITY;
    }
}

// As a kernel, one wavefront per head: with few ranges combine_splits_kernel is made of the trips between its sixteen
// wavefronts.  GPU time of a decode step of 32 heads with ranges of 32 keys, that / this: 1 range 8.0 / 7.0 us, 8 ranges
// 8.1 / 7.6, 16 ranges 8.6 / 8.3, 24 ranges 8.65 / 8.61, 32 ranges 8.84 / 8.92.
// A step whose launch merges its own ranges, up to kMergeRanges, is merged here as well where that launch cannot: same bits.
constexpr int kCombineFew = 24;
template <bool OUT_F32>
__global__ __launch_bounds__(64) void combine_few_kernel(const float* o_part, const float* lse_part, int n_splits, int n_heads,
                                                         void* out, float* lse) {
    combine_few<kMergeRanges, false>(o_part, lse_part, n_splits, n_heads, blockIdx.x, out, OUT_F32, lse);
}

// The same combination for the one-token sequences of a colocated batch: split_seqs lists
// (sequence, first slot, number of key ranges); the result goes to the sequence's row of the packed
// out [total_q, n_heads, 128] / lse [n_heads, total_q].  grid = (n_heads, up to batch).
template <bool OUT_F32>
__global__ __launch_bounds__(kCombineThreads) void combine_colocated_kernel(
    const float* __restrict__ o_part, const float* __restrict__ lse_part, const SplitSeq* __restrict__ split_seqs,
    const int32_t* __restrict__ n_split_seqs, const int32_t* __restrict__ cu_q, int total_q, int n_heads,
    void* __restrict__ out, float* __restrict__ lse) {
    const int h = blockIdx.x;
    const int n = *n_split_seqs;
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const SplitSeq ss = split_seqs[i];
        const int64_t row = min(max(cu_q[ss.seq], 0), total_q - 1);
        void* out_row = OUT_F32 ? static_cast<void*>(reinterpret_cast<float*>(out) + (row * n_heads + h) * kHeadDim)
                                : static_cast<void*>(reinterpret_cast<__bf16*>(out) + (row * n_heads + h) * kHeadDim);
        combine_one_head<OUT_F32>(o_part + (int64_t)ss.slot0 * n_heads * kHeadDim, lse_part + (int64_t)ss.slot0 * n_heads,
                                  ss.n_ranges, n_heads, h, out_row, lse + (int64_t)h * total_q + row);
    }
}

// Ulysses-style layout exchange, the on-GPU halves.  A GPU holding a sequence segment of all heads,
// x [s, H, 128], packs it into G messages of s x H/G heads, y [G, s, H/G, 128] (message g = the heads
// GPU g will own); the inverse turns G received messages back into [s, H, 128].  16 bytes per thread,
// both sides contiguous in runs of H/G * 256 bytes.  TO_MESSAGES selects the direction.
template <bool TO_MESSAGES>
__global__ __launch_bounds__(256) void ulysses_layout_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                             int64_t s, int n_heads, int n_gpus) {
    constexpr int kBatch = 4;                        // loads in flight per thread before the first store
    const int hg = n_heads / n_gpus;                 // heads per message
    const int64_t chunks_per_tok = (int64_t)n_heads * 16;   // 16-byte chunks per token (all heads)
    const int64_t total = s * chunks_per_tok;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    auto other_side = [&](int64_t i) {               // i indexes the [s, H, 16] side; returns the [G, s, H/G, 16] index
        const int64_t t = i / chunks_per_tok;
        const int r = (int)(i % chunks_per_tok);
        const int h = r >> 4, c = r & 15;
        const int g = h / hg, hh = h % hg;
        return (((int64_t)g * s + t) * hg + hh) * 16 + c;
    };
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < total; i0 += kBatch * stride) {
        u32x4 v[kBatch];
        int64_t j[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t i = i0 + u * stride;
            if (i < total) {
                j[u] = other_side(i);
                v[u] = __builtin_nontemporal_load(src + (TO_MESSAGES ? i : j[u]));
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t i = i0 + u * stride;
            if (i < total) __builtin_nontemporal_store(v[u], dst + (TO_MESSAGES ? j[u] : i));
        }
    }
}

// Exclusive suffix sum in place over a[0..n), by one workgroup of 1024 threads: a[t] <- sum of the old
// a[t'] for t' > t.  Returns the sum of all old elements.  `red` is int32[16] in LDS.
template <typename T>
__device__ __forceinline__ int block_suffix_sum_1024(T* a, int n, int32_t* red) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int chunk = (n + 1023) / 1024;
    const int lo = min(n, tid * chunk), hi = min(n, lo + chunk);
    int mine = 0;
    for (int t = lo; t < hi; ++t) mine += a[t];
    int run = mine;                              // everything owned by this lane and the later ones of its wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_down(run, off);
        if (lane + off < 64) run += x;
    }
    if (lane == 0) red[wave] = run;
    __syncthreads();
    run -= mine;
    int total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        total += red[w];
        if (w > wave) run += red[w];
    }
    for (int t = hi - 1; t >= lo; --t) {
        const int x = a[t];
        a[t] = run;
        run += x;
    }
    __syncthreads();
    return total;
}

// Work list of a packed or colocated batch.  A sequence with one query token and more than range_len keys (the decode
// step of a long request; range_len > 0 only in a colocated batch) is cut into key ranges of range_len keys, `group` of
// them per item (one for each of its work units), every other sequence into query tiles of bm rows.  Items are ordered by
// descending number of blocks of block_keys keys they have to read, so that the long ones start first and the launch ends
// on the short ones -- or, by_sequence, sequences by that number of their heaviest item, the items of one sequence
// together, the longest first: the workgroups of an XCD then work on one sequence at a time, whose keys its L2 holds
// (list_by_sequence() in kernel_choice.hpp).
// Single workgroup of 1024 threads.  counters: [0] number of items, [1] slots handed out, [2] number of split sequences,
// [8 .. 15] the attention kernel's draw counters, one per XCD.  bucket is int32[n_buckets], n_buckets larger than the
// number of such blocks in all keys.  Sequence bounds are clamped into [0, total], so no index leaves the arrays whatever
// the offsets are, and n_buckets and capacity bound the items of any clamped offsets.
// What it costs is latency, all other compute units waiting: sequences are brought to LDS once (a wavefront that reads its
// sequences' offsets one after the other pays a trip to memory for each), and so are the buckets, unless there are more
// than fit; only as many are touched as the heaviest item needs.  256 prompts and a decode step 47.5 -> 17.8 us, 8
// prompts 8.7 -> 5.8 us.
constexpr int kListSeqs = 1024, kListBuckets = 2048;
__global__ __launch_bounds__(1024) void build_worklist_kernel(const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
                                                              int batch, int total_q, int total_k, int bm, int block_keys,
                                                              int range_len, int group, int capacity, int slot_capacity,
                                                              int n_buckets, int by_sequence, WorkItem* __restrict__ work,
                                                              int32_t* __restrict__ counters, int32_t* __restrict__ bucket,
                                                              SplitSeq* __restrict__ split_seqs) {
    struct Seq {
        int q0, len_q, k0, len_k, slot0, n_items, pos0;   // slot0 -1: not split; pos0: list position of its first item
    };
    __shared__ Seq seqs[kListSeqs];
    __shared__ int32_t lds_bucket[kListBuckets];
    __shared__ int32_t red[16], n_slots, n_split;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (tid == 0) n_slots = n_split = 0;
    if (tid >= 8 && tid < 16) counters[tid] = 0;
    __syncthreads();
    auto bounds_of = [&](int b) {
        Seq s;
        s.q0 = min(max(cu_q[b], 0), total_q);
        s.len_q = min(max(cu_q[b + 1], s.q0), total_q) - s.q0;
        s.k0 = min(max(cu_k[b], 0), total_k);
        s.len_k = min(max(cu_k[b + 1], s.k0), total_k) - s.k0;
        s.slot0 = -1;
        s.n_items = (s.len_q + bm - 1) / bm;
        return s;
    };
    auto is_split = [&](const Seq& s) { return range_len > 0 && s.len_q == 1 && s.len_k > range_len; };
    auto weight_of = [&](const Seq& s, int i) {   // blocks item i of the sequence reads
        const int keys = is_split(s) ? min(range_len, s.len_k - i * group * range_len)
                                     : min(s.len_k, max(0, s.len_k - s.len_q + min(s.len_q, bm * (i + 1))));
        return min(n_buckets - 1, (keys + block_keys - 1) / block_keys);
    };
    auto heaviest_of = [&](const Seq& s) { return weight_of(s, is_split(s) ? 0 : max(0, s.n_items - 1)); };
    // Sequence c0 + tid into LDS; the first time round, slots for the key ranges of split ones.  (A sequence that finds no
    // room -- only possible with offsets that are not monotone, whose clamped lengths can add up to more than total_k -- is
    // left out altogether.)  Slots are handed out once per sequence: with more than kListSeqs sequences they are kept in
    // split_seqs and looked up there.
    auto load_seq = [&](int c0, bool first) {
        const int b = c0 + tid;
        if (b >= batch) return;
        Seq s = bounds_of(b);
        if (is_split(s)) {
            const int n_ranges = (s.len_k + range_len - 1) / range_len;
            s.n_items = (n_ranges + group - 1) / group;
            if (first) {
                s.slot0 = atomicAdd(&n_slots, n_ranges);
                if (s.slot0 + n_ranges <= slot_capacity) {
                    split_seqs[atomicAdd(&n_split, 1)] = SplitSeq{b, s.slot0, n_ranges, 0};
                } else {
                    s.n_items = 0;
                }
            } else {
                s.n_items = 0;
                for (int i = 0; i < n_split; ++i) {
                    const SplitSeq ss = split_seqs[i];
                    if (ss.seq != b) continue;
                    s.slot0 = ss.slot0;
                    s.n_items = (n_ranges + group - 1) / group;
                }
            }
        }
        seqs[tid] = s;
    };
    auto for_items = [&](int c0, auto&& f) {      // one wavefront per sequence, one lane per item
        __syncthreads();
        const int n = min(batch - c0, kListSeqs);
        for (int b = wave; b < n; b += 16) {
            const Seq s = seqs[b];
            for (int i = lane; i < s.n_items; i += 64) f(s, i);
        }
    };
    int mx = 0;   // heaviest item
    for (int b = tid; b < batch; b += 1024) mx = max(mx, heaviest_of(bounds_of(b)));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 16; ++w) mx = max(mx, red[w]);
    const int n_w = mx + 1;
    auto build = [&](auto* slots) {   // slots[w]: items of weight w (of sequences whose heaviest has it), then the next one's place
        for (int t = tid; t < n_w; t += 1024) slots[t] = 0;
        __syncthreads();
        for (int c0 = 0; c0 < batch; c0 += kListSeqs) {
            if (c0 > 0) __syncthreads();
            load_seq(c0, true);
            if (!by_sequence) for_items(c0, [&](const Seq& s, int i) { atomicAdd(&slots[weight_of(s, i)], 1); });
            else if (c0 + tid < batch) atomicAdd(&slots[heaviest_of(seqs[tid])], seqs[tid].n_items);
        }
        __syncthreads();
        const int total = block_suffix_sum_1024(slots, n_w, red);
        if (tid == 0) {
            counters[0] = min(total, capacity);
            counters[1] = n_slots;
            counters[2] = n_split;
        }
        for (int c0 = 0; c0 < batch; c0 += kListSeqs) {
            if (batch > kListSeqs) {
                __syncthreads();
                load_seq(c0, false);
            }
            if (by_sequence && c0 + tid < batch) seqs[tid].pos0 = atomicAdd(&slots[heaviest_of(seqs[tid])], seqs[tid].n_items);
            for_items(c0, [&](const Seq& s, int i) {
                const int pos = !by_sequence ? atomicAdd(&slots[weight_of(s, i)], 1) : s.pos0 + (s.slot0 >= 0 ? i : s.n_items - 1 - i);
                if ((uint32_t)pos >= (uint32_t)capacity) return;
                const int r0 = i * group;   // first key range of a split sequence's item
                work[pos] = s.slot0 >= 0 ? WorkItem{s.q0, 1, s.k0 + r0 * range_len, s.len_k - r0 * range_len, -1, s.slot0 + r0, {0, 0}}
                                         : WorkItem{s.q0, s.len_q, s.k0, s.len_k, i, 0, {0, 0}};
            });
        }
    };
    if (n_w <= kListBuckets) build(lds_bucket);
    else build(bucket);
}

// Merge of the pieces of every item that fwd_il_kernel<kFwdSpan> has cut, 32 rows of it per workgroup: grid (spans - 1, 8).
// Workgroup x does the item that span x + 1 starts inside, if no earlier span does.  Its pieces are the last one of span x
// and the first ones of the spans that start inside it.  Memory-bound: 132 KB per piece are read once, the item is written.
// An item is merged by the first launch that finds all its pieces done.
__global__ __launch_bounds__(256) void span_merge_kernel(const FwdParams p) {
    const int w0 = blockIdx.x + 1, strip = blockIdx.y;
    const int pos = span_start(p, w0), n_spans = gridDim.x + 1;
    const SpanPos at = span_locate(p, pos);
    const int unit_start = pos - at.tile;
    if (at.tile == 0 || unit_start < span_start(p, w0 - 1)) return;
    const int item = at.unit / p.group % p.n_items;
    const int unit_end = unit_start + span_steps_of(p, item);
    int w_last = w0;
    while (w_last + 1 < n_spans && span_start(p, w_last + 1) < unit_end) ++w_last;
    int32_t* const merged = p.progress + n_spans + 8 * w0 + strip;
    bool there = *merged == 0;
    for (int w = w0 - 1; w <= w_last; ++w)
        there = there && p.progress[w] >= min(unit_end, span_start(p, w + 1)) - span_start(p, w);
    if (!there) return;
    __syncthreads();      // everyone has read the word
    if (threadIdx.x == 0) {
        *merged = 1;
        if (strip == 0) atomicSub(p.pending, 1);
    }
    const int head = at.unit / p.group / p.n_items * p.group + at.unit % p.group;
    const int row0 = (p.causal ? p.n_items - 1 - item : item) * 256 + strip * 32;
    const int n_pieces = w_last - w0 + 2, c = threadIdx.x & 31;
    auto slot_row = [&](int i, int r) { return (int64_t)(2 * (w0 - 1 + i) + (i == 0 ? 1 : 0)) * 256 + strip * 32 + r; };
    for (int r = threadIdx.x >> 5; r < 32; r += 8) {
        const int row = row0 + r;
        if (row >= p.sq) return;
        float mx = -INFINITY, den = 0.f;
        for (int i = 0; i < n_pieces; ++i) mx = fmaxf(mx, p.slot_lse[slot_row(i, r)]);      // (NaN: as if it were not there)
        const float ref = mx == -INFINITY ? 0.f : mx;
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int i = 0; i < n_pieces; ++i) {     // a row without a key takes O = 0 from every piece, one with NaN weights NaN
            const int64_t s = slot_row(i, r);
            const float wgt = __builtin_amdgcn_exp2f((p.slot_lse[s] - ref) * kLog2e);
            const f32x4 x = *reinterpret_cast<const f32x4*>(p.slot_out + s * kHeadDim + 4 * c);
            den += wgt;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] += wgt * x[e];
        }
        const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] *= inv;
        const int64_t idx = ((int64_t)row * p.n_q_heads + head) * kHeadDim + 4 * c;
        if (p.out_f32) *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + idx) = a;
        else *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.out) + idx) = __builtin_convertvector(a, bf16x4);
        if (c == 0) p.lse[(int64_t)head * p.lse_stride + row] = den > 0.f ? ref + logf(den) : -INFINITY;
    }
}

// Start of a resumable sweep: nothing of it is done, all of its items are pending.  Or its end, where a plain call did the
// work: every item is through, none is pending.
__global__ void sweep_table_kernel(int32_t* progress, int64_t n_words, int32_t n_items, int32_t* pending, int32_t done) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += (int64_t)gridDim.x * blockDim.x)
        progress[i] = done ? kSweepDone : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *pending = done ? 0 : n_items;
}

}  // namespace pec
