// Stand-alone top-k kernels for gfx950 (the selection itself is in topk_select.hpp).
// One workgroup per (query set, slice) selects the k best keys of its slice; a single slice
// gives the final result directly, otherwise a second launch selects among the slices' keys.
#include "kernels.hpp"
#include "topk_select.hpp"

namespace dessert {

constexpr uint32_t TOPK_THREADS = 512;
constexpr uint64_t TOPK_SLICE = 1u << 16;

// Slices per query set: long lists are cut into 65536-element slices; shorter ones are still cut
// (down to 8192 elements per slice) when the batch alone would leave most CUs without a workgroup.
// Non-decreasing in max_scored, so a bound on the list length bounds the slice count.
uint32_t topk_slices(uint64_t max_scored, uint32_t n_queries) {
    uint64_t by_size = max_scored <= 2 * TOPK_SLICE ? 1 : (max_scored + TOPK_SLICE - 1) / TOPK_SLICE;
    uint64_t want = n_queries ? (1024 + n_queries - 1) / n_queries : 1;
    uint64_t by_fill = max_scored / 8192 < want ? max_scored / 8192 : want;
    uint64_t s = by_size > by_fill ? by_size : by_fill;
    return (uint32_t)(s ? s : 1);
}

// grid (slices, B).  slices == 1: final results; else per-slice keys to a.partial.
// KT: the width the keys are computed in (uint32_t when keys_fit_32).  T threads with U loads in flight each; a slice of
// at most T * U = 4096 scores stays in registers for all passes.  T = 512, U = 8 in general; T = 1024, U = 4 when no
// slice is longer than that (candidate lists): the phases of such a selection are short chains of LDS round trips and
// barriers, which sixteen waves get through sooner than eight (17 -> 14 us for 256 lists of 4096); on long slices the
// wider workgroup is slower (0.90 -> 1.20 ms on 8M documents).
// Slices of 4097 to 16 384 scores with 32-bit keys: 1024 threads, U = 16, so that these too are read once and stay in registers (114
// VGPRs); per search, one list of 8192, k = 10 31.7 -> 30.0 us, k = 1000 43.5 -> 40.0; 64 lists of 16 384, k = 1000 250.5 -> 246.1.
// Not with more workgroups than CUs, where the narrower ones share a CU better (64 query sets x 12 slices of 8334 scores, k = 100:
// 1269 -> 1285 us a search).
constexpr uint32_t TOPK_THREADS_SHORT = 1024;
template <typename KT, int T, int U>
__global__ __launch_bounds__(T) void topk_scores_kernel(TopkArgs a, KeyPlan plan, uint32_t slices, uint32_t kpad) {
    extern __shared__ uint64_t sorted[];
    __shared__ SelectShared sh;
    const uint32_t b = blockIdx.y, s = blockIdx.x;
    uint64_t base, count;
    if (a.cand_ids) {
        base = a.cand_uniform ? (uint64_t)b * a.cand_uniform : a.cand_off[b];
        count = a.cand_uniform ? a.cand_uniform : a.cand_off[b + 1] - base;
    } else {
        base = (uint64_t)b * a.n_docs;
        count = a.n_docs;
    }
    const uint64_t per = (count + slices - 1) / slices;
    const uint64_t lo = (uint64_t)s * per < count ? (uint64_t)s * per : count;
    const uint64_t hi = lo + per < count ? lo + per : count;
    ScoreKeysT<KT> keys{a.scores + base + lo, a.cand_ids ? a.cand_ids + base + lo : nullptr, lo, plan.id_bits};
    block_select<T, ScoreKeysT<KT>, U, true>(keys, hi - lo, a.k, kpad, sorted, sh, plan);
    if (slices == 1) {
        for (uint32_t i = threadIdx.x; i < a.k; i += T)
            write_result(sorted[i], plan.id_bits, a.out_ids + (size_t)b * a.k + i, a.out_scores + (size_t)b * a.k + i);
    } else {
        uint64_t* dst = a.partial + ((size_t)b * slices + s) * a.k;
        for (uint32_t i = threadIdx.x; i < a.k; i += T) dst[i] = sorted[i];
    }
}

// A few results from a short list (k <= TOPK_FEW, at most 4096 scores, 32-bit keys; such lists are never cut into slices): no histogram.  A lane holds eight keys in
// descending order; a round takes the largest head of the wave (six DPP maxima) and moves the lane that held it up, so a wave's
// k best of its 512 scores are k rounds with no barrier between them; the waves' lists meet in LDS once, where every key's place
// in the result is counted.  Bound: latency of the load and of k rounds of some 100 cycles; the selection above has some twenty
// barriers.  Whole searches of one list of 4096 ids: k = 1 26.3 -> 23.2 us, 10 27.6 -> 25.2, 16 28.7 -> 26.1, 24 28.4 -> 27.9, 32 29.4 -> 30.3 (64
// lists of 4096: k = 10 120.8 -> 117.8, 32 122.4 -> 123.0): taken up to 16 results.
constexpr uint32_t TOPK_FEW = 16, TOPK_FEW_KEYS = 8, TOPK_FEW_WAVES = 8;   // results; keys per lane; waves of a workgroup at most
// largest x of the wave, in every lane
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    auto step = [](uint32_t v, uint32_t o) { return v > o ? v : o; };
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true));   // row_shr 1, 2, 4, 8
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true));
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true));
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true));
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, true));   // row_bcast 15, 31
    x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, true));
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
// k <= 64 rounds over the lanes' descending lists: lane i ends with the i-th largest key of the wave (0: fewer than that)
template <int N>
__device__ __forceinline__ uint32_t wave_take_best(uint32_t (&key)[N], uint32_t k) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t mine = 0;
    for (uint32_t i = 0; i < k;) {
        const uint32_t top = wave_max_u32(key[0]);
        const bool held = key[0] == top;
        uint64_t holders = __ballot(held);   // more than one: an id listed twice, or no keys left
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t stays = key[j], follows = j + 1 < N ? key[j + 1 < N ? j + 1 : j] : 0u;
            key[j] = held ? follows : stays;
        }
        mine = lane == i ? top : mine;
        ++i;
        for (holders &= holders - 1; holders && i < k; holders &= holders - 1, ++i) mine = lane == i ? top : mine;
    }
    return mine;
}

__global__ __launch_bounds__(TOPK_FEW_WAVES * 64) void topk_few_kernel(TopkArgs a, uint32_t id_bits) {
    __shared__ uint32_t best[TOPK_FEW_WAVES][TOPK_FEW + 1];   // a list per wave; the odd row length keeps rows apart in the banks
    const uint32_t b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    uint64_t base, count;
    if (a.cand_ids) {
        base = a.cand_uniform ? (uint64_t)b * a.cand_uniform : a.cand_off[b];
        count = a.cand_uniform ? a.cand_uniform : a.cand_off[b + 1] - base;
    } else {
        base = (uint64_t)b * a.n_docs;
        count = a.n_docs;
    }
    const uint32_t n = (uint32_t)count;   // at most 8 * blockDim.x
    ScoreKeysT<uint32_t> keys{a.scores + base, a.cand_ids ? a.cand_ids + base : nullptr, 0, id_bits};
    uint32_t key[TOPK_FEW_KEYS];
#pragma unroll
    for (uint32_t u = 0; u < TOPK_FEW_KEYS; ++u) {
        uint32_t got[1];
        keys.load(tid + u * blockDim.x, n, got);
        key[u] = got[0];
    }
    auto order = [&](int i, int j) {
        const uint32_t x = key[i], y = key[j];
        key[i] = x > y ? x : y;
        key[j] = x > y ? y : x;
    };
    // Batcher's odd-even merge sort of eight
    order(0, 1); order(2, 3); order(4, 5); order(6, 7);
    order(0, 2); order(1, 3); order(4, 6); order(5, 7);
    order(1, 2); order(5, 6);
    order(0, 4); order(1, 5); order(2, 6); order(3, 7);
    order(2, 4); order(3, 5);
    order(1, 2); order(3, 4); order(5, 6);
    auto result = [&](uint32_t i, uint32_t top) {
        write_result(top, id_bits, a.out_ids + (size_t)b * a.k + i, a.out_scores + (size_t)b * a.k + i);
    };
    const uint32_t k = a.k, mine = wave_take_best(key, k);
    if (waves == 1) {
        if (lane < k) result(lane, mine);
        return;
    }
    if (lane < k) best[wave][lane] = mine;
    __syncthreads();
    // a key's place in the result = its place in its own list plus the keys of each other list that rank before it (of equal
    // keys the lower wave's): eight lanes per key, one list each
    const uint32_t other = tid & 7, keys_in_all = waves * k, per_pass = blockDim.x / 8;
    for (uint32_t e0 = 0; e0 < keys_in_all; e0 += per_pass) {
        const uint32_t e = e0 + tid / 8, w = e / k, i = e - w * k;
        const bool have = e < keys_in_all;
        const uint32_t x = have ? best[w][i] : 0u;
        uint32_t before = 0;
        if (have && other < waves && other != w)
            for (uint32_t j = 0; j < k; ++j) {
                const uint32_t o = best[other][j];
                before += (o > x || (o == x && other < w)) ? 1u : 0u;
            }
        before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x111, 0xF, 0xF, true);   // lane 7 and 15 of a row: sum over eight
        before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x112, 0xF, 0xF, true);
        before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x114, 0xF, 0xF, true);
        if (have && other == 7 && i + before < k) result(i + before, x);
    }
}

__global__ __launch_bounds__(TOPK_THREADS) void topk_merge_kernel(TopkArgs a, KeyPlan plan, uint32_t slices,
                                                                  uint32_t kpad) {
    extern __shared__ uint64_t sorted[];
    __shared__ SelectShared sh;
    const uint32_t b = blockIdx.x;
    StoredKeys keys{a.partial + (size_t)b * slices * a.k};
    block_select<TOPK_THREADS>(keys, (uint64_t)slices * a.k, a.k, kpad, sorted, sh, plan);
    for (uint32_t i = threadIdx.x; i < a.k; i += TOPK_THREADS)
        write_result(sorted[i], plan.id_bits, a.out_ids + (size_t)b * a.k + i, a.out_scores + (size_t)b * a.k + i);
}

// one workgroup per stored list whose length is read from device memory.  There are only as many workgroups
// as lists, so each is wide and keeps many loads in flight: a pass over a list is a few round trips.
constexpr uint32_t TOPK_LIST_THREADS = 1024;
template <typename KT, bool ORDERED>  // stored key type: uint64_t, or uint32_t when keys_fit_32; ORDERED: best first, else any order
__global__ __launch_bounds__(TOPK_LIST_THREADS) void topk_lists_kernel(const KT* __restrict__ lists, uint64_t list_stride,
                                                                       const uint32_t* __restrict__ counts, uint32_t k,
                                                                       KeyPlan plan, uint32_t kpad, uint32_t* __restrict__ out_ids,
                                                                       int32_t* __restrict__ out_scores,
                                                                       const uint32_t* __restrict__ hist0, uint32_t hist_bins,
                                                                       const uint32_t* __restrict__ segs, uint32_t slabs) {
    extern __shared__ uint64_t sorted[];
    __shared__ SelectShared sh;
    const uint32_t b = blockIdx.x;
    // segs != nullptr: hist0 holds rows per slab (see SlabDirectory); else one histogram per list, or nothing
    const uint32_t* first_hist = (hist0 && !segs) ? hist0 + (size_t)b * hist_bins : nullptr;
    SlabDirectory directory{nullptr, nullptr, 0, 0};
    if (segs) directory = SlabDirectory{hist0 + (size_t)b * slabs * hist_bins, segs + (size_t)b * slabs * 2, slabs, hist_bins};
    const SlabDirectory* dir = segs ? &directory : nullptr;
    if constexpr (sizeof(KT) == 8) {
        StoredKeysPairs keys{lists + (size_t)b * list_stride};
        block_select<TOPK_LIST_THREADS, StoredKeysPairs, 8, false, ORDERED>(keys, counts[b], k, kpad, sorted, sh, plan, first_hist, dir);
    } else {
        StoredKeys32 keys{lists + (size_t)b * list_stride};
        block_select<TOPK_LIST_THREADS, StoredKeys32, 8, false, ORDERED>(keys, counts[b], k, kpad, sorted, sh, plan, first_hist, dir);
    }
    for (uint32_t i = threadIdx.x; i < k; i += TOPK_LIST_THREADS)
        write_result(sorted[i], plan.id_bits, out_ids + (size_t)b * k + i, out_scores + (size_t)b * k + i);
}

// The same selection for a few long lists, in two launches: one workgroup per list finds the k-th key (everything
// block_select does short of its last pass over the list) and leaves it in emit_plan[b]; topk_lists_emit_kernel then
// copies the keys at or above it with many workgroups per list.  With one workgroup per list that last pass is the
// longest part of the selection, and with a handful of lists the rest of the chip idles meanwhile.  Unordered results.
// emit_plan[b] = {k-th key (low, high word), copies of it to take, done flag, output cursor, copies taken, -, -}.
constexpr uint32_t TOPK_EMIT_WORDS = TOPK_LISTS_EMIT_WORDS;
constexpr uint32_t TOPK_EMIT_PARTS = 32;   // workgroups per list in the second launch
template <typename KT>
__global__ __launch_bounds__(TOPK_LIST_THREADS) void topk_lists_plan_kernel(const KT* __restrict__ lists, uint64_t list_stride,
                                                                            const uint32_t* __restrict__ counts, uint32_t k,
                                                                            KeyPlan plan, uint32_t kpad, uint32_t* __restrict__ out_ids,
                                                                            int32_t* __restrict__ out_scores,
                                                                            const uint32_t* __restrict__ hist0, uint32_t hist_bins,
                                                                            const uint32_t* __restrict__ segs, uint32_t slabs,
                                                                            uint32_t* __restrict__ emit_plan) {
    extern __shared__ uint64_t sorted[];
    __shared__ SelectShared sh;
    const uint32_t b = blockIdx.x;
    const uint32_t* first_hist = (hist0 && !segs) ? hist0 + (size_t)b * hist_bins : nullptr;
    SlabDirectory directory{nullptr, nullptr, 0, 0};
    if (segs) directory = SlabDirectory{hist0 + (size_t)b * slabs * hist_bins, segs + (size_t)b * slabs * 2, slabs, hist_bins};
    const SlabDirectory* dir = segs ? &directory : nullptr;
    bool done;
    if constexpr (sizeof(KT) == 8) {
        StoredKeysPairs keys{lists + (size_t)b * list_stride};
        done = block_select<TOPK_LIST_THREADS, StoredKeysPairs, 8, false, false, false>(keys, counts[b], k, kpad, sorted, sh, plan, first_hist, dir);
    } else {
        StoredKeys32 keys{lists + (size_t)b * list_stride};
        done = block_select<TOPK_LIST_THREADS, StoredKeys32, 8, false, false, false>(keys, counts[b], k, kpad, sorted, sh, plan, first_hist, dir);
    }
    uint32_t* p = emit_plan + (size_t)b * TOPK_EMIT_WORDS;
    if (done) {  // a short list, or few keys at the top: the result is complete
        for (uint32_t i = threadIdx.x; i < k; i += TOPK_LIST_THREADS)
            write_result(sorted[i], plan.id_bits, out_ids + (size_t)b * k + i, out_scores + (size_t)b * k + i);
        if (threadIdx.x == 0) p[3] = 1;
    } else if (threadIdx.x == 0) {
        p[0] = (uint32_t)sh.prefix;
        p[1] = (uint32_t)(sh.prefix >> 32);
        p[2] = sh.need;
        p[3] = 0;
        p[4] = 0;
        p[5] = 0;
    }
}

// grid (parts, B): workgroup (x, b) copies, of its part of list b, the keys above the k-th key and as many copies of the
// k-th key itself as the plan says; output slots are taken with one atomic per wave and trip.
constexpr uint32_t TOPK_EMIT_THREADS = 256;
template <typename KT>
__global__ __launch_bounds__(TOPK_EMIT_THREADS) void topk_lists_emit_kernel(const KT* __restrict__ lists, uint64_t list_stride,
                                                                            const uint32_t* __restrict__ counts, uint32_t k,
                                                                            uint32_t id_bits, uint32_t* __restrict__ emit_plan,
                                                                            uint32_t* __restrict__ out_ids,
                                                                            int32_t* __restrict__ out_scores) {
    constexpr uint32_t V = 16 / sizeof(KT), U = 4, T = TOPK_EMIT_THREADS;
    const uint32_t b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    uint32_t* p = emit_plan + (size_t)b * TOPK_EMIT_WORDS;
    if (p[3]) return;
    const uint64_t n = counts[b];
    const KT kth = (KT)((uint64_t)p[0] | ((uint64_t)p[1] << 32));
    const uint32_t need_eq = p[2];
    const KT* keys = lists + (size_t)b * list_stride;
    uint64_t part = (n + gridDim.x - 1) / gridDim.x;
    part = (part + V - 1) / V * V;  // parts start on 16-byte boundaries
    const uint64_t lo = (uint64_t)blockIdx.x * part < n ? (uint64_t)blockIdx.x * part : n;
    const uint64_t hi = lo + part < n ? lo + part : n;
    for (uint64_t t0 = lo; t0 < hi; t0 += (uint64_t)U * T * V) {
        KT key[U][V];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint64_t i = t0 + ((uint64_t)u * T + tid) * V;
#pragma unroll
            for (uint32_t v = 0; v < V; ++v) key[u][v] = 0;
            if (i < hi) {  // a vector that starts below the list's end stays inside its allocation
                if constexpr (sizeof(KT) == 8) {
                    const ulonglong2 x = *(const ulonglong2*)(keys + i);
                    key[u][0] = x.x;
                    key[u][1] = x.y;
                } else {
                    const uint4 x = *(const uint4*)(keys + i);
                    key[u][0] = x.x;
                    key[u][1] = x.y;
                    key[u][2] = x.z;
                    key[u][3] = x.w;
                }
            }
        }
        uint32_t flags = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
#pragma unroll
            for (uint32_t v = 0; v < V; ++v) {
                const uint64_t i = t0 + ((uint64_t)u * T + tid) * V + v;
                bool take = i < hi && key[u][v] > kth;
                if (i < hi && key[u][v] == kth) take = atomicAdd(&p[5], 1u) < need_eq;
                flags |= (take ? 1u : 0u) << (u * V + v);
            }
        const uint32_t cnt = (uint32_t)__builtin_popcount(flags);
        uint32_t incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(incl, off, 64);
            if ((int)lane >= off) incl += o;
        }
        uint32_t base = 0;
        if (lane == 63 && incl) base = atomicAdd(&p[4], incl);
        base = __shfl(base, 63, 64);
        uint32_t pos = base + incl - cnt;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
#pragma unroll
            for (uint32_t v = 0; v < V; ++v)
                if ((flags >> (u * V + v)) & 1u) {
                    if (pos < k) write_result((uint64_t)key[u][v], id_bits, out_ids + (size_t)b * k + pos, out_scores + (size_t)b * k + pos);
                    ++pos;
                }
    }
}

static hipError_t allow_large_k() {  // large k: opt in to more dynamic LDS (the selection state is another 8.3 KB)
    static hipError_t a0 = hipFuncSetAttribute((const void*)topk_scores_kernel<uint32_t, TOPK_THREADS, 8>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a1 = hipFuncSetAttribute((const void*)topk_scores_kernel<uint64_t, TOPK_THREADS, 8>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a9 = hipFuncSetAttribute((const void*)topk_scores_kernel<uint32_t, TOPK_THREADS_SHORT, 4>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a11 = hipFuncSetAttribute((const void*)topk_scores_kernel<uint32_t, TOPK_THREADS_SHORT, 16>,
                                                hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a10 = hipFuncSetAttribute((const void*)topk_scores_kernel<uint64_t, TOPK_THREADS_SHORT, 4>,
                                                hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a2 = hipFuncSetAttribute((const void*)topk_merge_kernel,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a3 = hipFuncSetAttribute((const void*)topk_lists_kernel<uint64_t, true>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a4 = hipFuncSetAttribute((const void*)topk_lists_kernel<uint32_t, true>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a5 = hipFuncSetAttribute((const void*)topk_lists_kernel<uint64_t, false>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a6 = hipFuncSetAttribute((const void*)topk_lists_kernel<uint32_t, false>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a7 = hipFuncSetAttribute((const void*)topk_lists_plan_kernel<uint64_t>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    static hipError_t a8 = hipFuncSetAttribute((const void*)topk_lists_plan_kernel<uint32_t>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, TOPK_KMAX * 8);
    return a0 != hipSuccess ? a0 : a1 != hipSuccess ? a1 : a2 != hipSuccess ? a2 : a3 != hipSuccess ? a3 : a4 != hipSuccess ? a4
           : a5 != hipSuccess ? a5 : a6 != hipSuccess ? a6 : a7 != hipSuccess ? a7 : a8 != hipSuccess ? a8 : a9 != hipSuccess ? a9 : a11 != hipSuccess ? a11 : a10;
}

hipError_t launch_topk_lists(const uint64_t* lists, uint64_t list_stride, const uint32_t* counts, uint32_t n_queries,
                             uint32_t k, uint32_t max_score, uint64_t max_id, const FilterHistPlan* hp, uint32_t* out_ids,
                             int32_t* out_scores, bool ordered, hipStream_t stream, uint32_t* emit_plan) {
    if (n_queries == 0 || k == 0) return hipSuccess;
    if (emit_plan && ordered) return hipErrorInvalidValue;  // the two-launch form leaves the result unordered
    if (k > TOPK_KMAX) return hipErrorInvalidValue;
    // the lists are read 16 bytes at a time
    if ((uintptr_t)lists % 16 || list_stride % 4) return hipErrorInvalidValue;
    uint32_t kpad = 2;
    while (kpad < k) kpad <<= 1;
    const KeyPlan plan = make_key_plan(max_score, max_id);
    const size_t lds = (size_t)kpad * 8;
    if (lds > 48 * 1024) {
        hipError_t e = allow_large_k();
        if (e != hipSuccess) return e;
    }
    const uint32_t hist_bins = (hp && hp->bins) ? hp->bins : 0;
    if (hist_bins && hist_bins != leading_score_bins(max_score, max_id)) return hipErrorInvalidValue;
    if (hist_bins && hp->rows && hp->slabs > TOPK_LIST_THREADS) return hipErrorInvalidValue;
    const uint32_t* hist0 = hist_bins ? counts + hp->hist_off : nullptr;
    const uint32_t* segs = (hist_bins && hp->rows) ? counts + hp->seg_off : nullptr;
    const uint32_t slabs = hist_bins ? hp->slabs : 0;
    const dim3 grid(n_queries), block(TOPK_LIST_THREADS);
    if (emit_plan) {
        const dim3 egrid(TOPK_EMIT_PARTS, n_queries), eblock(TOPK_EMIT_THREADS);
        if (keys_fit_32(max_score, max_id)) {
            hipLaunchKernelGGL(topk_lists_plan_kernel<uint32_t>, grid, block, lds, stream, (const uint32_t*)lists, list_stride, counts,
                               k, plan, kpad, out_ids, out_scores, hist0, hist_bins, segs, slabs, emit_plan);
            hipLaunchKernelGGL(topk_lists_emit_kernel<uint32_t>, egrid, eblock, 0, stream, (const uint32_t*)lists, list_stride,
                               counts, k, plan.id_bits, emit_plan, out_ids, out_scores);
        } else {
            hipLaunchKernelGGL(topk_lists_plan_kernel<uint64_t>, grid, block, lds, stream, lists, list_stride, counts, k, plan, kpad,
                               out_ids, out_scores, hist0, hist_bins, segs, slabs, emit_plan);
            hipLaunchKernelGGL(topk_lists_emit_kernel<uint64_t>, egrid, eblock, 0, stream, lists, list_stride, counts, k,
                               plan.id_bits, emit_plan, out_ids, out_scores);
        }
        return hipGetLastError();
    }
    if (keys_fit_32(max_score, max_id)) {
        auto kern = ordered ? topk_lists_kernel<uint32_t, true> : topk_lists_kernel<uint32_t, false>;
        hipLaunchKernelGGL(kern, grid, block, lds, stream, (const uint32_t*)lists, list_stride, counts, k, plan, kpad, out_ids,
                           out_scores, hist0, hist_bins, segs, slabs);
    } else {
        auto kern = ordered ? topk_lists_kernel<uint64_t, true> : topk_lists_kernel<uint64_t, false>;
        hipLaunchKernelGGL(kern, grid, block, lds, stream, lists, list_stride, counts, k, plan, kpad, out_ids, out_scores, hist0,
                           hist_bins, segs, slabs);
    }
    return hipGetLastError();
}

hipError_t launch_topk(const TopkArgs& a, hipStream_t stream) {
    if (a.n_queries == 0 || a.k == 0) return hipSuccess;
    if (a.k > TOPK_KMAX || a.n_queries > 65535) return hipErrorInvalidValue;
    uint32_t kpad = 2;
    while (kpad < a.k) kpad <<= 1;
    const KeyPlan plan = make_key_plan(a.max_score, a.n_docs ? a.n_docs - 1 : 0);
    const uint32_t slices = topk_slices(a.max_scored, a.n_queries);
    const size_t lds = (size_t)kpad * 8;
    if (lds > 48 * 1024) {
        hipError_t e = allow_large_k();
        if (e != hipSuccess) return e;
    }
    const bool fit32 = keys_fit_32(a.max_score, a.n_docs ? a.n_docs - 1 : 0);
    const dim3 grid(slices, a.n_queries);
    const uint64_t slice_len = (a.max_scored + slices - 1) / slices;
    if (fit32 && a.k <= TOPK_FEW && slices == 1 && slice_len <= 4096) {   // 512 scores per wave
        const uint32_t waves = slice_len <= 512 ? 1 : (uint32_t)((slice_len + 511) / 512);
        hipLaunchKernelGGL(topk_few_kernel, dim3(a.n_queries), dim3(64 * waves), 0, stream, a, plan.id_bits);
    } else
    // every slice short enough to stay in the registers of the wider workgroup (see topk_scores_kernel)
    if ((a.max_scored + slices - 1) / slices <= (uint64_t)TOPK_THREADS_SHORT * 4) {
        if (fit32)
            hipLaunchKernelGGL((topk_scores_kernel<uint32_t, TOPK_THREADS_SHORT, 4>), grid, dim3(TOPK_THREADS_SHORT), lds, stream, a, plan,
                               slices, kpad);
        else
            hipLaunchKernelGGL((topk_scores_kernel<uint64_t, TOPK_THREADS_SHORT, 4>), grid, dim3(TOPK_THREADS_SHORT), lds, stream, a, plan,
                               slices, kpad);
    } else if (fit32 && slice_len <= (uint64_t)TOPK_THREADS_SHORT * 16 && (uint64_t)slices * a.n_queries <= 256) {
        hipLaunchKernelGGL((topk_scores_kernel<uint32_t, TOPK_THREADS_SHORT, 16>), grid, dim3(TOPK_THREADS_SHORT), lds, stream, a, plan, slices,
                           kpad);
    } else {
        if (fit32)
            hipLaunchKernelGGL((topk_scores_kernel<uint32_t, TOPK_THREADS, 8>), grid, dim3(TOPK_THREADS), lds, stream, a, plan, slices, kpad);
        else
            hipLaunchKernelGGL((topk_scores_kernel<uint64_t, TOPK_THREADS, 8>), grid, dim3(TOPK_THREADS), lds, stream, a, plan, slices, kpad);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || slices == 1) return e;
    hipLaunchKernelGGL(topk_merge_kernel, dim3(a.n_queries), dim3(TOPK_THREADS), lds, stream, a, plan, slices, kpad);
    return hipGetLastError();
}

}  // namespace dessert
