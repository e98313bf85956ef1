// Short jobs that the query-hashing launch carries along in workgroups of its own: they need nothing from the hashing, everything here is
// latency-bound, and a launch less is a kernel boundary less on the stream.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cand_order.hpp"

namespace dessert {

constexpr int64_t LIST_EMPTY = INT64_MIN;

template <int P>
__device__ __forceinline__ void list_insert(int64_t (&best)[P], int64_t x) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const bool gt = x > best[i];
        const int64_t lo = gt ? best[i] : x;
        best[i] = gt ? x : best[i];
        x = lo;
    }
}

// Joining the probe lists that filter_gemm_kernel leaves per range of centroids: the `probe` best of a vector's per_vec entries, closest
// first.  One wave per vector.
struct ProbeMergeArgs {
    const int64_t* lists;   // nullptr: nothing to join
    uint64_t n;             // query vectors
    uint32_t per_vec, probe, width;   // width: 1, 2, 4 or 8, at least probe
    uint32_t* probe_ids;    // [n][probe]
};

// Lanes stride over the entries and keep sorted lists of their own, then the wave's largest head is taken P times (entries differ: they
// end in their centroid's id).  Bound: the round trips of one pass over the entries; 4096 vectors x 512 entries, 4 probes: 96 -> 7 us
// (one thread walked a vector's entries before, uncoalesced and with 16 workgroups in all).
template <int P>
__device__ inline void probe_merge(const ProbeMergeArgs& a, uint64_t v, uint32_t lane) {
    const int64_t* src = a.lists + v * a.per_vec;
    int64_t best[P];
#pragma unroll
    for (int i = 0; i < P; ++i) best[i] = LIST_EMPTY;
    constexpr uint32_t U = 4;   // loads in flight
    for (uint32_t i = lane; i < a.per_vec; i += 64 * U) {
        int64_t e[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) e[u] = i + 64 * u < a.per_vec ? src[i + 64 * u] : LIST_EMPTY;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (e[u] > best[P - 1]) list_insert<P>(best, e[u]);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
        int64_t top = best[0];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const int64_t other = __shfl_xor((long long)top, o, 64);
            top = other > top ? other : top;
        }
        if (lane == 0 && (uint32_t)i < a.probe) a.probe_ids[v * a.probe + i] = top == LIST_EMPTY ? 0xFFFFFFFFu : ~(uint32_t)top;
        if (P > 1 && best[0] == top) {   // the lane that holds it moves up
#pragma unroll
            for (int j = 0; j + 1 < P; ++j) best[j] = best[j + 1];
            best[P - 1] = LIST_EMPTY;
        }
    }
}
__device__ inline void probe_merge_any(const ProbeMergeArgs& a, uint64_t v, uint32_t lane) {
    if (v >= a.n) return;
    if (a.width == 1) probe_merge<1>(a, v, lane);
    else if (a.width == 2) probe_merge<2>(a, v, lane);
    else if (a.width == 4) probe_merge<4>(a, v, lane);
    else probe_merge<8>(a, v, lane);
}

struct HashRiders {   // a grouping and words to clear, or a join
    CandOrderArgs order;     // n_lists = 0: none.  A workgroup per list
    int32_t* zero;           // words to clear (scores that partial sums are added to): RIDER_ZERO_PER_WG to a workgroup
    uint64_t zero_words;
    ProbeMergeArgs merge;    // a wave per query vector
    bool any() const { return order.n_lists || zero_words || merge.lists; }
};
constexpr uint32_t RIDER_ZERO_PER_WG = 4096;

}  // namespace dessert
