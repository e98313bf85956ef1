// Closest centroid by groups of centroids: exact, with most distances never computed.
//
// Centroids are put into groups, each around one of them, its leader.  A vector x is compared with the leaders.  If l is its
// closest leader and every other leader l' lies so far that
//     |x - l'|  >  |x - l| + r,      r = the largest distance of a centroid from its leader,
// then by the triangle inequality every centroid c' of another group has |x - c'| >= |x - l'| - r > |x - l|: it is further off than
// the centroid l, and x's closest centroid is one of l's own group, the only one that is then read.  The other vectors ("the rest") go to
// a list and are compared with every centroid as before.  Distances are integers, square roots are taken with a margin far above their
// rounding, and ties go to the lower id as everywhere: the assignment is the same bit for bit.
//
// How wide a group may be decides what it is good for: as narrow as the centroids' own distances it is of no use, since in many dimensions
// a vector is almost as far from its second closest centroid as from its closest; once groups are as wide as the clusters of the
// data, few vectors are near to two.  So the width follows the vectors: sqrt(3) times the median distance of a vector
// from its closest centroid, over a sample.  (Mixture of 1024 centres, 4096 to 16 384 centroids, before and after rounds of k-means: 0 to
// 2 % of the vectors are left over, 1010 to 1036 groups; at sqrt(2) 1 to 7 %, at sqrt(1.5) 6 to 45 %.)  Where the data have no clusters the
// groups are too many or the rest is too large; a trial on 4096 vectors tells that on the device, and everything goes the old way: in a
// training also the next rounds, without another trial.
#include "filter_common.hpp"
#include "kernels.hpp"

namespace dessert {

constexpr uint32_t GROUP_SAMPLE = 512;   // vectors whose median distance sets the groups' width
constexpr uint32_t GROUP_PARTS = 16;     // of the centroids, looked through side by side for that sample

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int32_t init_of(int32_t w) { return w << 5 >> 5; }   // a row's word without parity and tie-break
// squared norm of centroid c from its word: the accumulators start from -ceil(|c|^2 / 2), the top bit is |c|^2 & 1
__device__ __forceinline__ int32_t norm_of(uint32_t w) { return -2 * init_of((int32_t)w) - (int32_t)(w >> 31); }
__device__ __forceinline__ uint32_t word_at(uint32_t c) {   // index of centroid c's word
    const uint32_t row = c & 31;
    return (c >> 5) * 32 + ((row >> 2) & 1) * 16 + 4 * (row >> 3) + (row & 3);
}
__device__ __forceinline__ int32_t dot16(v4i a, v4i b, int32_t s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_sdot4(a[i], b[i], s, false);
    return s;
}

// Squared distance from GROUP_SAMPLE vectors, taken evenly, to the closest centroid of each of GROUP_PARTS parts of the tiles; clears the
// counters for the launches that follow.  A workgroup's 16 waves hold the same 32 vectors and take every 16th tile of a part.  Bound:
// latency (the parts are there because one CU takes 16 us to read 2 MB of centroids: 38 us in one part, 8 in eight).
// before: what the round before left, or nullptr; where its groups did not pay, all launches of this one end at once.
template <int KS>
__global__ __launch_bounds__(1024) void group_near_kernel(const int8_t* __restrict__ X, uint64_t n, const v4i* __restrict__ Cp,
                                                          const v4i* __restrict__ W, uint32_t tiles, uint32_t K, uint32_t* __restrict__ near,
                                                          uint32_t* __restrict__ size, GroupCtl* __restrict__ ctl,
                                                          const GroupCtl* __restrict__ before) {
    constexpr int D = KS * 32;
    __shared__ int32_t s_val[16][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x;
    if (before && !groups_pay(*before, K)) {
        if (block == 0 && threadIdx.x == 0) {
            GroupCtl none{};
            none.skip = 1;
            *ctl = none;
        }
        return;
    }
    for (uint32_t i = block * 1024 + threadIdx.x; i < K; i += gridDim.x * gridDim.y * 1024) size[i] = 0;
    if (block == 0 && threadIdx.x == 0) *ctl = GroupCtl{};
    const uint64_t v = (uint64_t)(blockIdx.x * 32 + col) * n / GROUP_SAMPLE;
    const v4i* src = (const v4i*)(X + v * D + g * 16);
    v4i b[KS];
    int32_t xx = 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        b[ks] = src[ks * 2];
        xx = dot16(b[ks], b[ks], xx);
    }
    xx += __shfl_xor(xx, 32, 64);
    int32_t best = 2 * FILTER_PAD_INIT;   // what a wave without a tile reports: above every distance
    const uint32_t end = (uint32_t)((uint64_t)tiles * (blockIdx.y + 1) / GROUP_PARTS);
    for (uint32_t tile = (uint32_t)((uint64_t)tiles * blockIdx.y / GROUP_PARTS) + wave; tile < end; tile += 16) {
        v4i a[KS], row[4];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[ks] = Cp[((size_t)tile * KS + ks) * 64 + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) row[q] = W[(size_t)tile * 8 + g * 4 + q];
        v16i acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = init_of(row[r / 4][r % 4]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[ks], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int32_t value = (int32_t)__builtin_amdgcn_alignbit((uint32_t)acc[r], (uint32_t)row[r / 4][r % 4], 31);
            best = value > best ? value : best;
        }
    }
    const int32_t other = __shfl_xor(best, 32, 64);
    best = other > best ? other : best;
    if (g == 0) s_val[wave][col] = xx - best;
    __syncthreads();
    if (threadIdx.x < 32) {
        int32_t least = s_val[0][threadIdx.x];
        for (int w = 1; w < 16; ++w) least = s_val[w][threadIdx.x] < least ? s_val[w][threadIdx.x] : least;
        near[blockIdx.y * GROUP_SAMPLE + blockIdx.x * 32 + threadIdx.x] = (uint32_t)least;
    }
}

// Every centroid's leader: the lowest centroid whose squared distance from it is at most tau = 3 * median(near).  A workgroup's waves hold
// the same 64 centroids (32 at d = 256) and take every 8th tile up to their own (a centroid is within tau of itself), 32 tiles between
// two looks at what has been found: lower tiles come first, so the walk ends once every centroid has its leader.  16 384 centroids
// around 1024 centres, d = 128: 40 us, the few walks that find a leader late or not at all.
// looks != 0: only counts, by so many workgroups spread over the centroids, how many lead themselves (groups_hopeless).
template <int KS>
__global__ __launch_bounds__(512) void group_leader_kernel(const v4i* __restrict__ Cp, const v4i* __restrict__ W, uint32_t tiles, uint32_t K,
                                                           const uint32_t* __restrict__ near, uint32_t* __restrict__ leader,
                                                           uint32_t* __restrict__ member, uint32_t* __restrict__ size, GroupCtl* __restrict__ ctl,
                                                           uint32_t looks) {
    constexpr int NT = KS == 8 ? 1 : 2;
    constexpr uint32_t WAVES = 8, ROUND = 4 * WAVES;
    static_assert(GROUP_SAMPLE == WAVES * 64, "a thread per vector of the sample");
    __shared__ uint32_t s_near[GROUP_SAMPLE];
    __shared__ unsigned long long s_found[32 * NT];   // (id, value) of the lowest so far
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    if (ctl->skip || (!looks && groups_hopeless(ctl->led, ctl->alone))) return;   // as the launches before left it
    const uint32_t* words = (const uint32_t*)W;
    v4i b[NT][KS];
    int32_t norm[NT];
    const uint32_t all = (tiles + NT - 1) / NT;   // workgroups for every centroid; the longest walks start first
    const uint32_t first = (all - 1 - (looks ? blockIdx.x * all / looks : blockIdx.x)) * NT;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const uint32_t tile = first + nt < tiles ? first + nt : tiles - 1;
        norm[nt] = norm_of(words[word_at(tile * 32 + col)]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[nt][ks] = Cp[((size_t)tile * KS + ks) * 64 + lane];
    }
    uint32_t mine = near[threadIdx.x];
    for (uint32_t p = 1; p < GROUP_PARTS; ++p) {
        const uint32_t x = near[p * GROUP_SAMPLE + threadIdx.x];
        mine = x < mine ? x : mine;
    }
    s_near[threadIdx.x] = mine;
    const uint32_t end = first + NT < tiles ? first + NT : tiles;
    if (threadIdx.x < 32 * NT) s_found[threadIdx.x] = first * 32 + threadIdx.x < K ? ~0ull : 0ull;
    __syncthreads();
    // the median, bit by bit from above: the largest value with at most GROUP_SAMPLE / 2 others below it (every wave finds it for itself)
    uint32_t sample[WAVES], median = 0;
#pragma unroll
    for (uint32_t i = 0; i < WAVES; ++i) sample[i] = s_near[i * 64 + lane];
    for (uint32_t bit = 1u << 24; bit; bit >>= 1) {
        uint32_t below = 0;
#pragma unroll
        for (uint32_t i = 0; i < WAVES; ++i) below += (uint32_t)__builtin_popcountll(__ballot(sample[i] < (median | bit)));
        if (below <= GROUP_SAMPLE / 2) median |= bit;
    }
    const int32_t tau = median < (1u << 21) ? 3 * (int32_t)median : 1 << 22;
    int32_t least[NT];   // a value must reach it: above -2^24, where rows past K are
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) least[nt] = norm[nt] - tau;
    v4i a[KS], row[4], a_next[KS], row_next[4];
    auto load = [&](uint32_t tile, v4i (&frag)[KS], v4i (&consts)[4]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) frag[ks] = Cp[((size_t)tile * KS + ks) * 64 + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) consts[q] = W[(size_t)tile * 8 + g * 4 + q];
    };
    if ((uint32_t)wave < end) load((uint32_t)wave, a, row);
    for (uint32_t t0 = 0; t0 < end; t0 += ROUND) {
        for (uint32_t tile = t0 + wave; tile < t0 + ROUND && tile < end; tile += WAVES) {
            load(tile + WAVES < end ? tile + WAVES : tile, a_next, row_next);
            v16i init;
#pragma unroll
            for (int r = 0; r < 16; ++r) init[r] = init_of(row[r / 4][r % 4]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                v16i acc;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[nt][ks], ks == 0 ? init : acc, 0, 0, 0);
                int32_t m = max3(acc[0], acc[1], acc[2]);
#pragma unroll
                for (int r = 3; r < 15; r += 2) m = max3(m, acc[r], acc[r + 1]);
                m = acc[15] > m ? acc[15] : m;
                if (2 * m + 1 >= least[nt]) {
                    uint32_t id = 0xFFFFFFFFu;
                    int32_t val = 0;
#pragma unroll
                    for (int r = 15; r >= 0; --r) {   // the lowest row stays
                        const int32_t value = (int32_t)__builtin_amdgcn_alignbit((uint32_t)acc[r], (uint32_t)row[r / 4][r % 4], 31);
                        if (value >= least[nt]) {
                            id = tile * 32 + tile_row(r, g);
                            val = value;
                        }
                    }
                    if (id != 0xFFFFFFFFu) atomicMin(&s_found[nt * 32 + col], ((unsigned long long)id << 32) | (uint32_t)val);
                }
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[ks] = a_next[ks];
#pragma unroll
            for (int q = 0; q < 4; ++q) row[q] = row_next[q];
        }
        // nothing in a later tile is lower than what has been found
        __syncthreads();
        if (!__syncthreads_or(threadIdx.x < 32 * NT && s_found[threadIdx.x] == ~0ull)) break;
    }
    __syncthreads();
    const uint32_t c = first * 32 + threadIdx.x;
    uint32_t d2 = 0;
    if (threadIdx.x < 32 * NT && c < K) {   // lanes of the first wave
        const uint32_t l = (uint32_t)(s_found[threadIdx.x] >> 32);   // at most c
        if (looks) {
            const uint64_t alone = __ballot(l == c), led = __ballot(true);
            if (threadIdx.x == 0) {
                atomicAdd(&ctl->led, (uint32_t)__builtin_popcountll(led));
                atomicAdd(&ctl->alone, (uint32_t)__builtin_popcountll(alone));
            }
            return;
        }
        leader[c] = l;
        // The centroid's number within its group.  Lanes that share the first lane's leader take theirs together: in data without clusters
        // there are few groups, and an atomic to the same word as others takes 11 ns.
        const uint32_t l0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)l);
        const uint64_t same = __ballot(l == l0);
        uint32_t at = 0;
        if (l != l0 || threadIdx.x == 0) at = atomicAdd(size + l, l == l0 ? (uint32_t)__builtin_popcountll(same) : 1u);
        const uint32_t at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        member[c] = l == l0 ? at0 + (uint32_t)__builtin_popcountll(same & ((1ull << threadIdx.x) - 1)) : at;
        d2 = (uint32_t)(norm_of(words[word_at(c)]) - (int32_t)(uint32_t)s_found[threadIdx.x]);
    }
    if (wave == 0) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t other = (uint32_t)__shfl_xor((int)d2, o, 64);
            d2 = other > d2 ? other : d2;
        }
        if (lane == 0 && d2) atomicMax(&ctl->radius2, d2);
    }
}

// One workgroup: group numbers in order of their leaders, starts[group] = members of the groups before it, and size[leader] becomes the
// same start.  No more than room groups are written; none where the leaders were not all looked for.  A thread's 16 sizes come in four
// reads (in 16 the lines that each wave asks for, one a lane, took 4 of 10 us for 16 384 centroids); size has room for whole reads.
__global__ __launch_bounds__(1024) void group_starts_kernel(uint32_t* __restrict__ size, uint32_t K, uint32_t room, uint32_t* __restrict__ leads,
                                                            uint32_t* __restrict__ starts, GroupCtl* __restrict__ ctl) {
    __shared__ uint64_t wsum[16];
    if (ctl->skip || groups_hopeless(ctl->led, ctl->alone)) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint64_t carry = 0;   // groups in the high word, members in the low one
    for (uint32_t base = 0; base < K; base += 1024 * 16) {
        uint32_t x[16];
        const uint32_t first = base + tid * 16;
        uint64_t sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < 16; i += 4) {
            uint4 four = make_uint4(0, 0, 0, 0);
            if (first + i < K) four = *(const uint4*)(size + first + i);
            x[i] = four.x; x[i + 1] = four.y; x[i + 2] = four.z; x[i + 3] = four.w;
        }
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i) {
            if (first + i >= K) x[i] = 0;
            sum += ((uint64_t)(x[i] != 0) << 32) | x[i];
        }
        uint64_t incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t y = __shfl_up((unsigned long long)incl, o, 64);
            if ((int)lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint64_t all = 0;
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < wave) incl += wsum[w];
            all += wsum[w];
        }
        uint64_t run = carry + incl - sum;
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i)
            if (x[i]) {
                const uint32_t group = (uint32_t)(run >> 32);
                if (group < room) {
                    leads[group] = first + i;
                    starts[group] = (uint32_t)run;
                }
                size[first + i] = (uint32_t)run;
                run += (1ull << 32) | x[i];
            }
        carry += all;
        __syncthreads();
    }
    if (tid == 0) {
        const uint32_t groups = (uint32_t)(carry >> 32);
        ctl->groups = groups;
        if (groups <= room) starts[groups] = K;
    }
}

// The centroids' rows in group order, with their squared norms and ~ids beside them, and the leaders in MFMA operand order
// with what their rows' accumulators start from, -ceil(|c|^2 / 2).
template <int KS>
__global__ __launch_bounds__(256) void group_fill_kernel(const v4i* __restrict__ Cp, const uint32_t* __restrict__ W, uint32_t K, uint32_t room,
                                                         const uint32_t* __restrict__ leader, const uint32_t* __restrict__ member,
                                                         const uint32_t* __restrict__ start,
                                                         const uint32_t* __restrict__ leads, const GroupCtl* __restrict__ ctl,
                                                         v4i* __restrict__ rows, int2* __restrict__ meta, v4i* __restrict__ Lp,
                                                         int32_t* __restrict__ Lw) {
    constexpr uint32_t LPV = KS * 2;   // lanes to a centroid: 16-byte pieces of a row
    const uint32_t groups = ctl->groups;
    if (groups == 0 || groups > room) return;
    const uint32_t sub = threadIdx.x & (LPV - 1);
    const uint32_t first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
    for (uint32_t i = first; i < K * LPV; i += stride) {
        const uint32_t c = i / LPV, pos = start[leader[c]] + member[c];
        rows[(size_t)pos * LPV + sub] = Cp[((size_t)(c >> 5) * KS + sub / 2) * 64 + (c & 31) + 32 * (sub & 1)];
        if (sub == 0) meta[pos] = make_int2(norm_of(W[word_at(c)]), (int)~c);
    }
    const uint32_t tiles = (groups + 31) / 32;
    for (uint32_t i = first; i < tiles * KS * 64; i += stride) {
        const uint32_t l = i & 63, ks = (i >> 6) % KS, group = (i >> 6) / KS * 32 + (l & 31);
        v4i x = {0, 0, 0, 0};
        if (group < groups) {
            const uint32_t c = leads[group];
            x = Cp[((size_t)(c >> 5) * KS + ks) * 64 + (c & 31) + (l & 32)];
        }
        Lp[i] = x;
    }
    for (uint32_t i = first; i < tiles * 32; i += stride) {
        const uint32_t group = (i >> 5) * 32 + tile_row(i & 15, (i >> 4) & 1);
        Lw[i] = group < groups ? init_of((int32_t)W[word_at(leads[group])]) : FILTER_PAD_INIT;
    }
}

// DPP lane exchanges within 16 lanes: lane i gets lane (LPV - 1) - i's value of its aligned LPV lanes
template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
template <int LANES>
__device__ __forceinline__ int32_t mirror(int32_t x) {
    if constexpr (LANES == 16) return dpp<0x140>(x);       // row_mirror
    else if constexpr (LANES == 8) return dpp<0x141>(x);   // row_half_mirror
    else if constexpr (LANES == 4) return dpp<0x1B>(x);    // quad_perm 3,2,1,0
    else return dpp<0xB1>(x);                              // quad_perm 1,0,3,2
}
// s[j] of the LANES lanes added up for every j < LANES; lane i ends with the sum for j = i (in s[0])
template <int LANES>
__device__ __forceinline__ void add_scatter(int32_t* s, uint32_t lane) {
    constexpr int H = LANES / 2;
    const bool upper = (lane & H) != 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const int32_t keep = upper ? s[j + H] : s[j], give = upper ? s[j] : s[j + H];
        s[j] = keep + mirror<LANES>(give);
    }
    if constexpr (H > 1) add_scatter<H>(s, lane);
}
// the largest key of the LANES lanes, in all of them
template <int LANES>
__device__ __forceinline__ void best_of(int64_t& key) {
    const int64_t other = (int64_t)(((uint64_t)(uint32_t)mirror<LANES>((int32_t)(key >> 32)) << 32) | (uint32_t)mirror<LANES>((int32_t)key));
    if (other > key) key = other;
    if constexpr (LANES > 2) best_of<LANES / 2>(key);
}

// Vectors x leaders on the matrix cores as filter_gemm_kernel, then, vector by vector with KS lanes each, the members of the one group
// that it needs.  Of the leaders a lane keeps the largest accumulator of a tile, the largest of any other tile, and the best tile's
// accumulators themselves: the row, and the best of the other rows of that tile, are looked for once at the end.  (Both kept by row and tile
// all along: two operations more per accumulator, and the vector ALU, not the matrix cores, bounds the loop.)  h = x.c - ceil(|c|^2 / 2)
// gives |x - c|^2 = |x|^2 - 2 h - (0 or 1), which is as good as exact here: the larger for the closest leader, the smaller for the others.
// trial: only counts the vectors that need one group, and its members, among trial vectors taken evenly.
// Bound: both halves alike, the loop over the leaders by matrix cores and vector ALU in turn, the members by the CU's 64 bytes a cycle
// from L2 (17 rows a vector).  4.2M vectors of 128 dimensions, 1024 leaders of 16 384 centroids: 0.89 ms, of which 0.55 and 0.65 by themselves;
// comparing with every centroid takes 7.4 ms.
template <int KS, int NT>
__global__ __launch_bounds__(256, KS >= 8 ? 2 : 3) void group_assign_kernel(const int8_t* __restrict__ X, uint64_t n, uint32_t K,
                                                               const v4i* __restrict__ Lp, const v4i* __restrict__ Lw,
                                                               const uint32_t* __restrict__ starts, const v4i* __restrict__ rows,
                                                               const int2* __restrict__ meta, uint32_t max_group, GroupCtl* __restrict__ ctl,
                                                               uint32_t* __restrict__ assign, uint32_t* __restrict__ list, uint32_t trial) {
    constexpr int D = KS * 32, TG = FILTER_TG;
    __shared__ v4i sA[2][TG * KS * 64];
    __shared__ v4i sW[2][TG * 8];
    __shared__ uint2 s_run[4][32 * NT];   // the members of a vector's group; none: start = end
    const GroupCtl now = *ctl;
    if (trial ? now.groups == 0 || now.groups > groups_room(K) : !groups_pay(now, K)) return;   // the same for every thread of the launch
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const uint64_t v0 = ((uint64_t)blockIdx.x * 4 + wave) * (32 * NT);
    const uint64_t count = trial ? trial : n;
    const uint32_t t_end = (now.groups + 31) / 32;

    v4i b[NT][KS];
    v16i kept[NT];
    int32_t best[NT], second[NT];   // the best tile's largest accumulator, the largest of the others'
    uint32_t best_tile[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        uint64_t v = v0 + nt * 32 + col;
        if (v >= count) v = count - 1;
        if (trial) v = v * n / trial;
        const v4i* src = (const v4i*)(X + v * D + g * 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[nt][ks] = src[ks * 2];
        best[nt] = second[nt] = (int32_t)0x80000000;
        best_tile[nt] = 0;
    }
    auto stage = [&](uint32_t t0, int buf) {
        const uint32_t tg = t_end - t0 < TG ? t_end - t0 : TG;
        for (uint32_t i = threadIdx.x; i < tg * KS * 64; i += 256)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Lp + (size_t)t0 * KS * 64 + i),
                                             (__attribute__((address_space(3))) void*)&sA[buf][i - lane], 16, 0, 0);
        if (wave == 0 && (uint32_t)lane < tg * 8)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Lw + (size_t)t0 * 8 + lane),
                                             (__attribute__((address_space(3))) void*)&sW[buf][0], 16, 0, 0);
    };
    stage(0, 0);
    int buf = 0;
    for (uint32_t t0 = 0; t0 < t_end; t0 += TG, buf ^= 1) {
        const uint32_t tg = t_end - t0 < TG ? t_end - t0 : TG;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's copies into sA[buf] have landed
        __syncthreads();                                   // everyone's have, and everyone is done with the other buffer
        if (t0 + TG < t_end) stage(t0 + TG, buf ^ 1);
#pragma unroll 1
        for (uint32_t tt = 0; tt < tg; ++tt) {
            v16i init;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i t = sW[buf][tt * 8 + g * 4 + q];
#pragma unroll
                for (int j = 0; j < 4; ++j) init[4 * q + j] = t[j];
            }
            v4i a[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[ks] = sA[buf][(tt * KS + ks) * 64 + lane];
            auto multiply = [&](v16i& acc, int nt) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[nt][ks], ks == 0 ? init : acc, 0, 0, 0);
            };
            auto take = [&](const v16i& acc, int nt) {
                int32_t m = max3(acc[0], acc[1], acc[2]);
#pragma unroll
                for (int r = 3; r < 15; r += 2) m = max3(m, acc[r], acc[r + 1]);
                m = acc[15] > m ? acc[15] : m;
                second[nt] = med3_i32(best[nt], second[nt], m);
                if (m > best[nt]) {
                    best[nt] = m;
                    best_tile[nt] = t0 + tt;
                    kept[nt] = acc;
                }
            };
            v16i acc[2];
            multiply(acc[0], 0);
#pragma unroll
            for (int nt = 1; nt < NT; ++nt) {
                multiply(acc[nt & 1], nt);
                take(acc[(nt - 1) & 1], nt - 1);
            }
            take(acc[(NT - 1) & 1], NT - 1);
        }
    }
    const float radius = __fsqrt_rn((float)now.radius2);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        int32_t xx = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) xx = dot16(b[nt][ks], b[nt][ks], xx);
        xx += __shfl_xor(xx, 32, 64);
        int32_t val = best[nt], top = (int32_t)0x80000000, sec = (int32_t)0x80000000;
        uint32_t row = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sec = med3_i32(top, sec, kept[nt][r]);
            top = kept[nt][r] > top ? kept[nt][r] : top;
            row = kept[nt][r] == val ? r : row;
        }
        sec = second[nt] > sec ? second[nt] : sec;
        uint32_t group = best_tile[nt] * 32 + tile_row(row, g);
        const int32_t oval = __shfl_xor(val, 32, 64), osec = __shfl_xor(sec, 32, 64);
        const uint32_t ogroup = (uint32_t)__shfl_xor((int)group, 32, 64);
        sec = max3(oval < val ? oval : val, sec, osec);
        if (oval > val) {
            val = oval;
            group = ogroup;
        }
        const uint64_t v = v0 + nt * 32 + col;
        const bool mine = g == 0 && v < count;
        const uint32_t start = starts[group], end = starts[group + 1];
        // squared distances are below 2^25: the roots are good to 2^-10, the margin is 2^-4
        const bool one = __fsqrt_rn((float)(xx - 2 * sec - 1)) > __fsqrt_rn((float)(xx - 2 * val)) + radius + 0.0625f && end - start <= max_group;
        const uint64_t easy = __ballot(mine && one), rest = __ballot(mine && !one);
        if (trial) {
            uint32_t members = mine && one ? end - start : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) members += (uint32_t)__shfl_xor((int)members, o, 64);
            if (lane == 0 && easy) {
                atomicAdd(&ctl->easy, (uint32_t)__builtin_popcountll(easy));
                atomicAdd(&ctl->members, members);
            }
            continue;
        }
        if (g == 0) s_run[wave][nt * 32 + col] = mine && one ? make_uint2(start, end) : make_uint2(0, 0);
        if (rest) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&ctl->rest, (uint32_t)__builtin_popcountll(rest));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__builtin_popcountll(rest & ((1ull << lane) - 1));
            if (mine && !one) list[at] = (uint32_t)v;
        }
    }
    if (trial) return;
    // a wave's LDS operations execute in order; the fences keep the compiler from moving them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    constexpr uint32_t LPV = KS, AT_ONCE = 64 / LPV, SETS = KS == 2 ? 2 : 1;   // sets of LPV rows in flight
    const uint32_t sub = (uint32_t)lane & (LPV - 1);
    auto vector = [&](uint32_t i, v4i (&x)[2]) {   // a lane's two pieces of a row: number sub of either half
        const uint64_t v = v0 + i + (uint32_t)lane / LPV;
        const v4i* src = (const v4i*)(X + (v < n ? v : n - 1) * D) + sub;
        x[0] = src[0];
        x[1] = src[LPV];
    };
    // at most 2^20 rows of 256 bytes; OUTSIDE + what is added to it stays outside and below 2^32
    constexpr uint32_t OUTSIDE = 0x80000000u;
    const auto rows_buf = __builtin_amdgcn_make_buffer_rsrc((void*)rows, 0, (int)(K * (uint32_t)D), 0x00027000);
    const auto meta_buf = __builtin_amdgcn_make_buffer_rsrc((void*)meta, 0, (int)(K * 8), 0x00027000);
    v4i x_next[2];
    vector(0, x_next);
#pragma unroll 1
    for (uint32_t i = 0; i < 32 * NT; i += AT_ONCE) {
        const uint32_t vi = i + (uint32_t)lane / LPV;
        const uint2 run = s_run[wave][vi];
        const v4i x[2] = {x_next[0], x_next[1]};
        if (i + AT_ONCE < 32 * NT) vector(i + AT_ONCE, x_next);
        int64_t best_member = INT64_MIN;   // value in the high word, ~id in the low one
        for (uint32_t p = run.x; __any(p < run.y); p += LPV * SETS) {
            v4i y[SETS][LPV][2];
            v2i m[SETS];
            // lanes of vectors that are done ask for a row past the buffer's end and get none: the CU's 64 bytes a cycle count
#pragma unroll
            for (uint32_t s = 0; s < SETS; ++s) {
                const uint32_t q = p + s * LPV;
                m[s] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(meta_buf, q + sub < run.y ? (q + sub) * 8 : OUTSIDE, 0, 0));
#pragma unroll
                for (uint32_t j = 0; j < LPV; ++j) {
                    const uint32_t at = q + j < run.y ? (q + j) * (uint32_t)D + sub * 16 : OUTSIDE;
                    y[s][j][0] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rows_buf, at, 0, 0));
                    y[s][j][1] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rows_buf, at, LPV * 16, 0));
                }
            }
#pragma unroll
            for (uint32_t s = 0; s < SETS; ++s) {
                int32_t dot[LPV];
#pragma unroll
                for (uint32_t j = 0; j < LPV; ++j) dot[j] = dot16(x[1], y[s][j][1], dot16(x[0], y[s][j][0], 0));
                add_scatter<(int)LPV>(dot, sub);
                const int64_t key = (int64_t)(((uint64_t)(uint32_t)(2 * dot[0] - m[s][0]) << 32) | (uint32_t)m[s][1]);
                if (p + s * LPV + sub < run.y && key > best_member) best_member = key;
            }
        }
        best_of<(int)LPV>(best_member);
        if (sub == 0 && run.x < run.y) assign[v0 + vi] = ~(uint32_t)best_member;
    }
}

struct GroupLayout {
    size_t ctl, near, leader, member, size, leads, starts, meta, rows, Lp, Lw, total;
    uint32_t room;   // groups at most: more of them do not pay
};
GroupLayout group_layout(uint32_t K, uint32_t d) {
    GroupLayout w{};
    size_t p = 0;
    auto take = [&](size_t bytes) {
        const size_t at = p;
        p += (bytes + 255) / 256 * 256;
        return at;
    };
    w.room = groups_room(K);
    w.ctl = take(2 * sizeof(GroupCtl));   // of this round of k-means and the one before, in turn
    w.near = take((size_t)GROUP_PARTS * GROUP_SAMPLE * 4);
    w.leader = take((size_t)K * 4);
    w.member = take((size_t)K * 4);
    w.size = take((size_t)K * 4);
    w.leads = take((size_t)w.room * 4);
    w.starts = take((size_t)(w.room + 1) * 4);
    w.meta = take((size_t)K * 8);
    w.rows = take((size_t)K * d);
    w.Lp = take(filter_centroid_bytes(w.room, d));
    w.Lw = take(filter_table_bytes(w.room));
    w.total = p;
    return w;
}

template <int KS, int NT>
hipError_t launch_groups(const int8_t* X, uint64_t n, uint32_t K, const v4i* Cp, const v4i* W, void* buffer, uint32_t* assign, uint32_t* list,
                         uint32_t round, hipStream_t stream) {
    const GroupLayout w = group_layout(K, KS * 32);
    char* base = (char*)buffer;
    GroupCtl* ctl = (GroupCtl*)(base + w.ctl) + (round & 1);
    const GroupCtl* before = group_round_tries(round) ? nullptr : (GroupCtl*)(base + w.ctl) + (~round & 1);
    uint32_t *near = (uint32_t*)(base + w.near), *leader = (uint32_t*)(base + w.leader), *member = (uint32_t*)(base + w.member), *size = (uint32_t*)(base + w.size);
    uint32_t *leads = (uint32_t*)(base + w.leads), *starts = (uint32_t*)(base + w.starts);
    int32_t* Lw = (int32_t*)(base + w.Lw);
    int2* meta = (int2*)(base + w.meta);
    v4i *rows = (v4i*)(base + w.rows), *Lp = (v4i*)(base + w.Lp);
    const uint32_t tiles = filter_tiles(K);
    const uint32_t max_group = groups_largest(K);
    const uint64_t blocks = (n + 128 * NT - 1) / (128 * NT);
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(group_near_kernel<KS>, dim3(GROUP_SAMPLE / 32, GROUP_PARTS), dim3(1024), 0, stream, X, n, Cp, W, tiles, K, near, size, ctl, before);
    auto leaders = [&](uint32_t workgroups, uint32_t looks) {
        hipLaunchKernelGGL(group_leader_kernel<KS>, dim3(workgroups), dim3(512), 0, stream, Cp, W, tiles, K, near, leader, member, size, ctl, looks);
    };
    if (K >= GROUP_MANY) leaders(GROUP_LOOKS, GROUP_LOOKS);
    leaders(KS == 8 ? tiles : (tiles + 1) / 2, 0);
    hipLaunchKernelGGL(group_starts_kernel, dim3(1), dim3(1024), 0, stream, size, K, w.room, leads, starts, ctl);
    hipLaunchKernelGGL(group_fill_kernel<KS>, dim3(512), dim3(256), 0, stream, Cp, (const uint32_t*)W, K, w.room, leader, member, size, leads, ctl,
                       rows, meta, Lp, Lw);
    hipLaunchKernelGGL((group_assign_kernel<KS, NT>), dim3(GROUP_TRIAL / (128 * NT)), dim3(256), 0, stream, X, n, K, Lp, (const v4i*)Lw, starts,
                       rows, meta, max_group, ctl, assign, list, GROUP_TRIAL);
    hipLaunchKernelGGL((group_assign_kernel<KS, NT>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, K, Lp, (const v4i*)Lw, starts,
                       rows, meta, max_group, ctl, assign, list, 0u);
    return hipGetLastError();
}

}  // namespace

size_t filter_group_bytes(uint32_t K, uint32_t d) { return group_layout(K, d).total; }

const GroupCtl* group_ctl(const void* buffer, uint32_t round) { return (const GroupCtl*)buffer + (round & 1); }

hipError_t launch_group_assign(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2, void* buffer,
                               uint32_t* assign, uint32_t* list, uint32_t round, hipStream_t stream) {
    if (d == 64) return launch_groups<2, 2>(X, n, K, (const v4i*)Cp, (const v4i*)T2, buffer, assign, list, round, stream);
    if (d == 128) return launch_groups<4, 2>(X, n, K, (const v4i*)Cp, (const v4i*)T2, buffer, assign, list, round, stream);
    if (d == 256) return launch_groups<8, 2>(X, n, K, (const v4i*)Cp, (const v4i*)T2, buffer, assign, list, round, stream);
    return hipErrorInvalidValue;
}

}  // namespace dessert
