// Candidate filter for gfx950 (Sec. 5 "Filtering"): an inverted index from centroid ids to
// document ids, built from the closest centroid of every document vector, and the query-side
// probe-and-count that keeps the filter_k documents whose buckets are hit most often.
//
// "Closest" is the squared Euclidean distance with ties to the lower centroid id.  Since
// |x|^2 is common to all centroids, argmin_k |x - c_k|^2 = argmax_k (2 x.c_k - |c_k|^2): the
// dense part is an int8 GEMM (vectors x centroids) on v_mfma_i32_32x32x32_i8, exact in int32.
#include "filter_common.hpp"
#include "hash_riders.hpp"
#include "kernels.hpp"
#include "topk_select.hpp"

namespace dessert {

static bool filter_shape(uint32_t d) { return d == 64 || d == 128 || d == 256; }

constexpr int FILTER_RANGE_TILES = 8;  // ranges of the query side are whole multiples of it
constexpr int32_t FILTER_BIAS = 1 << 24;  // 2 x.c - |c|^2 lies in (-2^24, 2^24) for int8 vectors up to d = 256

// ---------------------------------------------------------------------------
// Centroids in MFMA operand order, [tiles][KS][64 lanes][16 B] (tile = 32 centroids, rows past K
// are zero), and one constant per row, W[tiles][2][16] for accumulator register r of lane half g:
//   bits 0..26   -ceil(|c|^2 / 2), signed: the accumulators start from it, so that after the MFMAs
//                acc = x.c - ceil(|c|^2 / 2) =: h  and  2 x.c - |c|^2 = 2 h + (|c|^2 & 1);
//                rows past K start from -2^23: a value of -2^24, below every real one (at least -3 * 128^2 * 256)
//   bits 27..30  15 - r
//   bit 31       |c|^2 & 1
// so that shifting the top bit, or the top five, of W into an accumulator (one v_alignbit) gives the row's value, or the key
// 16 * value + 15 - r that decides ties within a tile.  A lane's largest h bounds its largest value (<= 2 h + 1): most tiles
// are dismissed by a max over the raw accumulators, without building any key.
// One thread per row for the constants (its bytes in 16-byte loads), then one per 16-byte fragment for the copy: 16 384
// centroids of 128 bytes 242 -> 5 us (one thread took 16 rows byte by byte before).
__global__ __launch_bounds__(256) void filter_prep_kernel(const int8_t* __restrict__ Cn, uint32_t K, uint32_t d, int8_t* __restrict__ Cp,
                                                          uint32_t* __restrict__ W, uint32_t tiles) {
    const uint32_t KS = d / 32, stride = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t idx = first; idx < tiles * KS * 64; idx += stride) {
        const uint32_t l = idx & 63, ks = (idx >> 6) % KS, tile = (idx >> 6) / KS;
        const uint32_t c = tile * 32 + (l & 31);
        v4i x = {0, 0, 0, 0};
        if (c < K) __builtin_memcpy(&x, Cn + (size_t)c * d + ks * 32 + 16 * (l >> 5), 16);   // the caller's array, at any address
        ((v4i*)Cp)[idx] = x;
    }
    for (uint32_t idx = first; idx < tiles * 32; idx += stride) {
        const uint32_t r = idx & 15, g = (idx >> 4) & 1, tile = idx >> 5;
        const uint32_t c = tile * 32 + tile_row(r, g);
        int32_t h = FILTER_PAD_INIT;
        uint32_t par = 0;
        if (c < K) {
            int32_t nrm = 0;
            for (uint32_t i = 0; i < d; i += 16) {
                v4i x;
                __builtin_memcpy(&x, Cn + (size_t)c * d + i, 16);
#pragma unroll
                for (int w = 0; w < 4; ++w)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int32_t v = (int32_t)(int8_t)((uint32_t)x[w] >> (8 * e));
                        nrm += v * v;
                    }
            }
            h = -((nrm + 1) >> 1);
            par = (uint32_t)(nrm & 1);
        }
        W[idx] = (par << 31) | ((15 - r) << 27) | ((uint32_t)h & 0x7FFFFFFu);
    }
}

// ---------------------------------------------------------------------------
// vectors x centroids.  Each wave keeps 32*NT vectors as MFMA B fragments in registers and walks
// over a range of centroid tiles (blockIdx.y selects the range); the workgroup keeps two groups of TG
// tiles of centroids (and their key constants) in LDS, one being multiplied, one being filled.  Three epilogues:
//   MODE = 0      closest centroid of every vector (running max of the keys; the two lane halves
//                 of a column are merged at the end); one tile range only.
//   MODE = P > 0  the P best centroids each lane has seen, as sorted lists of 64-bit entries
//                 (value in the high word, ~id in the low word: larger = closer, then lower id),
//                 lists[v][range][half][P]; filter_merge_kernel joins the lists of a vector.
//   MODE = -1     the values 2 x.c - |c|^2 themselves, out[v][tiles*32] (any probe count).
// Bound: matrix cores.  Column tiles are multiplied one after the other, each while the one before is compared: two accumulator
// sets instead of one per column tile (202 -> 168 VGPRs at d = 128, three waves per SIMD instead of two).  With 512 tiles
// 38 % of the tiles can improve some lane of a wave, so what such a tile costs matters: 16 shifts and 8 maxima (parity and
// tie-break come out of the row's constant with the shift; about 64 operations when they were computed per row).  (No registers are spilled: where a list
// gives the vectors, their places are made anew at the end, see there; d = 256, 500 000 vectors, 16 384 centroids with 24 bytes of scratch a
// lane 1.05 of the time.)  4.2M vectors x
// 16 384 centroids, d = 128: 8.7 -> 7.4 ms = 2.4 POP/s, the share of nominal that a large bf16 matrix product reaches here.
// Four probes of 4096 vectors in 32 768 centroids 116 -> 54 us (32-bit sorted keys; 64-bit list inserts per row before).
// Waves per SIMD that the registers leave room for: 32*NT vectors as fragments (4*KS*NT), two accumulator sets, a tile's constants
constexpr int gemm_min_waves(int KS, int NT, int MODE) { return KS >= 8 ? 2 : KS * NT >= 8 || MODE > 1 ? 3 : 4; }

// What an assignment by groups (filter_groups.hip) leaves to the kernels that compare with every centroid: the vectors of its list, or all of
// them where the groups do not pay.  Two launches share it, whichever suits the number that is known on the device only: one takes up to
// `few` vectors, one more than that; the other ends at once.
struct Rest {
    const GroupCtl* ctl;   // nullptr: all n vectors, no list
    const uint32_t* list;
    uint32_t few;
};
// The vectors to do; false: none for this launch.  list becomes nullptr where it is not to be used.
__device__ __forceinline__ bool rest_of(Rest& rest, uint32_t K, bool many, uint64_t& n) {
    const GroupCtl c = *rest.ctl;
    if (groups_pay(c, K)) n = c.rest;
    else rest.list = nullptr;
    return n != 0 && (n > rest.few) == many;
}

template <int KS, int NT, int MODE, bool REST = false>
__global__ __launch_bounds__(256, gemm_min_waves(KS, NT, MODE)) void filter_gemm_kernel(const int8_t* __restrict__ X, uint64_t n,
                                                          const v4i* __restrict__ Cp, const v4i* __restrict__ W,
                                                          uint32_t tiles, uint32_t K, uint32_t tiles_per_range,
                                                          uint32_t* __restrict__ assign, int32_t* __restrict__ out,
                                                          int64_t* __restrict__ lists, uint32_t zero_words, Rest rest) {
    constexpr int D = KS * 32;
    constexpr int P = MODE > 0 ? MODE : 1;
    if constexpr (REST) {
        if (!rest_of(rest, K, true, n) || (uint64_t)blockIdx.x * (128 * NT) >= n) return;   // the same for the whole workgroup
    }
    // list modes do not write `assign`: there it names zero_words words that the first workgroup clears for the kernel
    // that follows (the counting kernel's list lengths), which saves a launch on the single-query path
    if constexpr (MODE > 0) {
        if (zero_words && blockIdx.x == 0 && blockIdx.y == 0)
            for (uint32_t i = threadIdx.x; i < zero_words; i += 256) assign[i] = 0;
    }
    // a list of one entry is an argmax: MODE = 1 keeps the 32-bit running key of MODE = 0 (no 64-bit list
    // inserts in the loop) and forms its list entry at the end
    constexpr bool ARGMAX = MODE == 0 || MODE == 1;
    // centroid tiles per group: two buffers of 8 would leave a CU with fewer workgroups than the registers allow
    constexpr int TG = FILTER_TG;
    // two groups of centroid tiles in LDS: while the waves multiply one, the next is copied from global memory
    // straight into the other buffer (global_load ... lds: no staging registers; a wave's 64 lanes fill
    // consecutive LDS), one barrier per group
    __shared__ v4i sA[2][TG * KS * 64];
    __shared__ v4i sW[2][TG * 8];  // 32 words per tile
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const uint64_t v0 = ((uint64_t)blockIdx.x * 4 + wave) * (32 * NT);
    const uint32_t t_begin = blockIdx.y * tiles_per_range;
    const uint32_t t_end = tiles - t_begin < tiles_per_range ? tiles : t_begin + tiles_per_range;

    v4i b[NT][KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        uint64_t v = v0 + nt * 32 + col;
        if (v >= n) v = n - 1;
        if (REST && rest.list) v = rest.list[v];
        const v4i* src = (const v4i*)(X + v * D + g * 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[nt][ks] = src[ks * 2];
    }
    // ARGMAX: best_key = 16 * value + (15 - register) of the best row so far, best_tile its tile
    int32_t best_key[NT];
    uint32_t best_tile[NT];
    // lists: `best` over the chunks of LIST_CHUNK tiles that are done, `near` of the chunk at hand as 32-bit keys
    // (value << 7 | 127 - position): value needs 25 bits, a lane's 16 rows of 8 tiles the other 7.  A key goes into the sorted
    // `near` with one max or median per entry; its entries join the 64-bit list once per chunk.
    constexpr uint32_t LIST_CHUNK = 8;
    int64_t best[NT][P];
    int32_t near[NT][P], bar[NT];   // bar: a value must exceed it to matter
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        best_key[nt] = bar[nt] = (int32_t)0x80000000;
        best_tile[nt] = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            best[nt][i] = LIST_EMPTY;
            near[nt][i] = (int32_t)0x80000000;
        }
    }
    auto fold = [&](uint32_t chunk0) {   // the keys of the chunk that starts at tile chunk0 join `best`
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const uint32_t at = 127 - ((uint32_t)near[nt][i] & 127u);
                const uint32_t cid = (chunk0 + (at >> 4)) * 32 + tile_row(at & 15, g);
                const int64_t e = (int64_t)(((uint64_t)(uint32_t)(near[nt][i] >> 7) << 32) | (uint32_t)~cid);
                if (near[nt][i] != (int32_t)0x80000000 && cid < K && e > best[nt][P - 1]) list_insert<P>(best[nt], e);
                near[nt][i] = (int32_t)0x80000000;
            }
            bar[nt] = (int32_t)(best[nt][P - 1] >> 32);
        }
    };

    static_assert(TG * 8 <= 64, "the constants of a group are one wave's copy");
    auto stage = [&](uint32_t t0, int buf) {  // every copy instruction is issued by whole waves (exec masks the tail)
        const uint32_t tg = t_end - t0 < TG ? t_end - t0 : TG;
        for (uint32_t i = threadIdx.x; i < tg * KS * 64; i += 256)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Cp + (size_t)t0 * KS * 64 + i),
                                             (__attribute__((address_space(3))) void*)&sA[buf][i - lane], 16, 0, 0);
        if (wave == 0 && (uint32_t)lane < tg * 8)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(W + (size_t)t0 * 8 + lane),
                                             (__attribute__((address_space(3))) void*)&sW[buf][0], 16, 0, 0);
    };
    if (t_begin < t_end) stage(t_begin, 0);
    int buf = 0;
    uint32_t in_chunk = 0;   // lists: tiles of the chunk at hand that are done
    for (uint32_t t0 = t_begin; t0 < t_end; t0 += TG, buf ^= 1) {
        const uint32_t tg = t_end - t0 < TG ? t_end - t0 : TG;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's copies into sA[buf] have landed
        __syncthreads();                                   // everyone's have, and everyone is done with the other buffer
        if (t0 + TG < t_end) stage(t0 + TG, buf ^ 1);
#pragma unroll 1
        for (uint32_t tt = 0; tt < tg; ++tt) {
            uint32_t w[16];
            v16i init;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i t = sW[buf][tt * 8 + g * 4 + q];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    w[4 * q + j] = (uint32_t)t[j];
                    init[4 * q + j] = t[j] << 5 >> 5;
                }
            }
            v4i a[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[ks] = sA[buf][(tt * KS + ks) * 64 + lane];
            auto multiply = [&](v16i& acc, int nt) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[nt][ks], ks == 0 ? init : acc, 0, 0, 0);
            };
            auto value = [&](const v16i& acc, int r) { return (int32_t)__builtin_amdgcn_alignbit((uint32_t)acc[r], w[r], 31); };
            auto take = [&](const v16i& acc, int nt) {
                if constexpr (MODE < 0) {
                    const uint64_t v = v0 + nt * 32 + col;
                    if (v < n) {
                        int32_t* dst = out + v * ((uint64_t)tiles * 32) + (uint64_t)(t0 + tt) * 32 + 4 * g;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            v4i o;
#pragma unroll
                            for (int j = 0; j < 4; ++j) o[j] = value(acc, 4 * q + j);
                            *(v4i*)(dst + 8 * q) = o;
                        }
                    }
                } else {
                    int32_t m = max3(acc[0], acc[1], acc[2]);
#pragma unroll
                    for (int r = 3; r < 15; r += 2) m = max3(m, acc[r], acc[r + 1]);
                    m = acc[15] > m ? acc[15] : m;
                    // a lane meets centroid ids in increasing tile order, so only a strictly larger value can
                    // replace what it holds, and no value of this tile exceeds 2 m + 1
                    const int32_t bound = ARGMAX ? best_key[nt] >> 4 : bar[nt];
                    if (2 * m + 1 > bound) {
                        if constexpr (ARGMAX) {
                            int32_t key[16];   // equal values: the lower register = lower row
#pragma unroll
                            for (int r = 0; r < 16; ++r) key[r] = (int32_t)__builtin_amdgcn_alignbit((uint32_t)acc[r], w[r], 27);
                            int32_t km = max3(key[0], key[1], key[2]);
#pragma unroll
                            for (int r = 3; r < 15; r += 2) km = max3(km, key[r], key[r + 1]);
                            km = key[15] > km ? key[15] : km;
                            if ((km >> 4) > bound) {
                                best_key[nt] = km;
                                best_tile[nt] = t0 + tt;
                            }
                        } else {
                            const uint32_t top = 127 - in_chunk * 16;
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                const int32_t key = (int32_t)(((uint32_t)value(acc, r) << 7) + (top - r));
#pragma unroll
                                for (int i = P - 1; i > 0; --i) near[nt][i] = med3_i32(near[nt][i - 1], near[nt][i], key);
                                near[nt][0] = key > near[nt][0] ? key : near[nt][0];
                            }
                            const int32_t last = near[nt][P - 1] >> 7, far = (int32_t)(best[nt][P - 1] >> 32);
                            bar[nt] = last > far ? last : far;
                        }
                    }
                }
            };
            // the products of one column tile run on the matrix cores while the one before is compared
            v16i acc[2];
            multiply(acc[0], 0);
#pragma unroll
            for (int nt = 1; nt < NT; ++nt) {
                multiply(acc[nt & 1], nt);
                take(acc[(nt - 1) & 1], nt - 1);
            }
            take(acc[(NT - 1) & 1], NT - 1);
            if constexpr (MODE > 1) {
                if (++in_chunk == LIST_CHUNK) {
                    fold(t0 + tt + 1 - LIST_CHUNK);
                    in_chunk = 0;
                }
            }
        }
    }
    if constexpr (MODE > 1) {
        if (in_chunk) fold(t_end - in_chunk);
    }
    if constexpr (MODE == 0) {
        // the vectors' places anew from the thread: where the list gives them the compiler keeps their addresses all along otherwise, and spills
        uint32_t thread = threadIdx.x;
        if constexpr (REST) asm volatile("" : "+v"(thread));
        const uint64_t first = ((uint64_t)blockIdx.x * 4 + thread / 64) * (32 * NT) + (thread & 31);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            int32_t val = best_key[nt] >> 4;
            uint32_t c = best_tile[nt] * 32 + tile_row(15 - (best_key[nt] & 15), g);
            int32_t oval = __shfl_xor(val, 32, 64);
            uint32_t oc = (uint32_t)__shfl_xor((int)c, 32, 64);
            if (oval > val || (oval == val && oc < c)) c = oc;
            const uint64_t v = first + nt * 32;
            if (g == 0 && v < n) assign[REST && rest.list ? rest.list[v] : v] = c;
        }
    } else if constexpr (MODE > 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (MODE == 1) {
                const uint32_t cid = best_tile[nt] * 32 + tile_row(15 - (best_key[nt] & 15), g);
                const int32_t val = best_key[nt] >> 4;
                best[nt][0] = (best_key[nt] != (int32_t)0x80000000 && cid < K)
                                  ? (int64_t)(((uint64_t)(uint32_t)val << 32) | (uint32_t)~cid)
                                  : LIST_EMPTY;
            }
            const uint64_t v = v0 + nt * 32 + col;
            if (v < n) {
                int64_t* dst = lists + ((v * gridDim.y + blockIdx.y) * 2 + g) * P;
#pragma unroll
                for (int i = 0; i < P; ++i) dst[i] = best[nt][i];
            }
        }
    }
}

// Closest centroid of a few vectors (too few workgroups of the kernel above to fill the chip, and long walks over the centroids in
// each): a workgroup's 8 or 16 waves hold the SAME 32*NT vectors and take every 8th or 16th centroid tile, straight from L2 into
// registers, the next tile on its way while one is multiplied: a tile has one reader in the workgroup, so LDS would bring
// nothing.  No barrier until the waves' winners meet.  Bound: L2 to registers (the centroids once per 32*NT vectors).
// A k-means round of 12 000 vectors, 16 384 centroids, d = 128: 461 -> 177 us.
template <int KS, int NT, int WAVES, bool REST = false>
__global__ __launch_bounds__(WAVES * 64) void filter_assign_few_kernel(const int8_t* __restrict__ X, uint64_t n,
                                                                                const v4i* __restrict__ Cp, const v4i* __restrict__ W,
                                                                                uint32_t tiles, uint32_t K, uint32_t* __restrict__ assign,
                                                                                Rest rest) {
    constexpr int D = KS * 32;
    if constexpr (REST) {
        if (!rest_of(rest, K, false, n) || (uint64_t)blockIdx.x * (32 * NT) >= n) return;   // the same for the whole workgroup
    }
    __shared__ int32_t s_val[WAVES][32 * NT];
    __shared__ uint32_t s_id[WAVES][32 * NT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const uint64_t v0 = (uint64_t)blockIdx.x * (32 * NT);
    v4i b[NT][KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        uint64_t v = v0 + nt * 32 + col;
        if (v >= n) v = n - 1;
        if (REST && rest.list) v = rest.list[v];
        const v4i* src = (const v4i*)(X + v * D + g * 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[nt][ks] = src[ks * 2];
    }
    int32_t best_key[NT];      // as in the kernel above
    uint32_t best_tile[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        best_key[nt] = (int32_t)0x80000000;
        best_tile[nt] = 0;
    }
    v4i a[KS], row[4], a_next[KS], row_next[4];
    auto load = [&](uint32_t tile, v4i (&frag)[KS], v4i (&consts)[4]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) frag[ks] = Cp[((size_t)tile * KS + ks) * 64 + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) consts[q] = W[(size_t)tile * 8 + g * 4 + q];
    };
    uint32_t tile = (uint32_t)wave;
    if (tile < tiles) load(tile, a, row);
    for (; tile < tiles; tile += WAVES) {
        const uint32_t next = tile + WAVES < tiles ? tile + WAVES : tile;
        load(next, a_next, row_next);
        v16i init;
#pragma unroll
        for (int r = 0; r < 16; ++r) init[r] = row[r / 4][r % 4] << 5 >> 5;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            v16i acc;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], b[nt][ks], ks == 0 ? init : acc, 0, 0, 0);
            int32_t key[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) key[r] = (int32_t)__builtin_amdgcn_alignbit((uint32_t)acc[r], (uint32_t)row[r / 4][r % 4], 27);
            int32_t km = max3(key[0], key[1], key[2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) km = max3(km, key[r], key[r + 1]);
            km = key[15] > km ? key[15] : km;
            const bool better = (km >> 4) > (best_key[nt] >> 4);   // equal values: the lower tile stays
            best_key[nt] = better ? km : best_key[nt];
            best_tile[nt] = better ? tile : best_tile[nt];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[ks] = a_next[ks];
#pragma unroll
        for (int q = 0; q < 4; ++q) row[q] = row_next[q];
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        int32_t val = best_key[nt] >> 4;   // a wave without a tile: below every value
        uint32_t c = best_tile[nt] * 32 + tile_row(15 - (best_key[nt] & 15), g);
        const int32_t oval = __shfl_xor(val, 32, 64);
        const uint32_t oc = (uint32_t)__shfl_xor((int)c, 32, 64);
        if (oval > val || (oval == val && oc < c)) {
            val = oval;
            c = oc;
        }
        if (g == 0) {
            s_val[wave][nt * 32 + col] = val;
            s_id[wave][nt * 32 + col] = c;
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 32 * NT; i += WAVES * 64) {
        int32_t val = s_val[0][i];
        uint32_t c = s_id[0][i];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const int32_t oval = s_val[w][i];
            const uint32_t oc = s_id[w][i];
            if (oval > val || (oval == val && oc < c)) {
                val = oval;
                c = oc;
            }
        }
        if (v0 + i < n) assign[REST && rest.list ? rest.list[v0 + i] : v0 + i] = c;
    }
}

// the probe lists joined in a launch of its own (hash_riders.hpp)
template <int P>
__global__ __launch_bounds__(256) void filter_merge_kernel(ProbeMergeArgs a) {
    const uint64_t v = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v < a.n) probe_merge<P>(a, v, threadIdx.x & 63);
}

// ---------------------------------------------------------------------------
// Inverted index.  One wave per document; a vector counts if it is the one that puts its centroid into the document's set
// (a bucket holds a document once).  A document goes to sub-bucket c*S + (doc >> sub_shift) of its centroid c.  FILL = false counts
// sub-bucket sizes; FILL = true writes document ids at sub_off[...] + (atomic cursor), so the order inside
// a sub-bucket is unspecified.
// The set is an open-addressing table in LDS, per wave, when the document has at most DOC_SET_MAX vectors: some three
// compare-and-swap round trips per 64 vectors.  Longer documents compare each vector with all before it by lane broadcast, 64 of them
// per 64 vectors and chunk, as all documents did before: 60 000 documents of 70 vectors, 16 384 centroids 231 -> 199 us counting,
// 238 -> 201 us filling.  Bound now: the counters' atomics, 4.1M to random places at 20 G/s.  Few counters would share
// lines, and atomics to one line wait for each other (4.5 G/s over 932 counters in 59 lines): up to COUNTER_WORDS words counter i
// lies at word i << spread, a line of its own if they are few enough: 648 000 vectors, 932 centroids 145 -> 40 us a pass.
constexpr uint64_t COUNTER_WORDS = 65536;
static uint32_t counter_spread(uint64_t counters) {
    uint32_t spread = 0;
    while (spread < 4 && (counters << (spread + 1)) <= COUNTER_WORDS) ++spread;
    return spread;
}
constexpr uint32_t DOC_SET = 512, DOC_SET_MAX = 384, DOC_SET_EMPTY = 0xFFFFFFFFu;
template <bool FILL>
__global__ __launch_bounds__(256) void filter_bucket_kernel(const uint32_t* __restrict__ assign,
                                                            const uint64_t* __restrict__ doc_off, uint64_t n_docs,
                                                            uint32_t S, uint32_t sub_shift, uint32_t spread,
                                                            uint32_t* __restrict__ size_or_cursor,
                                                            const uint32_t* __restrict__ sub_off,
                                                            uint32_t* __restrict__ bucket_docs) {
    __shared__ uint4 sets[4][DOC_SET / 4];
    const uint32_t lane = threadIdx.x & 63;
    uint4* set4 = sets[threadIdx.x >> 6];
    uint32_t* set = (uint32_t*)set4;
    auto enter = [&](uint64_t doc, uint32_t c) {
        const uint32_t sub = c * S + (uint32_t)(doc >> sub_shift);
        uint32_t pos = atomicAdd(&size_or_cursor[(size_t)sub << spread], 1u);
        if constexpr (FILL) bucket_docs[sub_off[sub] + pos] = (uint32_t)doc;
    };
    for (uint64_t doc = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); doc < n_docs; doc += (uint64_t)gridDim.x * 4) {
        const uint64_t lo = doc_off[doc], hi = doc_off[doc + 1];
        if (hi - lo <= DOC_SET_MAX) {
            const uint32_t m = (uint32_t)(hi - lo);
            uint32_t log_slots = 7;   // at least a quarter of the slots stays free
            while (log_slots < 9 && (1u << log_slots) * 3 < m * 4) ++log_slots;
            const uint32_t slots = 1u << log_slots;
            for (uint32_t i = lane; i < slots / 4; i += 64) set4[i] = uint4{DOC_SET_EMPTY, DOC_SET_EMPTY, DOC_SET_EMPTY, DOC_SET_EMPTY};
            uint32_t next = lane < m ? assign[lo + lane] : 0;
            // a wave's LDS operations execute in order; the fences keep the compiler from moving them
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (uint32_t j0 = 0; j0 < m; j0 += 64) {
                const uint32_t c = next;
                if (j0 + 64 + lane < m) next = assign[lo + j0 + 64 + lane];
                bool pending = j0 + lane < m, first = false;
                uint32_t at = (c * 0x9E3779B1u) >> (32 - log_slots);
                while (__any(pending)) {   // ends: a free slot lies behind every start
                    if (pending) {
                        const uint32_t old = atomicCAS(&set[at], DOC_SET_EMPTY, c);
                        first = old == DOC_SET_EMPTY;
                        pending = !first && old != c;
                        at = (at + 1) & (slots - 1);
                    }
                }
                if (first) enter(doc, c);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        for (uint64_t j0 = lo; j0 < hi; j0 += 64) {  // 64 vectors of the document per pass, one per lane
            const bool valid = j0 + lane < hi;
            const uint32_t c = valid ? assign[j0 + lane] : 0xFFFFFFFFu;
            bool first = valid;
            for (uint64_t e0 = lo; e0 <= j0; e0 += 64) {  // against every earlier vector, 64 at a time
                const uint32_t ce = e0 == j0 ? c : assign[e0 + lane];  // e0 < j0: a full chunk
                const uint32_t cnt = e0 == j0 ? (uint32_t)(hi - j0 < 64 ? hi - j0 : 64) : 64u;
                for (uint32_t e = 0; e < cnt; ++e) {
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)ce, (int)e);
                    if (v == c && (e0 < j0 || e < lane)) first = false;
                }
            }
            if (first) enter(doc, c);
        }
    }
}

// Exclusive scan of size[0..K) into off[0..K]; size is zeroed for reuse as cursors.  Three launches: workgroup i adds up its
// SCAN_PART entries and leaves the sum in off[i * SCAN_PART], one workgroup scans those sums where they lie, workgroup i scans
// its entries from there on.  (One workgroup walked over all entries before, 1.1 us per 1024: 37 us for 32 768, 2.3 ms for 2M.)  One
// part needs the last of the three alone: with all of them the filter over one centroid and 10 documents took 71 -> 79 us to build.
constexpr uint32_t SCAN_THREADS = 256, SCAN_PART = SCAN_THREADS * 16;
// inclusive prefix sum over the workgroup's threads; wsum: SCAN_THREADS / 64 words, free again after the call's last barrier
__device__ inline uint32_t scan_threads(uint32_t x, uint32_t* wsum) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if ((int)lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    for (uint32_t w = 0; w < wave; ++w) incl += wsum[w];
    __syncthreads();
    return incl;
}
__device__ inline uint32_t scan_load16(const uint32_t* size, uint32_t first, uint32_t K, uint32_t spread, uint32_t (&x)[16]) {
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
        x[i] = first + i < K ? size[(size_t)(first + i) << spread] : 0;
        sum += x[i];
    }
    return sum;
}
__global__ __launch_bounds__(SCAN_THREADS) void filter_scan_sums_kernel(const uint32_t* __restrict__ size, uint32_t K, uint32_t spread,
                                                                        uint32_t* __restrict__ off) {
    __shared__ uint32_t wsum[SCAN_THREADS / 64];
    uint32_t x[16];
    const uint32_t sum = scan_load16(size, blockIdx.x * SCAN_PART + threadIdx.x * 16, K, spread, x);
    const uint32_t incl = scan_threads(sum, wsum);
    if (threadIdx.x == SCAN_THREADS - 1) off[(size_t)blockIdx.x * SCAN_PART] = incl;
}
__global__ __launch_bounds__(SCAN_THREADS) void filter_scan_parts_kernel(uint32_t* __restrict__ off, uint32_t parts, uint32_t K) {
    __shared__ uint32_t wsum[SCAN_THREADS / 64];
    __shared__ uint32_t last;
    uint32_t carry = 0;
    for (uint32_t p0 = 0; p0 < parts; p0 += SCAN_THREADS) {
        const uint32_t p = p0 + threadIdx.x;
        const uint32_t x = p < parts ? off[(size_t)p * SCAN_PART] : 0;
        const uint32_t incl = scan_threads(x, wsum);
        if (p < parts) off[(size_t)p * SCAN_PART] = carry + incl - x;
        if (threadIdx.x == SCAN_THREADS - 1) last = incl;
        __syncthreads();
        carry += last;
        __syncthreads();
    }
    if (threadIdx.x == 0) off[K] = carry;
}
__global__ __launch_bounds__(SCAN_THREADS) void filter_scan_kernel(uint32_t* __restrict__ size, uint32_t K, uint32_t spread,
                                                                   uint32_t* __restrict__ off, uint32_t alone) {
    __shared__ uint32_t wsum[SCAN_THREADS / 64];
    uint32_t x[16];
    const uint32_t first = blockIdx.x * SCAN_PART + threadIdx.x * 16;
    const uint32_t base = alone ? 0u : off[(size_t)blockIdx.x * SCAN_PART];   // read by all before scan_threads' barriers, rewritten after them
    const uint32_t sum = scan_load16(size, first, K, spread, x);
    const uint32_t incl = scan_threads(sum, wsum);
    if (alone && threadIdx.x == SCAN_THREADS - 1) off[K] = incl;
    uint32_t run = base + incl - sum;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i)
        if (first + i < K) {
            off[first + i] = run;
            size[(size_t)(first + i) << spread] = 0;
            run += x[i];
        }
}
static void launch_filter_scan(uint32_t* size, uint32_t K, uint32_t spread, uint32_t* off, hipStream_t stream) {   // K >= 1
    const uint32_t parts = (K + SCAN_PART - 1) / SCAN_PART;
    if (parts > 1) {
        hipLaunchKernelGGL(filter_scan_sums_kernel, dim3(parts), dim3(SCAN_THREADS), 0, stream, size, K, spread, off);
        hipLaunchKernelGGL(filter_scan_parts_kernel, dim3(1), dim3(SCAN_THREADS), 0, stream, off, parts, K);
    }
    hipLaunchKernelGGL(filter_scan_kernel, dim3(parts), dim3(SCAN_THREADS), 0, stream, size, K, spread, off, parts == 1 ? 1u : 0u);
}

// bucket_off[c] = sub_off[c*S] for c = 0..K: the caller-visible bucket starts
__global__ void filter_bucket_starts_kernel(const uint32_t* __restrict__ sub_off, uint32_t K, uint32_t S,
                                            uint32_t* __restrict__ bucket_off) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= K) bucket_off[c] = sub_off[(size_t)c * S];
}

// ---------------------------------------------------------------------------
// Query side.
struct DistKeys {  // key = (value + bias) above the centroid id: closest first, lower id first
    const int32_t* row;
    uint32_t id_bits;
    static constexpr int VEC = 1;
    static constexpr bool SEGMENTS = false;
    using key_t = uint64_t;
    __device__ uint64_t operator()(uint64_t i) const { return make_key(row[i] + FILTER_BIAS, (uint32_t)i, id_bits); }
    __device__ void load(uint64_t i, uint64_t n, uint64_t (&out)[1]) const { out[0] = i < n ? (*this)(i) : 0; }
};

// one workgroup per query vector: its `probe` closest centroids, closest first
__global__ __launch_bounds__(256) void filter_probe_kernel(const int32_t* __restrict__ dist, uint32_t row_stride,
                                                           uint32_t K, uint32_t probe, uint32_t kpad, KeyPlan plan,
                                                           uint32_t* __restrict__ probe_ids) {
    extern __shared__ uint64_t sorted[];
    __shared__ SelectShared sh;
    const uint32_t q = blockIdx.x;
    DistKeys keys{dist + (size_t)q * row_stride, plan.id_bits};
    block_select<256>(keys, K, probe, kpad, sorted, sh, plan);
    const uint64_t idmask = (1ull << plan.id_bits) - 1;
    for (uint32_t i = threadIdx.x; i < probe; i += 256)
        probe_ids[(size_t)q * probe + i] = sorted[i] ? (uint32_t)(idmask - (sorted[i] & idmask)) : 0xFFFFFFFFu;
}

__global__ void filter_zero_kernel(int32_t* __restrict__ p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Bucket counting without global atomics.  Workgroup (slab, query set) owns the documents
// [slab * slab_docs, +slab_docs) and keeps one counter per document in LDS (W bytes each, packed into
// 32-bit words; a count never exceeds the number of probed buckets, which the host bounds by the
// counter range).  It reads, of every bucket its query set probes, the sub-buckets that overlap its slab
// (long ranges 64 elements to a load, eight loads in flight; short ones as one concatenated run, see below),
// counts the ids that fall into the slab, and remembers each document at its first hit in a queue.  Then
// one key (count, id) in the top-k key format per queued document goes to the query set's list;
// cursor[b] ends as the number of distinct documents hit.  The order inside a list is unspecified.
// Only if the queue overflows (more than FILTER_QUEUE distinct documents of one slab hit) are the counters
// scanned instead.
// first-hit queue entries per workgroup (positions within the slab: QT = u16, or u32 for slabs over 65536 documents).
// 3456: with a slab of 32768 one-byte counters and the histogram below the workgroup then needs just under 40 KB
// of LDS and four fit a CU.
constexpr uint32_t FILTER_QUEUE = 3456;
// bins of the per-workgroup histogram of counts: all that one-byte counters can have (with 256 a count of 255 needs a way of its own: one query
// set 0.3 us more, 128 sets of 128 probed buckets 678 -> 673 us a search)
constexpr uint32_t FILTER_HSMALL = 257;

template <int W, int T, typename QT, typename KT>
__global__ __launch_bounds__(T) void filter_count_kernel(const uint32_t* __restrict__ probe_ids, uint32_t probe,
                                                            const uint32_t* __restrict__ q_off, uint32_t q_uniform,
                                                            const uint32_t* __restrict__ sub_off, uint32_t S,
                                                            uint32_t sub_shift,
                                                            const uint32_t* __restrict__ bucket_docs, uint64_t n_docs,
                                                            uint32_t slab_docs, uint32_t id_bits,
                                                            KT* __restrict__ lists, uint64_t list_stride,
                                                            uint32_t* __restrict__ cursor, uint32_t* __restrict__ hist,
                                                            uint32_t hist_bins, uint32_t* __restrict__ segs) {
    extern __shared__ uint32_t cnt[];
    __shared__ QT queue[FILTER_QUEUE];
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t base_sh, q_count;
    constexpr uint32_t PER = 4 / W, BITS = 8 * W, WAVES = T / 64;
    constexpr uint32_t MASK = W == 4 ? 0xFFFFFFFFu : (1u << (BITS % 32)) - 1;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t b = blockIdx.y;
    const uint32_t doc0 = blockIdx.x * slab_docs;
    const uint32_t here = n_docs - doc0 < slab_docs ? (uint32_t)(n_docs - doc0) : slab_docs;
    const uint32_t words = (here + PER - 1) / PER;
    const uint32_t q_lo = q_uniform ? b * q_uniform : q_off[b];
    const uint32_t q_hi = q_uniform ? q_lo + q_uniform : q_off[b + 1];
    const uint32_t pairs = (q_hi - q_lo) * probe;
    const uint32_t* mine = probe_ids + (uint64_t)q_lo * probe;
    // the sub-buckets that overlap this slab's document range (whole sub-buckets: ids outside the slab are skipped below)
    const uint32_t s_lo = doc0 >> sub_shift;
    uint32_t s_hi = (uint32_t)(((uint64_t)doc0 + here + ((1u << sub_shift) - 1)) >> sub_shift);
    s_hi = s_hi < S ? s_hi : S;
    // first batch of this wave's buckets: lane l takes pair wave + l*WAVES; its bounds are requested before the
    // counters are cleared
    auto bounds = [&](uint32_t p0, uint32_t& lo_l, uint32_t& n_l) {
        const uint32_t myp = p0 + lane * WAVES;
        lo_l = n_l = 0;
        if (myp < pairs) {
            const uint32_t c = mine[myp];
            if (c != 0xFFFFFFFFu) {
                lo_l = sub_off[(size_t)c * S + s_lo];
                n_l = sub_off[(size_t)c * S + s_hi] - lo_l;
            }
        }
    };
    // Histogram of the emitted keys' score fields (bin = count + 1) for the selection that follows.  Nearly every
    // document is hit once: a thread counts those in a register; the workgroup gathers its counts in a small LDS
    // histogram.  segs != nullptr: this workgroup's histogram and the run of the list it writes are stored as they
    // are, hist[b][slab][bins] and segs[b][slab][2] (counts that fit FILTER_HSMALL bins).  Else the occupied bins are added to
    // the query set's histogram hist[b][bins] (a handful of global atomics per workgroup; one per key made this kernel
    // four times slower: they all go to the same few addresses).
    __shared__ uint32_t hsmall[FILTER_HSMALL];
    const bool tallying = hist_bins != 0;
    uint32_t* my_hist = !tallying ? nullptr
                        : segs    ? hist + ((size_t)b * gridDim.x + blockIdx.x) * hist_bins
                                  : hist + (size_t)b * hist_bins;
    uint32_t ones = 0;
    if (tid < FILTER_HSMALL) hsmall[tid] = 0;  // ordered before the first tally by the barriers of the counting phase
    auto tally = [&](uint32_t c) {
        if (!tallying) return;
        if (c == 1) ++ones;
        else if (c + 1 < FILTER_HSMALL) atomicAdd(&hsmall[c + 1], 1u);
        else atomicAdd(&my_hist[c + 1], 1u);  // not with segs: the host gives rows only to histograms that fit hsmall
    };
    auto flush_tally = [&](uint32_t list_start, uint32_t list_len) {  // called by every thread of the workgroup
        if (!tallying) return;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) ones += __shfl_down(ones, o, 64);
        if (lane == 0 && ones) atomicAdd(&hsmall[2], ones);
        __syncthreads();
        if (segs) {
            for (uint32_t i = tid; i < hist_bins; i += T) my_hist[i] = i < FILTER_HSMALL ? hsmall[i] : 0;
            if (tid == 0) {
                uint32_t* sg = segs + ((size_t)b * gridDim.x + blockIdx.x) * 2;
                sg[0] = list_start;
                sg[1] = list_len;
            }
        } else if (tid < FILTER_HSMALL && tid < hist_bins && hsmall[tid]) {
            atomicAdd(&my_hist[tid], hsmall[tid]);
        }
    };
    uint32_t lo_l, n_l;
    bool full = false;   // this wave has seen the queue overflow
    bounds(wave, lo_l, n_l);
    for (uint32_t i = tid; i < words; i += T) cnt[i] = 0;
    if (tid == 0) q_count = 0;
    __syncthreads();
    for (uint32_t p0 = wave; p0 < pairs; p0 += WAVES * 64) {
        if (p0 != wave) bounds(p0, lo_l, n_l);
        // concatenate the ranges: inclusive prefix of the sizes over the lanes
        uint32_t incl = n_l;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            uint32_t y = __shfl_up(incl, o, 64);
            if ((int)lane >= o) incl += y;
        }
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t left = (pairs - p0 + WAVES - 1) / WAVES;
        const uint32_t n_ranges = left < 64 ? left : 64;
        constexpr int U = 8;  // elements per lane per trip
        // Count a trip's ids (0xFFFFFFFF: none) and queue the documents that are hit for the first time: all counter updates are
        // in flight together, and the wave takes its queue slots with one atomic per trip.
        auto count = [&](const uint32_t (&id)[U]) {
            uint32_t old[U], local[U];
            bool hit[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                local[u] = id[u] - doc0;  // wraps to a large value for ids below the slab
                hit[u] = id[u] != 0xFFFFFFFFu && local[u] < here;
                old[u] = hit[u] ? atomicAdd(&cnt[local[u] / PER], 1u << ((local[u] % PER) * BITS)) : 0u;
            }
            if (full) return;   // the counters will be scanned: nothing to queue any more
            uint64_t fm[U];
            uint32_t found = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                fm[u] = __ballot(hit[u] && ((old[u] >> ((local[u] % PER) * BITS)) & MASK) == 0);
                found += (uint32_t)__builtin_popcountll(fm[u]);
            }
            if (found == 0) return;
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&q_count, found);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            full = base + found > FILTER_QUEUE;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t pos = base + (uint32_t)__builtin_popcountll(fm[u] & ((1ull << lane) - 1));
                if (((fm[u] >> lane) & 1) && pos < FILTER_QUEUE) queue[pos] = (QT)local[u];
                base += (uint32_t)__builtin_popcountll(fm[u]);
            }
        };
        // Ranges of 24 and more elements on average (a few thousand documents per bucket): a load takes one range, 64 elements of it at
        // most, and its bounds are wave-uniform; a long range comes back for its rest.  Shorter ranges are read as one concatenated
        // run, where finding an element's range costs some nine operations per range and element.  (128 query sets of 128 probed
        // buckets, 65 elements per bucket and slab: 275 -> 176 us, together with the batched counting; one set of 32: 12.2 -> 9.6 us.)
        if (total >= 24 * n_ranges) {
            uint32_t j = 0, off = 0;   // next range, and what is done of it
            while (j < n_ranges) {
                uint32_t id[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    id[u] = 0xFFFFFFFFu;
                    if (j < n_ranges) {
                        const uint32_t lo_j = (uint32_t)__builtin_amdgcn_readlane((int)lo_l, (int)j);
                        const uint32_t n_j = (uint32_t)__builtin_amdgcn_readlane((int)n_l, (int)j);
                        if (off + lane < n_j) id[u] = bucket_docs[(size_t)lo_j + off + lane];
                        off += 64;
                        if (off >= n_j) {
                            off = 0;
                            ++j;
                        }
                    }
                }
                count(id);
            }
            continue;
        }
        for (uint32_t f0 = 0; f0 < total; f0 += 64 * U) {
            uint32_t id[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // element f of the concatenated run: the range j with excl_j <= f < incl_j
                const uint32_t f = f0 + u * 64 + lane;
                uint32_t addr = 0xFFFFFFFFu;
                if (f < total) {
                    for (uint32_t j = 0; j < n_ranges; ++j) {
                        const uint32_t in_j = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)j);
                        const uint32_t n_j = (uint32_t)__builtin_amdgcn_readlane((int)n_l, (int)j);
                        if (addr == 0xFFFFFFFFu && f < in_j)
                            addr = (uint32_t)__builtin_amdgcn_readlane((int)lo_l, (int)j) + (f - (in_j - n_j));
                    }
                }
                id[u] = addr != 0xFFFFFFFFu ? bucket_docs[addr] : 0xFFFFFFFFu;
            }
            count(id);
        }
    }
    __syncthreads();
    const uint32_t hits = q_count;
    if (hits <= FILTER_QUEUE) {
        if (tid == 0) base_sh = hits ? atomicAdd(&cursor[b], hits) : 0;
        __syncthreads();
        KT* dst = lists + (uint64_t)b * list_stride + base_sh;
        for (uint32_t i = tid; i < hits; i += T) {
            const uint32_t local = queue[i];
            const uint32_t c = (cnt[local / PER] >> ((local % PER) * BITS)) & MASK;
            dst[i] = (KT)make_key((int32_t)c, doc0 + local, id_bits);
            tally(c);
        }
        flush_tally(base_sh, hits);
        return;
    }
    // Queue overflow: scan the counters.  A wave takes 64 consecutive words at a time and its keys leave side by side: one thread walked
    // its words and stored key after key before, a memory request each (128 query sets of 128 probed buckets with 11 000 of a slab's
    // 32 768 documents hit: 177 -> 114 us).
    const uint32_t trips = (words + T - 1) / T;
    auto word_at = [&](uint32_t trip) {
        const uint32_t i = (trip * WAVES + wave) * 64 + lane;
        return i < words ? cnt[i] : 0u;
    };
    uint32_t nz = 0;   // of the thread, then of the wave
    for (uint32_t trip = 0; trip < trips; ++trip) {
        const uint32_t x = word_at(trip);
        if constexpr (W == 4) {
            nz += x != 0;
        } else {   // the top bit of every field that is not zero
            constexpr uint32_t TOP = W == 1 ? 0x80808080u : 0x80008000u;
            nz += (uint32_t)__builtin_popcount((((x & ~TOP) + ~TOP) | x) & TOP);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nz += (uint32_t)__shfl_xor((int)nz, o, 64);
    if (lane == 0) wsum[wave] = nz;
    __syncthreads();
    if (tid == 0) {
        uint32_t total = 0;
        for (int w = 0; w < (int)WAVES; ++w) total += wsum[w];
        base_sh = total ? atomicAdd(&cursor[b], total) : 0;
        q_count = total;
    }
    uint32_t at = 0;
    for (uint32_t w = 0; w < wave; ++w) at += wsum[w];
    __syncthreads();
    KT* dst = lists + (uint64_t)b * list_stride + base_sh;
    for (uint32_t trip = 0; trip < trips; ++trip) {
        const uint32_t x = word_at(trip), i = (trip * WAVES + wave) * 64 + lane;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            const uint32_t c = (x >> (j * BITS % 32)) & MASK;
            const uint64_t some = __ballot(c != 0);
            if (c) {
                dst[at + (uint32_t)__builtin_popcountll(some & ((1ull << lane) - 1))] = (KT)make_key((int32_t)c, doc0 + i * PER + j, id_bits);
                tally(c);
            }
            at += (uint32_t)__builtin_popcountll(some);
        }
    }
    flush_tally(base_sh, q_count);
}

// ---------------------------------------------------------------------------
// k-means for the centroids (Sec. 5 "Filtering": k-means on a sample of the vectors): Lloyd's iteration
// in integers.  The assignment step is the GEMM above; the kernels below are the update step.
// The sample's vectors are first ordered by centroid (a counting sort of their numbers), so that a vector's coordinates are added in
// registers to those of the same centroid's other vectors and only whole runs reach memory.  Without room for the order (a
// workspace of the older, smaller size), and for a few vectors per centroid in a small sample, every coordinate is added to the
// sums by itself.
// Bound: the vectors are read once, whole lines; 524 288 vectors of 128 dimensions, 16 384 centroids: 796 -> 128 us
// for the update's five kernels (67M atomics before, 1.1M now and the two per vector of the sort, at 20 G/s).
// While the vectors are ordered the sums' memory holds the counters, a centroid's at word c << spread (see COUNTER_WORDS).
__global__ __launch_bounds__(256) void kmeans_count_kernel(const uint32_t* __restrict__ assign, uint64_t n, uint32_t spread, uint32_t* counters) {
    const uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) atomicAdd(counters + ((size_t)assign[v] << spread), 1u);
}
// a centroid's counter becomes the start of its run = the sum of the counts before it; the counts are kept (one workgroup)
__global__ __launch_bounds__(1024) void kmeans_starts_kernel(uint32_t* counters, uint32_t K, uint32_t spread, uint32_t* __restrict__ counts) {
    __shared__ uint32_t wsum[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < K; base += 1024 * 16) {
        uint32_t x[16];
        const uint32_t first = base + tid * 16;
        const uint32_t sum = scan_load16(counters, first, K, spread, x);
        uint32_t incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if ((int)lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint32_t all = 0;
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < wave) incl += wsum[w];
            all += wsum[w];
        }
        uint32_t run = carry + incl - sum;
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i)
            if (first + i < K) {
                counters[(size_t)(first + i) << spread] = run;
                counts[first + i] = x[i];
                run += x[i];
            }
        carry += all;
        __syncthreads();
    }
}
__global__ __launch_bounds__(256) void kmeans_order_kernel(const uint32_t* __restrict__ assign, uint64_t n, uint32_t spread,
                                                           uint32_t* counters, uint32_t* __restrict__ order) {
    const uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) order[atomicAdd(counters + ((size_t)assign[v] << spread), 1u)] = (uint32_t)v;
}
// LR = d / 4 lanes take a vector, four coordinates each; a group of LR lanes walks over pieces * LR consecutive
// positions of the order and adds to the sums where the centroid changes.  (More pieces: fewer runs cut in two; fewer: more
// workgroups.  14 000 vectors of 15 000 centroids take 63 us with four pieces, in 14 workgroups, 20 with one.)
template <int LR>
__global__ __launch_bounds__(256) void kmeans_runs_kernel(const int8_t* __restrict__ X, uint64_t n, const uint32_t* __restrict__ assign,
                                                          const uint32_t* __restrict__ order, uint32_t pieces,
                                                          int32_t* __restrict__ sums) {
    constexpr uint32_t D = LR * 4;
    const uint32_t l = threadIdx.x & (LR - 1), group_lane = (threadIdx.x & 63) & ~(LR - 1);
    const uint64_t p0 = ((uint64_t)blockIdx.x * (256 / LR) + threadIdx.x / LR) * (pieces * LR);
    int32_t acc[4] = {0, 0, 0, 0};
    uint32_t at = 0xFFFFFFFFu;   // the run's centroid
    auto flush = [&]() {
        if (at == 0xFFFFFFFFu) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (acc[i]) atomicAdd(sums + (size_t)at * D + 4 * l + i, acc[i]);
            acc[i] = 0;
        }
    };
    for (uint32_t piece = 0; piece < pieces; ++piece) {
        const uint64_t p = p0 + (uint64_t)piece * LR;
        if (!__any(p < n)) break;   // the groups of a wave stay together for the lane exchanges
        const uint32_t have = p >= n ? 0u : n - p < LR ? (uint32_t)(n - p) : (uint32_t)LR;
        const uint32_t my_v = l < have ? order[p + l] : 0u;
        const uint32_t my_c = l < have ? assign[my_v] : 0u;
        constexpr int U = 8;
        for (uint32_t i0 = 0; i0 < LR; i0 += U) {
            uint32_t x[U], c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t v = (uint32_t)__shfl((int)my_v, (int)(group_lane + i0 + u), 64);
                c[u] = (uint32_t)__shfl((int)my_c, (int)(group_lane + i0 + u), 64);
                x[u] = i0 + u < have ? *(const uint32_t*)(X + (size_t)v * D + 4 * l) : 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u >= have) continue;
                if (c[u] != at) {
                    flush();
                    at = c[u];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] += (int32_t)(int8_t)(x[u] >> (8 * i));
            }
        }
    }
    flush();
}
// One thread per (vector, 4 coordinates): sums[c][i] += x[i]; the thread of the first coordinates counts the vector.
__global__ __launch_bounds__(256) void kmeans_accumulate_kernel(const int8_t* __restrict__ X, uint64_t n, uint32_t d,
                                                                const uint32_t* __restrict__ assign,
                                                                int32_t* __restrict__ sums, uint32_t* __restrict__ counts) {
    const uint32_t parts = d / 4;
    const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * parts) return;
    const uint64_t v = idx / parts;
    const uint32_t part = (uint32_t)(idx - v * parts);
    const uint32_t c = assign[v];
    const uint32_t x = *(const uint32_t*)(X + v * d + part * 4);
    int32_t* dst = sums + (size_t)c * d + part * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int32_t xi = (int32_t)(int8_t)(x >> (8 * i));
        if (xi) atomicAdd(dst + i, xi);
    }
    if (part == 0) atomicAdd(counts + c, 1u);
}

// centroid = coordinate-wise mean rounded to the nearest integer, half up: floor((2 sum + n) / (2 n));
// a centroid that received no vector stays
__global__ __launch_bounds__(256) void kmeans_update_kernel(const int32_t* __restrict__ sums,
                                                            const uint32_t* __restrict__ counts, uint32_t K, uint32_t d,
                                                            int8_t* __restrict__ Cn) {
    const uint32_t idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= K * d) return;
    const int64_t cnt = counts[idx / d];
    if (cnt == 0) return;
    const int64_t a = 2 * (int64_t)sums[idx] + cnt, b = 2 * cnt;
    int64_t q = a / b;
    if (a % b != 0 && a < 0) --q;  // floor division
    Cn[idx] = (int8_t)q;
}

hipError_t launch_kmeans_update(const int8_t* X, uint64_t n, uint32_t d, const uint32_t* assign, uint32_t K,
                                int32_t* sums, uint32_t* counts, int8_t* Cn, uint32_t* order, hipStream_t stream) {
    if (d % 4 || K == 0 || (uint64_t)K * d > 0x7fffffffull) return hipErrorInvalidValue;
    const uint64_t cells = (uint64_t)K * d;
    auto zero = [&](void* p, uint64_t words) {
        hipLaunchKernelGGL(filter_zero_kernel, dim3((unsigned)((words + 2047) / 2048)), dim3(256), 0, stream, (int32_t*)p, words);
    };
    // The order's three more launches and its walks over runs pay where runs are long or many: from n = 370 sqrt(K) vectors on, the line
    // at which a round takes the same time either way for K = 1 to 8192 at d = 64, 128 and 256.  (K = 64 to 512, n = 200 to 1500:
    // 20 -> 41 and 25 -> 44 us with the order; K = 32 at d = 128, n = 1500 27 -> 30, n = 3000 39 -> 33, n = 100 000 821 -> 324.)
    const bool ordered = n && order && filter_shape(d) && n * n >= 140000ull * K;
    if (ordered) {
        const uint32_t spread = counter_spread(K);   // K << 4 words fit the sums: d is at least 64
        const dim3 per_vector((unsigned)((n + 255) / 256)), block(256);
        zero(sums, (uint64_t)K << spread);
        hipLaunchKernelGGL(kmeans_count_kernel, per_vector, block, 0, stream, assign, n, spread, (uint32_t*)sums);
        hipLaunchKernelGGL(kmeans_starts_kernel, dim3(1), dim3(1024), 0, stream, (uint32_t*)sums, K, spread, counts);
        hipLaunchKernelGGL(kmeans_order_kernel, per_vector, block, 0, stream, assign, n, spread, (uint32_t*)sums, order);
        zero(sums, cells);
        const uint32_t pieces = n >= (1u << 19) ? 4 : n >= (1u << 17) ? 2 : 1;   // 512 workgroups where there are enough vectors
        const dim3 runs((unsigned)((n + 256 * pieces - 1) / (256 * pieces)));    // a workgroup walks over 256 * pieces positions
        if (d == 64) hipLaunchKernelGGL(kmeans_runs_kernel<16>, runs, block, 0, stream, X, n, assign, order, pieces, sums);
        else if (d == 128) hipLaunchKernelGGL(kmeans_runs_kernel<32>, runs, block, 0, stream, X, n, assign, order, pieces, sums);
        else hipLaunchKernelGGL(kmeans_runs_kernel<64>, runs, block, 0, stream, X, n, assign, order, pieces, sums);
    } else {
        zero(sums, cells);
        zero(counts, K);
    }
    if (n && !ordered) {
        const uint64_t blocks = (n * (d / 4) + 255) / 256;
        if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(kmeans_accumulate_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, X, n, d, assign, sums,
                           counts);
    }
    hipLaunchKernelGGL(kmeans_update_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, stream, sums, counts, K,
                       d, Cn);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
bool filter_supported(uint32_t d) { return filter_shape(d); }
uint32_t filter_tiles(uint32_t K) { return (K + 31) / 32; }
size_t filter_centroid_bytes(uint32_t K, uint32_t d) { return (size_t)filter_tiles(K) * (d / 32) * 1024; }
size_t filter_table_bytes(uint32_t K) { return (size_t)filter_tiles(K) * 32 * 4; }

hipError_t launch_filter_prep(const int8_t* Cn, uint32_t K, uint32_t d, void* Cp, void* T2, hipStream_t stream) {
    if (!filter_shape(d) || K == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(filter_prep_kernel, dim3(1024), dim3(256), 0, stream, Cn, K, d, (int8_t*)Cp, (uint32_t*)T2,
                       filter_tiles(K));
    return hipGetLastError();
}

template <int NT, int MODE>
static hipError_t launch_gemm(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2,
                              uint32_t ranges, uint32_t tiles_per_range, uint32_t* assign, int32_t* out, int64_t* lists,
                              hipStream_t stream, uint32_t zero_words = 0) {
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 4 * 32 * NT - 1) / (4 * 32 * NT);
    if (blocks > 0x7fffffffull || ranges == 0 || ranges > 65535) return hipErrorInvalidValue;
    const uint32_t tiles = filter_tiles(K);
    if ((uint64_t)ranges * tiles_per_range < tiles || (uint64_t)(ranges - 1) * tiles_per_range >= tiles)
        return hipErrorInvalidValue;  // every range must hold at least one tile and together they cover all
    dim3 grid((unsigned)blocks, ranges), block(256);
    if (d == 64)
        hipLaunchKernelGGL((filter_gemm_kernel<2, NT, MODE>), grid, block, 0, stream, X, n, (const v4i*)Cp, (const v4i*)T2, tiles, K, tiles_per_range, assign, out, lists, zero_words, Rest{});
    else if (d == 128)
        hipLaunchKernelGGL((filter_gemm_kernel<4, NT, MODE>), grid, block, 0, stream, X, n, (const v4i*)Cp, (const v4i*)T2, tiles, K, tiles_per_range, assign, out, lists, zero_words, Rest{});
    else if (d == 256)
        hipLaunchKernelGGL((filter_gemm_kernel<8, NT, MODE>), grid, block, 0, stream, X, n, (const v4i*)Cp, (const v4i*)T2, tiles, K, tiles_per_range, assign, out, lists, zero_words, Rest{});
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// up to so many vectors the kernel whose waves split the centroids is the faster one
static uint32_t assign_few_max(uint32_t d) { return d <= 128 ? 160000u : 80000u; }

template <int KS, int NT, int WAVES, bool REST>
static void launch_few(const int8_t* X, uint64_t n, uint32_t K, const void* Cp, const void* T2, uint32_t* assign, Rest rest, hipStream_t stream) {
    const uint64_t most = REST && rest.few < n ? rest.few : n;   // vectors that the launch may have to do
    hipLaunchKernelGGL((filter_assign_few_kernel<KS, NT, WAVES, REST>), dim3((unsigned)((most + 32 * NT - 1) / (32 * NT))), dim3(WAVES * 64), 0, stream, X, n,
                       (const v4i*)Cp, (const v4i*)T2, filter_tiles(K), K, assign, rest);
}

template <int KS>
static hipError_t launch_rest(const int8_t* X, uint64_t n, uint32_t K, const void* Cp, const void* T2, uint32_t* assign, Rest rest, hipStream_t stream) {
    const uint64_t blocks = (n + 511) / 512;
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    launch_few<KS, 2, KS == 8 ? 8 : 16, true>(X, n, K, Cp, T2, assign, rest, stream);
    const uint32_t tiles = filter_tiles(K);
    hipLaunchKernelGGL((filter_gemm_kernel<KS, 4, 0, true>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, (const v4i*)Cp, (const v4i*)T2, tiles, K,
                       tiles, assign, nullptr, nullptr, 0u, rest);
    return hipGetLastError();
}

// Assignment by groups (filter_groups.hip) saves the more the more centroids there are to a group and the more vectors there are to pay
// for the eight launches.  Measured where it helps, vectors around 1024 centres (time of a k-means round against the comparison with
// every centroid, first and later rounds): d = 128, K = 4096, 500 000 vectors 0.94, 1.05; 1.5M 0.66, 0.71; K = 6000, 170 000 0.77, 0.76;
// K = 8192, 170 000 0.67, 0.68; K = 16 384, 500 000 0.37, 0.37, 1.5M 0.26, 0.24; K = 3000, 1.5M 1.14, 1.06.  d = 64 and 256 lie on the same line in
// n * d: 500 000 vectors, K = 6000 0.98, 0.66 and 0.55, 0.53.  Where it does not help, the launches that find
// that out cost the first of eight rounds 32 to 55 us, up to 100 where groups form that vectors lie between, and the others 15: eight rounds of
// 500 000 vectors, d = 128, from all directions K = 16 384 1.014, K = 8192 1.026, mixture of 1024 wide clusters 1.021, 1.041, 64 narrow ones 1.014,
// 1.031; 170 000 vectors, K = 8192 1.05 to 1.07; one round alone 1.03 to 1.09, 170 000 vectors up to 1.2; 600 000 vectors, K = 65 536, one round 1.00 to 1.04.
bool filter_groups_pay_from(uint32_t K) { return K >= 4096; }
bool filter_groups_try(uint64_t n, uint32_t d, uint32_t K) {
    return filter_shape(d) && n > assign_few_max(d) && n <= 0xFFFFFFFFull && filter_groups_pay_from(K) && n >= 8ull * K &&
           (double)n * d * (K - 3300) >= 1e11;
}

hipError_t launch_filter_assign(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2,
                                uint32_t* assign, void* groups, uint32_t* list, uint32_t round, hipStream_t stream) {
    if (groups && list && filter_groups_try(n, d, K)) {
        const hipError_t e = launch_group_assign(X, n, d, K, Cp, T2, groups, assign, list, round, stream);
        if (e != hipSuccess) return e;
        const Rest rest{group_ctl(groups, round), list, 65536};
        if (d == 64) return launch_rest<2>(X, n, K, Cp, T2, assign, rest, stream);
        if (d == 128) return launch_rest<4>(X, n, K, Cp, T2, assign, rest, stream);
        return launch_rest<8>(X, n, K, Cp, T2, assign, rest, stream);
    }
    // measured over n, K = 1024 .. 16 384: at d = 128 and 16 384 centroids 30 000 vectors 211 us per k-means round instead of
    // 455, 120 000 383 instead of 447, 250 000 655 instead of 590; at d = 256 60 000 515 instead of 702, 120 000 832 instead of 699.
    // With many vectors, where the kernel above comes near to filling the chip, it takes centroids enough to keep the waves in work:
    // d = 128, 120 000 vectors, 256 centroids 121 -> 134 us, 1024 116 -> 122, 1536 115 -> 116, 2048 120 -> 118; d = 256, 79 000 vectors, 256
    // 134 -> 149, 1536 117 -> 118, 2048 130 -> 127; d = 64 and fewer vectors are no slower at any K (60 000, d = 128, 256: 114 -> 117).
    const bool many = (d == 128 && n > 65536) || (d == 256 && n > 49152);
    if (n && n <= assign_few_max(d) && (!many || K >= 1536)) {
        const bool wide = n > 32 * 1024 && d <= 128;   // 128 vectors per workgroup where that still gives every CU one
        if (d == 64 && wide) launch_few<2, 4, 8, false>(X, n, K, Cp, T2, assign, Rest{}, stream);
        else if (d == 64) launch_few<2, 2, 16, false>(X, n, K, Cp, T2, assign, Rest{}, stream);
        else if (d == 128 && wide) launch_few<4, 4, 8, false>(X, n, K, Cp, T2, assign, Rest{}, stream);
        else if (d == 128) launch_few<4, 2, 16, false>(X, n, K, Cp, T2, assign, Rest{}, stream);
        else if (d == 256) launch_few<8, 2, 8, false>(X, n, K, Cp, T2, assign, Rest{}, stream);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    return launch_gemm<4, 0>(X, n, d, K, Cp, T2, 1, filter_tiles(K), assign, nullptr, nullptr, stream);
}

hipError_t launch_filter_distances(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2,
                                   int32_t* out, hipStream_t stream) {
    return launch_gemm<2, -1>(X, n, d, K, Cp, T2, 1, filter_tiles(K), nullptr, out, nullptr, stream);
}

// Query side with a small probe count: the centroid tiles are split into ranges so that the few query
// vectors of a batch still fill the chip, and every range keeps its best P = 2^ceil(log2 probe) in registers.
static uint32_t list_width(uint32_t probe) { return probe <= 1 ? 1 : probe <= 2 ? 2 : probe <= 4 ? 4 : 8; }

FilterProbePlan filter_probe_plan(uint64_t n, uint32_t K, uint32_t probe) {
    FilterProbePlan pl{};
    if (probe == 0 || probe > FILTER_LIST_MAX || n == 0) return pl;  // ranges = 0: use the distance matrix
    const uint32_t tiles = filter_tiles(K);
    const uint32_t groups = (tiles + FILTER_RANGE_TILES - 1) / FILTER_RANGE_TILES;
    // more vectors per workgroup halve the centroid bytes staged through LDS per vector
    pl.nt = n >= 4096 ? 2 : 1;
    const uint64_t blocks = (n + 128 * pl.nt - 1) / (128 * pl.nt);
    uint64_t want = (2048 + blocks - 1) / blocks;  // aim at ~2048 workgroups
    if (want > groups) want = groups;
    // a few query vectors alone (one query set): the launch is a chain of global -> LDS stages per workgroup, so more,
    // shorter ranges cut its latency.  With more probes the merge has as many times the entries to read: 65 536 centroids, 256
    // ranges instead of 128 for one set of 32 vectors, d = 128, 2 probes 43.8 -> 41.2 us a filter query, 8 probes 97.9 -> 104.7
    const uint64_t cap = blocks <= 4 ? (probe == 1 ? 512 : 128) : 64;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    const uint32_t per = (groups + (uint32_t)want - 1) / (uint32_t)want;
    pl.tiles_per_range = per * FILTER_RANGE_TILES;
    pl.ranges = (tiles + pl.tiles_per_range - 1) / pl.tiles_per_range;
    pl.width = list_width(probe);
    pl.list_bytes = (size_t)n * pl.ranges * 2 * pl.width * 8;
    return pl;
}

template <int P>
static hipError_t launch_probe_gemm(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2,
                                    const FilterProbePlan& pl, int64_t* lists, hipStream_t stream, uint32_t* zero, uint32_t zero_words) {
    return pl.nt == 2 ? launch_gemm<2, P>(X, n, d, K, Cp, T2, pl.ranges, pl.tiles_per_range, zero, nullptr, lists, stream, zero_words)
                      : launch_gemm<1, P>(X, n, d, K, Cp, T2, pl.ranges, pl.tiles_per_range, zero, nullptr, lists, stream, zero_words);
}

hipError_t launch_filter_probe_lists(const int8_t* X, uint64_t n, uint32_t d, uint32_t K, const void* Cp, const void* T2,
                                     uint32_t probe, const FilterProbePlan& pl, int64_t* lists, uint32_t* probe_ids,
                                     hipStream_t stream, uint32_t* zero, uint32_t zero_words, ProbeMergeArgs* merge) {
    if (merge) *merge = ProbeMergeArgs{};
    if (n == 0) return hipSuccess;
    if (pl.ranges == 0 || probe > K || pl.width != list_width(probe)) return hipErrorInvalidValue;
    const hipError_t e = pl.width == 1   ? launch_probe_gemm<1>(X, n, d, K, Cp, T2, pl, lists, stream, zero, zero_words)
                         : pl.width == 2 ? launch_probe_gemm<2>(X, n, d, K, Cp, T2, pl, lists, stream, zero, zero_words)
                         : pl.width == 4 ? launch_probe_gemm<4>(X, n, d, K, Cp, T2, pl, lists, stream, zero, zero_words)
                                         : launch_probe_gemm<8>(X, n, d, K, Cp, T2, pl, lists, stream, zero, zero_words);
    if (e != hipSuccess) return e;
    const ProbeMergeArgs args{lists, n, pl.ranges * 2 * pl.width, probe, pl.width, probe_ids};
    if (merge) {
        *merge = args;
        return hipSuccess;
    }
    const dim3 mgrid((unsigned)((n + 3) / 4)), mblock(256);
    if (pl.width == 1) hipLaunchKernelGGL(filter_merge_kernel<1>, mgrid, mblock, 0, stream, args);
    else if (pl.width == 2) hipLaunchKernelGGL(filter_merge_kernel<2>, mgrid, mblock, 0, stream, args);
    else if (pl.width == 4) hipLaunchKernelGGL(filter_merge_kernel<4>, mgrid, mblock, 0, stream, args);
    else hipLaunchKernelGGL(filter_merge_kernel<8>, mgrid, mblock, 0, stream, args);
    return hipGetLastError();
}

FilterSubPlan filter_sub_plan(uint64_t n_docs, uint32_t K) {
    // ranges of 32768 documents (the smallest slab of the counting kernel), wider while K*S would pass 2^22 entries
    FilterSubPlan sp{1, 15};
    for (;;) {
        const uint64_t S = n_docs ? ((n_docs - 1) >> sp.sub_shift) + 1 : 1;
        if (S * K <= (1ull << 22) || sp.sub_shift >= 31) {
            sp.S = (uint32_t)S;
            return sp;
        }
        ++sp.sub_shift;
    }
}

size_t filter_cursor_bytes(uint64_t n_sub) { return (size_t)(n_sub << counter_spread(n_sub)) * 4; }

hipError_t launch_filter_buckets(const uint32_t* assign, const uint64_t* doc_off, uint64_t n_docs, uint32_t K,
                                 FilterSubPlan sp, uint32_t* cursor, uint32_t* sub_off, uint32_t* bucket_off,
                                 uint32_t* bucket_docs, hipStream_t stream) {
    uint64_t blocks = (n_docs + 3) / 4;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) blocks = 1;
    const uint64_t KS = (uint64_t)K * sp.S;
    if (KS > 0x7fffffffull) return hipErrorInvalidValue;
    const uint32_t spread = counter_spread(KS);
    uint64_t zb = ((KS << spread) + 255) / 256;
    if (zb > 65536) zb = 65536;
    hipLaunchKernelGGL(filter_zero_kernel, dim3((unsigned)zb), dim3(256), 0, stream, (int32_t*)cursor, KS << spread);
    hipLaunchKernelGGL(filter_bucket_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, assign, doc_off, n_docs,
                       sp.S, sp.sub_shift, spread, cursor, sub_off, bucket_docs);
    launch_filter_scan(cursor, (uint32_t)KS, spread, sub_off, stream);
    hipLaunchKernelGGL(filter_bucket_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, assign, doc_off, n_docs,
                       sp.S, sp.sub_shift, spread, cursor, sub_off, bucket_docs);
    hipLaunchKernelGGL(filter_bucket_starts_kernel, dim3(K / 256 + 1), dim3(256), 0, stream, sub_off, K, sp.S, bucket_off);
    return hipGetLastError();
}

hipError_t launch_filter_probe(const int32_t* dist, uint64_t total_q, uint32_t K, uint32_t probe, uint32_t* probe_ids,
                               hipStream_t stream) {
    if (total_q == 0) return hipSuccess;
    if (total_q > 0x7fffffffull || probe == 0 || probe > K || probe > 1024) return hipErrorInvalidValue;
    uint32_t kpad = 2;
    while (kpad < probe) kpad <<= 1;
    KeyPlan plan = make_key_plan((uint32_t)(2 * FILTER_BIAS), K - 1);
    hipLaunchKernelGGL(filter_probe_kernel, dim3((unsigned)total_q), dim3(256), (size_t)kpad * 8, stream, dist,
                       filter_tiles(K) * 32, K, probe, kpad, plan, probe_ids);
    return hipGetLastError();
}

constexpr uint32_t FILTER_SLAB_BYTES = 128 * 1024;  // most LDS counters one workgroup may hold (the queue takes up to 16 KB more)

template <int W, int T, typename QT, typename KT>
static hipError_t launch_filter_count_t(dim3 grid, size_t lds, hipStream_t stream, const uint32_t* probe_ids, uint32_t probe,
                                        const uint32_t* q_off, uint32_t q_uniform, const uint32_t* sub_off, FilterSubPlan sp,
                                        const uint32_t* bucket_docs, uint64_t n_docs, uint32_t slab_docs, uint32_t id_bits,
                                        uint64_t* lists, uint64_t list_stride, uint32_t* cursor, uint32_t* hist,
                                        uint32_t hist_bins, uint32_t* segs) {
    static hipError_t attr = hipFuncSetAttribute((const void*)filter_count_kernel<W, T, QT, KT>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, FILTER_SLAB_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((filter_count_kernel<W, T, QT, KT>), grid, dim3(T), lds, stream, probe_ids, probe, q_off, q_uniform, sub_off,
                       sp.S, sp.sub_shift, bucket_docs, n_docs, slab_docs, id_bits, (KT*)lists, list_stride, cursor, hist, hist_bins, segs);
    return hipGetLastError();
}

FilterHistPlan filter_hist_plan(uint32_t n_queries, uint32_t max_pairs, uint64_t n_docs, FilterSubPlan sp, bool wide_rows) {
    FilterHistPlan hp{};
    hp.counter_bytes = max_pairs <= 255 ? 1 : max_pairs <= 65535 ? 2 : 4;  // a count is at most the number of probed buckets
    // A slab is one sub-bucket range of documents when its counters fit (32768 documents: 32 KB of LDS with
    // one-byte counters; four workgroups of 512 threads per CU overlap their phases), else as many documents as fit.
    uint64_t slab_docs = 1ull << sp.sub_shift;
    if (slab_docs * hp.counter_bytes > FILTER_SLAB_BYTES) slab_docs = FILTER_SLAB_BYTES / hp.counter_bytes;
    if (slab_docs > n_docs) slab_docs = (n_docs + 3) & ~3ull;
    hp.slab_docs = (uint32_t)slab_docs;
    const uint64_t slabs = slab_docs ? (n_docs + slab_docs - 1) / slab_docs : 0;
    hp.slabs = slabs > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)slabs;
    hp.bins = n_docs ? leading_score_bins(max_pairs, n_docs - 1) : 0;
    // One thread per slab in the selection.  Without rows it makes a pass over the whole list per digit of the id: 128 query sets of
    // 128 probed buckets (counts up to 128, 256 bins of which 130 occur), 180 000 keys each, 70 -> 51 us.  A whole filter query with counts up
    // to 136 .. 254, 300 000 to 700 000 documents: 0.95 of the time on average (22 queries, 0.86 to 1.02), with 30 000 to 100 000 the same.
    hp.rows = hp.bins != 0 && (hp.bins <= 128 || (wide_rows && hp.bins <= 256 && max_pairs + 2 <= FILTER_HSMALL)) && hp.slabs <= 1024;
    hp.hist_off = ((size_t)n_queries + 63) / 64 * 64;
    const size_t hist_words = hp.rows ? (size_t)n_queries * hp.slabs * hp.bins : (size_t)n_queries * hp.bins;
    hp.seg_off = hp.hist_off + hist_words;
    hp.words = hp.seg_off + (hp.rows ? (size_t)n_queries * hp.slabs * 2 : 0);
    return hp;
}

uint64_t filter_count_zero_words(const FilterHistPlan& hp, uint32_t n_queries) { return hp.rows ? n_queries : hp.seg_off; }

hipError_t launch_filter_count(const uint32_t* probe_ids, uint64_t total_q, uint32_t probe, uint32_t max_pairs,
                               const uint32_t* q_off, uint32_t q_uniform, uint32_t n_queries, const uint32_t* sub_off,
                               FilterSubPlan sp, const uint32_t* bucket_docs, uint64_t n_docs, const FilterHistPlan& hp, uint64_t* lists,
                               uint64_t list_stride, uint32_t* cursor, hipStream_t stream, bool zeroed) {
    if (n_queries == 0) return hipSuccess;
    if (n_queries > 65535 || n_docs > 0xFFFFFFFEull) return hipErrorInvalidValue;
    const uint32_t hist_bins = hp.bins;
    uint32_t* hist = hist_bins ? cursor + hp.hist_off : nullptr;
    uint32_t* segs = hp.rows ? cursor + hp.seg_off : nullptr;
    // the list lengths start from zero, and so does a histogram that is added up with atomics (rows are stored)
    const uint64_t zero_words = filter_count_zero_words(hp, n_queries);
    uint64_t zb = (zero_words + 1023) / 1024;
    if (!zeroed)
        hipLaunchKernelGGL(filter_zero_kernel, dim3((unsigned)(zb > 4096 ? 4096 : zb)), dim3(256), 0, stream, (int32_t*)cursor,
                           zero_words);
    if (n_docs == 0 || total_q == 0) return hipGetLastError();
    const uint32_t W = hp.counter_bytes;
    const uint64_t slab_docs = hp.slab_docs;
    const uint64_t slabs = hp.slabs;
    if (slabs > 0x7fffffffull) return hipErrorInvalidValue;
    const size_t lds = (size_t)slab_docs * W;
    const uint32_t id_bits = bits_for(n_docs - 1);
    const dim3 grid((unsigned)slabs, n_queries);
#define DESSERT_COUNT_ARGS grid, lds, stream, probe_ids, probe, q_off, q_uniform, sub_off, sp, bucket_docs, n_docs, \
                           (uint32_t)slab_docs, id_bits, lists, list_stride, cursor, hist, hist_bins, segs
#define DESSERT_COUNT_CASE(W_, T_)                                                                              \
    do {                                                                                                        \
        if (slab_docs <= 65536)                                                                                 \
            return k32 ? launch_filter_count_t<W_, T_, uint16_t, uint32_t>(DESSERT_COUNT_ARGS)                    \
                       : launch_filter_count_t<W_, T_, uint16_t, uint64_t>(DESSERT_COUNT_ARGS);                   \
        return k32 ? launch_filter_count_t<W_, T_, uint32_t, uint32_t>(DESSERT_COUNT_ARGS)                        \
                   : launch_filter_count_t<W_, T_, uint32_t, uint64_t>(DESSERT_COUNT_ARGS);                       \
    } while (0)
    const bool k32 = keys_fit_32(max_pairs, n_docs - 1);  // the lists hold u32 keys then (launch_topk_lists reads them so)
    if (W == 1) DESSERT_COUNT_CASE(1, 512);
    if (W == 2) DESSERT_COUNT_CASE(2, 512);
    DESSERT_COUNT_CASE(4, 512);
#undef DESSERT_COUNT_ARGS
#undef DESSERT_COUNT_CASE
}

}  // namespace dessert
