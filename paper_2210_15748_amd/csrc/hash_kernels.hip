// SRP hashing kernels for gfx950.
//
// A vector's code for table t is C sign bits, bit c = [ r_{t*C+c} . x >= 0 ]
// (Sec. 3: signed random projections; Sec. 5: C hashes concatenated per
// table; Alg. 1 "h = f_t(x_j)", Alg. 2 "h_{t,q} = f_t(q)").  Codes are written
// vector-major, one byte per table: codes[v*L + t].
#include "kernels.hpp"

#include <type_traits>

namespace dessert {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// Seed-derived Rademacher matrix: entry (row, col) = +1 iff the top bit of
// mix64(seed + GOLDEN*(row*d+col+1)) is set (SplitMix64 output function).
__device__ inline uint64_t splitmix_out(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void rademacher_kernel(uint64_t seed, uint64_t total, int8_t* R) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    uint64_t z = splitmix_out(seed + 0x9E3779B97F4A7C15ull * (i + 1));
    R[i] = (z >> 63) ? 1 : -1;
}

hipError_t launch_rademacher(uint64_t seed, uint32_t P, uint32_t d, int8_t* R, hipStream_t stream) {
    uint64_t total = (uint64_t)P * d;
    unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(rademacher_kernel, dim3(blocks), dim3(256), 0, stream, seed, total, R);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Generic kernel: one thread per (vector, table).  int8 x int8 accumulates in
// int32 (exact), everything else in fp32 with fused multiply-add in index
// order.
template <typename XT, typename RT, typename AccT, typename CT>
__global__ __launch_bounds__(256) void hash_scalar_kernel(const XT* __restrict__ X, uint64_t n, uint32_t d,
                                                          const RT* __restrict__ R, uint32_t L, uint32_t C,
                                                          CT* __restrict__ codes) {
    uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * L) return;
    uint64_t v = idx / L;
    uint32_t t = (uint32_t)(idx - v * L);
    const XT* x = X + v * d;
    uint32_t code = 0;
    for (uint32_t c = 0; c < C; ++c) {
        const RT* r = R + (size_t)(t * C + c) * d;
        AccT acc = 0;
        for (uint32_t i = 0; i < d; ++i) {
            if constexpr (std::is_same<AccT, float>::value)
                acc = __builtin_fmaf((float)r[i], (float)x[i], acc);
            else
                acc += (AccT)r[i] * (AccT)x[i];
        }
        code |= (acc >= (AccT)0 ? 1u : 0u) << c;
    }
    codes[idx] = (CT)code;
}

hipError_t launch_hash_scalar(const void* X, uint32_t dtype, uint64_t n, uint32_t d, const void* R, uint32_t proj_kind,
                              uint32_t L, uint32_t C, uint8_t* codes, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    uint64_t total = n * L;
    uint64_t blocks64 = (total + 255) / 256;
    if (blocks64 > 0x7fffffffull) return hipErrorInvalidValue;
    dim3 grid((unsigned)blocks64), block(256);
    if (C < 1 || C > 16) return hipErrorInvalidValue;
#define DESSERT_SCALAR_CASE(XT_, RT_, ACC_)                                                                            \
    do {                                                                                                               \
        if (C <= 8)                                                                                                    \
            hipLaunchKernelGGL((hash_scalar_kernel<XT_, RT_, ACC_, uint8_t>), grid, block, 0, stream, (const XT_*)X, n, \
                               d, (const RT_*)R, L, C, codes);                                                         \
        else                                                                                                           \
            hipLaunchKernelGGL((hash_scalar_kernel<XT_, RT_, ACC_, uint16_t>), grid, block, 0, stream, (const XT_*)X,  \
                               n, d, (const RT_*)R, L, C, (uint16_t*)codes);                                           \
    } while (0)
    if (dtype == 0 && proj_kind == 0)
        DESSERT_SCALAR_CASE(int8_t, int8_t, int32_t);
    else if (dtype == 0 && proj_kind == 1)
        DESSERT_SCALAR_CASE(int8_t, float, float);
    else if (dtype == 1 && proj_kind == 0)
        DESSERT_SCALAR_CASE(_Float16, int8_t, float);
    else
        DESSERT_SCALAR_CASE(_Float16, float, float);
#undef DESSERT_SCALAR_CASE
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// int8 MFMA kernel.  Computes P^T = R * X^T with v_mfma_i32_32x32x32_i8: the M
// dimension runs over projection rows, the N dimension over vectors, so a
// lane's 16 accumulators belong to ONE vector and the sign bits are packed in
// registers without any cross-lane traffic.
//
// Accumulator layout of the 32x32 tile: lane l, register r holds
//   row i = 8*(r/4) + 4*(l/32) + (r%4),   column j = l%32.
// The rows of R are re-ordered (launch_repack_proj_i8) so that within M-tile mt
// register r of lane-half g = l/32 is  table t = g*(L/2) + 2*mt + r/8,  bit r%8.
// Bits c >= C are zero rows and are masked off.  A lane therefore owns L/2
// consecutive code bytes of its vector: lanes 0..31 bytes [0, L/2), lanes
// 32..63 bytes [L/2, L), and the wave's stores cover whole 32*L-byte runs.
//
// Operand layout: lane l supplies row (l%32) of its operand and the 16
// consecutive k-indices 32*ks + 16*(l/32) .. +15; A and B use the same rule,
// so whatever order the instruction walks k in, matching elements meet.
//
// The re-ordered matrix ([LT][KS][64 lanes][16 B], LT = L/4 M-tiles, KS = d/32
// k-steps) is staged in LDS once per workgroup; each wave then loops over
// tiles of 32*NT vectors, reading every A fragment once per NT MFMAs.
//
// WIDE (9 <= C <= 16, 16-bit codes): an M-tile holds 2 tables of 16 bit rows instead of 4 tables of
// 8; register r of lane-half g is bit r of table g*(L/2) + mt, so a lane's 16 accumulators of one
// M-tile make one code.  A code row is LT*4 bytes either way (LT = L/4 M-tiles, or L/2 when WIDE)
// and lane-half g owns the g-th half of it.
// Table groups: with more tables than one launch takes (a code row of more than 64 bytes: L = 128 one-byte codes, L = 64
// 16-bit codes; or a matrix over 64 KB: d = 256 from 32 bytes of code row on) the tables are hashed in groups, one launch
// per group: `codes` then points at the group's first byte of row 0, Rp at the group's matrix, and row_bytes (bytes from
// one vector's codes to the next) is the full row.  The vectors are read once per group.
// RIDERS: the workgroups from hash_blocks on do not hash but carry out riders (hash_riders.hpp), of either kind in instantiations of their own
// (the join holds lists of keys in registers: with both in one kernel 128 dimensions and 16 tables took 128 of them where the grouping needs
// 88, and at 32 tables a launch that carries a grouping of 128 lists of 8192 took 14.5 us instead of 14.1, of 256 lists of 4096 10.2 instead of 9.8);
// a grouping has its bins in the LDS that holds R otherwise.
// Threads per workgroup: a 64 KB matrix lets a CU hold two workgroups, and with four waves each the MFMA, the sign packing
// and the loads of only two waves per SIMD do not overlap enough; eight waves share such a matrix.
constexpr int mfma_threads(int KS, int LT) { return LT * KS * 1024 >= 64 * 1024 ? 512 : 256; }

struct NoRiders {};

constexpr int RIDERS_NONE = 0, RIDERS_LISTS = 1, RIDERS_MERGE = 2;   // none; a grouping and words to clear; a join of probe lists

template <int KS, int LT, int NT, bool WIDE, int RIDERS>
__global__ __launch_bounds__(mfma_threads(KS, LT)) void hash_mfma_i8_kernel(const int8_t* __restrict__ X, uint64_t n,
                                                           const v4i* __restrict__ Rp, uint32_t cmask,
                                                           uint8_t* __restrict__ codes, uint32_t row_bytes,
                                                           uint32_t hash_blocks, std::conditional_t<RIDERS != RIDERS_NONE, HashRiders, NoRiders> riders) {
    constexpr int D = KS * 32;
    constexpr int L = LT * 4;   // bytes per code row
    constexpr int OW = LT / 2;  // output dwords per lane (half a code row)
    constexpr int T = mfma_threads(KS, LT);
    constexpr int WAVES = T / 64;
    extern __shared__ v4i sR[];
    if constexpr (RIDERS == RIDERS_LISTS) {
        if (blockIdx.x >= hash_blocks) {
            __shared__ uint32_t wave_sum[WAVES];
            uint32_t job = blockIdx.x - hash_blocks;
            if (job < riders.order.n_lists) {
                cand_order_body<T>(riders.order, job, reinterpret_cast<uint32_t*>(sR), wave_sum);
                return;
            }
            job -= riders.order.n_lists;
            const uint64_t at = (uint64_t)job * RIDER_ZERO_PER_WG;
            for (uint32_t i = threadIdx.x; i < RIDER_ZERO_PER_WG && at + i < riders.zero_words; i += T) riders.zero[at + i] = 0;
            return;
        }
    } else if constexpr (RIDERS == RIDERS_MERGE) {
        if (blockIdx.x >= hash_blocks) {
            probe_merge_any(riders.merge, (uint64_t)(blockIdx.x - hash_blocks) * WAVES + (threadIdx.x >> 6), threadIdx.x & 63);
            return;
        }
    }
    for (int i = threadIdx.x; i < LT * KS * 64; i += T) sR[i] = Rp[i];
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int col = lane & 31;
    const int g = lane >> 5;
    const uint64_t n_tiles = (n + 32 * NT - 1) / (32 * NT);

    for (uint64_t tile = (uint64_t)blockIdx.x * WAVES + wave; tile < n_tiles; tile += (uint64_t)hash_blocks * WAVES) {
        const uint64_t v0 = tile * (32 * NT);
        v4i b[NT][KS];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint64_t v = v0 + nt * 32 + col;
            if (v >= n) v = n - 1;
            const v4i* src = (const v4i*)(X + v * D + g * 16);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) b[nt][ks] = src[ks * 2];
        }
        uint32_t outw[NT][OW];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int w = 0; w < OW; ++w) outw[nt][w] = 0;

        // One iteration = two M-tiles = one output dword per lane.  The loop is kept rolled so
        // that only one pair of tiles' accumulators is live; finished dwords shift through outw.
#pragma unroll 1
        for (int mp = 0; mp < OW; ++mp) {
            uint32_t word[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) word[nt] = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int mt = mp * 2 + h;
                v16i acc[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[nt][r] = 0;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    v4i a = sR[(mt * KS + ks) * 64 + lane];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[nt][ks], acc[nt], 0, 0, 0);
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    // shift in the sign bits, most significant code bit first: neg = sum_c [p_c < 0] << c
                    if constexpr (!WIDE) {
#pragma unroll
                        for (int s = 0; s < 2; ++s) {
                            uint32_t neg = 0;
#pragma unroll
                            for (int c = 7; c >= 0; --c)
                                neg = __builtin_amdgcn_alignbit(neg, (uint32_t)acc[nt][8 * s + c], 31);
                            uint32_t code = ~neg & cmask;  // bit = [p >= 0]
                            word[nt] |= code << (8 * (2 * h + s));
                        }
                    } else {
                        uint32_t neg = 0;
#pragma unroll
                        for (int c = 15; c >= 0; --c) neg = __builtin_amdgcn_alignbit(neg, (uint32_t)acc[nt][c], 31);
                        uint32_t code = ~neg & cmask;
                        word[nt] |= code << (16 * h);
                    }
                }
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int w = 0; w + 1 < OW; ++w) outw[nt][w] = outw[nt][w + 1];
                outw[nt][OW - 1] = word[nt];
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint64_t v = v0 + nt * 32 + col;
            if (v < n) {
                uint32_t* dst = (uint32_t*)(codes + v * row_bytes + g * (L / 2));
                if constexpr (OW % 4 == 0) {
#pragma unroll
                    for (int w = 0; w < OW; w += 4) {
                        v4i o = {(int)outw[nt][w], (int)outw[nt][w + 1], (int)outw[nt][w + 2], (int)outw[nt][w + 3]};
                        *(v4i*)(dst + w) = o;
                    }
                } else {
#pragma unroll
                    for (int w = 0; w < OW; ++w) dst[w] = outw[nt][w];
                }
            }
        }
    }
}

__global__ void repack_proj_i8_kernel(const int8_t* __restrict__ R, uint32_t d, uint32_t L, uint32_t C,
                                      int8_t* __restrict__ Rp, uint32_t total) {
    uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const uint32_t KS = d / 32;
    uint32_t e = idx & 15;          // byte within the lane's 16
    uint32_t l = (idx >> 4) & 63;   // lane
    uint32_t ks = (idx >> 10) % KS;
    uint32_t mt = (idx >> 10) / KS;
    uint32_t i = l & 31;            // row of the M-tile
    uint32_t kk = ks * 32 + 16 * (l >> 5) + e;
    uint32_t g = (i >> 2) & 1;                // lane half that receives the row
    uint32_t r = 4 * (i >> 3) + (i & 3);      // its accumulator register
    uint32_t t, c;
    if (C <= 8) {  // 4 tables of 8 bit rows
        t = g * (L / 2) + 2 * mt + (r >> 3);
        c = r & 7;
    } else {       // 2 tables of 16 bit rows
        t = g * (L / 2) + mt;
        c = r;
    }
    Rp[idx] = (c < C) ? R[(size_t)(t * C + c) * d + kk] : (int8_t)0;
}

// M-tiles of 32 projection rows: L/4 with one-byte codes, L/2 with 16-bit codes
static uint32_t mfma_tiles(uint32_t L, uint32_t C) { return C <= 8 ? L / 4 : L / 2; }

// shapes of the fp16 kernel (one-byte codes only); L = 128 is hashed as two groups of 64 tables, one launch each
static bool mfma_shape(uint32_t d, uint32_t L) {
    return (d == 64 || d == 128 || d == 256) && (L == 8 || L == 16 || L == 32 || L == 64 || L == 128);
}
static uint32_t f16_group_tables(uint32_t L) { return L < 64 ? L : 64; }

static bool group_supported(uint32_t d, uint32_t Lg, uint32_t C) {
    if (!(d == 64 || d == 128 || d == 256) || C < 1 || C > 16) return false;
    if (!(Lg == 8 || Lg == 16 || Lg == 32 || (Lg == 64 && C <= 8))) return false;
    const uint32_t lt = mfma_tiles(Lg, C);  // 2, 4, 8 or 16
    return (size_t)lt * (d / 32) * 1024 <= 64 * 1024;
}
// Tables per launch: the largest group (at most 64 bytes of code row) whose re-ordered matrix fits 64 KB of LDS;
// 0 if L is not a multiple of a supported group
static uint32_t group_tables(uint32_t d, uint32_t L, uint32_t C) {
    for (uint32_t Lg = 64; Lg >= 8; Lg /= 2)
        if (Lg <= L && L % Lg == 0 && group_supported(d, Lg, C)) return Lg;
    return 0;
}
static size_t group_proj_bytes(uint32_t d, uint32_t Lg, uint32_t C) { return (size_t)mfma_tiles(Lg, C) * (d / 32) * 64 * 16; }

size_t mfma_proj_bytes(uint32_t d, uint32_t L, uint32_t C) {
    if (!hash_mfma_supported(d, L, C)) return 0;
    const uint32_t Lg = group_tables(d, L, C);
    return (L / Lg) * group_proj_bytes(d, Lg, C);
}

// L in {8, 16, 32, 64, 128}, hashed in groups of tables whose matrix fits LDS (one group up to 64 bytes of code row
// at d <= 128)
bool hash_mfma_supported(uint32_t d, uint32_t L, uint32_t C) {
    if (C < 1 || C > 16) return false;
    if (!(L == 8 || L == 16 || L == 32 || L == 64 || L == 128)) return false;
    return group_tables(d, L, C) != 0;
}

hipError_t launch_repack_proj_i8(const int8_t* R, uint32_t d, uint32_t L, uint32_t C, void* Rp, hipStream_t stream) {
    if (!hash_mfma_supported(d, L, C)) return hipErrorInvalidValue;
    const uint32_t Lg = group_tables(d, L, C);
    const uint32_t total = (uint32_t)group_proj_bytes(d, Lg, C);
    for (uint32_t grp = 0; grp < L / Lg; ++grp) {   // group grp = tables grp*Lg .. : rows grp*Lg*C .. of R
        hipLaunchKernelGGL(repack_proj_i8_kernel, dim3((total + 255) / 256), dim3(256), 0, stream,
                           R + (size_t)grp * Lg * C * d, d, Lg, C, (int8_t*)Rp + (size_t)grp * total, total);
    }
    return hipGetLastError();
}

template <int KS, int LT>
static hipError_t launch_mfma_t(const int8_t* X, uint64_t n, uint32_t C, const void* Rp, uint8_t* codes, uint32_t row_bytes,
                                const HashRiders* riders, hipStream_t stream) {
    constexpr int NT = 2;
    constexpr int T = mfma_threads(KS, LT), WAVES = T / 64;
    const uint64_t n_tiles = (n + 32 * NT - 1) / (32 * NT);
    uint64_t blocks = (n_tiles + WAVES - 1) / WAVES;
    // waves loop over tiles; 16384 waves (sixteen workgroups of four per CU, four or five of them resident at a time)
    // measured 3 % faster on 70M vectors than exactly one resident set: the tail of the launch is shorter
    if (blocks > 16384 / WAVES) blocks = 16384 / WAVES;
    size_t lds = (size_t)LT * KS * 64 * 16;
    const uint32_t cmask = (1u << C) - 1u;
    using Kernel = void (*)(const int8_t*, uint64_t, const v4i*, uint32_t, uint8_t*, uint32_t, uint32_t, HashRiders);
    if (riders) {
        const bool merge = riders->merge.lists != nullptr;
        if (merge && (riders->order.n_lists || riders->zero_words)) return hipErrorInvalidValue;   // one kind to a launch
        const uint64_t jobs = merge ? (riders->merge.n + WAVES - 1) / WAVES
                                    : riders->order.n_lists + (riders->zero_words + RIDER_ZERO_PER_WG - 1) / RIDER_ZERO_PER_WG;
        if ((riders->order.n_lists && (size_t)riders->order.ranges * 4 > lds) || blocks + jobs > 0x7fffffffull) return hipErrorInvalidValue;
        const Kernel kern = C <= 8 ? (merge ? hash_mfma_i8_kernel<KS, LT, NT, false, RIDERS_MERGE> : hash_mfma_i8_kernel<KS, LT, NT, false, RIDERS_LISTS>)
                                   : (merge ? hash_mfma_i8_kernel<KS, LT, NT, true, RIDERS_MERGE> : hash_mfma_i8_kernel<KS, LT, NT, true, RIDERS_LISTS>);
        hipLaunchKernelGGL(kern, dim3((unsigned)(blocks + jobs)), dim3(T), lds, stream, X, n, (const v4i*)Rp, cmask, codes, row_bytes, (uint32_t)blocks,
                           *riders);
        return hipGetLastError();
    }
    if (C <= 8)
        hipLaunchKernelGGL((hash_mfma_i8_kernel<KS, LT, NT, false, RIDERS_NONE>), dim3((unsigned)blocks), dim3(T), lds, stream, X,
                           n, (const v4i*)Rp, cmask, codes, row_bytes, (uint32_t)blocks, NoRiders{});
    else
        hipLaunchKernelGGL((hash_mfma_i8_kernel<KS, LT, NT, true, RIDERS_NONE>), dim3((unsigned)blocks), dim3(T), lds, stream, X,
                           n, (const v4i*)Rp, cmask, codes, row_bytes, (uint32_t)blocks, NoRiders{});
    return hipGetLastError();
}

// ranges the fused grouping may use: the bins live in the LDS that holds R in the hashing workgroups
uint32_t hash_mfma_fused_ranges(uint32_t d, uint32_t L, uint32_t C) {
    if (!hash_mfma_supported(d, L, C)) return 0;
    const size_t words = group_proj_bytes(d, group_tables(d, L, C), C) / 4;
    uint32_t r = 1;
    while ((size_t)r * 2 <= words && r < 4096) r *= 2;
    return r;
}

hipError_t launch_hash_mfma_i8(const int8_t* X, uint64_t n, uint32_t d, uint32_t L, uint32_t C, const void* Rp,
                               uint8_t* codes, const HashRiders* riders, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (!hash_mfma_supported(d, L, C)) return hipErrorInvalidValue;
    const uint32_t Lg = group_tables(d, L, C), groups = L / Lg;
    const uint32_t lt = mfma_tiles(Lg, C);
    const uint32_t code_bytes = C <= 8 ? 1 : 2;
    const uint32_t row_bytes = L * code_bytes;
    for (uint32_t grp = 0; grp < groups; ++grp) {
        const void* Rg = (const char*)Rp + (size_t)grp * group_proj_bytes(d, Lg, C);
        uint8_t* cg = codes + (size_t)grp * Lg * code_bytes;
        const HashRiders* rg = grp == 0 ? riders : nullptr;   // they ride in the first launch
        hipError_t e = hipErrorInvalidValue;
#define DESSERT_MFMA_CASE(KS_, LT_) \
    if (d == KS_ * 32 && lt == LT_) e = launch_mfma_t<KS_, LT_>(X, n, C, Rg, cg, row_bytes, rg, stream);
        DESSERT_MFMA_CASE(2, 2)
        DESSERT_MFMA_CASE(2, 4)
        DESSERT_MFMA_CASE(2, 8)
        DESSERT_MFMA_CASE(2, 16)
        DESSERT_MFMA_CASE(4, 2)
        DESSERT_MFMA_CASE(4, 4)
        DESSERT_MFMA_CASE(4, 8)
        DESSERT_MFMA_CASE(4, 16)
        DESSERT_MFMA_CASE(8, 2)
        DESSERT_MFMA_CASE(8, 4)
        DESSERT_MFMA_CASE(8, 8)
#undef DESSERT_MFMA_CASE
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// fp16 vectors x fp32 Gaussian projections on v_mfma_f32_32x32x16_f16.
//
// An fp16 copy of R alone would perturb r.x by about 3e-4*|x| and flip more sign bits than the
// 1e-4 budget allows, so R is split as  R = hi + lo/2048  with hi = fp16(R) and
// lo = fp16((R - hi) * 2048): both parts are normal fp16 numbers, every product is exact in
// fp32, and the two parts accumulate in separate fp32 accumulators that are joined as
// p = accL/2048 + accH.  What is left is fp32 accumulation error (about 1e-6*|x|).
//
// Tiling and sign packing follow the int8 kernel (same accumulator layout, same row order of
// R).  R does not fit LDS here (512 KB at L=64, d=256), so the workgroup stages one M-tile of
// R (hi and lo, 2*d*64 bytes) in LDS at a time; its four waves multiply it with their own
// vectors, which stay in registers for all M-tiles.
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

template <int KS, int LT, int NT, int WV>  // KS = d/16 k-steps, LT = L/4 M-tiles, NT n-tiles of 32 vectors per wave, WV waves per workgroup
__global__ __launch_bounds__(WV * 64, 2) void hash_mfma_f16_kernel(const _Float16* __restrict__ X, uint64_t n,
                                                            const v8h* __restrict__ Rp, uint32_t cmask,
                                                            uint8_t* __restrict__ codes, uint32_t row_bytes) {
    constexpr int D = KS * 16;
    constexpr int L = LT * 4;
    constexpr int OW = LT / 2;
    constexpr int TILE_FRAGS = 2 * KS * 64;  // 16-byte fragments of one M-tile (hi then lo)
    constexpr int T = WV * 64;
    constexpr int FPT = TILE_FRAGS / T;      // fragments each thread moves per tile
    static_assert(TILE_FRAGS % T == 0, "a tile of R divides over the threads");
    // two tiles of R in LDS: while the waves multiply tile mt, the next one is copied from global memory
    // straight into the other buffer (global_load ... lds: no staging registers; a wave's 64 lanes fill
    // 1 KB of consecutive LDS per instruction), one barrier per tile
    __shared__ v8h sA[2][TILE_FRAGS];
    auto copy_tile = [&](int mt, int buf) {
#pragma unroll
        for (int f = 0; f < FPT; ++f) {
            const v8h* src = Rp + (size_t)mt * TILE_FRAGS + threadIdx.x + f * T;
            v8h* dst = &sA[buf][(threadIdx.x & ~63) + f * T];  // wave-uniform; lane i lands 16*i bytes further
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
        }
    };

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int col = lane & 31;
    const int g = lane >> 5;
    const uint64_t block_vecs = WV * 32 * NT;
    const uint64_t n_blocks = (n + block_vecs - 1) / block_vecs;

    for (uint64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
        const uint64_t v0 = blk * block_vecs + (uint64_t)wave * 32 * NT;
        __syncthreads();  // every wave is done with both buffers (previous block of vectors)
        copy_tile(0, 0);
        v8h b[NT][KS];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint64_t v = v0 + nt * 32 + col;
            if (v >= n) v = n - 1;
            const v8h* src = (const v8h*)(X + v * D + g * 8);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) b[nt][ks] = src[ks * 2];
        }
        uint32_t outw[NT][OW];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int w = 0; w < OW; ++w) outw[nt][w] = 0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();

        uint32_t word[NT];
#pragma unroll 1
        for (int mt = 0; mt < LT; ++mt) {
            const int h = mt & 1;
            const v8h* tile = sA[h];
            // the other buffer was last read during tile mt-1, before the barrier that ended it
            if (mt + 1 < LT) copy_tile(mt + 1, h ^ 1);
            if (h == 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) word[nt] = 0;
            }
            v16f accH[NT], accL[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    accH[nt][r] = 0.f;
                    accL[nt][r] = 0.f;
                }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                v8h ah = tile[ks * 64 + lane];
                v8h al = tile[(KS + ks) * 64 + lane];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    accH[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b[nt][ks], accH[nt], 0, 0, 0);
                    accL[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, b[nt][ks], accL[nt], 0, 0, 0);
                }
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    uint32_t neg = 0;
#pragma unroll
                    for (int c = 7; c >= 0; --c) {
                        float p = __builtin_fmaf(accL[nt][8 * s2 + c], 1.0f / 2048.0f, accH[nt][8 * s2 + c]);
                        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(p), 31);  // sign bit: p < 0
                    }
                    uint32_t code = ~neg & cmask;
                    word[nt] |= code << (8 * (2 * h + s2));
                }
            if (h == 1) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int w = 0; w + 1 < OW; ++w) outw[nt][w] = outw[nt][w + 1];
                    outw[nt][OW - 1] = word[nt];
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of tile mt+1 has landed
            __syncthreads();  // tile mt+1 is in place, and nobody reads tile mt any more
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint64_t v = v0 + nt * 32 + col;
            if (v < n) {
                uint32_t* dst = (uint32_t*)(codes + v * row_bytes + g * (L / 2));
#pragma unroll
                for (int w = 0; w < OW; ++w) dst[w] = outw[nt][w];
            }
        }
    }
}

// Rp layout: [LT M-tiles][2 parts: hi, lo][KS k-steps][64 lanes][8 halves]
__global__ void repack_proj_f16_kernel(const float* __restrict__ R, uint32_t d, uint32_t L, uint32_t C,
                                       _Float16* __restrict__ Rp, uint32_t total) {
    uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const uint32_t KS = d / 16;
    uint32_t e = idx & 7;
    uint32_t l = (idx >> 3) & 63;
    uint32_t rest = idx >> 9;
    uint32_t ks = rest % KS;
    uint32_t part = (rest / KS) & 1;
    uint32_t mt = rest / (2 * KS);
    uint32_t i = l & 31;
    uint32_t kk = ks * 16 + 8 * (l >> 5) + e;
    uint32_t g = (i >> 2) & 1;
    uint32_t s = i >> 4;
    uint32_t c = 4 * ((i >> 3) & 1) + (i & 3);
    uint32_t t = g * (L / 2) + 2 * mt + s;
    float r = (c < C) ? R[(size_t)(t * C + c) * d + kk] : 0.f;
    _Float16 hi = (_Float16)r;
    _Float16 lo = (_Float16)((r - (float)hi) * 2048.0f);
    Rp[idx] = part ? lo : hi;
}

size_t mfma_f16_proj_bytes(uint32_t d, uint32_t L) {
    if (!mfma_shape(d, L)) return 0;
    return (size_t)(L / 4) * 2 * (d / 16) * 64 * 16;  // the groups' matrices one after the other
}

bool hash_mfma_f16_supported(uint32_t d, uint32_t L, uint32_t C) { return mfma_shape(d, L) && C >= 1 && C <= 8; }

hipError_t launch_repack_proj_f16(const float* R, uint32_t d, uint32_t L, uint32_t C, void* Rp, hipStream_t stream) {
    if (!mfma_shape(d, L)) return hipErrorInvalidValue;
    const uint32_t Lg = f16_group_tables(L);
    const uint32_t total = (uint32_t)(mfma_f16_proj_bytes(d, Lg) / 2);  // halves per group
    for (uint32_t grp = 0; grp < L / Lg; ++grp)
        hipLaunchKernelGGL(repack_proj_f16_kernel, dim3((total + 255) / 256), dim3(256), 0, stream,
                           R + (size_t)grp * Lg * C * d, d, Lg, C, (_Float16*)Rp + (size_t)grp * total, total);
    return hipGetLastError();
}

template <int KS, int LT>
static hipError_t launch_mfma_f16_t(const void* X, uint64_t n, uint32_t C, const void* Rp, uint8_t* codes,
                                    uint32_t row_bytes, hipStream_t stream) {
    constexpr int NT = 2;
    // eight waves share each staged tile of R when a tile is large (d = 256: 32 KB), four otherwise
    constexpr int WV = KS >= 16 ? 8 : 4;
    const uint64_t block_vecs = WV * 32 * NT;
    uint64_t blocks = (n + block_vecs - 1) / block_vecs;
    const uint64_t persistent = 256 * (8 / WV);  // 256 CUs x 8 waves
    if (blocks > persistent) blocks = persistent;
    auto kern = hash_mfma_f16_kernel<KS, LT, NT, WV>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(WV * 64), 0, stream, (const _Float16*)X, n, (const v8h*)Rp,
                       (1u << C) - 1u, codes, row_bytes);
    return hipGetLastError();
}

hipError_t launch_hash_mfma_f16(const void* X, uint64_t n, uint32_t d, uint32_t L, uint32_t C, const void* Rp,
                                uint8_t* codes, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (!hash_mfma_f16_supported(d, L, C)) return hipErrorInvalidValue;
    const uint32_t Lg = f16_group_tables(L);
    for (uint32_t grp = 0; grp < L / Lg; ++grp) {
        const void* Rg = (const char*)Rp + (size_t)grp * mfma_f16_proj_bytes(d, Lg);
        uint8_t* cg = codes + (size_t)grp * Lg;
        hipError_t e = hipErrorInvalidValue;
#define DESSERT_MFMA_F16_CASE(KS_, LT_) \
    if (d == KS_ * 16 && Lg == LT_ * 4) e = launch_mfma_f16_t<KS_, LT_>(X, n, C, Rg, cg, L, stream);
        DESSERT_MFMA_F16_CASE(4, 2)
        DESSERT_MFMA_F16_CASE(4, 4)
        DESSERT_MFMA_F16_CASE(4, 8)
        DESSERT_MFMA_F16_CASE(4, 16)
        DESSERT_MFMA_F16_CASE(8, 2)
        DESSERT_MFMA_F16_CASE(8, 4)
        DESSERT_MFMA_F16_CASE(8, 8)
        DESSERT_MFMA_F16_CASE(8, 16)
        DESSERT_MFMA_F16_CASE(16, 2)
        DESSERT_MFMA_F16_CASE(16, 4)
        DESSERT_MFMA_F16_CASE(16, 8)
        DESSERT_MFMA_F16_CASE(16, 16)
#undef DESSERT_MFMA_F16_CASE
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Hashing on the matrix cores for every other shape: any dimension from one k-step up to HASH_ANY_KS k-steps, any number
// of tables, up to 16 bits per table, all four pairings of vector and projection type.
//
// Same product and lane layout as above (M = projection rows, N = vectors, a lane's 16 accumulators belong to one vector),
// with three differences that make the shape a run-time value:
//  - Bits are packed without padding: lane half g owns the tables [g*La, ...) of its vector and their bits are one stream, 16
//    to an M-tile, cut into codes as they leave.  (A table of 11 bits takes 11 rows, not 16.)  The stream starts anew every
//    16 tables of a half (a "segment": C tiles), so that a launch with few vectors can give the segments to different
//    workgroups.
//  - The k-steps of a row are whole 16-byte fragments at any byte offset; the last one, if d is no multiple of a k-step, is
//    the window that ends at the row's end, with the elements that the step before has covered set to zero.  So every
//    load stays inside its row, whatever d is.
//  - A fragment loop is unrolled KS times with a uniform exit at the shape's own ks_n.
// fp16 arithmetic (everything but int8 x +-1): each row of R is first scaled by a power of two that brings its largest entry
// to [2^14, 2^15) (a sign does not change), then split in hi + lo/4096 (PARTS = 2; +-1 entries are exact in one part).  At that
// scale both parts of an entry are normal fp16 numbers down to 2^-28 of the row's largest, and the two hold it to 2^-23 of
// itself; below that it is off by up to 2^-51 of the row's largest.  Vectors may be zero wherever a row is large, so a matrix
// with an entry that is off by more than 2^-22 of itself stays with the plain kernel (the repacking reports it; of
// Gaussian matrices with 786 432 entries one in several hundred has such an entry).
// A projection that is not a number gives bit 0, as the comparison p >= 0 does, and an infinite element decides its
// sign alone: hi is never 0 for an entry that is not, and the lo part is clamped to finite values before it joins.
//
// All of R stays in LDS when it fits ANY_RESIDENT bytes (two workgroups to a CU); else one tile is multiplied while the next
// arrives.  Bound: HBM for a few tables, the matrix cores for many.  1.02M fp16 vectors of 200 dimensions, L = 8, C = 11:
// 17.2 ms on the plain kernel (2.1 TFLOP/s of the method's), 0.130 ms here (3.3 TB/s of 4.8 that a copy reaches).  Against 64-bit
// projections 2 of 88M bits differ here, 4 on the plain kernel (its fp32 sum is one chain of d additions).
// The fixed-shape kernels above stay where they exist: int8 2M vectors of 128 dimensions, L = 32, C = 7 take 0.071 ms there and
// 0.113 ms here; fp16 1M of 256, L = 64, C = 8 0.467 and 0.522 ms.
constexpr uint32_t HASH_ANY_SEG = 16;            // tables of a lane half per segment
constexpr size_t ANY_RESIDENT = 80 * 1024;
constexpr int ANY_ROW_EXP = 14;                  // of a scaled row's largest entry; 2^15 * 65504 * 384 is far inside fp32
constexpr float ANY_LO_SCALE = 4096.0f;          // hi is off by 2^3 at most: lo stays below 2^15

struct HashAnyShape {
    uint32_t d, L, C;
    uint32_t La;          // tables of lane half 0 (half 1 has the other L - La <= La)
    uint32_t ks;          // k-steps of a row
    uint32_t segs, tiles; // segments, and M-tiles in all
};

template <bool F16>
struct AnyAcc { typedef v16i type; };
template <>
struct AnyAcc<true> { typedef v16f type; };

// XT: element type of the vectors; F16: fp16 arithmetic (else int8); KS >= shape.ks; NT n-tiles of 32 vectors per wave
template <typename XT, bool F16, int PARTS, int KS, int NT>
__global__ __launch_bounds__(256, 2) void hash_mfma_any_kernel(const XT* __restrict__ X, uint64_t n, HashAnyShape sh,
                                                               const v4i* __restrict__ Rp, uint8_t* __restrict__ codes,
                                                               uint32_t seg_first_step, uint32_t resident) {
    constexpr int E = F16 ? 8 : 16;          // elements of a lane's fragment
    constexpr int XB = E * (int)sizeof(XT);  // their bytes in memory (8 for int8 vectors in fp16 arithmetic)
    typedef typename AnyAcc<F16>::type Acc;
    extern __shared__ v4i sR[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, g = lane >> 5;
    const uint32_t frags = PARTS * sh.ks;    // of 64 lanes each, per tile
    const uint32_t cw = sh.C <= 8 ? 1 : 2, row_bytes = sh.L * cw;
    const uint32_t cmask = (1u << sh.C) - 1u;
    const uint32_t full = sh.d / (2 * E);    // whole k-steps
    const uint32_t mine = g ? sh.L - sh.La : sh.La;   // tables of this lane half

    auto copy_tile = [&](uint32_t tile, uint32_t slot) {  // whole waves; lane i lands 16*i bytes further
        for (uint32_t f = (uint32_t)wave; f < frags; f += 4)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Rp + ((size_t)tile * frags + f) * 64 + lane),
                                             (__attribute__((address_space(3))) void*)&sR[((size_t)slot * frags + f) * 64], 16, 0, 0);
    };
    // elements of the last, overlapping window that the whole k-steps have not covered
    const int tail_base = (int)sh.d - 2 * E + g * E - (int)(full * 2 * E);   // window element e is new if tail_base + e >= 0
    const bool has_tail = full * 2 * E != sh.d;

    // grid.y > 1: segments are dealt round-robin (seg_first_step = grid.y), else this workgroup does all of them
    const uint32_t seg0 = seg_first_step ? blockIdx.y : 0, seg_step = seg_first_step ? seg_first_step : 1;
    if (resident) {
        for (uint32_t t = 0; t < sh.tiles; ++t) copy_tile(t, t);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    const uint64_t block_vecs = 4 * 32 * NT;
    const uint64_t n_blocks = (n + block_vecs - 1) / block_vecs;
    for (uint64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
        const uint64_t v0 = blk * block_vecs + (uint64_t)wave * 32 * NT;
        uint32_t slot = 0;
        if (!resident) {
            __syncthreads();   // every wave is done with both buffers
            copy_tile(seg0 * sh.C, 0);
        }
        v4i b[NT][KS];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint64_t v = v0 + nt * 32 + col;
            if (v >= n) v = n - 1;
            const XT* row = X + v * sh.d + g * E;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint32_t at = (uint32_t)ks < full ? ks * 2 * E : sh.d - 2 * E;   // uniform, inside the row
                XT raw[E];
                __builtin_memcpy(raw, row + at, XB);
                if constexpr (F16 && sizeof(XT) == 1) {
                    v8h h;
#pragma unroll
                    for (int e = 0; e < 8; ++e) h[e] = (_Float16)(short)raw[e];
                    __builtin_memcpy(&b[nt][ks], &h, 16);
                } else {
                    __builtin_memcpy(&b[nt][ks], raw, 16);
                }
            }
            if (has_tail) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if ((uint32_t)ks == full) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            uint32_t keep = 0;
#pragma unroll
                            for (int e = 0; e < E / 4; ++e)
                                if (tail_base + w * (E / 4) + e >= 0) keep |= (E == 16 ? 0xFFu : 0xFFFFu) << (e * (E == 16 ? 8 : 16));
                            b[nt][ks][w] &= (int)keep;
                        }
                    }
            }
        }
        for (uint32_t seg = seg0; seg < sh.segs; seg += seg_step) {
            const uint32_t seg_tables = sh.La - seg * HASH_ANY_SEG < HASH_ANY_SEG ? sh.La - seg * HASH_ANY_SEG : HASH_ANY_SEG;
            const uint32_t tile0 = seg * sh.C;
            const uint32_t seg_tiles = (seg_tables * sh.C + 15) / 16;
            uint32_t buf[NT], word[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) buf[nt] = word[nt] = 0;
            uint32_t nbits = 0, pos = 0, done = 0;   // bits waiting in buf, bit position in word, codes cut off so far
            for (uint32_t t = 0; t < seg_tiles; ++t) {
                const v4i* tile = sR + (size_t)(resident ? tile0 + t : slot) * frags * 64;
                if (!resident) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the tile has landed
                    __syncthreads();                                    // everyone's has, and nobody reads the other buffer any more
                    const bool more = t + 1 < seg_tiles;
                    if (more || seg + seg_step < sh.segs) copy_tile(more ? tile0 + t + 1 : (seg + seg_step) * sh.C, slot ^ 1);
                    slot ^= 1;
                }
                Acc acc[PARTS][NT];
#pragma unroll
                for (int p = 0; p < PARTS; ++p)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[p][nt][r] = 0;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    if ((uint32_t)ks < sh.ks) {
#pragma unroll
                        for (int p = 0; p < PARTS; ++p) {
                            const v4i a = tile[((uint32_t)p * sh.ks + ks) * 64 + lane];
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) {
                                if constexpr (F16)
                                    acc[p][nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a),
                                                                                       __builtin_bit_cast(v8h, b[nt][ks]), acc[p][nt], 0, 0, 0);
                                else
                                    acc[p][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[nt][ks], acc[p][nt], 0, 0, 0);
                            }
                        }
                    }
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    uint32_t neg = 0;
#pragma unroll
                    for (int r = 15; r >= 0; --r) {
                        uint32_t bits;
                        if constexpr (F16) {
                            float p = acc[0][nt][r];
                            if constexpr (PARTS == 2)
                                p = __builtin_fmaf(__builtin_amdgcn_fmed3f(acc[PARTS - 1][nt][r], -1e30f, 1e30f), 1.0f / ANY_LO_SCALE, p);
                            bits = __float_as_uint(__builtin_fmaxf(p, -1.0f));   // not a number: negative
                        } else {
                            bits = (uint32_t)acc[0][nt][r];
                        }
                        neg = __builtin_amdgcn_alignbit(neg, bits, 31);
                    }
                    buf[nt] |= (~neg & 0xFFFFu) << nbits;   // fewer than C <= 16 bits were waiting
                }
                nbits += 16;
                while (nbits >= sh.C && done < seg_tables) {   // the same for the whole grid
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        word[nt] |= (buf[nt] & cmask) << pos;
                        buf[nt] >>= sh.C;
                    }
                    nbits -= sh.C;
                    pos += 8 * cw;
                    ++done;
                    if (pos == 32) {   // tables are owned in whole dwords of codes
                        const uint32_t first = seg * HASH_ANY_SEG + done - 4 / cw;   // the dword's first table in this half
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const uint64_t v = v0 + nt * 32 + col;
                            if (v < n && first < mine)
                                *(uint32_t*)(codes + v * row_bytes + ((g ? sh.La : 0u) + first) * cw) = word[nt];
                            word[nt] = 0;
                        }
                        pos = 0;
                    }
                }
            }
        }
    }
}

// Re-ordered matrix: [tiles][PARTS][ks][64 lanes][16 bytes].  One workgroup per tile: the scale of each of its 32 rows first.
// *lost (PARTS = 2) becomes 1 if an entry is off by more than 2^-22 of itself.
template <typename RT, bool F16, int PARTS>
__global__ __launch_bounds__(256) void repack_proj_any_kernel(const RT* __restrict__ R, HashAnyShape sh, void* __restrict__ Rp,
                                                              uint32_t* __restrict__ lost) {
    constexpr uint32_t E = F16 ? 8 : 16;
    __shared__ int scale[32];         // exponent
    __shared__ uint32_t row_of[32];   // row of R, all ones: no such table
    const uint32_t tile = blockIdx.x, seg = tile / sh.C, tid = threadIdx.x;
    if (tid < 32) {
        const uint32_t i = tid, g = (i >> 2) & 1, r = 4 * (i >> 3) + (i & 3);   // accumulator r of lane half g
        const uint32_t bit = (tile - seg * sh.C) * 16 + r;                     // of the segment's stream
        const uint32_t j = seg * HASH_ANY_SEG + bit / sh.C, c = bit % sh.C;
        const bool have = bit / sh.C < HASH_ANY_SEG && j < (g ? sh.L - sh.La : sh.La);
        const uint32_t row = have ? ((g ? sh.La : 0u) + j) * sh.C + c : 0xFFFFFFFFu;
        row_of[i] = row;
        int s = 0;
        if constexpr (F16) {
            float top = 0.0f;
            if (have)
                for (uint32_t k = 0; k < sh.d; ++k) {
                    const float a = __builtin_fabsf((float)R[(size_t)row * sh.d + k]);
                    if (a < __builtin_inff() && a > top) top = a;
                }
            if (top > 0.0f) s = ANY_ROW_EXP - ilogbf(top);
        }
        scale[i] = s;
    }
    __syncthreads();
    const uint32_t total = PARTS * sh.ks * 64 * E;
    for (uint32_t idx = tid; idx < total; idx += 256) {
        const uint32_t e = idx % E, l = (idx / E) & 63, ks = (idx / E / 64) % sh.ks, part = idx / E / 64 / sh.ks;
        const uint32_t row = row_of[l & 31];
        // element of the row: whole k-steps, then the window that ends at d, whose covered elements count nothing
        const uint32_t full = sh.d / (2 * E), in = (l >> 5) * E + e;
        const uint32_t k = ks < full ? ks * 2 * E + in : sh.d - 2 * E + in;
        const bool have = row != 0xFFFFFFFFu && (ks < full || k >= full * 2 * E);
        if constexpr (F16) {
            const float entry = have ? (float)R[(size_t)row * sh.d + k] : 0.0f;
            const float x = ldexpf(entry, scale[l & 31]);
            _Float16 hi = (_Float16)x;
            if ((float)hi == 0.0f && entry != 0.0f) hi = (_Float16)(entry > 0.0f ? 0x1p-24f : -0x1p-24f);
            const float rest = (x - (float)hi) * ANY_LO_SCALE;
            const _Float16 lo = (rest - rest == 0.0f) ? (_Float16)rest : (_Float16)0.0f;   // an entry that is not finite: hi alone
            if constexpr (PARTS == 2) {
                const double exact = ldexp((double)entry, scale[l & 31]), off = ((double)(float)hi + (double)(float)lo / ANY_LO_SCALE) - exact;
                if (fabs(off) > fabs(exact) * 0x1p-22) *lost = 1;   // (not for infinities: off is not a number or 0)
            }
            ((_Float16*)Rp)[(size_t)tile * total + idx] = part ? lo : hi;
        } else {
            ((int8_t*)Rp)[(size_t)tile * total + idx] = have ? (int8_t)R[(size_t)row * sh.d + k] : (int8_t)0;
        }
    }
}

// dtype / proj_kind as in dessert.h (0: int8 / +-1, 1: fp16 / Gaussian)
static bool any_is_f16(uint32_t dtype, uint32_t proj_kind) { return dtype != 0 || proj_kind != 0; }
static uint32_t any_parts(uint32_t proj_kind) { return proj_kind == 0 ? 1 : 2; }
static HashAnyShape any_shape(uint32_t dtype, uint32_t d, uint32_t L, uint32_t C, uint32_t proj_kind) {
    HashAnyShape s{};
    const uint32_t kstep = any_is_f16(dtype, proj_kind) ? 16 : 32;
    s.d = d; s.L = L; s.C = C;
    s.La = C <= 8 ? 4 * ((L + 7) / 8) : L / 2;   // whole dwords of codes: 4 one-byte codes, 2 of 16 bits
    s.ks = (d + kstep - 1) / kstep;
    s.segs = (s.La + HASH_ANY_SEG - 1) / HASH_ANY_SEG;
    s.tiles = (s.segs - 1) * C + ((s.La - (s.segs - 1) * HASH_ANY_SEG) * C + 15) / 16;   // a full segment: C tiles
    return s;
}

bool hash_any_supported(uint32_t dtype, uint32_t proj_kind, uint32_t d, uint32_t L, uint32_t C) {
    const uint32_t kstep = any_is_f16(dtype, proj_kind) ? 16 : 32;
    return d >= kstep && d <= HASH_ANY_MAX_D && L >= 4 && L % 4 == 0 && L <= 128 && C >= 1 && C <= 16;
}

size_t hash_any_proj_bytes(uint32_t dtype, uint32_t proj_kind, uint32_t d, uint32_t L, uint32_t C) {
    const HashAnyShape s = any_shape(dtype, d, L, C, proj_kind);
    return (size_t)s.tiles * any_parts(proj_kind) * s.ks * 1024;
}

bool hash_any_rounds(uint32_t proj_kind) { return any_parts(proj_kind) == 2; }

hipError_t launch_repack_proj_any(const void* R, uint32_t dtype, uint32_t proj_kind, uint32_t d, uint32_t L, uint32_t C, void* Rp,
                                  uint32_t* lost, hipStream_t stream) {
    if (!hash_any_supported(dtype, proj_kind, d, L, C) || (hash_any_rounds(proj_kind) && !lost)) return hipErrorInvalidValue;
    const HashAnyShape s = any_shape(dtype, d, L, C, proj_kind);
    const dim3 grid(s.tiles), block(256);
    if (!any_is_f16(dtype, proj_kind))
        hipLaunchKernelGGL((repack_proj_any_kernel<int8_t, false, 1>), grid, block, 0, stream, (const int8_t*)R, s, Rp, lost);
    else if (proj_kind == 0)
        hipLaunchKernelGGL((repack_proj_any_kernel<int8_t, true, 1>), grid, block, 0, stream, (const int8_t*)R, s, Rp, lost);
    else
        hipLaunchKernelGGL((repack_proj_any_kernel<float, true, 2>), grid, block, 0, stream, (const float*)R, s, Rp, lost);
    return hipGetLastError();
}

template <typename XT, bool F16, int PARTS, int KS, int NT>
static hipError_t launch_any_t(const void* X, uint64_t n, const HashAnyShape& s, const void* Rp, uint8_t* codes, hipStream_t stream) {
    auto kern = hash_mfma_any_kernel<XT, F16, PARTS, KS, NT>;
    static hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * 2 * KS * 1024 > (int)ANY_RESIDENT ? 2 * 2 * KS * 1024 : (int)ANY_RESIDENT);
    if (attr != hipSuccess) return attr;
    const size_t tile_bytes = (size_t)PARTS * s.ks * 1024, all = tile_bytes * s.tiles;
    const uint64_t block_vecs = 4 * 32 * NT;
    uint64_t blocks = (n + block_vecs - 1) / block_vecs;
    // few vectors: the segments go to different workgroups (a workgroup then walks over C tiles instead of all)
    const uint32_t gy = (s.segs > 1 && blocks < 256) ? s.segs : 1;
    const bool resident = gy == 1 && all <= ANY_RESIDENT && blocks > 512;   // short runs would wait for tiles they use once
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks, gy), dim3(256), resident ? all : 2 * tile_bytes, stream, (const XT*)X, n, s,
                       (const v4i*)Rp, codes, gy > 1 ? gy : 0u, resident ? 1u : 0u);
    return hipGetLastError();
}

template <typename XT, bool F16, int PARTS>
static hipError_t launch_any_ks(const void* X, uint64_t n, const HashAnyShape& s, const void* Rp, uint8_t* codes, hipStream_t stream) {
    // two n-tiles per wave while their fragments leave room for the accumulators of two waves per SIMD; one when two would
    // leave CUs without a workgroup (a workgroup's walk over the tiles of R is the latency of a small launch: searches
    // of 4 sets of 20 vectors, L = 24, 32.9 -> 29.8 us; 10 800 fp16 vectors of 200 dimensions, L = 48, C = 10 37.9 -> 36.6).
    // The steps of KS are where the registers of the unused fragments cost most: 13 instead of 16 for up to 208 (fp16) or 416 (int8)
    // dimensions saves 1 to 12 % (1M fp16 vectors of 200 dimensions x +-1, L = 8, C = 11: 112 us against 126); 16 and 24 serve what is left.
    if (n * s.segs <= 256 * 256) {
        if (s.ks <= 4) return launch_any_t<XT, F16, PARTS, 4, 1>(X, n, s, Rp, codes, stream);
        if (s.ks <= 8) return launch_any_t<XT, F16, PARTS, 8, 1>(X, n, s, Rp, codes, stream);
        if (s.ks <= 13) return launch_any_t<XT, F16, PARTS, 13, 1>(X, n, s, Rp, codes, stream);
    }
    if (s.ks <= 4) return launch_any_t<XT, F16, PARTS, 4, 2>(X, n, s, Rp, codes, stream);
    if (s.ks <= 8) return launch_any_t<XT, F16, PARTS, 8, 2>(X, n, s, Rp, codes, stream);
    if constexpr (F16) {
        if (s.ks <= 13) return launch_any_t<XT, F16, PARTS, 13, 2>(X, n, s, Rp, codes, stream);
        if (s.ks <= 16) return launch_any_t<XT, F16, PARTS, 16, 2>(X, n, s, Rp, codes, stream);
        if (s.ks <= 24) return launch_any_t<XT, F16, PARTS, 24, 1>(X, n, s, Rp, codes, stream);
    } else {
        if (s.ks <= 12) return launch_any_t<XT, F16, PARTS, 12, 2>(X, n, s, Rp, codes, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_hash_any(const void* X, uint32_t dtype, uint32_t proj_kind, uint64_t n, uint32_t d, uint32_t L, uint32_t C,
                           const void* Rp, uint8_t* codes, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (!hash_any_supported(dtype, proj_kind, d, L, C) || (uintptr_t)codes % 4) return hipErrorInvalidValue;
    const HashAnyShape s = any_shape(dtype, d, L, C, proj_kind);
    if (dtype == 0)
        return proj_kind == 0 ? launch_any_ks<int8_t, false, 1>(X, n, s, Rp, codes, stream)
                              : launch_any_ks<int8_t, true, 2>(X, n, s, Rp, codes, stream);
    return proj_kind == 0 ? launch_any_ks<_Float16, true, 1>(X, n, s, Rp, codes, stream)
                          : launch_any_ks<_Float16, true, 2>(X, n, s, Rp, codes, stream);
}

// ---------------------------------------------------------------------------
// Plain streaming read (measurement aid): what HBM delivers to a kernel that does nothing but
// read, for comparison with the 8 TB/s nameplate and with the scoring kernel's rate.
__global__ __launch_bounds__(256) void read_probe_kernel(const v4i* __restrict__ p, size_t n16, int* sink) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    v4i acc = {0, 0, 0, 0};
    for (; i + 3 * stride < n16; i += 4 * stride) {
        v4i a = p[i], b = p[i + stride], c = p[i + 2 * stride], d = p[i + 3 * stride];
        acc += a; acc += b; acc += c; acc += d;
    }
    for (; i < n16; i += stride) acc += p[i];
    // a store that practically never happens keeps the loads alive
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x5ee1c0de && sink) *sink = 1;
}

// The traffic of index building with the arithmetic taken out: every thread reads 64 bytes and writes 16 (the 4 : 1
// read : write mix of d = 128 bytes in, L = 32 bytes out per vector), whole lines, grid-stride.
__global__ __launch_bounds__(256) void mix_probe_kernel(const v4i* __restrict__ in, v4i* __restrict__ out, size_t n_out) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_out; i += (size_t)gridDim.x * blockDim.x) {
        const v4i* p = in + i * 4;
        const v4i a = p[0], b = p[1], c = p[2], d = p[3];
        out[i] = a ^ b ^ c ^ d;
    }
}

hipError_t launch_mix_probe(const void* in, void* out, size_t out_bytes, hipStream_t stream) {
    hipLaunchKernelGGL(mix_probe_kernel, dim3(65536), dim3(256), 0, stream, (const v4i*)in, (v4i*)out, out_bytes / 16);
    return hipGetLastError();
}

hipError_t launch_read_probe(const void* buf, size_t bytes, hipStream_t stream) {
    hipLaunchKernelGGL(read_probe_kernel, dim3(65536), dim3(256), 0, stream, (const v4i*)buf, bytes / 16, (int*)nullptr);
    return hipGetLastError();
}

}  // namespace dessert
