// Dense rows: the few hottest rows of a table appear in a large share of its bags (at Zipf exponents around 1.1 a hundred
// rows take half of all lookups).  Reducing them lookup by lookup reads every bag's gradient row once per hot row that the
// bag holds.  Here the table's gradient block is streamed ONCE and contracted with the count matrix of its dense rows,
//     partial[row, :] = sum over the chunk's bags of count[row, bag] * scale[bag] * grad[bag, :]
// on the matrix cores: M = up to 128 dense rows, N = the table's columns, K = bags.
//
// Precision: counts are small integers, exact in bfloat16; an fp32 gradient element is split into three bfloat16 pieces of
// 8 significant bits each, so that x = hi + mid + lo exactly; every product count * piece is exact in fp32 and the matrix
// core accumulates in fp32, i.e. this is an fp32 sum of exact products.  16-bit gradients (sum pooling) are one piece.
// Counts above 255 (a bag that holds one id very often) take a second pass with the count's upper byte, a multiple of 256
// and as exact; bags of more than 65535 ids are counted in rounds.
//
// Work split: a workgroup of 4 wavefronts takes a run of 256-bag blocks of one table and 256 of its columns.  Per block it
// builds the 128 x 256 count table in LDS from the rows' sorted bag lists (two bags per word, integer LDS additions), turns
// it into bfloat16 in place, and streams the block's gradient rows: a wavefront owns 64 columns (two per lane: 8-byte loads,
// 256 contiguous bytes per bag), 16 bags per step, the next step's 8 loads in flight while the current one multiplies.
// Tables narrower than 256 columns give the spare wavefronts a share of the bags.  Two workgroups per compute unit (68 KB of
// LDS, 128 accumulator registers) overlap each other's counting.  The partial sums of a row, one per workgroup run, are added
// in order by the kernel that applies the step, so the result does not depend on scheduling.
// Bound: the stream of the gradient block (matrix work at 128 rows and fp32 gradients is about a third of it).
// (Gradients are taken to be finite: 0 * Inf is NaN, so a non-finite element of one bag's gradient may reach every dense row
// of its table.)
#include "tbe_rows.h"

namespace tbe {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kDThreads = 256;
constexpr int kCntPitch = kDenseBags + 8;   // 16 bytes more than a power of two: the rows a wavefront reads lie in different banks
constexpr int kMTiles = kDenseRows / 32;
static_assert(kDenseBags == kDThreads, "one thread per bag of a block");

// the two columns a lane holds of one bag's gradient row
template <typename GT>
struct Pair;
template <>
struct Pair<float> {
    using raw_t = float2;
    static __device__ __forceinline__ raw_t load(const float* p) { return *reinterpret_cast<const float2*>(p); }
    static __device__ __forceinline__ raw_t zero() { return make_float2(0.f, 0.f); }
    static __device__ __forceinline__ float2 to_float(const raw_t r) { return r; }
};
template <>
struct Pair<__half> {
    using raw_t = uint32_t;
    static __device__ __forceinline__ raw_t load(const __half* p) { return *reinterpret_cast<const uint32_t*>(p); }
    static __device__ __forceinline__ raw_t zero() { return 0u; }
    static __device__ __forceinline__ float2 to_float(const raw_t r) {
        return make_float2(__half2float(__ushort_as_half((unsigned short)(r & 0xFFFFu))),
                           __half2float(__ushort_as_half((unsigned short)(r >> 16))));
    }
};
template <>
struct Pair<bf16_t> {
    using raw_t = uint32_t;
    static __device__ __forceinline__ raw_t load(const bf16_t* p) { return *reinterpret_cast<const uint32_t*>(p); }
    static __device__ __forceinline__ raw_t zero() { return 0u; }
    static __device__ __forceinline__ float2 to_float(const raw_t r) {
        return make_float2(__uint_as_float(r << 16), __uint_as_float(r & 0xFFFF0000u));
    }
};

__device__ __forceinline__ uint32_t upper_halves(const uint32_t lo, const uint32_t hi) {   // (hi's upper half : lo's upper half)
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}
__device__ __forceinline__ uint32_t lower_halves(const uint32_t lo, const uint32_t hi) {
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
template <bool F16>
__device__ __forceinline__ f32x16 mfma(const uint4 a, const uint4 b, const f32x16 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// a count below 256, or a multiple of 256 below 65536, as bfloat16 / binary16 bits (exact)
template <bool F16>
__device__ __forceinline__ uint32_t count_bits(const uint32_t c) {
    if constexpr (F16) return (uint32_t)__half_as_ushort(__float2half_rn((float)c));
    else return __float_as_uint((float)c) >> 16;
}

template <bool MEAN, typename GT>
__global__ __launch_bounds__(kDThreads, 2) void seg_dense_kernel(const SegArgs a, const uint32_t col_blocks) {
    constexpr bool kExact = !MEAN && sizeof(GT) == 2;                 // a gradient element is one piece
    constexpr bool kF16 = kExact && __is_same(GT, __half);            // binary16 pieces, else bfloat16
    constexpr int kPieces = kExact ? 1 : 3;
    using raw_t = typename Pair<GT>::raw_t;
    __shared__ __align__(16) uint16_t s_cnt[kDenseRows * kCntPitch];
    __shared__ uint32_t s_lo[kDenseRows], s_pref[kDenseRows + 1], s_scan[kDThreads / kWave], s_flags;
    __shared__ __align__(16) float s_scale[MEAN ? kDenseBags : 4];
    uint32_t bx = blockIdx.x;
    const uint32_t cb = bx % col_blocks;
    bx /= col_blocks;
    const uint32_t chunk = bx % a.dense_chunks;
    const int t = (int)(bx / a.dense_chunks);
    const uint32_t nd = a.dense_n[t];
    if (nd == 0u) return;
    const int d0 = a.D_off[t];
    const int D = a.D_off[t + 1] - d0;
    if ((int)cb * 256 >= D) return;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id();
    const int w = (int)(tid >> 6);
    const int groups = D - (int)cb * 256 > 128 ? 4 : (D - (int)cb * 256 > 64 ? 2 : 1);   // 64-column groups, a power of two
    const int cg = w & (groups - 1);
    const int split = w / groups, splits = 4 / groups;   // which share of the bags this wavefront takes
    const int kh = lane >> 5;                            // which half of a 16-bag step
    const int col = (int)cb * 256 + cg * 64 + 2 * (lane & 31);
    const bool col_on = col < D;
    const uint32_t mt = (nd + 31u) >> 5;                 // row tiles in use
    const GT* gcol = static_cast<const GT*>(a.grad_out) + d0 + col;
    const uint32_t B = (uint32_t)a.B;
    const int64_t bag0 = (int64_t)t * B;
    uint32_t* const cnt32 = reinterpret_cast<uint32_t*>(s_cnt);
    f32x16 acc[kMTiles][2];
#pragma unroll
    for (int m = 0; m < kMTiles; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][0][r] = acc[m][1][r] = 0.f;

    const uint32_t k_lo = chunk * a.dense_per_chunk;
    const uint32_t k_hi = k_lo + a.dense_per_chunk < a.dense_blocks ? k_lo + a.dense_per_chunk : a.dense_blocks;
    for (uint32_t k = k_lo; k < k_hi; ++k) {
        const uint32_t b0 = k * kDenseBags;
        const uint32_t nb = B - b0 < (uint32_t)kDenseBags ? B - b0 : (uint32_t)kDenseBags;   // bags of the block
        for (uint32_t pass = 0;; ++pass) {   // pass 2r + d: counts' digit d (low, high byte) of round r
            const uint32_t round = pass >> 1, digit = pass & 1u;
            __syncthreads();   // the table is free (previous block, or pass)
            // ---- counts of the block: zero, then one LDS addition per lookup of a dense row
            for (uint32_t i = tid; i < mt * 32u * (kCntPitch / 8); i += kDThreads)
                reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
            uint32_t n = 0;
            if (tid < nd) {
                const uint32_t* ix = a.dense_index + ((size_t)t * kDenseRows + tid) * (a.dense_blocks + 1u) + k;
                const uint32_t lo = ix[0];
                n = ix[1] - lo;
                s_lo[tid] = lo;
            }
            if (tid == 0) s_flags = 0u;
            uint32_t L = 0;
            if (tid < nb) L = a.offsets.length(bag0 + b0 + tid);
            if (MEAN) s_scale[tid] = L > 0u ? 1.f / (float)L : 0.f;
            uint32_t all;
            const uint32_t ex = block_excl_scan<kDThreads>(n, s_scan, &all);
            if (tid < nd) s_pref[tid] = ex;
            if (L > 255u) atomicOr(&s_flags, L > 65535u ? 3u : 1u);   // (a count cannot exceed its bag's length)
            __syncthreads();
            const uint32_t flags = s_flags;
            bool more = false;   // lookups left for a later round
            for (uint32_t e = tid; e < all; e += kDThreads) {
                uint32_t lo = 0, hi = nd;   // the row: last h with s_pref[h] <= e
                while (hi - lo > 1u) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_pref[mid] <= e) lo = mid;
                    else hi = mid;
                }
                const uint32_t p = s_lo[lo] + (e - s_pref[lo]);
                const uint32_t bag = a.bag_sorted[p];
                bool take = true;
                if (flags & 2u) {   // position among the row's lookups of this bag: 65535 of them per round
                    uint32_t q0 = s_lo[lo], q1 = p;   // first position in [q0, p] that holds this bag
                    while (q0 < q1) {
                        const uint32_t mid = q0 + ((q1 - q0) >> 1);
                        if (a.bag_sorted[mid] < bag) q0 = mid + 1u;
                        else q1 = mid;
                    }
                    const uint32_t r = (p - q0) / 65535u;
                    take = r == round;
                    more |= r > round;
                }
                const uint32_t b = (uint32_t)((int64_t)bag - bag0) - b0;
                if (take && b < nb) atomicAdd(&cnt32[lo * (kCntPitch / 2) + (b >> 1)], 1u << (16u * (b & 1u)));
            }
            if (more) atomicOr(&s_flags, 8u);
            __syncthreads();
            bool big = false;
            for (uint32_t i = tid; i < mt * 32u * (kCntPitch / 8); i += kDThreads) {
                uint4 v = reinterpret_cast<uint4*>(s_cnt)[i];
                uint32_t* x = &v.x;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (flags) big |= (x[q] & 0xFF00FF00u) != 0u;
                    const uint32_t c = digit ? x[q] & 0xFF00FF00u : (flags ? x[q] & 0x00FF00FFu : x[q]);
                    x[q] = count_bits<kF16>(c & 0xFFFFu) | (count_bits<kF16>(c >> 16) << 16);
                }
                reinterpret_cast<uint4*>(s_cnt)[i] = v;
            }
            if (big) atomicOr(&s_flags, 4u);
            __syncthreads();
            // ---- stream the block's gradient rows, 16 bags per step; a wavefront takes every splits-th step
            const int steps = (int)((nb + 15u) >> 4);
            raw_t x[8];
            auto load_step = [&](const int j) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t b = (uint32_t)(j * 16 + kh * 8 + i);
                    x[i] = (col_on && j < steps && b < nb) ? Pair<GT>::load(gcol + (int64_t)(b0 + b) * a.sumD) : Pair<GT>::zero();
                }
            };
            load_step(split);
            for (int j = split; j < steps; j += splits) {
                // pieces of the 8 bags, packed for the matrix core: [piece][column of the pair]
                uint4 f[kPieces][2];
                if constexpr (kExact) {
                    uint32_t* f0 = &f[0][0].x;
                    uint32_t* f1 = &f[0][1].x;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f0[i] = lower_halves(x[2 * i], x[2 * i + 1]);
                        f1[i] = upper_halves(x[2 * i], x[2 * i + 1]);
                    }
                } else {
                    float v[8][2];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float2 g = Pair<GT>::to_float(x[i]);
                        v[i][0] = g.x;
                        v[i][1] = g.y;
                    }
                    if constexpr (MEAN) {
                        const float4 sa = *reinterpret_cast<const float4*>(&s_scale[j * 16 + kh * 8]);
                        const float4 sb = *reinterpret_cast<const float4*>(&s_scale[j * 16 + kh * 8 + 4]);
                        const float sc[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            v[i][0] *= sc[i];
                            v[i][1] *= sc[i];
                        }
                    }
#pragma unroll
                    for (int p = 0; p < 3; ++p)
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            uint32_t* o = &f[p][c].x;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const uint32_t u0 = __float_as_uint(v[2 * i][c]), u1 = __float_as_uint(v[2 * i + 1][c]);
                                o[i] = upper_halves(u0, u1);
                                if (p < 2) {   // what the upper 16 bits leave, exactly
                                    v[2 * i][c] -= __uint_as_float(u0 & 0xFFFF0000u);
                                    v[2 * i + 1][c] -= __uint_as_float(u1 & 0xFFFF0000u);
                                }
                            }
                        }
                }
                load_step(j + splits);
#pragma unroll
                for (int m = 0; m < kMTiles; ++m) {
                    if ((uint32_t)m < mt) {
                        const uint4 av = *reinterpret_cast<const uint4*>(&s_cnt[(m * 32 + (lane & 31)) * kCntPitch + j * 16 + kh * 8]);
#pragma unroll
                        for (int p = kPieces - 1; p >= 0; --p) {   // small pieces first
                            acc[m][0] = mfma<kF16>(av, f[p][0], acc[m][0]);
                            acc[m][1] = mfma<kF16>(av, f[p][1], acc[m][1]);
                        }
                    }
                }
            }
            const uint32_t fl = s_flags;
            if (digit == 0u && !(fl & 4u)) {        // no count has an upper byte: skip that pass
                if (!(fl & 8u)) break;
                ++pass;
            } else if (digit == 1u && !(fl & 8u)) {
                break;
            }
        }
    }
    // ---- add up the wavefronts that shared the bags of a column group, in order
    float* const red = reinterpret_cast<float*>(s_cnt);   // [32 * mt rows][64 * groups columns]: at most 64 KB (splits > 1: groups <= 2)
    for (int sp = 1; sp < splits; ++sp) {
        __syncthreads();
        if (split == sp) {
#pragma unroll
            for (int m = 0; m < kMTiles; ++m)
                if ((uint32_t)m < mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int h = m * 32 + (r & 3) + 8 * (r >> 2) + 4 * kh;
                        *reinterpret_cast<float2*>(&red[h * (64 * groups) + cg * 64 + 2 * (lane & 31)]) = make_float2(acc[m][0][r], acc[m][1][r]);
                    }
        }
        __syncthreads();
        if (split == 0) {
#pragma unroll
            for (int m = 0; m < kMTiles; ++m)
                if ((uint32_t)m < mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int h = m * 32 + (r & 3) + 8 * (r >> 2) + 4 * kh;
                        const float2 o = *reinterpret_cast<const float2*>(&red[h * (64 * groups) + cg * 64 + 2 * (lane & 31)]);
                        acc[m][0][r] += o.x;
                        acc[m][1][r] += o.y;
                    }
        }
    }
    if (split == 0 && col_on) {
        const size_t slot0 = (size_t)a.dense_slot0 + (size_t)t * kDenseRows * a.dense_chunks + chunk;
#pragma unroll
        for (int m = 0; m < kMTiles; ++m)
            if ((uint32_t)m < mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t h = (uint32_t)(m * 32 + (r & 3) + 8 * (r >> 2) + 4 * kh);
                    if (h < nd)
                        *reinterpret_cast<float2*>(a.partial + (slot0 + (size_t)h * a.dense_chunks) * a.maxD + col) = make_float2(acc[m][0][r], acc[m][1][r]);
                }
    }
}

template <typename GT>
static void launch_dense_gt(const SegArgs& a, bool mean, hipStream_t s) {
    const uint32_t col_blocks = ((uint32_t)a.maxD + 255u) / 256u;
    const unsigned grid = (unsigned)a.T * a.dense_chunks * col_blocks;
    if (mean) seg_dense_kernel<true, GT><<<grid, kDThreads, 0, s>>>(a, col_blocks);
    else seg_dense_kernel<false, GT><<<grid, kDThreads, 0, s>>>(a, col_blocks);
}

void launch_dense(const SegArgs& a, int grad_io, bool mean, hipStream_t s) {
    if (grad_io == 0) launch_dense_gt<float>(a, mean, s);
    else if (grad_io == 1) launch_dense_gt<__half>(a, mean, s);
    else launch_dense_gt<bf16_t>(a, mean, s);
}

}  // namespace tbe
