// Dense rows: the few hottest rows of a table appear in a large share of its bags (at Zipf exponents around 1.1 a hundred
// rows take half of all lookups).  Reducing them lookup by lookup reads every bag's gradient row once per hot row that the
// bag holds.  Here the table's gradient block is streamed ONCE and contracted with the count matrix of its dense rows,
//     partial[row, :] = sum over the chunk's bags of count[row, bag] * scale[bag] * grad[bag, :]
// on the matrix cores: M = up to 128 dense rows, N = the table's columns, K = bags.
//
// Precision: counts are small integers, exact in bfloat16; an fp32 gradient element is split into three bfloat16 pieces of
// 8 significant bits each, so that x = hi + mid + lo exactly down to elements of 2^-110 (below, the last piece is subnormal and
// ends at 2^-133: the kernel that adds the partial sums looks for sums that this could reach); every product count * piece is
// exact in fp32, and the matrix core adds them in fp32, one rounding for 8 products (checked on the device: to nearest even,
// with subnormal operands kept).  16-bit gradients (sum pooling) are one piece.  Under mean pooling an element is multiplied by
// its bag's 1 / length first, which rounds once.
// What decides the error is how many terms go into one running sum, since every addition rounds at its magnitude: after 512
// bags (kRunBlocks) a wavefront adds its accumulators to the partial sum in memory and starts again.  Relative error of the
// rows' gradient sums against 64 bits, N(0,1) gradients, 64 tables x 32768 bags x 256 columns, Zipf 1.1: ranks 0 to 15 / 16 to
// 127 2.1e-7 / 1.3e-7 (without the runs 4.0e-7 / 2.2e-7; before the matrix cores 5.2e-7 / 1.4e-7); 32 tables x 65536 bags x 32
// columns, mean pooling, 2.2e-7 / 1.4e-7 (before 2.9e-7 / 1.2e-7).
// Counts above 255 (a bag that holds one id very often) take a second pass with the count's upper byte, a multiple of 256
// and as exact; bags of more than 65535 ids are counted in rounds.
//
// Work split: a workgroup of 4 wavefronts takes a run of 256-bag blocks of one table and 256 of its columns.  Per block it
// builds the 128 x 256 count table in LDS from the rows' sorted bag lists (two bags per word, integer LDS additions), turns
// it into bfloat16 in place, and streams the block's gradient rows: a wavefront owns 64 columns (two per lane: 8-byte loads,
// 256 contiguous bytes per bag), 16 bags per step, the next step's 8 loads in flight while the current one multiplies.
// Tables narrower than 256 columns give the spare wavefronts a share of the bags.  Two workgroups per compute unit (68 KB of
// LDS, 128 accumulator registers) overlap each other's counting.  The partial sums of a row, one per workgroup, are added
// in order by the kernel that applies the step, so the result does not depend on scheduling.
// Tables of up to 64 columns have a form of their own (dense_run_narrow), for there the count table, whose size does not shrink with
// the columns, is what takes the time: 30 tables x 65536 bags x 32 columns, long-tailed bags, Zipf 1.3, mean pooling, 277 -> 175 us;
// 16 x 32768 x 64, Zipf 1.1, binary16 gradients 76 -> 68, fp32 and mean pooling 85 -> 78.  Taken for 65 to 128 columns too (four
// groups, each turning all counts into bfloat16 again) 137 -> 145.
// Bound: wide tables by the stream of the gradient block, at about half the copy rate (64 tables x 32768 bags, 48 of 256
// columns: 1.9 GB in 0.64 ms), narrow ones by the chain of searches, list loads and LDS additions that fills the count table (a block
// of 256 bags takes 11 us, two at a time per compute unit, for about 4 us of instructions).
// Measured, whole training step, against 16 dense rows on the vector units and sweeps over the rest: the former 9.5 -> 8.2 ms, the
// latter, mean pooling, 2.5 -> 1.7 ms.  Of that, the loads ahead of the matrix instructions 20 us of 690; the runs cost 85 us of 607
// (and 8 of 296 at 32 columns); the counting as a function of its own, whose registers the compiler then lays out apart, 690 -> 645.
// Spilled vector registers: 6 to 9 under mean pooling, 1 or 2 with 16-bit gradients, none else.
// 0 * Inf is NaN, so a non-finite element of one bag's gradient reaches every dense row of its table here; the kernel that
// adds the partial sums reduces such rows again from their own lookups.
#include "tbe_rows.h"

namespace tbe {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kDThreads = 256;
constexpr int kCntPitch = kDenseBags + 8;   // 16 bytes more than a power of two: the rows a wavefront reads lie in different banks
static_assert(kDenseBags == kDThreads, "one thread per bag of a block");
constexpr uint32_t kRunBlocks = 2;   // blocks whose bags a wavefront's accumulators take before they are emptied

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

struct DenseLds {
    __align__(16) uint16_t cnt[kDenseRows * kCntPitch];
    __align__(16) float scale[kDenseBags];
    uint32_t lo[kDenseRows], pref[kDenseRows], scan[kDThreads / kWave], flags;
};

// The counts of a block of bags, in the table: ix0 and ix1 where the thread's dense row starts and ends in the block, L its bag's
// length.  `round`: bags of more than 65535 ids are counted 65535 at a time.  Returns 0, or whether a bag of the block has more
// ids than a byte counts (bit 0), or than a round does (bit 1).
template <int MT, bool MEAN, int kU>
__device__ __forceinline__ uint32_t count_block(const SegArgs& a, const uint32_t nd, const uint32_t ix0, const uint32_t ix1, const uint32_t L,
                                                const int64_t bag0, const uint32_t b0, const uint32_t nb, const uint32_t round, DenseLds* S) {
    const uint32_t tid = threadIdx.x;
    uint16_t* const s_cnt = S->cnt;
    uint32_t* const s_lo = S->lo;
    uint32_t* const s_pref = S->pref;
    uint32_t* const cnt32 = reinterpret_cast<uint32_t*>(s_cnt);
    __syncthreads();   // the table is free (previous block, or pass)
    // ---- counts of the block: zero, then one LDS addition per lookup of a dense row
    for (uint32_t i = tid; i < MT * 32u * (kCntPitch / 8); i += kDThreads)
        reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t n = ix1 - ix0;
    if (tid < nd) s_lo[tid] = ix0;
    if (tid == 0) S->flags = 0u;
    if (MEAN) S->scale[tid] = L > 0u ? 1.f / (float)L : 0.f;
    uint32_t all;
    const uint32_t ex = block_excl_scan<kDThreads>(n, S->scan, &all);
    if (tid < (uint32_t)kDenseRows) s_pref[tid] = tid < nd ? ex : 0xFFFFFFFFu;
    if (L > 255u) atomicOr(&S->flags, L > 65535u ? 3u : 1u);   // (a count cannot exceed its bag's length)
    __syncthreads();
    const uint32_t flags = S->flags;
    bool more = false;   // lookups left for a later round
    // kU lookups in flight per thread: the searches and loads of one are a chain of LDS and L2 trips
    for (uint32_t e0 = tid; e0 < all; e0 += kU * kDThreads) {
        uint32_t row[kU], p[kU], bag[kU];
#pragma unroll
        for (int q = 0; q < kU; ++q) row[q] = 0u;
#pragma unroll
        for (uint32_t step = kDenseRows / 2; step > 0u; step >>= 1)   // the row: last h < nd with s_pref[h] <= e
#pragma unroll
            for (int q = 0; q < kU; ++q)
                if (s_pref[row[q] + step] <= e0 + q * kDThreads) row[q] += step;   // (s_pref[nd ..] is above every e)
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            const uint32_t e = e0 + q * kDThreads;
            p[q] = s_lo[row[q]] + (e - s_pref[row[q]]);
            bag[q] = a.bag_sorted[e < all ? p[q] : s_lo[0]];
        }
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            if (e0 + q * kDThreads >= all) continue;
            bool take = true;
            if (flags & 2u) {   // position among the row's lookups of this bag: 65535 of them per round
                uint32_t q0 = s_lo[row[q]], q1 = p[q];   // first position in [q0, p] that holds this bag
                while (q0 < q1) {
                    const uint32_t mid = q0 + ((q1 - q0) >> 1);
                    if (a.bag_sorted[mid] < bag[q]) q0 = mid + 1u;
                    else q1 = mid;
                }
                const uint32_t r = (p[q] - q0) / 65535u;
                take = r == round;
                more |= r > round;
            }
            const uint32_t b = (uint32_t)((int64_t)bag[q] - bag0) - b0;
            if (take && b < nb) atomicAdd(&cnt32[row[q] * (kCntPitch / 2) + (b >> 1)], 1u << (16u * (b & 1u)));
        }
    }
    if (more) atomicOr(&S->flags, 8u);
    return flags;
}

// MT: row tiles of 32 (compiled apart, so that the matrix instructions of a step are one straight run)
template <int MT, bool MEAN, typename GT>
__device__ __forceinline__ void dense_run(const SegArgs& a, const uint32_t cb, const uint32_t chunk, const int t,
                                          const uint32_t nd, const uint2 tab, const int d0, const int D, DenseLds* S) {
    constexpr bool kExact = !MEAN && sizeof(GT) == 2;                 // a gradient element is one piece
    constexpr bool kF16 = kExact && __is_same(GT, __half);            // binary16 pieces, else bfloat16
    constexpr int kPieces = kExact ? 1 : 3;
    using raw_t = typename Pair<GT>::raw_t;
    uint16_t* const s_cnt = S->cnt;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id();
    const int w = (int)(tid >> 6);
    const int groups = D - (int)cb * 256 > 128 ? 4 : (D - (int)cb * 256 > 64 ? 2 : 1);   // 64-column groups, a power of two
    const int cg = w & (groups - 1);
    const int split = w / groups, splits = 4 / groups;   // which share of the bags this wavefront takes
    const int kh = lane >> 5;                            // which half of a 16-bag step
    const int col = (int)cb * 256 + cg * 64 + 2 * (lane & 31);
    const bool col_on = col < D;                         // (other lanes read column 0 and store nothing)
    // a lane's address: wavefront-uniform start of a bag's gradient row + 32-bit byte offset
    const char* const gtab = static_cast<const char*>(a.grad_out) + (int64_t)d0 * (int)sizeof(GT);
    const int64_t pitch = (int64_t)a.sumD * (int)sizeof(GT);
    const uint32_t lane_col = (uint32_t)(col_on ? col : 0) * (uint32_t)sizeof(GT);
    const uint32_t B = (uint32_t)a.B;
    const int64_t bag0 = (int64_t)t * B;
    const uint32_t* const my_ix = a.dense_index + ((size_t)tab.x * kDenseRows + (tid < nd ? tid : 0u)) * (a.dense_blocks + 1u);
    char* const sums = reinterpret_cast<char*>(a.dense_partial + (size_t)tab.y * 4u + (size_t)chunk * nd * (uint32_t)D);
    const uint32_t run = kRunBlocks * (uint32_t)splits;   // blocks that go into the accumulators before they are emptied
    const uint32_t k_lo = chunk * a.dense_per_chunk;
    const uint32_t k_hi = k_lo + a.dense_per_chunk < a.dense_blocks ? k_lo + a.dense_per_chunk : a.dense_blocks;
#pragma unroll 1
    for (uint32_t k0 = k_lo; k0 < k_hi; k0 += run) {
        const uint32_t k1 = k0 + run < k_hi ? k0 + run : k_hi;
        f32x16 acc[MT][2];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][0][r] = acc[m][1][r] = 0.f;
        for (uint32_t k = k0; k < k1; ++k) {
            const uint32_t b0 = k * kDenseBags;
            const uint32_t nb = B - b0 < (uint32_t)kDenseBags ? B - b0 : (uint32_t)kDenseBags;   // bags of the block
            uint32_t ix0 = 0, ix1 = 0;   // this thread's row's lookups in the block
            if (tid < nd) {
                ix0 = my_ix[k];
                ix1 = my_ix[k + 1u];
            }
            const uint32_t L = b0 + tid < B ? a.offsets.length(bag0 + b0 + tid) : 0u;   // this thread's bag's length
            for (uint32_t pass = 0;; ++pass) {   // pass 2r + d: counts' digit d (low, high byte) of round r
                const uint32_t round = pass >> 1, digit = pass & 1u;
                const uint32_t flags = count_block<MT, MEAN, 8>(a, nd, ix0, ix1, L, bag0, b0, nb, round, S);
                __syncthreads();
                bool big = false;
                for (uint32_t i = tid; i < MT * 32u * (kCntPitch / 8); i += kDThreads) {
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
                if (big) atomicOr(&S->flags, 4u);
                __syncthreads();
                // ---- stream the block's gradient rows, 16 bags per step; a wavefront takes every splits-th step
                const int steps = (int)((nb + 15u) >> 4);
                const char* const gblk = gtab + (int64_t)b0 * pitch;
                // (a bag behind the batch's end has zero counts: the block's last will do, and where that is not finite the sums are redone)
                auto load_step = [&](raw_t (&x)[8], const int j) {
                    if (nb == (uint32_t)kDenseBags) {
                        const char* const row0 = gblk + (int64_t)(j * 16) * pitch;
                        const uint32_t off = lane_col + (uint32_t)(kh * 8) * (uint32_t)pitch;
#pragma unroll
                        for (int i = 0; i < 8; ++i) x[i] = Pair<GT>::load(reinterpret_cast<const GT*>(row0 + i * pitch + off));
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const uint32_t b = (uint32_t)(j * 16 + kh * 8 + i);
                            x[i] = Pair<GT>::load(reinterpret_cast<const GT*>(gblk + (int64_t)(b < nb ? b : nb - 1u) * pitch + lane_col));
                        }
                    }
                };
                auto multiply_step = [&](raw_t (&x)[8], const int j, const int next) {
                    uint4 f[2][kPieces];   // per column of the pair: pieces of the 8 bags, packed for the matrix core
                    if constexpr (kExact) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            (&f[0][0].x)[i] = lower_halves(x[2 * i], x[2 * i + 1]);
                            (&f[1][0].x)[i] = upper_halves(x[2 * i], x[2 * i + 1]);
                        }
                    } else {
                        float sc[8];
                        if constexpr (MEAN) {
                            const float4 sa = *reinterpret_cast<const float4*>(&S->scale[j * 16 + kh * 8]);
                            const float4 sb = *reinterpret_cast<const float4*>(&S->scale[j * 16 + kh * 8 + 4]);
                            sc[0] = sa.x; sc[1] = sa.y; sc[2] = sa.z; sc[3] = sa.w;
                            sc[4] = sb.x; sc[5] = sb.y; sc[6] = sb.z; sc[7] = sb.w;
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float2 g0 = Pair<GT>::to_float(x[2 * i]), g1 = Pair<GT>::to_float(x[2 * i + 1]);
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                float v0 = c ? g0.y : g0.x, v1 = c ? g1.y : g1.x;
                                if constexpr (MEAN) {
                                    v0 *= sc[2 * i];
                                    v1 *= sc[2 * i + 1];
                                }
#pragma unroll
                                for (int p = 0; p < 3; ++p) {
                                    const uint32_t u0 = __float_as_uint(v0), u1 = __float_as_uint(v1);
                                    (&f[c][p].x)[i] = upper_halves(u0, u1);
                                    v0 -= __uint_as_float(u0 & 0xFFFF0000u);   // what the upper 16 bits leave, exactly
                                    v1 -= __uint_as_float(u1 & 0xFFFF0000u);
                                }
                            }
                        }
                    }
                    load_step(x, next);
                    // (without this line the compiler turns "loaded here or ahead of the loop" into one load at the top of the next
                    // step, right before its use: nothing would be in flight while the matrix cores work)
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        const uint4 av = *reinterpret_cast<const uint4*>(&s_cnt[(m * 32 + (lane & 31)) * kCntPitch + j * 16 + kh * 8]);
#pragma unroll
                        for (int p = kPieces - 1; p >= 0; --p) {   // small pieces first
                            acc[m][0] = mfma<kF16>(av, f[0][p], acc[m][0]);
                            acc[m][1] = mfma<kF16>(av, f[1][p], acc[m][1]);
                        }
                    }
                };
                raw_t x[8];   // the next step's rows are in flight while a step multiplies
                const int last = steps - 1;
                load_step(x, split < last ? split : last);
#pragma unroll 1
                for (int j = split; j < steps; j += splits) multiply_step(x, j, j + splits < last ? j + splits : last);
                const uint32_t fl = S->flags;
                if (digit == 0u && !(fl & 4u)) {        // no count has an upper byte: skip that pass
                    if (!(fl & 8u)) break;
                    ++pass;
                } else if (digit == 1u && !(fl & 8u)) {
                    break;
                }
            }
        }
        // ---- the accumulators go to the rows' partial sums and start again.  First the wavefronts that shared the bags of a column
        // group, in order.  (The addresses below are kept from being computed ahead of the loops: there are no registers for them.)
#pragma unroll 1
        for (int sp = 1; sp < splits; ++sp) {
            uint32_t red_pitch = 64u * (uint32_t)groups;
            asm volatile("" : "+s"(red_pitch));
            // [32 * MT rows][64 * groups columns]: at most 64 KB (splits > 1: groups <= 2)
            float* red = reinterpret_cast<float*>(s_cnt) + 4u * (uint32_t)kh * red_pitch + (uint32_t)(cg * 64 + 2 * (lane & 31));
            __syncthreads();
            if (split == sp) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q, red += 8u * red_pitch)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            *reinterpret_cast<float2*>(red + (uint32_t)r * red_pitch) = make_float2(acc[m][0][4 * q + r], acc[m][1][4 * q + r]);
            }
            __syncthreads();
            if (split == 0) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q, red += 8u * red_pitch)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float2 o = *reinterpret_cast<const float2*>(red + (uint32_t)r * red_pitch);
                            acc[m][0][4 * q + r] += o.x;
                            acc[m][1][4 * q + r] += o.y;
                        }
            }
        }
        if (split == 0 && col_on) {
            const bool add = k0 > k_lo;   // not the chunk's first run: this lane has written the sum before
            uint32_t row_bytes = (uint32_t)D * 4u;
            int left = (int)nd - 4 * kh;   // dense rows from this lane's first on
            asm volatile("" : "+s"(row_bytes), "+v"(left));
            uint32_t at = (uint32_t)(4 * kh) * row_bytes + (uint32_t)col * 4u;
#pragma unroll
            for (int m = 0; m < MT; ++m, at += 32u * row_bytes) {
                if (add) {   // all loads of a row tile in flight
                    float2 o[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int h = (r & 3) + 8 * (r >> 2);
                        o[r] = *reinterpret_cast<const float2*>(sums + (m * 32 + h < left ? at + (uint32_t)h * row_bytes : (uint32_t)col * 4u));
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        acc[m][0][r] += o[r].x;
                        acc[m][1][r] += o[r].y;
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int h = (r & 3) + 8 * (r >> 2);
                    if (m * 32 + h < left) *reinterpret_cast<float2*>(sums + (at + (uint32_t)h * row_bytes)) = make_float2(acc[m][0][r], acc[m][1][r]);
                }
            }
        }
    }
}

__device__ __forceinline__ float grad_float(const float x) { return x; }
__device__ __forceinline__ float grad_float(const __half x) { return __half2float(x); }
__device__ __forceinline__ float grad_float(const bf16_t x) { return bf16_to_float(__builtin_bit_cast(unsigned short, x)); }

// Tables of up to 64 columns.  A lane holds one column, not two, so that 32 columns fill the matrix instructions and need half the
// accumulators: the registers freed hold four steps of gradient rows, which are loaded, like the next block's list ends and bag
// lengths, ahead of the counting and arrive during it.  A count is turned into bfloat16 where it is multiplied (once, or twice above
// 32 columns), which saves a pass over the table and a barrier.
template <int MT, int GROUPS, bool MEAN, typename GT>
__device__ __forceinline__ void dense_run_narrow(const SegArgs& a, const uint32_t chunk, const int t, const uint32_t nd, const uint2 tab,
                                                 const int d0, const int D, DenseLds* S) {
    constexpr bool kExact = !MEAN && sizeof(GT) == 2;
    constexpr bool kF16 = kExact && __is_same(GT, __half);
    constexpr int kPieces = kExact ? 1 : 3;
    constexpr int kAhead = GROUPS == 2 ? 2 : 4;   // steps whose gradient rows are in flight
    uint16_t* const s_cnt = S->cnt;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id();
    const int w = (int)(tid >> 6);
    constexpr int splits = 4 / GROUPS;                   // wavefronts that share the bags of a 32-column group
    const int cg = w & (GROUPS - 1), split = w / GROUPS;
    const int kh = lane >> 5;
    const int col = cg * 32 + (lane & 31);
    const bool col_on = col < D;                         // (other lanes read column 0 and store nothing)
    const char* const gtab = static_cast<const char*>(a.grad_out) + (int64_t)(d0 + (col_on ? col : 0)) * (int)sizeof(GT);
    const int64_t pitch = (int64_t)a.sumD * (int)sizeof(GT);
    const uint32_t B = (uint32_t)a.B;
    const int64_t bag0 = (int64_t)t * B;
    const uint32_t* const my_ix = a.dense_index + ((size_t)tab.x * kDenseRows + (tid < nd ? tid : 0u)) * (a.dense_blocks + 1u);
    float* const sums = a.dense_partial + (size_t)tab.y * 4u + (size_t)chunk * nd * (uint32_t)D;
    constexpr uint32_t run = 4 * kRunBlocks;
    const uint32_t k_lo = chunk * a.dense_per_chunk;
    const uint32_t k_hi = k_lo + a.dense_per_chunk < a.dense_blocks ? k_lo + a.dense_per_chunk : a.dense_blocks;
    if (k_lo >= k_hi) return;
    uint32_t next0 = my_ix[k_lo], next1 = my_ix[k_lo + 1u];   // the next block's
    uint32_t nextL = k_lo * kDenseBags + tid < B ? a.offsets.length(bag0 + k_lo * kDenseBags + tid) : 0u;
#pragma unroll 1
    for (uint32_t k0 = k_lo; k0 < k_hi; k0 += run) {
        const uint32_t k1 = k0 + run < k_hi ? k0 + run : k_hi;
        f32x16 acc[MT], acc2[GROUPS == 2 ? MT : 1];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[m][r] = 0.f;
                if (GROUPS == 2) acc2[m][r] = 0.f;
            }
#pragma unroll 1
        for (uint32_t k = k0; k < k1; ++k) {
            const uint32_t b0 = k * kDenseBags;
            const uint32_t nb = B - b0 < (uint32_t)kDenseBags ? B - b0 : (uint32_t)kDenseBags;
            const uint32_t ix0 = tid < nd ? next0 : 0u, ix1 = tid < nd ? next1 : 0u, L = nextL;
            GT x[kAhead][8];
            const char* const gblk = gtab + (int64_t)b0 * pitch;
            auto load_step = [&](GT (&v)[8], const int j) {   // (a bag behind the batch's end has zero counts: the block's last will do)
                uint32_t bag = (uint32_t)(j * 16 + kh * 8);
                asm volatile("" : "+v"(bag));   // (or 16 addresses are computed ahead of the loops, and spilled)
#pragma unroll
                for (uint32_t i = 0; i < 8; ++i) {
                    const uint32_t b = bag + i;
                    v[i] = *reinterpret_cast<const GT*>(gblk + (uint64_t)(b < nb ? b : nb - 1u) * (uint32_t)pitch);
                }
            };
#pragma unroll
            for (int q = 0; q < kAhead; ++q) load_step(x[q], split + q * splits);
            if (k + 1u < k_hi) {
                next0 = next1;
                next1 = my_ix[k + 2u];
                nextL = b0 + kDenseBags + tid < B ? a.offsets.length(bag0 + b0 + kDenseBags + tid) : 0u;
            }
            for (uint32_t pass = 0;; ++pass) {
                const uint32_t round = pass >> 1, digit = pass & 1u;
                const uint32_t flags = count_block<MT, MEAN, 8>(a, nd, ix0, ix1, L, bag0, b0, nb, round, S);
                __syncthreads();
                const uint32_t keep = flags == 0u ? 0xFFFFFFFFu : (digit ? 0xFF00FF00u : 0x00FF00FFu);
                uint32_t upper = 0;   // bits of counts above 255
                auto multiply_step = [&](GT (&v)[8], const int j, f32x16* const to) {
                    uint4 f[kPieces];
                    if constexpr (kExact) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            (&f[0].x)[i] = (uint32_t)__builtin_bit_cast(uint16_t, v[2 * i]) | (uint32_t)__builtin_bit_cast(uint16_t, v[2 * i + 1]) << 16;
                    } else {
                        float sc[8];
                        if constexpr (MEAN) {
                            const float4 sa = *reinterpret_cast<const float4*>(&S->scale[j * 16 + kh * 8]);
                            const float4 sb = *reinterpret_cast<const float4*>(&S->scale[j * 16 + kh * 8 + 4]);
                            sc[0] = sa.x; sc[1] = sa.y; sc[2] = sa.z; sc[3] = sa.w;
                            sc[4] = sb.x; sc[5] = sb.y; sc[6] = sb.z; sc[7] = sb.w;
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float v0 = grad_float(v[2 * i]), v1 = grad_float(v[2 * i + 1]);
                            if constexpr (MEAN) {
                                v0 *= sc[2 * i];
                                v1 *= sc[2 * i + 1];
                            }
#pragma unroll
                            for (int p = 0; p < 3; ++p) {
                                const uint32_t u0 = __float_as_uint(v0), u1 = __float_as_uint(v1);
                                (&f[p].x)[i] = upper_halves(u0, u1);
                                v0 -= __uint_as_float(u0 & 0xFFFF0000u);
                                v1 -= __uint_as_float(u1 & 0xFFFF0000u);
                            }
                        }
                    }
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        uint4 av = *reinterpret_cast<const uint4*>(&s_cnt[(m * 32 + (lane & 31)) * kCntPitch + j * 16 + kh * 8]);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            uint32_t c = (&av.x)[q];
                            upper |= c & 0xFF00FF00u;
                            c &= keep;
                            (&av.x)[q] = count_bits<kF16>(c & 0xFFFFu) | (count_bits<kF16>(c >> 16) << 16);
                        }
#pragma unroll
                        for (int p = kPieces - 1; p >= 0; --p) to[m] = mfma<kF16>(av, f[p], to[m]);   // small pieces first
                    }
                };
#pragma unroll 1
                for (int j0 = split; j0 < kDenseBags / 16; j0 += kAhead * splits) {   // (all of a short block's: no counts, no branches)
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) {
                        multiply_step(x[q], j0 + q * splits, GROUPS == 2 && (q & 1) ? acc2 : acc);
                        load_step(x[q], j0 + (q + kAhead) * splits);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (flags == 0u) break;
                if (upper) atomicOr(&S->flags, 4u);
                __syncthreads();
                const uint32_t fl = S->flags;
                if (digit == 0u && !(fl & 4u)) {        // no count has an upper byte: skip that pass
                    if (!(fl & 8u)) break;
                    ++pass;
                } else if (digit == 1u && !(fl & 8u)) {
                    break;
                }
#pragma unroll
                for (int q = 0; q < kAhead; ++q) load_step(x[q], split + q * splits);
            }
        }
        // ---- the wavefronts that shared a column group's bags, in order, then the rows' partial sums
        if constexpr (GROUPS == 2) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[m][r] += acc2[m][r];
        }
#pragma unroll 1
        for (int sp = 1; sp < splits; ++sp) {
            uint32_t rp = 32u * (uint32_t)GROUPS;
            asm volatile("" : "+s"(rp));
            float* const red = reinterpret_cast<float*>(s_cnt) + 4u * (uint32_t)kh * rp + (uint32_t)(cg * 32 + (lane & 31));
            __syncthreads();
            if (split == sp) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[(uint32_t)(m * 32 + (r & 3) + 8 * (r >> 2)) * rp] = acc[m][r];
            }
            __syncthreads();
            if (split == 0) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[m][r] += red[(uint32_t)(m * 32 + (r & 3) + 8 * (r >> 2)) * rp];
            }
        }
        if (split == 0 && col_on) {
            const bool add = k0 > k_lo;
            uint32_t row_floats = (uint32_t)D;
            int left = (int)nd - 4 * kh;
            asm volatile("" : "+s"(row_floats), "+v"(left));
            uint32_t at = (uint32_t)(4 * kh) * row_floats + (uint32_t)col;
#pragma unroll
            for (int m = 0; m < MT; ++m, at += 32u * row_floats) {
                if (add) {
                    float o[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int h = (r & 3) + 8 * (r >> 2);
                        o[r] = sums[m * 32 + h < left ? at + (uint32_t)h * row_floats : (uint32_t)col];
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[m][r] += o[r];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int h = (r & 3) + 8 * (r >> 2);
                    if (m * 32 + h < left) sums[at + (uint32_t)h * row_floats] = acc[m][r];
                }
            }
        }
    }
}

template <int GROUPS, bool MEAN, typename GT>
__device__ __forceinline__ void dense_any_narrow(const SegArgs& a, const uint32_t chunk, const int t, const uint32_t nd, const uint2 tab,
                                                 const int d0, const int D, DenseLds* S) {
    if (nd > 96u) dense_run_narrow<4, GROUPS, MEAN, GT>(a, chunk, t, nd, tab, d0, D, S);
    else if (nd > 64u) dense_run_narrow<3, GROUPS, MEAN, GT>(a, chunk, t, nd, tab, d0, D, S);
    else if (nd > 32u) dense_run_narrow<2, GROUPS, MEAN, GT>(a, chunk, t, nd, tab, d0, D, S);
    else dense_run_narrow<1, GROUPS, MEAN, GT>(a, chunk, t, nd, tab, d0, D, S);
}

template <bool MEAN, typename GT>
__global__ __launch_bounds__(kDThreads, 2) void seg_dense_kernel(const SegArgs a, const uint32_t col_blocks) {
    __shared__ DenseLds S;
    uint32_t bx = blockIdx.x;
    const uint32_t cb = bx % col_blocks;
    bx /= col_blocks;
    const uint32_t chunk = bx % a.dense_chunks;
    const int t = (int)(bx / a.dense_chunks);
    const uint32_t nd = a.dense_n[t];
    const uint2 tab = a.dense_tab[t];   // (with dense_n's load, not behind it; written where nd is not 0)
    if (nd == 0u) return;
    const int d0 = a.D_off[t];
    const int D = a.D_off[t + 1] - d0;
    if ((int)cb * 256 >= D) return;
    if (D <= 32) return dense_any_narrow<1, MEAN, GT>(a, chunk, t, nd, tab, d0, D, &S);
    if (D <= 64) return dense_any_narrow<2, MEAN, GT>(a, chunk, t, nd, tab, d0, D, &S);
    if (nd > 96u) dense_run<4, MEAN, GT>(a, cb, chunk, t, nd, tab, d0, D, &S);
    else if (nd > 64u) dense_run<3, MEAN, GT>(a, cb, chunk, t, nd, tab, d0, D, &S);
    else if (nd > 32u) dense_run<2, MEAN, GT>(a, cb, chunk, t, nd, tab, d0, D, &S);
    else dense_run<1, MEAN, GT>(a, cb, chunk, t, nd, tab, d0, D, &S);
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
