// Forward: pooled lookup, one wavefront per bag.
//
// A bag's rows are D_t * sizeof(weight) contiguous bytes each (128 B .. 1 KB for the shapes of interest),
// so a 64-lane wavefront would waste most lanes on one row.  The wavefront is therefore split into
// G = 64 / LPR groups of LPR lanes, LPR = D_t / kVec lanes covering one row with one 16-byte load per
// lane; the groups walk the bag in an interleaved fashion, four rows per group in flight, and a
// butterfly over the groups folds the partial sums at the end.  The bag's ids are read with one
// coalesced 64-wide load and handed to the groups with cross-lane reads.
#include <type_traits>

#include "tbe_device.h"
#include "tbe_internal.h"

namespace tbe {

constexpr int kFwdThreads = 256;

// Lane-group classes: a bag with more ids than this is walked by a whole wavefront instead of one lane group.  The
// more bags share a wavefront, the more lanes one long bag keeps waiting, so the bound falls with the lanes per row
// (measured at lognormal bag lengths, 8 bags per wavefront: 2.28 ms without, 2.07 / 2.01 / 1.94 / 1.86 ms at 96 / 64 /
// 48 / 32; a bound below the typical length would send ordinary bags the slower way).
__device__ __forceinline__ int long_bag_min(const int lanes_per_row) {
    return lanes_per_row > 16 ? 64 : (lanes_per_row > 8 ? 48 : 32);
}
// Of a table whose ordinary bags are that long themselves a lane group walks them all the same: only bags of more than twice the
// table's mean length are long, and those of more than kLongBagMax ids.  The mean is the table's own: one table of bags of 100 ids among
// 25 of 5, 32 fp32 columns, us, class bounds alone / twice the mean of the whole batch / of the table: 4096 bags 908 / 71 / 28, 65536
// bags 1145 / 1153 / 189.  Class bounds alone against this: 17000 bags of 40 ids, 32 fp32 columns 444 / 13; 26 tables x 4096 bags,
// 1 + Poisson(30) ids, 64 binary16 columns 283 / 43; of 100 ids, 128 fp32 columns 2625 / 318 (part of that by the shorter runs of
// long_scan_log2).  Bags of 200 ids with the limit at 128 / 512: 17000 bags, 32 columns 37 / 53 us, 16 tables x 32768 bags 1084 / 715.
constexpr int kLongBagMax = 128;
// len: of a bag above long_bag_min; lookups: ids of its table (of a malformed offsets array any number, and any answer will do)
__device__ __forceinline__ bool long_bag(const int len, const int64_t lookups, const int32_t B) {
    return len > kLongBagMax || (uint64_t)(uint32_t)len * (uint32_t)B > 2u * (uint64_t)lookups;
}
// the same as a bound, for a kernel that needs it before it has seen a bag
__device__ __forceinline__ int long_bag_bound(const int lanes_per_row, const int64_t lookups, const int32_t B) {
    int mean2 = 0;   // the largest number up to kLongBagMax that is at most twice the mean
#pragma unroll
    for (int step = kLongBagMax; step > 0; step >>= 1)
        if (mean2 + step <= kLongBagMax && (uint64_t)(uint32_t)(mean2 + step) * (uint32_t)B <= 2u * (uint64_t)lookups) mean2 += step;
    const int least = long_bag_min(lanes_per_row);
    return least > mean2 ? least : mean2;
}
// first position and ids of bag b of table t (0 ids from bag B on), clamped so that a malformed offsets array can never take a read
// outside indices[0, nnz); positions are below 2^32
struct BagSpan {
    uint32_t start;
    int len;
};
__device__ __forceinline__ BagSpan bag_span(const IdxView offsets, const int32_t t, const int32_t B, const uint32_t b, const int64_t nnz) {
    BagSpan r{0u, 0};
    if (b < (uint32_t)B) {
        const int64_t bag = (int64_t)t * B + b;
        int64_t start = offsets[bag], end = offsets[bag + 1];
        start = start < 0 ? 0 : (start > nnz ? nnz : start);
        end = end < start ? start : (end > nnz ? nnz : end);
        r.start = (uint32_t)start;
        r.len = (int)((end - start) < (int64_t)0x7FFFFFFF ? (end - start) : (int64_t)0x7FFFFFFF);
    }
    return r;
}
__device__ __forceinline__ int64_t table_lookups(const IdxView offsets, const int32_t t, const int32_t B) {
    return offsets[(int64_t)(t + 1) * B] - offsets[(int64_t)t * B];
}

// NC = number of 64-lane column chunks a row needs (1 when D <= 64 * kVec); U = rows in flight per group.
// The pooled value that is stored: the sum, or for mean pooling sum / L - the product with the reciprocal, corrected
// once by its exact residual (the usual refinement step of a division), so that a mean that is exactly representable
// (a bag whose ids are all equal, say) comes out exact and a 16-bit `out` rounds it the way the definition does.
// An empty bag has L = 0 and inv = 0: the result is the (zero) sum.
template <bool MEAN>
__device__ __forceinline__ float pooled(const float sum, const float L, const float inv) {
    if (!MEAN) return sum;
    const float q = sum * inv;
    return fmaf(fmaf(-q, L, sum), inv, q);
}

template <typename WT, int NC, int U, bool MEAN>
__device__ __forceinline__ void forward_bag(const WT* __restrict__ table, const int D, const int64_t R,
                                            const IdxView indices, const int64_t start, const int64_t end,
                                            void* __restrict__ out, const int out_io, const int64_t out_elem,
                                            int32_t* err) {
    constexpr int V = RowIO<WT>::kVec;
    using raw_t = typename RowIO<WT>::raw_t;
    const int lane = lane_id();
    const int nl = (D + V - 1) / V;  // lanes needed by one row
    const int LPR = nl >= kWave ? kWave : pow2ceil64(nl);
    const int G = kWave / LPR;
    const int sub = lane / LPR;
    const int lc = (lane & (LPR - 1)) * V;

    float acc[NC][V];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[c][v] = 0.f;

    for (int64_t base = start; base < end; base += kWave) {
        const int n = (int)((end - base) < (int64_t)kWave ? (end - base) : (int64_t)kWave);
        int32_t my = -1;
        if (lane < n) {
            const int64_t id = indices[base + lane];
            if (id >= 0 && id < R) my = (int32_t)id;
            else atomicOr(err, 1);
        }
        for (int k0 = 0; k0 < n; k0 += U * G) {
            raw_t x[U][NC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * G + sub;
                const int32_t got = __shfl(my, k & (kWave - 1), kWave);
                const int32_t id = (k < n) ? got : -1;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int col = lc + c * kWave * V;
                    x[u][c] = (id >= 0 && col < D) ? RowIO<WT>::load_raw(table + (int64_t)id * D + col)
                                                   : RowIO<WT>::zero_raw();
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < NC; ++c) RowIO<WT>::accumulate(x[u][c], acc[c]);
        }
    }
    // fold the groups
    for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[c][v] += __shfl_xor(acc[c][v], o, kWave);
    }
    float scale = 1.f, lenf = 0.f;
    if (MEAN) {
        const int64_t L = end - start;
        lenf = (float)L;
        scale = L > 0 ? 1.f / lenf : 0.f;
    }
    if (sub == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int col = lc + c * kWave * V;
            if (col < D) {
#pragma unroll
                for (int v4 = 0; v4 < V; v4 += 4) {
                    store4_from_float(out, out_io, out_elem + col + v4, pooled<MEAN>(acc[c][v4], lenf, scale),
                                      pooled<MEAN>(acc[c][v4 + 1], lenf, scale), pooled<MEAN>(acc[c][v4 + 2], lenf, scale),
                                      pooled<MEAN>(acc[c][v4 + 3], lenf, scale));
                }
            }
        }
    }
}

// One kernel per NC so that the common narrow-row case (NC = 1) keeps its register count low enough for
// 8 wavefronts per SIMD; the host launches one per width class that has tables.  `tables_of_class` lists the
// tables this launch covers (those whose rows need more than 64 * (NC / 2) and at most 64 * NC lanes).
template <typename WT, int NC, int U, bool MEAN>
__global__ __launch_bounds__(kFwdThreads, NC * U <= 4 ? 8 : 4) void forward_kernel(
    const WT* __restrict__ weights, const IdxView indices, const IdxView offsets,
    const int32_t* __restrict__ D_off, const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base,
    const int32_t* __restrict__ tables_of_class, const int32_t n_tables, const int32_t B, const int64_t nnz,
    const int32_t sumD, void* __restrict__ out, const int out_io, int32_t* err) {
    const uint32_t q = blockIdx.x * (kFwdThreads / kWave) + (threadIdx.x >> 6);   // (bags in all: below 2^31)
    const uint32_t i = q / (uint32_t)B;
    if (i >= (uint32_t)n_tables) return;
    const int32_t t = tables_of_class[i];
    const int32_t b = (int32_t)(q - i * (uint32_t)B);
    const int64_t bag = (int64_t)t * B + b;
    const int32_t d0 = D_off[t];
    const int D = D_off[t + 1] - d0;
    const int64_t R = row_base[t + 1] - row_base[t];
    // clamped so that a malformed offsets array can never take a read outside indices[0, nnz)
    int64_t start = offsets[bag];
    int64_t end = offsets[bag + 1];
    start = start < 0 ? 0 : (start > nnz ? nnz : start);
    end = end < start ? start : (end > nnz ? nnz : end);
    forward_bag<WT, NC, U, MEAN>(weights + w_off[t], D, R, indices, start, end, out, out_io, (int64_t)b * sumD + d0, err);
}

// Bags of more than long_bag_min ids that a lane group walks all the same: a single running sum of up to 128 terms would have up to
// 2.5 times the error of the 2 to 16 interleaved ones of a whole wavefront, so such a bag's sum is moved to a 64-bit total every
// 8 ids, or 16 of rows of 32 lanes.  Wavefronts without such a bag take the loop without totals.  rms error of fp32 rows (normal
// values, units of 2^-24), one running sum / a whole wavefront / this: 40 ids of 32 columns 12.5 / 7.0 / 6.6, 62 of 64 19.2 / 11.2 /
// 8.1, 100 of 8 30.6 / 11.9 / 8.1, 100 of 128 30.8 / 22.4 / 13.4.  The totals cost 3 to 15 % of launches of such bags: 26 tables x 4096
// bags, 1 + Poisson(30) ids, 64 binary16 columns 40.1 -> 42.3 us, 17000 bags of 40 ids, 32 columns 13.1 -> 13.5; nothing elsewhere.
__device__ __forceinline__ bool split_run_ends(const int k, const int lpr_log2) {   // k ids of a round of 2^lpr_log2 are summed
    return (k & (lpr_log2 >= 5 ? 15 : 7)) == 0;
}
template <bool SPLIT, int V>
struct Totals {
    __device__ __forceinline__ void add(float (&)[V], bool) {}
    __device__ __forceinline__ void finish(float (&)[V], bool) {}
};
template <int V>
struct Totals<true, V> {
    double sum[V];
    __device__ __forceinline__ Totals() {
#pragma unroll
        for (int v = 0; v < V; ++v) sum[v] = 0.0;
    }
    __device__ __forceinline__ void add(float (&acc)[V], const bool split) {   // `split`: of this lane's bag
#pragma unroll
        for (int v = 0; v < V; ++v) {
            sum[v] += split ? (double)acc[v] : 0.0;
            acc[v] = split ? 0.f : acc[v];
        }
    }
    __device__ __forceinline__ void finish(float (&acc)[V], const bool split) const {
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = split ? (float)sum[v] : acc[v];
    }
};

constexpr int kGroupThreads = 256;   // of the kernel of plain lane groups
// ... in LDS, for a kernel that can spare it: [V][threads of the workgroup]
template <bool SPLIT, int V>
struct LdsTotals {
    __device__ __forceinline__ LdsTotals(double (*)[kGroupThreads]) {}
    __device__ __forceinline__ void add(float (&)[V], bool) {}
    __device__ __forceinline__ void finish(float (&)[V], bool) {}
};
template <int V>
struct LdsTotals<true, V> {
    double (*sum)[kGroupThreads];
    __device__ __forceinline__ LdsTotals(double (*s)[kGroupThreads]) : sum(s) {
#pragma unroll
        for (int v = 0; v < V; ++v) sum[v][threadIdx.x] = 0.0;
    }
    __device__ __forceinline__ void add(float (&acc)[V], const bool split) {
        if (!split) return;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            __hip_atomic_fetch_add(&sum[v][threadIdx.x], (double)acc[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            acc[v] = 0.f;
        }
    }
    __device__ __forceinline__ void finish(float (&acc)[V], const bool split) const {
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = split ? (float)sum[v][threadIdx.x] : acc[v];
    }
};

// Narrow rows (at most 32 lanes per row): every lane group of the wavefront takes a bag of its own, G = 64 / LPR bags of one table per
// wavefront.  A bag of a dozen narrow rows is a few hundred bytes; with one wavefront per bag the step is bound by the latency of the
// offsets -> ids -> rows chain, not by bandwidth.  A group reads LPR ids with one coalesced load, then walks them U rows at a time.
// BY_LENGTH: the workgroup hands its bags out by length, longest first, so that those that share a wavefront are of a length: a
// wavefront walks as far as the longest of its bags.  Every wavefront finds the order of all of them by itself, and none where they are of
// one length, so that the workgroup's wavefronts never wait for each other (with counts in LDS and four barriers instead, bags of one to
// five ids took 6 to 14 % longer than consecutive ones).  Consecutive bags / this, us: 32 tables x 65536 bags, lognormal of 12 ids on
// average, 2 of 128 and 30 of 32 fp32 columns 481 / 414; 16 tables x 32768 bags: 8 fp32 columns, lognormal of 12 and 35 ids 94 201 / 82
// 173; 32 fp32 122 297 / 111 258, 1 + Poisson(30) 133 / 126, fixed 5 and 40 36.6 156 / 36.7 156; 64 binary16, lognormal 171 344 / 162 324;
// 8192 bags of 128 fp32, Poisson(3) 34.7 / 35.6, fixed 3 33.9 / 32.8.  Several such rounds per workgroup level the lengths further (the
// first 372 with 8) but spread the workgroups that run at a time over more tables: fixed 40 of 32 fp32 columns 169, 179, 190 with 2, 4, 8
// of them; workgroups of 512 threads 432 at the first.
// Place of every lane's number, below 2^bits, among those of the lanes `in`, the largest first, equal ones by lane: a bit at a time from
// the top, the lanes that agree so far and have a bit that this one lacks come before it.
__device__ __forceinline__ uint32_t place_by_size(const uint32_t x, const int bits, const uint64_t in) {
    uint32_t lo = (uint32_t)in, hi = (uint32_t)(in >> 32), place = 0;
#pragma unroll 1
    for (int b = bits - 1; b >= 0; --b) {
        const uint32_t has = (uint32_t)__builtin_amdgcn_sbfe((int)x, b, 1);   // all ones or nothing
        const uint64_t m = __builtin_amdgcn_uicmp(has, 0u, 33 /* != */);
        const uint32_t before = (uint32_t)__popc(lo & (uint32_t)m) + (uint32_t)__popc(hi & (uint32_t)(m >> 32));
        place += before & ~has;
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, has, 0x90);           // lo & ~(m ^ has)
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), has, 0x90);
    }
    return place + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
}
static_assert(kLongBagMax < 256 && kGroupThreads / 4 <= kWave, "a length in a byte, a workgroup's bags in the lanes of a wavefront");
template <typename WT, int U, bool MEAN, bool BY_LENGTH, bool STREAM>
__global__ __launch_bounds__(kGroupThreads, 8) void forward_groups_kernel(
    const WT* __restrict__ weights, const IdxView indices, const IdxView offsets,
    const int32_t* __restrict__ D_off, const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base,
    const int32_t* __restrict__ tables_of_class, const int32_t n_tables, const int lpr_log2, const int32_t B,
    const int64_t nnz, const int32_t sumD, void* __restrict__ out, const int out_io, int32_t* err) {
    constexpr int V = RowIO<WT>::kVec;
    using raw_t = typename RowIO<WT>::raw_t;
    __shared__ double s_total[V][kGroupThreads];
    const int lane = lane_id();
    const int LPR = 1 << lpr_log2;
    const int G = kWave >> lpr_log2;
    const int sub = lane >> lpr_log2;
    const int li = lane & (LPR - 1);        // lane inside its group
    const int lc = li * V;
    const int wv = (int)(threadIdx.x >> 6);
    // ---- the table, and the first bag of this wavefront or (BY_LENGTH) workgroup
    const int bags = BY_LENGTH ? kGroupThreads >> lpr_log2 : G;
    const int64_t per_table = ((int64_t)B + bags - 1) / bags;   // wavefronts or workgroups per table
    const int64_t wid = BY_LENGTH ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * (kGroupThreads / kWave) + wv;
    const int64_t i = wid / per_table;
    if (i >= n_tables) return;
    const int32_t t = __builtin_amdgcn_readfirstlane(tables_of_class[i]);   // (the same for the wavefront: its table's numbers stay scalar)
    const uint32_t b0 = (uint32_t)((wid - i * per_table) * bags);   // (below 2^31)
    const int32_t d0 = D_off[t];
    const int D = D_off[t + 1] - d0;
    const int64_t R = row_base[t + 1] - row_base[t];
    const WT* table = weights + w_off[t];
    const bool col_on = lc < D;
    // a bag far longer than its neighbours would keep the other groups of the wavefront waiting: such bags are left to
    // forward_long_bags_kernel, where a whole wavefront walks one bag
    const int long_min = long_bag_min(LPR);
    uint32_t b = b0 + (uint32_t)sub, start;
    int len;
    bool is_long = false;
    if constexpr (BY_LENGTH) {
        // every wavefront by itself, without a barrier: a lane per bag of the workgroup
        const BagSpan bag = bag_span(offsets, t, B, b0 + umin((uint32_t)lane, (uint32_t)bags - 1u), nnz);
        bool lng = false;
        if (__any(bag.len > long_min)) lng = bag.len > long_min && long_bag(bag.len, table_lookups(offsets, t, B), B);
        const uint32_t my_len = lng ? 0u : (uint32_t)bag.len;
        uint32_t word = my_len | (lng ? 256u : 0u) | (uint32_t)lane << 16;
        start = bag.start;
        if (__ballot(my_len != (uint32_t)__builtin_amdgcn_readfirstlane((int)my_len)) != 0ull) {   // (a bag's sum does not depend on those beside it)
            const uint64_t in = bags == kWave ? ~0ull : (1ull << bags) - 1ull;
            const uint32_t place = place_by_size(my_len, 32 - __clz(wave_max_i32((int)my_len)), in);
            const int to = 4 * (int)(lane < bags ? place : (uint32_t)lane);
            word = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)word);
            start = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)start);
        }
        word = __shfl(word, wv * G + sub, kWave);
        start = __shfl(start, wv * G + sub, kWave);
        b = b0 + (word >> 16);
        len = (int)(word & 0xFFu);
        is_long = (word & 256u) != 0u;
    } else {
        const BagSpan bag = bag_span(offsets, t, B, b, nnz);
        start = bag.start;
        len = bag.len;
        if (__any(len > long_min)) is_long = len > long_min && long_bag(len, table_lookups(offsets, t, B), B);
        len = is_long ? 0 : len;
    }
    const bool split = len > long_min;
    const bool has_bag = b < (uint32_t)B;
    const int maxlen = wave_max_i32(len);   // longest bag of the wavefront: the loop bounds below are wave-uniform
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    auto walk = [&](auto split_c) {
        constexpr bool kSplit = decltype(split_c)::value;
        LdsTotals<kSplit, V> total(s_total);
        for (int base = 0; base < maxlen; base += LPR) {
            int32_t my = -1;
            if (base + li < len) {
                const int64_t id = indices[(int64_t)start + base + li];
                if (id >= 0 && id < R) my = (int32_t)id;
                else atomicOr(err, 1);
            }
            const int nk = maxlen - base < LPR ? maxlen - base : LPR;
            for (int k0 = 0; k0 < nk; k0 += U) {
                raw_t x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    // cross-lane read outside any lane-dependent condition; lanes of a finished bag read -1
                    const int32_t id = __shfl(my, (sub << lpr_log2) + ((k0 + u) & (LPR - 1)), kWave);
                    const bool on = (k0 + u) < nk && id >= 0 && col_on;
                    x[u] = on ? RowIO<WT>::load_raw(table + (int64_t)id * D + lc) : RowIO<WT>::zero_raw();
                }
#pragma unroll
                for (int u = 0; u < U; ++u) RowIO<WT>::accumulate(x[u], acc);
                if (kSplit && (split_run_ends(k0 + U, lpr_log2) || k0 + U >= nk)) total.add(acc, split);
            }
        }
        total.finish(acc, split);
    };
    if (__any(split)) walk(std::true_type{});
    else walk(std::false_type{});
    const float lenf = (float)len;
    float scale = 1.f;
    if (MEAN) scale = len > 0 ? 1.f / lenf : 0.f;
    if (has_bag && col_on && !is_long) {
        const int64_t out_elem = (int64_t)b * sumD + d0 + lc;
        float y[V];
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] = pooled<MEAN>(acc[v], lenf, scale);
        if constexpr (V == 4) {
            store4_from_float<STREAM>(out, out_io, out_elem, y[0], y[1], y[2], y[3]);
        } else if (out_io != 0) {
            store8_from_float<STREAM>(out, out_io, out_elem, y);
        } else {
            store4_from_float(out, 0, out_elem, y[0], y[1], y[2], y[3]);
            store4_from_float(out, 0, out_elem + 4, y[4], y[5], y[6], y[7]);
        }
    }
}

// ---- the lane-group classes with the tables' hottest rows held in LDS --------------------------------------------
// In a skewed batch a hundred rows of a table take half of its lookups.  Their rows come from the L2, but every read
// that leaves a compute unit's vector L1 occupies one of its few dozen miss slots for the length of the trip, and it
// is those slots times the trip time that bound this kernel.  A workgroup of 16 wavefronts therefore takes a long run of
// consecutive bags of ONE table, copies the rows that the handle lists as the table's hottest (the rows that had the
// most lookups in the last backward call - a hint: any list of valid ids gives the same result) into LDS once, and
// serves every lookup of one of those rows from there.  A lookup finds out through a small open-addressing table of
// ids in LDS.  Per round of LPR ids a lane group first walks its cold ids (global loads, U rows in flight), then its
// hot ones (LDS reads); the two lists are compacted through an LDS stage, so that no lane issues a load it does not
// need.  The sum is taken in that order, which is fixed, so results do not depend on timing.
constexpr int kHotThreads = 1024;
constexpr int kHotWaves = kHotThreads / kWave;
constexpr int kHotTab = 1024;                // slots of the id table (at most kHotRows ids: a quarter full)
constexpr int kHotRowBytes = 64 << 10;       // LDS bytes for rows
constexpr int kHotPasses = 8;               // rounds of kHotWaves * G bags per workgroup
constexpr uint32_t kHotEmpty = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t hot_hash(const uint32_t id) { return (id * 0x9E3779B1u) >> 22; }   // 10 bits

template <typename WT, int U, bool MEAN>
__global__ __launch_bounds__(kHotThreads, 8) void forward_hot_kernel(
    const WT* __restrict__ weights, const IdxView indices, const IdxView offsets,
    const int32_t* __restrict__ D_off, const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base,
    const int32_t* __restrict__ tables_of_class, const int32_t n_tables, const int lpr_log2, const int32_t B,
    const int64_t nnz, const int32_t sumD, void* __restrict__ out, const int out_io, int32_t* err,
    const uint32_t* __restrict__ hot_ids, const uint32_t* __restrict__ hot_n, const int32_t chunks_per_table) {
    constexpr int V = RowIO<WT>::kVec;
    using raw_t = typename RowIO<WT>::raw_t;
    __shared__ raw_t s_rows[kHotRowBytes / 16];
    __shared__ uint32_t s_tab_id[kHotTab];
    __shared__ uint16_t s_tab_slot[kHotTab];
    __shared__ uint32_t s_ids[kHotRows];
    __shared__ uint32_t s_n;
    __shared__ int64_t s_lookups;
    __shared__ uint32_t s_cold[kHotWaves][kWave];
    __shared__ uint16_t s_hot[kHotWaves][kWave];
    const int lane = lane_id();
    const int wv = threadIdx.x >> 6;
    const int LPR = 1 << lpr_log2;
    const int G = kWave >> lpr_log2;
    const int32_t i = (int32_t)(blockIdx.x / (uint32_t)chunks_per_table);
    const int32_t chunk = (int32_t)(blockIdx.x - (uint32_t)i * (uint32_t)chunks_per_table);
    if (i >= n_tables) return;
    const int32_t t = tables_of_class[i];
    const int sub = lane >> lpr_log2;
    const int li = lane & (LPR - 1);        // lane inside its group
    const int lc = li * V;
    const int32_t d0 = D_off[t];
    const int D = D_off[t + 1] - d0;
    const int64_t R = row_base[t + 1] - row_base[t];
    const WT* table = weights + w_off[t];
    const bool col_on = lc < D;
    // ---- the table's hot rows: id table, then the rows themselves (one lane group per row).  The list's length and
    // each listed id are read once, for both: a backward call over other tables of this shape may rewrite the list meanwhile,
    // and an id table that named one row where another, or none, was copied would give wrong sums.
    const int cap = (kHotRowBytes / 16) >> lpr_log2;
    if (threadIdx.x == 0) s_n = hot_n[t];
    if (threadIdx.x == kWave) s_lookups = table_lookups(offsets, t, B);
    for (int k = threadIdx.x; k < kHotTab; k += kHotThreads) s_tab_id[k] = kHotEmpty;
    __syncthreads();
    int nh = s_n < (uint32_t)kHotRows ? (int)s_n : kHotRows;
    nh = nh > cap ? cap : nh;
    if ((int)threadIdx.x < nh) {
        const uint32_t id = hot_ids[(size_t)t * kHotRows + threadIdx.x];
        s_ids[threadIdx.x] = id;
        if ((int64_t)id < R) {
            uint32_t hsh = hot_hash(id);
            for (;;) {   // ends: the table is at most a quarter full
                const uint32_t old = atomicCAS(&s_tab_id[hsh], kHotEmpty, id);
                if (old == kHotEmpty) {
                    s_tab_slot[hsh] = (uint16_t)threadIdx.x;
                    break;
                }
                if (old == id) break;   // listed twice: the first entry serves
                hsh = (hsh + 1u) & (kHotTab - 1u);
            }
        }
    }
    __syncthreads();
    for (int k = (int)(threadIdx.x >> lpr_log2); k < nh; k += kHotThreads >> lpr_log2) {
        const uint32_t id = s_ids[k];
        s_rows[(k << lpr_log2) + li] = ((int64_t)id < R && col_on) ? RowIO<WT>::load_raw(table + (int64_t)id * D + lc)
                                                                     : RowIO<WT>::zero_raw();
    }
    __syncthreads();
    // ---- the bags
    const uint32_t gmask = LPR >= 32 ? 0xFFFFFFFFu : ((1u << LPR) - 1u);   // (LPR <= 32 in these classes)
    const uint32_t below = (1u << li) - 1u;
    uint32_t* const cold = &s_cold[wv][sub << lpr_log2];
    uint16_t* const hot = &s_hot[wv][sub << lpr_log2];
    for (int pass = 0; pass < kHotPasses; ++pass) {
        const uint32_t b0 = (uint32_t)((chunk * kHotPasses + pass) * kHotWaves + wv) * (uint32_t)G, b = b0 + (uint32_t)sub;
        if (b0 >= (uint32_t)B) break;   // (the same for all lanes)
        const bool has_bag = b < (uint32_t)B;
        const BagSpan bag = bag_span(offsets, t, B, b, nnz);
        const int full_len = bag.len;
        bool split = full_len > long_bag_min(LPR);
        const bool is_long = split && long_bag(full_len, s_lookups, B);   // left to forward_long_bags_kernel
        split = split && !is_long;
        const int len = is_long ? 0 : full_len;
        const int maxlen = wave_max_i32(len);
        float acc[V];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = 0.f;
        auto walk = [&](auto split_c) {
            constexpr bool kSplit = decltype(split_c)::value;
            constexpr int kU = kSplit ? (V == 8 ? 2 : 4) : U;   // the totals take the registers of the other rows   // rows in flight: the totals take the registers of the others
            Totals<kSplit, V> total;
            for (int base = 0; base < maxlen; base += LPR) {
                int32_t my = -1;
                if (base + li < len) {
                    const int64_t id = indices[(int64_t)bag.start + base + li];
                    if (id >= 0 && id < R) my = (int32_t)id;
                    else atomicOr(err, 1);
                }
                int slot = -1;
                if (my >= 0 && nh > 0) {
                    uint32_t hsh = hot_hash((uint32_t)my);
                    for (;;) {
                        const uint32_t tid = s_tab_id[hsh];
                        if (tid == kHotEmpty) break;
                        if (tid == (uint32_t)my) {
                            slot = (int)s_tab_slot[hsh];
                            break;
                        }
                        hsh = (hsh + 1u) & (kHotTab - 1u);
                    }
                }
                // this lane group's cold ids and hot slots, each list in bag order
                const bool is_cold = my >= 0 && slot < 0, is_hot = slot >= 0;
                const uint32_t mc = (uint32_t)(__ballot(is_cold) >> (sub << lpr_log2)) & gmask;
                const uint32_t mh = (uint32_t)(__ballot(is_hot) >> (sub << lpr_log2)) & gmask;
                if (is_cold) cold[__popc(mc & below)] = (uint32_t)my;
                if (is_hot) hot[__popc(mh & below)] = (uint16_t)slot;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const int nc = __popc(mc), nhh = __popc(mh);
                const int ncmax = wave_max_i32(nc), nhmax = wave_max_i32(nhh);
                for (int k0 = 0; k0 < ncmax; k0 += kU) {
                    raw_t x[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const uint32_t id = cold[(k0 + u) & (LPR - 1)];
                        const bool on = (k0 + u) < nc && col_on;
                        x[u] = on ? RowIO<WT>::load_raw(table + (int64_t)id * D + lc) : RowIO<WT>::zero_raw();
                    }
#pragma unroll
                    for (int u = 0; u < kU; ++u) RowIO<WT>::accumulate(x[u], acc);
                    if (kSplit && (split_run_ends(k0 + kU, lpr_log2) || k0 + kU >= ncmax)) total.add(acc, split);
                }
                for (int k0 = 0; k0 < nhmax; k0 += 4) {
                    raw_t x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int sl = hot[(k0 + u) & (LPR - 1)];
                        const bool on = (k0 + u) < nhh;
                        x[u] = on ? s_rows[(sl << lpr_log2) + li] : RowIO<WT>::zero_raw();
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) RowIO<WT>::accumulate(x[u], acc);
                    if (kSplit && (split_run_ends(k0 + 4, lpr_log2) || k0 + 4 >= nhmax)) total.add(acc, split);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the lists are free for the next round
            }
            total.finish(acc, split);
        };
        if (__any(split)) walk(std::true_type{});
        else walk(std::false_type{});
        const float lenf = (float)len;
        float scale = 1.f;
        if (MEAN) scale = len > 0 ? 1.f / lenf : 0.f;
        if (has_bag && col_on && !is_long) {
            const int64_t out_elem = (int64_t)b * sumD + d0 + lc;
#pragma unroll
            for (int v4 = 0; v4 < V; v4 += 4)
                store4_from_float(out, out_io, out_elem + v4, pooled<MEAN>(acc[v4], lenf, scale),
                                  pooled<MEAN>(acc[v4 + 1], lenf, scale), pooled<MEAN>(acc[v4 + 2], lenf, scale),
                                  pooled<MEAN>(acc[v4 + 3], lenf, scale));
        }
    }
}

// The long bags of the lane-group classes.  A wavefront looks at 2^scan_log2 consecutive bags of one table, at most 64 at
// a time with one bag per lane, and walks every bag with more than long_bag_min ids with all of its lanes
// (forward_bag, as for wide rows).  A kernel of its own: inside the lane-group kernel the second phase pushed the
// binary16 variant over its 64 registers (8.0 -> 9.3 ms at the largest workload).
template <typename WT, bool MEAN>
__global__ __launch_bounds__(kFwdThreads, 4) void forward_long_bags_kernel(
    const WT* __restrict__ weights, const IdxView indices, const IdxView offsets,
    const int32_t* __restrict__ D_off, const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base,
    const int32_t* __restrict__ tables_of_class, const int32_t n_tables, const int scan_log2, const int32_t B, const int64_t nnz,
    const int32_t sumD, void* __restrict__ out, const int out_io, int32_t* err) {
    constexpr int V = RowIO<WT>::kVec;
    const int lane = lane_id();
    const int64_t scan = (int64_t)1 << scan_log2;
    const int64_t per_table = ((int64_t)B + scan - 1) >> scan_log2;   // wavefronts per table
    const int64_t wid = (int64_t)blockIdx.x * (kFwdThreads / kWave) + (threadIdx.x >> 6);
    const int64_t i = wid / per_table;
    if (i >= n_tables) return;
    const int32_t t = __builtin_amdgcn_readfirstlane(tables_of_class[i]);   // (the same for the wavefront: its table's numbers stay scalar)
    const int32_t d0 = D_off[t];
    const int D = D_off[t + 1] - d0;
    // the bound of the table's class: lanes per row as the host classifies them (power of two, at least 4)
    const int nl = (D + V - 1) / V;
    const int bound = long_bag_bound(nl > 16 ? 32 : (nl > 8 ? 16 : (nl > 4 ? 8 : 4)), table_lookups(offsets, t, B), B);
    const int64_t first = (wid - i * per_table) << scan_log2;
    const int64_t last = first + scan < (int64_t)B ? first + scan : (int64_t)B;
    for (int64_t b0 = first; b0 < last; b0 += kWave) {   // (wave-uniform)
        const int64_t b = b0 + lane;
        int64_t start = 0, end = 0;
        if (b < last) {   // clamped as in the lane-group kernel
            const int64_t bag = (int64_t)t * B + b;
            start = offsets[bag];
            end = offsets[bag + 1];
            start = start < 0 ? 0 : (start > nnz ? nnz : start);
            end = end < start ? start : (end > nnz ? nnz : end);
        }
        uint64_t todo = __ballot(end - start > (int64_t)bound);
        while (todo != 0ull) {
            const int src = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1ull;
            const int64_t s = (int64_t)(((uint64_t)bcast_lane((uint32_t)((uint64_t)start >> 32), src) << 32) |
                                        (uint64_t)bcast_lane((uint32_t)((uint64_t)start & 0xFFFFFFFFull), src));
            const int64_t e = (int64_t)(((uint64_t)bcast_lane((uint32_t)((uint64_t)end >> 32), src) << 32) |
                                        (uint64_t)bcast_lane((uint32_t)((uint64_t)end & 0xFFFFFFFFull), src));
            forward_bag<WT, 1, 4, MEAN>(weights + w_off[t], D, row_base[t + 1] - row_base[t], indices, s, e, out,
                                                out_io, (b0 + src) * (int64_t)sumD + d0, err);
        }
    }
}

// A small batch is a matter of latency: one wavefront per bag then is the shortest chain (the lane groups of a narrow row's
// wavefront share one bag, and a long bag keeps nobody waiting), and the classes 0 to 4 take one launch instead of up to
// six.  Lane groups need fewer wavefronts and win back what the longer chain costs from some number of bags on: the sooner,
// the narrower the rows (more bags per wavefront) and the shorter the bags (less to walk for a group of lanes).  The border
// follows the measured break-even by the narrowest rows of the handle and the mean bag length.  Lane groups against one
// wavefront per bag, us, at 4096 / 8192 / 16384 bags (100000 rows, Zipf 1.05):
//   8 fp32 columns       1 id  6.0 4.4 / 6.0 5.4 / 6.1 8.1     3 ids 7.5 4.3 / 7.7 5.4 / 7.7 8.0     10 ids 10.2 4.3 / 10.1 5.4 / 10.3 8.0
//   16 binary16 columns  1 id  6.2 5.3 / 6.2 7.1 / 6.3 10.9    3 ids 7.8 5.3 / 8.0 7.1 / 8.0 10.9    10 ids 10.5 5.2 / 10.5 7.1 / 10.7 10.9
//   64 fp32 columns      1 id  6.1 4.1 / 6.5 5.2 / 7.2 7.8     3 ids 6.8 4.1 / 7.1 5.2 / 7.7 8.0     10 ids 7.9 4.5 / 8.3 5.7 / 10.4 9.5
//   256 binary16 columns 1 id  7.1 4.6 / 8.4 6.1 / 11.5 9.5    3 ids 7.5 4.8 / 9.4 6.2 / 12.9 10.3   10 ids 9.2 5.5 / 11.5 8.2 / 16.3 13.5
// Lognormal lengths, 32 columns, 16384 bags: 73 against 13 us.
constexpr int64_t kFwdSmallBags = 16384;
// (not with the hot rows asked for at every size: they live in the lane-group classes)
static bool forward_small(const tbe_handle* h, const int32_t B, const int64_t nnz) {
    const int64_t bags = (int64_t)(h->fwd_first[5] - h->fwd_first[0]) * B;   // of rows of at most 64 lanes, classes 0 to 4
    if (h->hot_min_workgroups == 0 || bags > kFwdSmallBags) return false;
    const double ids = (double)nnz / ((double)h->T * B);
    double border = 12288.0 + 1024.0 * ids;
    if (h->fwd_count[3] + h->fwd_count[4] > 0)   // rows of at most 8 lanes
        border = h->dtype == TBE_F32 ? 7168.0 + 2560.0 * ids : 5120.0 + 1280.0 * ids;
    return (double)bags <= border;
}
// Rows in flight per lane group: 4 leaves registers for 8 wavefronts per SIMD and covers most bags in one round; 8 pay where
// every row takes at least half a wavefront and bags are long (256 fp32 columns, 16384 bags: 40 ids 45.9 -> 44.5 us, but 1
// id 8.6 -> 9.7).
static bool forward_small_long(const tbe_handle* h, const int32_t B, const int64_t nnz) {
    return h->fwd_count[2] + h->fwd_count[3] + h->fwd_count[4] == 0 && nnz >= (int64_t)24 * h->T * B;
}
// Workgroups from which the lane-group classes 1 (32 lanes per row) and 2 (16) keep hot rows in LDS where no tunable says so:
// 512 of its large workgroups run at a time, so a launch needs some rounds of them before LDS hits outweigh the last, part-filled
// one and the copying of the rows.  Plain lane groups against hot rows, us (Zipf 1.2, the list filled by a backward call):
//   128 fp32 columns, 1 + Poisson(30) ids   416 workgroups 92 101   640 132 137   768 189 173   1664 361 296
//   256 binary16 columns, the same          416 121 126             640 173 174   768 229 198   1664 442 377
//   64 fp32 columns, the same               384 94 108              832 200 199
//   64 fp32 columns, 1 + Poisson(10) ids    384 44 53               832 100 99    3840 488 388
//   128 binary16 columns, the same          384 52 69               832 147 146   3840 640 520
// Rows of at most 8 lanes gain nothing at any size (1 + Poisson(10) ids): 32 fp32 columns 416 workgroups 51 69, 1920 278 275; 64
// binary16 columns 416 58 94, 1920 359 359.
constexpr int64_t kHotWorkgroups[2] = {768, 1024};
// workgroups per table with which the lane-group class c keeps hot rows in LDS; 0: it does not
static int hot_chunks(const tbe_handle* h, const int c, const int32_t B) {
    const bool by_class = h->hot_min_workgroups == TBE_TUNE_AUTO;
    if (!h->d_hot_ids || (by_class ? c > 2 : h->hot_min_workgroups < 0)) return 0;
    const int64_t bags_per_wg = (int64_t)kHotPasses * kHotWaves * (kWave >> (6 - c));
    const int cpt = (int)(((int64_t)B + bags_per_wg - 1) / bags_per_wg);
    return (int64_t)h->fwd_count[c] * cpt >= (by_class ? kHotWorkgroups[c - 1] : h->hot_min_workgroups) ? cpt : 0;
}
// Bags that a wavefront of forward_long_bags_kernel looks at: 256 where that fills the chip, fewer (down to 4) in smaller
// batches, where long bags would wait for one another in a few wavefronts.  Lognormal bags of 35 ids on average, us, 256 bags a
// wavefront -> this: 26 tables x 4096 bags x 32 fp32 columns 324 -> 82, 16 tables x 32768 bags 470 -> 347; where no bag is long
// the launch takes 4.4 us either way.
constexpr int64_t kLongScanWaves = 4096;
static int long_scan_log2(const int64_t bags) {
    int l = 2;
    while (l < 8 && (bags >> (l + 1)) >= kLongScanWaves) ++l;
    return l;
}
unsigned forward_kernels(const tbe_handle* h, const int32_t B, const int64_t nnz) {
    unsigned m = h->fwd_count[5] + h->fwd_count[6] > 0 ? TBE_FWD_WAVEFRONT_PER_BAG : 0u;
    if (forward_small(h, B, nnz)) return h->fwd_first[5] > 0 ? m | TBE_FWD_WAVEFRONT_PER_BAG : m;
    if (h->fwd_count[0] > 0) m |= TBE_FWD_WAVEFRONT_PER_BAG;
    for (int c = 1; c < 5; ++c)
        if (h->fwd_count[c] > 0) m |= TBE_FWD_LONG_BAGS | (hot_chunks(h, c, B) > 0 ? TBE_FWD_HOT_ROWS : TBE_FWD_LANE_GROUPS);
    return m;
}

template <typename WT, int NC, int U>
static void launch_forward_nc(const tbe_handle* h, int first, int n, const void* tables, const int32_t* d_D_off,
                              const IdxView indices, const IdxView offsets, int32_t B, int64_t nnz, bool mean, void* out,
                              int out_io, hipStream_t s) {
    if (n == 0) return;
    const int32_t* list = h->d_fwd_tables + first;
    const int wpb = kFwdThreads / kWave;
    const dim3 grid((unsigned)(((int64_t)n * B + wpb - 1) / wpb));
    const WT* w = static_cast<const WT*>(tables);
    if (mean)
        forward_kernel<WT, NC, U, true><<<grid, kFwdThreads, 0, s>>>(w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base,
                                                                     list, n, B, nnz, h->sumD, out, out_io, h->d_err);
    else
        forward_kernel<WT, NC, U, false><<<grid, kFwdThreads, 0, s>>>(w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base,
                                                                      list, n, B, nnz, h->sumD, out, out_io, h->d_err);
}

// A launch of lane groups hands bags out by length if it has as many workgroups as the chip holds at a time - smaller ones gain nothing
// by it that can be told from the noise: 8 tables x 4096 bags, 1 + Poisson(10) ids, 8 fp32 columns 13.9 / 14.0 us, 64 binary16 14.1 / 13.6,
// 64 fp32 14.5 / 14.2 - and if the bags are long enough on average for what they then save each other.  The order is a chain of a few
// hundred cycles for every wavefront, and two bags beside each other have less to save than sixteen: hence the square of the lanes per
// row.  64 tables x 16384 bags, for 32 lanes 26 x 4096, of 100 rows, fp32, Poisson(3), (8), (25), lognormal of mean 1.3, 3, 7, 20, not / by
// length: 4 lanes 48 67 140, 50 78 117 232 / 45 62 127, 51 66 97 197; 8 lanes 67 90 177, 68 95 143 293 / 70 87 162, 73 92 128 259; 16 lanes
// (26 x 4096) 18.8 23.1 40.5, 22.0 27.2 38.8 72 / 20.4 23.6 39.4, 23.4 28.5 38.3 68; 32 lanes 30.5 37.2 60.6, 30.7 49.7 58.0 102 / 32.7 38.3
// 59.8, 32.3 52.0 59.0 99.  Of 100000 rows, which are fetched from further away, 8 lanes 106 189 497, 87 141 227 487 / 100 184 514, 85 124 209
// 470, 16 and 32 lanes 0 to 4 % slower below a mean of 7, then the same.
constexpr int64_t kByLengthWorkgroups = 2048;
static bool by_length(const int64_t workgroups, const int64_t lookups, const int64_t bags, const int lpr) {
    return workgroups >= kByLengthWorkgroups && lookups >= bags * (lpr * lpr) / 32;   // (of the whole batch: the host does not know whose they are)
}
// Do the lane groups of class c write their parts of the output past the caches, which are then left to the rows?  Not where that leaves
// parts of 64-byte pieces to other workgroups, which are then fetched and written again: 26 tables x 32768 bags of one id, us, plain / past
// the caches: 12 fp32 columns 33.5 / 51, 28 55 / 83, 4 and 8 columns into bfloat16 34 / 36; but 16 columns, 64 bytes, 33.5 / 33, of 5 and 10
// ids 51 / 48 and 70 / 66.  And wider parts not where the output is small enough for its reader to find it in a cache: forward and one
// kernel that reads its output, 14, 27, 54, 80, 109 MB of 64 to 512 bytes a part: 0.91 to 1.0, 0.96 to 1.0, 0.95 to 1.04, 0.99 to 1.04,
// 0.98 to 1.06 times as fast (the forward alone 1.01 to 1.06, 1.01 to 1.05, 1.0 to 1.1, 1.0 to 1.2, 1.0 to 1.2; of 64 tables x 3001 bags of 31
// ids, 128 and 256 binary16 columns into binary16, 86 MB, 198 -> 192 us).  Parts of 64 bytes gain both, 1.0 to 1.03, from the smallest on.
constexpr size_t kLargeOutput = (size_t)48 << 20;   // bytes
static bool stream_output(const tbe_handle* h, const int c, const int32_t B, const void* out, const int out_io) {
    const size_t eb = out_io == 0 ? 4 : 2, pitch = (size_t)h->sumD * eb;
    if (h->dtype == TBE_F16 && out_io == 0) return false;   // (a lane's eight elements are two stores)
    if (((h->fwd_columns[c] * eb | pitch | reinterpret_cast<uintptr_t>(out)) & 63u) != 0u) return false;
    return (size_t)B * pitch > kLargeOutput || (size_t)h->fwd_maxD[c] * eb == 64u;
}
// the narrow-row classes: 32, 16, 8 and 4 lanes per row
template <typename WT>
static void launch_forward_groups(const tbe_handle* h, const void* tables, const int32_t* d_D_off, const IdxView indices,
                                  const IdxView offsets, int32_t B, int64_t nnz, bool mean, void* out, int out_io,
                                  hipStream_t s) {
    const WT* w = static_cast<const WT*>(tables);
    const int wpb = kFwdThreads / kWave;
    for (int c = 1; c < 5; ++c) {
        const int n = h->fwd_count[c];
        if (n == 0) continue;
        const int lpr_log2 = 6 - c;              // 32, 16, 8, 4 lanes per row
        const int G = kWave >> lpr_log2;
        const int64_t waves = (int64_t)n * (((int64_t)B + G - 1) / G);
        dim3 grid((unsigned)((waves + kGroupThreads / kWave - 1) / (kGroupThreads / kWave)));
        const int32_t* list = h->d_fwd_tables + h->fwd_first[c];
        // with a hot-row list in the handle, and enough bags per table to fill a workgroup's rounds
        const int cpt = hot_chunks(h, c, B);
        if (cpt > 0) {
            const dim3 hgrid((unsigned)((int64_t)n * cpt));
            if (mean)
                forward_hot_kernel<WT, 8, true><<<hgrid, kHotThreads, 0, s>>>(
                    w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base, list, n, lpr_log2, B, nnz, h->sumD, out, out_io,
                    h->d_err, h->d_hot_ids, h->d_hot_n, cpt);
            else
                forward_hot_kernel<WT, 8, false><<<hgrid, kHotThreads, 0, s>>>(
                    w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base, list, n, lpr_log2, B, nnz, h->sumD, out, out_io,
                    h->d_err, h->d_hot_ids, h->d_hot_n, cpt);
            continue;
        }
        const int64_t bags = kGroupThreads >> lpr_log2;   // of a workgroup
        const int64_t groups = (int64_t)n * (((int64_t)B + bags - 1) / bags);
        const bool stream = stream_output(h, c, B, out, out_io);
        auto launch = [&](auto mean_c, auto by_length_c, auto stream_c) {
            forward_groups_kernel<WT, 8, decltype(mean_c)::value, decltype(by_length_c)::value, decltype(stream_c)::value>
                <<<grid, kGroupThreads, 0, s>>>(w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base, list, n, lpr_log2, B, nnz,
                                                h->sumD, out, out_io, h->d_err);
        };
        auto go = [&](auto mean_c, auto by_length_c) {
            if (stream) launch(mean_c, by_length_c, std::true_type{});
            else launch(mean_c, by_length_c, std::false_type{});
        };
        if (by_length(groups, nnz, (int64_t)h->T * B, 1 << lpr_log2)) {
            grid = dim3((unsigned)groups);
            if (mean) go(std::true_type{}, std::true_type{});
            else go(std::false_type{}, std::true_type{});
        } else {
            if (mean) go(std::true_type{}, std::false_type{});
            else go(std::false_type{}, std::false_type{});
        }
    }
    // the bags those launches left out (the four classes' tables follow one another in the list)
    const int n_all = h->fwd_count[1] + h->fwd_count[2] + h->fwd_count[3] + h->fwd_count[4];
    if (n_all > 0) {
        const int scan_log2 = long_scan_log2((int64_t)n_all * B);
        const int64_t waves = (int64_t)n_all * (((int64_t)B + (1 << scan_log2) - 1) >> scan_log2);
        const dim3 grid((unsigned)((waves + wpb - 1) / wpb));
        const int32_t* list = h->d_fwd_tables + h->fwd_first[1];
        if (mean)
            forward_long_bags_kernel<WT, true><<<grid, kFwdThreads, 0, s>>>(
                w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base, list, n_all, scan_log2, B, nnz, h->sumD, out, out_io, h->d_err);
        else
            forward_long_bags_kernel<WT, false><<<grid, kFwdThreads, 0, s>>>(
                w, indices, offsets, d_D_off, h->d_w_off, h->d_row_base, list, n_all, scan_log2, B, nnz, h->sumD, out, out_io, h->d_err);
    }
}

template <typename WT>
static void launch_forward_classes(const tbe_handle* h, const void* tables, const int32_t* d_D_off, const IdxView indices,
                                   const IdxView offsets, int32_t B, int64_t nnz, bool mean, void* out, int out_io,
                                   hipStream_t s) {
    const int32_t *first = h->fwd_first, *count = h->fwd_count;
    if (forward_small(h, B, nnz)) {
        const int n = first[5] - first[0];
        if (forward_small_long(h, B, nnz)) launch_forward_nc<WT, 1, 8>(h, first[0], n, tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
        else launch_forward_nc<WT, 1, 4>(h, first[0], n, tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
    } else {
        launch_forward_nc<WT, 1, 4>(h, first[0], count[0], tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
        launch_forward_groups<WT>(h, tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
    }
    launch_forward_nc<WT, 2, 4>(h, first[5], count[5], tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
    if constexpr (sizeof(WT) == 4)   // (128 lanes hold 1024 binary16 columns, the widest row)
        launch_forward_nc<WT, 4, 2>(h, first[6], count[6], tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
}

hipError_t launch_forward(const tbe_handle* h, const void* tables, const int32_t* d_D_off, const void* indices_p,
                          const void* offsets_p, int idx32, int32_t B, int64_t nnz, tbe_pooling pooling, void* out,
                          int out_io, hipStream_t s) {
    const IdxView indices{indices_p, idx32}, offsets{offsets_p, idx32};
    const int64_t nbags = (int64_t)h->T * B;
    if (nbags == 0) return hipSuccess;
    LaunchTimer tm(h, s, "forward_pool");
    const bool mean = pooling == TBE_MEAN;
    if (h->dtype == TBE_F32) launch_forward_classes<float>(h, tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
    else launch_forward_classes<__half>(h, tables, d_D_off, indices, offsets, B, nnz, mean, out, out_io, s);
    tm.done();
    return hipGetLastError();
}

// ---- non-pooled lookup -------------------------------------------------------------------------------------
// out block of table t = [n_t, D_t], row i = W_t[indices[offsets[t] + i]]; the blocks follow one another.
// A wavefront takes up to 64 consecutive positions.  As a rule they lie in one table: then its lanes look at 64 tables at a time, each
// lane with one id finds its row, and what the wavefront writes is one contiguous run of rows, which its lanes fill fragment after
// fragment, kSeqInFlight of them under way before the first is converted and stored.  Only a fragment's row goes from lane to
// lane.  Positions of several tables, or of an offsets array that does not add up, take the general path below, where every lane
// resolves its own position and finds out for every fragment whose row it is.
// Bound: the gather of the rows and the stream of the output, which is written past the caches: nothing here reads it again, and the
// rows stay in the L2.  With a search per lane, a division and five cross-lane reads per fragment and one of them in flight / this with
// plain stores / this, us: 14 tables of 100 k rows x 32 and 2 of 2 M x 128 fp32 columns, 3.1 M positions, Zipf 1.3, bfloat16 out 143 /
// 110 / 66; 8 tables of 300 k rows, 1.3 M positions, Zipf 1.1: 64 fp32 columns 121 / 111 / 67, 256 fp32 430 / 412 / 359, 256 binary16
// into fp32 433 / 378 / 255, into bfloat16 260 / 224 / 139, 32 fp32 into bfloat16 35 / 27 / 26; 8 in flight instead of 4 0 to 30 % slower.
constexpr int kSeqInFlight = 4;

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)(v & 0xFFFFFFFFll), o, kWave);
        const uint32_t hi = __shfl_xor((uint32_t)((uint64_t)v >> 32), o, kWave);
        v += (int64_t)(((uint64_t)hi << 32) | lo);
    }
    return v;
}

// What a lane copies at a time: a 16-byte piece of a row, or where binary16 rows go into fp32 an 8-byte one, so that neighbouring
// lanes' stores are 16 bytes next to each other.
template <typename WT, int IO>
struct SeqFragment {
    static constexpr int kElems = RowIO<WT>::kVec;
    using raw_t = typename RowIO<WT>::raw_t;
    static __device__ __forceinline__ raw_t load(const WT* p) { return RowIO<WT>::load_raw(p); }
    static __device__ __forceinline__ raw_t zero() { return RowIO<WT>::zero_raw(); }
    static __device__ __forceinline__ void store(const raw_t raw, void* __restrict__ out, const int64_t elem) {
        float x[kElems];
        RowIO<WT>::unpack(raw, x);
        if constexpr (IO != 0 && kElems == 8) store8_from_float<true>(out, IO, elem, x);
        else store4_from_float<true>(out, IO, elem, x[0], x[1], x[2], x[3]);
    }
};
template <>
struct SeqFragment<__half, 0> {
    static constexpr int kElems = 4;
    using raw_t = uint2;
    static __device__ __forceinline__ raw_t load(const __half* p) { return RowIO<__half>::load4_raw(p); }
    static __device__ __forceinline__ raw_t zero() { return make_uint2(0u, 0u); }
    static __device__ __forceinline__ void store(const raw_t raw, void* __restrict__ out, const int64_t elem) {
        float x[4];
        RowIO<__half>::unpack4(raw, x);
        store4_from_float<true>(out, 0, elem, x[0], x[1], x[2], x[3]);
    }
};

// The general path: every position by itself.
template <typename WT, typename IT, int IO>
__device__ __forceinline__ void lookup_seq_rows(
    const WT* __restrict__ weights, const IT* __restrict__ indices, const IT* __restrict__ offsets, const int32_t* __restrict__ D_off,
    const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base, const int T, const int64_t p0, const int n,
    void* __restrict__ out, const int64_t out_elems, int32_t* err) {
    using F4 = SeqFragment<WT, IO>;
    constexpr uint32_t kF = F4::kElems;
    const int lane = lane_id();
    const int64_t p = p0 + lane;
    const bool valid = lane < n;
    // table of the position: the last t with offsets[t] <= p (empty tables are skipped by construction)
    int t = 0;
    {
        const int64_t q = valid ? p : p0;
        int lo = 0, hi = T;  // invariant: offsets[lo] <= q, answer in [lo, hi)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)offsets[mid] <= q) lo = mid;
            else hi = mid;
        }
        t = lo;
    }
    // element offset of the table's block: sum over earlier tables of n_t' * D_t'
    const int t0 = __shfl(t, 0, kWave);
    int64_t part = 0;
    for (int tt = lane; tt < t0; tt += kWave) {
        const int64_t n = (int64_t)offsets[tt + 1] - (int64_t)offsets[tt];
        part += (n > 0 ? n : 0) * (int64_t)(D_off[tt + 1] - D_off[tt]);
    }
    int64_t base = wave_sum_i64(part);
    for (int tt = t0; tt < t; ++tt) {
        const int64_t n = (int64_t)offsets[tt + 1] - (int64_t)offsets[tt];
        base += (n > 0 ? n : 0) * (int64_t)(D_off[tt + 1] - D_off[tt]);
    }
    const int D = D_off[t + 1] - D_off[t];
    int64_t id = valid ? (int64_t)indices[p] : 0;
    const int64_t R = row_base[t + 1] - row_base[t];
    bool bad = false;
    if (valid && (id < 0 || id >= R)) {
        atomicOr(err, 1);   // as in the pooled forward: flagged, and the row reads as zeros
        bad = true;
        id = 0;
    }
    const int64_t src_elem = w_off[t] + id * D;
    int64_t dst_elem = base + (p - (int64_t)offsets[t]) * D;
    // a malformed offsets array (not ascending from 0 to nnz) must never take a store outside out[0, out_elems)
    if (valid && (dst_elem < 0 || dst_elem + D > out_elems)) {
        atomicOr(err, 1);
        dst_elem = -1;
    }
    // all fragments of the rows, one behind the other: a row's first is number `first`
    const uint32_t F = valid && dst_elem >= 0 ? (uint32_t)D / kF : 0u, behind = wave_incl_scan(F), first = behind - F;
    const uint32_t total = bcast_lane(behind, kWave - 1);
    const int64_t src = bad ? -1 : src_elem;
    const uint32_t F0 = bcast_lane(F, 0);   // (of the first position, which exists)
    const uint32_t inv = __all(!valid || F == F0) && F0 > 0u ? ((1u << 31) + F0 - 1u) / F0 : 0u;   // all the same: as in one table
    for (uint32_t q0 = (uint32_t)lane; q0 - (uint32_t)lane < total; q0 += kSeqInFlight * kWave) {
        typename F4::raw_t x[kSeqInFlight];
        int64_t to[kSeqInFlight];
#pragma unroll
        for (int u = 0; u < kSeqInFlight; ++u) {
            const uint32_t q = q0 + (uint32_t)u * kWave;
            int k = 0;   // the last row whose first fragment is q or one before it
            if (inv != 0u) {
                k = (int)umin(__umulhi(2u * q, inv), kWave - 1u);
            } else {
#pragma unroll
                for (int step = kWave / 2; step > 0; step >>= 1) k += (uint32_t)__shfl(first, k + step, kWave) <= q ? step : 0;
            }
            const int64_t f = (int64_t)(q - (uint32_t)__shfl(first, k, kWave)) * kF;
            const int64_t from = (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)src >> 32), k, kWave) << 32) | (uint32_t)__shfl((int)(uint64_t)src, k, kWave));
            to[u] = f + (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)dst_elem >> 32), k, kWave) << 32) | (uint32_t)__shfl((int)(uint64_t)dst_elem, k, kWave));
            x[u] = q < total && from >= 0 ? F4::load(weights + from + f) : F4::zero();
        }
#pragma unroll
        for (int u = 0; u < kSeqInFlight; ++u)
            if (q0 + (uint32_t)u * kWave < total) F4::store(x[u], out, to[u]);
    }
}

// IT: int64 or int32 ids and offsets, compiled apart: with the width as a run-time flag every step of a search branches around two
// loads.
template <typename WT, typename IT, int IO>
__global__ __launch_bounds__(kFwdThreads, 8) void lookup_seq_kernel(
    const WT* __restrict__ weights, const IT* __restrict__ indices, const IT* __restrict__ offsets, const int32_t* __restrict__ D_off,
    const int64_t* __restrict__ w_off, const int64_t* __restrict__ row_base, const int T, const int64_t nnz, const int each,
    void* __restrict__ out, const int64_t out_elems, int32_t* err) {
    const int lane = lane_id();
    const int64_t p0 = ((int64_t)blockIdx.x * (kFwdThreads / kWave) + (threadIdx.x >> 6)) * each;
    if (p0 >= nnz) return;
    const int n = (int)((nnz - p0) < (int64_t)each ? (nnz - p0) : (int64_t)each);
    const int64_t my_id = (int64_t)indices[p0 + (lane < n ? lane : n - 1)];
    // the first table that ends behind p0, all that is needed of it, and the elements of the blocks before its own; 64 tables a round
    int t = -1, D = 0;
    int64_t part = 0, start = 0, end = 0, R = 0, w0 = 0;
    for (int t0 = 0; t0 < T; t0 += kWave) {
        const bool on = t0 + lane < T;
        const int tt = on ? t0 + lane : T - 1;
        const int64_t s = (int64_t)offsets[tt], e = (int64_t)offsets[tt + 1], rows = row_base[tt + 1] - row_base[tt], w = w_off[tt];
        const int cols = D_off[tt + 1] - D_off[tt];
        const uint64_t m = __ballot(on && e > p0);
        const int f = m != 0ull ? __ffsll((unsigned long long)m) - 1 : kWave;
        if (on && lane < f && e > s) part += (e - s) * (int64_t)cols;
        if (m != 0ull) {
            t = t0 + f;
            start = lane_i64(s, f);
            end = lane_i64(e, f);
            R = lane_i64(rows, f);
            w0 = lane_i64(w, f);
            D = bcast_lane(cols, f);
            break;
        }
    }
    const int64_t dst = wave_sum_i64(part) + (p0 - start) * D;
    if (t < 0 || start < 0 || start > p0 || end < p0 + n || dst < 0 || dst + (int64_t)n * D > out_elems) {
        lookup_seq_rows<WT, IT, IO>(weights, indices, offsets, D_off, w_off, row_base, T, p0, n, out, out_elems, err);
        return;
    }
    const WT* const table = weights + w0;
    const bool ok = my_id >= 0 && my_id < R;
    if (!ok) atomicOr(err, 1);   // as in the pooled forward: flagged, and the row reads as zeros
    const int row = ok ? (int)my_id : -1;   // (tables have fewer than 2^31 rows)
    using F4 = SeqFragment<WT, IO>;
    constexpr uint32_t kF = F4::kElems;
    const uint32_t F = (uint32_t)D / kF, total = (uint32_t)n * F;   // fragments per row, in all
    const uint32_t inv = ((1u << 31) + F - 1u) / F;   // q / F by a multiplication: exact, as q * F stays below 2^31
    for (uint32_t q0 = (uint32_t)lane; q0 - (uint32_t)lane < total; q0 += kSeqInFlight * kWave) {
        typename F4::raw_t x[kSeqInFlight];
#pragma unroll
        for (int u = 0; u < kSeqInFlight; ++u) {
            const uint32_t q = q0 + (uint32_t)u * kWave;
            const uint32_t k = __umulhi(2u * q, inv), f = q - k * F;
            const int r = __shfl(row, (int)(k < (uint32_t)n ? k : 0u), kWave);
            x[u] = r >= 0 && q < total ? F4::load(table + (int64_t)r * D + f * kF) : F4::zero();
        }
#pragma unroll
        for (int u = 0; u < kSeqInFlight; ++u) {
            const uint32_t q = q0 + (uint32_t)u * kWave;
            if (q < total) F4::store(x[u], out, dst + (int64_t)q * kF);
        }
    }
}

// Positions per wavefront, at most 64 and in whole powers of two.  64 rows of 1024 columns are 64 steps of loads one behind the other:
// a small batch waits for that chain, and in a large one the wavefronts write 128 to 256 KB apart, which meets the same channels.  So a
// wavefront gets about 1024 fragments (by the mean width of the tables, as the host does not know where the positions lie), at least
// 16 positions, for it looks its table up once; and where that leaves fewer than 2048 wavefronts, down to a step's 256 fragments.
// A search per lane and 64 positions / this with 64 / 32 / 16 / 8, us, tables of 100 k rows, Zipf 1.2 (the last: of 9 to 84 rows):
//   8 x 1000 of 64, 256, 1024 fp32 columns into bfloat16   11.1 35.5 137 / 9.7 27.6 99.7 / 9.3 15.7 52.6 / 9.3 9.9 28.8 / 9.1 8.7 15.9
//   8 x 10000, 1024 columns, and a reader of the output    278 / 199 / 155 / 131 / 129; 256 binary16 columns into fp32 51 / 52 / 49 / 45 / 44
//   8 x 100000 of 16, 64, 256 fp32 columns                 16.7 52 272 / 11.8 40 180 / 12.8 39 148 / 19.4 38 147 / 35 43 142
//   5 x 430000 of 16 and 1024 columns into bfloat16        727 / 566 / 524 / 483 / 557
static int seq_positions(const tbe_handle* h, const int64_t nnz, const int out_io) {
    const int elems = h->dtype == TBE_F32 || out_io == 0 ? 4 : 8;   // of a fragment
    const int64_t row = h->sumD / ((int64_t)h->T * elems) > 0 ? h->sumD / ((int64_t)h->T * elems) : 1;
    int each = kWave;
    while (each > 16 && each * row > 1024 && nnz < (int64_t)1 << 30) each /= 2;   // (a grid has fewer than 2^32 lanes)
    while (each > 4 && each * row > kSeqInFlight * kWave && nnz < (int64_t)each * 2048) each /= 2;
    return each;
}

template <typename WT, typename IT>
static void launch_lookup_seq_as(const tbe_handle* h, const dim3 grid, const int each, const void* tables, const void* indices, const void* offsets,
                                 int64_t nnz, void* out, int out_io, int64_t out_elems, hipStream_t s) {
    auto go = [&](auto io) {
        lookup_seq_kernel<WT, IT, decltype(io)::value><<<grid, kFwdThreads, 0, s>>>(
            static_cast<const WT*>(tables), static_cast<const IT*>(indices), static_cast<const IT*>(offsets), h->d_D_off, h->d_w_off,
            h->d_row_base, h->T, nnz, each, out, out_elems, h->d_err);
    };
    if (out_io == 0) go(std::integral_constant<int, 0>{});
    else if (out_io == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
}

hipError_t launch_lookup_seq(const tbe_handle* h, const void* tables, const void* indices, const void* offsets,
                             int idx32, int64_t nnz, void* out, int out_io, int64_t out_elems, hipStream_t s) {
    if (nnz == 0) return hipSuccess;
    const int each = seq_positions(h, nnz, out_io);
    const int64_t per_block = (int64_t)(kFwdThreads / kWave) * each;
    const dim3 grid((unsigned)((nnz + per_block - 1) / per_block));
    LaunchTimer tm(h, s, "lookup_seq");
    if (h->dtype == TBE_F32) {
        if (idx32) launch_lookup_seq_as<float, int32_t>(h, grid, each, tables, indices, offsets, nnz, out, out_io, out_elems, s);
        else launch_lookup_seq_as<float, int64_t>(h, grid, each, tables, indices, offsets, nnz, out, out_io, out_elems, s);
    } else {
        if (idx32) launch_lookup_seq_as<__half, int32_t>(h, grid, each, tables, indices, offsets, nnz, out, out_io, out_elems, s);
        else launch_lookup_seq_as<__half, int64_t>(h, grid, each, tables, indices, offsets, nnz, out, out_io, out_elems, s);
    }
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
