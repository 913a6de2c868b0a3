// Floating-point half of the backward pass: per unique row, sum the upstream gradient slices of the
// row's segment and apply one moment-scaled row-wise AdaGrad step in place (Algorithm 1, steps 5-6).
//
// Every unique row has exactly one owner (a group of lanes, a wavefront, or the workgroup that combines
// a long row's partial sums), so weights and moments have a single writer and the result does not depend
// on scheduling.  A row of D floats is covered by LPR = D/4 lanes (one float4 each), which leaves
// G = 64/LPR lane groups per wavefront.  Rows are binned by the number of lookups that hit them:
//   - short  (a run of <= G consecutive rows of one table with <= 64 lookups in total): one row per lane group, the
//     lookups' bag ids arrive in windows of 64 with one coalesced load and are handed out with cross-lane reads;
//   - medium (65 .. long_min lookups): the whole wavefront walks the row, groups interleaved;
//   - long   (> long_min lookups): listed by tbe_lists.hip; the hottest of a large gradient block go through the matrix
//     cores (tbe_dense.hip), the others are cut into parts that wavefronts of the kernels here reduce into partial sums.
// Row metadata (segment bounds, key, table, moment) is fetched for up to 64 rows at a time, one row per lane.
#include "tbe_rows.h"

namespace tbe {

constexpr int kSegThreads = 256;
// Rows of one wavefront pass: 16 in batches of many rows, 32 from so many rows per wavefront on that the last round of passes does
// not count.  Every pass starts with a chain of four dependent loads (bounds, first bag, table, moment) and one for its bag ids, which
// longer passes do less often; shorter ones share out rows of unequal length better, and rows of many lookups lie together, in the
// small tables of a handle.  Row updates with passes of 16 / 32 / 64 rows, ms: 256 tables x 32768 bags of 31 ids, 256 binary16 columns
// (4500 rows per wavefront) 20.5 / 19.8 / 19.7; 64 such tables x 65536 bags (1400) 8.64 / 8.70 / 8.72, with mean pooling 9.36 / 9.39 /
// 9.46, of half the bags (600) 2.47 / 2.58 / 2.62; 26 tables of 1000 to 1 M rows x 32768 bags, uniform, 128 columns (260) 1.25 / 1.54 /
// 2.34.  Tables of at most 8 columns have 32 or 64 rows side by side, and a pass of 16 leaves lanes idle: 8 tables of 1 M rows x
// 16384 bags of 20 uniform ids, 4 / 8 columns (270) 73 / 107 us with 16, 66 / 92 with 32; the 26 tables x 16384 bags at 4 columns
// (180) 216 with 16, 240 with 32, 424 with 64.
// Where registers allow (8 wavefronts per SIMD), the loads at the start serve as many of a wavefront's passes as 64 rows are: the same
// 8 tables at 16 / 32 / 64 / 128 columns 131 / 187 / 330 / 615 us with the loads in every pass, 119 / 172 / 317 / 609 with this;
// the variant of 7 wavefronts loses by it, 20.5 -> 21.2 ms at the first of the workloads above with passes of 16 rows.
constexpr int kPassRowsLog2 = 4, kLongPassRowsLog2 = 5;
constexpr uint32_t kLongPassNeed = 2048, kLongPassNeedNarrow = 128;   // rows per wavefront; tables of at most 8 columns
// Rows of few lookups are read and written past the caches (as streams) where the batch's rows and its gradients together are more
// than the Infinity Cache holds: the gradients, which are gathered again and again, stay there instead.  Where everything fits, the next
// forward finds the rows in it.  Whole steps without / with this, us: 12 tables x 8192 bags of 20 uniform ids, 128 fp32 columns (928 MB
// of rows + 50 MB) 591 / 547; 64 tables x 4096 bags of 31 ids, bfloat16 gradients (663 + 117) 1261 / 1245; 16 tables x 16384 bags of 21
// ids (271 + 151) 766 / 754; but where it all fits 26 tables x 4096 bags of 11 ids (56 + 27) 162 / 165, sequences of 3.1 M events (34 + 275)
// 343 / 361.  The reads or the writes alone: 561 and 576 of the first 577.
constexpr uint64_t kInfinityCacheBytes = (uint64_t)256 << 20;
constexpr int kSegBlocks = 2048;  // persistent grids: waves stride over passes of unique rows, or over rows
constexpr int kSegBlocks7 = 1792;   // ... of the variants of 7 wavefronts per SIMD
// Long spans count a die's wavefronts as an eighth of the grid: a pass would be left out or taken twice otherwise.
static_assert(kSegBlocks % kDies == 0 && kSegBlocks7 % kDies == 0, "as many workgroups on every die");
// Gradient fragments in flight per lane while a row is reduced: as many as the registers of the variant allow
// without spilling at the WAVES wavefronts per SIMD its kernel is compiled for.  Measured at the largest workload with
// 32-bit gradients: 2 / 4 / 6 / 8 in flight give 21.6 / 20.4 / 20.2 / 19.8 ms for the row updates; 8 needs more than
// the 64 registers of 8 wavefronts per SIMD, which is why seg_update runs 7 (6: 20.7 ms); 16-bit fragments are half
// the size: 8 in flight with mean pooling too, row updates with 6 / 8, us: 32 tables x 8192 bags of 21 ids, 128 and 256 binary16
// columns, bfloat16 gradients 518 / 505; 26 tables x 8192 bags, 64 binary16 columns, binary16 gradients 219 / 214.
template <int NC, bool MEAN, typename GT, int WAVES>
__device__ __host__ constexpr int seg_unroll() {
    return NC > 1 ? 4 : (sizeof(GT) == 4 ? (WAVES < 8 ? (MEAN ? 6 : 8) : (MEAN ? 4 : 6)) : 8);
}


struct RowGeom {
    int D, LPR, G, sub, lc;
};

__device__ __forceinline__ RowGeom row_geom(int D) {
    RowGeom g;
    const int lane = lane_id();
    const int nl = (D + 3) >> 2;
    g.D = D;
    g.LPR = nl >= kWave ? kWave : pow2ceil64(nl);
    const int lpr_log2 = __builtin_ctz((unsigned)g.LPR);   // LPR is a power of two: shifts, not divisions
    g.G = kWave >> lpr_log2;
    g.sub = lane >> lpr_log2;
    g.lc = (lane & (g.LPR - 1)) * 4;
    return g;
}

template <bool MEAN>
__device__ __forceinline__ float bag_scale(const OffsetWords offsets, uint32_t bag) {
    if (!MEAN) return 1.f;
    const uint32_t L = offsets.length(bag);
    return L > 0u ? 1.f / (float)L : 0.f;
}

// Where the upstream gradient of a lookup of table t lives: element base + (row - row0) * pitch (+ column).
// Pooled: row = bag id, one [B, sum(D)] matrix.  Non-pooled: row = original position, one [n_t, D_t] block per table.
struct GradAddr {
    int64_t base;
    uint32_t pitch, row0;   // (a 32-bit pitch: one 32 x 32 + 64 bit multiply-add per address instead of a 64-bit product)
};
__device__ __forceinline__ GradAddr grad_addr(const SegArgs& a, const int t, const int D) {
    GradAddr ga;
    if (a.seq) {
        ga.base = a.seq_gbase[t]; ga.pitch = (uint32_t)D; ga.row0 = 0u;
    } else {
        ga.base = a.D_off[t]; ga.pitch = (uint32_t)a.sumD; ga.row0 = (uint32_t)t * (uint32_t)a.B;
    }
    return ga;
}

// Whole-wavefront reduction of sorted positions [s, e) of ONE row:
// acc += sum of scale(bag) * grad_out[b, d0 + col .. col+3]; the groups take interleaved positions and
// fold_groups() completes the sum.  NC = 256-column chunks per row.
template <int NC, bool MEAN, typename GT, int WAVES = 8>
__device__ __forceinline__ void segment_reduce(float (&acc)[NC][4], const RowGeom& g, const GT* __restrict__ gcol,
                                               const uint32_t pitch, const uint32_t row0,
                                               const uint32_t* __restrict__ bag_sorted, const OffsetWords offsets,
                                               const uint32_t s, const uint32_t e) {
    constexpr int kSegUnroll = seg_unroll<NC, MEAN, GT, WAVES>();
    const int lane = lane_id();
    for (uint32_t base = s; base < e; base += kWave) {
        const int n = (int)((e - base) < (uint32_t)kWave ? (e - base) : (uint32_t)kWave);
        uint32_t my_b = 0;
        float my_s = 1.f;
        if (lane < n) {
            const uint32_t bag = bag_sorted[base + lane];
            my_b = bag - row0;
            my_s = bag_scale<MEAN>(offsets, bag);
        }
        for (int k0 = 0; k0 < n; k0 += kSegUnroll * g.G) {
            typename GradIO<GT>::raw_t x[kSegUnroll][NC];
            float sc[kSegUnroll];
#pragma unroll
            for (int u = 0; u < kSegUnroll; ++u) {
                const int k = k0 + u * g.G + g.sub;
                const uint32_t b = __shfl(my_b, k & (kWave - 1), kWave);
                sc[u] = MEAN ? __shfl(my_s, k & (kWave - 1), kWave) : 1.f;
                const bool on = k < n;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int col = g.lc + c * kWave * 4;
                    x[u][c] = (on && col < g.D) ? GradIO<GT>::load(gcol + (uint64_t)b * pitch + col) : GradIO<GT>::zero();
                }
            }
#pragma unroll
            for (int u = 0; u < kSegUnroll; ++u)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const float4 f = GradIO<GT>::to_float(x[u][c]);
                    if (MEAN) {
                        acc[c][0] = fmaf(sc[u], f.x, acc[c][0]);
                        acc[c][1] = fmaf(sc[u], f.y, acc[c][1]);
                        acc[c][2] = fmaf(sc[u], f.z, acc[c][2]);
                        acc[c][3] = fmaf(sc[u], f.w, acc[c][3]);
                    } else {
                        acc[c][0] += f.x;
                        acc[c][1] += f.y;
                        acc[c][2] += f.z;
                        acc[c][3] += f.w;
                    }
                }
        }
    }
}

template <int NC>
__device__ __forceinline__ void fold_groups(float (&acc)[NC][4], const RowGeom& g) {
    for (int o = g.LPR; o < kWave; o <<= 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (o == 32) acc[c][v] = pair_sum<32>(acc[c][v]);        // the two halves / odd and even rows: in place
                else if (o == 16) acc[c][v] = pair_sum<16>(acc[c][v]);
                else acc[c][v] += __shfl_xor(acc[c][v], o, kWave);
            }
    }
}

// the step size of Algorithm 1, step 6: lr / (sqrt(v / c) + eps), from the hardware square root and reciprocal (one
// unit in the last place each); v == 0 means the row's gradient is zero and nothing is applied
__device__ __forceinline__ float adagrad_step(const float v_new, const float lr, const float eps, const float inv_c) {
    const float denom = __builtin_amdgcn_sqrtf(v_new * inv_c) + eps;
    return v_new > 0.f ? lr * __builtin_amdgcn_rcpf(denom) : 0.f;
}

// The optimizer step for one row.  acc holds the complete row gradient in the LPR lanes that `on`
// marks (all groups after fold_groups, or each group its own row).  v_old is the row's moment.
//   v <- v + ||g||^2 ;  w <- w - lr / (sqrt(v / c) + eps) * g      (updated v; v stored unscaled)
// Lanes with write == true store their 4 columns; the lane with lc == 0 among them stores the moment.
// With sgd == true the step is plain SGD instead, w <- w - lr * g, and the moment is neither read nor written.
template <int NC>
__device__ __forceinline__ float row_step(const float (&acc)[NC][4], const RowGeom& g, float* __restrict__ vptr,
                                          const float v_old, const bool write, const float lr, const float eps,
                                          const float inv_c, const bool sgd) {   // the moment; returns the step size
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int col = g.lc + c * kWave * 4;
        if (col < g.D) {
#pragma unroll
            for (int v = 0; v < 4; ++v) sq = fmaf(acc[c][v], acc[c][v], sq);
        }
    }
    sq = group_sum(sq, g.LPR);  // within the LPR lanes that cover the row
    const float v_new = v_old + sq;
    if (write && g.lc == 0 && !sgd) *vptr = v_new;
    return sgd ? lr : adagrad_step(v_new, lr, eps, inv_c);
}
template <typename WT, int NC>
__device__ __forceinline__ void adagrad_row(const float (&acc)[NC][4], const RowGeom& g, WT* __restrict__ wrow,
                                            float* __restrict__ vptr, const float v_old, const bool write,
                                            const float lr, const float eps, const float inv_c, const bool sgd = false,
                                            const bool stream = false) {
    const float step = row_step<NC>(acc, g, vptr, v_old, write, lr, eps, inv_c, sgd);
    if (!write) return;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int col = g.lc + c * kWave * 4;
        if (col < g.D) {
            float w[4];
            RowIO<WT>::unpack4(stream ? RowIO<WT>::template load4_raw<true>(wrow + col) : RowIO<WT>::load4_raw(wrow + col), w);
#pragma unroll
            for (int v = 0; v < 4; ++v) w[v] = fmaf(-step, acc[c][v], w[v]);
            if (stream) RowIO<WT>::template store4<true>(wrow + col, w);
            else RowIO<WT>::store4(wrow + col, w);
        }
    }
}
// ... of a row of at most 256 columns whose weights are in registers already
template <typename WT>
__device__ __forceinline__ void adagrad_row_loaded(const float (&acc)[1][4], const RowGeom& g, WT* __restrict__ wrow,
                                                   const typename RowIO<WT>::raw4_t wraw, float* __restrict__ vptr,
                                                   const float v_old, const bool write, const float lr, const float eps,
                                                   const float inv_c, const bool sgd, const bool stream) {
    const float step = row_step<1>(acc, g, vptr, v_old, write, lr, eps, inv_c, sgd);
    if (write && g.lc < g.D) {
        float w[4];
        RowIO<WT>::unpack4(wraw, w);
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = fmaf(-step, acc[0][v], w[v]);
        if (stream) RowIO<WT>::template store4<true>(wrow + g.lc, w);
        else RowIO<WT>::store4(wrow + g.lc, w);
    }
}

// ---- short rows ---------------------------------------------------------------------------------------------------
// Most rows of a batch have one or two lookups, and their bookkeeping is vector-ALU work: before the three things below the row
// updates of 64 tables x 4096 bags of 31 ids (Zipf 1.1, bfloat16 gradients) issued 32183 vector instructions per wavefront in
// 800 us, now 21746 in 702.  A round has as many slots as its longest row needs (1, 2, 4 or the variant's unroll, not always the
// last); the bag ids of 64 lookups serve all the rounds they cover; a round's rows are of one table, so that its addresses start
// from scalars and each costs one 32 x 32 + 64 bit multiply-add.  12 tables x 8192 bags of 20 uniform ids, 128 columns: 544 ->
// 507 us.  The weights are loaded behind the gradients: ahead of them 507 -> 612 us there (the read and the write of a row then
// lie further apart), 702 -> 727 us above.  The variant of 7 wavefronts per SIMD, 32-bit gradients of wide binary16 rows, has them
// ahead: 64 tables x 32768 bags of 31 ids 4271 -> 4242 us, half of the bags with mean pooling 2604 -> 2582, but 12 tables x 8192
// bags of 20 uniform ids 833 -> 837 and x 4096 299 -> 302.
//
// NS lookups of short rows, of every lane group its own: number q0 .. q0+NS-1 of the group's glen, which lie in lanes off, off+1,
// ... of (my_b, my_s).  UNIFORM: one group, so that all of this is the same in all lanes and stays on the scalar unit.
template <int NS, bool UNIFORM, bool MEAN, typename GT>
__device__ __forceinline__ void add_lookups(float (&acc)[1][4], const GT* __restrict__ gcol, const uint32_t pitch,
                                            const uint32_t lane_col, const uint32_t my_b, const float my_s, const uint32_t off,
                                            const uint32_t q0, const uint32_t glen) {
    typename GradIO<GT>::raw_t x[NS];
    float sc[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int src = (int)((off + q0 + (uint32_t)u) & (kWave - 1));
        uint32_t b;
        if (UNIFORM) {
            b = bcast_lane(my_b, src);
            sc[u] = MEAN ? bcast_lane(my_s, src) : 1.f;
            const GT* row = gcol + (uint64_t)b * pitch;
            x[u] = q0 + u < glen ? GradIO<GT>::load(row + lane_col) : GradIO<GT>::zero();
        } else {
            b = __shfl(my_b, src, kWave);
            sc[u] = MEAN ? __shfl(my_s, src, kWave) : 1.f;
            x[u] = q0 + u < glen ? GradIO<GT>::load(gcol + lane_col + (uint64_t)b * pitch) : GradIO<GT>::zero();
        }
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const float4 f = GradIO<GT>::to_float(x[u]);
        if (MEAN) {
            acc[0][0] = fmaf(sc[u], f.x, acc[0][0]);
            acc[0][1] = fmaf(sc[u], f.y, acc[0][1]);
            acc[0][2] = fmaf(sc[u], f.z, acc[0][2]);
            acc[0][3] = fmaf(sc[u], f.w, acc[0][3]);
        } else {
            acc[0][0] += f.x;
            acc[0][1] += f.y;
            acc[0][2] += f.z;
            acc[0][3] += f.w;
        }
    }
}
// all lookups of short rows, lmax of the longest: as many slots a round as are needed
template <int NS, bool UNIFORM, bool MEAN, typename GT>
__device__ __forceinline__ void add_short(float (&acc)[1][4], const GT* __restrict__ gcol, const uint32_t pitch,
                                          const uint32_t lane_col, const uint32_t my_b, const float my_s, const uint32_t off,
                                          const uint32_t lmax, const uint32_t glen) {
    uint32_t q0 = 0;
    for (; q0 + 4u < lmax; q0 += NS) add_lookups<NS, UNIFORM, MEAN, GT>(acc, gcol, pitch, lane_col, my_b, my_s, off, q0, glen);
    if (q0 >= lmax) return;
    const uint32_t left = lmax - q0;
    if (left == 1u) add_lookups<1, UNIFORM, MEAN, GT>(acc, gcol, pitch, lane_col, my_b, my_s, off, q0, glen);
    else if (left == 2u) add_lookups<2, UNIFORM, MEAN, GT>(acc, gcol, pitch, lane_col, my_b, my_s, off, q0, glen);
    else add_lookups<4, UNIFORM, MEAN, GT>(acc, gcol, pitch, lane_col, my_b, my_s, off, q0, glen);
}

// ---- parts of long rows ----------------------------------------------------------------------------------------
// One wavefront per part: partial[slot] = sum of an equal share of the row's lookups.
template <int NC, bool MEAN, typename GT, int WAVES>
__device__ __forceinline__ void reduce_part(const SegArgs& a, const RowGeom& g, const uint4 ent, const uint32_t c) {
    const uint32_t s = a.seg_start[ent.x];
    const uint64_t len = a.seg_start[ent.x + 1] - s;
    const uint32_t lo = s + (uint32_t)(len * c / ent.z);
    const uint32_t hi = s + (uint32_t)(len * (c + 1u) / ent.z);
    float acc[NC][4];
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) acc[cc][0] = acc[cc][1] = acc[cc][2] = acc[cc][3] = 0.f;
    const GradAddr ga = grad_addr(a, (int)ent.w, g.D);
    segment_reduce<NC, MEAN, GT, WAVES>(acc, g, static_cast<const GT*>(a.grad_out) + ga.base, ga.pitch, ga.row0, a.bag_sorted,
                                        a.offsets, lo, hi);
    fold_groups<NC>(acc, g);
    if (g.sub == 0) {
        float* dst = a.partial + (size_t)(ent.y + c) * a.maxD;
#pragma unroll
        for (int cc = 0; cc < NC; ++cc) {
            const int col = g.lc + cc * kWave * 4;
            if (col < g.D) *reinterpret_cast<float4*>(dst + col) = make_float4(acc[cc][0], acc[cc][1], acc[cc][2], acc[cc][3]);
        }
    }
}

// All parts of the tables of one width class (WIDE: more than 256 columns), one per wavefront and round.  Parts are of
// similar size, so a fixed stride keeps the wavefronts level.
template <bool WIDE, bool MEAN, typename GT, int WAVES>
__device__ __forceinline__ void reduce_parts(const SegArgs& a) {
    const uint32_t nunits = a.counters[3];
    const uint32_t nwaves = gridDim.x * (kSegThreads / kWave);
    for (uint32_t e = blockIdx.x * (kSegThreads / kWave) + (threadIdx.x >> 6); e < nunits; e += nwaves) {
        const uint2 un = a.unit_list[e];
        const uint4 ent = a.long_list[un.x];
        const int t = (int)ent.w;
        const int D = a.D_off[t + 1] - a.D_off[t];
        if ((D > 256) != WIDE) continue;
        reduce_part<WIDE ? 4 : 1, MEAN, GT, WAVES>(a, row_geom(D), ent, un.y);
    }
}

// The hint for the next forward: the handle's copy of the rows listed as having the most lookups.
__device__ __forceinline__ void copy_hint(const SegArgs& a) {
    if (!a.hint_n) return;
    for (int t = blockIdx.x; t < a.T; t += gridDim.x) {
        const uint32_t n = a.hot_n[t];
        if (threadIdx.x == 0) a.hint_n[t] = n;
        if (threadIdx.x < n) a.hint_ids[(size_t)t * kHotRows + threadIdx.x] = a.hot_ids[(size_t)t * kHotRows + threadIdx.x];
    }
}
static_assert(kHotRows <= kSegThreads, "one thread per listed row");

// ---- rows with at most long_min lookups (after the parts of longer ones), tables at most 256 columns wide ------------------
// kSegWaves = wavefronts per SIMD the kernel is compiled and launched for: 8, or 7 with more fragments in flight; the
// host picks (see the launch).
template <typename WT, bool MEAN, typename GT, int kSegWaves>
__global__ __launch_bounds__(kSegThreads, kSegWaves) void seg_update_kernel(const SegArgs a) {
    constexpr int kSegUnroll = seg_unroll<1, MEAN, GT, kSegWaves>();
    // ... of rows side by side: 8 would spill registers where every fragment comes with its bag's scale (ten tables of odd widths,
    // 777 bags, binary16 gradients, the step with 8 / 6: 108.4 / 107.2 us; 32 tables x 8192 bags, 128 and 256 columns 497 / 492)
    constexpr int kSideUnroll = MEAN && sizeof(GT) == 2 ? 6 : kSegUnroll;
    constexpr bool kFetch = kSegWaves == 8;   // the start of a pass is loaded for several of them (see kPassRowsLog2)
    constexpr bool kAhead = kSegWaves < 8;   // a row's weights are loaded ahead of its gradients (see the short rows above)
    const int lane = lane_id();
    copy_hint(a);
    if (a.counters[4] != 0u) return;
    reduce_parts<false, MEAN, GT, kSegWaves>(a);
    const uint32_t U = a.counters[0];
    const bool stream = (uint64_t)U * a.row_bytes > a.stream_from;
    const uint32_t nwaves = gridDim.x * (kSegThreads / kWave);
    // rows per pass: 2^lg (see kPassRowsLog2), fewer where the batch touches so few rows that whole wavefronts would go idle while
    // others walk a pass one round after the other - down to as many as the widest table's rows a wavefront takes side by side
    int lg = kPassRowsLog2;
    if (U / nwaves >= a.long_pass_need) lg = kLongPassRowsLog2;
    else while (lg > a.min_rows_log2 && (U >> lg) < 2u * nwaves) --lg;
    const uint32_t nblk = (U + (1u << lg) - 1u) >> lg;
    const uint32_t e_all = a.seg_start[U];   // lookups in all
    // The wavefronts of the chip take the passes in turn.  With long spans those of a die take the passes of its two spans in turn
    // instead, so that a die reads the gradient blocks of a few tables only: pass first + i of the first span, i < n1, then again + i
    // of the second.  All of it is the same for the whole wavefront and stays on the scalar unit; with two divisions by the length of
    // a span in every pass, and more scalar registers spilled than now, small batches paid 0.5 to 2 us (34 tables x 40 bags x 32
    // columns 14.1 us, now 12.5; one table x 512 bags x 64 columns 8.8, now 8.1).
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t i = blockIdx.x * (kSegThreads / kWave) + wave, step = nwaves, n1 = nblk, n = nblk, first = 0, again = 0;
    if (a.long_spans) {
        const uint32_t die = blockIdx.x & (kDies - 1u);
        auto border = [&](const uint32_t k) {   // (as a scalar: it came from a vector load)
            return (uint32_t)__builtin_amdgcn_readfirstlane((int)a.counters[kSpanWord + k]) >> lg;
        };
        const uint32_t b0 = border(die), b1 = border(die + 1u), b2 = border(die + kDies);
        const uint32_t b3 = die + 1u < kDies ? border(die + kDies + 1u) : nblk;
        i = (blockIdx.x / kDies) * (kSegThreads / kWave) + wave;
        step = nwaves / kDies;
        n1 = b1 - b0;
        n = n1 + (b3 - b2);
        first = b0;
        again = b2 - n1;
    }
    WT* tables = static_cast<WT*>(a.tables);
    const int fetch_log2 = kFetch ? 6 : lg;
    for (; i < n; i += step << (fetch_log2 - lg)) {
        // ---- one row per lane, of the next pass or (kFetch) the next 64 / 2^lg: bounds, key, table, width, moment
        const uint32_t i_l = i + ((uint32_t)lane >> lg) * step;
        const uint32_t u = ((i_l + (i_l < n1 ? first : again)) << lg) + ((uint32_t)lane & ((1u << lg) - 1u));
        const bool row_on = i_l < n && u < U && lane >> fetch_log2 == 0;
        uint32_t s = 0, e = e_all, key = 0;
        if (row_on) {
            s = a.seg_start[u];
            e = a.seg_start[u + 1];
            key = a.keys_unique[u];
        }
        bool live = row_on && e != s && e - s <= a.long_min && key < a.total_rows;
        int t = 0, D = 4;
        float v = 0.f;
        if (live) {
            t = table_of_row(a, s, key);
            D = a.D_off[t + 1] - a.D_off[t];
            if (D > 256) {   // a wider table's row: the one-wavefront-per-row kernel takes it
                live = false;
                D = 4;
            } else {
                v = a.state ? a.state[key] : 0.f;
            }
        }
        // a window of 64 lookups of one table, lane's lookup win + lane: loaded once for all the short rows that lie in it
        uint32_t win = 0, my_b = 0;
        int win_t = -1;
        float my_s = 1.f;
        auto load_window = [&](const int r, const uint32_t s0, const int t_w, const uint32_t row0) {
            win = s0;
            win_t = t_w;
            const uint32_t at = s0 + (uint32_t)lane;
            const uint32_t end = bcast_lane(e, r | ((1 << lg) - 1));   // of the lookups of row r's pass
            const uint32_t bag = a.bag_sorted[at < end ? at : end - 1u];
            my_b = bag - row0;
            my_s = bag_scale<MEAN>(a.offsets, bag);
        };
        uint64_t todo = __ballot(live);
        while (todo != 0ull) {
            const int r = __ffsll((unsigned long long)todo) - 1;
            const RowGeom g = row_geom(bcast_lane(D, r));   // r is the same in all lanes: scalar reads
            const uint32_t s_r = bcast_lane(s, r);
            const uint32_t len_r = bcast_lane(e, r) - s_r;
            if (len_r > (uint32_t)kWave) {
                // ---- medium row: the whole wavefront reduces it
                const uint32_t key_r = bcast_lane(key, r);
                const int t_r = bcast_lane(t, r);
                const float v_r = bcast_lane(v, r);
                float acc[1][4] = {{0.f, 0.f, 0.f, 0.f}};
                const GradAddr ga = grad_addr(a, t_r, g.D);
                segment_reduce<1, MEAN, GT, kSegWaves>(acc, g, static_cast<const GT*>(a.grad_out) + ga.base, ga.pitch, ga.row0,
                                            a.bag_sorted, a.offsets, s_r, s_r + len_r);
                fold_groups<1>(acc, g);
                WT* wrow = tables + a.w_off[t_r] + ((int64_t)key_r - a.row_base[t_r]) * g.D;
                adagrad_row<WT, 1>(acc, g, wrow, a.state + key_r, v_r, g.sub == 0, a.lr, a.eps, a.inv_c, a.state == nullptr);
                todo &= todo - 1ull;
                continue;
            }
            // ---- short rows: rows r .. r+k-1 of one pass share the table of row r and have at most 64 lookups in total
            const int t_r = bcast_lane(t, r);
            const GradAddr ga = grad_addr(a, t_r, g.D);
            const GT* const gcol = static_cast<const GT*>(a.grad_out) + ga.base;
            WT* const wtab = tables + a.w_off[t_r];
            const uint32_t rb = (uint32_t)a.row_base[t_r];
            const bool col_on = g.lc < g.D;
            const uint32_t lane_col = col_on ? (uint32_t)g.lc : 0u;   // (what other lanes sum is not used)
            if (g.G == 1) {
                // a row as wide as the wavefront (more than 128 columns): one row per round, so its bookkeeping is the same in
                // all lanes and stays on the scalar unit (key, bag ids, addresses)
                const uint32_t key_r = bcast_lane(key, r);
                const float v_r = bcast_lane(v, r);
                if (win_t != t_r || s_r + len_r - win > (uint32_t)kWave) load_window(r, s_r, t_r, ga.row0);
                WT* const wrow = wtab + (uint64_t)(key_r - rb) * (uint32_t)g.D;
                typename RowIO<WT>::raw4_t wraw;
                if constexpr (kAhead) wraw = stream ? RowIO<WT>::template load4_raw<true>(wrow + lane_col) : RowIO<WT>::load4_raw(wrow + lane_col);
                float acc[1][4] = {{0.f, 0.f, 0.f, 0.f}};
                add_short<kSegUnroll, true, MEAN, GT>(acc, gcol, ga.pitch, lane_col, my_b, my_s, s_r - win, len_r, len_r);
                if constexpr (kAhead)
                    adagrad_row_loaded<WT>(acc, g, wrow, wraw, a.state + key_r, v_r, true, a.lr, a.eps, a.inv_c, a.state == nullptr, stream);
                else adagrad_row<WT, 1>(acc, g, wrow, a.state + key_r, v_r, true, a.lr, a.eps, a.inv_c, a.state == nullptr, stream);
                todo &= todo - 1ull;
                continue;
            }
            const bool q = live && t == t_r && lane >= r && lane < r + g.G && (lane ^ r) >> lg == 0 && (e - s_r) <= (uint32_t)kWave;
            const uint64_t m = __ballot(q) >> r;                       // bit j: row r+j qualifies
            const int k = __ffsll((unsigned long long)(~m)) - 1;       // trailing ones, 1 .. 2^lg
            if (win_t != t_r || bcast_lane(e, r + k - 1) - win > (uint32_t)kWave) load_window(r, s_r, t_r, ga.row0);
            // this lane group's row
            const bool gon = g.sub < k;
            const int gi = (r + g.sub) & (kWave - 1);
            const uint32_t gs = __shfl(s, gi, kWave);
            // cross-lane reads stay outside any lane-dependent condition: a lane that sits out cannot be read from
            const uint32_t glen_any = __shfl(e, gi, kWave) - gs;
            const uint32_t glen = gon ? glen_any : 0u;
            const uint32_t gkey = __shfl(key, gi, kWave);
            const float gv = __shfl(v, gi, kWave);
            WT* const wrow = wtab + (uint64_t)(gkey - rb) * (uint32_t)g.D;
            const uint32_t lmax = (uint32_t)wave_max_i32((int)glen);   // longest row of the round (wave-uniform loop bound)
            float acc[1][4] = {{0.f, 0.f, 0.f, 0.f}};
            add_short<kSideUnroll, false, MEAN, GT>(acc, gcol, ga.pitch, lane_col, my_b, my_s, gs - win, lmax, glen);
            adagrad_row<WT, 1>(acc, g, wrow, a.state + gkey, gv, gon, a.lr, a.eps, a.inv_c, a.state == nullptr, stream);
            todo &= ~(((1ull << k) - 1ull) << r);
        }
    }
}

// ---- the same for tables wider than 256 columns: one wavefront per row ----------------------------
template <typename WT, bool MEAN, typename GT>
__global__ __launch_bounds__(kSegThreads, 4) void seg_update_wide_kernel(const SegArgs a) {
    copy_hint(a);
    if (a.counters[4] != 0u) return;
    reduce_parts<true, MEAN, GT, 4>(a);
    const uint32_t U = a.counters[0];
    const uint32_t nwaves = gridDim.x * (kSegThreads / kWave);
    WT* tables = static_cast<WT*>(a.tables);
    for (uint32_t u = blockIdx.x * (kSegThreads / kWave) + (threadIdx.x >> 6); u < U; u += nwaves) {
        const uint32_t s = a.seg_start[u];
        const uint32_t e = a.seg_start[u + 1];
        const uint32_t key = a.keys_unique[u];
        if (key >= a.total_rows) continue;  // invalid ids: no row
        if (e - s > a.long_min) continue;   // long rows are reduced part by part
        const int t = table_of_row(a, s, key);
        const int d0 = a.D_off[t];
        if (a.D_off[t + 1] - d0 <= 256) continue;   // done by seg_update_kernel
        const RowGeom g = row_geom(a.D_off[t + 1] - d0);
        WT* wrow = tables + a.w_off[t] + ((int64_t)key - a.row_base[t]) * g.D;
        float acc[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c][0] = acc[c][1] = acc[c][2] = acc[c][3] = 0.f;
        const GradAddr ga = grad_addr(a, t, g.D);
        segment_reduce<4, MEAN, GT>(acc, g, static_cast<const GT*>(a.grad_out) + ga.base, ga.pitch, ga.row0, a.bag_sorted,
                                    a.offsets, s, e);
        fold_groups<4>(acc, g);
        adagrad_row<WT, 4>(acc, g, wrow, a.state + key, a.state ? a.state[key] : 0.f, g.sub == 0, a.lr, a.eps, a.inv_c,
                           a.state == nullptr);
    }
}

// ---- one workgroup per long row: add its partial sums, then the step ----------------------------------
// Wavefront w adds slots w, w+4, ... in ascending order, the four sums are added in wavefront order, and
// wavefront 0 applies the step: a fixed order, so the result does not depend on scheduling.
// A dense row whose sum is not finite is reduced again from its own lookups, each wavefront a quarter of them: its partial
// sums hold count * gradient for every bag of the table, and a count of zero times an infinity or NaN of a bag that the row
// is not in is NaN.  So a non-finite gradient reaches the rows of its own bag and no others.  The same for a sum so small that
// the last bits of its terms lay below the smallest number of a bfloat16 piece (2^-133): they would be missing from it (with
// gradients around 1e-36 the relative error of such sums was 5e-5, and 7e-4 under mean pooling).  Only a column whose every
// term is below that number still sums to zero.
constexpr float kDenseSmall = 0x1p-80f;   // 2^53 times as large: 2^29 terms lose less than the sum's own rounding
constexpr uint32_t kAgainRun = 256;       // lookups of one running sum
__device__ __forceinline__ bool sum_unsafe(const float x) {
    return !(fabsf(x) <= 3.402823466e38f) || (fabsf(x) < kDenseSmall && x != 0.f);
}
template <typename WT, bool MEAN, typename GT>
__global__ __launch_bounds__(kSegThreads) void seg_long_update_kernel(const SegArgs a) {
    __shared__ __align__(16) float s_sum[kSegThreads / kWave][1024];
    if (a.counters[4] != 0u) return;
    const uint32_t nlong = a.counters[1] < a.cap_long ? a.counters[1] : a.cap_long;
    WT* tables = static_cast<WT*>(a.tables);
    const int wv = threadIdx.x >> 6;
    constexpr uint32_t kW = kSegThreads / kWave;
    for (uint32_t li = blockIdx.x; li < nlong; li += gridDim.x) {
        const uint4 ent = a.long_list[li];
        const uint32_t key = a.keys_unique[ent.x];
        const int t = (int)ent.w;
        const int D = a.D_off[t + 1] - a.D_off[t];
        const bool dense = (ent.z & kDenseFlag) != 0u;
        const uint32_t nch = dense ? a.dense_chunks : ent.z;   // partial sums of the row
        const uint32_t pitch = dense ? a.dense_n[t] * (uint32_t)D : (uint32_t)a.maxD;
        // here all 64 lanes cover the row (or a 256-column part of it); groups are not used
        RowGeom g;
        g.D = D; g.LPR = kWave; g.G = 1; g.sub = 0; g.lc = lane_id() * 4;
        float acc[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            acc[c][0] = acc[c][1] = acc[c][2] = acc[c][3] = 0.f;
            const int col = g.lc + c * 256;
            if (col < D) {
                const float* src = (dense ? a.dense_partial + (size_t)ent.y * 4u : a.partial + (size_t)ent.y * a.maxD) + col;
                for (uint32_t k = (uint32_t)wv; k < nch; k += 8 * kW) {   // eight loads in flight
                    float4 v[8];
#pragma unroll
                    for (uint32_t q = 0; q < 8; ++q) {
                        const uint32_t kk = k + q * kW;
                        v[q] = *reinterpret_cast<const float4*>(src + (size_t)(kk < nch ? kk : (uint32_t)wv) * pitch);
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 8; ++q)
                        if (k + q * kW < nch) {
                            acc[c][0] += v[q].x; acc[c][1] += v[q].y; acc[c][2] += v[q].z; acc[c][3] += v[q].w;
                        }
                }
                *reinterpret_cast<float4*>(&s_sum[wv][col]) = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
            }
        }
        __syncthreads();
        if (dense) {   // (the same for the whole workgroup, and so is what the wavefronts find in s_sum)
            bool again = false;
            for (int col = g.lc; col < D; col += 256) {
                float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (uint32_t w2 = 0; w2 < kW; ++w2) {
                    const float4 o = *reinterpret_cast<const float4*>(&s_sum[w2][col]);
                    sum.x += o.x; sum.y += o.y; sum.z += o.z; sum.w += o.w;
                }
                again |= sum_unsafe(sum.x) || sum_unsafe(sum.y) || sum_unsafe(sum.z) || sum_unsafe(sum.w);
            }
            if (__any(again)) {
                __syncthreads();   // (all wavefronts have read s_sum)
                const uint32_t s0 = a.seg_start[ent.x];
                const uint64_t len = a.seg_start[ent.x + 1] - s0;
                const uint32_t lo = s0 + (uint32_t)(len * (uint32_t)wv / kW);
                const uint32_t hi = s0 + (uint32_t)(len * ((uint32_t)wv + 1u) / kW);
                const GradAddr ga = grad_addr(a, t, D);
#pragma unroll 1
                for (int c0 = 0; c0 < D; c0 += 256) {
                    RowGeom gc = g;
                    gc.D = D - c0;
                    float4 all = make_float4(0.f, 0.f, 0.f, 0.f);
                    for (uint32_t p = lo; p < hi; p += kAgainRun) {
                        float sum[1][4] = {{0.f, 0.f, 0.f, 0.f}};
                        segment_reduce<1, MEAN, GT>(sum, gc, static_cast<const GT*>(a.grad_out) + ga.base + c0, ga.pitch, ga.row0,
                                                    a.bag_sorted, a.offsets, p, hi - p < kAgainRun ? hi : p + kAgainRun);
                        all.x += sum[0][0]; all.y += sum[0][1]; all.z += sum[0][2]; all.w += sum[0][3];
                    }
                    if (c0 + g.lc < D) *reinterpret_cast<float4*>(&s_sum[wv][c0 + g.lc]) = all;
                }
                __syncthreads();
            }
        }
        if (wv == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int col = g.lc + c * 256;
                if (col < D) {
                    const float4 first = *reinterpret_cast<const float4*>(&s_sum[0][col]);
                    acc[c][0] = first.x; acc[c][1] = first.y; acc[c][2] = first.z; acc[c][3] = first.w;
#pragma unroll
                    for (int w2 = 1; w2 < kSegThreads / kWave; ++w2) {
                        const float4 o = *reinterpret_cast<const float4*>(&s_sum[w2][col]);
                        acc[c][0] += o.x; acc[c][1] += o.y; acc[c][2] += o.z; acc[c][3] += o.w;
                    }
                }
            }
            WT* wrow = tables + a.w_off[t] + ((int64_t)key - a.row_base[t]) * D;
            adagrad_row<WT, 4>(acc, g, wrow, a.state + key, a.state ? a.state[key] : 0.f, true, a.lr, a.eps, a.inv_c,
                               a.state == nullptr);
        }
        __syncthreads();
    }
}

// the two row-update kernels and the hot-row reduction for one gradient element type
template <typename GT>
static void launch_row_updates(const tbe_handle* h, const SegArgs& a, bool mean, bool narrow, bool wide,
                               hipStream_t s) {
    const bool f32 = h->dtype == TBE_F32;
    if (narrow) {
        // every CU filled once; 7 wavefronts per SIMD for 32-bit gradients on binary16 tables when most of their rows
        // are as wide as the wavefront (measured: 20.2 -> 19.8 ms there, but 2.43 -> 2.55 ms on fp32 tables of the
        // same widths, which therefore keep 8)
        if (sizeof(GT) == 4 && !f32 && h->seg_mostly_wavefront_rows) {
            const unsigned grid = kSegBlocks7;
            if (mean) seg_update_kernel<__half, true, GT, 7><<<grid, kSegThreads, 0, s>>>(a);
            else seg_update_kernel<__half, false, GT, 7><<<grid, kSegThreads, 0, s>>>(a);
        } else {
            const unsigned grid = kSegBlocks;
            if (f32) {
                if (mean) seg_update_kernel<float, true, GT, 8><<<grid, kSegThreads, 0, s>>>(a);
                else seg_update_kernel<float, false, GT, 8><<<grid, kSegThreads, 0, s>>>(a);
            } else {
                if (mean) seg_update_kernel<__half, true, GT, 8><<<grid, kSegThreads, 0, s>>>(a);
                else seg_update_kernel<__half, false, GT, 8><<<grid, kSegThreads, 0, s>>>(a);
            }
        }
    }
    if (wide) {
        if (f32) {
            if (mean) seg_update_wide_kernel<float, true, GT><<<kSegBlocks, kSegThreads, 0, s>>>(a);
            else seg_update_wide_kernel<float, false, GT><<<kSegBlocks, kSegThreads, 0, s>>>(a);
        } else {
            if (mean) seg_update_wide_kernel<__half, true, GT><<<kSegBlocks, kSegThreads, 0, s>>>(a);
            else seg_update_wide_kernel<__half, false, GT><<<kSegBlocks, kSegThreads, 0, s>>>(a);
        }
    }
}

template <typename GT>
static void launch_long_update(const tbe_handle* h, const SegArgs& a, bool mean, unsigned grid, hipStream_t s) {
    if (h->dtype == TBE_F32) {
        if (mean) seg_long_update_kernel<float, true, GT><<<grid, kSegThreads, 0, s>>>(a);
        else seg_long_update_kernel<float, false, GT><<<grid, kSegThreads, 0, s>>>(a);
    } else {
        if (mean) seg_long_update_kernel<__half, true, GT><<<grid, kSegThreads, 0, s>>>(a);
        else seg_long_update_kernel<__half, false, GT><<<grid, kSegThreads, 0, s>>>(a);
    }
}

SegArgs seg_args(const tbe_handle* h, const Workspace& w, char* ws, const void* offsets, int idx32, int32_t B, int seq) {
    SegArgs a;
    const int sorted = w.sort.passes & 1;
    a.keys_unique = reinterpret_cast<const uint32_t*>(ws + w.vals[sorted ^ 1]);
    a.seg_start = reinterpret_cast<const uint32_t*>(ws + w.seg_start);
    a.counters = reinterpret_cast<uint32_t*>(ws + w.counters);
    a.bag_sorted = reinterpret_cast<const uint32_t*>(ws + w.vals[sorted]);   // the sorted payload stream
    a.offsets = OffsetWords{static_cast<const uint32_t*>(offsets), idx32 ? 0 : 1};
    a.grad_out = nullptr;
    a.seq_gbase = reinterpret_cast<int64_t*>(ws + w.seq_gbase);
    a.seq = seq;
    a.D_off = h->d_D_off;
    a.row_base = h->d_row_base;
    a.w_off = h->d_w_off;
    a.T = h->T;
    a.B = B;
    a.sumD = h->sumD;
    a.maxD = h->maxD;
    a.total_rows = (uint32_t)h->total_rows;
    a.stream_from = 0;
    a.row_bytes = (uint32_t)(h->total_elems / h->total_rows) * (h->dtype == TBE_F32 ? 4u : 2u);
    a.lr = a.eps = a.inv_c = 0.f;
    a.tables = nullptr;
    a.state = nullptr;
    a.long_min = w.long_min;
    a.part = w.part;
    a.cap_long = (uint32_t)w.cap_long;
    a.long_rows = reinterpret_cast<const uint2*>(ws + w.long_rows);
    a.long_list = reinterpret_cast<uint4*>(ws + w.long_list);
    a.unit_list = reinterpret_cast<uint2*>(ws + w.unit_list);
    a.partial = reinterpret_cast<float*>(ws + w.partial);
    const bool hint = h->d_hot_ids && !seq;
    a.hot_ids = hint ? reinterpret_cast<uint32_t*>(ws + w.hot_ids) : nullptr;
    a.hot_n = hint ? reinterpret_cast<uint32_t*>(ws + w.hot_n) : nullptr;
    a.hint_ids = hint ? h->d_hot_ids : nullptr;
    a.hint_n = hint ? h->d_hot_n : nullptr;
    // side by side: 64 / (lanes per row) rows of the widest table up to 256 columns
    a.min_rows_log2 = h->maxD > 128 ? 0 : (h->maxD > 64 ? 1 : (h->maxD > 32 ? 2 : 3));
    a.long_pass_need = h->maxD <= 8 ? kLongPassNeedNarrow : kLongPassNeed;
    a.long_spans = 0;
    const bool dense = w.dense && !seq;
    a.dense_n = dense ? reinterpret_cast<uint32_t*>(ws + w.dense_n) : nullptr;
    a.dense_rows = reinterpret_cast<uint32_t*>(ws + w.dense_rows);
    a.dense_index = reinterpret_cast<uint32_t*>(ws + w.dense_index);
    a.dense_tab = reinterpret_cast<uint2*>(ws + w.dense_tab);
    a.dense_partial = reinterpret_cast<float*>(ws + w.dense_partial);
    a.dense_blocks = w.dense_blocks;
    a.dense_chunks = w.dense_chunks;
    a.dense_per_chunk = w.dense_per_chunk;
    return a;
}

// Whether the rows that are streamed gain by it, in all, as far as the host can know which those are.  Rows that fill whole 64-byte
// pieces do, and those so wide that the first and the last piece count little.  Of other rows neighbours share pieces, and past the caches
// a part of a piece is a read and a write of its own: that costs a row about as much as 256 bytes of the others gain.  8 tables, 564 MB
// of rows in use with one or two lookups each, update alone, cached / streamed, us: fp32 of 8, 12, 16, 20, 24, 32, 36, 40 columns 1175 984
// 636 732 628 385 569 515 / 1422 1172 594 853 711 349 629 529; of 48, 52, 84, 92, 100, 104, 116, 132 436 488 441 415 383 396 396 489 / 399
// 507 449 421 394 377 380 474; binary16 of 16, 24, 32, 40, 56, 120, 136, 200 1027 990 669 888 678 588 895 661 / 1229 1149 653 918 759 594
// 890 648.  Asked for every table in the kernel itself, it cost the loop the scalar registers that it spills: 886 -> 991 at the 40.
static bool rows_gain_by_streams(const tbe_handle* h, const int64_t n) {
    const int64_t size = h->dtype == TBE_F32 ? 4 : 2, each = n / h->T + 1;
    int64_t gain = 0;
    for (int t = 0; t < h->T; ++t) {
        if (h->D[t] > 256) continue;   // (never streamed)
        const int64_t bytes = h->D[t] * size;
        const bool good = ((h->w_off[t] * size | bytes) & 63) == 0 || bytes > 400 || h->D[t] > 128;
        gain += (h->rows[t] < each ? h->rows[t] : each) * (good ? bytes : -256);
    }
    return gain > 0;
}

hipError_t launch_segment_update(const tbe_handle* h, const Workspace& w, char* ws, const void* grad_out, int grad_io,
                                 const void* offsets, int idx32, int32_t B, tbe_pooling pooling, float lr, float eps, float c,
                                 void* tables, float* state, int seq, hipStream_t s) {
    SegArgs a = seg_args(h, w, ws, offsets, idx32, B, seq);
    a.grad_out = grad_out;
    a.lr = lr;
    a.eps = eps;
    a.inv_c = 1.0f / c;
    a.tables = tables;
    a.state = state;
    const uint64_t grad_bytes = (uint64_t)B * (uint64_t)h->sumD * (grad_io == 0 ? 4u : 2u);   // (of sequences next to nothing: they are read once)
    a.stream_from = grad_bytes < kInfinityCacheBytes ? kInfinityCacheBytes - grad_bytes : 0u;
    if ((uint64_t)(w.n < h->total_rows ? w.n : h->total_rows) * a.row_bytes > a.stream_from && !rows_gain_by_streams(h, w.n)) a.stream_from = UINT64_MAX;
    a.long_spans = long_spans(h, B, seq, grad_io == 0 ? 4u : 2u);
    const bool mean = pooling == TBE_MEAN;
    if (a.dense_n) {
        LaunchTimer tm(h, s, "seg_dense_partial");
        launch_dense(a, grad_io, mean, s);
        tm.done();
    }
    // Rows of tables up to 256 columns wide go to the kernel that takes them in passes of up to 32, rows of wider tables
    // to the one-wavefront-per-row kernel; a handle that holds both kinds runs both, each skipping the other's rows.
    const bool narrow = h->minD <= 256;
    const bool wide = h->maxD > 256;
    {
        LaunchTimer tm(h, s, "seg_update");
        if (grad_io == 0) launch_row_updates<float>(h, a, mean, narrow, wide, s);
        else if (grad_io == 1) launch_row_updates<__half>(h, a, mean, narrow, wide, s);
        else launch_row_updates<bf16_t>(h, a, mean, narrow, wide, s);
        tm.done();
    }
    if ((int64_t)w.n > (int64_t)w.long_min) {   // (no row of a smaller batch can be long)
        LaunchTimer tm(h, s, "seg_long_update");
        // one row per workgroup and round, a dependent chain of loads each: enough workgroups to fill every CU's slots
        const unsigned grid = (unsigned)(w.cap_long < kSegBlocks ? w.cap_long : kSegBlocks);
        if (grad_io == 0) launch_long_update<float>(h, a, mean, grid, s);
        else if (grad_io == 1) launch_long_update<__half>(h, a, mean, grid, s);
        else launch_long_update<bf16_t>(h, a, mean, grid, s);
        tm.done();
    }
    return hipGetLastError();
}

}  // namespace tbe
