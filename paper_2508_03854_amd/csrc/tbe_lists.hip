// Between the sort and the row updates: what is known of the batch's long rows from the ids alone.  Run by the calls that
// sort a batch, so that applying a step needs none of it again.
//
// The run-length kernels leave the rows with more than long_min lookups in key order, i.e. table by table.  One workgroup
// per table lists its own:
//   - the kHotRows longest of those with more than kHotMin lookups, a hint for the next forward (with shorter rows listed, as
//     long_min falls with the batch, the forward of 256 tables x 512 bags of 4 ids, 16 columns, went from 16.4 to 18.6 us);
//   - the dense rows: up to kDenseRows longest, if together they hold at least two lookups per bag of a gradient block that
//     no L2 holds.  Streaming the block once and adding every bag's gradient to all of them (tbe_dense.hip) then reads less
//     than gathering it once per lookup;
//   - the others, cut into parts of about `part` lookups, one work unit and one partial sum each.
// Partial-sum slots need no counting: row number i of the list with its first lookup at sorted position s gets the slots
// from s / part + i on.  A row of len lookups takes ceil(len / part) <= (s + len) / part - s / part + 1 of them, so the
// next row's start behind its own, and n lookups in rows longer than long_min need at most n / part + n / long_min.
//
// Bound: latency - a table has at most a few thousand long rows, and the launch is one chain of dependent loads.  Hence one
// launch (two with dense rows) in place of the up to 20 that counted, scanned, filled, ranked and sliced before.  With parts
// sized to the batch the whole step went from 67 to 46 us (one table, 10 k lookups), 353 to 163 us (ten tables of odd widths,
// 47 k lookups, mean pooling) and 254 to 193 us (26 tables, 1.2 M lookups).
#include "tbe_rows.h"

namespace tbe {

constexpr int kListThreads = 1024;
constexpr uint32_t kListRank = 1024;   // long rows of one table that are ranked; a table with more lists the first kHotRows as hot and has no dense rows

// first i in [0, n) with rows[i].y >= x, or n; a whole wavefront, 64 probes per round
__device__ __forceinline__ uint32_t wave_lower_bound_key(const uint2* __restrict__ rows, const uint32_t n, const int64_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint64_t i = lo + (uint64_t)(lane_id() + 1) * step - 1;
        const bool ge = i < hi ? (int64_t)rows[i].y >= x : true;
        const uint64_t m = __ballot(ge);
        if (m == 0ull) return hi;
        const uint32_t f = (uint32_t)__ffsll((unsigned long long)m) - 1u;
        const uint64_t i_f = lo + (uint64_t)(f + 1u) * step - 1;
        lo += f * step;
        hi = i_f < hi ? (uint32_t)i_f : hi;
    }
    return lo;
}

__device__ __forceinline__ uint32_t row_parts(const SegArgs& a, const uint32_t len) {
    const uint32_t c = (len + a.part - 1u) / a.part;
    return c < (uint32_t)kMaxParts ? c : (uint32_t)kMaxParts;
}

// Non-pooled mode: element offset of every table's gradient block, minus start_t * D_t, so that the kernels address a lookup
// by its original position alone.  If offsets is not ascending from 0 to nnz, or the blocks do not fit grad_elems, no
// gradient address can be trusted: the batch is then flagged as an index error and counters[4] turns the kernels that
// follow into no-ops.
template <typename IT>
__device__ __forceinline__ void seq_blocks(const SegArgs& a, const IT* __restrict__ offsets, const int64_t nnz,
                                           const int64_t grad_elems, int32_t* __restrict__ err) {
    __shared__ int64_t s_sum[kListThreads / kWave];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    int64_t carry = 0;
    bool ok = (int64_t)offsets[0] == 0 && (int64_t)offsets[a.T] == nnz;
    for (int t0 = 0; t0 < a.T; t0 += kListThreads) {
        const int t = t0 + (int)threadIdx.x;
        int64_t s0 = 0, e = 0, D = 0;
        if (t < a.T) {
            s0 = (int64_t)offsets[t];
            const int64_t s1 = (int64_t)offsets[t + 1];
            D = a.D_off[t + 1] - a.D_off[t];
            ok = ok && s1 >= s0;
            e = (s1 > s0 ? s1 - s0 : 0) * D;
        }
        int64_t inc = e;   // inclusive scan over the wavefront
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t l32 = __shfl_up((uint32_t)(inc & 0xFFFFFFFFll), o, kWave);
            const uint32_t h32 = __shfl_up((uint32_t)((uint64_t)inc >> 32), o, kWave);
            if (lane >= o) inc += (int64_t)(((uint64_t)h32 << 32) | l32);
        }
        if (lane == kWave - 1) s_sum[w] = inc;
        __syncthreads();
        int64_t before = carry, all = 0;
        for (int i = 0; i < kListThreads / kWave; ++i) {
            before += i < w ? s_sum[i] : 0;
            all += s_sum[i];
        }
        if (t < a.T) a.seq_gbase[t] = before + inc - e - s0 * D;
        carry += all;
        __syncthreads();
    }
    if (!ok || carry > grad_elems) {
        a.counters[4] = 1u;
        atomicOr(err, 1);
    }
}

// grid: one workgroup per table, and in non-pooled mode one more for the gradient blocks
template <typename IT>
__global__ __launch_bounds__(kListThreads) void list_rows_kernel(const SegArgs a, const IT* __restrict__ offsets,
                                                                 const int64_t nnz, const int64_t grad_elems,
                                                                 int32_t* __restrict__ err) {
    __shared__ uint32_t s_len[kListRank], s_start[kListRank], s_row[kListRank], s_rank[kListRank];
    __shared__ uint32_t smem[kListThreads / kWave];
    __shared__ uint32_t s_range[2], s_sum, s_base, s_first;
    const int t = blockIdx.x;
    if (t == a.T) {
        seq_blocks<IT>(a, offsets, nnz, grad_elems, err);
        return;
    }
    const uint32_t nlong = a.counters[1] < a.cap_long ? a.counters[1] : a.cap_long;
    const uint32_t tid = threadIdx.x;
    if (tid < 2 * kWave) {
        const uint32_t i = wave_lower_bound_key(a.long_rows, nlong, a.row_base[t + (int)(tid >> 6)]);
        if ((tid & (kWave - 1)) == 0) s_range[tid >> 6] = i;
    }
    if (tid == 0) s_sum = 0u;
    __syncthreads();
    const uint32_t i0 = s_range[0], n = s_range[1] - s_range[0];
    const uint32_t rb = (uint32_t)a.row_base[t];
    const uint32_t D = (uint32_t)(a.D_off[t + 1] - a.D_off[t]);
    if (tid == 0) {
        if (a.hot_n) a.hot_n[t] = 0u;
        if (a.dense_n) a.dense_n[t] = 0u;
    }
    if (n == 0u) return;
    const bool ranked = n <= kListRank;
    uint32_t nd = 0;   // dense rows
    if (ranked) {
        uint32_t my_len = 0, my_key = 0;
        if (tid < n) {
            const uint2 r = a.long_rows[i0 + tid];
            const uint32_t s0 = a.seg_start[r.x];
            my_len = a.seg_start[r.x + 1] - s0;
            my_key = r.y;
            s_len[tid] = my_len;
            s_start[tid] = s0;
            s_row[tid] = r.x;
        }
        __syncthreads();
        if (tid < n) {   // longest first, ties by key (the list is ascending by key)
            uint32_t rank = 0;
            for (uint32_t j = 0; j < n; ++j) {
                const uint32_t l = s_len[j];
                rank += (l > my_len || (l == my_len && j < tid)) ? 1u : 0u;
            }
            s_rank[tid] = rank;
            if (a.hot_ids && rank < (uint32_t)kHotRows && my_len > kHotMin) a.hot_ids[(size_t)t * kHotRows + rank] = my_key - rb;
            if (rank < (uint32_t)kDenseRows) atomicAdd(&s_sum, my_len < 0x01000000u ? my_len : 0x01000000u);
        }
        const uint32_t hot = (uint32_t)__syncthreads_count(tid < n && my_len > kHotMin);
        if (a.hot_n && tid == 0) a.hot_n[t] = hot < (uint32_t)kHotRows ? hot : (uint32_t)kHotRows;
        if (a.dense_n && dense_block((uint32_t)a.B, D) && s_sum >= 2u * (uint32_t)a.B) nd = n < (uint32_t)kDenseRows ? n : (uint32_t)kDenseRows;
        if (tid == 0 && nd > 0u) {   // (which table gets which place decides nothing but addresses)
            a.dense_n[t] = nd;
            s_first = atomicAdd(&a.counters[2], nd * a.dense_chunks * (D / 4u));
            a.dense_tab[t] = make_uint2(atomicAdd(&a.counters[5], 1u), s_first);
        }
    } else if (a.hot_ids && tid < (uint32_t)kHotRows) {
        a.hot_ids[(size_t)t * kHotRows + tid] = a.long_rows[i0 + tid].y - rb;
        if (tid == 0) a.hot_n[t] = (uint32_t)kHotRows;
    }
    // parts of the rows that are not dense: their number first, then the table's place in the unit list (which tables come
    // first decides the order in which units are worked on, nothing else)
    uint32_t total = 0;
    for (uint32_t k0 = 0; k0 < n; k0 += kListThreads) {
        const uint32_t k = k0 + tid;
        uint32_t c = 0;
        if (k < n && !(ranked && s_rank[k] < nd)) {
            const uint32_t u = a.long_rows[i0 + k].x;
            c = row_parts(a, ranked ? s_len[k] : a.seg_start[u + 1] - a.seg_start[u]);
        }
        uint32_t tot;
        block_excl_scan<kListThreads>(c, smem, &tot);
        total += tot;
    }
    if (tid == 0) s_base = total > 0u ? atomicAdd(&a.counters[3], total) : 0u;
    __syncthreads();
    uint32_t base = s_base;
    for (uint32_t k0 = 0; k0 < n; k0 += kListThreads) {
        const uint32_t k = k0 + tid;
        uint32_t c = 0;
        if (k < n) {
            const uint32_t u = ranked ? s_row[k] : a.long_rows[i0 + k].x;
            const uint32_t s0 = ranked ? s_start[k] : a.seg_start[u];
            if (ranked && s_rank[k] < nd) {
                a.dense_rows[(size_t)t * kDenseRows + s_rank[k]] = i0 + k;
                a.long_list[i0 + k] = make_uint4(u, s_first + s_rank[k] * a.dense_chunks * (D / 4u), kDenseFlag, (uint32_t)t);
            } else {
                c = row_parts(a, ranked ? s_len[k] : a.seg_start[u + 1] - s0);
                a.long_list[i0 + k] = make_uint4(u, s0 / a.part + i0 + k, c, (uint32_t)t);
            }
        }
        uint32_t tot;
        const uint32_t at = base + block_excl_scan<kListThreads>(c, smem, &tot);
        for (uint32_t q = 0; q < c; ++q) a.unit_list[at + q] = make_uint2(i0 + k, q);
        base += tot;
    }
}

// Handles of very many tables (no hint, no dense rows): one thread per long row.
template <typename IT>
__global__ __launch_bounds__(kListThreads) void list_rows_flat_kernel(const SegArgs a, const IT* __restrict__ offsets,
                                                                      const int64_t nnz, const int64_t grad_elems,
                                                                      int32_t* __restrict__ err) {
    if (a.seq && blockIdx.x == gridDim.x - 1) {
        seq_blocks<IT>(a, offsets, nnz, grad_elems, err);
        return;
    }
    const uint32_t nlong = a.counters[1] < a.cap_long ? a.counters[1] : a.cap_long;
    const uint32_t i = blockIdx.x * kListThreads + threadIdx.x;
    if (i >= nlong) return;
    const uint2 r = a.long_rows[i];
    const uint32_t s0 = a.seg_start[r.x];
    const uint32_t c = row_parts(a, a.seg_start[r.x + 1] - s0);
    a.long_list[i] = make_uint4(r.x, s0 / a.part + i, c, (uint32_t)table_of_row(a, s0, r.y));
    const uint32_t at = atomicAdd(&a.counters[3], c);
    for (uint32_t q = 0; q < c; ++q) a.unit_list[at + q] = make_uint2(i, q);
}

// Where every block of kDenseBags bags starts in a dense row's segment.  The lookups of a table's dense rows, row after
// row, are shared out evenly to kIndexSplit workgroups; a lookup whose bag lies in a later block than its predecessor's
// writes the borders between them.  (A binary search per border is a chain of 17 dependent loads; this reads every lookup
// of a dense row once, coalesced.)
constexpr int kIndexSplit = 32;
__global__ __launch_bounds__(256) void dense_index_kernel(const SegArgs a) {
    __shared__ uint32_t s_start[kDenseRows], s_end[kDenseRows], s_pref[kDenseRows];
    __shared__ uint32_t smem[256 / kWave];
    const int t = blockIdx.x / kIndexSplit;
    const uint32_t y = blockIdx.x % kIndexSplit;
    const uint32_t nd = a.dense_n[t];
    if (nd == 0u) return;
    const uint32_t tid = threadIdx.x;
    uint32_t len = 0;
    if (tid < nd) {
        const uint32_t u = a.long_list[a.dense_rows[(size_t)t * kDenseRows + tid]].x;
        s_start[tid] = a.seg_start[u];
        s_end[tid] = a.seg_start[u + 1];
        len = s_end[tid] - s_start[tid];
    }
    uint32_t all;
    const uint32_t ex = block_excl_scan<256>(len, smem, &all);
    if (tid < (uint32_t)kDenseRows) s_pref[tid] = tid < nd ? ex : 0xFFFFFFFFu;
    __syncthreads();
    const uint32_t bag0 = (uint32_t)t * (uint32_t)a.B, place = a.dense_tab[t].x;
    const uint32_t e0 = (uint32_t)((uint64_t)all * y / kIndexSplit), e1 = (uint32_t)((uint64_t)all * (y + 1u) / kIndexSplit);
    constexpr int kU = 8;   // lookups in flight per thread
    for (uint32_t f = e0 + tid; f < e1; f += kU * 256) {
        uint32_t row[kU], p[kU], bag[kU], prev[kU];
#pragma unroll
        for (int q = 0; q < kU; ++q) row[q] = 0u;
#pragma unroll
        for (uint32_t step = kDenseRows / 2; step > 0u; step >>= 1)   // the row: last h < nd with s_pref[h] <= e
#pragma unroll
            for (int q = 0; q < kU; ++q)
                if (s_pref[row[q] + step] <= f + q * 256) row[q] += step;   // (s_pref[nd ..] is above every e)
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            const uint32_t e = f + q * 256 < e1 ? f + q * 256 : e1 - 1u;
            if (f + q * 256 >= e1) row[q] = nd - 1u;
            p[q] = f + q * 256 < e1 ? s_start[row[q]] + (e - s_pref[row[q]]) : s_start[nd - 1u];
            bag[q] = a.bag_sorted[p[q]];
            prev[q] = a.bag_sorted[p[q] > s_start[row[q]] ? p[q] - 1u : p[q]];
        }
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            if (f + q * 256 >= e1) continue;
            const bool first = p[q] == s_start[row[q]], last = p[q] + 1u == s_end[row[q]];
            const uint32_t b1 = (bag[q] - bag0) / kDenseBags;
            const uint32_t b0 = first ? 0u : (prev[q] - bag0) / kDenseBags + 1u;   // borders b0 .. b1 are p
            uint32_t* ix = a.dense_index + ((size_t)place * kDenseRows + row[q]) * (a.dense_blocks + 1u);
            for (uint32_t k = b0; k <= b1 && k <= a.dense_blocks; ++k) ix[k] = p[q];
            if (last)
                for (uint32_t k = b1 + 1u; k <= a.dense_blocks; ++k) ix[k] = p[q] + 1u;
        }
    }
}

hipError_t launch_lists(const tbe_handle* h, const Workspace& w, char* ws, const void* offsets, int idx32, int32_t B, int seq,
                        int64_t grad_elems, hipStream_t s) {
    const SegArgs a = seg_args(h, w, ws, offsets, idx32, B, seq);
    LaunchTimer tm(h, s, "seg_long_list");
    const int64_t nnz = w.n;
    if (h->T <= kMaxSortSegments) {
        const unsigned grid = (unsigned)(h->T + (seq ? 1 : 0));
        if (idx32) list_rows_kernel<int32_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int32_t*>(offsets), nnz, grad_elems, h->d_err);
        else list_rows_kernel<int64_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int64_t*>(offsets), nnz, grad_elems, h->d_err);
        if (a.dense_n) dense_index_kernel<<<(unsigned)(h->T * kIndexSplit), 256, 0, s>>>(a);
    } else {
        const unsigned grid = (unsigned)((w.cap_long + kListThreads - 1) / kListThreads + (seq ? 1 : 0));
        if (idx32) list_rows_flat_kernel<int32_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int32_t*>(offsets), nnz, grad_elems, h->d_err);
        else list_rows_flat_kernel<int64_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int64_t*>(offsets), nnz, grad_elems, h->d_err);
    }
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
