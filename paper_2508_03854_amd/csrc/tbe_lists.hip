// Between the sort and the row updates: what is known of the batch's long rows from the ids alone.  Run by the calls that
// sort a batch, so that applying a step needs none of it again.
//
// The run-length kernels leave the rows with more than long_min lookups in key order, i.e. table by table.  One workgroup
// per table lists its own:
//   - the kHotRows longest of those with more than kHotMin lookups, a hint for the next forward (with shorter rows listed, as
//     long_min falls with the batch, the forward of 256 tables x 512 bags of 4 ids, 16 columns, went from 16.4 to 18.6 us);
//   - the dense rows: up to kDenseRows longest, if together they hold at least two lookups per bag of a large gradient block
//     (dense_block).  Streaming the block once and adding every bag's gradient to all of them (tbe_dense.hip) then reads less
//     than gathering it once per lookup;
//   - the others, cut into parts of about `part` lookups, one work unit and one partial sum each.
// Partial-sum slots need no counting: row number i of the list with its first lookup at sorted position s gets the slots
// from s / part + i on.  A row of len lookups takes at most ceil(len / part) <= (s + len) / part - s / part + 1 of them, so the
// next row's start behind its own, and n lookups in rows longer than long_min need at most n / part + n / long_min.
//
// Bound: latency - most tables have at most a thousand long rows, ranked by one workgroup at one row per thread, and the launch
// is one chain of dependent loads; of more rows the longest are selected first (one table, 16.8 M lookups, Zipf 1.05: 20 us).  Hence one
// launch (two with dense rows) in place of the up to 20 that counted, scanned, filled, ranked and sliced before.  With parts
// sized to the batch the whole step went from 67 to 46 us (one table, 10 k lookups), 353 to 163 us (ten tables of odd widths,
// 47 k lookups, mean pooling) and 254 to 193 us (26 tables, 1.2 M lookups).
#include "tbe_rows.h"

namespace tbe {

constexpr int kListThreads = 1024;
constexpr uint32_t kListRank = 1024;   // long rows of one table that are ranked; of more, the kHotRows longest are found first
constexpr uint32_t kDenseMinLen = 64;  // dense rows have more lookups than this
static_assert(kDenseRows <= kHotRows && kHotRows <= (int)kListRank && kListRank <= (uint32_t)kListThreads, "one thread per ranked row");

// first i in [lo, hi) with ge(i), which is false before some i and true from it on, or hi; a whole wavefront, 64 probes per round
template <typename F>
__device__ __forceinline__ uint32_t wave_first(uint32_t lo, uint32_t hi, F ge) {
    while (lo < hi) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint64_t i = lo + (uint64_t)(lane_id() + 1) * step - 1;
        const uint64_t m = __ballot(i < hi ? ge((uint32_t)i) : true);
        if (m == 0ull) return hi;
        const uint32_t f = (uint32_t)__ffsll((unsigned long long)m) - 1u;
        const uint64_t i_f = lo + (uint64_t)(f + 1u) * step - 1;
        lo += f * step;
        hi = i_f < hi ? (uint32_t)i_f : hi;
    }
    return lo;
}

// Parts of a row.  Those finer than kCoarsePart lookups shorten the longest chain of loads, but cost the table's workgroup a unit each and
// the row's a sum: a row has at most kFineParts of them, and more only where parts of kCoarsePart make more.  Backward, us, with the passes
// and parts of 64 that a batch of any size can have / fine parts for all rows / this: 10 tables, 30000 lookups, nine tenths in one of 60
// rows, Zipf 1.3, 1024 columns 82 / 101 / 66; 8 x 512 columns, 1000 rows 73 / 76 / 58; 81 tables of 32 and 512, 16000 lookups 52 / 62 / 49;
// 30000 spread over these 74 / 56 / 56.  With at most 32 the same within 2 %, but 7200 of 8000 lookups in one of two tables of 1000 rows,
// 1024 columns, 49 where this takes 47.
constexpr uint32_t kFineParts = 64, kCoarsePart = 64;
__device__ __forceinline__ uint32_t row_parts(const SegArgs& a, const uint32_t len) {
    uint32_t c = (len + a.part - 1u) / a.part;
    if (a.part < kCoarsePart && c > kFineParts) {
        const uint32_t coarse = (len + kCoarsePart - 1u) / kCoarsePart;
        c = coarse > kFineParts ? coarse : kFineParts;
    }
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

__device__ __forceinline__ uint32_t long_row_len(const SegArgs& a, const uint32_t i) {
    const uint32_t u = a.long_rows[i].x;
    return a.seg_start[u + 1] - a.seg_start[u];
}

// The lengths of a table's long rows [i0, i0 + n), row k0 + thread for k0 = 0, kListThreads, ...: the first HELD rounds in
// registers (a length is two dependent loads away), the others loaded again by every pass.  Called by the whole workgroup.
template <int HELD>
struct Lengths {
    static constexpr int kHeld = HELD;
    uint32_t held[kHeld], u0, s0;   // u0, s0: unique row and first lookup of the first round's row
    __device__ __forceinline__ void load(const SegArgs& a, const uint32_t i0, const uint32_t n) {
#pragma unroll
        for (int q = 0; q < kHeld; ++q) {
            const uint32_t k = (uint32_t)q * kListThreads + threadIdx.x;
            held[q] = 0u;
            if (k - (uint32_t)lane_id() < n) {   // (a wavefront without a row loads nothing)
                const uint32_t u = a.long_rows[i0 + (k < n ? k : n - 1u)].x;
                const uint32_t s = a.seg_start[u], len = a.seg_start[u + 1] - s;
                held[q] = k < n ? len : 0u;
                if (q == 0) {
                    u0 = u;
                    s0 = s;
                }
            }
        }
    }
    // f(k, length) for k of every round, length 0 behind the end (no long row is as short)
    template <typename F>
    __device__ __forceinline__ void each(const SegArgs& a, const uint32_t i0, const uint32_t n, F f) const {
#pragma unroll
        for (int q = 0; q < kHeld; ++q)
            if ((uint32_t)q * kListThreads < n) f((uint32_t)q * kListThreads + threadIdx.x, held[q]);
        for (uint32_t k0 = kHeld * kListThreads; k0 < n; k0 += kListThreads) {
            const uint32_t k = k0 + threadIdx.x;
            f(k, k < n ? long_row_len(a, i0 + k) : 0u);
        }
    }
};

struct ListLds {
    uint32_t len[kListRank], k[kHotRows], hist[256], scan[kListThreads / kWave];
    uint32_t sum, base, first, cut_len, cut_k;
};

// The kHotRows longest of the n > kListRank long rows of a table, ties by their place in the list (the key): their places k in
// list order into S->k, their lengths into S->len.  A radix selection finds the length of the last one, eight bits a pass from
// the top; what is longer is taken, and of that length as many as are missing, the first ones.
template <typename LENS>
__device__ __forceinline__ void select_longest(const SegArgs& a, const LENS& lens, const uint32_t i0, const uint32_t n, ListLds* S) {
    uint32_t* const s_hist = S->hist;
    const uint32_t tid = threadIdx.x;
    uint32_t cut = 0u, need = (uint32_t)kHotRows;   // length so far, and rows still missing among those that share its upper bits
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256u) s_hist[tid] = 0u;
        __syncthreads();
        lens.each(a, i0, n, [&](const uint32_t, const uint32_t len) {
            hist_add(s_hist, (len >> shift) & 255u, len != 0u && (shift == 24 || (len >> (shift + 8)) == (cut >> (shift + 8))));
        });
        __syncthreads();
        const uint32_t c = tid < 256u ? s_hist[255u - tid] : 0u;   // digits from the largest down
        uint32_t all;
        const uint32_t above = block_excl_scan<kListThreads>(c, S->scan, &all);
        if (above < need && need <= above + c) {
            s_hist[0] = 255u - tid;
            s_hist[1] = need - above;
        }
        __syncthreads();
        cut |= s_hist[0] << shift;
        need = s_hist[1];
        __syncthreads();
    }
    uint32_t longer = 0u, equal = 0u;   // ... than / to the cut, among the rows before
    lens.each(a, i0, n, [&](const uint32_t k, const uint32_t len) {
        const bool gt = len > cut, eq = len == cut;
        uint32_t tot;
        const uint32_t ex = block_excl_scan<kListThreads>((gt ? 0x10000u : 0u) | (eq ? 1u : 0u), S->scan, &tot);
        const uint32_t e = equal + (ex & 0xFFFFu);
        if (gt || (eq && e < need)) {
            const uint32_t at = longer + (ex >> 16) + (e < need ? e : need);   // below kHotRows
            S->k[at] = k;
            S->len[at] = len;
        }
        longer += tot >> 16;
        equal += tot & 0xFFFFu;
    });
    __syncthreads();
}

// a row k of many that is dense, or (length 0) does not exist
__device__ __forceinline__ bool dense_or_end(const uint32_t len, const uint32_t k, const uint32_t cut_len, const uint32_t cut_k) {
    return len == 0u || len > cut_len || (len == cut_len && k <= cut_k);
}

// The n long rows of table t, from place i0 of the list on.  MANY: more than kListRank of them (compiled apart: the launch is
// a chain of latencies, fetching its instructions among them).
template <bool MANY>
__device__ __forceinline__ void list_table(const SegArgs& a, ListLds* S, const int t, const uint32_t i0, const uint32_t n) {
    const uint32_t tid = threadIdx.x;
    const uint32_t rb = (uint32_t)a.row_base[t];
    const uint32_t D = (uint32_t)(a.D_off[t + 1] - a.D_off[t]);
    const bool ranked = a.hot_ids || a.dense_n;
    // ---- rank the candidates, one per thread: all long rows of the table, or the kHotRows longest
    const uint32_t nc = MANY ? (uint32_t)kHotRows : n;
    Lengths<MANY ? 8 : 1> lens;
    lens.load(a, i0, n);
    if (!MANY) {
        if (tid < n) S->len[tid] = lens.held[0];
    } else if (ranked) select_longest(a, lens, i0, n, S);
    __syncthreads();
    uint32_t my_k = tid, my_len = 0, rank = 0xFFFFFFFFu, nd = 0;   // nd: dense rows
    if (ranked) {
        if (tid < nc) {   // longest first, ties by key (the list is ascending by key)
            if (MANY) my_k = S->k[tid];
            my_len = S->len[tid];
            rank = 0u;
            for (uint32_t j = 0; j < nc; ++j) {
                const uint32_t l = S->len[j];
                rank += (l > my_len || (l == my_len && j < tid)) ? 1u : 0u;
            }
            if (a.hot_ids && rank < (uint32_t)kHotRows && my_len > kHotMin) a.hot_ids[(size_t)t * kHotRows + rank] = a.long_rows[i0 + my_k].y - rb;
            if (rank < (uint32_t)kDenseRows && my_len > kDenseMinLen) atomicAdd(&S->sum, my_len < 0x01000000u ? my_len : 0x01000000u);
        }
        const uint32_t hot = (uint32_t)__syncthreads_count(my_len > kHotMin);
        if (a.hot_n && tid == 0) a.hot_n[t] = hot < (uint32_t)kHotRows ? hot : (uint32_t)kHotRows;
        // A table with that many long rows has most of its lookups in parts anyway, and those fill the chip: the dense rows
        // pay only if their kernel does as well.  Measured, backward without and with them: 4 tables x 131072 bags of 128 ids,
        // 128 columns (128 workgroups) 5.82 and 5.35 ms; 1 table x 65536 bags of 256 ids (32 workgroups) 1.24 and 1.71 ms.
        const bool filled = !MANY || (uint32_t)a.T * a.dense_chunks * ((D + 255u) / 256u) >= 128u;
        if (a.dense_n && filled && dense_block((uint32_t)a.B, D) && S->sum >= 2u * (uint32_t)a.B)
            nd = nc < (uint32_t)kDenseRows ? nc : (uint32_t)kDenseRows;
        if (a.long_min < kDenseMinLen) {   // (the same for all) parts cut finer than dense rows are looked for
            const uint32_t many = (uint32_t)__syncthreads_count(tid < nc && my_len > kDenseMinLen);
            nd = nd < many ? nd : many;
        }
    }
    // ---- parts of the rows that are not dense: their number, then the table's place in the unit list, and the dense rows'
    // places (which tables come first decides the order in which units are worked on, and addresses, nothing else)
    uint32_t c = 0, ex = 0, total = 0;
    if (!MANY) {
        if (tid < n && rank >= nd) c = row_parts(a, lens.held[0]);
        ex = block_excl_scan<kListThreads>(c, S->scan, &total);
    } else {
        if (tid == 0) {
            S->cut_len = 0xFFFFFFFFu;   // dense are the rows down to the last ranked so
            S->cut_k = 0u;
        }
        __syncthreads();
        if (rank < nd && rank + 1u == nd) {
            S->cut_len = my_len;
            S->cut_k = my_k;
        }
        __syncthreads();
        lens.each(a, i0, n, [&](const uint32_t k, const uint32_t len) { c += dense_or_end(len, k, S->cut_len, S->cut_k) ? 0u : row_parts(a, len); });
        block_excl_scan<kListThreads>(c, S->scan, &total);
    }
    if (tid == 0) S->base = total > 0u ? atomicAdd(&a.counters[3], total) : 0u;
    if (tid == kWave && nd > 0u) {
        const uint32_t place = atomicAdd(&a.counters[5], 1u);
        S->first = atomicAdd(&a.counters[2], nd * a.dense_chunks * (D / 4u));
        a.dense_n[t] = nd;
        a.dense_tab[t] = make_uint2(place, S->first);
    }
    __syncthreads();
    if (rank < nd) {
        a.dense_rows[(size_t)t * kDenseRows + rank] = i0 + my_k;
        a.long_list[i0 + my_k] = make_uint4(MANY ? a.long_rows[i0 + my_k].x : lens.u0, S->first + rank * (D / 4u), kDenseFlag, (uint32_t)t);
    }
    if (!MANY) {
        if (c > 0u) a.long_list[i0 + tid] = make_uint4(lens.u0, lens.s0 / a.part + i0 + tid, c, (uint32_t)t);
        for (uint32_t q = 0; q < c; ++q) a.unit_list[S->base + ex + q] = make_uint2(i0 + tid, q);
        return;
    }
    uint32_t base = S->base;
    const uint32_t cut_len = S->cut_len, cut_k = S->cut_k;
    for (uint32_t k0 = 0; k0 < n; k0 += kListThreads) {
        const uint32_t k = k0 + tid;
        c = 0;
        if (k < n) {
            const uint32_t u = a.long_rows[i0 + k].x;
            const uint32_t s0 = a.seg_start[u], len = a.seg_start[u + 1] - s0;
            if (!dense_or_end(len, k, cut_len, cut_k)) {
                c = row_parts(a, len);
                a.long_list[i0 + k] = make_uint4(u, s0 / a.part + i0 + k, c, (uint32_t)t);
            }
        }
        uint32_t tot;
        const uint32_t at = base + block_excl_scan<kListThreads>(c, S->scan, &tot);
        for (uint32_t q = 0; q < c; ++q) a.unit_list[at + q] = make_uint2(i0 + k, q);
        base += tot;
    }
}

// Where each of the kSpans long spans of rows starts that the dies take (seg_update_kernel), so that all of them hold the same work: a
// row counts kSpanRow lookups besides its own, those of long rows not at all, which are reduced elsewhere.  Spans of equally many rows
// were level only where tables of all sizes alternate: of 26 tables of 1000 to 1 M rows in ascending order, uniform ids, one die had 3.1
// times the mean's lookups.  Row updates without long spans / with equally many rows / with these, us (tables in mixed, ascending and
// descending order of size): 26 tables x 4096 bags of 11 ids x 64 columns 82 77 72, 87 80 75, 84 80 74; uniform ids 174 162 164,
// 174 180 166, 176 173 169; 57 tables x 1410 bags of 21 ids x 128 columns 195 160 161, 199 180 157, 189 164 153; 40 tables x 4096 bags
// of 20 ids, Zipf 1.2, x 64 columns 154 125 129, 143 148 132, 147 138 123.  With 4 / 8 / 24 lookups a row: uniform ids gain (ascending
// 153 / 155 / 166), but many lookups of one row cost less than those of many, and skewed ids lose: the 57 tables in mixed order 178 /
// 166 / 160.
// One workgroup: the weight before every long row into LDS, then a wavefront per border finds the long row it lies before, and its
// place between that row and the one before.  Five dependent loads, no more than the lists of a table take, beside which it runs
// (measured: 0.2 us of the launch's 10).
constexpr uint32_t kSpanRow = 16;
constexpr uint32_t kSpanChunk = 2 * kListThreads;   // long rows in LDS at a time
__device__ __forceinline__ void span_borders(const SegArgs& a) {
    __shared__ uint64_t s_weight[kSpanChunk];                         // of the rows before a long row
    __shared__ uint32_t s_row[kSpanChunk], s_long[kSpanChunk];        // its number; lookups of the long rows up to and with it
    __shared__ uint32_t s_scan[kListThreads / kWave];
    const uint32_t tid = threadIdx.x;
    const uint32_t U = a.counters[0], nlong = a.counters[1] < a.cap_long ? a.counters[1] : a.cap_long;
    const uint32_t N = a.seg_start[U];
    auto load_chunk = [&](const uint32_t k0, const uint32_t carry) {   // returns the lookups of its rows
        uint32_t u[2], s0[2], len[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) u[j] = k0 + 2u * tid + j < nlong ? a.long_rows[k0 + 2u * tid + j].x : U;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            s0[j] = a.seg_start[u[j]];
            len[j] = u[j] < U ? a.seg_start[u[j] + 1] - s0[j] : 0u;
        }
        uint32_t tot;
        uint32_t before = carry + block_excl_scan<kListThreads>(len[0] + len[1], s_scan, &tot);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            s_weight[2u * tid + j] = (uint64_t)kSpanRow * u[j] + (s0[j] - before);
            before += len[j];
            s_row[2u * tid + j] = u[j];
            s_long[2u * tid + j] = before;
        }
        __syncthreads();
        return tot;
    };
    uint32_t all = 0;
    for (uint32_t k0 = 0; k0 < nlong; k0 += kSpanChunk) {
        all += load_chunk(k0, all);
        __syncthreads();
    }
    const uint64_t whole = (uint64_t)kSpanRow * U + (N - all);
    const uint32_t q = tid >> 6;
    const uint64_t x = whole * q / kSpans;   // the border's weight
    uint32_t lo = 0, hi = U, before = 0, carry = 0;
    for (uint32_t k0 = 0; k0 < nlong; k0 += kSpanChunk) {
        const uint32_t n = umin(nlong - k0, kSpanChunk);
        if (nlong > kSpanChunk) carry += load_chunk(k0, carry);
        if (hi == U) {   // (no long row so far has the border's weight before it)
            const uint32_t i = wave_first(0u, n, [&](const uint32_t k) { return s_weight[k] >= x; });
            if (i < n) hi = s_row[i];
            if (i > 0u) {
                lo = s_row[i - 1u] + 1u;
                before = s_long[i - 1u];
            }
        }
        __syncthreads();
    }
    if (q >= kSpans) return;
    const uint32_t border = wave_first(lo, hi, [&](const uint32_t u) { return (uint64_t)kSpanRow * u + (a.seg_start[u] - before) >= x; });
    if (lane_id() == 0) a.counters[kSpanWord + q] = border;
}
static_assert(kSpans <= kListThreads / kWave, "a wavefront per border");

// grid: one workgroup per table, and one more for the gradient blocks (non-pooled mode) or the borders of long spans
template <typename IT>
__global__ __launch_bounds__(kListThreads) void list_rows_kernel(const SegArgs a, const IT* __restrict__ offsets,
                                                                 const int64_t nnz, const int64_t grad_elems,
                                                                 int32_t* __restrict__ err) {
    __shared__ ListLds S;
    __shared__ uint32_t s_range[2];
    const int t = blockIdx.x;
    if (t == a.T) {
        if (a.seq) seq_blocks<IT>(a, offsets, nnz, grad_elems, err);
        else span_borders(a);
        return;
    }
    const uint32_t nlong = a.counters[1] < a.cap_long ? a.counters[1] : a.cap_long;
    const uint32_t tid = threadIdx.x;
    if (tid < 2 * kWave) {
        const int64_t x = a.row_base[t + (int)(tid >> 6)];
        const uint32_t i = wave_first(0u, nlong, [&](const uint32_t k) { return (int64_t)a.long_rows[k].y >= x; });
        if ((tid & (kWave - 1)) == 0) s_range[tid >> 6] = i;
    }
    if (tid == 0) {
        S.sum = 0u;
        if (a.hot_n) a.hot_n[t] = 0u;
        if (a.dense_n) a.dense_n[t] = 0u;
    }
    __syncthreads();
    const uint32_t i0 = s_range[0], n = s_range[1] - s_range[0];
    if (n == 0u) return;
    if (n <= kListRank) list_table<false>(a, &S, t, i0, n);
    else list_table<true>(a, &S, t, i0, n);
}

// Handles of very many tables (no hint, no dense rows): one thread per long row.
template <typename IT>
__global__ __launch_bounds__(kListThreads) void list_rows_flat_kernel(const SegArgs a, const IT* __restrict__ offsets,
                                                                      const int64_t nnz, const int64_t grad_elems,
                                                                      int32_t* __restrict__ err) {
    if ((a.seq || a.long_spans) && blockIdx.x == gridDim.x - 1) {
        if (a.seq) seq_blocks<IT>(a, offsets, nnz, grad_elems, err);
        else span_borders(a);
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
    SegArgs a = seg_args(h, w, ws, offsets, idx32, B, seq);
    a.long_spans = long_spans(h, B, seq, 2);   // (the gradient's type is not known yet: where any type would take them)
    const unsigned more = seq || a.long_spans ? 1u : 0u;
    LaunchTimer tm(h, s, "seg_long_list");
    const int64_t nnz = w.n;
    if (h->T <= kMaxSortSegments) {
        const unsigned grid = (unsigned)h->T + more;
        if (idx32) list_rows_kernel<int32_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int32_t*>(offsets), nnz, grad_elems, h->d_err);
        else list_rows_kernel<int64_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int64_t*>(offsets), nnz, grad_elems, h->d_err);
        if (a.dense_n) dense_index_kernel<<<(unsigned)(h->T * kIndexSplit), 256, 0, s>>>(a);
    } else {
        const unsigned grid = (unsigned)((w.cap_long + kListThreads - 1) / kListThreads) + more;
        if (idx32) list_rows_flat_kernel<int32_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int32_t*>(offsets), nnz, grad_elems, h->d_err);
        else list_rows_flat_kernel<int64_t><<<grid, kListThreads, 0, s>>>(a, static_cast<const int64_t*>(offsets), nnz, grad_elems, h->d_err);
    }
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
