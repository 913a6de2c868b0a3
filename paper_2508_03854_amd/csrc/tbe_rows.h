// What the kernels that list the rows of a sorted batch (tbe_lists.hip) and those that reduce and step them
// (tbe_backward.hip, tbe_dense.hip) share.
#pragma once
#include "tbe_device.h"
#include "tbe_internal.h"

namespace tbe {

// Bag lengths from the offsets array, whose values are below 2^32: the low word of every entry is enough, so int64 and
// int32 offsets differ in an index shift only.
struct OffsetWords {
    const uint32_t* p;
    int shift;   // 1: int64, 0: int32
    __device__ __forceinline__ uint32_t length(const int64_t bag) const {
        return p[(bag + 1) << shift] - p[bag << shift];
    }
};

constexpr uint32_t kDenseFlag = 0x80000000u;   // long_list entry: the dense-row kernel reduces the row

// Dies of the chip, each with an L2 of its own; workgroup i of a launch runs on die i % kDies.
constexpr uint32_t kDies = 8;
constexpr uint32_t kSpans = 2 * kDies;   // long spans of rows that the row updates may share out to the dies, two each
constexpr uint32_t kSpanWord = 16;       // counters[kSpanWord + k]: first row of span k
static_assert(kSpanWord + kSpans <= (uint32_t)kCounterWords, "borders among the counters");

struct SegArgs {
    const uint32_t* keys_unique;  // unique_rows
    const uint32_t* seg_start;
    uint32_t* counters;           // [0] unique rows, [1] long rows, [2] dense partials, [3] work units, [4] != 0: apply nothing,
                                  // [5] tables with dense rows, [kSpanWord ..] first rows of the long spans
    const uint32_t* bag_sorted;   // the sorted payload: linear bag id of every sorted lookup
    OffsetWords offsets;
    const void* grad_out;         // [B, sum(D)] float / binary16 / bfloat16, per the kernel's GT (or the sequence layout)
    int64_t* seq_gbase;           // non-pooled mode only: element offset of table t's gradient block minus start_t * D_t
    int seq;                      // 1: non-pooled; bag_sorted then holds the original positions
    const int32_t* D_off;
    const int64_t* row_base;
    const int64_t* w_off;
    int32_t T, B, sumD, maxD;
    uint32_t total_rows;
    uint32_t row_bytes;           // of the handle's mean row
    uint64_t stream_from;         // bytes of unique rows from which they are read and written past the caches
    float lr, eps, inv_c;
    void* tables;
    float* state;          // nullptr: plain SGD step, no moments
    // rows with more than long_min lookups
    uint32_t long_min, part;      // ... are cut into equal parts of about `part` lookups
    uint32_t cap_long;
    const uint2* long_rows;       // [counters[1]] (unique row, key), ascending
    uint4* long_list;             // [counters[1]] (unique row, first partial-sum slot, parts, table); a dense row: (unique row,
                                  // first partial sum in dense_partial in units of four floats, kDenseFlag, table)
    uint2* unit_list;             // [counters[3]] (position in long_list, part)
    float* partial;               // [slots][maxD] partial sums
    uint32_t* hot_ids;            // [T][kHotRows] rows with the most lookups, for the handle's hint (null: not kept)
    uint32_t* hot_n;              // [T]
    uint32_t* hint_ids;           // the handle's hint (null: not kept)
    uint32_t* hint_n;
    int long_spans;               // seg_update: 1: each die takes two long spans of rows (counters[kSpanWord ..]); 0: the whole chip
                                  // takes all passes in turn
    uint32_t long_pass_need;      // seg_update: rows per wavefront from which a pass has 32 rows
    int min_rows_log2;            // seg_update: a pass has at least 2^this consecutive rows
    // dense rows (tbe_dense.hip); null dense_n: no table can have any
    uint32_t* dense_n;            // [T] number of dense rows
    uint32_t* dense_rows;         // [T][kDenseRows] their positions in long_list, longest first
    uint2* dense_tab;             // [T] (place in dense_index, first partial sum as in long_list) of a table with dense rows
    uint32_t* dense_index;        // [place][kDenseRows][dense_blocks + 1] where each block of bags starts in the row's segment
    float* dense_partial;         // per table with dense rows [dense_chunks][dense rows][its columns] partial sums
    uint32_t dense_blocks;        // blocks of kDenseBags bags per table
    uint32_t dense_chunks;        // partial sums per dense row: runs of dense_per_chunk blocks
    uint32_t dense_per_chunk;
};

// Whether the row updates share long spans of rows out to the dies, for gradient elements of so many bytes.
// They gather a table's gradient block at random, and every die that works on the table reads it through its own L2.  Where the blocks
// are small enough to stay there next to the rows themselves (1.5 MiB of 4), a die takes two long spans of rows, equal in work
// (span_borders); from 16 tables on, so that a span is no small part of one table.  Row updates without / with them, us: 26 tables x
// 4096 bags x 64 fp32 columns (1 MiB) 82 / 72; 31 x 1699 x 224 fp32 (1.5 MB) 201 / 182; 57 x 1410 x 128 fp32 195 / 161; but 64 tables x
// 4096 bags x 224 bfloat16 (1.8 MB) 702 / 706, 12 tables x 1548 x 224 binary16 39.1 / 41.5, and at 16384 x 149 fp32 (9.8 MB) 288 / 310.
// Tables of more than 256 columns have rows in a span but no work for seg_update_kernel, and a row's lookups cost what its width says;
// the widest may have twice the mean width (16 tables x 650 bags, 8 to 520 columns, as spans of equally many rows 26.0 / 31.9 us).
inline int long_spans(const tbe_handle* h, const int32_t B, const int seq, const unsigned elem_bytes) {
    const uint64_t block = (uint64_t)B * (uint64_t)h->sumD * elem_bytes;   // of all tables
    const bool level = (int64_t)h->maxD * h->T <= 2 * (int64_t)h->sumD;
    return !seq && h->T >= 16 && level && block <= (uint64_t)h->T * (3u << 19) ? 1 : 0;
}

// Dense rows exist only where a table's gradient block is large, 2 MiB at four bytes per element (half an L2: a block that fits
// one is gathered from at L2 speed), and has enough bags to share out.  The lists are made before the gradient's type is known,
// so 16-bit blocks count as if they were 32-bit ones.  Measured around the line, backward with / without dense rows, us: 64
// tables, 31 ids, Zipf 1.1, 4096 bags x 256 columns fp32 (4 MiB) 1294 / 1460, bfloat16 (2 MiB) 1175 / 1255; 8192 x 128 fp32
// 1336 / 1535, bfloat16 1264 / 1324; 16 tables, 20 ids, 6000 x 128 fp32 (2.9 MiB) 222 / 252, bfloat16 208 / 212; but 26 tables,
// 11 ids, Zipf 1.05, 16384 x 64 fp32 435 / 418, bfloat16 416 / 380, and 8 tables, 20 ids, 1200 x 512 fp32 177 / 161.
__device__ __host__ __forceinline__ bool dense_block(const uint32_t B, const uint32_t D) {
    return B >= (uint32_t)kDenseMinBags && (uint64_t)B * D * 4u > ((uint64_t)2 << 20);
}

// table of a linearised row key: the t with row_base[t] <= key < row_base[t+1]
__device__ __forceinline__ int table_of_key(const int64_t* __restrict__ row_base, int T, uint32_t key) {
    int lo = 0, hi = T;  // first t in [0, T] with row_base[t] > key, minus 1
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (row_base[mid] > (int64_t)key) hi = mid;
        else lo = mid + 1;
    }
    return lo - 1;
}

// ... of a row whose first sorted lookup is s0: from that lookup's bag where the payload is one (one load instead of a
// search), else from the key
__device__ __forceinline__ int table_of_row(const SegArgs& a, const uint32_t s0, const uint32_t key) {
    return a.seq ? table_of_key(a.row_base, a.T, key) : (int)(a.bag_sorted[s0] / (uint32_t)a.B);
}

}  // namespace tbe
