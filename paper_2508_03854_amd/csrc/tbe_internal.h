// Internal declarations shared by the translation units of libtbe355 (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "tbe355.h"

namespace tbe {

// ---- tunables that fix the workspace layout -------------------------------------------------
constexpr int kRadixTile = 4096;  // elements per radix-sort tile (256 threads x 16) of a large batch; smaller ones take 2048 or 1024
constexpr int kRadixMaxBlocks = 8192;  // large batches: each radix block owns one contiguous slice of the input
constexpr int kRleTile = 2048;  // elements per run-length tile (at most 4096: one wavefront scans its runs of 64)
constexpr int64_t kRleOneBlock = 32768;  // batches up to this size are segmented by one workgroup
// Batches that are sorted in one launch (tbe_sort_small.hip): of at most kSmallMax lookups, or of at most kSmallMaxMany that are no
// more than kSmallSegment per table on average; of at most kSmallTables tables.
constexpr int kSmallTables = 512;
constexpr int64_t kSmallMax = 12288, kSmallMaxMany = 65536, kSmallSegment = 8192;
constexpr int kSmallChunk = 512;         // places of the sorted order that a workgroup owns
constexpr int kMaxParts = 1024;          // parts that a long row is cut into at most
constexpr int kMaxSortSegments = 4096;  // tables beyond this are sorted as one segment on the linearised key
constexpr int kDenseRows = 128;  // rows per table that the dense-row kernel reduces at most (multiple of 32)
constexpr int kDenseBags = 256;  // bags per block of that kernel
constexpr int kDenseMinBags = 1024;   // batches of fewer samples have no dense rows
constexpr int kFwdGroupMaxLanes = 32;   // rows of at most this many lanes use one bag per lane group
constexpr int kHotRows = 256;           // rows per table that the forward may hold in LDS (the handle's hot-row list)
constexpr uint32_t kHotMin = 512;       // ... of those with more lookups than this
constexpr int kMaxReplicas = 16;        // replicas of one buffer that tbe_replica_mean averages in one call
constexpr int kCounterWords = 64;      // device counters: [0]=U [1]=long rows [2]=dense partials handed out [3]=units [4]=apply nothing [5]=tables with dense rows

struct TimingSlot {
    const char* name;
    hipEvent_t beg, end;
};

}  // namespace tbe

struct tbe_handle {
    int32_t T = 0;
    tbe_dtype dtype = TBE_F32;
    int device = 0;
    int64_t total_rows = 0;
    int64_t total_elems = 0;
    int32_t sumD = 0;
    int32_t maxD = 0;
    int32_t minD = 0;
    bool seg_mostly_wavefront_rows = false;  // most rows of the tables up to 256 columns need all 64 lanes (D > 128)
    int key_bits = 1;  // bits needed to hold the value total_rows (the key given to invalid ids)
    // Sort plan.  Positions arrive grouped by table, so sorting every table's run of positions on its table-local id
    // alone gives the same order as sorting all of them on the linearised key, with no more key bits and no search for a
    // position's table.  Keys of at most 8 bits take one pass either way.
    bool segmented = false;  // true: one sort segment per table, local keys; false: one segment, linearised keys
    int sort_bits = 1;       // key bits the radix passes cover
    std::vector<int64_t> rows, row_base, w_off;
    std::vector<int32_t> D, D_off;
    // device metadata, one allocation
    void* d_meta = nullptr;
    int32_t* d_D_off = nullptr;     // [T+1]
    int64_t* d_row_base = nullptr;  // [T+1]
    int64_t* d_w_off = nullptr;     // [T+1]
    void* static_scratch = nullptr; // device address, on this handle's device, of the library's fixed scratch array
    int32_t* d_err = nullptr;       // sticky invalid-id flag
    // Forward classes: 0, 5, 6 = one wavefront per bag, rows of at most 64 / 128 / 256 sixteen-byte fragments;
    // 1..4 = narrow rows (32 / 16 / 8 / <=4 lanes per row), where every lane group of a wavefront takes a bag of its
    // own (2 / 4 / 8 / 16 bags per wavefront).  d_fwd_tables lists the tables class by class.
    int32_t* d_fwd_tables = nullptr;  // [T]
    // Hot-row hint: the table-local ids of the rows of every table that had the most lookups in the last backward
    // call (at most kHotRows each), written by that call's kernels and read by the next forward.  Any contents give
    // the same forward result; null when the handle has too many tables to keep one.
    uint32_t* d_hot_ids = nullptr;    // [T][kHotRows]
    uint32_t* d_hot_n = nullptr;      // [T]
    // The forward stages hot rows in LDS when a width class fills this many workgroups; < 0: never, except TBE_TUNE_AUTO, where the
    // line follows the class (hot_chunks).
    int64_t hot_min_workgroups = TBE_TUNE_AUTO;
    int fwd_first[7] = {0, 0, 0, 0, 0, 0, 0};
    int fwd_count[7] = {0, 0, 0, 0, 0, 0, 0};
    uint32_t fwd_columns[7] = {0};   // of the class's tables: all bits of their numbers of columns and first columns
    int fwd_maxD[7] = {0};           // ... and the most columns
    // timing
    bool timing = false;
    std::vector<tbe::TimingSlot> slots;  // pool of event pairs
    int n_used = 0;                      // slots used by the calls since timing was (re)enabled
};

namespace tbe {

// How the keys of a batch of N lookups are sorted (see tbe_sort.hip).
struct SortShape {
    int nseg;          // sort segments
    bool small;        // one launch for the whole sort; of what follows the chunks alone are used, its workgroups' ranges
    int passes, bits;  // radix passes, digit bits of each
    size_t hist_bytes; // chunk histograms
    int bins;          // 256, 1024 or 2048: histogram width of the kernels that run
    bool self_scan;    // scatter workgroups add up their segment's chunk histograms themselves
    int tile;          // 1024, 2048 or 4096 positions
    int64_t chunk;     // positions per chunk (a multiple of the tile)
    int max_chunks;    // N / chunk + number of segments (every segment may end in a partial chunk)
};
SortShape sort_shape(const tbe_handle* h, int64_t N);

// Workspace carving for a batch of N lookups (all offsets in bytes, 256-byte aligned).
struct Workspace {
    // keys/vals: radix double buffers of N+1 words each.  The payload of a key is the linear bag id of its lookup
    // (pooled calls) or its position (non-pooled calls), so vals[sorted] is the per-lookup stream the gradient
    // kernels read.  After the sort vals[spare] receives unique_rows.
    size_t keys[2], vals[2], seg_start, counters, long_rows, long_list, unit_list, hot_ids, hot_n, seq_gbase, dense_n, dense_tab,
        dense_rows, dense_index, radix_hist, nchunks, chunk_desc, rle_counts, partial, dense_partial, total;
    SortShape sort;
    int rle_blocks;
    uint32_t long_min, part;      // a row with more lookups is long: it is cut into parts of about `part`
    int64_t cap_long, cap_main;   // long rows; partial-sum slots of their parts
    bool dense;           // dense rows are looked for; their sizes:
    uint32_t dense_blocks, dense_chunks, dense_per_chunk;
    int64_t n;            // number of lookups the workspace was carved for
};
Workspace carve(const tbe_handle* h, int32_t B, int64_t N);

// RAII-free helper: brackets one kernel launch with events when timing is on.
struct LaunchTimer {
    tbe_handle* h;
    hipStream_t s;
    int slot = -1;
    LaunchTimer(const tbe_handle* h_, hipStream_t s_, const char* name);
    void done();
};

// launchers (each returns hipGetLastError() after its launches).  idx32: ids and offsets are int32 instead of
// int64; out_io / grad_io: 0 float, 1 binary16, 2 bfloat16.
hipError_t launch_forward(const tbe_handle* h, const void* tables, const int32_t* d_D_off, const void* indices,
                          const void* offsets, int idx32, int32_t B, int64_t nnz, tbe_pooling pooling, void* out,
                          int out_io, hipStream_t s);
// the kernels that launch_forward would launch for B samples and nnz ids (TBE_FWD_* bits), by the rules it launches them by
unsigned forward_kernels(const tbe_handle* h, int32_t B, int64_t nnz);
// every replicas[m] (device pointers, M <= kMaxReplicas) becomes the element-wise mean; count elements each
hipError_t launch_replica_mean(const tbe_handle* h, void* const* replicas, int M, size_t count, bool f32, hipStream_t s);
// Sorts the batch's ids, segment by segment, into (linearised row key, payload) pairs; the payload is the lookup's bag, or
// its position when seq is set.  The result lies in buffer pair w.sort.passes & 1 of the workspace.
// Then the run lengths: vals of the other pair receive unique_rows.
hipError_t launch_sort(const tbe_handle* h, const Workspace& w, char* ws, const void* indices, const void* offsets, int idx32,
                       int32_t B, int64_t N, bool seq, hipStream_t s);
struct SegArgs;
SegArgs seg_args(const tbe_handle* h, const Workspace& w, char* ws, const void* offsets, int idx32, int32_t B, int seq);
// lists the long rows of the sorted batch (and, seq != 0, the gradient blocks of the non-pooled layout)
hipError_t launch_lists(const tbe_handle* h, const Workspace& w, char* ws, const void* offsets, int idx32, int32_t B, int seq,
                        int64_t grad_elems, hipStream_t s);
void launch_dense(const SegArgs& a, int grad_io, bool mean, hipStream_t s);
// state == nullptr: plain SGD step.  seq != 0: grad_out is the non-pooled layout (one [n_t, D_t] block per table),
// offsets has T+1 entries and B is 1.
hipError_t launch_segment_update(const tbe_handle* h, const Workspace& w, char* ws, const void* grad_out, int grad_io,
                                 const void* offsets, int idx32, int32_t B, tbe_pooling pooling, float lr, float eps, float c,
                                 void* tables, float* state, int seq, hipStream_t s);
// non-pooled lookup: out block of table t = rows indices[offsets[t] .. offsets[t+1]) of table t, one after the other
hipError_t launch_lookup_seq(const tbe_handle* h, const void* tables, const void* indices, const void* offsets, int idx32,
                             int64_t nnz, void* out, int out_io, int64_t out_elems, hipStream_t s);

}  // namespace tbe
