// What the kernels that sort a batch's ids and segment the sorted keys share: tbe_sort.hip (batches of any size) and
// tbe_sort_small.hip (small ones, one launch).
#pragma once
#include "tbe_device.h"
#include "tbe_internal.h"

namespace tbe {

constexpr int kRsThreads = 256;

struct ChunkDesc {            // written by pass 0, one per workgroup; e == s: no chunk
    uint32_t s, e;            // positions [s, e)
    uint32_t seg;             // segment
    uint32_t first, count;    // the segment's first chunk, its number of chunks
    uint32_t seg_start;       // the segment's first position
    uint32_t seg_end;         // ... and the position behind its last
    uint32_t pad;
};

// everything a pass needs to know about where its elements come from
struct SortArgs {
    const void* indices;     // int64 or int32, both the same: the kernels that read them are compiled for either (a run-time
    const void* offsets;     // flag costs every load of the divergent searches a branch around two forms of it)
    const int64_t* row_base;
    ChunkDesc* desc;
    uint32_t* nchunks;       // chunks of all segments (large batches; else null)
    void* ghist;             // self-scan: uint16 [chunk][NB] (a chunk is one tile); else uint32 at hist_word(chunk, digit)
    const uint32_t* keys_in;
    const uint32_t* vals_in;
    uint32_t* keys_out;
    uint32_t* vals_out;
    int32_t* err;
    int64_t N, chunk, nbags;
    int32_t B, nseg, max_chunks;
    int32_t shift;
    uint32_t mask, invalid_key;
    int32_t by_table;        // keys are table-local (a single table counts as such)
    int32_t iota;            // the payload is the position
    int32_t globalize;       // last pass of a table-by-table sort: write linearised keys
};

// first i in [lo, hi] with a[i] > x   (caller guarantees a[hi] > x)
template <typename IT>
__device__ __forceinline__ int64_t upper_bound_i64(const IT* __restrict__ a, int64_t lo, int64_t hi, int64_t x) {
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] > x) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// The same search by a whole wavefront: 64 probes per round cut the range 64-fold, so 8 M offsets take 4 dependent
// loads instead of 23.  Every lane returns the result.  Terminates for any contents of a (the range shrinks every
// round) and never reads outside [lo, hi).
template <typename IT>
__device__ __forceinline__ int64_t wave_upper_bound_i64(const IT* __restrict__ a, int64_t lo, int64_t hi, const int64_t x) {
    const int lane = lane_id();
    while (lo < hi) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t i = lo + (int64_t)(lane + 1) * step - 1;   // lane's probe; the last lane's is >= hi - 1
        const bool gt = i < hi ? (a[i] > x) : true;
        const uint64_t m = __ballot(gt);                         // (a probe beyond hi counts as greater)
        if (m == 0ull) return hi;                                // all of [lo, hi) is <= x
        const int f = __ffsll((unsigned long long)m) - 1;        // first probe above x
        const int64_t i_f = lo + (int64_t)(f + 1) * step - 1;
        lo += (int64_t)f * step;                                 // the probe before it was <= x
        hi = i_f < hi ? i_f : hi;
    }
    return lo;
}

// Inclusive running maximum across a block of NT threads (smem: NT / 64 words, free again on return).
template <int NT>
__device__ __forceinline__ uint32_t block_incl_max(uint32_t v, uint32_t* smem) {
    const int l = lane_id();
    v = wave_incl_max(v);
    const int w = threadIdx.x >> 6;
    if (l == kWave - 1) smem[w] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i)
        if (i < w) v = smem[i] > v ? smem[i] : v;
    __syncthreads();
    return v;
}

// Which chunk is this workgroup's?  Segment borders are offsets[t * B], forced into [0, N] and made ascending, so that
// the chunks always tile [0, N) exactly, whatever the offsets array holds.  NT segments (the workgroup's threads) per round; every round
// scans borders and chunk counts.  Workgroup 0 also leaves the number of chunks for the scan of the histograms, if there is one.
template <typename IT, int NT>
__device__ __forceinline__ ChunkDesc find_chunk(const SortArgs& a, const uint32_t c, uint32_t* smem, ChunkDesc* s_desc) {
    if (threadIdx.x == 0) *s_desc = ChunkDesc{0, 0, 0, 0, 0, 0, 0, 0};
    __syncthreads();
    if (a.nseg == 1) {
        if (threadIdx.x == 0) {
            const int64_t s = (int64_t)c * a.chunk, n = (a.N + a.chunk - 1) / a.chunk;
            if (s < a.N) *s_desc = ChunkDesc{(uint32_t)s, (uint32_t)(s + a.chunk < a.N ? s + a.chunk : a.N), 0, 0, (uint32_t)n, 0, (uint32_t)a.N, 0};
            if (c == 0 && a.nchunks) *a.nchunks = (uint32_t)n;
        }
        __syncthreads();
        return *s_desc;
    }
    uint32_t carry_b = 0, carry_c = 0;   // border and chunk count before this round's segments
    for (int t0 = 0; t0 < a.nseg; t0 += NT) {
        const int t = t0 + (int)threadIdx.x;
        uint32_t b1 = 0;                 // end of segment t
        if (t < a.nseg) {
            int64_t b = t + 1 == a.nseg ? a.N : (int64_t)static_cast<const IT*>(a.offsets)[(int64_t)(t + 1) * a.B];
            b = b < 0 ? 0 : (b > a.N ? a.N : b);
            b1 = (uint32_t)b;
        }
        b1 = block_incl_max<NT>(b1 > carry_b ? b1 : carry_b, smem);
        uint32_t b0 = __shfl_up(b1, 1, kWave);   // its start: the segment before
        if (lane_id() == kWave - 1) smem[threadIdx.x >> 6] = b1;
        __syncthreads();
        if (lane_id() == 0) b0 = threadIdx.x == 0 ? carry_b : smem[(threadIdx.x >> 6) - 1];
        const uint32_t last = smem[NT / kWave - 1];
        __syncthreads();
        const uint32_t n = t < a.nseg ? (uint32_t)(((int64_t)(b1 - b0) + a.chunk - 1) / a.chunk) : 0u;
        uint32_t tot;
        const uint32_t f = carry_c + block_excl_scan<NT>(n, smem, &tot);
        if (c >= f && c - f < n) {
            const int64_t s = (int64_t)b0 + (int64_t)(c - f) * a.chunk;
            const int64_t e = s + a.chunk < (int64_t)b1 ? s + a.chunk : (int64_t)b1;
            *s_desc = ChunkDesc{(uint32_t)s, (uint32_t)e, (uint32_t)t, f, n, b0, b1, 0};
        }
        if (c == 0 && a.nchunks && t == a.nseg - 1) *a.nchunks = f + n;
        carry_b = last;
        carry_c += tot;
        if (carry_c > c && !(c == 0 && a.nchunks)) break;   // (the same for all threads) found
    }
    __syncthreads();
    return *s_desc;
}

// The lanes among `valid` that hold the same digit of `bits` bits: per bit one ballot, and the lanes that agree with this lane's bit
// are ~(ballot ^ (all ones if the bit is set)), taken into the running set by one three-operand instruction per half.
__device__ __forceinline__ void same_bit(const uint32_t d, const int b, uint32_t& lo, uint32_t& hi) {
    const uint32_t sel = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);           // all ones if this lane's digit has bit b
    const uint64_t m = __builtin_amdgcn_uicmp(sel, 0u, 33 /* != */);
    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, sel, 0x90);                 // lo & ~(m ^ sel)
    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), sel, 0x90);
}
__device__ __forceinline__ uint64_t same_digit(const uint32_t d, const int bits, const uint64_t valid) {
    uint32_t lo = (uint32_t)valid, hi = (uint32_t)(valid >> 32);
#pragma unroll 1
    for (int b = 0; b < bits; ++b) same_bit(d, b, lo, hi);
    return ((uint64_t)hi << 32) | lo;
}

// =================================================================================================
// run-length segmentation of the sorted keys: unique_rows, seg_start, num_unique, and in row order the long rows, i.e.
// those with more than long_min lookups (element i starts one if it is a head and element i + long_min has its key).
// Element order inside a tile: 8 rows of NT, row k / wave w / lane l is element k*NT + w*64 + l, so every (k, w) pair is
// a run of 64 consecutive elements and ballots give exact ranks.
// =================================================================================================
constexpr int kRleThreads = 256;
constexpr int kRleItems = kRleTile / kRleThreads;            // 8
static_assert(kRleItems == 8, "the kernels below take eight elements per thread");

struct RleArgs {
    const uint32_t* keys;
    int64_t N;
    uint32_t long_min, total_rows;
    uint2* counts;            // per tile: heads, long rows
    uint32_t* unique_rows;
    uint32_t* seg_start;
    uint2* long_rows;         // (index of the unique row, key)
    uint32_t* counters;       // [0] unique rows, [1] long rows, [2] .. [5] = 0
};

// Head flags of a thread's eight elements (element k*NT + tid of the tile, which ends before `end`): element i is a head if it
// exists and its key differs from its predecessor's; lng: a head of a long row (ids outside their table form no row).  The loads are
// unconditional (indices clamped into the array, which always holds at least one element) and all issued before the first
// comparison, so that they overlap.
template <int NT>
__device__ __forceinline__ void head_flags(const RleArgs& a, const int64_t base, const int64_t end,
                                           uint32_t (&cur)[kRleItems], bool (&head)[kRleItems], bool (&lng)[kRleItems]) {
    uint32_t prev[kRleItems], far[kRleItems];
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        const int64_t i = base + k * NT + threadIdx.x;
        const bool in = i < end;
        cur[k] = a.keys[in ? i : 0];
        prev[k] = a.keys[(in && i > 0) ? i - 1 : 0];
        far[k] = a.keys[i + a.long_min < a.N ? i + a.long_min : a.N - 1];
    }
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        const int64_t i = base + k * NT + threadIdx.x;
        head[k] = i < end && (i == 0 || cur[k] != prev[k]);
        lng[k] = head[k] && i + a.long_min < a.N && far[k] == cur[k] && cur[k] < a.total_rows;
    }
}

// Writes a tile's unique_rows, seg_start and long rows; the tile's first head is unique row bb, its first long row number
// bl.  Returns the tile's (heads, long rows).  s_run: 8 * NT / 64 + 1 words.
template <int NT>
__device__ __forceinline__ uint2 rle_write_tile(const RleArgs& a, const int64_t base, const uint32_t bb, const uint32_t bl,
                                                const uint32_t (&cur)[kRleItems], const bool (&head)[kRleItems],
                                                const bool (&lng)[kRleItems], uint32_t* s_run) {
    constexpr int kRuns = kRleItems * (NT / kWave);   // runs of 64 elements per tile: 32 or 128
    const int lane = lane_id();
    const int w = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    uint64_t heads[kRleItems], longs[kRleItems];
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        heads[k] = __ballot(head[k]);
        longs[k] = __ballot(lng[k]);
        if (lane == 0) s_run[k * (NT / kWave) + w] = (uint32_t)__popcll(heads[k]) | ((uint32_t)__popcll(longs[k]) << 16);
    }
    __syncthreads();
    if (threadIdx.x < kWave) {  // one wavefront scans the run counts (heads and long rows in one word: at most 8192 each)
        uint32_t carry = 0;
#pragma unroll
        for (int r0 = 0; r0 < kRuns; r0 += kWave) {
            const uint32_t v = (r0 + lane < kRuns) ? s_run[r0 + lane] : 0u;
            const uint32_t inc = wave_incl_scan(v);
            if (r0 + lane < kRuns) s_run[r0 + lane] = carry + inc - v;
            carry += __shfl(inc, kWave - 1, kWave);
        }
        if (lane == 0) s_run[kRuns] = carry;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        const uint32_t run = s_run[k * (NT / kWave) + w];
        if (head[k]) {
            const int64_t i = base + k * NT + threadIdx.x;
            const uint32_t u = bb + (run & 0xFFFFu) + (uint32_t)__popcll(heads[k] & lt);
            a.unique_rows[u] = cur[k];
            a.seg_start[u] = (uint32_t)i;
            if (lng[k]) a.long_rows[bl + (run >> 16) + (uint32_t)__popcll(longs[k] & lt)] = make_uint2(u, cur[k]);
        }
    }
    const uint32_t tot = s_run[kRuns];
    return make_uint2(tot & 0xFFFFu, tot >> 16);
}

__device__ __forceinline__ void rle_finish(const RleArgs& a, const uint32_t U, const uint32_t nlong) {
    a.counters[0] = U;
    a.counters[1] = nlong;
    a.counters[2] = a.counters[3] = a.counters[5] = 0u;   // handed out by the kernel that lists the long rows
    a.counters[4] = 0u;   // set when a non-pooled batch must not be applied
    a.seg_start[U] = (uint32_t)a.N;
}

// Sort and run lengths of a small batch whose keys are local to their segment (tbe_sort_small.hip).
hipError_t launch_sort_small(const tbe_handle* h, const SortArgs& a, const RleArgs& r, int idx32, hipStream_t s);

}  // namespace tbe
