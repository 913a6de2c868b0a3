// Integer half of the backward pass: linearise ids into row keys, stable LSD radix sort of (key, payload) with the
// lookup's bag id (pooled calls) or position (non-pooled calls) as payload, run-length segmentation into unique rows.  Everything here is exact integer work.
#include "tbe_sort.h"

namespace tbe {

// =================================================================================================
// Ids to sorted (key, payload) pairs: a stable LSD radix sort whose first pass reads the ids themselves.
//
// The positions are cut into segments (one per table, or a single one) and every segment into chunks of at most `chunk`
// positions; a chunk never crosses a segment border.  One workgroup owns one chunk in every pass:
//   hist    : counts the digits of its chunk (pass 0: of the keys it makes from the ids, and leaves the chunk's
//             descriptor for the kernels that follow)
//   scan    : large batches only - adds up the chunks' histograms
//   scatter : ranks the chunk tile by tile and writes (key, payload) to its final place inside the segment
// Chunk k precedes chunk k+1, and the scatter ranks elements in input order, so the sort is stable.  The last pass
// turns table-local keys into linearised ones as it writes them.
//   key     : the table-local id when the sort goes table by table, else row_base[t] + id; an id outside its table gets
//             the table's number of rows (sum(rows) when the keys are linearised)
//   payload : the lookup's bag (pooled calls) or its position (non-pooled calls)
// Making the keys inside pass 0, twice, instead of storing them and their bags first costs one more read of the ids and
// saves 8 bytes written and 4 read per lookup and two launches.
//
// The smallest batches have a sort of one launch instead (tbe_sort_small.hip; sort_shape draws the line).
//
// Digits: up to 11 bits in batches of at most kSelfScanMax lookups, 8 bits beyond.  A small batch's time is its chain of
// launches (about 4 us each), so it takes wide digits (fewer passes) and lets every scatter workgroup add up the
// histograms of its segment's chunks by itself (no launch for the scan).  In a large batch 2048 bins would leave runs of two
// keys per tile and bin to write, and the chunk histograms would be too many to add up per workgroup.
//
// Bound: launches and latency in small batches, the streams and the ranking beyond.  Measured, whole training step, against
// a sort that stored keys and bags first and took 8-bit digits throughout: 26 tables, 1.2 M lookups 295 -> 254 us; 64 tables, 65 M
// lookups 9.50 -> 9.18 ms.
// =================================================================================================
constexpr int kRsWaves = kRsThreads / kWave;

struct OwnerLds {
    int64_t lo, hi;
    int32_t wmax[kRsWaves];
};

// The bag of every position of the tile [p0, p1): thread's item k is position p0 + w*64*ITEMS + k*64 + lane.  Two
// wavefronts find the bags of the first and the last position among bags [blo, bhi); every bag that starts inside the
// tile marks its first position in LDS, and a running maximum over the positions gives each position the last bag that
// starts at or before it, i.e. its owner (empty bags start where the next one does and lose against it).  A tile that
// spans more bags than it has positions (runs of empty bags) searches position by position instead.  Whatever the
// offsets hold, the result lies in [blo, bhi).  s_own: 256 * ITEMS words.
template <typename IT, int ITEMS>
__device__ __forceinline__ void tile_owners(const IT* __restrict__ offsets, const int64_t blo, const int64_t bhi, const int64_t p0,
                                            const int64_t p1, int32_t* s_own, OwnerLds* o, uint32_t (&bag)[ITEMS]) {
    constexpr int kTile = ITEMS * kRsThreads;
    const int lane = lane_id();
    const int w = threadIdx.x >> 6;
    if (w < 2) {
        const int64_t r = wave_upper_bound_i64(offsets, blo, bhi, w == 0 ? p0 : p1 - 1) - 1;
        if (lane == 0) *(w == 0 ? &o->lo : &o->hi) = r;
    }
    for (int i = threadIdx.x; i < kTile; i += kRsThreads) s_own[i] = 0;
    __syncthreads();
    int64_t lo = o->lo, hi = o->hi;
    lo = lo < blo ? blo : (lo > bhi - 1 ? bhi - 1 : lo);
    hi = hi < lo ? lo : (hi > bhi - 1 ? bhi - 1 : hi);
    const int64_t nb = hi - lo + 1;              // bags touched by this tile (>= 1)
    const bool marked = nb <= kTile;
    if (marked) {
        for (int i = 1 + (int)threadIdx.x; i < (int)nb; i += kRsThreads) {
            const int64_t rel = (int64_t)offsets[lo + i] - p0;
            if (rel >= 0 && rel < kTile) atomicMax(&s_own[rel], i);   // bag lo+i starts here
        }
    }
    __syncthreads();
    if (marked) {
        // running maximum, in place: every thread over ITEMS consecutive positions, then across lanes and wavefronts
        int32_t* const mine = s_own + threadIdx.x * ITEMS;
        int32_t run[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; k += 4) {
            const int4 v = *reinterpret_cast<const int4*>(mine + k);
            run[k] = v.x; run[k + 1] = v.y; run[k + 2] = v.z; run[k + 3] = v.w;
        }
#pragma unroll
        for (int k = 1; k < ITEMS; ++k) run[k] = run[k] > run[k - 1] ? run[k] : run[k - 1];
        const int32_t top = (int32_t)wave_incl_max((uint32_t)run[ITEMS - 1]);   // (places among the tile's bags: not negative)
        int32_t prev = __shfl_up(top, 1, kWave);
        if (lane == 0) prev = 0;
        if (lane == kWave - 1) o->wmax[w] = top;
        __syncthreads();
        for (int ww = 0; ww < w; ++ww) prev = o->wmax[ww] > prev ? o->wmax[ww] : prev;
#pragma unroll
        for (int k = 0; k < ITEMS; k += 4)
            *reinterpret_cast<int4*>(mine + k) = make_int4(run[k] > prev ? run[k] : prev, run[k + 1] > prev ? run[k + 1] : prev,
                                                           run[k + 2] > prev ? run[k + 2] : prev, run[k + 3] > prev ? run[k + 3] : prev);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) bag[k] = (uint32_t)(lo + s_own[w * (kWave * ITEMS) + k * kWave + lane]);
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t p = p0 + w * (kWave * ITEMS) + k * kWave + lane;
            int64_t b = upper_bound_i64(offsets, lo, hi + 1, p < p1 ? p : p1 - 1) - 1;
            bag[k] = (uint32_t)(b < lo ? lo : (b > hi ? hi : b));
        }
    }
    __syncthreads();   // s_own may be reused by the caller
}

// The ids of a thread's items, all loads issued before the first use (a position behind the tile's end reads its last).
template <typename IT, int ITEMS>
__device__ __forceinline__ void load_ids(const IT* __restrict__ indices, const int64_t p0, const int64_t p1, IT (&id)[ITEMS]) {
    const int64_t first = p0 + (threadIdx.x >> 6) * (kWave * ITEMS) + lane_id();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) id[k] = indices[first + k * kWave < p1 ? first + k * kWave : p1 - 1];
}

// Chunk histograms of a large batch: [group of kScanDigits digits][chunk][digit of the group], max_chunks + 1 chunks.  A workgroup of the
// scan reads one group from end to end, a chunk's workgroups in pieces of 32 bytes.
constexpr int kScanDigits = 8;
__device__ __forceinline__ size_t hist_word(const SortArgs& a, const uint32_t chunk, const uint32_t d) {
    return ((size_t)(d / kScanDigits) * ((uint32_t)a.max_chunks + 1u) + chunk) * kScanDigits + d % kScanDigits;
}

// Private histograms: lanes are spread over kCopies of them, which divides the number of lanes that meet on one LDS word
// or bank (the kernel is bound by these LDS additions, not by the key stream: 1.04 ms with one copy per wavefront, 0.83 ms
// with two, for the three passes of the largest workload).
// IDS: pass 0.  OWNER: keys are linearised over several tables, so a position's table comes from its bag.
template <typename IT, int NB, int ITEMS, bool IDS, bool OWNER, bool SELF>
__global__ __launch_bounds__(kRsThreads) void radix_hist_kernel(const SortArgs a) {
    constexpr int kTile = ITEMS * kRsThreads;
    constexpr int kCopies = NB >= 2048 ? 1 : 2048 / NB;   // 8 KB of LDS
    __shared__ uint32_t h[kCopies][NB];
    __shared__ uint32_t s_scan[kRsWaves];
    __shared__ ChunkDesc s_desc;
    __shared__ OwnerLds s_o;
    __shared__ __align__(16) int32_t s_own[OWNER ? kTile : 1];
    ChunkDesc ds;
    if (IDS) {
        ds = find_chunk<IT, kRsThreads>(a, blockIdx.x, s_scan, &s_desc);
        if (threadIdx.x == 0) a.desc[blockIdx.x] = ds;
    } else {
        ds = a.desc[blockIdx.x];
    }
    if (ds.e <= ds.s) return;
    for (int i = threadIdx.x; i < kCopies * NB; i += kRsThreads) (&h[0][0])[i] = 0u;
    __syncthreads();
    uint32_t* hw = h[kCopies >= 8 ? 2 * (threadIdx.x >> 6) + (threadIdx.x & 1) : (threadIdx.x & (kCopies - 1))];
    const int64_t s = ds.s, e = ds.e;
    int64_t R = 0;
    if (IDS && !OWNER) R = a.row_base[ds.seg + 1] - a.row_base[ds.seg];
    bool bad = false;
    for (int64_t tile = s; tile < e; tile += kTile) {
        const int64_t te = tile + kTile < e ? tile + kTile : e;
        const int64_t first = tile + (threadIdx.x >> 6) * (kWave * ITEMS) + lane_id();
        uint32_t key[ITEMS];
        if (IDS) {
            IT id[ITEMS];
            load_ids<IT, ITEMS>(static_cast<const IT*>(a.indices), tile, te, id);
            if (OWNER) {
                uint32_t bag[ITEMS];
                tile_owners<IT, ITEMS>(static_cast<const IT*>(a.offsets), 0, a.nbags, tile, te, s_own, &s_o, bag);
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    const int64_t rb = a.row_base[bag[k] / (uint32_t)a.B], re = a.row_base[bag[k] / (uint32_t)a.B + 1];
                    const bool ok = id[k] >= 0 && id[k] < re - rb;
                    bad |= !ok;
                    key[k] = ok ? (uint32_t)(rb + id[k]) : a.invalid_key;
                }
            } else {
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    const bool ok = id[k] >= 0 && id[k] < R;
                    bad |= !ok;
                    key[k] = ok ? (uint32_t)id[k] : (uint32_t)R;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) key[k] = a.keys_in[first + k * kWave < te ? first + k * kWave : te - 1];
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) hist_add(hw, (key[k] >> a.shift) & a.mask, first + k * kWave < te);
    }
    if (IDS && bad) atomicOr(a.err, 1);   // (positions behind a tile's end repeat a valid position's id)
    __syncthreads();
    for (int d = threadIdx.x; d < NB; d += kRsThreads) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < kCopies; ++q) c += h[q][d];
        if (SELF) static_cast<uint16_t*>(a.ghist)[(size_t)blockIdx.x * NB + d] = (uint16_t)c;
        else static_cast<uint32_t*>(a.ghist)[hist_word(a, blockIdx.x, d)] = c;
    }
}

// Large batches: every chunk's count of a digit becomes the sum of those of all chunks before it, chunk nchunks gets the sum of all; a
// chunk's place within its segment is the difference to the segment's first.  A workgroup takes kScanDigits digits of all chunks, a
// thread one of them in a run of consecutive chunks, held in registers (up to 66 of 128: four others are spilled, 20 bytes a lane, at
// every size, for all sizes share the kernel).
// Bound: latency.  All histograms, scans and scatters of a step with a row of all chunks per digit (256 scattered words for every
// chunk's workgroups) / a row of all digits per chunk (every scan workgroup reads all of it) / this, us: 32 tables,
// 26 M lookups 124 + 58 + 301 / 98 + 98 + 287 / 101 + 54 + 289; 16 tables, 5.5 M 45 + 24 + 92 / 39 + 28 + 89 / 39 + 19 + 89; 64 tables, 65 M
// 301 + 72 + 851 / 274 + 110 + 844 / 284 + 57 + 851.
constexpr int kScanThreads = 1024, kScanParts = kScanThreads / kScanDigits;
// exclusive prefix of the threads' sums over the parts of a digit
__device__ __forceinline__ uint32_t scan_parts(uint32_t (&s_part)[kScanDigits][kScanParts], const uint32_t dl, const uint32_t part, const uint32_t sum) {
    s_part[dl][part] = sum;
    __syncthreads();
    if (threadIdx.x < kScanDigits * kWave) {   // a wavefront per digit: two parts per lane
        uint2* const p = reinterpret_cast<uint2*>(s_part[threadIdx.x / kWave]) + lane_id();
        const uint2 v = *p;
        const uint32_t before = wave_incl_scan(v.x + v.y) - v.x - v.y;
        *p = make_uint2(before, before + v.x);
    }
    __syncthreads();
    return s_part[dl][part];
}
template <int HELD>
__device__ __forceinline__ void scan_held(uint32_t (&s_part)[kScanDigits][kScanParts], const uint32_t dl, const uint32_t part, uint32_t* const col,
                                          const uint32_t r0, const uint32_t r1, const uint32_t rows, const uint32_t nchunks) {
    uint32_t v[HELD], sum = 0;
#pragma unroll
    for (int u = 0; u < HELD; ++u) v[u] = col[(size_t)umin(r0 + u, nchunks - 1u) * kScanDigits];
#pragma unroll
    for (int u = 0; u < HELD; ++u) sum += r0 + u < r1 ? v[u] : 0u;
    uint32_t run = scan_parts(s_part, dl, part, sum);
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
        if (r0 + u < r1 || (r0 + u == nchunks && (uint32_t)u < rows)) col[(size_t)(r0 + u) * kScanDigits] = run;   // (the part's own rows alone)
        run += r0 + u < r1 ? v[u] : 0u;
    }
}
__global__ __launch_bounds__(kScanThreads) void radix_scan_kernel(const SortArgs a) {
    __shared__ uint32_t s_part[kScanDigits][kScanParts];
    const uint32_t nchunks = *a.nchunks;   // at most max_chunks
    const uint32_t dl = threadIdx.x & (kScanDigits - 1), part = threadIdx.x / kScanDigits;
    uint32_t* const col = static_cast<uint32_t*>(a.ghist) + hist_word(a, 0u, blockIdx.x * kScanDigits + dl);
    const uint32_t rows = (nchunks + kScanParts) / kScanParts;   // of every part: nchunks + 1 of them in all
    const uint32_t r0 = part * rows, r1 = umin(r0 + rows, nchunks);
    if (rows <= 12u) {
        scan_held<12>(s_part, dl, part, col, r0, r1, rows, nchunks);
    } else if (rows <= 32u) {
        scan_held<32>(s_part, dl, part, col, r0, r1, rows, nchunks);
    } else if (rows <= 66u) {
        scan_held<66>(s_part, dl, part, col, r0, r1, rows, nchunks);
    } else {
        uint32_t sum = 0;
        for (uint32_t r = r0; r < r1; ++r) sum += col[(size_t)r * kScanDigits];
        uint32_t run = scan_parts(s_part, dl, part, sum);
        for (uint32_t r = r0; r < r1; ++r) {
            const uint32_t v = col[(size_t)r * kScanDigits];
            col[(size_t)r * kScanDigits] = run;
            run += v;
        }
        if (nchunks >= r0 && nchunks < r0 + rows) col[(size_t)nchunks * kScanDigits] = run;
    }
}
static_assert(kScanParts == 2 * kWave && kScanDigits * kWave <= kScanThreads, "two parts per lane, a wavefront per digit");

template <int NB, int ITEMS>
struct ScatterLds {
    uint32_t cnt[kRsWaves][NB];     // per-wave digit counts, then per-wave exclusive offsets
    uint32_t base[NB];              // where this chunk's next element of digit d goes
    uint32_t dstart[NB];            // start of digit d inside the locally sorted tile
    __align__(16) uint32_t keys[ITEMS * kRsThreads];
    uint32_t vals[ITEMS * kRsThreads];
    uint32_t scan[kRsWaves];
    OwnerLds own;
};

// One tile of a chunk.  FULL: all positions of the tile exist, so nothing is predicated (all but a chunk's last tile).
template <typename IT, int NB, int ITEMS, bool FIRST, bool FULL>
__device__ __forceinline__ void scatter_tile(const SortArgs& a, const ChunkDesc& ds, const int64_t rb, const int64_t R,
                                             const int64_t tile, const int64_t e, ScatterLds<NB, ITEMS>* L) {
    constexpr int K = NB / kRsThreads;   // digits per thread in the scans
    constexpr int kTile = ITEMS * kRsThreads;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid >> 6;
    const int64_t wbase = tile + (int64_t)w * (kWave * ITEMS);
    uint32_t key[ITEMS], val[ITEMS], off[ITEMS];
    if (FIRST) {
        const int64_t te = FULL ? tile + kTile : e;
        IT id[ITEMS];
        load_ids<IT, ITEMS>(static_cast<const IT*>(a.indices), tile, te, id);
        if (!a.iota || !a.by_table) {
            const int64_t blo = a.by_table ? (int64_t)ds.seg * a.B : 0, bhi = a.by_table ? blo + a.B : a.nbags;
            tile_owners<IT, ITEMS>(static_cast<const IT*>(a.offsets), blo, bhi, tile, te, reinterpret_cast<int32_t*>(L->keys), &L->own, val);
        }
        if (a.by_table) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) key[k] = (id[k] >= 0 && id[k] < R) ? (uint32_t)id[k] : (uint32_t)R;
        } else {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int64_t b0 = a.row_base[val[k] / (uint32_t)a.B], b1 = a.row_base[val[k] / (uint32_t)a.B + 1];
                key[k] = (id[k] >= 0 && id[k] < b1 - b0) ? (uint32_t)(b0 + id[k]) : a.invalid_key;
            }
        }
        if (a.iota) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) val[k] = (uint32_t)(wbase + k * kWave + lane);
        }
    } else {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = wbase + k * kWave + lane;
            const bool valid = FULL || i < e;
            key[k] = valid ? a.keys_in[i] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = wbase + k * kWave + lane;
            val[k] = FULL || i < e ? a.vals_in[i] : 0u;
        }
    }
    for (int i = tid; i < kRsWaves * NB; i += kRsThreads) (&L->cnt[0][0])[i] = 0u;
    __syncthreads();  // also orders the base update / key reads of the previous tile
    // Rank inside the wave, item by item in input order: the lanes that hold the same digit, whose first adds their number to the
    // wave's count.  The additions are all under way before the first result is waited for (LDS operations of a wave stay in order).
    // With two instructions more per bit and a wait for every addition, all scatters of a step, us: 32 tables, 26 M lookups 315 -> 298;
    // 64 tables, 65 M 869 -> 846; sequences of 3.1 M 66.7 -> 62.3; the rest is the streams (64 tables: 3.7 TB/s read and written).
    constexpr int kBits = NB == 256 ? 8 : (NB == 1024 ? 10 : 11);
    uint32_t old[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const bool valid = FULL || wbase + k * kWave + lane < e;
        const uint32_t d = (key[k] >> a.shift) & a.mask;
        const uint64_t vmask = FULL ? ~0ull : __builtin_amdgcn_ballot_w64(valid);
        uint32_t plo = (uint32_t)vmask, phi = (uint32_t)(vmask >> 32);
#pragma unroll
        for (int b = 0; b < kBits; ++b) same_bit(d, b, plo, phi);   // (bits above the digit's width are zero in every lane)
        const uint64_t peers = ((uint64_t)phi << 32) | plo;   // never empty for a valid lane: it holds the lane itself
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        const uint32_t leader = (uint32_t)__ffsll((unsigned long long)peers) - 1u;
        off[k] = rank | leader << 8;
        old[k] = 0;
        if (valid && rank == 0u) old[k] = atomicAdd(&L->cnt[w][d], (uint32_t)__popcll(peers));
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) off[k] = (off[k] & 0xFFu) + __shfl(old[k], (int)(off[k] >> 8), kWave);
    __syncthreads();
    // per digit: exclusive offsets over the waves, tile total, exclusive scan over the digits
    uint32_t mine[K], sum = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        uint32_t run = 0;
#pragma unroll
        for (int ww = 0; ww < kRsWaves; ++ww) {
            const uint32_t c = L->cnt[ww][tid * K + j];
            L->cnt[ww][tid * K + j] = run;
            run += c;
        }
        mine[j] = run;
        sum += run;
    }
    {
        uint32_t tot;
        uint32_t ex = block_excl_scan<kRsThreads>(sum, L->scan, &tot);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            L->dstart[tid * K + j] = ex;
            ex += mine[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = wbase + k * kWave + lane;
        if (FULL || i < e) {
            const uint32_t d = (key[k] >> a.shift) & a.mask;
            const uint32_t pos = L->dstart[d] + L->cnt[w][d] + off[k];
            L->keys[pos] = key[k];
            L->vals[pos] = val[k];
        }
    }
    __syncthreads();
    const int cnt = FULL ? kTile : (int)(e - tile);
    for (int j = tid; j < cnt; j += kRsThreads) {
        const uint32_t kk = L->keys[j];
        const uint32_t d = (kk >> a.shift) & a.mask;
        const uint32_t dst = L->base[d] + ((uint32_t)j - L->dstart[d]);
        // last pass of a table-by-table sort: table-local id -> linearised row key
        a.keys_out[dst] = a.globalize ? ((int64_t)kk >= R ? a.invalid_key : (uint32_t)(rb + kk)) : kk;
        a.vals_out[dst] = L->vals[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < K; ++j) L->base[tid * K + j] += mine[j];
}

template <typename IT, int NB, int ITEMS, bool FIRST, bool SELF>
__global__ __launch_bounds__(kRsThreads, NB == 256 && !FIRST ? 4 : 1) void radix_scatter_kernel(const SortArgs a) {
    constexpr int K = NB / kRsThreads;
    constexpr int kTile = ITEMS * kRsThreads;
    __shared__ ScatterLds<NB, ITEMS> L;
    const uint32_t chunk = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);   // (the grid is a multiple of 8)
    if (chunk >= (uint32_t)a.max_chunks) return;
    const ChunkDesc ds = a.desc[chunk];
    if (ds.e <= ds.s) return;
    const int tid = threadIdx.x;
    const int64_t rb = a.by_table ? a.row_base[ds.seg] : 0;
    const int64_t R = a.by_table ? a.row_base[ds.seg + 1] - rb : 0;
    {   // base of every digit for this chunk: segment start + (digits below d, whole segment) + (digit d, the
        // segment's chunks before this one)
        uint32_t tot[K], pre[K], sum = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) tot[j] = pre[j] = 0u;
        if (SELF) {
            struct __align__(2 * K) Counts { uint16_t c[K]; };
            const uint16_t* q = static_cast<const uint16_t*>(a.ghist) + (size_t)ds.first * NB + tid * K;
            const uint32_t before = chunk - ds.first;
            constexpr int kU = 16;   // chunk histograms in flight
            for (uint32_t i0 = 0; i0 < ds.count; i0 += kU) {
                Counts v[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint32_t i = i0 + u < ds.count ? i0 + u : ds.count - 1u;
                    v[u] = *reinterpret_cast<const Counts*>(q + (size_t)i * NB);
                }
#pragma unroll
                for (int u = 0; u < kU; ++u)
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        tot[j] += i0 + u < ds.count ? (uint32_t)v[u].c[j] : 0u;
                        pre[j] += i0 + u < before ? (uint32_t)v[u].c[j] : 0u;
                    }
            }
        } else {
            const uint32_t* const q = static_cast<const uint32_t*>(a.ghist);
            const uint32_t first = q[hist_word(a, ds.first, tid)];
            tot[0] = q[hist_word(a, ds.first + ds.count, tid)] - first;
            pre[0] = q[hist_word(a, chunk, tid)] - first;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) sum += tot[j];
        uint32_t all;
        uint32_t ex = ds.seg_start + block_excl_scan<kRsThreads>(sum, L.scan, &all);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            L.base[tid * K + j] = ex + pre[j];
            ex += tot[j];
        }
    }
    const int64_t s = ds.s, e = ds.e;
    for (int64_t tile = s; tile < e; tile += kTile) {
        if (e - tile >= (int64_t)kTile) scatter_tile<IT, NB, ITEMS, FIRST, true>(a, ds, rb, R, tile, e, &L);
        else scatter_tile<IT, NB, ITEMS, FIRST, false>(a, ds, rb, R, tile, e, &L);
    }
}

template <typename IT, int NB, int ITEMS, bool SELF>
static void launch_hist0(const SortArgs& a, const unsigned grid, hipStream_t s) {
    if (a.by_table) radix_hist_kernel<IT, NB, ITEMS, true, false, SELF><<<grid, kRsThreads, 0, s>>>(a);
    else radix_hist_kernel<IT, NB, ITEMS, true, true, SELF><<<grid, kRsThreads, 0, s>>>(a);
}

template <int NB, int ITEMS, bool SELF>
static void launch_pass(const tbe_handle* h, const SortArgs& a, const SortShape& sh, bool first, bool idx32, hipStream_t s) {
    const unsigned grid = (unsigned)sh.max_chunks;
    const unsigned sgrid = (grid + 7u) & ~7u;
    {
        LaunchTimer tm(h, s, "radix_hist");
        if (!first) radix_hist_kernel<int32_t, NB, ITEMS, false, false, SELF><<<grid, kRsThreads, 0, s>>>(a);
        else if (idx32) launch_hist0<int32_t, NB, ITEMS, SELF>(a, grid, s);
        else launch_hist0<int64_t, NB, ITEMS, SELF>(a, grid, s);
        tm.done();
    }
    if (!SELF) {
        LaunchTimer tm(h, s, "radix_scan");
        radix_scan_kernel<<<256 / kScanDigits, kScanThreads, 0, s>>>(a);
        tm.done();
    }
    LaunchTimer tm(h, s, "radix_scatter");
    if (!first) radix_scatter_kernel<int32_t, NB, ITEMS, false, SELF><<<sgrid, kRsThreads, 0, s>>>(a);
    else if (idx32) radix_scatter_kernel<int32_t, NB, ITEMS, true, SELF><<<sgrid, kRsThreads, 0, s>>>(a);
    else radix_scatter_kernel<int64_t, NB, ITEMS, true, SELF><<<sgrid, kRsThreads, 0, s>>>(a);
    tm.done();
}

__global__ __launch_bounds__(kRleThreads) void rle_count_kernel(const RleArgs a) {
    __shared__ uint2 s_w[kRleThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kRleTile;
    uint32_t c = 0, l = 0;   // heads seen by this wavefront: one ballot and one population count per run of 64 keys
    uint32_t cur[kRleItems];
    bool head[kRleItems], lng[kRleItems];
    head_flags<kRleThreads>(a, base, a.N, cur, head, lng);
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        c += (uint32_t)__popcll(__ballot(head[k]));
        l += (uint32_t)__popcll(__ballot(lng[k]));
    }
    if (lane_id() == 0) s_w[threadIdx.x >> 6] = make_uint2(c, l);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint2 tot = make_uint2(0u, 0u);
#pragma unroll
        for (int w = 0; w < kRleThreads / kWave; ++w) {
            tot.x += s_w[w].x;
            tot.y += s_w[w].y;
        }
        a.counts[blockIdx.x] = tot;
    }
}

// single block, batches of many tiles: exclusive scan of the per-tile counts in place
__global__ __launch_bounds__(1024) void rle_scan_kernel(uint2* __restrict__ counts, const int nblocks) {
    __shared__ uint32_t smem[1024 / kWave];
    uint32_t carry_h = 0, carry_l = 0;
    for (int base = 0; base < nblocks; base += 4 * 1024) {   // four counts per thread and round: a quarter of the barriers
        const int i = base + 4 * (int)threadIdx.x;
        uint2 v[4];
        uint32_t sh = 0, sl = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = (i + q < nblocks) ? counts[i + q] : make_uint2(0u, 0u);
            sh += v[q].x;
            sl += v[q].y;
        }
        uint32_t th, tl;
        uint32_t rh = carry_h + block_excl_scan<1024>(sh, smem, &th);
        uint32_t rl = carry_l + block_excl_scan<1024>(sl, smem, &tl);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i + q < nblocks) counts[i + q] = make_uint2(rh, rl);
            rh += v[q].x;
            rl += v[q].y;
        }
        carry_h += th;
        carry_l += tl;
    }
}

// What lies before a tile: the sum of the counts of the tiles before it, or (SCANNED, batches of many tiles) their scan.
constexpr int kRleSumTiles = 2048;  // at most 8 counts per thread
template <bool SCANNED>
__global__ __launch_bounds__(kRleThreads) void rle_write_kernel(const RleArgs a) {
    __shared__ uint32_t s_run[kRleItems * (kRleThreads / kWave) + 1];
    __shared__ uint2 s_sum[kRleThreads / kWave];
    const uint32_t tile = blockIdx.x;
    const int64_t base = (int64_t)tile * kRleTile;
    uint32_t cur[kRleItems];
    bool head[kRleItems], lng[kRleItems];
    head_flags<kRleThreads>(a, base, a.N, cur, head, lng);
    uint32_t bb = 0, bl = 0;
    if (SCANNED) {
        const uint2 v = a.counts[tile];
        bb = v.x;
        bl = v.y;
    } else {
        for (uint32_t i0 = 0; i0 < tile; i0 += 4 * kRleThreads) {
            uint2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t i = i0 + u * kRleThreads + threadIdx.x;
                v[u] = a.counts[i < tile ? i : 0u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = i0 + u * kRleThreads + threadIdx.x < tile;
                bb += in ? v[u].x : 0u;
                bl += in ? v[u].y : 0u;
            }
        }
        bb = wave_incl_scan(bb);
        bl = wave_incl_scan(bl);
        if (lane_id() == kWave - 1) s_sum[threadIdx.x >> 6] = make_uint2(bb, bl);
        __syncthreads();
        bb = bl = 0;
#pragma unroll
        for (int i = 0; i < kRleThreads / kWave; ++i) {
            bb += s_sum[i].x;
            bl += s_sum[i].y;
        }
    }
    const uint2 tot = rle_write_tile<kRleThreads>(a, base, bb, bl, cur, head, lng, s_run);
    if (tile == gridDim.x - 1 && threadIdx.x == 0) rle_finish(a, bb + tot.x, bl + tot.y);
}

// Small batches (up to kRleOneBlock lookups): one workgroup walks all tiles of 8192 - one launch, nothing to add up.
__global__ __launch_bounds__(1024) void rle_one_block_kernel(const RleArgs a) {
    __shared__ uint32_t s_run[kRleItems * (1024 / kWave) + 1];
    uint32_t bb = 0, bl = 0;
    for (int64_t base = 0; base < a.N; base += kRleItems * 1024) {
        uint32_t cur[kRleItems];
        bool head[kRleItems], lng[kRleItems];
        head_flags<1024>(a, base, a.N, cur, head, lng);
        const uint2 tot = rle_write_tile<1024>(a, base, bb, bl, cur, head, lng, s_run);
        bb += tot.x;
        bl += tot.y;
        __syncthreads();   // s_run is written again
    }
    if (threadIdx.x == 0) rle_finish(a, bb, bl);
}

static hipError_t launch_run_lengths(const tbe_handle* h, const Workspace& w, const RleArgs& a, hipStream_t s) {
    const int64_t N = a.N;
    const int n = w.rle_blocks;
    if (N <= kRleOneBlock) {
        LaunchTimer tm(h, s, "rle_write");
        rle_one_block_kernel<<<1, 1024, 0, s>>>(a);
        tm.done();
        return hipGetLastError();
    }
    {
        LaunchTimer tm(h, s, "rle_count");
        rle_count_kernel<<<n, kRleThreads, 0, s>>>(a);
        tm.done();
    }
    if (n > kRleSumTiles) {
        LaunchTimer tm(h, s, "rle_scan");
        rle_scan_kernel<<<1, 1024, 0, s>>>(a.counts, n);
        tm.done();
    }
    LaunchTimer tm(h, s, "rle_write");
    if (n <= kRleSumTiles) rle_write_kernel<false><<<n, kRleThreads, 0, s>>>(a);
    else rle_write_kernel<true><<<n, kRleThreads, 0, s>>>(a);
    tm.done();
    return hipGetLastError();
}

hipError_t launch_sort(const tbe_handle* h, const Workspace& w, char* ws, const void* indices, const void* offsets, int idx32,
                       int32_t B, int64_t N, bool seq, hipStream_t s) {
    const SortShape& sh = w.sort;
    SortArgs a;
    a.indices = indices;
    a.offsets = offsets;
    a.row_base = h->d_row_base;
    a.desc = reinterpret_cast<ChunkDesc*>(ws + w.chunk_desc);
    a.nchunks = sh.self_scan ? nullptr : reinterpret_cast<uint32_t*>(ws + w.nchunks);
    a.ghist = ws + w.radix_hist;
    a.err = h->d_err;
    a.N = N;
    a.chunk = sh.chunk;
    a.nbags = (int64_t)h->T * B;
    a.B = B;
    a.nseg = sh.nseg;
    a.max_chunks = sh.max_chunks;
    a.mask = (1u << sh.bits) - 1u;
    a.invalid_key = (uint32_t)h->total_rows;
    a.by_table = h->segmented || h->T == 1;
    a.iota = seq;
    const int sorted = sh.passes & 1;   // every pass flips the double buffer, starting from 0
    RleArgs r;
    r.keys = reinterpret_cast<const uint32_t*>(ws + w.keys[sorted]);
    r.N = N;
    r.long_min = w.long_min;
    r.total_rows = (uint32_t)h->total_rows;
    r.counts = reinterpret_cast<uint2*>(ws + w.rle_counts);
    r.unique_rows = reinterpret_cast<uint32_t*>(ws + w.vals[sorted ^ 1]);
    r.seg_start = reinterpret_cast<uint32_t*>(ws + w.seg_start);
    r.long_rows = reinterpret_cast<uint2*>(ws + w.long_rows);
    r.counters = reinterpret_cast<uint32_t*>(ws + w.counters);
    if (sh.small) {
        a.keys_out = reinterpret_cast<uint32_t*>(ws + w.keys[sorted]);
        a.vals_out = reinterpret_cast<uint32_t*>(ws + w.vals[sorted]);
        return launch_sort_small(h, a, r, idx32, s);
    }
    for (int p = 0; p < sh.passes; ++p) {
        a.keys_in = reinterpret_cast<const uint32_t*>(ws + w.keys[p & 1]);
        a.vals_in = reinterpret_cast<const uint32_t*>(ws + w.vals[p & 1]);
        a.keys_out = reinterpret_cast<uint32_t*>(ws + w.keys[(p & 1) ^ 1]);
        a.vals_out = reinterpret_cast<uint32_t*>(ws + w.vals[(p & 1) ^ 1]);
        a.shift = p * sh.bits;
        a.globalize = h->segmented && p == sh.passes - 1;
        const bool first = p == 0;
        const bool idx = idx32 != 0;
        // (the digits a.mask can hold never exceed the bins a kernel is compiled for)
        if (!sh.self_scan && sh.bins == 256 && sh.tile == 4096) launch_pass<256, 16, false>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 256 && sh.tile == 4096) launch_pass<256, 16, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 256 && sh.tile == 2048) launch_pass<256, 8, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 1024 && sh.tile == 2048) launch_pass<1024, 8, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 2048 && sh.tile == 2048) launch_pass<2048, 8, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 256 && sh.tile == 1024) launch_pass<256, 4, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 1024 && sh.tile == 1024) launch_pass<1024, 4, true>(h, a, sh, first, idx, s);
        else if (sh.self_scan && sh.bins == 2048 && sh.tile == 1024) launch_pass<2048, 4, true>(h, a, sh, first, idx, s);
        else return hipErrorInvalidValue;
    }
    return launch_run_lengths(h, w, r, s);
}

}  // namespace tbe
