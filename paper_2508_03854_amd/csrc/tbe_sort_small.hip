// Small batches: ids to sorted (key, payload) pairs in one launch, and the counts that the run lengths need with it.
//
// Passes over digits are a chain of launches, two each, that a small batch cannot fill.  Here a workgroup owns a range of at most
// kSmallChunk places of one segment's SORTED order and finds the elements that belong there by itself, from the segment's ids
// alone, so that nothing has to be exchanged between workgroups:
//   1. the segment's keys are made from its ids (and kept in LDS, up to kSmallHeld of them);
//   2. a radix selection, histograms of digits of up to ten bits from the top, finds the keys at the range's first and last place:
//      their first digits, unless more elements than there are threads share those or lie between, then as many more as it takes;
//   3. the elements from the one to the other are compacted in order of position;
//   4. a stable radix sort in LDS on what distinguishes them, up to six bits a pass, one element per thread;
//   5. the payload (a binary search for the position's bag, most steps in LDS), and the range's heads and long rows counted.
// What workgroups repeat is the reading of the segment and steps 2 and 3 on it.  It is the same for any distribution of the ids
// over the segments and over the rows: a range has its places, whether they hold as many rows or one.
//
// Bound: latency, a chain of about ten barriers, and the instructions spent on the whole segment.  So a wavefront per border scans
// the histograms and every wavefront the counts, and loops are kept rolled: instructions come from memory too, and the same steps
// unrolled over up to 64 keys in registers took 23 us where this takes 11.6 (one table, 10240 uniform ids of 100000 rows: find the
// range 1.6, keys and first histogram 1.6, borders 1.5, count and compact 2.4, sort 2.6, bags and output 1.0).  In ranges of 1024
// places 14.6.
// Against passes over digits, prepare call with run lengths and lists, us: one table, 100 / 2000 / 8000 / 12288 uniform ids of 100000
// rows 24 26 28 31 / 16 17 18 19, of Zipf 1.3 24 30 33 35 / 16 21 26 31, of 3 rows (long runs everywhere) 19 20 22 23 / 17 18 22 24;
// 10 tables x 6000 35 / 23, 26 x 2500 34 / 20, 64 x 1000 34 / 19, 200 x 300 39 / 27.  The whole step of one table, 512 bags of 20 ids,
// 64 columns 44.4 / 34.0; of ten tables of odd widths x 777 bags 104 / 93.
#include "tbe_sort.h"

namespace tbe {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSelBits = 10, kSelBins = 1 << kSelBits;   // 16 bins per lane in a wavefront's scan
constexpr int kSmallHeld = 32 * kSmallThreads;           // keys in LDS; of larger segments they are made from the ids again
constexpr int kBagSteps = 2048;                          // offsets of a table in LDS: all, or every 2nd, 4th, ...
static_assert(kSmallChunk <= kSmallThreads && kSelBins == 16 * kWave, "an element per thread, 16 bins per lane");
constexpr uint32_t kNoKey = 0xFFFFFFFFu;                 // (keys are below 2^31)
// in a range's counts: it starts a segment with an id outside its table, or ends in one
constexpr uint32_t kRangeStartsInvalid = 0x80000000u, kRangeEndsInvalid = 0x40000000u;

struct SmallLds {
    union {
        __align__(16) uint32_t hist[4][kSelBins];   // spread over the lanes at first, then one per border
        struct { uint32_t key[kSmallThreads], pos[kSmallThreads]; } buf[2];
    };
    uint32_t cnt[kSmallWaves][kWave];
    uint32_t off[kBagSteps];
    uint4 taken[kSmallWaves], place[2];
    uint32_t scan[kSmallWaves], total;
    ChunkDesc desc;
};

struct Place { uint32_t bin, before, count; };   // a bin, the elements in bins below, and in it
// The bin of element number x (x below their sum) of a histogram, or of four that follow one another added up.  By one wavefront.
template <int COPIES>
__device__ __forceinline__ Place find_place(const uint32_t* h, const uint32_t x) {
    const int lane = lane_id();
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < COPIES; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // (in an order that spreads the lanes over the banks)
            const uint4 v = *reinterpret_cast<const uint4*>(h + q * kSelBins + 16 * lane + 4 * ((j + lane) & 3));
            sum += v.x + v.y + v.z + v.w;
        }
    const uint32_t incl = wave_incl_scan(sum);
    const int f = __ffsll((unsigned long long)__ballot(incl > x)) - 1;
    const uint32_t below = bcast_lane(incl - sum, f);
    const int bin = 16 * f + (lane & 15);
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < COPIES; ++q) c += h[q * kSelBins + bin];
    uint32_t in_row = c;   // inclusive, within the 16 lanes of a row, which hold the same
    in_row += dpp_or_zero<0x111, 0xF>(in_row);
    in_row += dpp_or_zero<0x112, 0xF>(in_row);
    in_row += dpp_or_zero<0x114, 0xF>(in_row);
    in_row += dpp_or_zero<0x118, 0xF>(in_row);
    const int g = (__ffsll((unsigned long long)__ballot(below + in_row > x)) - 1) & 15;
    return Place{(uint32_t)(16 * f + g), below + bcast_lane(in_row - c, g), bcast_lane(c, g)};
}

// The range of a workgroup, as find_chunk; up to 64 segments by every wavefront for itself, without a barrier.
template <typename IT, int NT>
__device__ __forceinline__ ChunkDesc find_range(const SortArgs& a, const uint32_t c, uint32_t* smem, ChunkDesc* s_desc) {
    if (a.nseg == 1 || a.nseg > kWave) return find_chunk<IT, NT>(a, c, smem, s_desc);
    const int t = lane_id();
    int64_t b = t + 1 >= a.nseg ? a.N : (int64_t)static_cast<const IT*>(a.offsets)[(int64_t)(t + 1) * a.B];
    b = b < 0 ? 0 : (b > a.N ? a.N : b);
    const uint32_t b1 = wave_incl_max((uint32_t)b);
    const uint32_t up = __shfl_up(b1, 1, kWave), b0 = t == 0 ? 0u : up;
    const uint32_t chunk = (uint32_t)a.chunk, n = (b1 - b0 + chunk - 1u) / chunk;   // (lanes behind the last segment: none)
    const uint32_t f = wave_incl_scan(n) - n;
    const uint64_t m = __ballot(c >= f && c - f < n);
    if (m == 0ull) return ChunkDesc{0, 0, 0, 0, 0, 0, 0, 0};
    const int seg = __ffsll((unsigned long long)m) - 1;
    const uint32_t first = bcast_lane(f, seg), start = bcast_lane(b0, seg), end = bcast_lane(b1, seg);
    const uint32_t s = start + (c - first) * chunk, e = umin(s + chunk, end);
    return ChunkDesc{s, e, (uint32_t)seg, first, bcast_lane(n, seg), start, end, 0};
}

template <typename IT>
__global__ __launch_bounds__(kSmallThreads) void sort_small_kernel(const SortArgs a, uint2* __restrict__ counts, const uint32_t long_min) {
    __shared__ SmallLds S;
    extern __shared__ uint32_t s_keys[];   // min(N, kSmallHeld), whole rounds of the workgroup
    // (neighbouring ranges read the same ids: on one die.  The grid is a multiple of 8)
    const uint32_t chunk = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (chunk >= (uint32_t)a.max_chunks) return;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id();
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const ChunkDesc ds = find_range<IT, kSmallThreads>(a, chunk, S.scan, &S.desc);
    if (tid == 0) {
        a.desc[chunk] = ds;
        if (ds.e <= ds.s) counts[chunk] = make_uint2(0u, 0u);
    }
    if (ds.e <= ds.s) return;
    const int64_t rb = a.row_base[ds.seg];
    const uint32_t R = (uint32_t)(a.row_base[ds.seg + 1] - rb);
    reinterpret_cast<uint4*>(S.hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) S.total = 0u;
    // ---- the table's offsets: every 2^bag_log2-th
    const IT* const offsets = static_cast<const IT*>(a.offsets) + (int64_t)ds.seg * a.B;
    int bag_log2 = 0;
    while ((a.B - 1) >> bag_log2 >= kBagSteps) ++bag_log2;
    const uint32_t bag_steps = ((uint32_t)(a.B - 1) >> bag_log2) + 1u;
    if (!a.iota) {
        for (uint32_t j = tid; j < bag_steps; j += kSmallThreads) {
            const int64_t o = (int64_t)offsets[(int64_t)j << bag_log2];
            S.off[j] = (uint32_t)(o < 0 ? 0 : (o > a.N ? a.N : o));
        }
    }
    __syncthreads();
    // ---- the segment's keys: element k of this lane is the segment's element number first + 64 k
    const uint32_t n = ds.seg_end - ds.seg_start;
    const uint32_t per = (n + kSmallThreads - 1u) / kSmallThreads;   // elements per lane
    const uint32_t first = w * per * kWave + (uint32_t)lane;
    const bool held = n <= (uint32_t)kSmallHeld;
    const IT* const ids = static_cast<const IT*>(a.indices) + ds.seg_start;
    bool bad = false;
    auto from_ids = [&](auto f) {
        constexpr uint32_t kU = 8;   // ids in flight
#pragma unroll 1
        for (uint32_t k0 = 0; k0 < per; k0 += kU) {
            IT id[kU];
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u) id[u] = ids[umin(first + (k0 + u) * kWave, n - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u) {
                if (k0 + u >= per) break;
                const bool in = first + (k0 + u) * kWave < n;
                const bool ok = id[u] >= 0 && (int64_t)id[u] < (int64_t)R;
                bad |= in && !ok;
                f(in ? (ok ? (uint32_t)id[u] : R) : kNoKey, first + (k0 + u) * kWave);
            }
        }
    };
    auto each_key = [&](auto f) {
        if (held) {
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < per; k0 += 2u) {
                const uint32_t at = first + k0 * kWave, next = at + (k0 + 1u < per ? kWave : 0u);
                const uint32_t x = s_keys[at], y = s_keys[next];
                f(x, at);
                f(k0 + 1u < per ? y : kNoKey, next);
            }
        } else {
            from_ids(f);
        }
    };
    // ---- the keys at places r0 and r0 + cnt - 1 (0: the lower border, 1: the upper one), digit by digit from the top
    const uint32_t r0 = ds.s - ds.seg_start, cnt = ds.e - ds.s;
    const uint32_t bits = 32u - (uint32_t)__clz((int)R);
    const uint32_t levels = (bits + kSelBits - 1u) / kSelBits, width = (bits + levels - 1u) / levels;
    const uint32_t mask = (1u << width) - 1u;
    uint32_t low = (levels - 1u) * width;   // bits below the digit
    {
        uint32_t* const h = S.hist[lane & 3];
        from_ids([&](const uint32_t k, const uint32_t at) {
            if (held) s_keys[at] = k;
            if (k != kNoKey) atomicAdd(&h[k >> low], 1u);
        });
    }
    if (bad) atomicOr(a.err, 1);
    __syncthreads();
    // (a wavefront per border; all of them reading the histogram would take as long as 16 of these in turn)
    if (w < 2u) {
        const Place p = find_place<4>(S.hist[0], w == 0u ? r0 : r0 + cnt - 1u);
        if (lane == 0) S.place[w] = make_uint4(p.bin, p.before, p.count, 0u);
    }
    __syncthreads();
    // digits so far, smaller keys, keys from border to border (at first as far as those digits tell), keys of the upper border's
    uint32_t key0 = 0, key1 = 0, before0 = 0, before1 = 0, between = 0, count1 = 0;
    auto take_borders = [&] {
        const uint4 p = S.place[lane & 1];
        key0 = key0 << width | bcast_lane(p.x, 0);
        key1 = key1 << width | bcast_lane(p.x, 1);
        before0 += bcast_lane(p.y, 0);
        before1 += bcast_lane(p.y, 1);
        count1 = bcast_lane(p.z, 1);
        between = before1 + count1 - before0;
    };
    take_borders();
    while (low > 0u && between > (uint32_t)kSmallThreads) {
        const uint32_t high = low;
        low -= width;
        if (tid < 2u * kSelBins / 4u) reinterpret_cast<uint4*>(S.hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        each_key([&](const uint32_t k, uint32_t) {
            const uint32_t d = k >> high;
            if (d == key0) atomicAdd(&S.hist[0][(k >> low) & mask], 1u);
            else if (d == key1) atomicAdd(&S.hist[1][(k >> low) & mask], 1u);
        });
        __syncthreads();
        if (w < 2u) {
            const Place p = find_place<1>(S.hist[key0 == key1 ? 0u : w], w == 0u ? r0 - before0 : r0 + cnt - 1u - before1);
            if (lane == 0) S.place[w] = make_uint4(p.bin, p.before, p.count, 0u);
        }
        __syncthreads();
        take_borders();
    }
    // ---- the elements from border to border, in order of position.  As many as there are threads: all of them, and the range is a
    // part of them once they are sorted.  More: the borders are whole keys, and of the lower one's the elements from number a_lo on are
    // taken (and, if it is the upper one too, before a_hi), of the upper one's those before number b_hi.
    const bool whole = between <= (uint32_t)kSmallThreads, one_key = key0 == key1;
    const uint32_t base = key0 << low, top = ((key1 - key0 + 1u) << low) - 1u;
    const uint32_t a_lo = r0 - before0, a_hi = one_key ? a_lo + cnt : kNoKey, b_hi = r0 + cnt - before1;
    uint32_t nr = 0, na = 0, nb = 0;   // elements from border to border, of the lower border's key, of the upper one's
    if (whole)
        each_key([&](const uint32_t k, uint32_t) { nr += (uint32_t)__popcll(__ballot(k - base <= top)); });
    else
        each_key([&](const uint32_t k, uint32_t) {
            nr += (uint32_t)__popcll(__ballot(k - base <= top));
            na += (uint32_t)__popcll(__ballot(k == key0));
            nb += (uint32_t)__popcll(__ballot(k == key1));
        });
    if (lane == 0) S.taken[w] = make_uint4(nr, na, nb, 0u);
    __syncthreads();
    {
        const uint4 v = S.taken[lane & (kSmallWaves - 1)];
        const bool before = (uint32_t)lane < w;
        nr = bcast_lane(wave_incl_scan(before ? v.x : 0u), kWave - 1);
        na = bcast_lane(wave_incl_scan(before ? v.y : 0u), kWave - 1);
        nb = bcast_lane(wave_incl_scan(before ? v.z : 0u), kWave - 1);
    }
    const uint64_t lt = lanemask_lt();
    if (whole) {
        each_key([&](const uint32_t k, const uint32_t p) {
            const bool on = k - base <= top;
            const uint64_t mr = __ballot(on);
            if (on) {
                const uint32_t at = nr + (uint32_t)__popcll(mr & lt);
                S.buf[0].key[at] = k - base;
                S.buf[0].pos[at] = ds.seg_start + p;
            }
            nr += (uint32_t)__popcll(mr);
        });
    } else {
        // the range's elements among the first r, x, y
        auto place = [&](const uint32_t r, const uint32_t x, const uint32_t y) {
            const uint32_t t = (x < a_lo ? a_lo : (x > a_hi ? a_hi : x)) - a_lo;
            return one_key ? t : r - x - y + t + umin(y, b_hi);
        };
        each_key([&](const uint32_t k, const uint32_t p) {
            const uint64_t mr = __ballot(k - base <= top), ma = __ballot(k == key0), mb = __ballot(k == key1);
            if (mr == 0ull) return;
            const uint32_t x = na + (uint32_t)__popcll(ma & lt), y = nb + (uint32_t)__popcll(mb & lt);
            const bool on = k == key0 ? x >= a_lo && x < a_hi : (k == key1 ? y < b_hi : k - base <= top);
            if (on) {
                const uint32_t at = place(nr + (uint32_t)__popcll(mr & lt), x, y);
                S.buf[0].key[at] = k - base;
                S.buf[0].pos[at] = ds.seg_start + p;
            }
            nr += (uint32_t)__popcll(mr);
            na += (uint32_t)__popcll(ma);
            nb += (uint32_t)__popcll(mb);
        });
    }
    __syncthreads();
    // ---- sorted by what the keys differ in, stably; one element per thread, a digit's counts per wavefront
    const uint32_t m = whole ? between : cnt;
    const bool on = tid < m;
    uint32_t my = S.buf[0].key[tid], pos = S.buf[0].pos[tid];
    const int diff = top == 0u ? 0 : 32 - __clz((int)top);
    const int passes = (diff + 5) / 6, db = passes == 0 ? 0 : (diff + passes - 1) / passes;
    for (int ps = 0; ps < passes; ++ps) {
        const uint32_t d = (my >> (ps * db)) & ((1u << db) - 1u);
        uint32_t rank = 0;
        S.cnt[w][lane] = 0u;
        if (w * kWave < m) {
            const uint64_t peers = same_digit(d, db, __ballot(on));
            rank = (uint32_t)__popcll(peers & lt);
            if (on && rank == 0u) S.cnt[w][d] = (uint32_t)__popcll(peers);
        }
        __syncthreads();
        auto& out = S.buf[(ps + 1) & 1];
        if (w * kWave < m) {
            uint32_t c[kSmallWaves], all = 0, mine = 0;   // of digit `lane`: in all wavefronts, in those before this one
#pragma unroll
            for (int i = 0; i < kSmallWaves; ++i) c[i] = S.cnt[i][lane];
#pragma unroll
            for (int i = 0; i < kSmallWaves; ++i) {
                if ((uint32_t)i == w) mine = all;
                all += c[i];
            }
            const uint32_t start = wave_incl_scan(all) - all + mine;
            const uint32_t at = __shfl(start, (int)d, kWave) + rank;
            if (on) {
                out.key[at] = my;
                out.pos[at] = pos;
            }
        }
        __syncthreads();
        my = out.key[tid];
        pos = out.pos[tid];
    }
    // ---- out: the elements that are the range's
    const uint32_t* const sorted = S.buf[passes & 1].key;
    const uint32_t o = whole ? r0 - before0 : 0u;
    bool head = false, lng = false;
    if (tid >= o && tid < o + cnt) {
        // (where the range is not a part of all there is: the elements of the lower border's key before it, and the length of the run
        // of the upper one's that goes on behind it)
        head = tid == 0u ? whole || a_lo == 0u : my != sorted[tid - 1u];
        if (head && base + my < R)
            lng = tid + long_min < m ? sorted[tid + long_min] == my : !whole && my == top && r0 + tid + long_min < before1 + count1;
        uint32_t val = pos;
        if (!a.iota) {   // the last bag of the table that starts at or before the position
            uint32_t lo = 0, hi = bag_steps;   // S.off[lo] <= pos (or lo == 0), S.off[hi] > pos (or the end)
            while (hi - lo > 1u) {
                const uint32_t mid = (lo + hi) >> 1;
                if (S.off[mid] <= pos) lo = mid;
                else hi = mid;
            }
            uint32_t b0 = lo << bag_log2, b1 = umin(b0 + (1u << bag_log2), (uint32_t)a.B);
            while (b1 - b0 > 1u) {
                const uint32_t mid = (b0 + b1) >> 1;
                if ((int64_t)offsets[mid] <= (int64_t)pos) b0 = mid;
                else b1 = mid;
            }
            val = ds.seg * (uint32_t)a.B + b0;
        }
        a.keys_out[ds.s + tid - o] = base + my >= R ? a.invalid_key : (uint32_t)(rb + base + my);
        a.vals_out[ds.s + tid - o] = val;
    }
    const uint32_t found = (uint32_t)__popcll(__ballot(head)) | (uint32_t)__popcll(__ballot(lng)) << 16;
    if (lane == 0 && found != 0u) atomicAdd(&S.total, found);
    __syncthreads();
    // (ids outside their table have one key: where a segment that holds nothing else follows one that ends in them, its first
    // element is no head after all)
    const uint32_t starts = r0 == 0u && base + sorted[o] >= R ? kRangeStartsInvalid : 0u;
    const uint32_t ends = base + sorted[o + cnt - 1u] >= R ? kRangeEndsInvalid : 0u;
    if (tid == 0) counts[chunk] = make_uint2((S.total & 0xFFFFu) | starts | ends, S.total >> 16);
}

// One workgroup per range: unique_rows, seg_start and long rows, behind those of the ranges before it.
constexpr int kSmallRleThreads = kSmallChunk / kRleItems;
__global__ __launch_bounds__(kSmallRleThreads) void rle_small_kernel(const RleArgs a, const ChunkDesc* __restrict__ desc) {
    constexpr int kW = kSmallRleThreads / kWave;
    __shared__ uint32_t s_run[kRleItems * kW + 1];
    __shared__ uint2 s_sum[kW];
    const uint32_t c = blockIdx.x;
    const ChunkDesc ds = desc[c];
    if (ds.e <= ds.s) return;
    uint32_t bb = 0, bl = 0;
    for (uint32_t i = threadIdx.x; i < c; i += kSmallRleThreads) {
        const uint2 v = a.counts[i], p = a.counts[i > 0u ? i - 1u : 0u];
        const bool joined = i > 0u && (v.x & kRangeStartsInvalid) != 0u && (p.x & kRangeEndsInvalid) != 0u;
        bb += (v.x & ~(kRangeStartsInvalid | kRangeEndsInvalid)) - (joined ? 1u : 0u);
        bl += v.y;
    }
    uint32_t cur[kRleItems];
    bool head[kRleItems], lng[kRleItems];
    head_flags<kSmallRleThreads>(a, ds.s, ds.e, cur, head, lng);
    bb = wave_incl_scan(bb);
    bl = wave_incl_scan(bl);
    if (lane_id() == kWave - 1) s_sum[threadIdx.x >> 6] = make_uint2(bb, bl);
    __syncthreads();
    bb = bl = 0;
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        bb += s_sum[i].x;
        bl += s_sum[i].y;
    }
    const uint2 tot = rle_write_tile<kSmallRleThreads>(a, ds.s, bb, bl, cur, head, lng, s_run);
    if ((int64_t)ds.e == a.N && threadIdx.x == 0) rle_finish(a, bb + tot.x, bl + tot.y);
}

hipError_t launch_sort_small(const tbe_handle* h, const SortArgs& a, const RleArgs& r, int idx32, hipStream_t s) {
    const unsigned grid = ((unsigned)a.max_chunks + 7u) & ~7u;
    const int64_t held = a.N < kSmallHeld ? a.N : (int64_t)kSmallHeld;
    const size_t lds = 4 * (size_t)((held + kSmallThreads - 1) / kSmallThreads * kSmallThreads);
    {
        LaunchTimer tm(h, s, "sort_small");
        if (idx32) sort_small_kernel<int32_t><<<grid, kSmallThreads, lds, s>>>(a, r.counts, r.long_min);
        else sort_small_kernel<int64_t><<<grid, kSmallThreads, lds, s>>>(a, r.counts, r.long_min);
        tm.done();
    }
    LaunchTimer tm(h, s, "rle_write");
    rle_small_kernel<<<(unsigned)a.max_chunks, kSmallRleThreads, 0, s>>>(r, a.desc);
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
