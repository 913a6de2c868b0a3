// Small batches: ids to sorted (key, payload) pairs in one launch, and the counts that the run lengths need with it.
//
// Passes over digits are a chain of launches, two each, that a small batch cannot fill.  Here a workgroup owns a range of at most
// kSmallChunk places of one segment's SORTED order and finds the elements that belong there by itself, from the segment's ids
// alone, so that nothing has to be exchanged between workgroups:
//   1. the segment's keys are made from its ids, once, and kept: 31 per thread in LDS, the others in registers;
//   2. a radix selection, histograms of digits of up to ten bits from the top, finds the keys at the range's first and last place:
//      their first digits, unless more elements than there are threads share those or lie between, then as many more as it takes;
//   3. the elements from the one to the other become bits of masks, and the masks' bits positions, in order;
//   4. a stable radix sort in LDS on what distinguishes them, up to six bits a pass, one element per thread;
//   5. the payload (a binary search for the position's bag, most steps in LDS), and the range's heads and long rows counted.
// What workgroups repeat is the reading of the segment and steps 2 and 3 on it.  It is the same for any distribution of the ids
// over the segments and over the rows: a range has its places, whether they hold as many rows or one.
//
// Bound: latency, a chain of about ten barriers, and in long segments the instructions and LDS additions spent on the whole of them.  So
// a wavefront per border scans the histograms and every wavefront the counts; loops are kept rolled, for instructions come from memory
// too (keys in registers with these steps unrolled over them 23 us where rolled loops took 11.6; registers are read by number instead);
// and no step branches on an element.  One table, 10240 uniform ids of 100000 rows, us: find the range 1.2, keys and first histogram 2.3,
// borders 0.6, masks 0.4, positions 0.9, sort 2.5, bags and output 1.2.  In ranges of 1024 places 14.6.
// Against passes over digits, prepare call with run lengths and lists, us: one table, 2000 / 10240 / 12288 uniform ids of 100000 rows 27
// 31 32 / 16 18 18, of Zipf 1.3 30 36 36 / 19 25 26; 10 tables x 4662 30 / 17.5, 26 x 2307 34 / 18.5, 200 x 300 32 / 26, 512 x 128 34.5 /
// 36.  With nearly all ids in one of several tables of 100000 rows, uniform, Zipf 1.1, Zipf 1.3, of 3 rows, of one row: 32000 ids 41 48 50
// 47 59 / 19 32 37 33 46, 48000 ids 36 47 50 47 65 / 24 41 48 44 61, 65536 ids 39 50 55 52 74 / 28 49 57 54 76.  (Where keys beyond 32768
// were made from the ids again in every step, and the lanes of one row added to one LDS word one after the other: 65000 ids 45 79 89 107
// 154.)  The sort alone is then 30 us of 48000 ids: first histogram 7.5, second 6 to 9, masks 4.5.
#include <type_traits>

#include "tbe_sort.h"

namespace tbe {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSelBits = 10, kSelBins = 1 << kSelBits;   // 16 bins per lane in a wavefront's scan
constexpr int kSelPitch = kSelBins + 4;                  // of the copies of a histogram: one bin's lie in different banks
constexpr int kSmallHeld = 31 * kSmallThreads;           // keys in LDS at most
constexpr int kSmallRows = 32;                           // rows of 64 further ones in registers of a wavefront, and one more
constexpr int kBagSteps = 2048;                          // offsets of a table in LDS: all, or every 2nd, 4th, ...
static_assert(kSmallChunk <= kSmallThreads && kSelBins == 16 * kWave, "an element per thread, 16 bins per lane");
static_assert(kSmallHeld / kSmallThreads % 2 == 1 && kSmallHeld / kSmallThreads < 32, "a thread's kept elements in 32 bits");
static_assert(kSmallMax <= kSmallMaxMany && kSmallMaxMany <= kSmallHeld + (kSmallRows + 1) * kSmallThreads, "a batch may be one segment's");
constexpr uint32_t kNoKey = 0xFFFFFFFFu;                 // (keys are below 2^31)
// in a range's counts: it starts a segment with an id outside its table, or ends in one
constexpr uint32_t kRangeStartsInvalid = 0x80000000u, kRangeEndsInvalid = 0x40000000u;

struct SmallLds {
    union {
        __align__(16) uint32_t hist[4][kSelPitch];   // copies that the lanes are spread over; of two borders two each
        struct { uint32_t key[kSmallThreads], pos[kSmallThreads]; } buf[2];
    };
    uint32_t cnt[kSmallWaves][kWave];
    uint32_t off[kBagSteps];
    uint4 place[2];
    uint32_t borders[2 * kSmallWaves], taken[2 * kSmallWaves], none[kWave];
    uint32_t scan[kSmallWaves], total;
    ChunkDesc desc;
};

struct Place { uint32_t bin, before, count; };   // a bin, the elements in bins below, and in it
// The bin of element number x (x below their sum) of a histogram's copies added up.  By one wavefront.
template <int COPIES>
__device__ __forceinline__ Place find_place(const uint32_t* h, const uint32_t x) {
    const int lane = lane_id();
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < COPIES; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // (in an order that spreads the lanes over the banks)
            const uint4 v = *reinterpret_cast<const uint4*>(h + q * kSelPitch + 16 * lane + 4 * ((j + lane) & 3));
            sum += v.x + v.y + v.z + v.w;
        }
    const uint32_t incl = wave_incl_scan(sum);
    const int f = __ffsll((unsigned long long)__ballot(incl > x)) - 1;
    const uint32_t below = bcast_lane(incl - sum, f);
    const int bin = 16 * f + (lane & 15);
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < COPIES; ++q) c += h[q * kSelPitch + bin];
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

// E digits per lane into a histogram.  Lanes that all hold the same one, as where a segment's upper digits agree, would queue on one LDS
// word: then one of them adds their number.  (Looked for only where the first digits agree.)
template <uint32_t E>
__device__ __forceinline__ void add_digits(uint32_t* const h, const uint32_t (&d)[E]) {
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d[0]);
    if (__ballot(d[0] != d0) == 0ull) {
        uint32_t other = 0;
#pragma unroll
        for (uint32_t u = 1; u < E; ++u) other |= d[u] ^ d0;
        if (__ballot(other != 0u) == 0ull) {
            if (lane_id() == 0) atomicAdd(&h[d0], E * (uint32_t)kWave);
            return;
        }
    }
#pragma unroll
    for (uint32_t u = 0; u < E; ++u) atomicAdd(&h[d[u]], 1u);
}

// the set bits of m but the lowest q
__device__ __forceinline__ uint64_t without_lowest(uint64_t m, const uint32_t q) {
    if (q >= (uint32_t)__popcll(m)) return 0ull;
    for (uint32_t i = 0; i < q; ++i) m &= m - 1ull;
    return m;
}

// m = 2 m + (x <= y), m = 2 m + (x == y): a comparison and an addition with its carry
__device__ __forceinline__ void push_le(uint32_t& m, const uint32_t x, const uint32_t y) {
    asm("v_cmp_ge_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(m) : "v"(x), "s"(y) : "vcc");
}
__device__ __forceinline__ void push_eq(uint32_t& m, const uint32_t x, const uint32_t y) {
    asm("v_cmp_eq_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(m) : "v"(x), "s"(y) : "vcc");
}

// held: keys that LDS has room for, an odd number of rounds of the workgroup
template <typename IT>
__global__ __launch_bounds__(kSmallThreads) void sort_small_kernel(const SortArgs a, uint2* __restrict__ counts, const uint32_t long_min,
                                                                   const uint32_t held) {
    __shared__ SmallLds S;
    extern __shared__ __align__(16) uint32_t s_keys[];
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
    // (256 threads per copy, a uint4 each)
    auto clear_hist = [&] { *reinterpret_cast<uint4*>(&S.hist[tid >> 8][4u * (tid & 255u)]) = make_uint4(0u, 0u, 0u, 0u); };
    clear_hist();
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
    // ---- the segment's elements.  The keys of the first `kept` stay in LDS, `per` that follow one another of each thread (an odd number,
    // which spreads the lanes over the banks; from n on they are kNoKey).  Those behind stay in registers, in rows of 64, at most
    // row_per to a wavefront.
    const uint32_t n = ds.seg_end - ds.seg_start;
    const uint32_t kept = umin(n, held), per = umin((n + kSmallThreads - 1u) / kSmallThreads | 1u, held / kSmallThreads);
    const uint32_t rows = (n - kept + kWave - 1u) / kWave, row_per = (rows + kSmallWaves - 1u) / kSmallWaves;
    const uint32_t row0 = umin(w * row_per, rows), my_rows = umin(row_per, rows - row0);
    const IT* const ids = static_cast<const IT*>(a.indices) + ds.seg_start;
    auto key_of = [&](const IT id) { return (sizeof(IT) == 8 ? (uint64_t)id < (uint64_t)R : (uint32_t)id < R) ? (uint32_t)id : R; };
    typedef uint32_t rows_t __attribute__((ext_vector_type(kSmallRows)));
    rows_t row = 0u;
    uint32_t last_row = 0u;   // number kSmallRows
    // of_kept(key) for this thread's kept elements, the last one first; of_row(key, the row's number among the wavefront's)
    auto each = [&](auto of_kept, auto of_row) {
        const uint32_t* mine = s_keys + tid * per + per - 1u;
        uint32_t left = per;
#pragma unroll 1
        for (; (left & 3u) != 0u; --left) of_kept(*mine--);
#pragma unroll 1
        for (; left > 0u; left -= 4u, mine -= 4) {
            uint32_t k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) k[u] = mine[-u];
#pragma unroll
            for (int u = 0; u < 4; ++u) of_kept(k[u]);
        }
#pragma unroll 1
        for (uint32_t r = 0; r < umin(my_rows, kSmallRows); ++r) of_row(row[r], r);
        if (my_rows > (uint32_t)kSmallRows) of_row(last_row, (uint32_t)kSmallRows);
    };
    // ---- the keys at places r0 and r0 + cnt - 1 (0: the lower border, 1: the upper one), digit by digit from the top
    const uint32_t r0 = ds.s - ds.seg_start, cnt = ds.e - ds.s;
    const uint32_t bits = 32u - (uint32_t)__clz((int)R);
    const uint32_t levels = (bits + kSelBits - 1u) / kSelBits, width = (bits + levels - 1u) / levels;
    const uint32_t mask = (1u << width) - 1u;
    uint32_t low = (levels - 1u) * width;   // bits below the digit
    {
        uint32_t* const h = S.hist[lane & 3];
        bool bad = false;
        constexpr uint32_t kU = 8;   // ids in flight, and as many more while these are used
        IT id[kU];
        // f(keys, number of the first) for elements first, first + stride, ...; from n on the segment's last
        auto from_ids = [&](const uint32_t first, const uint32_t stride, const uint32_t rounds, auto f) {
            auto load = [&](const uint32_t k0) {
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u)
                    if (u < 4u || k0 + 4u < rounds) id[u] = ids[umin(first + (k0 + u) * stride, n - 1u)];
            };
            load(0u);
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < rounds; k0 += kU) {
                uint32_t k[kU];
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) k[u] = key_of(id[u]);
                if (k0 + kU < rounds) load(k0 + kU);
                f(k, k0);
            }
        };
        from_ids(tid, kSmallThreads, per, [&](uint32_t (&k)[kU], const uint32_t k0) {
            uint32_t* const to = s_keys + tid + k0 * kSmallThreads;
            if ((k0 + kU) * kSmallThreads <= kept) {   // (without a branch per element, which would take as long as the rest of it)
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) {
                    bad |= k[u] == R;
                    to[u * kSmallThreads] = k[u];
                    k[u] >>= low;
                }
                add_digits(h, k);
            } else {
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) {
                    if (k0 + u >= per) break;
                    bad |= k[u] == R;
                    const bool in = tid + (k0 + u) * kSmallThreads < n;
                    to[u * kSmallThreads] = in ? k[u] : kNoKey;
                    atomicAdd(&h[k[u] >> low], in ? 1u : 0u);
                }
            }
        });
        const uint32_t first = kept + row0 * kWave + (uint32_t)lane, most = umin(my_rows, kSmallRows);
        auto add_row = [&](const uint32_t k, const uint32_t r) {   // returns what a row holds of it
            bad |= k == R;
            const bool in = first + r * kWave < n;
            atomicAdd(&h[k >> low], in ? 1u : 0u);
            return in ? k : kNoKey;
        };
        if (most > 0u)
            from_ids(first, kWave, most, [&](const uint32_t (&k)[kU], const uint32_t r) {
#pragma unroll
                for (uint32_t u = 0; u < kU; ++u) {
                    if (r + u >= most) break;
                    row[r + u] = add_row(k[u], r + u);
                }
            });
        if (my_rows > most) last_row = add_row(key_of(ids[umin(first + kSmallRows * kWave, n - 1u)]), kSmallRows);
        if (bad) atomicOr(a.err, 1);
    }
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
        clear_hist();
        __syncthreads();
        const bool one = key0 == key1;
        uint32_t* const h = one ? S.hist[lane & 3] : S.hist[lane & 1];
        // (the upper border's histograms lie behind the lower one's; the other lanes add to a word of their own instead of branching)
        const uint32_t upper = one ? 0u : 2u * kSelPitch;
        auto add = [&](const uint32_t k) {
            const uint32_t d = k >> high;
            uint32_t* const to = &h[((k >> low) & mask) + (d == key1 ? upper : 0u)];
            atomicAdd(((d == key0) | (d == key1)) ? to : &S.none[lane], 1u);
        };
        each(add, [&](const uint32_t k, uint32_t) { add(k); });
        __syncthreads();
        if (w < 2u) {
            const uint32_t x = w == 0u ? r0 - before0 : r0 + cnt - 1u - before1;
            const Place p = one ? find_place<4>(S.hist[0], x) : find_place<2>(S.hist[2u * w], x);
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
    const uint64_t lt = lanemask_lt();
    // masks of them: of the thread's kept elements, and of a row of the wavefront's others in each lane
    uint32_t kept_sel = 0;
    uint64_t row_sel = 0;
    if (whole) {
        each([&](const uint32_t k) { push_le(kept_sel, k - base, top); },
             [&](const uint32_t k, const uint32_t r) {
                 const uint64_t m = __ballot(k - base <= top);
                 row_sel = (uint32_t)lane == r ? m : row_sel;
             });
    } else {
        uint32_t kept_a = 0, kept_b = 0;
        uint64_t row_a = 0, row_b = 0;
        if (one_key) {
            each([&](const uint32_t k) { push_eq(kept_a, k, key0); },
                 [&](const uint32_t k, const uint32_t r) {
                     const uint64_t m = __ballot(k == key0);
                     row_a = (uint32_t)lane == r ? m : row_a;
                 });
        } else {
            each([&](const uint32_t k) {
                     push_le(kept_sel, k - base, top);
                     push_eq(kept_a, k, key0);
                     push_eq(kept_b, k, key1);
                 },
                 [&](const uint32_t k, const uint32_t r) {
                     const uint64_t m = __ballot(k - base <= top), ma = __ballot(k == key0), mb = __ballot(k == key1);
                     if ((uint32_t)lane == r) {
                         row_sel = m;
                         row_a = ma;
                         row_b = mb;
                     }
                 });
        }
        // the numbers of their first elements of either key: both in one word within a wavefront, which has at most 4096 elements of a kind
        const uint32_t of_kept = (uint32_t)__popc(kept_a) | (uint32_t)__popc(kept_b) << 16;
        const uint32_t of_row = (uint32_t)__popcll(row_a) | (uint32_t)__popcll(row_b) << 16;
        const uint32_t in_kept = wave_incl_scan(of_kept), in_row = wave_incl_scan(of_row);
        if (lane == kWave - 1) {
            S.borders[w] = in_kept;
            S.borders[kSmallWaves + w] = in_row;
        }
        __syncthreads();
        const uint32_t v = lane < 2 * kSmallWaves ? S.borders[lane] : 0u, va = v & 0xFFFFu, vb = v >> 16;
        const uint32_t xa = wave_incl_scan(va) - va, xb = wave_incl_scan(vb) - vb;
        const uint32_t a_lo = r0 - before0, a_hi = a_lo + cnt, b_hi = r0 + cnt - before1;
        auto from = [](const uint32_t number, const uint32_t first) { return number > first ? number - first : 0u; };
        auto choose = [&](const uint64_t sel, const uint64_t ma, const uint64_t mb, const uint32_t before, const int wave) {
            const uint32_t x = (before & 0xFFFFu) + bcast_lane(xa, wave), y = (before >> 16) + bcast_lane(xb, wave);
            const uint64_t lower = without_lowest(ma, from(a_lo, x));
            return one_key ? lower & ~without_lowest(ma, from(a_hi, x)) : (sel & ~ma & ~mb) | lower | (mb & ~without_lowest(mb, from(b_hi, y)));
        };
        kept_sel = (uint32_t)choose(kept_sel, kept_a, kept_b, in_kept - of_kept, (int)w);
        if (row_per > 0u) row_sel = choose(row_sel, row_a, row_b, in_row - of_row, kSmallWaves + (int)w);
    }
    {   // their positions
        const uint32_t c = (uint32_t)__popc(kept_sel), in_kept = wave_incl_scan(c);
        const uint32_t cr = (uint32_t)__popcll(row_sel), in_row = wave_incl_scan(cr);
        if (lane == kWave - 1) {
            S.taken[w] = in_kept;
            S.taken[kSmallWaves + w] = in_row;
        }
        __syncthreads();
        const uint32_t v = lane < 2 * kSmallWaves ? S.taken[lane] : 0u, xs = wave_incl_scan(v) - v;
        // a lane its own, bit by bit, or where few lanes hold many, lane after lane
        auto write = [&](uint64_t sel, uint32_t at, const uint32_t p0, const uint32_t count) {
            uint64_t any = __ballot(sel != 0ull);
            if (wave_max_i32((int)count) <= __popcll(any)) {
                while (sel != 0ull) {
                    S.buf[0].pos[at++] = p0 + (uint32_t)__ffsll((unsigned long long)sel) - 1u;
                    sel &= sel - 1ull;
                }
            } else {
                for (; any != 0ull; any &= any - 1ull) {
                    const int r = __ffsll((unsigned long long)any) - 1;
                    const uint64_t m = (uint64_t)lane_i64((int64_t)sel, r);
                    const uint32_t first = bcast_lane(at, r), pr = bcast_lane(p0, r);
                    if (m >> lane & 1ull) S.buf[0].pos[first + (uint32_t)__popcll(m & lt)] = pr + (uint32_t)lane;
                }
            }
        };
        write(kept_sel, bcast_lane(xs, (int)w) + in_kept - c, ds.seg_start + tid * per, c);
        if (row_per > 0u) write(row_sel, bcast_lane(xs, kSmallWaves + (int)w) + in_row - cr, ds.seg_start + kept + (row0 + (uint32_t)lane) * kWave, cr);
    }
    __syncthreads();
    // ---- sorted by what the keys differ in, stably; one element per thread, a digit's counts per wavefront
    const uint32_t m = whole ? between : cnt;
    const bool on = tid < m;
    uint32_t my = 0, pos = 0;
    if (on) {
        pos = S.buf[0].pos[tid];
        const uint32_t p = pos - ds.seg_start;
        my = (p < held ? s_keys[p] : key_of(ids[p])) - base;
    }
    S.buf[0].key[tid] = my;   // (where all are of one key, this is what is read below)
    const int diff = top == 0u ? 0 : 32 - __clz((int)top);
    const int passes = (diff + 5) / 6, db = passes == 0 ? 0 : (diff + passes - 1) / passes;
    if (passes == 0) __syncthreads();
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
        head = tid == 0u ? whole || r0 == before0 : my != sorted[tid - 1u];
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
    const int64_t rounds = ((a.N + kSmallThreads - 1) / kSmallThreads) | 1;
    const int64_t held = rounds * kSmallThreads < kSmallHeld ? rounds * kSmallThreads : kSmallHeld;
    const size_t lds = 4 * (size_t)held;
    {
        LaunchTimer tm(h, s, "sort_small");
        if (idx32) sort_small_kernel<int32_t><<<grid, kSmallThreads, lds, s>>>(a, r.counts, r.long_min, (uint32_t)held);
        else sort_small_kernel<int64_t><<<grid, kSmallThreads, lds, s>>>(a, r.counts, r.long_min, (uint32_t)held);
        tm.done();
    }
    LaunchTimer tm(h, s, "rle_write");
    rle_small_kernel<<<(unsigned)a.max_chunks, kSmallRleThreads, 0, s>>>(r, a.desc);
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
