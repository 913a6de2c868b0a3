// C ABI of libtbe355: argument checks, table metadata, workspace carving, stream plumbing, timing.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>

#include "tbe_rows.h"

namespace tbe {

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Batches up to kSelfScanMax lookups: the histograms of a segment's chunks are few enough for every scatter workgroup to
// add up itself (at most 512 chunks of 4096 in all).  What that reads grows with the square of the chunks per segment and
// with the digit's width, so small tiles (more workgroups) and digits of more than 8 bits (fewer passes) are for batches
// with at most kSelfScanChunks chunks per segment.  Measured: 26 tables of 45 k lookups, 20-bit ids, two 10-bit passes on
// 22 chunks per segment 50 us against 59 us for three 8-bit ones; 12 tables of 164 k lookups, 80 chunks per segment: 108
// against 75 us.
constexpr int64_t kSelfScanMax = (int64_t)1 << 21;
constexpr int64_t kSelfScanChunks = 32;
// Bytes of chunk histograms that wide digits may take, ascending in N, so that a workspace made for more lookups serves
// fewer as well.
static size_t hist_cap(int64_t N, int nseg) {
    const size_t c = (size_t)(N < kSelfScanMax ? N : kSelfScanMax) * 5 / 4;
    const size_t few = std::min((size_t)512 << 10, (size_t)4096 * ((size_t)N / 1024 + (size_t)nseg + 2));   // 2048 bins, tiles of 1024
    return c > few ? c : few;
}
// ... by passes over digits
static SortShape pass_shape(const tbe_handle* h, int64_t N) {
    SortShape sh;
    sh.nseg = h->segmented ? h->T : 1;
    sh.small = false;
    sh.self_scan = N <= kSelfScanMax;
    const int64_t few = kSelfScanChunks * sh.nseg;   // chunks in all
    if (sh.self_scan && N <= 32 * 4096 && N <= few * 1024) sh.tile = 1024;
    else if (sh.self_scan && N <= 4 * few * 2048) sh.tile = 2048;
    else sh.tile = kRadixTile;
    const int64_t tile = sh.tile;
    const int64_t tiles = (N + tile - 1) / tile;
    const int64_t blocks = tiles < kRadixMaxBlocks ? tiles : kRadixMaxBlocks;
    sh.chunk = (tiles + blocks - 1) / blocks * tile;
    sh.max_chunks = (int)((N + sh.chunk - 1) / sh.chunk) + sh.nseg;
    // few passes of wide digits where the batch is small enough for them and their histograms stay within hist_cap
    for (int wide = sh.self_scan && tiles <= few ? 1 : 0; wide >= 0; --wide) {
        const int most = wide ? 11 : 8;
        sh.passes = (h->sort_bits + most - 1) / most;
        sh.bits = (h->sort_bits + sh.passes - 1) / sh.passes;
        sh.bins = sh.bits <= 8 ? 256 : (sh.bits <= 10 ? 1024 : 2048);
        sh.hist_bytes = (size_t)(sh.self_scan ? 2 : 4) * (size_t)sh.bins * (size_t)(sh.max_chunks + 1);
        if (sh.hist_bytes <= hist_cap(N, sh.nseg)) break;
    }
    return sh;
}
SortShape sort_shape(const tbe_handle* h, int64_t N) {
    SortShape sh = pass_shape(h, N);
    // One launch where keys are local to their segment and reading a segment once per range of it costs less than two launches a
    // pass.  That grows with the longest segment, of which the host knows only that all of them together are N: hence the bound on N for
    // the batch that is one table's after all, and on the average, beyond which most batches have such a table.  Prepare calls with nearly
    // all ids in one of 26 tables, passes / one launch, us: 48000 ids 36 to 65 / 24 to 61, 65536 ids of 100000 rows 39 to 74 / 28 to 76,
    // and of tables of at most 2000 rows, which take one pass of wide digits, 30 to 44 / 33 to 52, where spread over the tables 23 to 28 /
    // 17 to 22.
    // A compute unit has room for one of its workgroups, and a round of 256 of them costs about as much as a pass.  A round more than
    // passes is slower, whatever the ids: 236 tables x 161 ids of 60 / 1000 / 100000 rows (1 / 2 / 3 passes, two rounds) 22 30 38 / 24 25
    // 26, 500 tables x 15 (three rounds) 22 30 38 / 32 33 34, 300 tables x 7 (two) 20 28 36 / 23 23 25, 150 x 400 (two) of 60, 3000 rows 25
    // 33 / 27 28.  As many rounds as passes, but more than one, lose more with long segments than they gain without: three quarters of
    // 38000 and of 60000 ids in one of 250 tables 32 39 47, 36 44 52 / 44 42 45, 54 53 58, of 13000 28 35 43 / 30 30 31.
    const int64_t ranges = (N + kSmallChunk - 1) / kSmallChunk + sh.nseg, rounds = (ranges + 255) / 256;
    if ((h->segmented || h->T == 1) && sh.nseg <= kSmallTables && rounds <= (rounds > 1 && N > 2 * kSmallMax ? sh.passes - 1 : sh.passes) &&
        (N <= kSmallMax || (N <= kSmallMaxMany && N <= kSmallSegment * sh.nseg))) {
        sh.small = true;
        sh.passes = 1;
        sh.bits = h->sort_bits;
        sh.bins = 0;
        sh.hist_bytes = 0;
        sh.self_scan = true;
        sh.chunk = sh.tile = kSmallChunk;
        sh.max_chunks = (int)ranges;
    }
    return sh;
}

// At least sort_shape(h, n).max_chunks for every n <= N: tiles of 1024 end at 128 K lookups and tiles of 2048 at
// kSelfScanMax, so a batch above such a border may have fewer chunks than one below it.
static size_t most_chunks(const tbe_handle* h, int64_t N) {
    const int64_t small = std::min(N, (int64_t)32 * 4096) / 1024, middle = std::min(N, kSelfScanMax) / 2048;
    const int64_t large = std::min(N / kRadixTile, (int64_t)kRadixMaxBlocks);
    return (size_t)(std::max(std::max(small, middle), large) + 1 + (h->segmented ? h->T : 1));
}

// A row with more than so many lookups is long, i.e. shared out to several wavefronts in parts.  A wavefront
// walks 512 lookups of a wide row in about 60 us, so small batches, whose row updates take less than that, cut finer; the
// borders follow from the memory of the partial sums (at most n / part + n / min slots): never more than n / 48 plus a constant.
// The smallest batches are a matter of the longest chain of loads.  Where rows take a wavefront each they cut finer still, as long as
// few lookups of a table keep the one workgroup that lists its long rows from becoming that chain.  Parts of 64 / 32 / 16, backward us:
// ten tables x 777 bags of 6 ids, 8 to 1024 columns 70 / 59 / 59; 10 tables x 1200 lookups of 64, 256, 1024 columns 33.5 33.4 49.9 / 33.1
// 32.5 46.7 / 32.4 31.9 42.6; one table x 12000 42.3 44.4 63.8 / 44.0 44.1 57.9 / 47.3 47.0 62.0; x 24000 53 55 93 / 57 58 94 / 63 62 96.
// But a batch that has any long row pays for it: its list 3 to 4 us, the parts 1.6, their sums 2 to 4.  So with fewer than 512 lookups per
// table, where a row has hardly more than a wavefront walks in that time, rows of up to 64 stay whole.  Against parts of 64, rows of 17
// and more cut / this: 59 tables x 33 lookups, 1024 columns 29.7 -> 40.6 / 30.0, 2 x 85 27 -> 37 / 27, 9 x 286 of 512 columns 35 -> 45 /
// 35.6; the mean over 1394 random batches of up to 65536 lookups, tables of 129 to 1024 columns, is 5 % faster with either, 63 / 11 of
// them more than 3 % slower than with the passes and parts that a batch of any size can have.
struct PartSteps {
    int64_t top[8];             // batches of at most so many lookups
    uint32_t min[8], part[8];   // ... cut rows of more than `min` of them into parts of `part`
    int of(const int64_t N) const {
        int i = 0;
        while (N > top[i]) ++i;
        return i;
    }
    // the most long rows, and slots for partial sums, that a batch of N lookups or fewer has: ascending in N
    int64_t most(const int64_t N, const bool slots) const {
        int64_t m = 0;
        for (const int64_t t : top) {
            const int64_t n = std::min(t, N), i = of(n);
            m = std::max(m, n / (int64_t)min[i] + (slots ? n / (int64_t)part[i] : 0) + 1);
        }
        return m;
    }
};
static PartSteps part_steps(const tbe_handle* h, const bool fine) {
    const int64_t D = fine ? h->maxD : 0, T = h->T, least = (int64_t)1 << 15, less = (int64_t)1 << 16;
    return {{D > 256 ? std::min(least, 512 * T) : 0, D > 256 ? std::min(least, 4096 * T) : 0, D > 128 ? std::min(less, 512 * T) : 0,
             D > 128 ? std::min(less, 8192 * T) : 0, (int64_t)1 << 17, (int64_t)3 << 17, (int64_t)3 << 19, INT64_MAX},
            {64, 16, 64, 32, 64, 128, 256, 512},
            {16, 16, 32, 32, 64, 128, 256, 512}};
}

// What the dense rows may make of a workspace.  A dense row leaves one partial sum per chunk of bags, so their area grows with
// the columns of all tables whose gradient block is large, not with the lookups: a batch of few lookups per bag would pay
// several times its other memory for it (32 tables of 128 columns, 16384 bags of one id: 20 + 58 MB).  So the layout with
// dense rows takes at most 20 bytes per lookup (the five streams once more) and 16 MiB over 20.5 bytes per lookup and n / 192 +
// 4096 + 512 T partial sums of the widest row, and a batch that would fit the library's own scratch array by the latter does
// so with dense rows as well; within that as many chunks as are useful.  Fewer chunks cost time only below about 512 workgroups
// (measured: 64 tables, 4096 bags, 16 / 8 / 4 chunks 63 / 58 / 90 us; 12 tables, 8192 bags, 32 / 16 / 8 chunks 21 / 29 / 50 us),
// which is what small batches have: the 16 MiB, next to nothing of this memory, let 2 tables x 5399 bags x 256 columns (86 k
// lookups) share their 22 blocks of bags out to 22 workgroups a table rather than 11, 33 -> 19 us, and 12 tables x 6478 bags
// (909 k lookups) to 26 rather than 13, 35 -> 25 us.
static size_t dense_allowance(const tbe_handle* h, size_t n) {
    const size_t lean = 41 * n / 2 + 4 * (n / 192 + 4096 + 512 * (size_t)h->T) * (size_t)h->maxD;
    const size_t full = lean + 20 * n + ((size_t)16 << 20);
    return lean <= (size_t)TBE_STATIC_SCRATCH_BYTES ? std::min(full, (size_t)TBE_STATIC_SCRATCH_BYTES) : full;
}

// Memory is used twice where lifetimes allow it: what the sort alone needs lies where the run lengths then write seg_start;
// the sort's spare key buffer and the run-length counts lie where the partial sums of a step go.
static Workspace lay_out(const tbe_handle* h, int32_t B, int64_t N, const PartSteps& steps) {
    Workspace w;
    memset(&w, 0, sizeof(w));
    const size_t n = (size_t)(N > 0 ? N : 1);
    w.n = N;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align256(off + bytes);
        return at;
    };
    w.sort = sort_shape(h, (int64_t)n);
    const int sorted = w.sort.passes & 1;   // every pass flips the double buffer, starting from 0
    w.keys[sorted] = take(4 * (n + 1));
    w.vals[0] = take(4 * (n + 1));
    w.vals[1] = take(4 * (n + 1));
    {   // seg_start; until the run lengths write it, what the sort needs only while it runs, at its end: few batches have so
        // many unique rows that they get there (lines that other dies have just written cost 0.6 of rle_write's 8.2 us)
        const size_t at = off;
        // (8-bit digits in a handle of many tables may exceed the cap; their histograms grow with N by themselves)
        const size_t chunks = most_chunks(h, (int64_t)n);
        const size_t hist8 = (size_t)(w.sort.self_scan ? 2 : 4) * 256 * (chunks + 1);
        w.radix_hist = take(std::max(std::max(w.sort.hist_bytes, hist_cap((int64_t)n, w.sort.nseg)), hist8));
        w.nchunks = take(w.sort.self_scan ? 0 : 4);
        w.chunk_desc = take(32 * chunks);
        const size_t need = off - at;
        off = at;
        w.seg_start = take(std::max(4 * (n + 1), need));
        const size_t shift = off - at - need;
        w.radix_hist += shift;
        w.nchunks += shift;
        w.chunk_desc += shift;
    }
    w.counters = take(4 * kCounterWords);
    w.long_min = steps.min[steps.of((int64_t)n)];
    w.part = steps.part[steps.of((int64_t)n)];
    w.cap_long = steps.most((int64_t)n, false);    // at most n / (long_min + 1) rows are long
    w.cap_main = steps.most((int64_t)n, true) + 1; // ceil(len / part) slots for each of them
    w.long_rows = take(8 * (size_t)w.cap_long);
    w.long_list = take(16 * (size_t)w.cap_long);
    w.unit_list = take(8 * (size_t)w.cap_main);
    const bool hint = h->T <= kMaxSortSegments;
    w.hot_ids = take(hint ? 4 * (size_t)kHotRows * (size_t)h->T : 0);
    w.hot_n = take(hint ? 4 * (size_t)h->T : 0);
    w.seq_gbase = take(8 * (size_t)h->T);
    const size_t parts = 4 * (size_t)w.cap_main * (size_t)h->maxD;
    w.rle_blocks = (int)(((int64_t)n + kRleTile - 1) / kRleTile);
    // spare keys and run-length counts; or the ranges of a small batch and their counts
    const size_t ranges = (std::min(n, (size_t)kSmallMaxMany) + kSmallChunk - 1) / kSmallChunk + (size_t)w.sort.nseg;
    const size_t front = std::max(align256(4 * (n + 1)) + align256(8 * (size_t)w.rle_blocks), align256(32 * ranges) + align256(8 * ranges));
    const size_t base = off + std::max(front, align256(parts));
    size_t reserve = base;
    // Dense rows: for the tables whose gradient block is large.  Enough chunks for about a thousand workgroups in all, at most
    // 32, as far as the allowance goes.
    uint32_t tables = 0;
    uint64_t columns = 0;
    if (h->T <= kMaxSortSegments)
        for (const int32_t D : h->D)
            if (dense_block((uint32_t)B, (uint32_t)D)) {
                ++tables;
                columns += (uint64_t)D;
            }
    if (tables > 0) {
        const uint32_t blocks = ((uint32_t)B + kDenseBags - 1) / kDenseBags;
        const uint32_t useful = std::min(blocks, h->T >= 1024 ? 1u : (h->T <= 32 ? 32u : 1024u / (uint32_t)h->T));
        const size_t per_chunk = 4 * (size_t)kDenseRows * (size_t)columns;
        const size_t lists = off;
        w.dense_n = take(4 * (size_t)h->T);
        w.dense_tab = take(8 * (size_t)h->T);
        w.dense_rows = take(4 * (size_t)h->T * kDenseRows);
        w.dense_index = take(4 * (size_t)tables * kDenseRows * (blocks + 1));
        const size_t allowed = dense_allowance(h, n);
        uint32_t chunks = 0;
        if (off + std::max(front, parts) + 256 <= allowed) chunks = (uint32_t)std::min((size_t)useful, (allowed - 256 - off - parts) / per_chunk);
        reserve = std::max(base, std::min(off + std::max(front, align256(parts + per_chunk * useful)), allowed));
        w.dense = chunks > 0;
        if (w.dense) {
            w.dense_blocks = blocks;
            w.dense_per_chunk = (blocks + chunks - 1) / chunks;
            w.dense_chunks = (blocks + w.dense_per_chunk - 1) / w.dense_per_chunk;
        } else {
            off = lists;
        }
    }
    const size_t shared = off;
    if (w.sort.small) {
        w.chunk_desc = take(32 * ranges);
        w.rle_counts = take(8 * ranges);
    } else {
        w.keys[sorted ^ 1] = take(4 * (n + 1));
        w.rle_counts = take(8 * (size_t)w.rle_blocks);
    }
    w.partial = shared;
    w.dense_partial = shared + parts;   // (a multiple of 16)
    w.total = reserve;   // (covers both uses: at least base, and with dense rows no less than what they were fitted into)
    return w;
}

// The total never shrinks when B or N grows: a workspace made for a batch serves every smaller one.  The finer parts of small batches
// take up to four times the memory for partial sums, so they are taken only where that neither leaves less to the dense rows nor costs
// the batch its place in the library's own scratch array (30 tables x 912 columns, 1024 bags, 28247 lookups: 69.7 MB with parts of 16,
// 60.0 with 64).
Workspace carve(const tbe_handle* h, int32_t B, int64_t N) {
    Workspace w = lay_out(h, B, N, part_steps(h, true));
    const PartSteps coarse = part_steps(h, false);
    if (w.cap_main == coarse.most(N > 0 ? N : 1, true) + 1) return w;
    Workspace c = lay_out(h, B, N, coarse);
    // (of all sizes up to this one: what the finer parts take, up to the array's end as long as the coarser ones fit into it)
    const size_t total = c.total <= (size_t)TBE_STATIC_SCRATCH_BYTES ? std::min(w.total, (size_t)TBE_STATIC_SCRATCH_BYTES) : w.total;
    const bool dense = N >= 2 * (int64_t)B;   // (no table has dense rows of fewer lookups)
    if (w.total > total || w.part == c.part || (dense && w.dense_chunks < c.dense_chunks)) w = c;
    w.total = total;
    return w;
}

LaunchTimer::LaunchTimer(const tbe_handle* h_, hipStream_t s_, const char* name) : h(const_cast<tbe_handle*>(h_)), s(s_) {
    if (!h->timing) return;
    if (h->n_used == (int)h->slots.size()) {
        TimingSlot t;
        t.name = name;
        if (hipEventCreate(&t.beg) != hipSuccess || hipEventCreate(&t.end) != hipSuccess) return;
        h->slots.push_back(t);
    }
    slot = h->n_used++;
    h->slots[slot].name = name;
    (void)hipEventRecord(h->slots[slot].beg, s);
}

void LaunchTimer::done() {
    if (slot >= 0) (void)hipEventRecord(h->slots[slot].end, s);
}

// ---- scratch memory for the entry point that allocates nothing ------------------------------------------------------
// A fixed array in the library's device image, one copy per GPU at that GPU's own address.  In host code the array's
// name is only a handle for the runtime: its device address is looked up once per device, with that device current,
// and kept; kernels, copies and fills always get that address, never the name.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[TBE_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on device i, once looked up

// address of `scratch` on the CURRENT device (which is `device`), or nullptr if the runtime cannot give it
static void* static_scratch_address(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[device] = ptr;
    }
    return g_scratch_ptr[device];
}

static int bits_for(uint64_t v) {  // number of bits needed to represent v (>= 1)
    int b = 1;
    while ((v >> b) != 0) ++b;
    return b;
}

}  // namespace tbe

using namespace tbe;

extern "C" {

#ifndef TBE_SOURCE_DIGEST
#define TBE_SOURCE_DIGEST "unknown"
#endif
const char* tbe_build_info(void) { return "tbe355 gfx950 " TBE_SOURCE_DIGEST; }

const char* tbe_status_string(tbe_status s) {
    switch (s) {
        case TBE_OK: return "ok";
        case TBE_EINVAL: return "invalid argument";
        case TBE_ESHAPE: return "size outside the supported limits";
        case TBE_EDTYPE: return "unknown dtype or pooling mode";
        case TBE_EWORKSPACE: return "workspace too small";
        case TBE_EINDEX: return "an id outside its table was seen";
        case TBE_EHIP: return "HIP runtime error";
    }
    return "unknown status";
}

tbe_status tbe_create(int32_t T, const int64_t* rows, const int32_t* D, tbe_dtype weight_dtype, tbe_handle** out) {
    if (!out) return TBE_EINVAL;
    *out = nullptr;
    if (!rows || !D) return TBE_EINVAL;
    if (weight_dtype != TBE_F32 && weight_dtype != TBE_F16) return TBE_EDTYPE;
    if (T < 1 || T > (1 << 20)) return TBE_ESHAPE;
    const int dmul = weight_dtype == TBE_F16 ? 8 : 4;
    tbe_handle* h = new (std::nothrow) tbe_handle;
    if (!h) return TBE_EHIP;
    h->T = T;
    h->dtype = weight_dtype;
    h->rows.assign(rows, rows + T);
    h->D.assign(D, D + T);
    h->row_base.assign(T + 1, 0);
    h->w_off.assign(T + 1, 0);
    h->D_off.assign(T + 1, 0);
    int64_t sumD = 0;
    for (int t = 0; t < T; ++t) {
        if (rows[t] < 1 || rows[t] >= ((int64_t)1 << 31) || D[t] < 4 || D[t] > 1024 || D[t] % dmul != 0) {
            delete h;
            return TBE_ESHAPE;
        }
        h->row_base[t + 1] = h->row_base[t] + rows[t];
        h->w_off[t + 1] = h->w_off[t] + rows[t] * (int64_t)D[t];
        sumD += D[t];
        h->D_off[t + 1] = (int32_t)sumD;
        if (D[t] > h->maxD) h->maxD = D[t];
        if (t == 0 || D[t] < h->minD) h->minD = D[t];
        if (h->row_base[t + 1] >= (int64_t)0xFFFFFFFFll || sumD > (int64_t)0x7FFFFFF0ll) {
            delete h;
            return TBE_ESHAPE;
        }
    }
    h->total_rows = h->row_base[T];
    h->total_elems = h->w_off[T];
    h->sumD = (int32_t)sumD;
    h->key_bits = bits_for((uint64_t)h->total_rows);
    {
        int64_t max_rows = 0;
        for (int t = 0; t < T; ++t) max_rows = rows[t] > max_rows ? rows[t] : max_rows;
        const int local_bits = bits_for((uint64_t)max_rows);  // the local key of an invalid id is rows[t] itself
        // table by table whenever that sorts fewer key bits; a single 8-bit pass gains nothing from it
        h->segmented = T > 1 && T <= kMaxSortSegments && h->key_bits > 8;
        h->sort_bits = h->segmented ? local_bits : h->key_bits;
    }
    {   // row-weighted share of the rows as wide as a wavefront (129..256 columns) among the tables up to 256 columns
        double wide = 0.0, all = 0.0;
        for (int t = 0; t < T; ++t) {
            if (D[t] > 256) continue;
            all += (double)rows[t];
            if (D[t] > 128) wide += (double)rows[t];
        }
        h->seg_mostly_wavefront_rows = all > 0.0 && wide >= 0.5 * all;
    }
    if (hipGetDevice(&h->device) != hipSuccess) {
        delete h;
        return TBE_EHIP;
    }
    h->static_scratch = static_scratch_address(h->device);   // (null: the entry point that needs it reports TBE_EHIP)
    const size_t b_doff = align256(4 * (size_t)(T + 1)), b_rb = align256(8 * (size_t)(T + 1)), b_wo = b_rb;
    const size_t b_cls = align256(4 * (size_t)T);
    const bool keep_hot = T <= kMaxSortSegments;
    const size_t b_hot = keep_hot ? align256(4 * (size_t)T * kHotRows) + align256(4 * (size_t)T) : 0;
    const size_t total = b_doff + b_rb + b_wo + 256 + b_cls + b_hot;
    std::vector<int32_t> cls_tables;
    {   // forward classes by lanes per row (D / elements per 16-byte fragment, rounded up to a power of two)
        const int vec = weight_dtype == TBE_F16 ? 8 : 4;
        std::vector<int32_t> lists[7];
        for (int t = 0; t < T; ++t) {
            const int nl = (D[t] + vec - 1) / vec;
            const int c = nl > 128 ? 6 : (nl > 64 ? 5 : (nl > kFwdGroupMaxLanes ? 0 : (nl > 16 ? 1 : (nl > 8 ? 2 : (nl > 4 ? 3 : 4)))));
            lists[c].push_back(t);
            h->fwd_columns[c] |= (uint32_t)D[t] | (uint32_t)h->D_off[t];
            h->fwd_maxD[c] = std::max(h->fwd_maxD[c], (int)D[t]);
        }
        for (int c = 0; c < 7; ++c) {
            h->fwd_first[c] = (int)cls_tables.size();
            h->fwd_count[c] = (int)lists[c].size();
            cls_tables.insert(cls_tables.end(), lists[c].begin(), lists[c].end());
        }
    }
    if (hipMalloc(&h->d_meta, total) != hipSuccess) {
        delete h;
        return TBE_EHIP;
    }
    char* base = static_cast<char*>(h->d_meta);
    h->d_D_off = reinterpret_cast<int32_t*>(base);
    h->d_row_base = reinterpret_cast<int64_t*>(base + b_doff);
    h->d_w_off = reinterpret_cast<int64_t*>(base + b_doff + b_rb);
    h->d_err = reinterpret_cast<int32_t*>(base + b_doff + b_rb + b_wo);
    h->d_fwd_tables = reinterpret_cast<int32_t*>(base + b_doff + b_rb + b_wo + 256);
    if (keep_hot) {   // (zeroed below: no hot rows until a backward call has listed some)
        h->d_hot_ids = reinterpret_cast<uint32_t*>(base + b_doff + b_rb + b_wo + 256 + b_cls);
        h->d_hot_n = h->d_hot_ids + align256(4 * (size_t)T * kHotRows) / 4;
    }
    bool ok = hipMemset(h->d_meta, 0, total) == hipSuccess;
    ok = ok && hipMemcpy(h->d_fwd_tables, cls_tables.data(), 4 * (size_t)T, hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_D_off, h->D_off.data(), 4 * (size_t)(T + 1), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_row_base, h->row_base.data(), 8 * (size_t)(T + 1), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_w_off, h->w_off.data(), 8 * (size_t)(T + 1), hipMemcpyHostToDevice) == hipSuccess;
    if (!ok) {
        (void)hipFree(h->d_meta);
        delete h;
        return TBE_EHIP;
    }
    *out = h;
    return TBE_OK;
}

tbe_status tbe_destroy(tbe_handle* h) {
    if (!h) return TBE_OK;
    for (auto& t : h->slots) {
        (void)hipEventDestroy(t.beg);
        (void)hipEventDestroy(t.end);
    }
    if (h->d_meta) (void)hipFree(h->d_meta);
    delete h;
    return TBE_OK;
}

static tbe_status check_batch(const tbe_handle* h, int32_t B, int64_t nnz) {
    if (B < 1) return TBE_ESHAPE;
    // positions are 32-bit; the margin keeps every strided position loop (steps of at most one tile) from wrapping
    if (nnz < 0 || nnz > (int64_t)0xFFFF0000ll) return TBE_ESHAPE;
    if ((int64_t)h->T * B >= ((int64_t)1 << 31)) return TBE_ESHAPE;
    return TBE_OK;
}

tbe_status tbe_workspace_bytes(const tbe_handle* h, int32_t B, int64_t max_nnz, size_t* bytes) {
    if (!h || !bytes) return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, max_nnz);
    if (st != TBE_OK) return st;
    *bytes = carve(h, B, max_nnz).total;
    return TBE_OK;
}

static bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

static bool io_ok(int io) { return io == TBE_IO_F32 || io == TBE_IO_F16 || io == TBE_IO_BF16; }
static bool idx_ok(int d) { return d == TBE_I64 || d == TBE_I32; }

tbe_status tbe_forward_ex(const tbe_handle* h, const void* tables, const int32_t* D_offsets, const void* indices,
                          const void* offsets, tbe_index_dtype index_dtype, int32_t B, int64_t nnz, tbe_pooling pooling,
                          void* out, tbe_io_dtype out_dtype, void* hip_stream) {
    if (!h || !tables || !offsets || !out || (!indices && nnz > 0)) return TBE_EINVAL;
    if (pooling != TBE_SUM && pooling != TBE_MEAN) return TBE_EDTYPE;
    if (!io_ok(out_dtype) || !idx_ok(index_dtype)) return TBE_EDTYPE;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    const size_t ia = index_dtype == TBE_I32 ? 4 : 8;
    if (!aligned(tables, 16) || !aligned(out, 16) || !aligned(indices, ia) || !aligned(offsets, ia)) return TBE_EINVAL;
    const hipError_t e = launch_forward(h, tables, D_offsets ? D_offsets : h->d_D_off, indices, offsets,
                                        index_dtype == TBE_I32, B, nnz, pooling, out, (int)out_dtype,
                                        static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? TBE_OK : TBE_EHIP;
}

tbe_status tbe_forward(const tbe_handle* h, const void* tables, const int32_t* D_offsets, const int64_t* indices,
                       const int64_t* offsets, int32_t B, int64_t nnz, tbe_pooling pooling, float* out,
                       void* hip_stream) {
    return tbe_forward_ex(h, tables, D_offsets, indices, offsets, TBE_I64, B, nnz, pooling, out, TBE_IO_F32, hip_stream);
}

// phases of the backward: steps a2-a4 need the ids only, steps a5-a6 need what a2-a4 left in the workspace
constexpr int kPrepare = 1, kApply = 2;

// shared body of the backward entry points; state == nullptr selects the plain SGD step
// seq != 0: the non-pooled layout (B is 1, offsets has T+1 entries, grad_out holds grad_elems elements)
static tbe_status backward_impl(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype, const void* indices,
                                const void* offsets, tbe_index_dtype index_dtype, int32_t B, int64_t nnz,
                                tbe_pooling pooling, float lr, float eps, float momentum_scale, void* tables, float* state,
                                void* workspace, size_t workspace_bytes, void* hip_stream, int seq = 0,
                                int64_t grad_elems = 0, int phases = kPrepare | kApply) {
    const bool prep = (phases & kPrepare) != 0, apply = (phases & kApply) != 0;
    if (!h || !offsets || (apply && !tables)) return TBE_EINVAL;
    if (nnz > 0 && ((prep && !indices) || (apply && !grad_out))) return TBE_EINVAL;
    if (pooling != TBE_SUM && pooling != TBE_MEAN) return TBE_EDTYPE;
    if (!io_ok(grad_dtype) || !idx_ok(index_dtype)) return TBE_EDTYPE;
    if (!isfinite(lr) || !isfinite(eps) || eps < 0.f || !isfinite(momentum_scale) || !(momentum_scale > 0.f))
        return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    const size_t ia = index_dtype == TBE_I32 ? 4 : 8;
    if (!aligned(tables, 16) || !aligned(grad_out, 16) || !aligned(state, 4) || !aligned(indices, ia) ||
        !aligned(offsets, ia))
        return TBE_EINVAL;
    if (nnz == 0) return TBE_OK;  // no id appears in the batch: no row has a gradient
    if (!workspace || !aligned(workspace, 256)) return TBE_EINVAL;
    const Workspace w = carve(h, B, nnz);
    if (workspace_bytes < w.total) return TBE_EWORKSPACE;
    char* ws = static_cast<char*>(workspace);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int idx32 = index_dtype == TBE_I32;
    hipError_t e = hipSuccess;
    if (prep) {
        e = launch_sort(h, w, ws, indices, offsets, idx32, B, nnz, seq != 0, s);
        if (e != hipSuccess) return TBE_EHIP;
        e = launch_lists(h, w, ws, offsets, idx32, B, seq, grad_elems, s);
        if (e != hipSuccess) return TBE_EHIP;
    }
    if (!apply) return TBE_OK;
    e = launch_segment_update(h, w, ws, grad_out, (int)grad_dtype, offsets, idx32, B, pooling, lr, eps, momentum_scale, tables,
                              state, seq, s);
    return e == hipSuccess ? TBE_OK : TBE_EHIP;
}

tbe_status tbe_backward_rowwise_adagrad_ex(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype,
                                           const void* indices, const void* offsets, tbe_index_dtype index_dtype,
                                           int32_t B, int64_t nnz, tbe_pooling pooling, float lr, float eps,
                                           float momentum_scale, void* tables, float* state, void* workspace,
                                           size_t workspace_bytes, void* hip_stream) {
    if (!state) return TBE_EINVAL;
    return backward_impl(h, grad_out, grad_dtype, indices, offsets, index_dtype, B, nnz, pooling, lr, eps, momentum_scale,
                         tables, state, workspace, workspace_bytes, hip_stream);
}

tbe_status tbe_backward_rowwise_adagrad_static(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype,
                                               const void* indices, const void* offsets, tbe_index_dtype index_dtype,
                                               int32_t B, int64_t nnz, tbe_pooling pooling, float lr, float eps,
                                               float momentum_scale, void* tables, float* state, void* hip_stream) {
    if (!h || !state) return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    if (carve(h, B, nnz).total > (size_t)TBE_STATIC_SCRATCH_BYTES) return TBE_EWORKSPACE;   // beyond the fixed array
    if (!h->static_scratch) return TBE_EHIP;
    // per-kernel timing creates events and grows a host-side list on first use: not in a call that allocates nothing
    tbe_handle* hm = const_cast<tbe_handle*>(h);
    const bool timing = hm->timing;
    hm->timing = false;
    const tbe_status r = backward_impl(h, grad_out, grad_dtype, indices, offsets, index_dtype, B, nnz, pooling, lr, eps,
                                       momentum_scale, tables, state, h->static_scratch, (size_t)TBE_STATIC_SCRATCH_BYTES,
                                       hip_stream);
    hm->timing = timing;
    return r;
}

tbe_status tbe_backward_prepare(const tbe_handle* h, const void* indices, const void* offsets,
                                tbe_index_dtype index_dtype, int32_t B, int64_t nnz, void* workspace,
                                size_t workspace_bytes, void* hip_stream) {
    return backward_impl(h, nullptr, TBE_IO_F32, indices, offsets, index_dtype, B, nnz, TBE_SUM, 0.f, 0.f, 1.f, nullptr,
                         nullptr, workspace, workspace_bytes, hip_stream, 0, 0, kPrepare);
}

tbe_status tbe_backward_apply_rowwise_adagrad(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype,
                                              const void* offsets, tbe_index_dtype index_dtype, int32_t B, int64_t nnz,
                                              tbe_pooling pooling, float lr, float eps, float momentum_scale,
                                              void* tables, float* state, void* workspace, size_t workspace_bytes,
                                              void* hip_stream) {
    if (!state) return TBE_EINVAL;
    return backward_impl(h, grad_out, grad_dtype, nullptr, offsets, index_dtype, B, nnz, pooling, lr, eps, momentum_scale,
                         tables, state, workspace, workspace_bytes, hip_stream, 0, 0, kApply);
}

tbe_status tbe_lookup_seq(const tbe_handle* h, const void* tables, const void* indices, const void* offsets,
                          tbe_index_dtype index_dtype, int64_t nnz, void* out, tbe_io_dtype out_dtype, int64_t out_elems,
                          void* hip_stream) {
    if (!h || !tables || !offsets || (!indices && nnz > 0) || (!out && out_elems > 0) || out_elems < 0) return TBE_EINVAL;
    if (!io_ok(out_dtype) || !idx_ok(index_dtype)) return TBE_EDTYPE;
    const tbe_status st = check_batch(h, 1, nnz);
    if (st != TBE_OK) return st;
    const size_t ia = index_dtype == TBE_I32 ? 4 : 8;
    if (!aligned(tables, 16) || !aligned(out, 16) || !aligned(indices, ia) || !aligned(offsets, ia)) return TBE_EINVAL;
    const hipError_t e = launch_lookup_seq(h, tables, indices, offsets, index_dtype == TBE_I32, nnz, out, (int)out_dtype,
                                           out_elems, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? TBE_OK : TBE_EHIP;
}

tbe_status tbe_backward_seq_rowwise_adagrad(const tbe_handle* h, const void* grad_seq, tbe_io_dtype grad_dtype,
                                            int64_t grad_elems, const void* indices, const void* offsets,
                                            tbe_index_dtype index_dtype, int64_t nnz, float lr, float eps,
                                            float momentum_scale, void* tables, float* state, void* workspace,
                                            size_t workspace_bytes, void* hip_stream) {
    if (!state || grad_elems < 0) return TBE_EINVAL;
    return backward_impl(h, grad_seq, grad_dtype, indices, offsets, index_dtype, 1, nnz, TBE_SUM, lr, eps, momentum_scale,
                         tables, state, workspace, workspace_bytes, hip_stream, 1, grad_elems);
}

tbe_status tbe_backward_sgd(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype, const void* indices,
                            const void* offsets, tbe_index_dtype index_dtype, int32_t B, int64_t nnz, tbe_pooling pooling,
                            float lr, void* tables, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return backward_impl(h, grad_out, grad_dtype, indices, offsets, index_dtype, B, nnz, pooling, lr, 0.f, 1.f, tables,
                         nullptr, workspace, workspace_bytes, hip_stream);
}

tbe_status tbe_backward_apply_sgd(const tbe_handle* h, const void* grad_out, tbe_io_dtype grad_dtype, const void* offsets,
                                  tbe_index_dtype index_dtype, int32_t B, int64_t nnz, tbe_pooling pooling, float lr,
                                  void* tables, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return backward_impl(h, grad_out, grad_dtype, nullptr, offsets, index_dtype, B, nnz, pooling, lr, 0.f, 1.f, tables,
                         nullptr, workspace, workspace_bytes, hip_stream, 0, 0, kApply);
}

tbe_status tbe_backward_rowwise_adagrad(const tbe_handle* h, const float* grad_out, const int64_t* indices,
                                        const int64_t* offsets, int32_t B, int64_t nnz, tbe_pooling pooling, float lr,
                                        float eps, float momentum_scale, void* tables, float* state, void* workspace,
                                        size_t workspace_bytes, void* hip_stream) {
    return tbe_backward_rowwise_adagrad_ex(h, grad_out, TBE_IO_F32, indices, offsets, TBE_I64, B, nnz, pooling, lr, eps,
                                           momentum_scale, tables, state, workspace, workspace_bytes, hip_stream);
}

tbe_status tbe_debug_sorted(const tbe_handle* h, void* workspace, int32_t B, int64_t nnz, const uint32_t** keys_sorted,
                            const uint32_t** vals_sorted, const uint32_t** unique_rows, const uint32_t** seg_start,
                            const uint32_t** num_unique) {
    if (!h || !workspace) return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    const Workspace w = carve(h, B, nnz);
    const int buf = w.sort.passes & 1;  // every pass flips the double buffer, starting from 0
    char* ws = static_cast<char*>(workspace);
    if (keys_sorted) *keys_sorted = reinterpret_cast<const uint32_t*>(ws + w.keys[buf]);
    if (vals_sorted) *vals_sorted = reinterpret_cast<const uint32_t*>(ws + w.vals[buf]);
    if (unique_rows) *unique_rows = reinterpret_cast<const uint32_t*>(ws + w.vals[buf ^ 1]);
    if (seg_start) *seg_start = reinterpret_cast<const uint32_t*>(ws + w.seg_start);
    if (num_unique) *num_unique = reinterpret_cast<const uint32_t*>(ws + w.counters);
    return TBE_OK;
}

tbe_status tbe_debug_hot_rows(const tbe_handle* h, void* workspace, int32_t B, int64_t nnz, const uint32_t** hot_ids,
                              const uint32_t** hot_n, const uint32_t** dense_rows, const uint32_t** dense_n,
                              const uint32_t** long_rows) {
    if (!h || !workspace || !hot_ids || !hot_n || !dense_rows || !dense_n || !long_rows) return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    const Workspace w = carve(h, B, nnz);
    char* ws = static_cast<char*>(workspace);
    const bool hint = h->d_hot_ids != nullptr;
    *hot_ids = hint ? reinterpret_cast<uint32_t*>(ws + w.hot_ids) : nullptr;
    *hot_n = hint ? reinterpret_cast<uint32_t*>(ws + w.hot_n) : nullptr;
    *dense_rows = w.dense ? reinterpret_cast<uint32_t*>(ws + w.dense_rows) : nullptr;
    *dense_n = w.dense ? reinterpret_cast<uint32_t*>(ws + w.dense_n) : nullptr;
    *long_rows = reinterpret_cast<uint32_t*>(ws + w.long_rows);
    return TBE_OK;
}

tbe_status tbe_debug_forward_kernels(const tbe_handle* h, int32_t B, int64_t nnz, uint32_t* kernels) {
    if (!h || !kernels) return TBE_EINVAL;
    const tbe_status st = check_batch(h, B, nnz);
    if (st != TBE_OK) return st;
    *kernels = forward_kernels(h, B, nnz);
    return TBE_OK;
}

tbe_status tbe_poll_index_error(tbe_handle* h) {
    if (!h) return TBE_EINVAL;
    int32_t flag = 0;
    if (hipDeviceSynchronize() != hipSuccess) return TBE_EHIP;
    if (hipMemcpy(&flag, h->d_err, sizeof(flag), hipMemcpyDeviceToHost) != hipSuccess) return TBE_EHIP;
    if (flag) {
        if (hipMemset(h->d_err, 0, sizeof(flag)) != hipSuccess) return TBE_EHIP;
        return TBE_EINDEX;
    }
    return TBE_OK;
}

tbe_status tbe_replica_mean(tbe_handle* h, void* const* replicas, int32_t M, size_t count, tbe_dtype dtype,
                            void* hip_stream) {
    if (!h || !replicas || M < 1 || M > kMaxReplicas) return TBE_EINVAL;
    if (dtype != TBE_F32 && dtype != TBE_F16) return TBE_EDTYPE;
    const size_t bytes = count * (dtype == TBE_F32 ? 4u : 2u);
    for (int m = 0; m < M; ++m) {
        if (!replicas[m] || !aligned(replicas[m], 16)) return TBE_EINVAL;
        const uintptr_t a0 = reinterpret_cast<uintptr_t>(replicas[m]);
        for (int k = 0; k < m; ++k) {   // two replicas that share bytes would race (equal pointers, or ranges that overlap)
            const uintptr_t b0 = reinterpret_cast<uintptr_t>(replicas[k]);
            if (a0 == b0 || (a0 < b0 + bytes && b0 < a0 + bytes)) return TBE_EINVAL;
        }
    }
    if (count == 0 || M == 1) return TBE_OK;   // the mean over one replica is that replica
    const hipError_t e = launch_replica_mean(h, replicas, M, count, dtype == TBE_F32, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? TBE_OK : TBE_EHIP;
}

tbe_status tbe_set_tunable(tbe_handle* h, tbe_tunable which, int64_t value) {
    if (!h) return TBE_EINVAL;
    switch (which) {
        case TBE_TUNE_HOT_ROWS_MIN_WORKGROUPS: h->hot_min_workgroups = value; return TBE_OK;
    }
    return TBE_EINVAL;
}

tbe_status tbe_timing_enable(tbe_handle* h, int enable) {
    if (!h) return TBE_EINVAL;
    h->timing = enable != 0;
    h->n_used = 0;
    return TBE_OK;
}

tbe_status tbe_timing_count(tbe_handle* h, int32_t* n) {
    if (!h || !n) return TBE_EINVAL;
    *n = h->n_used;
    return TBE_OK;
}

tbe_status tbe_timing_read(tbe_handle* h, int32_t i, const char** name, float* ms) {
    if (!h || !name || !ms || i < 0 || i >= h->n_used) return TBE_EINVAL;
    TimingSlot& t = h->slots[i];
    if (hipEventSynchronize(t.end) != hipSuccess) return TBE_EHIP;
    if (hipEventElapsedTime(ms, t.beg, t.end) != hipSuccess) return TBE_EHIP;
    *name = t.name;
    return TBE_OK;
}

}  // extern "C"
