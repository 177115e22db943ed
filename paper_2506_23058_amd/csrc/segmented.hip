// segmented.hip -- partition2L / filter_seg on gfx950: partition2 applied to
// every row of a jagged array given by its shape (Section 6, "Segmented
// operations"; the flat-form helpers mkSgmDescr / mkII of Section 2.1).
//
// Row k covers [o_k, o_k + s_k), o_k = s_0 + ... + s_{k-1}.  Partition writes
//   idx[i] = o_k + (c_i ? #trues before i in row k : T_k + #falses before i in row k)
// (the index function the paper infers for partition2L); filter packs the kept
// elements of all rows one row after the other (so a kept element goes to the
// number of kept elements before it in the whole array) and gives -1 to the
// others.  T_k (trues of row k) is written for every row, and optionally the
// segment descriptor: a byte array with 1 at o_k for every non-empty row.
//
// Work decomposition.  Each non-empty row is cut into work items of at most
// one tile (TILE = block * rows * 4 elements), aligned to 4-element groups so
// that loads stay vector loads: item j of row k covers
//   [A_k + j*TILE, A_k + (j+1)*TILE) ∩ [o_k, o_k + s_k),
// A_k = o_k rounded down to 32 (a 128-byte line) when that gives the row no
// more items than rounding down to 4, else o_k rounded down to 4.
// Where rows are short on average, rows of at most a quarter tile are packed:
// an item holds the whole short rows that start in one window of 3 quarter
// tiles (up to the next longer row, and inside one block of rows).
// Kernels (all stream-ordered, capturable in one HIP graph):
//   seg_shape -- (up to 16384 rows) row offsets, item offsets and item
//                descriptors in one launch: each workgroup rescans the sizes
//                before its rows; the last one validates the shape;
//   seg_sizes, seg_rows, seg_records -- (more rows) the same in three launches
//                over chunks of rows, each workgroup adding up the chunk
//                totals before its own;
//   seg_count -- one wave per 1024-element chunk counts the trues of the items
//                whose row spans several items and is not synchronised in
//                seg_main (partition), or of every item (filter), into a
//                dense array of item counts;
//   seg_scan_items / seg_item_bases -- one scan of all item counts, then per
//                item its output bases and T_k of its row;
//   seg_main  -- workgroups take items round-robin (the default grid of 64
//                workgroups per CU oversubscribes the chip, so the hardware
//                starts the items in order as slots free); each
//                loads its item, ranks the trues by ballot/mbcnt, writes the
//                indices and descriptor bytes in input order and the keys,
//                staged in LDS, as two runs per wave.  A row that fits one
//                item is read once: its T_k comes from the item itself.  A
//                row of 2..kSibMax items is read once too (partition, row
//                sync WAIT): its items publish their counts to one another.
#include <type_traits>

#include "device.hpp"
#include "host.hpp"

namespace ixp {
namespace {

constexpr size_t kSegHeader = 256;   // error i32 @4, item count i64 @8, scan ticket u32 @16,
                                     // counted items u64 @24
constexpr int64_t kScanChunk = 8192;  // item counts per workgroup of seg_scan_items
#ifndef IXP_SEG_COUNT_ROWS
#define IXP_SEG_COUNT_ROWS 4
#endif
constexpr int kSegCountLog = IXP_SEG_COUNT_ROWS == 16 ? 12 : IXP_SEG_COUNT_ROWS == 8 ? 11 : 10;   // log2(256 * rows)
// Rows of 2..kSibMax items exchange their counts inside seg_main.  A
// published count is kCntReady | trues.  A waiting item polls at most
// kSibPolls times before counting the rest itself.
constexpr int kSibMax = 256;
constexpr uint64_t kCntReady = kStA;
constexpr uint32_t kSibPolls = 64;

// Per-item descriptor written by write_item and completed by seg_item_bases.
struct alignas(16) SegItem {
    int64_t lo, hi;      // valid positions [lo, hi)
    int64_t base;        // first position of the item's tile (4-aligned; see row_first_base)
    int64_t tbase;       // output position of the item's first true
    int64_t fbase;       // output position of the item's first false (until seg_item_bases
                         // sets it, the number of items of the row)
    int32_t row;         // row k
    int32_t kind;        // bit 0: row fits one item; bit 1: first item of its row;
                         // bit 2: row synchronised in seg_main, with its item
                         // count in bits 8..23 (tbase then holds o_k);
                         // bit 3: packed item, the whole short rows [row, first)
    int64_t first;       // first item of the row, or end row (bit 3)
};
constexpr int32_t kOwnRows = 1 | 8;        // the item holds whole rows
constexpr int32_t kPacked = 8;

struct SegArgs {
    const uint32_t *keys;
    int64_t n;
    const int64_t *shape;
    int64_t m;
    uint32_t *out_keys;
    void *out_idx;
    int64_t *seg_split;
    uint8_t *flags_out;
    int64_t *offsets;     // [m + 1] row offsets
    int64_t *item_off;    // [m + 1] first item of each row inside its chunk (three-launch shape scan)
    SegItem *items;       // [max_items]
    int64_t *prefix;      // [max_items + 1] exclusive scan of item counts
    unsigned long long *counts;   // [max_items] trues per counted item
    uint64_t *scan_desc;          // [ceil(max_items / kScanChunk)] look-back descriptors
    uint32_t *scan_ticket;
    int64_t max_items;
    int32_t *err;
    int64_t *num_items;
    unsigned long long *num_counted;   // items whose trues seg_count counts
    int64_t tile;
    int32_t tile_shift;   // tile = 2^tile_shift
    int32_t mode;
    int32_t need_keys;
    int32_t row_sync;     // IXP_ROW_SYNC_COUNT, _WAIT or _NOWAIT
    int32_t keep;         // plain loads of the keys (see prepare)
    int64_t short_max;    // rows of at most this many elements are packed (0: none)
    int64_t chunk_rows;   // rows per workgroup of seg_sizes / seg_rows / seg_records
    int64_t nchunks;
    int64_t *csum, *citems, *ccounted, *cbad;   // [kShapeChunks] of a chunk: elements, items, counted
                                                // items, whether a size is bad
};

constexpr int64_t kShapeFusedRows = 16384;   // up to here the shape takes one launch (seg_shape)
constexpr int kFusedPackShift = 8, kChunkPackShift = 10;
constexpr int64_t kShapeChunks = 1024;

// Packed rows have at most tile / 4 elements and start in one window of
// 3 tile / 4, so an item of them spans less than a tile whatever their sizes.
int64_t seg_max_items(int64_t n, int64_t m, int64_t tile, bool pack) {
    const int64_t plain = ceil_div(n + 3 * m, tile) + m + 1;
    if (!pack) return plain;
    // long rows; windows, each cut once more by every long row and block edge
    const int64_t longs = n / (tile / 4 + 1) < m ? n / (tile / 4 + 1) : m;
    const int64_t edges = (m >> (m <= kShapeFusedRows ? kFusedPackShift : kChunkPackShift)) + 1;
    const int64_t packed = n / (tile / 4 * 3) + 1 + longs + edges;
    const int64_t bound = packed + (n + 3 * longs) / tile + longs + 2;
    return bound < plain ? bound : plain;
}

// A row's size as it is counted.  One outside [0, n] makes the shape invalid and
// counts 0: then the offsets' and items' sums cannot wrap, and the records of an
// invalid shape stay inside [0, max_items) (they are written before the last
// chunk has found it invalid).
__device__ __forceinline__ bool size_bad(const SegArgs &a, int64_t v) { return v < 0 || v > a.n; }
__device__ __forceinline__ int64_t size_counted(const SegArgs &a, int64_t v) { return size_bad(a, v) ? 0 : v; }

// The items a row begins: 0 for an empty row and for a short row that joins
// the item of the row before it (`prev` elements, 0 if the block of rows
// holds no non-empty row before this one).
__device__ __forceinline__ int64_t row_items(const SegArgs &a, int64_t o, int64_t sk, int64_t prev) {
    if (sk <= a.short_max) {   // (never a non-empty row when nothing is packed)
        // windows of 3 quarter tiles, counted in 32 bits (2^42 elements)
        const int32_t q = a.tile_shift - 2;
        const uint32_t w0 = static_cast<uint32_t>((o - prev) >> q) / 3, w1 = static_cast<uint32_t>(o >> q) / 3;
        return (sk > 0) & ((prev == 0) | (prev > a.short_max) | (w0 != w1));
    }
    return ((o & 3) + sk + a.tile - 1) >> a.tile_shift;
}

// True when a row of nit items has its items counted by the counting pass.
__device__ __forceinline__ bool row_synced(const SegArgs &a, int64_t nit) {
    return a.mode == IXP_MODE_PARTITION && a.row_sync != IXP_ROW_SYNC_COUNT && nit > 1 && nit <= kSibMax;
}
__device__ __forceinline__ bool row_counted(const SegArgs &a, int64_t nit) {
    return a.mode != IXP_MODE_PARTITION || nit > (a.row_sync == IXP_ROW_SYNC_COUNT ? 1 : kSibMax);
}

// Rows are cut into items of `tile` elements from the 16-byte group holding
// the row's first element, which fixes the row's item count.  The first item
// starts one 128-byte line earlier when that keeps the count: then every
// boundary between two items of the row falls on a cache line, and the items
// (written by different workgroups, often on different XCDs with their own
// L2) share no output line inside the row.  Only row ends remain mid-line.
__device__ __forceinline__ int64_t row_first_base(int64_t o, int64_t sk, int64_t nit, int64_t tile,
                                                  int32_t shift) {
    const int64_t line = o & ~int64_t{31};
    return ((o + sk - line + tile - 1) >> shift) == nit ? line : (o & ~int64_t{3});
}

// ------------------------------------------------------------------ shape --
constexpr int kSetupThreads = 256;   // of the three-launch shape scan
constexpr int kSetupPer = 4;

// Exclusive scan over a workgroup of WAVES waves; `lds` holds WAVES words.
template <int WAVES>
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t *lds, int64_t *total) {
    const int lane = threadIdx.x & 63;
    const int wave = wave_id();
    const int64_t inc = wave_scan_i64(v);
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    int64_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int64_t x = lds[w];
        before += w < wave ? x : 0;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return before + inc - v;
}

// Sum over the workgroup of one value per thread, in every thread.
__device__ __forceinline__ int64_t block_sum_of(int64_t v, int64_t *lds16) {
    v = wave_sum_i64(v);
    if ((threadIdx.x & 63) == 0) lds16[wave_id()] = v;
    __syncthreads();
    int64_t tot = 0;
    for (uint32_t w = 0; w < blockDim.x / kWave; ++w) tot += lds16[w];
    __syncthreads();
    return tot;
}

// This thread's share of the sum of x[0..c), c <= kShapeChunks.
__device__ __forceinline__ int64_t chunks_before(const int64_t *x, int64_t c) {
    int64_t v = 0;
#pragma unroll
    for (int j = 0; j < kShapeChunks / kSetupThreads; ++j) {
        const int64_t i = j * kSetupThreads + static_cast<int64_t>(threadIdx.x);
        v += i < c ? x[i] : 0;
    }
    return v;
}

// Record `idx` of the items begun by rows [r0, r0 + own), whose offsets and
// first items, and those of the rows up to r0 + nr >= r0 + own, stand in
// s_off[0..nr], s_it[0..nr]; a packed item ends before r0 + nr.
__device__ __forceinline__ void write_item(const SegArgs &a, int64_t idx, const int64_t *s_off,
                                           const int64_t *s_it, int64_t r0, int own, int nr) {
    // the last rows with s_it <= idx and s_it <= idx + 1: both searches at once
    int j = 0, hi = own - 1, j1 = 0, hi1 = nr - 1;
    while (j < hi || j1 < hi1) {
        const int m0 = (j + hi + 1) >> 1, m1 = (j1 + hi1 + 1) >> 1;
        const int64_t x0 = s_it[m0], x1 = s_it[m1];
        if (x0 <= idx) j = m0;
        else hi = m0 - 1;
        if (x1 <= idx + 1) j1 = m1;
        else hi1 = m1 - 1;
    }
    const int64_t o = s_off[j], e = s_off[j + 1];
    SegItem d;
    d.fbase = 0;
    d.row = static_cast<int32_t>(r0 + j);
    // a short row's item reaches up to the row that begins the next item, or to the
    // end of the block; one that holds no other row's elements is an ordinary item
    // (rows of 1100 and 300 in turn, a filter by a row predicate: 187 -> 150 us)
    if (idx + 1 >= s_it[nr]) j1 = nr;
    if (e - o <= a.short_max && s_off[j1] > e) {
        d.lo = o;
        d.hi = s_off[j1];
        d.base = o & ~int64_t{31};
        d.tbase = 0;
        d.kind = kPacked | 2;
        d.first = r0 + j1;
    } else {
        const int64_t i0 = s_it[j], nit = s_it[j + 1] - i0, q = idx - i0;
        const bool sib = row_synced(a, nit);
        d.base = row_first_base(o, e - o, nit, a.tile, a.tile_shift) + q * a.tile;
        d.lo = d.base > o ? d.base : o;
        d.hi = d.base + a.tile < e ? d.base + a.tile : e;
        d.tbase = sib ? o : 0;
        d.fbase = nit;   // for seg_item_bases
        d.kind = (nit == 1 ? 1 : 0) | (q == 0 ? 2 : 0) | (sib ? 4 | static_cast<int32_t>(nit << 8) : 0);
        d.first = i0;
    }
    a.items[idx] = d;
    a.counts[idx] = 0;
}

// More than kShapeFusedRows rows: three launches over at most kShapeChunks
// chunks of whole 1024-row blocks.  Every workgroup adds up the chunk totals
// before its own, so none waits for another and nothing carries over between
// calls.  (One workgroup scanning the whole shape and one launch for the
// records took 340 us for 250,000 rows; the three launches take 25 us.)
//   seg_sizes   -- elements per chunk;
//   seg_rows    -- row offsets, and the items of a chunk;
//   seg_records -- the item records; the last chunk validates the shape.
__global__ __launch_bounds__(kSetupThreads) void seg_sizes_kernel(SegArgs a) {
    __shared__ int64_t lds[16];
    __shared__ int bad;
    const int64_t c = blockIdx.x, r0 = c * a.chunk_rows;
    const int64_t r1 = r0 + a.chunk_rows < a.m ? r0 + a.chunk_rows : a.m;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    int64_t sum = 0;
    bool wrong = false;
    for (int64_t b = r0; b < r1; b += kSetupThreads * kSetupPer) {
#pragma unroll
        for (int j = 0; j < kSetupPer; ++j) {
            const int64_t k = b + j * kSetupThreads + threadIdx.x;
            const int64_t v = k < r1 ? a.shape[k] : 0;
            wrong |= size_bad(a, v);
            sum += size_counted(a, v);
        }
    }
    if (ballot(wrong) != 0 && (threadIdx.x & 63) == 0) atomicOr(&bad, 1);
    sum = block_sum_of(sum, lds);
    if (threadIdx.x == 0) {
        a.csum[c] = sum;
        a.cbad[c] = bad;
    }
    // clear the item scan's ticket and look-back descriptors
    const int64_t g = c * kSetupThreads + threadIdx.x;
    const int64_t nd = (a.max_items + kScanChunk - 1) / kScanChunk;
    for (int64_t j = g; j < nd; j += static_cast<int64_t>(gridDim.x) * kSetupThreads) a.scan_desc[j] = 0;
    if (g == 0) *a.scan_ticket = 0;
}

__global__ __launch_bounds__(kSetupThreads) void seg_rows_kernel(SegArgs a) {
    constexpr int kBlockRows = kSetupThreads * kSetupPer;
    static_assert(kBlockRows == 1 << kChunkPackShift, "packing block");
    __shared__ int64_t lds[16];
    __shared__ int64_t sz[kBlockRows];
    __shared__ int wlast[kSetupThreads / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int64_t c = blockIdx.x, c0 = c * a.chunk_rows;
    const int64_t c1 = c0 + a.chunk_rows < a.m ? c0 + a.chunk_rows : a.m;
    int64_t off = block_sum_of(chunks_before(a.csum, c), lds);
    int64_t items = 0, counted = 0;
    for (int64_t b = c0; b < c1; b += kBlockRows) {
        __syncthreads();   // sz is reused
#pragma unroll
        for (int j = 0; j < kSetupPer; ++j) {
            const int64_t k = b + j * kSetupThreads + tid;
            const int64_t v = k < c1 ? a.shape[k] : 0;
            sz[j * kSetupThreads + tid] = size_counted(a, v);
        }
        __syncthreads();
        int64_t s[kSetupPer], sum_s = 0;
        int last = 0;   // 1 + this thread's last non-empty row in the block
#pragma unroll
        for (int j = 0; j < kSetupPer; ++j) {
            s[j] = sz[tid * kSetupPer + j];
            sum_s += s[j];
            if (s[j] > 0) last = tid * kSetupPer + j + 1;
        }
        int64_t tot_s;
        const int64_t off0 = off + block_exclusive_scan<kSetupThreads / kWave>(sum_s, lds, &tot_s);
        int64_t prev = 0;
        if (a.short_max) {
            // `last` grows with the thread: the nearest one before, in the wave, then the waves
            const uint64_t any = ballot(last != 0), under = any & ((1ull << lane) - 1);
            int before = __shfl(last, under ? 63 - __builtin_clzll(under) : 0, kWave);
            if (!under) before = 0;
            if (lane == kWave - 1) wlast[wave] = last ? last : before;
            __syncthreads();
            for (int w = 0; w < wave; ++w) before = wlast[w] > before ? wlast[w] : before;
            prev = before ? sz[before - 1] : 0;
            __syncthreads();   // wlast is reused
        }
        int64_t nit[kSetupPer], sum_it = 0, o = off0;
#pragma unroll
        for (int j = 0; j < kSetupPer; ++j) {
            nit[j] = row_items(a, o, s[j], prev);
            sum_it += nit[j];
            if (row_counted(a, nit[j])) counted += nit[j];
            if (s[j] > 0) prev = s[j];
            o += s[j];
        }
        int64_t tot_it;
        int64_t it = items + block_exclusive_scan<kSetupThreads / kWave>(sum_it, lds, &tot_it);
        o = off0;
#pragma unroll
        for (int j = 0; j < kSetupPer; ++j) {
            const int64_t k = b + tid * kSetupPer + j;
            if (k < c1) {
                a.offsets[k] = o;
                a.item_off[k] = it;   // inside the chunk
            }
            o += s[j];
            it += nit[j];
        }
        off += tot_s;
        items += tot_it;
    }
    counted = block_sum_of(counted, lds);
    if (tid == 0) {
        a.citems[c] = items;
        a.ccounted[c] = counted;
        if (c1 == a.m) a.offsets[a.m] = off;
    }
}

// Workgroup w takes rows [256 w, 256 w + 256); the other rows of their block
// tell where a packed item that reaches past them ends.
__global__ __launch_bounds__(kSetupThreads) void seg_records_kernel(SegArgs a) {
    constexpr int kBlockRows = kSetupThreads * kSetupPer;
    __shared__ int64_t lds[kSetupThreads / kWave];
    __shared__ int64_t s_off[kBlockRows + 1], s_it[kBlockRows + 1];
    const int tid = threadIdx.x;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kSetupThreads;
    const int own = static_cast<int>(a.m - r0 < kSetupThreads ? a.m - r0 : kSetupThreads);
    const int64_t bend = (r0 | (kBlockRows - 1)) + 1;   // end of the block of rows
    const int nr = static_cast<int>((a.m < bend ? a.m : bend) - r0);
    const int64_t c = r0 / a.chunk_rows, c1 = (c + 1) * a.chunk_rows < a.m ? (c + 1) * a.chunk_rows : a.m;
    const int64_t ibase = block_sum_of(chunks_before(a.citems, c), lds);
    const int64_t iend = ibase + a.citems[c];
    for (int j = tid; j <= nr; j += kSetupThreads) {
        s_off[j] = a.offsets[r0 + j];
        s_it[j] = r0 + j < c1 ? ibase + a.item_off[r0 + j] : iend;
    }
    __syncthreads();
    // (a bad shape may ask for more records than fit: the rest is left out)
    for (int64_t idx = s_it[0] + tid; idx < s_it[own] && idx < a.max_items; idx += kSetupThreads)
        write_item(a, idx, s_off, s_it, r0, own, nr);
    if (r0 + own < a.m) return;
    const int64_t bad = block_sum_of(chunks_before(a.cbad, a.nchunks), lds);
    const int64_t counted = block_sum_of(chunks_before(a.ccounted, a.nchunks), lds);
    if (tid == 0) {
        const bool ok = !bad && a.offsets[a.m] == a.n && iend <= a.max_items;
        *a.num_items = ok ? iend : 0;
        *a.num_counted = ok ? static_cast<unsigned long long>(counted) : 0ull;
        *a.err = ok ? 0 : kErrShape;
    }
}

// Shape scan and item records in one launch, for up to kShapeFusedRows rows.
// Workgroup j owns rows
// [256 j, 256 j + 256) and recomputes the scan of every row before and
// including its own (at most kShapeFusedRows sizes, read from L2), so no
// workgroup waits for another and no state carries over between calls.  The
// last workgroup scans all rows: it validates the shape and writes the totals,
// the item count and the number of items the counting pass will count.  It
// writes no output: T_k of empty rows is written by the counting kernel, once
// the shape is known good.
constexpr int kShapeThreads = 1024;

__global__ __launch_bounds__(kShapeThreads) void seg_shape_kernel(SegArgs a) {
    __shared__ int64_t lds_a[16], lds_b[16];
    __shared__ int64_t s_off[257], s_it[257];
    __shared__ int64_t sz[kShapeFusedRows];   // the sizes of rows [0, rend)
    __shared__ int bad;
    __shared__ int wlast[kShapeThreads / kWave];   // 1 + a wave's last non-empty row
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * 256;
    const int64_t rend = a.m - r0 < 256 ? a.m : r0 + 256;   // rows [0, rend) are scanned
    const int nr = static_cast<int>(rend - r0);
    const int part = blockIdx.y;   // of the workgroups that share these rows' records
    const bool last = rend == a.m && part == 0;
    if (tid == 0) bad = 0;
    if (part == 0) {   // clear the item scan's ticket and look-back descriptors
        const int64_t g = static_cast<int64_t>(blockIdx.x) * kShapeThreads + tid;
        const int64_t nd = (a.max_items + kScanChunk - 1) / kScanChunk;
        for (int64_t j = g; j < nd; j += static_cast<int64_t>(gridDim.x) * kShapeThreads) a.scan_desc[j] = 0;
        if (g == 0) *a.scan_ticket = 0;
    }
    __syncthreads();
    // coalesced loads into LDS, all in flight at once
    {
        constexpr int kLoads = kShapeFusedRows / kShapeThreads;
        int64_t v[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int64_t k = tid + static_cast<int64_t>(j) * kShapeThreads;
            v[j] = k < rend ? a.shape[k] : 0;
        }
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int64_t k = tid + static_cast<int64_t>(j) * kShapeThreads;
            if (size_bad(a, v[j])) atomicOr(&bad, 1);
            if (k < rend) sz[k] = size_counted(a, v[j]);
        }
    }
    __syncthreads();
    // thread t holds rows [t per, t per + per) of [0, rend)
    const int per = static_cast<int>((rend + kShapeThreads - 1) / kShapeThreads);
    const int64_t k0 = static_cast<int64_t>(tid) * per;
    const int64_t k1 = k0 + per < rend ? k0 + per : rend;
    const bool pack = a.short_max > 0;
    int64_t sum_s = 0;
    int filled = 0;   // 1 + this thread's last non-empty row, then 1 + the last one before its rows
    for (int64_t k = k0; k < k1; ++k) {
        sum_s += sz[k];
        if (sz[k] > 0) filled = static_cast<int>(k) + 1;
    }
    if (pack) {
        // the nearest one of the lanes below, then of the waves before; looking for it
        // row by row took 15 us where 1 row in 97 is not empty
        const uint64_t under = ballot(filled != 0) & ((1ull << lane) - 1);
        const int at = __shfl(filled, under ? 63 - __builtin_clzll(under) : 0, kWave);
        const int before = under ? at : 0;
        if (lane == kWave - 1) wlast[wave] = filled ? filled : before;
        filled = before;
    }
    int64_t tot_s;
    const int64_t off0 = block_exclusive_scan<16>(sum_s, lds_a, &tot_s);   // (its barriers publish wlast)
    if (pack)
        for (int w = 0; w < wave; ++w) filled = wlast[w] > filled ? wlast[w] : filled;
    // calls row(k, o, items) for this thread's rows; the packed form keeps the
    // last non-empty size before a row in its block of rows
    auto rows = [&](auto packed, auto &&row) {
        constexpr bool kPack = decltype(packed)::value;
        constexpr int64_t kBlock = int64_t{1} << kFusedPackShift;
        int64_t o = off0, prev = kPack && filled > (k0 & ~(kBlock - 1)) ? sz[filled - 1] : 0;
        for (int64_t k = k0; k < k1; ++k) {
            const int64_t sk = sz[k];
            if (kPack) {
                if ((k & (kBlock - 1)) == 0) prev = 0;
                row(k, o, row_items(a, o, sk, prev));
                if (sk > 0) prev = sk;
            } else {
                row(k, o, sk > 0 ? ((o & 3) + sk + a.tile - 1) >> a.tile_shift : int64_t{0});
            }
            o += sk;
        }
    };
    int64_t sum_it = 0, counted = 0;
    auto add = [&](int64_t, int64_t, int64_t nit) {
        sum_it += nit;
        counted += row_counted(a, nit) ? nit : 0;
    };
    if (pack) rows(std::true_type{}, add);
    else rows(std::false_type{}, add);
    int64_t tot_it;
    const int64_t it0 = block_exclusive_scan<16>(sum_it, lds_b, &tot_it);
    if (k1 > r0) {   // (the other threads' rows are other workgroups')
        int64_t it = it0;
        auto put = [&](int64_t k, int64_t o, int64_t nit) {
            if (k >= r0) {
                s_off[k - r0] = o;
                s_it[k - r0] = it;
                if (part == 0) a.offsets[k] = o;
            }
            it += nit;
        };
        if (pack) rows(std::true_type{}, put);
        else rows(std::false_type{}, put);
    }
    if (tid == 0) {
        s_off[nr] = tot_s;
        s_it[nr] = tot_it;
    }
    if (last) {
        int64_t tot_counted;
        (void)block_exclusive_scan<16>(counted, lds_a, &tot_counted);
        if (tid == 0) {
            const bool ok = !bad && tot_s == a.n && tot_it <= a.max_items;
            a.offsets[a.m] = tot_s;
            *a.num_items = ok ? tot_it : 0;
            *a.num_counted = ok ? static_cast<unsigned long long>(tot_counted) : 0ull;
            *a.err = ok ? 0 : kErrShape;
        }
    }
    __syncthreads();
    // this workgroup's item records (a bad shape may ask for more than fit:
    // those are not written, and the last workgroup reports the error)
    for (int64_t idx = s_it[0] + part * kShapeThreads + tid; idx < s_it[nr] && idx < a.max_items;
         idx += gridDim.y * kShapeThreads)
        write_item(a, idx, s_off, s_it, r0, nr, nr);
}

// ------------------------------------------------------------------ count --
// One wave per 1024-element chunk of a counted item (items of rows that span
// several items in partition mode, every item in filter mode); each wave adds
// its chunk's trues to the item's count.  Waves of one item hit one address
// at most tile/1024 times, so the atomics do not queue.
template <class Pred>
__global__ __launch_bounds__(256) void seg_count_kernel(SegArgs a, Pred pred) {
    using WT = Tile<kWave, IXP_SEG_COUNT_ROWS, 4>;   // one wave, 256 * rows elements
    constexpr int kCLog = kSegCountLog;
    const int lane = threadIdx.x & (kWave - 1);
    if (*a.err != 0) return;   // a bad shape: no output is written
    if (a.seg_split) {
        // T_k = 0 for empty rows, once the shape is known good
        for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < a.m;
             k += static_cast<int64_t>(gridDim.x) * blockDim.x)
            if (a.offsets[k] == a.offsets[k + 1]) a.seg_split[k] = 0;
    }
    if (*a.num_counted == 0) return;   // every item is counted in seg_main
    const int64_t nitems = *a.num_items;
    const int cshift = a.tile_shift > kCLog ? a.tile_shift - kCLog : 0;   // log2(chunks per item)
    const int64_t work = nitems << cshift;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * 4;
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * 4 + wave_id(); w < work; w += nw) {
        const int64_t it = w >> cshift;
        const int64_t c = w & ((int64_t{1} << cshift) - 1);
        const SegItem &d = a.items[it];
        if (a.mode == IXP_MODE_PARTITION && (d.kind & (kOwnRows | 4))) continue;   // counted in seg_main
        if (Pred::kRow && (d.kind & kPacked)) continue;   // (seg_count_packed)
        const int64_t b = d.base + (c << kCLog);
        if (b >= d.hi) continue;
        WT chunk;
        if (a.keep) chunk.template load<false>(a.keys, a.n, b, d.lo, d.hi, pred.at_row(d.row), !Pred::kUsesFlags, 0, lane);
        else chunk.load(a.keys, a.n, b, d.lo, d.hi, pred.at_row(d.row), !Pred::kUsesFlags, 0, lane);
        const uint32_t cnt = chunk.wave_count();
        if (lane == 0 && cnt) atomicAdd(a.counts + it, static_cast<unsigned long long>(cnt));
    }
}

// ------------------------------------------------------------------- scan --
// Exclusive scan of the item counts into prefix[0..num_items]; items of rows
// counted in place (partition, one item) count 0.  Workgroups take chunks of
// 8192 counts in ticket order, scan them (8 per thread, DPP wave scans, LDS)
// and chain the chunks with a decoupled look-back.
__global__ __launch_bounds__(1024) void seg_scan_items_kernel(SegArgs a) {
    __shared__ int64_t lds[16];
    __shared__ int64_t sh[2];
    constexpr int kPer = kScanChunk / 1024;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    if (*a.num_counted == 0) return;   // no item needs the prefix
    const int64_t nitems = *a.num_items;
    const int64_t nchunks = (nitems + kScanChunk - 1) / kScanChunk;
    if (tid == 0) sh[0] = atomicAdd(a.scan_ticket, 1u);
    __syncthreads();
    const int64_t c = sh[0];
    if (nitems == 0) {
        if (c == 0 && tid == 0) a.prefix[0] = 0;
        return;
    }
    if (c >= nchunks) return;
    const int64_t i0 = c * kScanChunk + static_cast<int64_t>(tid) * kPer;
    int64_t v[kPer];
    int64_t sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        v[j] = i0 + j < nitems ? static_cast<int64_t>(a.counts[i0 + j]) : 0;
        sum += v[j];
    }
    int64_t tot;
    const int64_t in_chunk = block_exclusive_scan<16>(sum, lds, &tot);
    if (wave == 0) {
        // a chunk holds at most 8192 * 16384 = 2^27 trues: below 2^32, as the
        // look-back's aggregates must be; 64 of them may pass 2^32, so the
        // window sums are taken wide
        if (lane == 0 && c > 0) desc_store(a.scan_desc + c, kStA | static_cast<uint64_t>(tot));
        const int64_t e = c == 0 ? 0 : lookback<4, true>(a.scan_desc, c, 0, a.err);
        if (lane == 0) {
            desc_store(a.scan_desc + c, kStP | static_cast<uint64_t>(e + tot));
            sh[1] = e;
            if (c == nchunks - 1) a.prefix[nitems] = e + tot;
        }
    }
    __syncthreads();
    int64_t acc = sh[1] + in_chunk;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (i0 + j < nitems) a.prefix[i0 + j] = acc;
        acc += v[j];
    }
}

// One thread per item: output bases from the prefix.  Partition: a row of
// several items gets o_k + (trues before the item in the row) for its trues
// and o_k + T_k + (falses before the item in the row) for its falses; the
// row's first item writes T_k.  Filter: kept elements of all rows are packed,
// so the base is the global prefix; the first item writes the row's T_k.
__global__ __launch_bounds__(256) void seg_item_bases_kernel(SegArgs a) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (*a.num_counted == 0) return;
    const int64_t nitems = *a.num_items;
    if (i >= nitems) return;
    const SegItem d = a.items[i];
    const int64_t k = d.row;
    const int64_t i0 = d.first, i1 = i0 + d.fbase;   // the row's items (not of a packed item)
    if (a.mode == IXP_MODE_PARTITION) {
        if (d.kind & (kOwnRows | 4)) return;   // finished by the main kernel
        const int64_t ok = a.offsets[k];
        const int64_t p0 = a.prefix[i0];
        const int64_t before = a.prefix[i] - p0;
        const int64_t tk = a.prefix[i1] - p0;
        a.items[i].tbase = ok + before;
        a.items[i].fbase = ok + tk + (d.lo - ok - before);
        if (i == i0 && a.seg_split) a.seg_split[k] = tk;
    } else {
        a.items[i].tbase = a.prefix[i];
        a.items[i].fbase = 0;
        if (i == i0 && a.seg_split && !(d.kind & kPacked)) a.seg_split[k] = a.prefix[i1] - a.prefix[i0];
    }
}

// ------------------------------------------------------------------- main --
// Count exchange of a row of 2..kSibMax items, run by one wave of the
// workgroup that holds item `it` (true count `tcount`): publishes the count,
// then reads the row's items' counts 64 at a time (lane j of chunk c reads
// item first + 64c + j).  Unpublished ones are polled again, kSibPolls times
// at most over the whole row; those still missing are counted from their
// keys here.  Leaves in out[0] the trues of the row before item `it` and in
// out[1] the row's total T_k.  Every count is exact whoever computes it, so
// the result does not depend on which items published in time.
template <class Pred>
__device__ __forceinline__ void row_counts(const SegArgs &a, const Pred &pred, int64_t it,
                                           const SegItem &d, uint32_t tcount, int lane,
                                           uint32_t *out) {
    uint64_t *cnt = reinterpret_cast<uint64_t *>(a.counts);
    const int nsib = (d.kind >> 8) & 0xffff;
    const int me = static_cast<int>(it - d.first);
    const bool nowait = a.row_sync == IXP_ROW_SYNC_NOWAIT;
    if (lane == 0) desc_store(cnt + it, kCntReady | tcount);
    uint32_t polls = kSibPolls;
    uint32_t before = 0, total = 0;
    for (int c0 = 0; c0 < nsib; c0 += kWave) {
        const int j = c0 + lane;
        const bool mine = j < nsib;
        uint64_t w = j == me ? (kCntReady | tcount) : 0;
        if (!nowait && mine && j != me) w = desc_load(cnt + d.first + j);
        uint64_t missing = ballot(mine && !(w & kCntReady));
        while (missing && !nowait && polls > 0) {
            --polls;
            __builtin_amdgcn_s_sleep(1);
            if (mine && !(w & kCntReady)) w = desc_load(cnt + d.first + j);   // this lane's bit of `missing`
            missing = ballot(mine && !(w & kCntReady));
        }
        while (missing) {
            // a plain strided loop: few registers are free while the tile is held
            const int b = __builtin_ctzll(missing);
            missing &= missing - 1;
            const auto p = pred.at_row(d.row);
            const SegItem &s = a.items[d.first + c0 + b];
            const int64_t shi = s.hi;
            uint32_t c = 0;
            for (int64_t q0 = s.lo; q0 < shi; q0 += 4 * kWave) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t q = q0 + u * kWave + lane;
                    if (q < shi) {
                        const uint32_t key = Pred::kUsesFlags ? 0u : a.keys[q];
                        uint8_t f = 0;
                        if constexpr (Pred::kUsesFlags) f = p.flags[q];
                        c += p(key, f) ? 1u : 0u;
                    }
                }
            }
            c = wave_sum_u32(c);
            if (lane == b) w = kCntReady | c;
        }
        const uint32_t v = mine ? static_cast<uint32_t>(w & kValMask) : 0u;
        before += wave_sum_u32(j < me ? v : 0u);
        total += wave_sum_u32(v);
    }
    if (lane == 0) {
        out[0] = before;
        out[1] = total;
    }
}

// ----------------------------------------------------------- packed items --
// A packed item holds the whole short rows [row, first): every row's elements
// and T_k are inside it, so it waits for no other item.  Where the rows start
// is kept as one bit per position of the tile (`head`); an element finds its
// row's start and the next row's start in its own 32-bit word or in a table of
// the nearest start before / after each word, so no per-element search is
// needed and rows may be of any size.  Window and limit (3/4 and 1/4 of the
// tile) let every such item fit its tile while filling three quarters of it.
// About 60 vector instructions an element and the chain of barriers bound it,
// not memory: 2^25 int32 keys in rows of 128 on average take 110 us in
// seg_main (3.7 TB/s), where a workgroup per row took 700 us.  Keeping keys and
// counts in one LDS array and 5 waves per SIMD (58 -> 35 us for 8 million keys in
// 250,000 rows) is what helped; 6 or 7 waves, or as many workgroups as fit that
// take many items each, changed nothing or were slower.
constexpr int kPackThreads = 256, kPackRows = 4;
constexpr int kPackTile = kPackThreads * kPackRows * 4;
constexpr int kPackWords = kPackTile / 32;
static_assert(kPackWords == 2 * kWave, "one wave scans the words");

struct PackLds {
    uint32_t head[kPackWords];
    int16_t before[kPackWords];   // last start before the word (or the item's first)
    int16_t after[kPackWords];    // first start after the word, or the item's end
};
// At a start: the trues of the tile before the row, and before the next row;
// at the item's end: all its trues.  One word per position: the same LDS
// holds each row's word before, and the keys in output order after.
struct PackRow {
    uint16_t trues, next;
};

// Start bits, and with `words` each row's word at its start; then (tables) the
// nearest starts of every word.  All threads of the workgroup; ends with a
// barrier.  `ok`, `oe` are the offsets of row d.row + tid and the one after it
// (equal past the last row), loaded by the caller beside the keys.
template <class WordOf>
__device__ __forceinline__ void pack_starts(const SegArgs &a, const SegItem &d, PackLds &p, uint32_t *words,
                                            const WordOf &word_of, bool tables, int64_t ok, int64_t oe) {
    const int tid = threadIdx.x;
    for (int64_t k = d.row + tid;;) {
        if (oe > ok) {
            const uint32_t l = static_cast<uint32_t>(ok - d.base);
            atomicOr(p.head + (l >> 5), 1u << (l & 31));
            if (words) words[l] = word_of(k);
        }
        k += kPackThreads;
        if (k >= d.first) break;
        ok = a.offsets[k];
        oe = a.offsets[k + 1];
    }
    __syncthreads();
    if (!tables) return;
    if (wave_id() == 0) {
        const int lane = tid & (kWave - 1);
        const uint32_t w0 = p.head[2 * lane], w1 = p.head[2 * lane + 1];
        const int f0 = w0 ? 64 * lane + __builtin_ctz(w0) : kPackTile;
        const int f1 = w1 ? 64 * lane + 32 + __builtin_ctz(w1) : kPackTile;
        const int l0 = w0 ? 64 * lane + 31 - __builtin_clz(w0) : -1;
        const int l1 = w1 ? 64 * lane + 63 - __builtin_clz(w1) : -1;
        const int last = l1 > l0 ? l1 : l0, next = f0 < f1 ? f0 : f1;
        // the nearest lanes on both sides with a start in their words
        const uint64_t any = ballot((w0 | w1) != 0);
        const uint64_t under = any & ((1ull << lane) - 1), over = any & ~((2ull << lane) - 1);
        int before = __shfl(last, under ? 63 - __builtin_clzll(under) : 0, kWave);
        int after = __shfl(next, over ? __builtin_ctzll(over) : 0, kWave);
        const int lo = static_cast<int>(d.lo - d.base), end = static_cast<int>(d.hi - d.base);
        if (!under || before < lo) before = lo;
        if (!over || after > end) after = end;
        p.before[2 * lane] = static_cast<int16_t>(before);
        p.before[2 * lane + 1] = static_cast<int16_t>(l0 >= 0 ? l0 : before);
        p.after[2 * lane + 1] = static_cast<int16_t>(after);
        p.after[2 * lane] = static_cast<int16_t>(f1 < kPackTile ? f1 : after);
    }
    __syncthreads();
}

// The starts around the element at position l of the tile, from its word.
__device__ __forceinline__ int row_start(uint32_t w, int l, int before) {
    const uint32_t m = w & ((2u << (l & 31)) - 1u);
    return m ? (l | 31) - __builtin_clz(m) : before;
}
__device__ __forceinline__ int row_end(uint32_t w, int l, int after) {
    const uint32_t m = w & ~((2u << (l & 31)) - 1u);
    return m ? (l & ~31) + __builtin_ctz(m) : after;
}

// Loads a packed item's keys and evaluates the predicate of each element's row.
// A wave past the item's end (`live` false) loads nothing.  Leaves the offsets
// of row d.row + tid and the one after it in ok, oe (equal past the last row).
template <class T, class Pred>
__device__ __forceinline__ void pack_load(const SegArgs &a, const Pred &pred, const SegItem &d, PackLds &p,
                                          uint32_t *words, bool tables, bool need_keys, bool live, T &tile, int wave,
                                          int lane, int64_t &ok, int64_t &oe) {
    const int tid = threadIdx.x;
    if (tid < kPackWords) p.head[tid] = 0;
    const int64_t k = d.row + tid;
    ok = k < d.first ? a.offsets[k] : 0;
    oe = k < d.first ? a.offsets[k + 1] : 0;
    if (!live) {
#pragma unroll
        for (int r = 0; r < kPackRows; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) tile.key[r][q] = 0;
    } else if constexpr (Pred::kRow) {
        tile.load(a.keys, a.n, d.base, d.lo, d.hi, PredNone{}, true, wave, lane);
    } else {
        tile.load(a.keys, a.n, d.base, d.lo, d.hi, pred, need_keys, wave, lane);
    }
    __syncthreads();   // head is clear
    if constexpr (Pred::kRow) {
        pack_starts(a, d, p, words, [&](int64_t r) { return pred.row_word(r); }, true, ok, oe);
        if (!live) return;
        int l0 = wave * T::kPerWave + lane * 4;
        asm volatile("" : "+v"(l0));   // (see packed_item)
#pragma unroll
        for (int r = 0; r < kPackRows; ++r) {
            const int lr = l0 + r * (kWave * 4);
            const uint32_t w = p.head[lr >> 5];
            int s = row_start(w, lr, p.before[lr >> 5]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q > 0) s = (w >> ((lr & 31) + q)) & 1u ? lr + q : s;
                const bool f = tile.valid(r, q) && pred.in_row(tile.key[r][q], words[s]);
                tile.fbits |= static_cast<uint32_t>(f) << (r * 4 + q);
            }
            __builtin_amdgcn_sched_barrier(0);   // a row's LDS words at a time, to hold few registers
        }
    } else {
        pack_starts(a, d, p, nullptr, [](int64_t) { return 0u; }, tables, ok, oe);
    }
}

// One packed item (see seg_main).  Its keys are staged in output order and
// leave as one run.  `stage` (kPackTile + 1 words) holds in turn the rows'
// words, the rows' counts and the keys.  Every barrier is reached by the whole
// workgroup.
template <class Pred, int MODE, class Idx>
__device__ __forceinline__ void packed_item(const SegArgs &a, const Pred &pred, const SegItem &d, PackLds &p,
                                            uint32_t *stage, uint32_t *wtot, int wave, int lane) {
    using T = Tile<kPackThreads, kPackRows, 4, uint32_t>;
    const int tid = threadIdx.x;
    Idx *out_idx = static_cast<Idx *>(a.out_idx);
    const bool part = MODE == IXP_MODE_PARTITION;
    const bool live = T::wave_live(d.base, d.lo, d.hi, wave);
    T tile;
    int64_t ok, oe;
    pack_load(a, pred, d, p, stage, part, a.need_keys != 0, live, tile, wave, lane, ok, oe);
    uint32_t pre[kPackRows];   // trues of the tile before this lane's group of a row
    uint32_t wt = 0;
#pragma unroll
    for (int r = 0; r < kPackRows; ++r) {
        uint32_t below = 0, row_total = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t m = ballot(tile.flag(r, q));
            below += rank_below(m);
            row_total += static_cast<uint32_t>(__builtin_popcountll(m));
        }
        pre[r] = wt + below;
        wt += row_total;
    }
    if (lane == 0) wtot[wave] = wt;
    __syncthreads();
    uint32_t tbefore = 0, tcount = 0;
#pragma unroll
    for (int w = 0; w < T::kWaves; ++w) {
        const uint32_t v = wtot[w];
        tbefore += w < wave ? v : 0u;
        tcount += v;
    }
    PackRow *at = reinterpret_cast<PackRow *>(stage);
    // opaque: the positions, words and masks derived from it would otherwise be
    // kept in registers across the whole item loop
    int l0 = wave * T::kPerWave + lane * 4;
    uint32_t fb = tile.fbits;
    asm volatile("" : "+v"(l0), "+v"(fb));
    const int end = static_cast<int>(d.hi - d.base);
    auto rank = [&](int r, int q) {   // trues of the tile before element (r, q)
        return pre[r] + static_cast<uint32_t>(__builtin_popcount((fb >> (4 * r)) & ((1u << q) - 1u)));
    };
#pragma unroll
    for (int r = 0; r < kPackRows; ++r) {
        pre[r] += tbefore;
        const int lr = l0 + r * (kWave * 4);
        const uint32_t h = live ? (p.head[lr >> 5] >> (lr & 31)) & 0xFu : 0u;
        if (h) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((h >> q) & 1u) at[lr + q].trues = static_cast<uint16_t>(rank(r, q));
        }
    }
    if (tid == 0) at[end].trues = static_cast<uint16_t>(tcount);
    __syncthreads();
    if (a.seg_split) {
        for (int64_t k = d.row + tid; k < d.first; k += kPackThreads) {
            if (oe > ok) a.seg_split[k] = at[oe - d.base].trues - at[ok - d.base].trues;   // (empty: seg_count)
            if (k + kPackThreads < d.first) {
                ok = a.offsets[k + kPackThreads];
                oe = a.offsets[k + kPackThreads + 1];
            }
        }
    }
    if (part) {
#pragma unroll
        for (int r = 0; r < kPackRows; ++r) {
            const int lr = l0 + r * (kWave * 4);
            const uint32_t w = p.head[lr >> 5];
            const uint32_t h = live ? (w >> (lr & 31)) & 0xFu : 0u;
            if (h) {
                const int after = p.after[lr >> 5];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((h >> q) & 1u) at[lr + q].next = at[row_end(w, lr + q, after)].trues;
            }
        }
        __syncthreads();
    }
    asm volatile("" : "+v"(l0), "+v"(fb));
    uint32_t to[kPackRows][4];   // place of the key in the stage
#pragma unroll
    for (int r = 0; r < kPackRows; ++r) {
        const int lr = l0 + r * (kWave * 4);
        const int64_t p0 = d.base + lr;
        const uint32_t w = p.head[lr >> 5];
        int s = part ? row_start(w, lr, p.before[lr >> 5]) : 0;
        const uint32_t h = (w >> (lr & 31)) & 0xFu;
        const uint32_t vm = (tile.vbits >> (4 * r)) & 0xFu;
        Idx v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t e = rank(r, q);
            const bool f = (fb >> (4 * r + q)) & 1u;
            if (MODE == IXP_MODE_PARTITION) {
                if (q > 0) s = (h >> q) & 1u ? lr + q : s;
                const uint32_t row = stage[s];   // (its two counts by one load)
                // a true: the row's start + its trues before; a false: after all of them
                const uint32_t t = s + e - (row & 0xFFFFu), u = static_cast<uint32_t>(lr + q) - e + (row >> 16);
                to[r][q] = f ? t : u;
                v[q] = static_cast<Idx>(d.base + to[r][q]);
            } else {
                to[r][q] = e;
                v[q] = static_cast<Idx>(f ? d.tbase + e : -1);
            }
        }
        if (vm) {
            if (out_idx) store_idx_group<4, Idx>(out_idx, p0, v, vm);
            if (a.flags_out) {
                const uint32_t fl = (h & 1u) | (h & 2u) << 7 | (h & 4u) << 14 | (h & 8u) << 21;
                if (vm == 0xFu) {
                    stream_store(reinterpret_cast<uint32_t *>(a.flags_out + p0), fl);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if ((vm >> q) & 1u) a.flags_out[p0 + q] = static_cast<uint8_t>(fl >> (8 * q));
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (a.out_keys) {
        __syncthreads();   // the rows' counts are read
#pragma unroll
        for (int r = 0; r < kPackRows; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (((MODE == IXP_MODE_PARTITION ? tile.vbits : fb) >> (4 * r + q)) & 1u)
                    stage[to[r][q]] = tile.key[r][q];
        __syncthreads();
        if (part)
            write_run<kPackThreads>(stage, static_cast<uint32_t>(d.lo - d.base), static_cast<uint32_t>(d.hi - d.lo),
                                    d.lo, a.out_keys, a.n, tid);
        else
            write_run<kPackThreads>(stage, 0, tcount, d.tbase, a.out_keys, a.n, tid);
    }
}

// Filter with a predicate of the row number: the trues of the packed items,
// one workgroup per item (seg_count's waves do not know their rows).
template <class Pred>
__global__ __launch_bounds__(kPackThreads) void seg_count_packed_kernel(SegArgs a, Pred pred) {
    using T = Tile<kPackThreads, kPackRows, 4, uint32_t>;
    __shared__ PackLds p;
    __shared__ uint32_t words[kPackTile];
    const int wave = wave_id(), lane = threadIdx.x & (kWave - 1);
    const int64_t nitems = *a.num_items;
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const SegItem d = a.items[it];
        if (!(d.kind & kPacked)) continue;
        T tile;
        int64_t ok, oe;
        const bool live = T::wave_live(d.base, d.lo, d.hi, wave);
        pack_load(a, pred, d, p, words, true, true, live, tile, wave, lane, ok, oe);
        const uint32_t cnt = tile.wave_count();
        if (lane == 0 && cnt) atomicAdd(a.counts + it, static_cast<unsigned long long>(cnt));
        __syncthreads();   // LDS is reused by the next item
    }
}

// Workgroups take items round-robin (item = blockIdx.x + k * gridDim.x: no
// shared queue counter, whose serialised atomics would cost ~10 ns per
// item); a grid smaller than the item count makes them persistent.  Wave 0
// prefetches the next item's 64-byte descriptor, one 8-byte word per lane,
// while the workgroup processes the current one.
//
// Each wave owns the LDS run of its own elements: right after ranking them it
// places its keys there, trues first, then falses, each in input order.  The
// keys then leave the registers before the workgroup's count exchange, and
// after it the wave writes its two runs straight to their places in the
// output (its trues follow the trues of the waves before it, its falses the
// falses before it).  No other wave reads that LDS run, so it needs no
// barrier of its own; the one at the top of the loop separates items.
// With PACK some items are packed ones (256 x 4 tiles only).
template <int BLOCK, int ROWS, class Pred, int MODE, class Idx, bool PACK = false>
__global__ __launch_bounds__(BLOCK, PACK ? 5 : 1) void seg_main_kernel(SegArgs a, Pred pred) {
    static_assert(!PACK || (BLOCK == kPackThreads && ROWS == kPackRows), "packed tiles");
    using T = Tile<BLOCK, ROWS, 4, uint32_t>;
    constexpr int kTile = T::kSize;
    constexpr int kPerWave = T::kPerWave;
    constexpr int kWords = sizeof(SegItem) / 8;
    static_assert(sizeof(SegItem) % 8 == 0 && kWords <= kWave, "descriptor words");
    __shared__ uint32_t stage[kTile + (PACK ? 1 : 0)];
    __shared__ uint32_t wtot[T::kWaves];
    __shared__ int64_t sh_desc[kWords];
    __shared__ int64_t sh_item;
    __shared__ uint32_t sh_row[2];

    const int tid = threadIdx.x;
    const int wave = wave_id();
    const int lane = tid & (kWave - 1);
    const int64_t nitems = *a.num_items;
    Idx *out_idx = static_cast<Idx *>(a.out_idx);
    const int64_t *words = reinterpret_cast<const int64_t *>(a.items);
    uint32_t *wstage = stage + wave * kPerWave;

    int64_t next = blockIdx.x, next_word = 0;
    auto prefetch = [&]() {
        if (lane < kWords && next < nitems) next_word = (words + next * kWords)[static_cast<uint32_t>(lane)];
    };
    if (wave == 0) prefetch();

    for (;;) {
        if (wave == 0) {
            if (lane < kWords) sh_desc[lane] = next_word;
            if (lane == 0) sh_item = next;
        }
        __syncthreads();
        const int64_t it = sh_item;
        if (it >= nitems) break;
        SegItem d;
        {
            // the record is the same for every lane: keep it in scalar registers
            int64_t w[kWords];
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                const uint64_t x = static_cast<uint64_t>(sh_desc[k]);
                const uint32_t xl = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
                const uint32_t xh = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
                w[k] = static_cast<int64_t>((static_cast<uint64_t>(xh) << 32) | xl);
            }
            __builtin_memcpy(&d, w, sizeof(SegItem));
        }
        if (wave == 0) {   // overlaps with this item
            next = it + gridDim.x;
            prefetch();
        }
        if constexpr (PACK) {
            if (d.kind & kPacked) {
                __shared__ PackLds pk;
                packed_item<Pred, MODE, Idx>(a, pred, d, pk, stage, wtot, wave, lane);
                continue;
            }
        }
        const int64_t lo = d.lo, hi = d.hi, base = d.base;
        const int32_t span = static_cast<int32_t>(hi - lo);
        // offsets from lo (a tile spans < 2^31): the wave's first element,
        // where its valid elements start, and how many there are
        const int32_t wl0 = static_cast<int32_t>(base - lo) + wave * kPerWave;
        const int32_t vbeg = wl0 < 0 ? 0 : (wl0 < span ? wl0 : span);
        const int32_t wl1 = wl0 + kPerWave;
        const int32_t vend = wl1 < 0 ? 0 : (wl1 < span ? wl1 : span);
        const uint32_t wvalid = static_cast<uint32_t>(vend - vbeg);

        T tile;
        const bool live = T::wave_live(base, lo, hi, wave);   // waves past a short item load nothing
        if (live) {
            if (MODE == IXP_MODE_FILTER && a.keep)
                tile.template load<false>(a.keys, a.n, base, lo, hi, pred.at_row(d.row), a.need_keys != 0, wave, lane);
            else
                tile.load(a.keys, a.n, base, lo, hi, pred.at_row(d.row), a.need_keys != 0, wave, lane);
        } else {
            // defined keys on every path: an undefined value here would keep
            // the last item's keys in registers across the whole loop
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) tile.key[r][q] = 0;
        }

        // rowpre[r]: trues of this wave before this lane's group of row r
        uint32_t rowpre[ROWS];
        uint32_t wt = 0;   // trues of this wave (uniform)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            uint32_t below = 0, row_total = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t m = ballot(tile.flag(r, q));
                below += rank_below(m);
                row_total += static_cast<uint32_t>(__builtin_popcountll(m));
            }
            rowpre[r] = wt + below;
            wt += row_total;
        }
        // rank of element (r, q) among the wave's trues (for a false: trues before it)
        auto wrank = [&](int r, int q) -> uint32_t {
            const uint32_t g = (tile.fbits >> (4 * r)) & ((1u << q) - 1u);
            return rowpre[r] + static_cast<uint32_t>(__builtin_popcount(g));
        };
        const int32_t l0 = wl0 + lane * 4;   // offset from lo of (row 0, q 0)

        if (a.out_keys && live) {
            // Every element is written, without a branch: a valid one at its
            // place in the run (falses too in filter mode, where they are
            // never read), an invalid one at lw mod kPerWave.  lw counts from
            // the wave's first valid element, so the invalid elements fill
            // exactly the slots past the valid ones, one each.
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t rw = wrank(r, q);
                    const uint32_t lw = static_cast<uint32_t>(l0 + r * (kWave * 4) + q - vbeg);
                    const uint32_t at = tile.flag(r, q) ? rw : wt + (lw - rw);
                    wstage[tile.valid(r, q) ? at : (lw & (kPerWave - 1))] = tile.key[r][q];
                }
            }
        }

        if (lane == 0) wtot[wave] = wt;
        __syncthreads();
        uint32_t tbefore = 0, tcount = 0;   // trues of the waves before this one; of the tile
#pragma unroll
        for (int w = 0; w < T::kWaves; ++w) {
            const uint32_t v = wtot[w];
            tbefore += w < wave ? v : 0u;
            tcount += v;
        }

        int64_t tbase = d.tbase, fbase = d.fbase;
        if (MODE == IXP_MODE_PARTITION && (d.kind & 1)) {
            tbase = lo;
            fbase = lo + tcount;
            if (tid == 0 && a.seg_split) a.seg_split[d.row] = tcount;
        }
        if (MODE == IXP_MODE_PARTITION && (d.kind & 4)) {
            if (wave == 0) row_counts(a, pred, it, d, tcount, lane, sh_row);
            __syncthreads();
            const int64_t ok = d.tbase, before = sh_row[0], tk = sh_row[1];
            tbase = ok + before;
            fbase = ok + tk + (lo - ok - before);
            if (tid == 0 && (d.kind & 2) && a.seg_split) a.seg_split[d.row] = tk;
        }
        const bool first = (d.kind & 2) != 0;

        if (out_idx || a.flags_out) {
            // Opaque copies of the flag words: every per-element bit and rank
            // below is recomputed from them, where the compiler would
            // otherwise keep the staging's sixteen of each in registers
            // through the exchange.
            uint32_t fb = tile.fbits, vb = tile.vbits;
            asm volatile("" : "+v"(fb), "+v"(vb));
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int64_t p0 = T::pos(base, wave, r, lane, 0);
                const int32_t lr = l0 + r * (kWave * 4);   // offset from lo of q = 0
                const uint32_t fr = (fb >> (4 * r)) & 0xFu;
                const uint32_t vm = (vb >> (4 * r)) & 0xFu;
                // the descriptor byte 1 sits at l == 0, i.e. at q = -lr
                const uint32_t fl = (first && lr <= 0 && lr > -4) ? 1u << (8 * -lr) : 0u;
                Idx v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int32_t l = lr + q;
                    const uint32_t rt = tbefore + rowpre[r] +   // rank among the tile's trues
                                        static_cast<uint32_t>(__builtin_popcount(fr & ((1u << q) - 1u)));
                    const uint32_t rf = static_cast<uint32_t>(l) - rt;
                    const bool f = (fr >> q) & 1u;
                    if (MODE == IXP_MODE_PARTITION)
                        v[q] = static_cast<Idx>(f ? tbase + rt : fbase + rf);
                    else
                        v[q] = static_cast<Idx>(f ? tbase + rt : -1);
                }
                if (vm) {
                    if (out_idx) store_idx_group<4, Idx>(out_idx, p0, v, vm);
                    if (a.flags_out) {
                        if (vm == 0xFu) {
                            stream_store(reinterpret_cast<uint32_t *>(a.flags_out + p0), fl);
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if ((vm >> q) & 1u)
                                    a.flags_out[p0 + q] = static_cast<uint8_t>(fl >> (8 * q));
                        }
                    }
                }
            }
        }
        if (a.out_keys) {
            // this wave's own LDS run, written by this wave before the exchange
            write_run<kWave>(wstage, 0, wt, tbase + tbefore, a.out_keys, a.n, lane);
            if (MODE == IXP_MODE_PARTITION) {
                const uint32_t fbefore = static_cast<uint32_t>(vbeg) - tbefore;   // falses before this wave
                write_run<kWave>(wstage, wt, wvalid - wt, fbase + fbefore, a.out_keys, a.n, lane);
            }
        }
    }
}

// ------------------------------------------------------------ shape tools --
// The segment helpers of Section 2.1 as device outputs, over the item records
// (each item knows its row; the first item of a non-empty row starts at o_k):
//   mkII:       ii[i] = k for o_k <= i < o_k + s_k;
//   mkSgmDescr: out[o_k] = xs[k] for every non-empty row k, 0 elsewhere.
// Workgroup w takes items w, w + grid, ...; consecutive threads write
// consecutive 16-byte groups of the item's aligned middle (when `out` is
// 16-byte aligned), and single elements at its ends.
// A packed item's rows start where its start bits say; each start also holds
// its row's number (from the item's first row), from which mkII fills and
// mkSgmDescr looks xs up.
template <int TOOL, class Out>
__device__ __forceinline__ void fill_packed(const SegArgs &a, const SegItem &d, Out *out, const int64_t *xs,
                                            bool vec_ok, PackLds &p, uint32_t *val) {
    constexpr int kV = 16 / sizeof(Out);   // elements per 16-byte group
    typedef Out vec_t __attribute__((ext_vector_type(kV)));
    const int tid = threadIdx.x;
    if (tid < kPackWords) p.head[tid] = 0;
    const int64_t k = d.row + tid;
    const int64_t ok = k < d.first ? a.offsets[k] : 0, oe = k < d.first ? a.offsets[k + 1] : 0;
    __syncthreads();
    pack_starts(a, d, p, val, [&](int64_t r) { return static_cast<uint32_t>(r - d.row); }, TOOL == 0, ok, oe);
    const int end = static_cast<int>(d.hi - d.base), lo = static_cast<int>(d.lo - d.base);
    for (int l = tid * kV; l < end; l += kPackThreads * kV) {   // (base is a multiple of 32)
        const uint32_t w = p.head[l >> 5];
        const int before = TOOL == 0 ? p.before[l >> 5] : 0;
        vec_t v;
#pragma unroll
        for (int q = 0; q < kV; ++q) {
            if (TOOL == 0) v[q] = static_cast<Out>(d.row + val[row_start(w, l + q, before)]);
            else v[q] = (w >> ((l + q) & 31)) & 1u ? static_cast<Out>(xs[d.row + val[l + q]]) : Out{0};
        }
        if (vec_ok && l >= lo && l + kV <= end) {
            stream_store(reinterpret_cast<vec_t *>(out + d.base + l), v);
        } else {
#pragma unroll
            for (int q = 0; q < kV; ++q)
                if (l + q >= lo && l + q < end) stream_store(out + d.base + l + q, v[q]);
        }
    }
    __syncthreads();   // the LDS is the next item's
}

template <int TOOL, class Out, bool PACK>
__global__ __launch_bounds__(256) void seg_fill_kernel(SegArgs a, Out *out, const int64_t *xs) {
    constexpr int kV = 16 / sizeof(Out);   // elements per 16-byte group
    typedef Out vec_t __attribute__((ext_vector_type(kV)));
    if (*a.err != 0) return;
    const int64_t nitems = *a.num_items;
    const bool vec_ok = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const SegItem d = a.items[it];
        if constexpr (PACK) {
            if (d.kind & kPacked) {
                __shared__ PackLds pk;
                __shared__ uint32_t val[kPackTile];
                fill_packed<TOOL, Out>(a, d, out, xs, vec_ok, pk, val);
                continue;
            }
        }
        const bool first = (d.kind & 2) != 0;
        const Out fill = TOOL == 0 ? static_cast<Out>(d.row) : static_cast<Out>(0);
        const Out head = TOOL == 0 ? fill : static_cast<Out>(first ? xs[d.row] : 0);
        // [v0, v1): whole groups; the rest element by element
        int64_t v0 = (d.lo + kV - 1) / kV * kV, v1 = d.hi / kV * kV;
        if (!vec_ok || v0 >= v1) v0 = v1 = d.hi;
        for (int64_t i = d.lo + threadIdx.x; i < v0; i += 256) stream_store(out + i, i == d.lo ? head : fill);
        for (int64_t i = v1 + threadIdx.x; i < d.hi; i += 256) stream_store(out + i, i == d.lo ? head : fill);
        vec_t fv;
#pragma unroll
        for (int q = 0; q < kV; ++q) fv[q] = fill;
        for (int64_t g = v0 / kV + threadIdx.x; g < v1 / kV; g += 256) {
            vec_t v = fv;
            if (TOOL == 1 && g * kV == d.lo) v[0] = head;
            stream_store(reinterpret_cast<vec_t *>(out) + g, v);
        }
    }
}

// Row offsets, item offsets and item records: one launch for up to
// kShapeFusedRows rows, else three.
int launch_shape(const SegArgs &a, hipStream_t st) {
    if (a.m <= kShapeFusedRows) {
        // few rows of many items: several workgroups share a group of 256 rows
        // (each rescans the shape), as far as they fit the chip at once
        const int64_t groups = ceil_div(a.m > 0 ? a.m : 1, 256);
        const int64_t want = a.n / (a.tile * groups * kShapeThreads) + 1, fit = device_cus() / groups;
        const int64_t parts = want < fit ? want : (fit > 0 ? fit : 1);
        IXP_LAUNCH("seg_shape", seg_shape_kernel, dim3(static_cast<uint32_t>(groups), static_cast<uint32_t>(parts)),
                   dim3(kShapeThreads), 0, st, a);
        return launch_status();
    }
    const dim3 chunks(static_cast<uint32_t>(a.nchunks));
    IXP_LAUNCH("seg_sizes", seg_sizes_kernel, chunks, dim3(kSetupThreads), 0, st, a);
    IXP_LAUNCH("seg_rows", seg_rows_kernel, chunks, dim3(kSetupThreads), 0, st, a);
    IXP_LAUNCH("seg_records", seg_records_kernel, dim3(static_cast<uint32_t>(ceil_div(a.m, kSetupThreads))),
               dim3(kSetupThreads), 0, st, a);
    return launch_status();
}

template <int TOOL, class Out>
int launch_tool(const SegArgs &a, Out *out, const int64_t *xs, hipStream_t st) {
    if (launch_shape(a, st) != IXP_OK) return IXP_EHIP;
    const int64_t cap = static_cast<int64_t>(device_cus()) * 16;
    const int64_t grid = a.max_items < cap ? (a.max_items > 0 ? a.max_items : 1) : cap;
    const char *name = TOOL == 0 ? "seg_mk_ii" : "seg_mk_sgm_descr";
    if (a.short_max > 0)
        IXP_LAUNCH(name, (seg_fill_kernel<TOOL, Out, true>), dim3(static_cast<uint32_t>(grid)), dim3(256), 0, st, a, out,
                   xs);
    else
        IXP_LAUNCH(name, (seg_fill_kernel<TOOL, Out, false>), dim3(static_cast<uint32_t>(grid)), dim3(256), 0, st, a, out,
                   xs);
    return launch_status();
}

// ----------------------------------------------------------------- launch --
constexpr int64_t kPackMinRows = 2048, kToolPackMinRows = 8192;   // (see packs)
struct SegGeom {
    int block, rows, wgs_per_cu, row_sync;
    int64_t pack_rows = kPackMinRows;
    int64_t tile() const { return static_cast<int64_t>(block) * rows * 4; }
};

// Every supported tile is a power of two (block and rows are).
bool geom_supported(const SegGeom &g) {
    const bool b = g.block == 256 || g.block == 512 || g.block == 1024;
    const bool r = g.rows == 2 || g.rows == 4 || g.rows == 8;
    return b && r && g.tile() <= 16384 && g.wgs_per_cu >= 1 && g.wgs_per_cu <= 64 &&
           (g.row_sync == IXP_ROW_SYNC_COUNT || g.row_sync == IXP_ROW_SYNC_NOWAIT ||
            g.row_sync == IXP_ROW_SYNC_WAIT);
}

SegGeom geom_from(const ixp_tuning *t) {
    // default: the tiling the autotuner picks for 10^4 log-normal rows
    SegGeom g{256, 4, 64, IXP_ROW_SYNC_AUTO};
    if (t) {
        if (t->block) g.block = t->block;
        if (t->rows) g.rows = t->rows;
        g.wgs_per_cu = t->wgs_per_cu > 0 ? t->wgs_per_cu : 0;
        g.row_sync = t->row_sync;
    }
    if (g.wgs_per_cu == 0) {
        // as many workgroups per CU as the LDS tile and 32 waves allow, at most 8
        const int64_t by_lds = (160 * 1024) / (g.tile() * 4 + 1024);
        const int64_t by_waves = 32 / (g.block / 64);
        int64_t w = by_lds < by_waves ? by_lds : by_waves;
        if (w > 8) w = 8;
        g.wgs_per_cu = static_cast<int>(w < 1 ? 1 : w);
    }
    // the in-kernel count exchange pays when a row's items run at the same
    // time, i.e. on oversubscribed grids that the hardware fills in order
    if (g.row_sync == IXP_ROW_SYNC_AUTO) g.row_sync = g.wgs_per_cu >= 16 ? IXP_ROW_SYNC_WAIT : IXP_ROW_SYNC_COUNT;
    return g;
}

// Of the segment helpers.
SegGeom tool_geom() {
    SegGeom g = geom_from(nullptr);
    g.pack_rows = kToolPackMinRows;
    return g;
}

template <int BLOCK, int ROWS, class Pred, bool PACK = false>
int launch_main_geom(const SegArgs &a, const Pred &p, int mode, int idx_t, int grid, hipStream_t st) {
    if (mode == IXP_MODE_PARTITION) {
        if (idx_t == IXP_I32)
            IXP_LAUNCH("seg_main_partition", (seg_main_kernel<BLOCK, ROWS, Pred, IXP_MODE_PARTITION, int32_t, PACK>),
                       dim3(grid), dim3(BLOCK), 0, st, a, p);
        else
            IXP_LAUNCH("seg_main_partition", (seg_main_kernel<BLOCK, ROWS, Pred, IXP_MODE_PARTITION, int64_t, PACK>),
                       dim3(grid), dim3(BLOCK), 0, st, a, p);
    } else {
        if (idx_t == IXP_I32)
            IXP_LAUNCH("seg_main_filter", (seg_main_kernel<BLOCK, ROWS, Pred, IXP_MODE_FILTER, int32_t, PACK>),
                       dim3(grid), dim3(BLOCK), 0, st, a, p);
        else
            IXP_LAUNCH("seg_main_filter", (seg_main_kernel<BLOCK, ROWS, Pred, IXP_MODE_FILTER, int64_t, PACK>),
                       dim3(grid), dim3(BLOCK), 0, st, a, p);
    }
    return launch_status();
}

template <class Pred>
int launch_main(const SegArgs &a, const Pred &p, const SegGeom &g, int mode, int idx_t, hipStream_t st) {
    const int64_t cap = static_cast<int64_t>(device_cus()) * g.wgs_per_cu;
    const int grid = static_cast<int>(a.max_items < cap ? a.max_items : cap);
    if (a.short_max > 0) {
        // about the number of items; a workgroup without one still costs its dispatch
        const int64_t want = a.n / (kPackTile / 2) + device_cus() * 4;
        return launch_main_geom<kPackThreads, kPackRows, Pred, true>(a, p, mode, idx_t,
                                                                     static_cast<int>(want < grid ? want : grid), st);
    }
#define IXP_SEG_GEOM(B, R) \
    if (g.block == B && g.rows == R) return launch_main_geom<B, R, Pred>(a, p, mode, idx_t, grid, st);
    IXP_SEG_GEOM(256, 2)
    IXP_SEG_GEOM(256, 4)
    IXP_SEG_GEOM(256, 8)
    IXP_SEG_GEOM(512, 2)
    IXP_SEG_GEOM(512, 4)
    IXP_SEG_GEOM(512, 8)
    IXP_SEG_GEOM(1024, 2)
    IXP_SEG_GEOM(1024, 4)
#undef IXP_SEG_GEOM
    return IXP_EUNSUPPORTED;
}

template <class Pred>
int launch_all(const SegArgs &a, const Pred &p, const SegGeom &g, int mode, int idx_t, hipStream_t st) {
    if (launch_shape(a, st) != IXP_OK) return IXP_EHIP;
    const int cus = device_cus();
    // one wave per chunk of the largest possible item list, capped
    const int64_t chunk_waves = a.max_items * (a.tile > (1 << kSegCountLog) ? a.tile >> kSegCountLog : 1);
    const int64_t cblocks = ceil_div(chunk_waves, 4) < static_cast<int64_t>(cus) * 16
                                ? ceil_div(chunk_waves, 4) : static_cast<int64_t>(cus) * 16;
    IXP_LAUNCH("seg_count", (seg_count_kernel<Pred>), dim3(static_cast<uint32_t>(cblocks)), dim3(256), 0,
               st, a, p);
    if constexpr (Pred::kRow) {
        if (a.short_max > 0 && mode == IXP_MODE_FILTER) {
            const int64_t cap = static_cast<int64_t>(cus) * 16;
            IXP_LAUNCH("seg_count_packed", (seg_count_packed_kernel<Pred>),
                       dim3(static_cast<uint32_t>(a.max_items < cap ? a.max_items : cap)), dim3(kPackThreads), 0, st,
                       a, p);
        }
    }
    IXP_LAUNCH("seg_scan_items", seg_scan_items_kernel,
               dim3(static_cast<uint32_t>(ceil_div(a.max_items > 0 ? a.max_items : 1, kScanChunk))), dim3(1024), 0,
               st, a);
    const uint32_t iblocks = static_cast<uint32_t>(ceil_div(a.max_items, 256));
    IXP_LAUNCH("seg_item_bases", seg_item_bases_kernel, dim3(iblocks), dim3(256), 0, st, a);
    if (launch_status() != IXP_OK) return IXP_EHIP;
    return launch_main(a, p, g, mode, idx_t, st);
}

// Short rows are packed when rows have at most kPackMean elements on average
// (the sizes themselves are known on the device only) and the tile is the
// default one.  A packed item costs more per element than a row of its own, rows
// above 1024 elements cut the packed items short, and the kernel that knows packed
// items runs fewer waves (a partition of long rows alone: 1.1 to 1.2 of the other
// one's time).  16,000 rows, item per row / packed, us, by the rows' mean: partition of
// log-normal sizes 256: 79 / 50, 512: 85 / 68, 768: 92 / 84, 1100: 99 / 100; of equal ones
// 512: 78 / 57, 768: 84 / 68; of uniform ones from 0 512: 84 / 57, 640: 88 / 81, 768: 90 / 92, 1100:
// 96 / 105; 60,000 rows, uniform 768: 245 / 243.  So the line is where uniform sizes break
// even; rows that are either 1100 or below 60 elements do at 448 (16,000 rows 640: 89 / 100,
// 768: 92 / 106), the worst there is.
// Below kPackMinRows rows a workgroup per row fills the chip in a wave or two, and a
// few packed items leave it idle.  Rows of 128, partition / filter / filter by a
// predicate of the row / the helpers, an item per row against packed: 1000 rows
// 23.5, 25.3, 25.2, 35.6 / 23.2, 25.6, 31.4, 37.6 us; 2000 rows 24.2, 30.7, 30.4,
// 37.3 / 24.7, 26.0, 31.8, 39.1; 4000 rows 30.9, 38.9, 38.8, 41.9 / 25.3, 27.4,
// 33.3, 41.6.  The helpers alone, which only write, gain later (the
// descriptor, rows of 32: 4000 rows 14.7 / 15.5, 8192 rows 19.8 / 18.0, 16,000 rows 30.7 / 25.2).
// (The tuning cache's key, _packs_short_rows in ops.py, follows this.)
constexpr int64_t kPackMean = 768;
bool packs(int64_t n, int64_t m, const SegGeom &g) {
    return g.block == kPackThreads && g.rows == kPackRows && m >= g.pack_rows && n / m <= kPackMean &&
           n < (int64_t{1} << 42);
}

// With room for an item per row also where rows are packed: calls of fewer rows, of
// larger tiles and the helpers may take one, and a workspace sized once, for the
// largest call, serves them all.
size_t seg_workspace(int64_t n, int64_t m, const SegGeom &g) {
    const int64_t mi = seg_max_items(n, m, g.tile(), false);
    return kSegHeader + round_up(static_cast<size_t>(m + 1) * 8, 256) * 2 +
           round_up(static_cast<size_t>(mi) * sizeof(SegItem), 256) +
           round_up(static_cast<size_t>(mi + 1) * 8, 256) + round_up(static_cast<size_t>(mi) * 8, 256) +
           round_up(static_cast<size_t>(ceil_div(mi > 0 ? mi : 1, kScanChunk)) * 8, 256) +
           (m > kShapeFusedRows ? 4 * kShapeChunks * sizeof(int64_t) : 0);
}

void set_layout(int64_t n, int64_t m, const int64_t *d_shape, const SegGeom &g, void *ws, SegArgs *a);

int prepare(const void *keys, int32_t key_t, int64_t n, const int64_t *d_shape, int64_t m,
            const ixp_pred *pred, int32_t mode, void *out_keys, void *out_idx, int32_t idx_t,
            int64_t *d_seg_split, uint8_t *d_flags_out, const SegGeom &g, void *ws,
            size_t ws_bytes, SegArgs *a, HostPred *hp) {
    if (n < 0 || m < 0 || (m > 0 && !d_shape)) return IXP_EINVAL;
    if (m > 0x7FFFFFFFll) return IXP_EINVAL;
    if (mode != IXP_MODE_PARTITION && mode != IXP_MODE_FILTER) return IXP_EINVAL;
    if (idx_t != IXP_I32 && idx_t != IXP_I64) return IXP_EINVAL;
    if (idx_t == IXP_I32 && n > 0x7FFFFFFFll) return IXP_EINVAL;
    if (key_t != IXP_I32 && key_t != IXP_F32) return key_t == IXP_I64 ? IXP_EUNSUPPORTED : IXP_EINVAL;
    if (!geom_supported(g)) return IXP_EINVAL;
    int rc = check_pred(pred, key_t, hp, n);
    if (rc != IXP_OK) return rc;
    const bool need_keys = hp->kind != IXP_PRED_FLAGS || out_keys != nullptr;
    if (n > 0 && need_keys && !keys) return IXP_EINVAL;
    if (!ws || ws_bytes < seg_workspace(n, m, g)) return IXP_EWORKSPACE;
    const size_t isz = idx_t == IXP_I32 ? 4 : 8;
    // vector groups of 4 elements: keys, indices and flag bytes must be
    // aligned to a whole group
    if (!aligned(keys, 16) || !aligned(out_keys, 4) || !aligned(out_idx, 4 * isz) ||
        !aligned(d_flags_out, 4) || !aligned(d_shape, 8) || !aligned(d_seg_split, 8) ||
        !aligned(ws, 16))
        return IXP_EINVAL;
    if (hp->kind == IXP_PRED_FLAGS && !aligned(hp->flags, 4)) return IXP_EINVAL;
    if (hp->kind == IXP_PRED_LT_ROW && !aligned(hp->row_s, 4)) return IXP_EINVAL;
    set_layout(n, m, d_shape, g, ws, a);
    a->keys = static_cast<const uint32_t *>(keys);
    a->out_keys = static_cast<uint32_t *>(out_keys);
    a->out_idx = out_idx;
    a->seg_split = d_seg_split;
    a->flags_out = d_flags_out;
    a->mode = mode;
    a->need_keys = need_keys ? 1 : 0;
    a->row_sync = g.row_sync;
    // A filter counts every item first; plain loads leave part of the keys in the
    // Infinity Cache for the main kernel.  Nontemporal / plain, rows of 5000, 32-bit
    // indices: 8 10^6 45.3 / 43.2 us, 2 10^7 75.9 / 70.1, 5 10^7 144 / 131, 8 10^7 215 / 211,
    // 10^8 260 / 262; 64-bit indices: 5 10^7 201 / 226.
    a->keep = mode == IXP_MODE_FILTER && idx_t == IXP_I32 && n >= (int64_t{1} << 22) && n <= int64_t{5} << 24;
    return IXP_OK;
}

// Shape-derived part of the arguments: the workspace layout (row offsets,
// item records, item counts and their scan) for n elements in m rows.
void set_layout(int64_t n, int64_t m, const int64_t *d_shape, const SegGeom &g, void *ws, SegArgs *a) {
    char *w = static_cast<char *>(ws);
    const size_t rows_bytes = round_up(static_cast<size_t>(m + 1) * 8, 256);
    a->keys = nullptr;
    a->n = n;
    a->shape = d_shape;
    a->m = m;
    a->out_keys = nullptr;
    a->out_idx = nullptr;
    a->seg_split = nullptr;
    a->flags_out = nullptr;
    a->err = reinterpret_cast<int32_t *>(w + 4);
    a->num_items = reinterpret_cast<int64_t *>(w + 8);
    a->num_counted = reinterpret_cast<unsigned long long *>(w + 24);
    a->offsets = reinterpret_cast<int64_t *>(w + kSegHeader);
    a->item_off = reinterpret_cast<int64_t *>(w + kSegHeader + rows_bytes);
    a->items = reinterpret_cast<SegItem *>(w + kSegHeader + 2 * rows_bytes);
    const bool pack = packs(n, m, g);
    a->max_items = seg_max_items(n, m, g.tile(), pack);
    a->prefix = reinterpret_cast<int64_t *>(
        w + kSegHeader + 2 * rows_bytes + round_up(static_cast<size_t>(a->max_items) * sizeof(SegItem), 256));
    a->counts = reinterpret_cast<unsigned long long *>(
        reinterpret_cast<char *>(a->prefix) + round_up(static_cast<size_t>(a->max_items + 1) * 8, 256));
    a->scan_desc = reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(a->counts) +
                                                round_up(static_cast<size_t>(a->max_items) * 8, 256));
    const int64_t nd = ceil_div(a->max_items > 0 ? a->max_items : 1, kScanChunk);
    a->csum = reinterpret_cast<int64_t *>(reinterpret_cast<char *>(a->scan_desc) +
                                          round_up(static_cast<size_t>(nd) * 8, 256));
    a->citems = a->csum + kShapeChunks;
    a->ccounted = a->citems + kShapeChunks;
    a->cbad = a->ccounted + kShapeChunks;
    a->chunk_rows = ceil_div(ceil_div(m, int64_t{1} << kChunkPackShift), kShapeChunks) << kChunkPackShift;
    a->nchunks = m > 0 ? ceil_div(m, a->chunk_rows) : 0;
    a->short_max = pack ? g.tile() / 4 : 0;
    a->scan_ticket = reinterpret_cast<uint32_t *>(w + 16);
    a->tile = g.tile();
    a->tile_shift = 0;
    while ((int64_t{1} << a->tile_shift) < a->tile) ++a->tile_shift;
    a->mode = IXP_MODE_PARTITION;
    a->keep = 0;
    a->need_keys = 0;
    a->row_sync = g.row_sync;
}

int run(const SegArgs &a, const HostPred &hp, const SegGeom &g, int mode, int idx_t, hipStream_t st) {
    switch (hp.kind) {
    case IXP_PRED_MOD_EQ: return launch_all(a, mod_eq_pred(hp.d, hp.r), g, mode, idx_t, st);
    case IXP_PRED_LT: return launch_all(a, PredLt{hp.s}, g, mode, idx_t, st);
    case IXP_PRED_LT_ROW: return launch_all(a, PredLtRow{hp.row_s, 0.f}, g, mode, idx_t, st);
    case IXP_PRED_MOD_ROW: return launch_all(a, mod_row_pred(hp.d), g, mode, idx_t, st);
    default: return launch_all(a, PredFlags{hp.flags}, g, mode, idx_t, st);
    }
}

}  // namespace
}  // namespace ixp

using namespace ixp;

struct ixp_graph_s {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

extern "C" size_t ixp_segmented_workspace(int64_t n, int64_t m, const ixp_tuning *tune) {
    if (n < 0 || m < 0) return 0;
    const SegGeom g = geom_from(tune);
    if (!geom_supported(g)) return 0;
    return seg_workspace(n, m, g);
}

extern "C" int ixp_segmented_partition(const void *keys, int32_t key_t, int64_t n,
                                       const int64_t *d_shape, int64_t m, const ixp_pred *pred,
                                       int32_t mode, void *out_keys, void *out_idx, int32_t idx_t,
                                       int64_t *d_seg_split, uint8_t *d_flags_out,
                                       const ixp_tuning *tune, void *ws, size_t ws_bytes,
                                       void *stream) {
    const SegGeom g = geom_from(tune);
    SegArgs a;
    HostPred hp;
    int rc = prepare(keys, key_t, n, d_shape, m, pred, mode, out_keys, out_idx, idx_t, d_seg_split,
                     d_flags_out, g, ws, ws_bytes, &a, &hp);
    if (rc != IXP_OK) return rc;
    return run(a, hp, g, mode, idx_t, as_stream(stream));
}

extern "C" int ixp_tune_segmented(const void *keys, int32_t key_t, int64_t n,
                                  const int64_t *d_shape, int64_t m, const ixp_pred *pred,
                                  int32_t mode, void *out_keys, void *out_idx, int32_t idx_t,
                                  int64_t *d_seg_split, uint8_t *d_flags_out, void *ws,
                                  size_t ws_bytes, int32_t reps, ixp_tuning *best, float *best_ms,
                                  void *stream) {
    if (!best) return IXP_EINVAL;
    if (reps < 1) reps = 1;
    hipStream_t st = as_stream(stream);
    static const int kCands[][2] = {{256, 2}, {256, 4}, {256, 8}, {512, 2}, {512, 4}, {512, 8},
                                    {1024, 2}, {1024, 4}};
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return IXP_EHIP;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return IXP_EHIP; }
    float best_t = -1.f;
    int rc_out = IXP_EUNSUPPORTED;
    // row sync matters in partition mode only
    const int nsync = mode == IXP_MODE_PARTITION ? 2 : 1;
    for (int sync = 0; sync < nsync; ++sync)
    for (const auto &c : kCands) {
        // persistent grids (as many workgroups per CU as fit, or one fewer),
        // and oversubscribed grids of 16, 32 or 64 per CU, where most
        // workgroups take a single item and the hardware overlaps them
        for (int wpc = 0; wpc < 5; ++wpc) {
            ixp_tuning t{c[0], c[1], 0, sync == 0 ? IXP_ROW_SYNC_WAIT : IXP_ROW_SYNC_COUNT};
            SegGeom g = geom_from(&t);
            if (wpc == 1) g.wgs_per_cu = g.wgs_per_cu > 1 ? g.wgs_per_cu - 1 : 1;
            if (wpc == 2) g.wgs_per_cu = 16;
            if (wpc == 3) g.wgs_per_cu = 64;
            if (wpc == 4) g.wgs_per_cu = 32;
            t.wgs_per_cu = g.wgs_per_cu;
            SegArgs a;
            HostPred hp;
            if (prepare(keys, key_t, n, d_shape, m, pred, mode, out_keys, out_idx, idx_t, d_seg_split,
                        d_flags_out, g, ws, ws_bytes, &a, &hp) != IXP_OK)
                continue;
            if (run(a, hp, g, mode, idx_t, st) != IXP_OK) continue;   // warm-up
            (void)hipEventRecord(e0, st);
            int rc = IXP_OK;
            for (int r = 0; r < reps && rc == IXP_OK; ++r) rc = run(a, hp, g, mode, idx_t, st);
            (void)hipEventRecord(e1, st);
            if (rc != IXP_OK || hipEventSynchronize(e1) != hipSuccess) continue;
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            ms /= static_cast<float>(reps);
            if (best_t < 0.f || ms < best_t) {
                best_t = ms;
                *best = t;
                rc_out = IXP_OK;
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (best_ms) *best_ms = best_t;
    return rc_out;
}

extern "C" int ixp_segmented_graph_create(ixp_graph *out, const void *keys, int32_t key_t, int64_t n,
                                          const int64_t *d_shape, int64_t m, const ixp_pred *pred,
                                          int32_t mode, void *out_keys, void *out_idx,
                                          int32_t idx_t, int64_t *d_seg_split,
                                          uint8_t *d_flags_out, const ixp_tuning *tune, void *ws,
                                          size_t ws_bytes) {
    if (!out) return IXP_EINVAL;
    *out = nullptr;
    const SegGeom g = geom_from(tune);
    SegArgs a;
    HostPred hp;
    int rc = prepare(keys, key_t, n, d_shape, m, pred, mode, out_keys, out_idx, idx_t, d_seg_split,
                     d_flags_out, g, ws, ws_bytes, &a, &hp);
    if (rc != IXP_OK) return rc;
    (void)device_cus();   // cache the CU count outside the capture
    hipStream_t cs = nullptr;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return IXP_EHIP;
    auto *gr = new (std::nothrow) ixp_graph_s;
    if (!gr) { (void)hipStreamDestroy(cs); return IXP_ENOMEM; }
    rc = IXP_EHIP;
    if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        const int lrc = run(a, hp, g, mode, idx_t, cs);
        hipGraph_t graph = nullptr;
        const hipError_t ec = hipStreamEndCapture(cs, &graph);
        if (lrc == IXP_OK && ec == hipSuccess && graph) {
            if (hipGraphInstantiate(&gr->exec, graph, nullptr, nullptr, 0) == hipSuccess) {
                gr->graph = graph;
                rc = IXP_OK;
            } else {
                (void)hipGraphDestroy(graph);
            }
        } else {
            rc = lrc != IXP_OK ? lrc : IXP_EHIP;
            if (graph) (void)hipGraphDestroy(graph);
        }
    }
    (void)hipStreamDestroy(cs);
    if (rc != IXP_OK) {
        delete gr;
        return rc;
    }
    *out = gr;
    return IXP_OK;
}

extern "C" int ixp_graph_launch(ixp_graph g, void *stream) {
    if (!g || !g->exec) return IXP_EINVAL;
    return hipGraphLaunch(g->exec, as_stream(stream)) == hipSuccess ? IXP_OK : IXP_EHIP;
}

extern "C" int ixp_graph_destroy(ixp_graph g) {
    if (!g) return IXP_EINVAL;
    int rc = IXP_OK;
    if (g->exec && hipGraphExecDestroy(g->exec) != hipSuccess) rc = IXP_EHIP;
    if (g->graph && hipGraphDestroy(g->graph) != hipSuccess) rc = IXP_EHIP;
    delete g;
    return rc;
}

extern "C" size_t ixp_mk_ii_workspace(int64_t n, int64_t m) {
    if (n < 0 || m < 0) return 0;
    return seg_workspace(n, m, tool_geom());
}

extern "C" int ixp_mk_ii(const int64_t *d_shape, int64_t m, int64_t n, void *out, int32_t out_t, void *ws,
                         size_t ws_bytes, void *stream) {
    if (n < 0 || m < 0 || m > 0x7FFFFFFFll || (m > 0 && !d_shape) || (n > 0 && !out)) return IXP_EINVAL;
    if (out_t != IXP_I32 && out_t != IXP_I64) return IXP_EINVAL;
    const SegGeom g = tool_geom();
    if (!ws || ws_bytes < seg_workspace(n, m, g)) return IXP_EWORKSPACE;
    if (!aligned(d_shape, 8) || !aligned(out, out_t == IXP_I32 ? 4 : 8) || !aligned(ws, 16)) return IXP_EINVAL;
    SegArgs a;
    set_layout(n, m, d_shape, g, ws, &a);
    hipStream_t st = as_stream(stream);
    return out_t == IXP_I32 ? launch_tool<0>(a, static_cast<int32_t *>(out), nullptr, st)
                            : launch_tool<0>(a, static_cast<int64_t *>(out), nullptr, st);
}

extern "C" int ixp_mk_sgm_descr(const int64_t *d_shape, int64_t m, int64_t n, const int64_t *d_xs,
                                int64_t *d_out, void *ws, size_t ws_bytes, void *stream) {
    if (n < 0 || m < 0 || m > 0x7FFFFFFFll || (m > 0 && (!d_shape || !d_xs)) || (n > 0 && !d_out))
        return IXP_EINVAL;
    const SegGeom g = tool_geom();
    if (!ws || ws_bytes < seg_workspace(n, m, g)) return IXP_EWORKSPACE;
    if (!aligned(d_shape, 8) || !aligned(d_xs, 8) || !aligned(d_out, 8) || !aligned(ws, 16)) return IXP_EINVAL;
    SegArgs a;
    set_layout(n, m, d_shape, g, ws, &a);
    return launch_tool<1>(a, d_out, d_xs, as_stream(stream));
}
