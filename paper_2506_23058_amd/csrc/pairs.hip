// pairs.hip -- get_smallest_pairs (Sections 5.4 and 6, maximal matching) in one
// call: H[v] = min(neutral, the least is[k] with es[k] = v), keep the entries k
// with H[es[k]] == is[k], and filter es and is by them, in input order.
//
// Step by step (hist with min, flags, filter, two scatters) every entry costs an
// atomic minimum and a read at a random place of H, each of which moves a cache
// line: 2.5 and 1.7 ms for 2^26 entries over 2^24 vertices.  Here the entries are
// routed to one workgroup per bucket of consecutive vertices, whose part of H
// sits in LDS, and everything in memory is read and written in order:
//   pairs_bucket -- one workgroup per chunk of 16384 entries: ranks them by
//                   bucket in LDS and writes, bucket by bucket, a 32-bit record
//                   (vertex in the bucket, place in the chunk) and the id, with
//                   a table of where each bucket starts in the chunk;
//   pairs_reduce -- one workgroup per bucket: reads its run of every chunk
//                   twice, first for the minima, then to set the top bit of the
//                   records that attain them; writes its part of H;
//   pairs_mark   -- one workgroup per chunk: the kept entries' bitmap and count;
//   pairs_scan   -- one workgroup: exclusive scan of the chunks' counts;
//   pairs_compact - one workgroup per chunk: copies the kept entries.
// 28 bytes per entry in pairs_bucket, 24 to 28 in pairs_reduce, 4 in pairs_mark,
// 16 to 32 in pairs_compact; for 2^26 entries over 2^24 vertices 356, 649, 46, 5 and
// 260 us by rocprofv3 (5.3, 2.7, 5.8, - and 5.1 TB/s); the call takes 1255 us, step by
// step 5130.  (The times of variants below are those of HIP events, without a
// profiler: 601 us for the same pairs_reduce.)
#include "device.hpp"
#include "host.hpp"

namespace ixp {
namespace {

constexpr int kPairChunkLog = 14;
constexpr int kPairChunk = 1 << kPairChunkLog;
constexpr int kPairThreads = 1024;
constexpr int kPairMaxBuckets = 2048;
constexpr int kPairMaxShift = 14;            // vertices per bucket: 128 KiB of LDS
constexpr uint32_t kKept = 1u << 31;
constexpr int kPairWords = kPairChunk / 32;
static_assert(kPairMaxShift + kPairChunkLog <= 31, "record fields below the kept bit");

struct PairArgs {
    const int64_t *es, *is;
    int64_t m, n_verts, neutral;
    int64_t *hist, *es_out, *is_out, *split;
    uint32_t *rec;      // [nchunks * kPairChunk] kept bit | place << shift | vertex in the bucket
    int64_t *ids;       // [nchunks * kPairChunk]
    uint16_t *ctab;     // [(nb + 1) * nchunks]: bucket starts per chunk; last row: chunk totals
    uint32_t *kept;     // [nchunks * kPairWords] bitmap of the kept entries
    int64_t *count;     // [nchunks] kept entries, then those before the chunk
    int64_t nchunks;
    int32_t shift, nb;
};

__global__ __launch_bounds__(kPairThreads) void pairs_bucket_kernel(PairArgs a) {
    constexpr int kPer = kPairChunk / kPairThreads;
    __shared__ int64_t lds[kPairChunk];   // ids in record order; before them, the records
    __shared__ uint32_t bstart[kPairMaxBuckets + 1];
    __shared__ uint32_t wtot[kPairThreads / kWave];
    uint32_t *stage = reinterpret_cast<uint32_t *>(lds);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int nb = a.nb;
    const int64_t c = xcd_tile(blockIdx.x, a.nchunks);
    const int64_t e0 = c << kPairChunkLog;
    const int live = static_cast<int>(a.m - e0 < kPairChunk ? a.m - e0 : kPairChunk);
    for (int b = tid; b <= nb; b += kPairThreads) bstart[b] = 0;
    __syncthreads();
    int64_t v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = u * kPairThreads + tid;
        v[u] = i < live ? __builtin_nontemporal_load(a.es + e0 + i) : -1;
    }
    // meta: bucket << 14 | rank in the bucket (a chunk holds at most 2^14), or ~0
    uint32_t meta[kPer], off[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const bool in = 0 <= v[u] && v[u] < a.n_verts;
        off[u] = static_cast<uint32_t>(v[u]) & ((1u << a.shift) - 1);
        meta[u] = ~0u;
        if (in) {
            const uint32_t b = static_cast<uint32_t>(v[u] >> a.shift);
            meta[u] = (b << kPairChunkLog) | atomicAdd(bstart + b, 1u);
        }
    }
    int64_t id[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = u * kPairThreads + tid;
        id[u] = i < live ? __builtin_nontemporal_load(a.is + e0 + i) : 0;
    }
    __syncthreads();
    {   // exclusive scan of the nb + 1 counts (the last is 0: it becomes the chunk's total)
        const int per = (nb + kPairThreads) / kPairThreads;
        const int b0 = tid * per;
        uint32_t mine = 0;
        for (int j = 0; j < per; ++j)
            if (b0 + j <= nb) mine += bstart[b0 + j];
        const uint32_t inc = wave_scan_u32(mine);
        if (lane == kWave - 1) wtot[wave] = inc;
        __syncthreads();
        uint32_t run = inc - mine;
        for (int w = 0; w < wave; ++w) run += wtot[w];
        for (int j = 0; j < per; ++j) {
            if (b0 + j <= nb) {
                const uint32_t cnt = bstart[b0 + j];
                bstart[b0 + j] = run;
                run += cnt;
            }
        }
    }
    __syncthreads();
    for (int b = tid; b <= nb; b += kPairThreads)
        a.ctab[static_cast<int64_t>(b) * a.nchunks + c] = static_cast<uint16_t>(bstart[b]);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (meta[u] != ~0u) {
            meta[u] = bstart[meta[u] >> kPairChunkLog] + (meta[u] & (kPairChunk - 1));   // its place now
            stage[meta[u]] = (static_cast<uint32_t>(u * kPairThreads + tid) << a.shift) | off[u];
        }
    }
    __syncthreads();
    const uint32_t total = bstart[nb];
    uint32_t *rec = a.rec + e0;
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    // (past the total up to a whole quad the stage holds anything, and nobody reads it)
    for (uint32_t j = tid; 4 * j < total; j += kPairThreads)
        *(reinterpret_cast<v4 *>(rec) + j) = *(reinterpret_cast<const v4 *>(stage) + j);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (meta[u] != ~0u) lds[meta[u]] = id[u];
    __syncthreads();
    typedef int64_t i64x2 __attribute__((ext_vector_type(2)));
    int64_t *ids = a.ids + e0;
    for (uint32_t j = tid; 2 * j < total; j += kPairThreads)
        *(reinterpret_cast<i64x2 *>(ids) + j) = *(reinterpret_cast<const i64x2 *>(lds) + j);
}

// Neighbouring buckets' runs share cache lines, so the buckets of one XCD are
// consecutive.  A run is 16384 / nb entries on average (8 with 2048 buckets), so a
// wave takes the runs of 16 chunks as one sequence of positions, 64 a row: a bit
// marks where a run starts, and a position's run is the number of such bits up to
// it.  (With 16 lanes to a run half of them were idle, and longer runs took a loop
// of their own: 7.7e6 entries over 6.2e5 vertices 61.6 us, so 39.4; 3e7 over 3e7
// 336 us, so 324; 2^26 over 2^24 597, now 601.)  Past that the lines bound it: the
// XCD's workgroups drift apart, and of 64 chunks to a wave too few of the shared
// lines stay in its L2 (2^26 entries over 2^24 vertices: 64 chunks 650 us, 8 642,
// 16 601).  With 1024 buckets of 128 KiB one workgroup fits a CU, and the kernel
// takes 964 us.
template <int SHIFT>   // at least a.shift
__global__ __launch_bounds__(kPairThreads) void pairs_reduce_kernel(PairArgs a) {
    constexpr int kWaves = kPairThreads / kWave, kUnroll = 4, kRows = 32, kRuns = 16;
    __shared__ uint64_t heads[kWaves][kRows];   // where runs start, among kRows * 64 positions
    __shared__ uint32_t places[kWaves][kWave];
    __shared__ int64_t lds[1 << SHIFT];   // this bucket's part of H
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int64_t b = xcd_tile(blockIdx.x, a.nb);
    const int64_t v0 = b << a.shift;
    const int width = static_cast<int>(a.n_verts - v0 < (int64_t{1} << a.shift) ? a.n_verts - v0
                                                                                : (int64_t{1} << a.shift));
    const uint32_t vmask = (1u << a.shift) - 1;
    for (int i = tid; i < width; i += kPairThreads) lds[i] = a.neutral;
    __syncthreads();
    const uint16_t *rs = a.ctab + b * a.nchunks, *re = rs + a.nchunks;
    // few chunks are dealt to all waves
    const int64_t each = ceil_div(a.nchunks, kWaves);
    const int runs = each < kRuns ? static_cast<int>(each) : kRuns;
    auto pass = [&](auto &&take) {
        for (int64_t cb = static_cast<int64_t>(wave) * runs; cb < a.nchunks; cb += kWaves * runs) {
            const int64_t c = cb + lane;
            const bool live = lane < runs && c < a.nchunks;
            const uint32_t s = live ? rs[c] : 0u, n = live ? re[c] - s : 0u;
            const uint32_t inc = wave_scan_u32(n), start = inc - n;
            const uint32_t total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), kWave - 1));
            // of the non-empty runs in turn: place of the run's first entry minus its position
            const uint64_t any = ballot(n > 0);
            if (n > 0) places[wave][rank_below(any)] = (static_cast<uint32_t>(lane) << kPairChunkLog) + s - start;
            uint32_t *rec = a.rec + (cb << kPairChunkLog);
            const int64_t *ids = a.ids + (cb << kPairChunkLog);
            int before = -1;   // runs that start before the row, minus 1
            for (uint32_t w0 = 0; w0 < total; w0 += kRows * kWave) {
                if (lane < kRows) heads[wave][lane] = 0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (n > 0 && start - w0 < static_cast<uint32_t>(kRows * kWave))
                    atomicOr(reinterpret_cast<unsigned long long *>(&heads[wave][(start - w0) >> 6]),
                             1ull << (start & 63));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (int r = 0; r < kRows && w0 + r * kWave < total; r += kUnroll) {
                    uint32_t at[kUnroll], x[kUnroll];
                    int64_t id[kUnroll];
                    const uint32_t p = w0 + r * kWave + lane;
#pragma unroll
                    for (int u = 0; u < kUnroll; ++u) {
                        const uint64_t m = readlane_u64(heads[wave][r + u], 0);
                        const int j = before + static_cast<int>(m & 1) + static_cast<int>(rank_below(m >> 1));
                        before += __builtin_popcountll(m);
                        at[u] = places[wave][j] + p + u * kWave;
                    }
#pragma unroll
                    for (int u = 0; u < kUnroll; ++u) {
                        const bool in = p + u * kWave < total;
                        x[u] = in ? rec[at[u]] : 0u;
                        id[u] = in ? ids[at[u]] : 0;
                    }
#pragma unroll
                    for (int u = 0; u < kUnroll; ++u)
                        if (p + u * kWave < total) take(rec + at[u], x[u], id[u]);
                }
            }
        }
    };
    pass([&](uint32_t *, uint32_t r, int64_t id) {
        atomicMin(reinterpret_cast<long long *>(lds) + (r & vmask), static_cast<long long>(id));
    });
    __syncthreads();
    pass([&](uint32_t *at, uint32_t r, int64_t id) {
        if (lds[r & vmask] == id) *at = r | kKept;
    });
    for (int i = tid; i < width; i += kPairThreads) stream_store(a.hist + v0 + i, lds[i]);
}

__global__ __launch_bounds__(256) void pairs_mark_kernel(PairArgs a) {
    __shared__ uint32_t bits[kPairWords];
    __shared__ uint32_t wsum[4];
    const int tid = threadIdx.x;
    const int64_t c = blockIdx.x;
    for (int w = tid; w < kPairWords; w += 256) bits[w] = 0;
    __syncthreads();
    const uint32_t total = a.ctab[static_cast<int64_t>(a.nb) * a.nchunks + c];
    const uint32_t *rec = a.rec + (c << kPairChunkLog);
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    constexpr int kLoads = 4;
    for (uint32_t j0 = tid; 4 * j0 < total; j0 += kLoads * 256) {
        v4 r[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const uint32_t j = j0 + k * 256;
            r[k] = 4 * j < total ? *(reinterpret_cast<const v4 *>(rec) + j) : v4{0, 0, 0, 0};
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = r[k][q], p = 4 * (j0 + k * 256) + q;
                if (p < total && (x & kKept)) {
                    const uint32_t i = (x & ~kKept) >> a.shift;
                    atomicOr(bits + (i >> 5), 1u << (i & 31));
                }
            }
    }
    __syncthreads();
    uint32_t n = 0;
    for (int w = tid; w < kPairWords; w += 256) {
        a.kept[c * kPairWords + w] = bits[w];
        n += static_cast<uint32_t>(__builtin_popcount(bits[w]));
    }
    n = wave_sum_u32(n);
    if ((tid & (kWave - 1)) == 0) wsum[wave_id()] = n;
    __syncthreads();
    if (tid == 0) a.count[c] = static_cast<int64_t>(wsum[0]) + wsum[1] + wsum[2] + wsum[3];
}

// One workgroup: exclusive scan of the chunks' counts in place, 8 per thread
// and step; the total is the number of kept pairs.
__global__ __launch_bounds__(1024) void pairs_scan_kernel(PairArgs a) {
    constexpr int kPer = 8;
    __shared__ int64_t wtot[16];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < a.nchunks; c0 += 1024 * kPer) {
        int64_t v[kPer], run = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t i = c0 + static_cast<int64_t>(tid) * kPer + k;
            v[k] = i < a.nchunks ? a.count[i] : 0;
            run += v[k];
        }
        const int64_t inc = wave_scan_i64(run);
        if (lane == kWave - 1) wtot[wave] = inc;
        __syncthreads();
        int64_t acc = carry + inc - run;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) acc += wtot[w];
            carry += wtot[w];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t i = c0 + static_cast<int64_t>(tid) * kPer + k;
            if (i < a.nchunks) a.count[i] = acc;
            acc += v[k];
        }
        __syncthreads();   // wtot is reused
    }
    if (tid == 0) *a.split = carry;
}

// A wave copies the kept entries of rows of 64: their places follow from the
// bitmap, consecutive kept lanes write consecutive elements.  kParts workgroups
// share a chunk, so that few chunks still fill the chip.
constexpr int kParts = 4;
__global__ __launch_bounds__(256) void pairs_compact_kernel(PairArgs a) {
    constexpr int kRows = 8, kPartRows = kPairChunk / kWave / kParts;
    __shared__ uint64_t mask[kPairChunk / kWave];
    __shared__ uint32_t before[kPairChunk / kWave];
    __shared__ uint32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int64_t c = blockIdx.x / kParts;
    const int part = blockIdx.x % kParts;
    static_assert(kPairChunk / kWave == 256, "a row of 64 per thread");
    {
        const uint64_t m = reinterpret_cast<const uint64_t *>(a.kept + c * kPairWords)[tid];
        const uint32_t n = static_cast<uint32_t>(__builtin_popcountll(m));
        const uint32_t inc = wave_scan_u32(n);
        if (lane == kWave - 1) wtot[wave] = inc;
        mask[tid] = m;
        __syncthreads();
        uint32_t acc = inc - n;
        for (int w = 0; w < wave; ++w) acc += wtot[w];
        before[tid] = acc;
    }
    __syncthreads();
    const int64_t e0 = c << kPairChunkLog, o0 = a.count[c];
    for (int r0 = part * kPartRows + wave * kRows; r0 < (part + 1) * kPartRows; r0 += 4 * kRows) {
        int64_t x[kRows], y[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const bool k = (mask[r0 + r] >> lane) & 1u;
            const int64_t i = e0 + (r0 + r) * kWave + lane;
            x[r] = k ? a.es[i] : 0;
            y[r] = k ? a.is[i] : 0;
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint64_t m = mask[r0 + r];
            if ((m >> lane) & 1u) {
                const int64_t o = o0 + before[r0 + r] + __builtin_popcountll(m & ((1ull << lane) - 1));
                a.es_out[o] = x[r];
                a.is_out[o] = y[r];
            }
        }
    }
}

// Bucket width: at most kPairMaxBuckets buckets.
int pair_shift(int64_t n_verts) {
    int s = 0;
    while (ceil_div(n_verts, int64_t{1} << s) > kPairMaxBuckets) ++s;
    return s;
}

struct PairLayout {
    size_t rec, ids, ctab, kept, count, total;
};
PairLayout pair_layout(int64_t m, int64_t n_verts) {
    const size_t nc = static_cast<size_t>(ceil_div(m, kPairChunk));
    const size_t nb = static_cast<size_t>(ceil_div(n_verts, int64_t{1} << pair_shift(n_verts)));
    PairLayout l;
    l.rec = 256;
    l.ids = l.rec + nc * kPairChunk * 4;
    l.ctab = l.ids + nc * kPairChunk * 8;
    l.kept = l.ctab + round_up((nb + 1) * nc * 2, 256);
    l.count = l.kept + nc * kPairWords * 4;
    l.total = l.count + round_up(nc * 8, 256);
    return l;
}

bool pairs_supported(int64_t m, int64_t n_verts) {
    return m > 0 && n_verts > 0 && n_verts <= static_cast<int64_t>(kPairMaxBuckets) << kPairMaxShift &&
           ceil_div(m, kPairChunk) <= 0x1FFFFFFF;
}

}  // namespace
}  // namespace ixp

using namespace ixp;

extern "C" size_t ixp_smallest_pairs_workspace(int64_t m, int64_t n_verts) {
    if (!pairs_supported(m, n_verts)) return 0;
    return pair_layout(m, n_verts).total;
}

extern "C" int ixp_smallest_pairs(const int64_t *es, const int64_t *is, int64_t m, int64_t n_verts, int64_t neutral,
                                  int64_t *d_hist, int64_t *es_out, int64_t *is_out, int64_t *d_split, void *ws,
                                  size_t ws_bytes, void *stream) {
    if (m < 0 || n_verts < 0) return IXP_EINVAL;
    if (!pairs_supported(m, n_verts)) return IXP_EUNSUPPORTED;
    if (!es || !is || !d_hist || !es_out || !is_out || !d_split) return IXP_EINVAL;
    if (!aligned(es, 8) || !aligned(is, 8) || !aligned(d_hist, 8) || !aligned(es_out, 8) || !aligned(is_out, 8) ||
        !aligned(d_split, 8) || !aligned(ws, 256))
        return IXP_EINVAL;
    const PairLayout l = pair_layout(m, n_verts);
    if (!ws || ws_bytes < l.total) return IXP_EWORKSPACE;
    char *w = static_cast<char *>(ws);
    PairArgs a;
    a.es = es;
    a.is = is;
    a.m = m;
    a.n_verts = n_verts;
    a.neutral = neutral;
    a.hist = d_hist;
    a.es_out = es_out;
    a.is_out = is_out;
    a.split = d_split;
    a.rec = reinterpret_cast<uint32_t *>(w + l.rec);
    a.ids = reinterpret_cast<int64_t *>(w + l.ids);
    a.ctab = reinterpret_cast<uint16_t *>(w + l.ctab);
    a.kept = reinterpret_cast<uint32_t *>(w + l.kept);
    a.count = reinterpret_cast<int64_t *>(w + l.count);
    a.nchunks = ceil_div(m, kPairChunk);
    a.shift = pair_shift(n_verts);
    a.nb = static_cast<int32_t>(ceil_div(n_verts, int64_t{1} << a.shift));
    hipStream_t st = as_stream(stream);
    const dim3 chunks(static_cast<uint32_t>(a.nchunks));
    IXP_LAUNCH("pairs_bucket", pairs_bucket_kernel, chunks, dim3(kPairThreads), 0, st, a);
    const dim3 buckets(static_cast<uint32_t>(a.nb));
    if (a.shift < kPairMaxShift)
        IXP_LAUNCH("pairs_reduce", pairs_reduce_kernel<kPairMaxShift - 1>, buckets, dim3(kPairThreads), 0, st, a);
    else
        IXP_LAUNCH("pairs_reduce", pairs_reduce_kernel<kPairMaxShift>, buckets, dim3(kPairThreads), 0, st, a);
    IXP_LAUNCH("pairs_mark", pairs_mark_kernel, chunks, dim3(256), 0, st, a);
    IXP_LAUNCH("pairs_scan", pairs_scan_kernel, dim3(1), dim3(1024), 0, st, a);
    IXP_LAUNCH("pairs_compact", pairs_compact_kernel, dim3(static_cast<uint32_t>(a.nchunks * kParts)), dim3(256), 0, st,
               a);
    return launch_status();
}
