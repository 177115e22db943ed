// sgmscan.hip -- sgmSum (Section 2.1, figure "Running Examples", right): the
// inclusive scan of int64 values under the lifted operator
//   (fx, vx) (+) (fy, vy) = (fx || fy, fy ? vy : vx + vy),
// i.e. a running sum that restarts at every flagged position.
//
// Reduce, scan, rescan over C <= 8192 chunks of whole 8192-element tiles:
//   reduce -- the aggregate of a chunk is (some flag, sum of the values from
//             its last flag on, that element included): one workgroup per
//             chunk finds the last flag from the flag bytes, then sums only
//             the values from there;
//   scan   -- one workgroup: exclusive scan of the C aggregates under the
//             lifted operator (8 per thread, DPP wave scans, LDS);
//   rescan -- one workgroup per chunk: a wave holds rows of 128 consecutive
//             elements, two per lane, and hands its last running sum to the
//             waves after it.
// No inter-workgroup waiting; the values from each chunk's last flag on are
// read twice, everything else once.
#include "device.hpp"
#include "host.hpp"

namespace ixp {
namespace {

constexpr int64_t kSgTile = 8192;      // chunks are multiples of this
constexpr int64_t kSgMaxChunks = 8192;

// The values are summed as unsigned words: the plain prefix sums used below pass
// segment borders and may wrap where no segment's sum does.
struct Pair {
    bool f;
    uint64_t v;
};

__device__ __forceinline__ Pair combine(Pair x, Pair y) { return Pair{x.f || y.f, y.f ? y.v : x.v + y.v}; }

struct SgArgs {
    const uint8_t *flags;
    const uint64_t *xs;
    uint64_t *out;
    int64_t n;
    int64_t chunk;      // elements per chunk, a multiple of kSgTile
    int64_t chunks;
    uint64_t *agg_v;    // [chunks] aggregate value, then exclusive prefix value
    int32_t *agg_f;     // [chunks] aggregate flag
};

// Reduce.  256 threads a chunk, so that eight chunks share a CU: with 1024 the
// chain flags, maximum, values, sum ran two chunks at a time (2^25 elements, a
// flag every 335: 39 us; now 14).
constexpr int kRedThreads = 256;

__device__ __forceinline__ int64_t block_max(int64_t x, int64_t *lds) {
    x = wave_max_i64(x);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
    __syncthreads();
    int64_t r = lds[0];
    for (int w = 1; w < kRedThreads / kWave; ++w) r = lds[w] > r ? lds[w] : r;
    __syncthreads();
    return r;
}

// The 8 flags of 8 consecutive elements, as one 8-byte load when
// the flag array is 8-byte aligned and the group lies inside [0, len).
__device__ __forceinline__ uint64_t flag_group(const uint8_t *f, int64_t p, int64_t len, bool vec) {
    if (vec && p + 8 <= len) return __builtin_nontemporal_load(reinterpret_cast<const uint64_t *>(f + p));
    uint64_t x = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (p + k < len) x |= static_cast<uint64_t>(f[p + k]) << (8 * k);
    return x;
}

__global__ __launch_bounds__(kRedThreads) void sg_reduce_kernel(SgArgs a) {
    constexpr int kLoads = kSgTile / (8 * kRedThreads);   // flag groups of a tile per thread
    constexpr int kVals = 8;                              // values in flight per thread
    __shared__ int64_t lds[kRedThreads / kWave];
    __shared__ uint64_t sums[kRedThreads / kWave];
    const int tid = threadIdx.x;
    const int64_t c = blockIdx.x;
    const int64_t lo = c * a.chunk;
    const int64_t hi = lo + a.chunk < a.n ? lo + a.chunk : a.n;
    // last flagged position of the chunk (lo - 1 if none)
    int64_t last = lo - 1;
    const bool fvec = (reinterpret_cast<uintptr_t>(a.flags) & 7) == 0;
    for (int64_t t = lo; t < hi; t += kSgTile) {
        uint64_t fg[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int64_t p = t - lo + (static_cast<int64_t>(j) * kRedThreads + tid) * 8;
            fg[j] = lo + p < hi ? flag_group(a.flags + lo, p, hi - lo, fvec) : 0;
        }
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int64_t p = t + (static_cast<int64_t>(j) * kRedThreads + tid) * 8;
            if (fg[j]) last = p + (63 - __builtin_clzll(fg[j])) / 8;
        }
    }
    last = block_max(last, lds);
    // a flagged element restarts the sum with its own value
    const int64_t start = last >= lo ? last : lo;
    uint64_t s = 0;
    for (int64_t p = start + tid; p < hi; p += kVals * kRedThreads) {
        uint64_t v[kVals];
#pragma unroll
        for (int j = 0; j < kVals; ++j) v[j] = p + j * kRedThreads < hi ? a.xs[p + j * kRedThreads] : 0;
#pragma unroll
        for (int j = 0; j < kVals; ++j) s += v[j];
    }
    s = wave_reduce_u64(s, [](uint64_t x, uint64_t y) { return x + y; });
    if ((tid & 63) == 0) sums[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        s = 0;
        for (int w = 0; w < kRedThreads / kWave; ++w) s += sums[w];
        a.agg_v[c] = s;
        a.agg_f[c] = last >= lo ? 1 : 0;
    }
}

// One workgroup: aggregates -> exclusive prefixes (in place, values only).
__global__ __launch_bounds__(1024) void sg_chunk_scan_kernel(SgArgs a) {
    constexpr int kPer = 8;
    static_assert(kPer * 1024 >= kSgMaxChunks, "scan capacity");
    __shared__ uint64_t wv[16];
    __shared__ int32_t wf[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    Pair e[kPer];
    Pair run{false, 0};
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = static_cast<int64_t>(tid) * kPer + k;
        e[k] = i < a.chunks ? Pair{a.agg_f[i] != 0, a.agg_v[i]} : Pair{false, 0};
        run = combine(run, e[k]);
    }
    // the sums wrap, so the sum since the last flag is a difference of plain
    // prefix sums, as in the rescan
    const uint64_t flagged = ballot(run.f);
    const uint64_t inc = wave_scan_u64(run.v), ex = inc - run.v;
    const uint64_t below = flagged & ((1ull << lane) - 1);
    const uint64_t from = __shfl(ex, below ? 63 - __builtin_clzll(below) : 0, kWave);
    const Pair before{below != 0, ex - from};
    if (lane == kWave - 1) {
        const Pair all = combine(before, run);
        wv[wave] = all.v;
        wf[wave] = all.f ? 1 : 0;
    }
    __syncthreads();
    Pair acc{false, 0};
    for (int w = 0; w < wave; ++w) acc = combine(acc, Pair{wf[w] != 0, wv[w]});
    acc = combine(acc, before);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = static_cast<int64_t>(tid) * kPer + k;
        if (i < a.chunks) a.agg_v[i] = acc.v;   // a flag only matters for later elements
        acc = combine(acc, e[k]);
    }
}

// Rescan.  The sums wrap, so a running sum since the last flag is a difference
// of plain prefix sums: a row of 128 elements takes one plain scan of the
// lanes' pairs, and an unflagged element looks up the prefix at the nearest
// flagged lane below it (from the ballot of the flags).  Loads and stores are
// 16 bytes a lane and consecutive, nothing is transposed, and the only barrier
// of a step publishes the waves' last running sums.
// 2^25 int64 values, a flag every 335: 101 us (17 bytes an element, 5.6 TB/s);
// 8 consecutive elements per thread, transposed through 64 KiB of LDS with four
// barriers a tile, took 165 us.
constexpr int kScThreads = 512;
constexpr int kScRows = 4;
constexpr int kScWave = kScRows * 2 * kWave;              // elements of a wave
constexpr int kScStep = kScThreads / kWave * kScWave;     // elements of a step
static_assert(kSgTile % kScStep == 0, "whole steps");

__global__ __launch_bounds__(kScThreads) void sg_rescan_kernel(SgArgs a) {
    constexpr int kWaves = kScThreads / kWave;
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    __shared__ uint64_t wv[2][kWaves];   // by parity of the step
    __shared__ int32_t wf[2][kWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = wave_id();
    const int64_t c = blockIdx.x;
    const int64_t lo_c = c * a.chunk;
    const int64_t hi_c = lo_c + a.chunk < a.n ? lo_c + a.chunk : a.n;
    uint64_t carry = a.agg_v[c];   // running sum before the chunk (a flag inside the chunk resets it)
    const bool fvec = (reinterpret_cast<uintptr_t>(a.flags) & 1) == 0;
    const bool xvec = (reinterpret_cast<uintptr_t>(a.xs) & 15) == 0;
    const bool ovec = (reinterpret_cast<uintptr_t>(a.out) & 15) == 0;
    int par = 0;
    for (int64_t lo = lo_c; lo < hi_c; lo += kScStep, par ^= 1) {
        const int64_t e0 = lo + wave * kScWave + 2 * lane;
        const bool whole = lo + (wave + 1) * kScWave <= hi_c;   // (wave-uniform)
        uint64_t v[kScRows][2];
        uint32_t fl[kScRows];   // the pair's flags: nonzero low byte, nonzero second byte
        if (whole && xvec && fvec) {
#pragma unroll
            for (int r = 0; r < kScRows; ++r) {
                const u64x2 x = __builtin_nontemporal_load(reinterpret_cast<const u64x2 *>(a.xs + e0 + r * 2 * kWave));
                fl[r] = __builtin_nontemporal_load(reinterpret_cast<const uint16_t *>(a.flags + e0 + r * 2 * kWave));
                v[r][0] = x.x;
                v[r][1] = x.y;
            }
        } else {
#pragma unroll
            for (int r = 0; r < kScRows; ++r) {
                const int64_t e = e0 + r * 2 * kWave;
                v[r][0] = e < hi_c ? a.xs[e] : 0;
                v[r][1] = e + 1 < hi_c ? a.xs[e + 1] : 0;
                fl[r] = (e < hi_c ? a.flags[e] : 0u) | (e + 1 < hi_c ? static_cast<uint32_t>(a.flags[e + 1]) << 8 : 0u);
            }
        }
        // run: running sum before the row, from the wave's start; seen: some
        // flag before the row; open: bit r*2+q, the element adds what comes
        // before the wave
        uint64_t run = 0;
        bool seen = false;
        uint32_t open = 0;
#pragma unroll
        for (int r = 0; r < kScRows; ++r) {
            const bool f0 = (fl[r] & 0xFFu) != 0, f1 = (fl[r] >> 8) != 0;
            const uint64_t inc = wave_scan_u64(v[r][0] + v[r][1]);
            const uint64_t excl = inc - v[r][0] - v[r][1];
            const uint64_t total = readlane_u64(inc, kWave - 1);
            const uint64_t m = ballot(f0 | f1);
            const uint64_t at = f1 ? excl + v[r][0] : excl;   // prefix before this lane's last flag
            const uint64_t below = m & ((1ull << lane) - 1);
            const uint64_t from = __shfl(at, below ? 63 - __builtin_clzll(below) : 0, kWave);
            const uint64_t x0 = f0 ? v[r][0] : v[r][0] + excl + (below ? -from : run);
            const bool o0 = !(f0 | seen | (below != 0));
            open |= (static_cast<uint32_t>(o0) | static_cast<uint32_t>(o0 & !f1) << 1) << (2 * r);
            v[r][1] += f1 ? 0 : x0;
            v[r][0] = x0;
            run = m ? total - readlane_u64(at, 63 - __builtin_clzll(m)) : run + total;
            seen |= m != 0;
        }
        if (lane == 0) {
            wv[par][wave] = run;
            wf[par][wave] = seen ? 1 : 0;
        }
        __syncthreads();
        uint64_t before = carry;   // running sum before this wave
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint64_t x = wv[par][w];
            const bool f = wf[par][w] != 0;
            carry = f ? x : carry + x;
            if (w < wave) before = carry;
        }
#pragma unroll
        for (int r = 0; r < kScRows; ++r) {
            const int64_t e = e0 + r * 2 * kWave;
            u64x2 y;
            y.x = v[r][0] + ((open >> (2 * r)) & 1u ? before : 0);
            y.y = v[r][1] + ((open >> (2 * r + 1)) & 1u ? before : 0);
            if (whole && ovec) {
                stream_store(reinterpret_cast<u64x2 *>(a.out + e), y);
            } else {
                if (e < hi_c) stream_store(a.out + e, static_cast<uint64_t>(y.x));
                if (e + 1 < hi_c) stream_store(a.out + e + 1, static_cast<uint64_t>(y.y));
            }
        }
    }
}

// Chunks of whole tiles, at most kSgMaxChunks of them.
void sg_geometry(int64_t n, int64_t *chunk, int64_t *chunks) {
    const int64_t tiles = ceil_div(n, kSgTile);
    const int64_t per = ceil_div(tiles, kSgMaxChunks);
    *chunk = per * kSgTile;
    *chunks = ceil_div(n, *chunk);
}

}  // namespace
}  // namespace ixp

using namespace ixp;

extern "C" size_t ixp_sgm_sum_workspace(int64_t n) {
    if (n < 0) return 0;
    int64_t chunk = 0, chunks = 0;
    sg_geometry(n > 0 ? n : 1, &chunk, &chunks);
    return round_up(static_cast<size_t>(chunks) * 8, 256) + static_cast<size_t>(chunks) * 4;
}

extern "C" int ixp_sgm_sum(const uint8_t *d_flags, const int64_t *d_xs, int64_t n, int64_t *d_out, void *ws,
                           size_t ws_bytes, void *stream) {
    if (n < 0 || (n > 0 && (!d_flags || !d_xs || !d_out))) return IXP_EINVAL;
    if (!aligned(d_xs, 8) || !aligned(d_out, 8) || !aligned(ws, 8)) return IXP_EINVAL;
    if (!ws || ws_bytes < ixp_sgm_sum_workspace(n)) return IXP_EWORKSPACE;
    if (n == 0) return IXP_OK;
    SgArgs a;
    a.flags = d_flags;
    a.xs = reinterpret_cast<const uint64_t *>(d_xs);
    a.out = reinterpret_cast<uint64_t *>(d_out);
    a.n = n;
    sg_geometry(n, &a.chunk, &a.chunks);
    a.agg_v = static_cast<uint64_t *>(ws);
    a.agg_f = reinterpret_cast<int32_t *>(static_cast<char *>(ws) + round_up(static_cast<size_t>(a.chunks) * 8, 256));
    hipStream_t st = as_stream(stream);
    const dim3 grid(static_cast<uint32_t>(a.chunks));
    IXP_LAUNCH("sgm_reduce", sg_reduce_kernel, grid, dim3(kRedThreads), 0, st, a);
    IXP_LAUNCH("sgm_chunk_scan", sg_chunk_scan_kernel, dim3(1), dim3(1024), 0, st, a);
    IXP_LAUNCH("sgm_rescan", sg_rescan_kernel, grid, dim3(kScThreads), 0, st, a);
    return launch_status();
}
