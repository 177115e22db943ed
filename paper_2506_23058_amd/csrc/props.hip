// props.hip -- run-time checkers of the array properties of Section 2.3
// (figure "Array Properties"): Range, Monotonic, Inj, Bij and FiltPart.
//
// Range / Monotonic / Inj / Bij share one streaming pass over X (16-byte
// nontemporal loads).  Every failing index is reduced to the least one with a
// wave minimum and an atomicMin, so verdicts do not depend on scheduling.
//
// Inj and Bij need to know which in-Rcd values occur more than once.  For
// large arrays whose Rcd spans at most 4096 buckets of up to 2^20 values, the pass
// over X also groups each workgroup's chunk of in-Rcd values by bucket in LDS
// and writes the chunk's values bucket by bucket into its own region, with a
// per-chunk table of where each bucket starts (no global histogram is
// needed); then one workgroup per bucket reads that bucket's runs from every
// chunk into an LDS bitmap.  Smaller arrays insert into a bitmap over
// Rcd in global memory directly.  A bit found already set says that its value
// repeats, not which occurrence is the first, so each repeated value is
// listed once (a second bitmap marks it).  One more streaming pass then looks
// every in-Rcd value up in an LDS hash table of the listed values and keeps,
// per listed value, the least index seen; an arrival that displaces an
// earlier least index, or finds one already there, proposes the larger of
// the two, and the least proposal is the earliest second occurrence.  When
// more values repeat than the list holds, two global passes over a per-value
// first-index table locate it instead.
//
// FiltPart checks the outputs of a flat partition: the split point against
// the number of trues, Bij of the indices (as above), the class order, the
// values moved, and stability (indices strictly increasing inside each class,
// InvFiltPart item 3).  Where class order and stability hold, nothing can
// repeat, so the bitmap is used only after one of them fails.
#include <type_traits>

#include "device.hpp"
#include "host.hpp"

namespace ixp {
namespace {

constexpr uint64_t kNone = 0x7FFFFFFFFFFFFFFFull;
constexpr int kPropsBlock = 256;
constexpr int kBucketShift = 20;              // at most 2^20 values a bucket: a 128 KiB LDS bitmap
constexpr int kMaxBuckets = 4096;
constexpr int kChunk = 16384;                 // elements per props_scan workgroup
constexpr int kScanThreads = 512;             // two workgroups per CU (64 KiB of LDS each)
constexpr int kRepCap = 2048;                 // repeated values one rescan can locate
constexpr int kRepSlots = 4 * kRepCap;        // hash table slots: load factor <= 1/4
constexpr uint64_t kEmptySlot = ~0ull;

// Device-side state at the start of the workspace.
struct PropsState {
    unsigned long long fv_range, fv_mono, fv_img, fv_inj;   // least failing index, kNone if none
    unsigned long long in_count;                            // entries inside Rcd
    unsigned long long missing;                             // least value of Img not attained, minus img_lo
    unsigned int dup_found;
    unsigned int nrep;                 // repeated values listed (may exceed the list)
    // FiltPart
    unsigned long long fp_fv;          // least index failing bits 1..4
    unsigned int fp_bits;              // OR of failing sub-check bits (2..16)
    unsigned int done;                 // workgroups of the last kernel that are through
};
constexpr size_t kPropsHeader = 256;
static_assert(sizeof(PropsState) <= kPropsHeader, "props header");

struct PropsArgs {
    const void *x;
    int32_t x64;          // 1: int64 elements, 0: int32
    int64_t n;
    uint32_t mask;
    int64_t lo, hi, ilo, ihi;
    int32_t mono_op;
    PropsState *st;
    uint32_t *seen;       // bitmap over [lo, hi)
    uint32_t *dup;        // repeated values
    uint32_t *first;      // least index of each repeated value (n < 2^32) or...
    unsigned long long *first64;   // ... 64-bit when n >= 2^32
    int64_t width;        // hi - lo when a bitmap is in use
    // Chunked Inj/Bij (props_scan / props_check): values of Rcd grouped in
    // buckets of 2^bshift consecutive values.
    int32_t bucketed;
    int32_t nbuckets;
    int32_t bshift;
    int64_t nchunks;
    uint16_t *ctab;       // [(nbuckets + 1) * nchunks]: bucket starts per chunk; last row: chunk totals
    uint32_t *records;    // [nchunks * kChunk]: value - lo - bucket base (20 bits)
    // Repeated values (Inj's first-violation search)
    uint64_t *rep;        // [kRepCap] value - lo of each repeated value
    unsigned long long *rep_min;   // [kRepCap] least index seen per listed value
    // FiltPart
    const uint32_t *fp_src;
    const uint32_t *fp_dst;
    const int64_t *fp_split;
    int32_t fp_mode;
    int64_t *fp_last;     // [2][kFpRanges] last index value of each class in a range (kNoZ if none)
    unsigned long long *fp_count;   // [kFpRanges] trues of a range
    int64_t fp_range;     // elements per range
    int64_t fp_nranges;
};

__device__ __forceinline__ int64_t load_x(const void *x, int32_t x64, int64_t i) {
    return x64 ? static_cast<const int64_t *>(x)[i] : static_cast<int64_t>(static_cast<const int32_t *>(x)[i]);
}

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    return wave_reduce_u64(v, [](uint64_t x, uint64_t y) { return x < y ? x : y; });
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
    return static_cast<unsigned long long>(wave_sum_i64(static_cast<int64_t>(v)));
}

__device__ __forceinline__ bool mono_ok(int64_t a, int64_t b, int op) {
    switch (op) {
    case IXP_MONO_LE: return a <= b;
    case IXP_MONO_LT: return a < b;
    case IXP_MONO_GE: return a >= b;
    default: return a > b;
    }
}

__global__ void props_init_kernel(PropsState *st, uint32_t *seen, uint32_t *dup, int64_t words,
                                  unsigned long long *rep_min) {
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (rep_min)
        for (int64_t i = i0; i < kRepCap; i += static_cast<int64_t>(gridDim.x) * blockDim.x) rep_min[i] = kNone;
    if (i0 == 0 && st) {
        st->fv_range = st->fv_mono = st->fv_img = st->fv_inj = kNone;
        st->in_count = 0;
        st->missing = kNone;
        st->dup_found = 0;
        st->nrep = 0;
        st->fp_fv = kNone;
        st->fp_bits = 0;
        st->done = 0;
    }
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    const int64_t w4 = words / 4;
    for (int64_t i = i0; i < w4; i += stride) {
        if (seen) __builtin_nontemporal_store(v4{0, 0, 0, 0}, reinterpret_cast<v4 *>(seen) + i);
        __builtin_nontemporal_store(v4{0, 0, 0, 0}, reinterpret_cast<v4 *>(dup) + i);
    }
    for (int64_t i = w4 * 4 + i0; i < words; i += stride) {
        if (seen) seen[i] = 0;
        dup[i] = 0;
    }
}

// A value found already set in the seen bitmap (o = value - lo): mark it in
// the dup bitmap, list it the first time, and reset its first-index slot for
// the global fallback passes.  Most repeats are of a value marked before, and
// the atomics of a few values' repeats fall on the same words one after the other,
// the more so where a narrow bucket's one workgroup makes them: a load finds
// those first.  (Range, Inj, Bij of 2^23 random int64 values, with / without
// the load: Rcd of 8192 values 1.1 / 16.4 ms, 65,536 0.68 / 1.32, 2^20 1.94 / 1.95; 2^26
// of 8192 5.8 / 128.  With one bucket of 2^20 values or the global bitmap for such Rcd,
// and no load, 4.6, 1.58, 2.04 and 35.5.)
__device__ __forceinline__ void note_repeat(const PropsArgs &a, uint64_t o, bool list) {
    const uint32_t bit = 1u << (o & 31);
    if (__hip_atomic_load(a.dup + (o >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) return;
    const uint32_t old = atomicOr(a.dup + (o >> 5), bit);
    if (list && !(old & bit)) {
        const uint32_t k = atomicAdd(&a.st->nrep, 1u);
        if (k < kRepCap) a.rep[k] = o;
    }
    if (a.first64) a.first64[o] = ~0ull;
    else a.first[o] = ~0u;
}

// Inserts v (inside [lo, hi)) into the seen bitmap; a repeat is noted.
template <bool LIST>
__device__ __forceinline__ void insert_value(const PropsArgs &a, int64_t v, bool *dup_seen) {
    const uint64_t o = static_cast<uint64_t>(v - a.lo);
    const uint32_t bit = 1u << (o & 31);
    const uint32_t old = atomicOr(a.seen + (o >> 5), bit);
    if (old & bit) {
        note_repeat(a, o, LIST);
        *dup_seen = true;
    }
}

// Monotonic comparison with the operator decoded once: LE a<=b, LT a<b,
// GE b<=a, GT b<a.
struct MonoCmp {
    bool swap, strict;
    __device__ __forceinline__ bool ok(int64_t a, int64_t b) const {
        const int64_t l = swap ? b : a, r = swap ? a : b;
        return strict ? l < r : l <= r;
    }
};

// Pass 1 (arrays without the chunked path): Range, Monotonic, the Img part of
// Bij, the in-Rcd count and the bitmap insertions of Inj / Bij, for every
// element.  Each thread takes 16-byte groups (2 int64 or 4 int32); a group's
// left neighbour for the monotonic check comes from the previous lane
// (consecutive lanes hold consecutive groups), lane 0 loads it.
template <bool X64, int UNROLL>
__global__ __launch_bounds__(kPropsBlock) void props_pass1_kernel(PropsArgs a) {
    constexpr int kPer = X64 ? 2 : 4;
    const bool want_range = a.mask & IXP_RANGE;
    const bool want_mono = a.mask & IXP_MONO;
    const bool want_set = a.mask & (IXP_INJ | IXP_BIJ);
    const bool want_img = a.mask & IXP_BIJ;
    const MonoCmp cmp{a.mono_op == IXP_MONO_GE || a.mono_op == IXP_MONO_GT,
                      a.mono_op == IXP_MONO_LT || a.mono_op == IXP_MONO_GT};
    const int lane = threadIdx.x & 63;
    unsigned long long c_range = kNone, c_mono = kNone, c_img = kNone, cnt = 0;
    bool dup_seen = false;
    const int64_t groups = a.n / kPer;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    // every lane of a wave runs the same number of iterations (shuffles below)
    const int64_t wave_g0 = g0 - lane;
    for (int64_t gb = g0; wave_g0 + (gb - g0) < groups; gb += UNROLL * stride) {
        v4 raw[UNROLL];
        int64_t gi[UNROLL], left[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            gi[u] = gb + u * stride;
            raw[u] = gi[u] < groups
                         ? __builtin_nontemporal_load(reinterpret_cast<const v4 *>(a.x) + gi[u])
                         : v4{0, 0, 0, 0};
        }
        // lane 0's left neighbours, loaded beside the groups rather than
        // one dependent load per group
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            left[u] = want_mono && lane == 0 && gi[u] < groups && gi[u] > 0
                          ? load_x(a.x, X64 ? 1 : 0, gi[u] * kPer - 1)
                          : 0;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int64_t val[kPer];
            if constexpr (X64) {
                val[0] = static_cast<int64_t>((static_cast<uint64_t>(raw[u].y) << 32) | raw[u].x);
                val[1 % kPer] = static_cast<int64_t>((static_cast<uint64_t>(raw[u].w) << 32) | raw[u].z);
            } else {
                val[0] = static_cast<int32_t>(raw[u].x);
                val[1 % kPer] = static_cast<int32_t>(raw[u].y);
                val[2 % kPer] = static_cast<int32_t>(raw[u].z);
                val[3 % kPer] = static_cast<int32_t>(raw[u].w);
            }
            const bool live = gi[u] < groups;
            const int64_t p0 = gi[u] * kPer;
            int64_t prev = 0;
            if (want_mono) {
                prev = __shfl_up(val[kPer - 1], 1, 64);
                if (lane == 0) prev = left[u];
            }
            if (!live) continue;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int64_t i = p0 + q;
                const int64_t v = val[q];
                if (want_range && !(a.lo <= v && v < a.hi) && static_cast<unsigned long long>(i) < c_range)
                    c_range = i;
                if (want_mono && i > 0 && !cmp.ok(prev, v) && static_cast<unsigned long long>(i) < c_mono)
                    c_mono = i;
                prev = v;
                if (want_set && a.lo <= v && v < a.hi) {
                    ++cnt;
                    if (want_img && !(a.ilo <= v && v < a.ihi) && static_cast<unsigned long long>(i) < c_img)
                        c_img = i;
                    insert_value<true>(a, v, &dup_seen);
                }
            }
        }
    }
    // the last n % kPer elements: thread 0 of block 0
    if (g0 == 0) {
        for (int64_t i = groups * kPer; i < a.n; ++i) {
            const int64_t v = load_x(a.x, X64 ? 1 : 0, i);
            if (want_range && !(a.lo <= v && v < a.hi) && static_cast<unsigned long long>(i) < c_range)
                c_range = i;
            if (want_mono && i > 0 && !cmp.ok(load_x(a.x, X64 ? 1 : 0, i - 1), v) &&
                static_cast<unsigned long long>(i) < c_mono)
                c_mono = i;
            if (want_set && a.lo <= v && v < a.hi) {
                ++cnt;
                if (want_img && !(a.ilo <= v && v < a.ihi) && static_cast<unsigned long long>(i) < c_img)
                    c_img = i;
                insert_value<true>(a, v, &dup_seen);
            }
        }
    }
    c_range = wave_min_u64(c_range);
    c_mono = wave_min_u64(c_mono);
    c_img = wave_min_u64(c_img);
    cnt = wave_sum_u64(cnt);
    const bool any_dup = ballot(dup_seen) != 0;
    if (lane == 0) {
        if (c_range != kNone) atomicMin(&a.st->fv_range, c_range);
        if (c_mono != kNone) atomicMin(&a.st->fv_mono, c_mono);
        if (c_img != kNone) atomicMin(&a.st->fv_img, c_img);
        if (cnt) atomicAdd(&a.st->in_count, cnt);
        if (any_dup) atomicOr(&a.st->dup_found, 1u);
    }
}

// Chunked Inj/Bij.  Random device-scope atomics on a bitmap in HBM run far
// below the memory bandwidth, so the in-Rcd values are routed to one
// workgroup per bucket of up to 2^20 values, whose bitmap sits in LDS.
//
// props_scan: workgroup c owns elements [c kChunk, (c+1) kChunk) (chunks in
// an XCD-aware order).  Besides Range / Monotonic / Img it ranks every in-Rcd
// value inside its bucket with an LDS atomic, scans the chunk's bucket
// counts, stages the values in bucket order in LDS and writes them as one
// contiguous run to the chunk's own region of `records`; ctab row b, column
// c receives the start of bucket b inside the chunk (row nbuckets: the
// chunk's in-Rcd total).  The values are written once and read once.
template <bool X64>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4)))
void props_scan_kernel(PropsArgs a) {
    constexpr int kPer = X64 ? 2 : 4;                       // elements per 16-byte group
    constexpr int kGroups = kChunk / kPer / kScanThreads;   // groups per thread
    constexpr int kElems = kGroups * kPer;
    constexpr uint32_t kOut = ~0u;
    __shared__ uint32_t stage[kChunk];
    __shared__ uint32_t wtot[kScanThreads / kWave];
    __shared__ unsigned long long wmin[3][kScanThreads / kWave];
    __shared__ int64_t wlast[kGroups][kScanThreads / kWave];   // Monotonic's left neighbours
    __shared__ int64_t wfirst;
    extern __shared__ uint32_t bstart[];                    // [nbuckets + 1]
    const int nb = a.nbuckets;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int64_t c = xcd_tile(blockIdx.x, a.nchunks);
    for (int b = tid; b <= nb; b += kScanThreads) bstart[b] = 0;
    __syncthreads();
    const bool want_range = a.mask & IXP_RANGE;
    const bool want_mono = a.mask & IXP_MONO;
    const bool want_img = a.mask & IXP_BIJ;
    const MonoCmp cmp{a.mono_op == IXP_MONO_GE || a.mono_op == IXP_MONO_GT,
                      a.mono_op == IXP_MONO_LT || a.mono_op == IXP_MONO_GT};
    const int64_t e0 = c * kChunk;
    const int64_t e1 = a.n < e0 + kChunk ? a.n : e0 + kChunk;
    const int64_t g_lo = e0 / kPer, g_hi = e1 / kPer;       // whole groups of the chunk
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    v4 raw[kGroups];
#pragma unroll
    for (int u = 0; u < kGroups; ++u) {
        const int64_t gi = g_lo + tid + u * kScanThreads;
        raw[u] = gi < g_hi ? __builtin_nontemporal_load(reinterpret_cast<const v4 *>(a.x) + gi)
                           : v4{0, 0, 0, 0};
    }
    unsigned long long c_range = kNone, c_mono = kNone, c_img = kNone;
    if (want_mono) {
        // the last element of every wave's group u, for the lane 0 of the
        // next wave (thread 0's group u follows thread kScanThreads-1's
        // group u-1); thread 0's first left neighbour comes from memory
        if (lane == kWave - 1) {
#pragma unroll
            for (int u = 0; u < kGroups; ++u)
                wlast[u][wave] = X64 ? static_cast<int64_t>((static_cast<uint64_t>(raw[u].w) << 32) | raw[u].z)
                                     : static_cast<int64_t>(static_cast<int32_t>(raw[u].w));
        }
        if (tid == 0 && e0 > 0) wfirst = load_x(a.x, X64 ? 1 : 0, e0 - 1);
        __syncthreads();
    }
    // Offsets in Rcd of the thread's elements and which of them lie inside; the
    // three other checks beside them, each skipped by the whole wave where it has
    // nothing to report.
    static_assert(kElems == 32, "a bit per element");
    const uint64_t width = static_cast<uint64_t>(a.hi) - static_cast<uint64_t>(a.lo);
    const bool whole = e1 - e0 == kChunk;   // (uniform)
    const bool img_all = a.ilo <= a.lo && a.hi <= a.ihi;
    uint32_t off[kElems], in_bits = 0;
#pragma unroll
    for (int u = 0; u < kGroups; ++u) {
        const int64_t gi = g_lo + tid + u * kScanThreads;
        int64_t val[kPer];
        if constexpr (X64) {
            val[0] = static_cast<int64_t>((static_cast<uint64_t>(raw[u].y) << 32) | raw[u].x);
            val[1 % kPer] = static_cast<int64_t>((static_cast<uint64_t>(raw[u].w) << 32) | raw[u].z);
        } else {
            val[0] = static_cast<int32_t>(raw[u].x);
            val[1 % kPer] = static_cast<int32_t>(raw[u].y);
            val[2 % kPer] = static_cast<int32_t>(raw[u].z);
            val[3 % kPer] = static_cast<int32_t>(raw[u].w);
        }
        const bool live = whole || gi < g_hi;
        const int64_t p0 = gi * kPer;
        int64_t prev = 0;
        if (want_mono) {
            // consecutive lanes hold consecutive groups
            prev = __shfl_up(val[kPer - 1], 1, 64);
            if (lane == 0)
                prev = wave > 0 ? wlast[u][wave - 1] : u > 0 ? wlast[u - 1][kScanThreads / kWave - 1] : wfirst;
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int k = u * kPer + q;
            const unsigned long long i = static_cast<unsigned long long>(p0 + q);
            const int64_t v = val[q];
            // (v - lo as an unsigned number is below the width exactly when lo <= v < hi)
            const uint64_t o = static_cast<uint64_t>(v) - static_cast<uint64_t>(a.lo);
            const bool in = live && o < width;
            off[k] = static_cast<uint32_t>(o);
            in_bits |= static_cast<uint32_t>(in) << k;
            if (want_range) {
                const bool bad = live && !in;
                if (ballot(bad) && bad && i < c_range) c_range = i;
            }
            if (want_mono) {
                const bool bad = live && i > 0 && !cmp.ok(prev, v);
                if (ballot(bad) && bad && i < c_mono) c_mono = i;
                prev = v;
            }
            if (want_img && !img_all) {
                const bool bad = in && !(a.ilo <= v && v < a.ihi);
                if (ballot(bad) && bad && i < c_img) c_img = i;
            }
        }
    }
    // Ranks inside the buckets.  A wave whose elements all lie in Rcd issues its
    // LDS atomics back to back; a branch around each, with its result combined at
    // once, made every one of them wait (2^27 int64: 294 -> 284 us, 2^28 811 -> 791 for
    // Range + Inj + Bij).
    uint32_t rank[kElems / 2];   // two 16-bit ranks each (a chunk holds 2^14 elements)
    const bool all_in = ballot(in_bits != ~0u) == 0;
    if (all_in) {
#pragma unroll
        for (int k = 0; k < kElems; k += 8) {
            uint32_t r[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = atomicAdd(bstart + (off[k + j] >> a.bshift), 1u);
#pragma unroll
            for (int j = 0; j < 8; j += 2) rank[(k + j) / 2] = r[j] | (r[j + 1] << 16);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kElems; k += 2) {
            uint32_t r0 = 0, r1 = 0;
            if ((in_bits >> k) & 1u) r0 = atomicAdd(bstart + (off[k] >> a.bshift), 1u);
            if ((in_bits >> (k + 1)) & 1u) r1 = atomicAdd(bstart + (off[k + 1] >> a.bshift), 1u);
            rank[k / 2] = r0 | (r1 << 16);
        }
    }
    auto rank_of = [&](int k) { return (rank[k / 2] >> (16 * (k % 2))) & 0xFFFFu; };
    // the chunk's last n % kPer elements (only in the chunk holding the end
    // of the array): thread 0, one at a time
    uint32_t toff[3] = {0, 0, 0}, tmeta[3] = {kOut, kOut, kOut};
    if (tid == 0) {
        for (int64_t i = g_hi * kPer; i < e1; ++i) {
            const int j = static_cast<int>(i - g_hi * kPer);
            const int64_t v = load_x(a.x, X64 ? 1 : 0, i);
            if (want_range && !(a.lo <= v && v < a.hi) && static_cast<unsigned long long>(i) < c_range)
                c_range = i;
            if (want_mono && i > 0 && !cmp.ok(load_x(a.x, X64 ? 1 : 0, i - 1), v) &&
                static_cast<unsigned long long>(i) < c_mono)
                c_mono = i;
            if (a.lo <= v && v < a.hi) {
                if (want_img && !(a.ilo <= v && v < a.ihi) && static_cast<unsigned long long>(i) < c_img)
                    c_img = i;
                const uint64_t o = static_cast<uint64_t>(v - a.lo);
                const uint32_t bk = static_cast<uint32_t>(o >> a.bshift);
                toff[j] = static_cast<uint32_t>(o) & ((1u << a.bshift) - 1);
                tmeta[j] = (bk << 16) | atomicAdd(bstart + bk, 1u);
            }
        }
    }
    __syncthreads();
    // exclusive scan of the nb + 1 bucket counts (the last is 0, so it
    // becomes the chunk's total): thread t owns `per` consecutive entries
    {
        const int per = (nb + 1 + kScanThreads - 1) / kScanThreads;
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
    for (int b = tid; b <= nb; b += kScanThreads)
        a.ctab[static_cast<int64_t>(b) * a.nchunks + c] = static_cast<uint16_t>(bstart[b]);
    const uint32_t bmask = (1u << a.bshift) - 1;
    if (all_in) {
#pragma unroll
        for (int k = 0; k < kElems; ++k) stage[bstart[off[k] >> a.bshift] + rank_of(k)] = off[k] & bmask;
    } else {
#pragma unroll
        for (int k = 0; k < kElems; ++k)
            if ((in_bits >> k) & 1u) stage[bstart[off[k] >> a.bshift] + rank_of(k)] = off[k] & bmask;
    }
    if (tid == 0) {
        for (int j = 0; j < 3; ++j)
            if (tmeta[j] != kOut) stage[bstart[tmeta[j] >> 16] + (tmeta[j] & 0xFFFFu)] = toff[j];
    }
    __syncthreads();
    const uint32_t total = bstart[nb];
    uint32_t *dst = a.records + c * kChunk;
    for (uint32_t j = tid; j < total / 4; j += kScanThreads) {
        const v4 w{stage[4 * j], stage[4 * j + 1], stage[4 * j + 2], stage[4 * j + 3]};
        __builtin_nontemporal_store(w, reinterpret_cast<v4 *>(dst) + j);
    }
    for (uint32_t j = total / 4 * 4 + tid; j < total; j += kScanThreads) dst[j] = stage[j];
    // least failing indices: one atomicMin per workgroup, and none when the
    // target already holds a smaller index (a permutation fails Monotonic
    // almost everywhere, and same-address atomics serialise)
    c_range = wave_min_u64(c_range);
    c_mono = wave_min_u64(c_mono);
    c_img = wave_min_u64(c_img);
    if (lane == 0) {
        wmin[0][wave] = c_range;
        wmin[1][wave] = c_mono;
        wmin[2][wave] = c_img;
    }
    __syncthreads();
    if (tid < 3) {
        unsigned long long m = kNone;
        for (int w = 0; w < kScanThreads / kWave; ++w) m = wmin[tid][w] < m ? wmin[tid][w] : m;
        unsigned long long *t = tid == 0 ? &a.st->fv_range : tid == 1 ? &a.st->fv_mono : &a.st->fv_img;
        if (m != kNone && m < __hip_atomic_load(t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(t, m);
    }
}

// props_check: workgroup b sets the bits of bucket b's values in an LDS
// bitmap of up to 128 KiB.  The bucket's records are one run per chunk; a wave takes 16
// chunks at a time, 4 lanes per chunk, and reads each run as the aligned
// 16-byte quads that cover it (records of neighbouring buckets in the edge
// quads are skipped), each lane up to kCheckDepth quads per pass, all loads
// issued before the bits are set, and the next chunks' run bounds fetched
// while the current ones are read.  Plain loads: the quads of one run are
// spread over several lanes and passes, so its cache lines are met more than
// once.  A bit found set lists its value as repeated.  For Bij it also finds
// the least value of Img inside the bucket whose bit is clear; the
// workgroup of the last bucket adds up the chunks' in-Rcd totals.
// Neighbouring buckets meet in the cache lines at the ends of their runs, so the
// buckets of one XCD are consecutive (2^28 entries: 268 -> 228 us).
constexpr int kCheckThreads = 1024;
constexpr int kCheckLanes = 4;
constexpr int kCheckDepth = 8;

template <int SHIFT>   // at least a.bshift
__global__ __launch_bounds__(kCheckThreads) void props_check_kernel(PropsArgs a) {
    __shared__ uint32_t bits[(1 << SHIFT) / 32];
    __shared__ unsigned long long wsum[kCheckThreads / kWave];
    const int b = static_cast<int>(xcd_tile(blockIdx.x, a.nbuckets));
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    for (int w = tid; w < (1 << a.bshift) / 32; w += kCheckThreads) bits[w] = 0;
    __syncthreads();
    const int64_t nc = a.nchunks;
    const uint16_t *rs = a.ctab + static_cast<int64_t>(b) * nc;
    const uint16_t *re = rs + nc;
    const int sub = lane / kCheckLanes, sl = lane % kCheckLanes;
    constexpr int kChunksPerWave = kWave / kCheckLanes;
    constexpr int kStride = (kCheckThreads / kWave) * kChunksPerWave;
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    bool dup_seen = false;
    unsigned long long tot = 0;
    // Sets the bits of the records at positions [s, e) of quads q, q + 4, ...
    // (one lane's share of a pass) whose values are in r.
    auto set_bits = [&](const v4 (&r)[kCheckDepth], uint32_t q0, uint32_t s, uint32_t e) {
#pragma unroll
        for (int d = 0; d < kCheckDepth; ++d) {
            const uint32_t q = q0 + sl + d * kCheckLanes;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t p = 4 * q + j;
                if (p < s || p >= e) continue;
                const uint32_t off = r[d][j];
                const uint32_t bit = 1u << (off & 31);
                const uint32_t old = atomicOr(bits + (off >> 5), bit);
                if (old & bit) {
                    note_repeat(a, (static_cast<uint64_t>(b) << a.bshift) + off, true);
                    dup_seen = true;
                }
            }
        }
    };
    auto load_pass = [&](v4 (&r)[kCheckDepth], int64_t c, uint32_t q0, uint32_t e) {
        const v4 *rq = reinterpret_cast<const v4 *>(a.records + c * kChunk);
        const uint32_t q_hi = (e + 3) >> 2;
#pragma unroll
        for (int d = 0; d < kCheckDepth; ++d) {
            const uint32_t q = q0 + sl + d * kCheckLanes;
            r[d] = q < q_hi ? rq[q] : v4{0, 0, 0, 0};
        }
    };
    // Software pipeline over this wave's chunk batches: the first pass of
    // batch k + 1 is loaded while batch k's bits are set; the run bounds of
    // batch k + 2 are loaded meanwhile.  Runs longer than one pass (rare
    // with many buckets) take their further passes in place.
    constexpr uint32_t kPassQuads = kCheckLanes * kCheckDepth;
    int64_t c = static_cast<int64_t>(wave) * kChunksPerWave + sub;
    uint32_t s = c < nc ? rs[c] : 0u, e = c < nc ? re[c] : 0u;
    int64_t c1 = c + kStride;
    uint32_t s1 = c1 < nc ? rs[c1] : 0u, e1 = c1 < nc ? re[c1] : 0u;
    v4 cur[kCheckDepth], nxt[kCheckDepth];
    load_pass(cur, c, s >> 2, e);
    while (c - sub < nc) {   // wave-uniform
        const int64_t c2 = c1 + kStride;
        const uint32_t s2 = c2 < nc ? rs[c2] : 0u, e2 = c2 < nc ? re[c2] : 0u;
        load_pass(nxt, c1, s1 >> 2, e1);
        if (sl == 0 && c < nc) tot += e;
        set_bits(cur, s >> 2, s, e);
        for (uint32_t q0 = (s >> 2) + kPassQuads; q0 < ((e + 3) >> 2); q0 += kPassQuads) {
            load_pass(cur, c, q0, e);
            set_bits(cur, q0, s, e);
        }
#pragma unroll
        for (int d = 0; d < kCheckDepth; ++d) cur[d] = nxt[d];
        c = c1;
        s = s1;
        e = e1;
        c1 = c2;
        s1 = s2;
        e1 = e2;
    }
    const bool any_dup = ballot(dup_seen) != 0;
    if (lane == 0 && any_dup) atomicOr(&a.st->dup_found, 1u);
    if (b == a.nbuckets - 1) {
        // re is the totals row for the last bucket
        tot = wave_sum_u64(tot);
        if (lane == 0) wsum[wave] = tot;
        __syncthreads();
        if (tid == 0) {
            unsigned long long all = 0;
            for (int w = 0; w < kCheckThreads / kWave; ++w) all += wsum[w];
            a.st->in_count = all;
        }
    }
    if (!(a.mask & IXP_BIJ)) return;
    __syncthreads();
    // least value of Img inside this bucket whose bit is clear
    const int64_t v0 = a.lo + (static_cast<int64_t>(b) << a.bshift);
    const int64_t lo_b = a.ilo > v0 ? a.ilo - v0 : 0;
    const int64_t hi_b = a.ihi - v0 < (int64_t{1} << a.bshift) ? a.ihi - v0 : (int64_t{1} << a.bshift);
    unsigned long long cm = kNone;
    if (lo_b < hi_b) {
        for (int64_t w = (lo_b >> 5) + tid; w <= ((hi_b - 1) >> 5); w += kCheckThreads) {
            uint32_t clear = ~bits[w];
            const int64_t wb = w << 5;
            if (wb < lo_b) clear &= ~0u << (lo_b - wb);
            if (wb + 32 > hi_b) clear &= (hi_b - wb) >= 32 ? ~0u : ((1u << (hi_b - wb)) - 1u);
            if (clear) {
                // offset from img_lo: values may be negative
                const unsigned long long v =
                    static_cast<unsigned long long>(v0 + wb + __builtin_ctz(clear) - a.ilo);
                if (v < cm) cm = v;
            }
        }
    }
    cm = wave_min_u64(cm);
    if (lane == 0 && cm != kNone) atomicMin(&a.st->missing, cm);
}

// ------------------------------------------- locating the first repeat --
__device__ __forceinline__ uint32_t rep_hash(uint64_t o, int log2_slots) {
    return static_cast<uint32_t>((o * 0x9E3779B97F4A7C15ull) >> (64 - log2_slots));
}

// Value inserted by the Inj / Bij bitmap for element i, or false.
__device__ __forceinline__ bool inserted_value(const PropsArgs &a, int64_t i, int64_t *v_out) {
    const int64_t v = load_x(a.x, a.x64, i);
    *v_out = v;
    return a.lo <= v && v < a.hi;
}

__device__ __forceinline__ bool is_dup(const PropsArgs &a, int64_t v) {
    const uint64_t o = static_cast<uint64_t>(v - a.lo);
    return (a.dup[o >> 5] >> (o & 31)) & 1u;
}

// When more values repeat than the list holds: least index of every repeated
// value, in the global table (the second pass over it is props_finish's).
__device__ __forceinline__ void props_first(const PropsArgs &a) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.n; i += stride) {
        int64_t v;
        if (!inserted_value(a, i, &v) || !is_dup(a, v)) continue;
        const uint64_t o = static_cast<uint64_t>(v - a.lo);
        if (a.first64) atomicMin(a.first64 + o, static_cast<unsigned long long>(i));
        else atomicMin(a.first + o, static_cast<uint32_t>(i));
    }
}

// Streams X once more (only when some value repeats and the list held every
// repeated value).  Each workgroup first builds an LDS hash table of the
// listed values (entry: value - lo << 12 | position in the list; the layout
// depends on the insertion order, the positions do not).  Each in-Rcd value
// is looked up; for a listed value at index i, m = atomicMin(least index of
// its list position, i) returns the previous least index, and when there
// was one, the larger of m and i is at least the value's second occurrence,
// with equality for the arrival that meets the least two.  The least such
// proposal over all values is Inj's first violation.
constexpr int kRescanThreads = 1024;   // two workgroups per CU (LDS, and at most 64 VGPRs)
constexpr int kRepPosBits = 12;
static_assert(kRepCap <= (1 << kRepPosBits), "list position field");

template <bool X64, int UNROLL>
__global__ __launch_bounds__(kRescanThreads) __attribute__((amdgpu_waves_per_eu(8)))
void props_rescan_kernel(PropsArgs a) {
    constexpr int kPer = X64 ? 2 : 4;
    __shared__ unsigned long long tab[kRepSlots];
    const uint32_t nrep = a.st->nrep;
    if (nrep == 0) return;
    if (nrep > static_cast<uint32_t>(kRepCap)) {
        props_first(a);
        return;
    }
    uint32_t tsz = 64;
    while (tsz < 4 * nrep) tsz <<= 1;
    const int lg = __builtin_ctz(tsz);
    for (uint32_t s = threadIdx.x; s < tsz; s += blockDim.x) tab[s] = kEmptySlot;
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < nrep; k += blockDim.x) {
        const uint64_t o = a.rep[k];
        uint32_t h = rep_hash(o, lg);
        while (atomicCAS(tab + h, static_cast<unsigned long long>(kEmptySlot),
                         static_cast<unsigned long long>((o << kRepPosBits) | k)) != kEmptySlot)
            h = (h + 1) & (tsz - 1);
    }
    __syncthreads();
    unsigned long long cand = kNone;
    // a listed value at index i: propose its second occurrence
    auto found = [&](int64_t i, uint32_t k) {
        const unsigned long long m = atomicMin(a.rep_min + k, static_cast<unsigned long long>(i));
        if (m != kNone) {
            const unsigned long long p = m > static_cast<unsigned long long>(i) ? m : i;
            if (p < cand) cand = p;
        }
    };
    // the slot of o starting at h whose entry t was already read, or none
    auto probe = [&](int64_t i, uint64_t o, uint32_t h, unsigned long long t) {
        while (t != kEmptySlot) {
            if ((t >> kRepPosBits) == o) {
                found(i, static_cast<uint32_t>(t & ((1u << kRepPosBits) - 1)));
                return;
            }
            h = (h + 1) & (tsz - 1);
            t = tab[h];
        }
    };
    constexpr int K = UNROLL * kPer;
    const int64_t groups = a.n / kPer;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    // the next iteration's groups are loaded while this one's are looked up
    v4 raw[UNROLL], nxt[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const int64_t gi = g0 + u * stride;
        raw[u] = gi < groups ? __builtin_nontemporal_load(reinterpret_cast<const v4 *>(a.x) + gi) : v4{0, 0, 0, 0};
    }
    for (int64_t gb = g0; gb < groups; gb += UNROLL * stride) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int64_t gi = gb + (UNROLL + u) * stride;
            nxt[u] = gi < groups ? __builtin_nontemporal_load(reinterpret_cast<const v4 *>(a.x) + gi)
                                 : v4{0, 0, 0, 0};
        }
        // every first probe is read before any is examined
        uint64_t o[K];
        uint32_t h[K];
        unsigned long long t[K];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const bool live = gb + u * stride < groups;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int k = u * kPer + q;
                int64_t v;
                if constexpr (X64)
                    v = static_cast<int64_t>((static_cast<uint64_t>(raw[u][2 * q + 1]) << 32) | raw[u][2 * q]);
                else
                    v = static_cast<int32_t>(raw[u][q]);
                const bool in = live && a.lo <= v && v < a.hi;
                o[k] = static_cast<uint64_t>(v - a.lo);
                h[k] = rep_hash(o[k], lg);
                t[k] = in ? tab[h[k]] : kEmptySlot;
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int k = u * kPer + q;
                if (t[k] != kEmptySlot) probe((gb + u * stride) * kPer + q, o[k], h[k], t[k]);
            }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) raw[u] = nxt[u];
    }
    if (g0 == 0) {
        for (int64_t i = groups * kPer; i < a.n; ++i) {
            const int64_t v = load_x(a.x, X64 ? 1 : 0, i);
            if (!(a.lo <= v && v < a.hi)) continue;
            const uint64_t ov = static_cast<uint64_t>(v - a.lo);
            const uint32_t hv = rep_hash(ov, lg);
            probe(i, ov, hv, tab[hv]);
        }
    }
    cand = wave_min_u64(cand);
    if ((threadIdx.x & 63) == 0 && cand != kNone) atomicMin(&a.st->fv_inj, cand);
}

// The table's second pass: least index that is not the first occurrence of its
// value.
__device__ __forceinline__ void props_second(const PropsArgs &a) {
    unsigned long long c = kNone;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.n; i += stride) {
        int64_t v;
        if (!inserted_value(a, i, &v) || !is_dup(a, v)) continue;
        const uint64_t o = static_cast<uint64_t>(v - a.lo);
        const uint64_t f = a.first64 ? a.first64[o] : static_cast<uint64_t>(a.first[o]);
        if (static_cast<uint64_t>(i) != f && static_cast<unsigned long long>(i) < c) c = i;
    }
    c = wave_min_u64(c);
    if ((threadIdx.x & 63) == 0 && c != kNone) atomicMin(&a.st->fv_inj, c);
}

// Bij failing only on the count: least value of Img whose bit is clear.
__device__ __forceinline__ void props_missing(const PropsArgs &a) {
    PropsState *st = a.st;
    const int64_t b0 = a.ilo - a.lo, b1 = a.ihi - a.lo;   // bit range inside the bitmap
    unsigned long long c = kNone;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t w = (b0 >> 5) + static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
         w <= ((b1 - 1) >> 5); w += stride) {
        uint32_t clear = ~a.seen[w];
        const int64_t wb = w << 5;
        if (wb < b0) clear &= ~0u << (b0 - wb);
        if (wb + 32 > b1) clear &= (b1 - wb) >= 32 ? ~0u : ((1u << (b1 - wb)) - 1u);
        if (clear) {
            // offset from img_lo: values may be negative
            const unsigned long long v = static_cast<unsigned long long>(wb + __builtin_ctz(clear) + a.lo - a.ilo);
            if (v < c) c = v;
        }
    }
    c = wave_min_u64(c);
    if ((threadIdx.x & 63) == 0 && c != kNone) atomicMin(&st->missing, c);
}

// ---------------------------------------------------------------- FiltPart --
// The array is cut into at most kFpRanges contiguous ranges, one per workgroup
// of fp_check, in whole steps of kFpStep elements.
constexpr int kFpThreads = 256;
constexpr int kFpWaves = kFpThreads / kWave;
constexpr int kFpRows = 8;            // rows of 64 elements a wave holds at once
constexpr int64_t kFpStep = static_cast<int64_t>(kFpThreads) * kFpRows;
constexpr int64_t kFpRanges = 2048;   // 8 workgroups per CU
constexpr int64_t kNoZ = INT64_MIN;   // no earlier kept element of the class

struct FpElem {
    bool c;        // predicate
    bool kept;     // takes part (partition: all; filter: trues)
    int cls;       // class for the stability check
    int64_t z;
};

template <class Pred>
__device__ __forceinline__ bool fp_true(const PropsArgs &a, const Pred &pred, int64_t i) {
    uint32_t key = 0;
    uint8_t fl = 0;
    if constexpr (Pred::kUsesFlags) fl = pred.flags[i];
    else key = a.fp_src[i];
    return pred(key, fl);
}

template <class Pred>
__device__ __forceinline__ FpElem fp_elem(const PropsArgs &a, const Pred &pred, int64_t i) {
    FpElem e;
    e.c = fp_true(a, pred, i);
    e.kept = a.fp_mode == IXP_MODE_PARTITION || e.c;
    e.cls = a.fp_mode == IXP_MODE_PARTITION ? (e.c ? 1 : 0) : 1;
    e.z = load_x(a.x, a.x64, i);
    return e;
}

// True when the element takes part in FiltPart's bijection (its index lies in
// the range the outputs cover).
__device__ __forceinline__ bool fp_inserts(const PropsArgs &a, const FpElem &e, int64_t split) {
    return a.fp_mode == IXP_MODE_PARTITION ? (0 <= e.z && e.z < a.n)
                                           : (e.c && 0 <= e.z && e.z < split && e.z < a.n);
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    return static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(v), 0));
}

// Per range and class, the index value of the range's last kept element (kNoZ
// if none): what the next range's first element is compared with.  Searched
// backwards from the range's end, so it reads a few hundred keys of a range
// unless a class is rare in it.  With `init` it also clears the state (a call
// that checks FiltPart alone launches no props_init).
template <class Pred>
__global__ __launch_bounds__(kFpThreads) void fp_last_kernel(PropsArgs a, Pred pred, int init) {
    __shared__ int64_t found[kFpWaves][2];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int64_t b = blockIdx.x;
    if (init && b == 0 && tid == 0) {
        a.st->dup_found = 0;
        a.st->fp_fv = kNone;
        a.st->fp_bits = 0;
        a.st->done = 0;
    }
    const int64_t e0 = b * a.fp_range;
    const int64_t e1 = e0 + a.fp_range < a.n ? e0 + a.fp_range : a.n;
    const bool part = a.fp_mode == IXP_MODE_PARTITION;
    int64_t last[2] = {-1, -1};   // greatest index of each class found so far (uniform)
    int64_t hi = e1;
    // the first step takes 256 elements, one per thread; the later ones kFpStep
    for (int per = 1; hi > e0 && (last[1] < 0 || (part && last[0] < 0)); per = kFpRows) {
        const int64_t lo = hi - static_cast<int64_t>(per) * kFpThreads > e0
                               ? hi - static_cast<int64_t>(per) * kFpThreads : e0;
        int64_t m[2] = {-1, -1};
#pragma unroll
        for (int r = 0; r < kFpRows; ++r) {
            const int64_t i = lo + r * kFpThreads + tid;
            if (r < per && i < hi) {
                const bool c = fp_true(a, pred, i);
                if (c) m[1] = i;
                else if (part) m[0] = i;
            }
        }
        m[0] = wave_max_i64(m[0]);
        m[1] = wave_max_i64(m[1]);
        if (lane == 0) {
            found[wave][0] = m[0];
            found[wave][1] = m[1];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            int64_t x = -1;
            for (int w = 0; w < kFpWaves; ++w) x = found[w][k] > x ? found[w][k] : x;
            if (last[k] < 0) last[k] = x;
        }
        __syncthreads();
        hi = lo;
    }
    if (tid < 2) a.fp_last[tid * kFpRanges + b] = last[tid] >= 0 ? load_x(a.x, a.x64, last[tid]) : kNoZ;
}

// The general test of one wave's elements [w0, e1), at most kFpRows rows of 64,
// a row at a time: Bij's range part (bit 2), class order (bit 4), stability
// (bit 8) and the values moved (bit 16).  run[k] is the index value of the
// last kept element of class k before w0 (kNoZ if none).
//
// Stability compares an element with its predecessor in the class.  Up to the
// first failure the class is strictly increasing, so its running maximum is
// the predecessor: the least failing index is that of a comparison with the
// maximum of all earlier elements.  The predecessor inside a row comes from one
// ballot per class and a lane permute.
template <class Pred>
__device__ __forceinline__ void fp_general(const PropsArgs &a, const Pred &pred, int64_t w0, int64_t e1,
                                                     int64_t split, int64_t run0, int64_t run1,
                                                     unsigned long long *cand, uint32_t *bits) {
    const int lane = lane_id();
    const bool part = a.fp_mode == IXP_MODE_PARTITION;
    const int64_t ylen = part ? a.n : split;
#pragma unroll 1
    for (int r = 0; r < kFpRows && w0 + r * kWave < e1; ++r) {
        const int64_t i = w0 + r * kWave + lane;
        const bool live = i < e1;
        FpElem e{false, false, 0, 0};
        if (live) e = fp_elem(a, pred, i);
        const bool kept = live && e.kept;
        const uint64_t m1 = ballot(kept && e.cls == 1), m0 = ballot(kept && e.cls == 0);
        const uint64_t below = (e.cls ? m1 : m0) & ((1ull << lane) - 1);
        const int64_t pz = __shfl(e.z, below ? 63 - __builtin_clzll(below) : 0, kWave);
        const int64_t prev = below ? pz : (e.cls ? run1 : run0);
        uint32_t bad = 0;
        if (part) {
            if (!(0 <= e.z && e.z < a.n)) bad |= 2;
            if ((e.z < split) != e.c) bad |= 4;
        } else if (e.c) {
            if (!(0 <= e.z && e.z < split) || e.z >= a.n) bad |= 2;
        } else if (0 <= e.z && e.z < split) {
            bad |= 2;
        }
        if (kept && 0 <= e.z && e.z < ylen && e.z < a.n && a.fp_dst[e.z] != a.fp_src[i]) bad |= 16;
        if (kept && prev != kNoZ && !(e.z > prev)) bad |= 8;
        if (bad && live) {
            *bits |= bad;
            if (static_cast<unsigned long long>(i) < *cand) *cand = static_cast<unsigned long long>(i);
        }
        if (m1) run1 = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(e.z), 63 - __builtin_clzll(m1)));
        if (m0) run0 = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(e.z), 63 - __builtin_clzll(m0)));
    }
}

// Every element once.  Workgroup b takes range b in steps of kFpStep elements,
// a wave 512 of them; ranges, steps and waves hand on the index value of each
// class's last element.
//
// In a correct partition the index values of each class simply count on, so a
// wave first makes one comparison per element with that count (the sides of
// the split are then a matter of where the counts start and end) and one of
// the value moved; only a wave where that fails, or whose elements are not all
// there, takes the general test.
//
// Injectivity needs no bitmap here: when the class order and stability hold,
// the classes' index values are disjoint and strictly increasing, so nothing
// repeats.  fp_insert looks for repeats only after a failure of one of the
// two; this kernel clears the bitmaps it would use.
//
// Bound by memory: src, X and the gathered dst are read once (12 bytes per
// element with int32 indices, the gather being two ascending streams).  2^24
// int32 keys and indices: 45 us (4.5 TB/s); a global bitmap with an atomic per
// element and a 64-bit max-scan per row took 995 us.
template <bool X64, class Pred>
__global__ __launch_bounds__(kFpThreads) void fp_check_kernel(PropsArgs a, Pred pred) {
    using Z = typename std::conditional<X64, int64_t, int32_t>::type;
    __shared__ int64_t sh_in[2];
    __shared__ int64_t wlast[2][kFpWaves][2];   // by parity of the step
    __shared__ unsigned long long wcount[kFpWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = wave_id();
    const int64_t b = blockIdx.x;
    const int64_t e0 = b * a.fp_range;
    const int64_t e1 = e0 + a.fp_range < a.n ? e0 + a.fp_range : a.n;
    const bool part = a.fp_mode == IXP_MODE_PARTITION;
    const int64_t split = *a.fp_split;
    const Z *x = static_cast<const Z *>(a.x);
    // last value of each class before this range, 64 ranges at a time
    if (wave < 2) {
        int64_t in = kNoZ;
        for (int64_t j = b - 1; j >= 0; j -= kWave) {
            const int64_t v = j - lane >= 0 ? a.fp_last[wave * kFpRanges + j - lane] : kNoZ;
            const uint64_t m = ballot(v != kNoZ);
            if (m) {
                in = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(v), __builtin_ctzll(m)));
                break;
            }
        }
        if (lane == 0) sh_in[wave] = in;
    }
    for (int64_t w = (e0 >> 5) + tid; w < ((e1 + 31) >> 5); w += kFpThreads) {
        a.seen[w] = 0;
        a.dup[w] = 0;
    }
    __syncthreads();
    // index values that fit both the type and the array end before zmax, those
    // of the trues before ymax1, those read from dst before ymax
    const int64_t zmax = X64 || a.n < (int64_t{1} << 31) ? a.n : (int64_t{1} << 31);
    const int64_t ymax1 = split < zmax ? split : zmax;
    const int64_t ymax = part ? zmax : ymax1;
    int64_t carry[2] = {uniform_i64(sh_in[0]), uniform_i64(sh_in[1])};
    unsigned long long cand = kNone, trues = 0;
    uint32_t bits = 0;
    int par = 0;
    for (int64_t base = e0; base < e1; base += kFpStep, par ^= 1) {
        const int64_t w0 = base + static_cast<int64_t>(wave) * (kFpRows * kWave);
        const bool whole = w0 + kFpRows * kWave <= e1 && ymax > 0;   // (wave-uniform)
        uint32_t src[kFpRows], dst[kFpRows];
        Z z[kFpRows];
        uint64_t m1[kFpRows];   // trues of a row
        int64_t p0 = -1, p1 = -1;   // this wave's last element of each class
        if (whole) {
            uint8_t fl[kFpRows];
#pragma unroll
            for (int r = 0; r < kFpRows; ++r) {
                src[r] = __builtin_nontemporal_load(a.fp_src + w0 + r * kWave + lane);
                z[r] = __builtin_nontemporal_load(x + w0 + r * kWave + lane);
                fl[r] = 0;
                if constexpr (Pred::kUsesFlags) fl[r] = pred.flags[w0 + r * kWave + lane];
            }
#pragma unroll
            for (int r = 0; r < kFpRows; ++r) {
                const bool in = 0 <= z[r] && z[r] < ymax;
                dst[r] = a.fp_dst[in ? z[r] : Z{0}];
                m1[r] = ballot(pred(src[r], fl[r]));
                const int64_t i0 = w0 + r * kWave + 63;
                if (m1[r]) p1 = i0 - __builtin_clzll(m1[r]);
                if (~m1[r]) p0 = i0 - __builtin_clzll(~m1[r]);
                trues += static_cast<uint32_t>(__builtin_popcountll(m1[r]));
            }
        } else {
#pragma unroll 1
            for (int r = 0; r < kFpRows && w0 + r * kWave < e1; ++r) {
                const int64_t i = w0 + r * kWave + lane;
                const bool c = i < e1 && fp_true(a, pred, i);
                const uint64_t t = ballot(c), f = ballot(i < e1 && !c);
                const int64_t i0 = w0 + r * kWave + 63;
                if (t) p1 = i0 - __builtin_clzll(t);
                if (f) p0 = i0 - __builtin_clzll(f);
                trues += static_cast<uint32_t>(__builtin_popcountll(t));
            }
        }
        if (!part) p0 = -1;
        if (lane < 2) {
            const int64_t p = lane ? p1 : p0;
            wlast[par][wave][lane] = p >= 0 ? static_cast<int64_t>(x[p]) : kNoZ;
        }
        __syncthreads();
        int64_t run0 = carry[0], run1 = carry[1];
#pragma unroll
        for (int w = 0; w < kFpWaves; ++w) {
            const int64_t v0 = uniform_i64(wlast[par][w][0]), v1 = uniform_i64(wlast[par][w][1]);
            if (v0 != kNoZ) {
                carry[0] = v0;
                if (w < wave) run0 = v0;
            }
            if (v1 != kNoZ) {
                carry[1] = v1;
                if (w < wave) run1 = v1;
            }
        }
        bool good = whole;
        if (whole) {
            int n1 = 0;   // trues of the rows before
            bool ok = true;
#pragma unroll
            for (int r = 0; r < kFpRows; ++r) {
                const bool c = (m1[r] >> lane) & 1u;
                const int k1 = n1 + static_cast<int>(rank_below(m1[r]));
                const Z want = c ? static_cast<Z>(run1 + 1) + k1 : static_cast<Z>(run0 + 1) + (r * kWave + lane - k1);
                const bool keep = part | c;
                ok &= keep ? (z[r] == want) & (dst[r] == src[r]) : !(0 <= z[r] && z[r] < split);
                n1 += __builtin_popcountll(m1[r]);
            }
            const int n0 = part ? kFpRows * kWave - n1 : 0;
            good = ballot(ok) == ~0ull && (n1 == 0 || (run1 >= 0 && run1 + n1 < ymax1)) &&
                   (n0 == 0 || (run0 >= 0 && run0 >= split - 1 && run0 + n0 < zmax));
        }
        if (!good) fp_general(a, pred, w0, e1, split, run0, run1, &cand, &bits);
    }
    if (lane == 0) wcount[wave] = trues;   // (uniform: counted by ballots)
    if (ballot(bits != 0)) {
        cand = wave_min_u64(cand);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) bits |= __shfl_xor(bits, off, kWave);
        if (lane == 0) {
            atomicMin(&a.st->fp_fv, cand);
            atomicOr(&a.st->fp_bits, bits);
        }
    }
    __syncthreads();
    // one store per range: an atomic on one total would serialise the ranges
    if (tid == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < kFpWaves; ++w) t += wcount[w];
        a.fp_count[b] = t;
    }
}

// OR of a 32-bit value over the 64 lanes, wave-uniform (as wave_sum_u32).
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t v) {
    v |= dpp_row_ror<8>(v);
    v |= dpp_row_ror<4>(v);
    v |= dpp_row_ror<2>(v);
    v |= dpp_row_ror<1>(v);
    const int iv = static_cast<int>(v);
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(iv, 0) | __builtin_amdgcn_readlane(iv, 16) |
                                 __builtin_amdgcn_readlane(iv, 32) | __builtin_amdgcn_readlane(iv, 48));
}

// After a failed class order or stability check, repeats are possible: the
// bitmap insertions of the elements that take part in the bijection.  Bound by
// the atomics, which queue at a word: 64 elements of a nearly right partition lie
// in a few words (each class's indices count on), so the lanes of a word make one
// atomic for up to kFpWords words, and one each beyond.  (The whole check of 4 10^7 int32
// entries rolled by one / with one repeat: an atomic per element 3240 / 3090 us, so 660 /
// 565; inside fp_check, as it once was, 2420 / 2550.)
constexpr int kFpWords = 6;

template <class Pred>
__global__ __launch_bounds__(kPropsBlock) void fp_insert_kernel(PropsArgs a, Pred pred) {
    if (!(a.st->fp_bits & 12u)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t split = *a.fp_split;
    bool dup_seen = false;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + wave_id() * kWave; i0 < a.n; i0 += stride) {
        FpElem e{false, false, 0, 0};
        bool ins = false;
        if (i0 + lane < a.n) {
            e = fp_elem(a, pred, i0 + lane);
            ins = fp_inserts(a, e, split);   // (then 0 <= z < n, and lo is 0)
        }
        const uint32_t word = static_cast<uint32_t>(e.z >> 5), bit = 1u << (e.z & 31);
        uint64_t left = ballot(ins);
        for (int k = 0; k < kFpWords && left; ++k) {
            const int lead = __builtin_ctzll(left);
            const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(word), lead));
            const bool mine = ins && word == w;
            const uint64_t m = ballot(mine);
            const uint32_t bits = wave_or_u32(mine ? bit : 0u);
            left &= ~m;
            if (__builtin_popcount(bits) != __builtin_popcountll(m)) {   // repeats among these lanes
                if (mine) insert_value<false>(a, e.z, &dup_seen);
                continue;
            }
            uint32_t old = 0;
            if (lane == lead) old = atomicOr(a.seen + w, bits);
            old = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(old), lead));
            if (mine && (old & bit)) {
                note_repeat(a, static_cast<uint64_t>(e.z), false);
                dup_seen = true;
            }
        }
        if ((left >> lane) & 1u) insert_value<false>(a, e.z, &dup_seen);
    }
    if (ballot(dup_seen) != 0 && lane == 0) atomicOr(&a.st->dup_found, 1u);
}

// FiltPart's repeats, among the values fp_insert inserted: pass 0 takes the least
// index of each repeated value, pass 1 the least index that is not one of those.
template <class Pred>
__device__ __forceinline__ void fp_repeats(const PropsArgs &a, const Pred &pred, int pass) {
    const int64_t split = *a.fp_split;
    unsigned long long c = kNone;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.n; i += stride) {
        const FpElem e = fp_elem(a, pred, i);
        if (!fp_inserts(a, e, split) || !is_dup(a, e.z)) continue;
        const uint64_t o = static_cast<uint64_t>(e.z - a.lo);
        if (pass == 0) {
            if (a.first64) atomicMin(a.first64 + o, static_cast<unsigned long long>(i));
            else atomicMin(a.first + o, static_cast<uint32_t>(i));
        } else {
            const uint64_t f = a.first64 ? a.first64[o] : static_cast<uint64_t>(a.first[o]);
            if (static_cast<uint64_t>(i) != f && static_cast<unsigned long long>(i) < c) c = i;
        }
    }
    if (pass == 1) {
        c = wave_min_u64(c);
        if ((threadIdx.x & 63) == 0 && c != kNone) {
            atomicMin(&a.st->fp_fv, c);
            atomicOr(&a.st->fp_bits, 2u);
        }
    }
}

template <class Pred>
__global__ __launch_bounds__(kPropsBlock) void fp_first_kernel(PropsArgs a, Pred pred) {
    if (a.st->dup_found != 0) fp_repeats(a, pred, 0);
}

// Writes the five verdicts (one workgroup of at most 1024 threads, which first
// adds up the ranges' counts of trues for FiltPart).  The state is read past the
// caches: other workgroups of the same launch may have written it.
__device__ __forceinline__ void props_verdicts(const PropsArgs &a, ixp_verdict *out) {
    __shared__ unsigned long long wsum[1024 / kWave];
    unsigned long long fp_trues = 0;
    if (a.mask & IXP_FILTPART) {
        for (int64_t r = threadIdx.x; r < a.fp_nranges; r += blockDim.x) fp_trues += a.fp_count[r];
        fp_trues = wave_sum_u64(fp_trues);
        if ((threadIdx.x & (kWave - 1)) == 0) wsum[wave_id()] = fp_trues;
        __syncthreads();
        fp_trues = 0;
        for (uint32_t w = 0; w < blockDim.x / kWave; ++w) fp_trues += wsum[w];
    }
    if (threadIdx.x != 0) return;
    PropsState *s = a.st;
    auto get = [](const unsigned long long *p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const unsigned long long fv_range = get(&s->fv_range), fv_mono = get(&s->fv_mono), fv_img = get(&s->fv_img),
                             fv_inj = get(&s->fv_inj), in_count = get(&s->in_count), missing = get(&s->missing),
                             fp_fv = get(&s->fp_fv);
    uint32_t fp_bits = __hip_atomic_load(&s->fp_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int b = 0; b < 5; ++b) {
        out[b].holds = 1;
        out[b].reserved = 0;
        out[b].first_violation = -1;
        out[b].aux = 0;
    }
    auto fail = [&](int b, int64_t fv, int64_t aux) {
        out[b].holds = 0;
        out[b].first_violation = fv;
        out[b].aux = aux;
    };
    if ((a.mask & IXP_RANGE) && fv_range != kNone) fail(0, fv_range, load_x(a.x, a.x64, fv_range));
    if ((a.mask & IXP_MONO) && fv_mono != kNone) fail(1, fv_mono, 0);
    if ((a.mask & IXP_INJ) && fv_inj != kNone) fail(2, fv_inj, load_x(a.x, a.x64, fv_inj));
    if (a.mask & IXP_BIJ) {
        const unsigned long long f = fv_inj < fv_img ? fv_inj : fv_img;
        if (f != kNone) fail(3, f, load_x(a.x, a.x64, f));
        else if (static_cast<int64_t>(in_count) != a.ihi - a.ilo)
            fail(3, a.n, a.ilo + static_cast<int64_t>(missing));
    }
    if (a.mask & IXP_FILTPART) {
        if (static_cast<int64_t>(fp_trues) != *a.fp_split) fp_bits |= 1u;
        if (fp_bits) fail(4, fp_fv != kNone ? static_cast<int64_t>(fp_fv) : a.n, fp_bits);
    }
}

// True for the workgroup that passes here last of those that have `items` to go
// over.  They have made atomics on the state and no stores, so waiting for those
// orders them (so props_second, props_missing and fp_repeats may write nothing but
// such atomics, and props_verdicts reads past the caches): a fence in each of 2048 workgroups, with every workgroup counted,
// cost 100 us (a missing value among 5000 entries: 130 us, so 18.4).
__device__ __forceinline__ bool last_workgroup(const PropsArgs &a, int64_t items) {
    __shared__ int last;
    int64_t parts = (items + blockDim.x - 1) / blockDim.x;
    if (parts > gridDim.x) parts = gridDim.x;
    if (parts < 1) parts = 1;
    if (blockIdx.x >= parts) return false;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(&a.st->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == parts;
    __syncthreads();
    return last != 0;
}

// The last kernel of a call without FiltPart (`out` is NULL when FiltPart's
// follow): usually workgroup 0 writes the verdicts at once; a pass that is still
// needed (the table's second one, or the least missing value) takes the whole
// grid, and whichever workgroup ends last writes them.  A small call is bound by
// its launches, about 2 us each: with the table's two passes, the missing value
// and the verdicts in kernels of their own, Range, Inj and Bij of 5000 int64
// entries took 24 us, now 18 us (1e6 entries: 30.6, now 28.7).
__global__ __launch_bounds__(kPropsBlock) void props_finish_kernel(PropsArgs a, ixp_verdict *out) {
    const PropsState *st = a.st;
    const bool second = (a.mask & (IXP_INJ | IXP_BIJ)) && st->nrep > static_cast<uint32_t>(kRepCap);
    const bool missing = !second && (a.mask & IXP_BIJ) && !a.bucketed && st->fv_inj == kNone && st->fv_img == kNone &&
                         static_cast<int64_t>(st->in_count) != a.ihi - a.ilo;
    if (second) props_second(a);
    else if (missing) props_missing(a);
    if (!out) return;
    if (second || missing ? last_workgroup(a, second ? a.n : ((a.ihi - a.lo) >> 5) - ((a.ilo - a.lo) >> 5) + 1)
                          : blockIdx.x == 0)
        props_verdicts(a, out);
}

// The last kernel of a call with FiltPart.
template <class Pred>
__global__ __launch_bounds__(kPropsBlock) void fp_finish_kernel(PropsArgs a, PropsArgs main, Pred pred,
                                                                ixp_verdict *out) {
    const bool second = a.st->dup_found != 0;
    if (second) fp_repeats(a, pred, 1);
    if (second ? last_workgroup(a, a.n) : blockIdx.x == 0) props_verdicts(main, out);
}

template <class Pred>
int launch_filtpart(const PropsArgs &a, const PropsArgs &main, const Pred &pred, ixp_verdict *out, hipStream_t st,
                    int grid, bool init) {
    if (a.fp_nranges > 0) {
        const dim3 ranges(static_cast<uint32_t>(a.fp_nranges));
        IXP_LAUNCH("fp_last", (fp_last_kernel<Pred>), ranges, dim3(kFpThreads), 0, st, a, pred, init ? 1 : 0);
        if (a.x64) IXP_LAUNCH("fp_check", (fp_check_kernel<true, Pred>), ranges, dim3(kFpThreads), 0, st, a, pred);
        else IXP_LAUNCH("fp_check", (fp_check_kernel<false, Pred>), ranges, dim3(kFpThreads), 0, st, a, pred);
        IXP_LAUNCH("fp_insert", (fp_insert_kernel<Pred>), dim3(grid), dim3(kPropsBlock), 0, st, a, pred);
        IXP_LAUNCH("fp_first", (fp_first_kernel<Pred>), dim3(grid), dim3(kPropsBlock), 0, st, a, pred);
    }
    IXP_LAUNCH("fp_finish", (fp_finish_kernel<Pred>), dim3(grid), dim3(kPropsBlock), 0, st, a, main, pred, out);
    return launch_status();
}

}  // namespace
}  // namespace ixp

using namespace ixp;

namespace {
constexpr int kPass1Grid = 2048;   // fixed, so the workspace size does not depend on the device
constexpr int kRescanGrid = 512;

// Values per bucket: the narrowest power of two that leaves at most 256 buckets
// (one workgroup reads a bucket), so that props_check fills the chip whatever the
// width.  Range + Inj + Bij of a permutation, with buckets of 2^20 values / this
// rule: 2^17 entries 659 / 39 us, 2^20 762 / 42, 2^24 312 / 83, 2^27 538 / 431.  Up
// to 512 buckets: 2^27 490, 1024: 617 (the runs get shorter than two lines).
constexpr int64_t kBuckets = 256;
int bucket_shift(int64_t w) {
    int s = 5;   // whole bitmap words
    while (s < kBucketShift && ceil_div(w, int64_t{1} << s) > kBuckets) ++s;
    return s;
}

// Inj/Bij take the chunked path when Rcd spans at most kMaxBuckets buckets
// and the array is large enough for the extra pass to pay.
int buckets_for(int64_t n, uint32_t mask, const ixp_prop_args *a) {
    if (!(mask & (IXP_INJ | IXP_BIJ)) || !a) return 0;
    const int64_t w = a->hi - a->lo;
    if (w <= 0 || n < (int64_t{1} << 16) || n >= (int64_t{1} << 43)) return 0;
    const int64_t b = ceil_div(w, int64_t{1} << bucket_shift(w));
    // one workgroup reads each bucket: with more than 2^22 values per bucket
    // on average the global bitmap is faster
    if (n > (b << 22)) return 0;
    return b <= kMaxBuckets ? static_cast<int>(b) : 0;
}

// Buckets that a workspace has room for: the most that any Rcd of no more values
// takes (wider buckets may be fewer), so that one sized for the widest serves all.
int buckets_room(int64_t n, uint32_t mask, const ixp_prop_args *a) {
    if (!(mask & (IXP_INJ | IXP_BIJ)) || !a) return 0;
    const int64_t w = a->hi - a->lo;
    if (w > static_cast<int64_t>(kMaxBuckets) << kBucketShift) return 0;
    ixp_prop_args narrow{};
    narrow.hi = w < kBuckets << 5 ? w : kBuckets << 5;
    const int at = buckets_for(n, mask, a), most = buckets_for(n, mask, &narrow);
    return at > most ? at : most;
}

int64_t chunks_for(int64_t n) { return ceil_div(n, kChunk); }

// Chunked path: the chunks' records and the bucket-start table.
size_t bucket_bytes(int64_t n, int nb) {
    if (!nb) return 0;
    const int64_t nc = chunks_for(n);
    return round_up(static_cast<size_t>(nc) * kChunk * 4, 256) +
           round_up(static_cast<size_t>(nb + 1) * nc * 2, 256);
}

// The repeated-value list, its hash table and each slot's least index.
constexpr size_t kRepBytes = 2 * static_cast<size_t>(kRepCap) * 8;

// FiltPart's per-range records: two last values and a count each.
constexpr size_t kFpBytes = static_cast<size_t>(kFpRanges) * 24;

int64_t rcd_width(int64_t n, uint32_t mask, const ixp_prop_args *a) {
    int64_t w = 0;
    if ((mask & (IXP_INJ | IXP_BIJ)) && a) w = a->hi - a->lo;
    if (mask & IXP_FILTPART) w = w > n ? w : n;
    return w;
}
}  // namespace

extern "C" size_t ixp_check_props_workspace(int64_t n, uint32_t mask, const ixp_prop_args *a) {
    if (n < 0) return 0;
    if ((mask & (IXP_INJ | IXP_BIJ | IXP_FILTPART)) && !a) return 0;
    if ((mask & (IXP_INJ | IXP_BIJ)) && (a->hi < a->lo || a->hi - a->lo > (int64_t{1} << 36))) return 0;
    const int64_t w = rcd_width(n, mask, a);
    const size_t words = static_cast<size_t>((w + 127) / 128 * 4);   // multiple of 4 words
    const size_t first_bytes = static_cast<size_t>(w) * (n >= (int64_t{1} << 32) ? 8 : 4);
    return kPropsHeader + 2 * round_up(words * 4, 256) + round_up(first_bytes, 256) +
           ((mask & IXP_FILTPART) ? kFpBytes : 0) + kRepBytes +
           bucket_bytes(n, buckets_room(n, mask, a));
}

extern "C" int ixp_check_props(const void *x, int32_t x_t, int64_t n, uint32_t mask,
                               const ixp_prop_args *args, ixp_verdict *d_out, void *ws,
                               size_t ws_bytes, void *stream) {
    if (n < 0 || !d_out || (mask & ~31u)) return IXP_EINVAL;
    if (x_t != IXP_I32 && x_t != IXP_I64) return IXP_EINVAL;
    if (n > 0 && !x) return IXP_EINVAL;
    const size_t esz = x_t == IXP_I64 ? 8 : 4;
    if (!aligned(x, 16) || !aligned(d_out, 8) || !aligned(ws, 256)) return IXP_EINVAL;
    if ((mask & ~static_cast<uint32_t>(IXP_MONO)) && !args) return IXP_EINVAL;
    ixp_prop_args dflt{};
    const ixp_prop_args *pa = args ? args : &dflt;
    if (mask & (IXP_INJ | IXP_BIJ)) {
        if (pa->hi < pa->lo || pa->hi - pa->lo > (int64_t{1} << 36)) return IXP_EINVAL;
    }
    if (mask & IXP_BIJ) {
        if (pa->img_lo > pa->img_hi || pa->img_lo < pa->lo || pa->img_hi > pa->hi) return IXP_EINVAL;
    }
    if ((mask & IXP_MONO) && (pa->mono_op < 0 || pa->mono_op > 3)) return IXP_EINVAL;
    HostPred hp{};
    if (mask & IXP_FILTPART) {
        if (pa->fp_mode != IXP_MODE_PARTITION && pa->fp_mode != IXP_MODE_FILTER) return IXP_EINVAL;
        if (!pa->fp_split || !pa->fp_dst || (n > 0 && !pa->fp_src && pa->fp_pred.kind != IXP_PRED_FLAGS))
            return IXP_EINVAL;
        int rc = check_pred(&pa->fp_pred, pa->fp_key_t, &hp, n);
        if (rc != IXP_OK) return rc;
        if (is_row_pred(hp.kind)) return IXP_EINVAL;
        if (!pa->fp_src) return IXP_EINVAL;
        if (!aligned(pa->fp_src, 4) || !aligned(pa->fp_dst, 4) || !aligned(pa->fp_split, 8)) return IXP_EINVAL;
    }
    if (!ws || ws_bytes < ixp_check_props_workspace(n, mask, pa)) return IXP_EWORKSPACE;
    (void)esz;

    hipStream_t st = as_stream(stream);
    const int64_t w = rcd_width(n, mask, pa);
    const int64_t words = (w + 127) / 128 * 4;
    char *p = static_cast<char *>(ws);
    PropsArgs a{};
    a.x = x;
    a.x64 = x_t == IXP_I64 ? 1 : 0;
    a.n = n;
    a.mask = mask;
    a.lo = (mask & (IXP_INJ | IXP_BIJ)) ? pa->lo : 0;
    a.hi = (mask & (IXP_INJ | IXP_BIJ)) ? pa->hi : 0;
    a.ilo = pa->img_lo;
    a.ihi = pa->img_hi;
    a.mono_op = pa->mono_op;
    a.st = reinterpret_cast<PropsState *>(p);
    a.seen = reinterpret_cast<uint32_t *>(p + kPropsHeader);
    a.dup = reinterpret_cast<uint32_t *>(p + kPropsHeader + round_up(words * 4, 256));
    char *fp = p + kPropsHeader + 2 * round_up(words * 4, 256);
    if (n >= (int64_t{1} << 32)) {
        a.first64 = reinterpret_cast<unsigned long long *>(fp);
        a.first = nullptr;
    } else {
        a.first = reinterpret_cast<uint32_t *>(fp);
        a.first64 = nullptr;
    }
    a.width = w;
    const size_t first_bytes = static_cast<size_t>(w) * (n >= (int64_t{1} << 32) ? 8 : 4);
    a.fp_last = reinterpret_cast<int64_t *>(fp + round_up(first_bytes, 256));
    a.fp_count = reinterpret_cast<unsigned long long *>(a.fp_last + 2 * kFpRanges);
    if (mask & IXP_FILTPART) {
        a.fp_range = ceil_div(ceil_div(n, kFpRanges), kFpStep) * kFpStep;
        a.fp_nranges = n > 0 ? ceil_div(n, a.fp_range) : 0;
    }
    a.nbuckets = buckets_for(n, mask, pa);
    a.bucketed = a.nbuckets > 0 ? 1 : 0;
    if (a.bucketed) a.bshift = bucket_shift(pa->hi - pa->lo);
    char *rp = reinterpret_cast<char *>(a.fp_last) + ((mask & IXP_FILTPART) ? kFpBytes : 0);
    a.rep = reinterpret_cast<uint64_t *>(rp);
    a.rep_min = reinterpret_cast<unsigned long long *>(a.rep + kRepCap);
    if (a.bucketed) {
        char *bp = rp + kRepBytes;
        a.nchunks = chunks_for(n);
        a.records = reinterpret_cast<uint32_t *>(bp);
        a.ctab = reinterpret_cast<uint16_t *>(bp + round_up(static_cast<size_t>(a.nchunks) * kChunk * 4, 256));
    }
    a.fp_src = static_cast<const uint32_t *>(pa->fp_src);
    a.fp_dst = static_cast<const uint32_t *>(pa->fp_dst);
    a.fp_split = pa->fp_split;
    a.fp_mode = pa->fp_mode;

    const int grid = kPass1Grid;
    const int64_t iwords = words > 0 ? words : 1;
    const uint32_t iblocks = static_cast<uint32_t>(ceil_div(iwords / 4 + 1, 256) < 4096 ? ceil_div(iwords / 4 + 1, 256) : 4096);
    const uint32_t main_mask = mask & (IXP_RANGE | IXP_MONO | IXP_INJ | IXP_BIJ);
    // FiltPart alone initialises what it uses itself
    const bool fp_only = main_mask == 0 && a.fp_nranges > 0;
    // the chunked path reads no seen bitmap: only the dup bitmap is cleared
    if (!fp_only)
        IXP_LAUNCH("props_init", props_init_kernel, dim3(iblocks), dim3(256), 0, st, a.st,
               a.bucketed ? static_cast<uint32_t *>(nullptr) : a.seen, a.dup, words, a.rep_min);
    if (launch_status() != IXP_OK) return IXP_EHIP;

    if (main_mask && n > 0) {
        PropsArgs b = a;
        b.mask = main_mask;
        if (b.bucketed) {
            const size_t scan_lds = static_cast<size_t>(b.nbuckets + 1) * 4;   // bucket counts
            if (b.x64)
                IXP_LAUNCH("props_scan", props_scan_kernel<true>, dim3(static_cast<uint32_t>(b.nchunks)),
                           dim3(kScanThreads), scan_lds, st, b);
            else
                IXP_LAUNCH("props_scan", props_scan_kernel<false>, dim3(static_cast<uint32_t>(b.nchunks)),
                           dim3(kScanThreads), scan_lds, st, b);
            if (b.bshift < kBucketShift)
                IXP_LAUNCH("props_check", props_check_kernel<kBucketShift - 1>, dim3(b.nbuckets), dim3(kCheckThreads),
                           0, st, b);
            else
                IXP_LAUNCH("props_check", props_check_kernel<kBucketShift>, dim3(b.nbuckets), dim3(kCheckThreads), 0,
                           st, b);
        } else if (b.x64) {
            IXP_LAUNCH("props_pass1", (props_pass1_kernel<true, 4>), dim3(grid), dim3(kPropsBlock), 0, st, b);
        } else {
            IXP_LAUNCH("props_pass1", (props_pass1_kernel<false, 4>), dim3(grid), dim3(kPropsBlock), 0, st, b);
        }
        if (main_mask & (IXP_INJ | IXP_BIJ)) {
            if (b.x64)
                IXP_LAUNCH("props_rescan", (props_rescan_kernel<true, 2>), dim3(kRescanGrid), dim3(kRescanThreads),
                           0, st, b);
            else
                IXP_LAUNCH("props_rescan", (props_rescan_kernel<false, 1>), dim3(kRescanGrid), dim3(kRescanThreads),
                           0, st, b);
        }
        if (launch_status() != IXP_OK) return IXP_EHIP;
    }
    ixp_verdict *const fp_none = nullptr;
    if (main_mask || !(mask & IXP_FILTPART)) {
        PropsArgs b = a;
        b.mask = main_mask;
        IXP_LAUNCH("props_finish", props_finish_kernel, dim3(grid), dim3(kPropsBlock), 0, st, b,
                   (mask & IXP_FILTPART) ? fp_none : d_out);
    }
    if (mask & IXP_FILTPART) {
        // FiltPart's bijection check uses its own bitmap over [0, n): the
        // Inj/Bij passes above are done with it.
        PropsArgs f = a;
        f.lo = 0;
        f.hi = n;
        int rc = IXP_OK;
        switch (hp.kind) {
        case IXP_PRED_MOD_EQ: rc = launch_filtpart(f, a, mod_eq_pred(hp.d, hp.r), d_out, st, grid, fp_only); break;
        case IXP_PRED_LT: rc = launch_filtpart(f, a, PredLt{hp.s}, d_out, st, grid, fp_only); break;
        default: rc = launch_filtpart(f, a, PredFlags{hp.flags}, d_out, st, grid, fp_only); break;
        }
        if (rc != IXP_OK) return rc;
    }
    return launch_status();
}
