// flatv.hip -- v-way stable partition on gfx950 (FiltPart with v pairwise
// exclusive predicates, Section 2.3; partition3 of Section 6 is v = 3).
//
// Element i has a class c(i) in [0, v); class 0 comes first, then class 1,
// and so on, each class in input order:
//   idx[i] = B_{c(i)} + (number of earlier elements of class c(i)),
//   B_c = N_0 + ... + N_{c-1},   N_c = size of class c.
// It is partition2 with v - 1 counters instead of one.  Three kernels, as for
// partition2:
//   count   -- one workgroup per tile up to 8192 tiles, else one wave per
//              contiguous run of tiles: per-class counts by cumulative ballots
//              + popcount (each tile's prefix inside its run and the totals);
//   scan    -- one workgroup: exclusive scan of the totals of every class but
//              the last, and the class sizes N_c;
//   scatter -- one workgroup per tile: per-class in-tile ranks from one packed
//              DPP scan per row, indices in input order, keys staged in LDS
//              class by class and written as v contiguous runs.
#include "device.hpp"
#include "host.hpp"

namespace ixp {
namespace {

constexpr int kVBlockThreads = 256;   // scatter tile: 256 threads x 4 rows x 4
constexpr int kVRows = 4;
constexpr int64_t kVCountWaves = 8192;
constexpr size_t kVHeader = 256;

// ------------------------------------------------------------------ classes --
// floor-mod(key, V) of an int32 key: the low bits for V = 2 and 4; for V = 3
// u = key + 2^31 has the key's floor modulus plus 2, and u / 3 is the high
// half of u (2^33 + 1) / 3 by 2.
template <int V>
struct ClassMod {
    static constexpr bool kUsesBytes = false;
    __device__ __forceinline__ uint32_t operator()(uint32_t bits, uint8_t) const {
        if (V != 3) return bits & static_cast<uint32_t>(V - 1);
        const uint32_t u = bits ^ 0x80000000u;
        const uint32_t m = u - 3u * (__umulhi(u, 0xAAAAAAABu) >> 1);
        return m == 2 ? 0u : m + 1;
    }
    // class <= K, for the counts
    template <int K>
    __device__ __forceinline__ bool upto(uint32_t bits, uint8_t b) const { return (*this)(bits, b) <= K; }
};

// f32 thresholds s0 <= s1 <= s2: class h for s_{h-1} <= x < s_h, the last
// class for x >= s_{v-2} and for NaN (which no earlier predicate takes).
template <int V>
struct ClassThresh {
    static constexpr bool kUsesBytes = false;
    float s0, s1, s2;
    __device__ __forceinline__ uint32_t operator()(uint32_t bits, uint8_t) const {
        const float x = __uint_as_float(bits);
        if (x < s0) return 0;
        if (V > 2 && x < s1) return 1;
        if (V > 3 && x < s2) return 2;
        return V - 1;
    }
    template <int K>   // (the thresholds do not decrease)
    __device__ __forceinline__ bool upto(uint32_t bits, uint8_t) const {
        return __uint_as_float(bits) < (K == 0 ? s0 : K == 1 ? s1 : s2);
    }
};

// A caller byte per element; values past the last class count as the last.
template <int V>
struct ClassBytes {
    static constexpr bool kUsesBytes = true;
    const uint8_t *cls;
    __device__ __forceinline__ uint32_t operator()(uint32_t, uint8_t b) const {
        return b < V - 1 ? b : V - 1;
    }
    template <int K>
    __device__ __forceinline__ bool upto(uint32_t, uint8_t b) const { return b <= K; }
};

// a[c] for a class c < V, as a[0] plus the steps a[k] - a[k-1] of every
// k <= c.  Compares and adds only: a chain of selects on c == k is turned by
// the compiler into an indexed load from a per-lane scratch copy of a[].
template <int V, class T>
struct Picker {
    T a0;
    T step[V - 1];
    __device__ __forceinline__ explicit Picker(const T (&a)[V]) : a0(a[0]) {
#pragma unroll
        for (int k = 1; k < V; ++k) step[k - 1] = a[k] - a[k - 1];
    }
    __device__ __forceinline__ T operator()(uint32_t c) const {
        T r = a0;
#pragma unroll
        for (int k = 1; k < V; ++k) r += c >= static_cast<uint32_t>(k) ? step[k - 1] : T{0};
        return r;
    }
};

// --------------------------------------------------------------------- tile --
// Same element layout as the partition2 tile (wave w owns a contiguous run,
// row r, lane l, quad q); the class of each element is kept as two bit planes.
template <int BLOCK, int ROWS, int V>
struct TileV {
    static constexpr int kWaves = BLOCK / kWave;
    static constexpr int kPerWave = ROWS * kWave * 4;
    static constexpr int kSize = BLOCK * ROWS * 4;
    static_assert(ROWS * 4 <= 32, "class bit planes");

    uint32_t key[ROWS][4];
    uint32_t rank[ROWS][4];   // rank among the tile's elements of the same class
    uint32_t c0 = 0, c1 = 0, vbits = 0;
    uint64_t wtotal = 0;   // packed per-class counts of this wave's run

    __device__ static __forceinline__ int64_t pos(int64_t base, int wave, int r, int lane) {
        return base + static_cast<int64_t>(wave) * kPerWave + r * (kWave * 4) + lane * 4;
    }
    __device__ __forceinline__ uint32_t cls(int r, int q) const {
        const int i = r * 4 + q;
        return ((c0 >> i) & 1u) | (((c1 >> i) & 1u) << 1);
    }
    __device__ __forceinline__ bool valid(int r, int q) const { return (vbits >> (r * 4 + q)) & 1u; }

    // Keys (if need_keys) and class bytes (for byte classes) of [lo, hi):
    // one unconditional 16-byte load per row for whole tiles, parked loads
    // for partial tiles, guarded element loads where the array's last group
    // is incomplete.
    // NT = false: plain loads.
    template <bool NT, class Cls>
    __device__ __forceinline__ void load(const uint32_t *keys, int64_t n, int64_t base, int64_t lo, int64_t hi,
                                         const Cls &cl, bool need_keys, int wave, int lane) {
        const bool tail = (n & 3) != 0 && hi > (n & ~int64_t{3});
        uint32_t kv[ROWS][4];
        uint8_t bv[ROWS][4];
        if (!tail) {
            const bool whole = base >= lo && base + kSize <= hi;
            const int64_t park = lo & ~int64_t{3};
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int64_t p0 = pos(base, wave, r, lane);
                const bool live = whole || (p0 + 4 > lo && p0 < hi);
                const int64_t src = live ? p0 : park;
                uint32_t k4[4];
                if (need_keys) load_group<4, NT>(keys + src, k4);
                else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) k4[q] = 0;
                }
                uint8_t b4[4] = {0, 0, 0, 0};
                if constexpr (Cls::kUsesBytes) load_flags<4, NT>(cl.cls + src, b4);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    kv[r][q] = k4[q];
                    bv[r][q] = b4[q];
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int64_t p0 = pos(base, wave, r, lane);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t p = p0 + q;
                    const bool ok = p >= lo && p < hi;
                    kv[r][q] = (need_keys && ok) ? keys[p] : 0u;
                    if constexpr (Cls::kUsesBytes) bv[r][q] = ok ? cl.cls[p] : 0;
                    else bv[r][q] = 0;
                }
            }
        }
        const int32_t l0 = static_cast<int32_t>(base - lo) + wave * kPerWave + lane * 4;
        const uint32_t span = static_cast<uint32_t>(hi - lo);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t l = l0 + r * (kWave * 4) + q;
                const bool ok = static_cast<uint32_t>(l) < span;
                key[r][q] = kv[r][q];
                const uint32_t c = ok ? cl(kv[r][q], bv[r][q]) : 0u;
                const int i = r * 4 + q;
                vbits |= static_cast<uint32_t>(ok) << i;
                c0 |= (c & 1u) << i;
                c1 |= ((c >> 1) & 1u) << i;
            }
        }
    }

    // Counts of the classes, packed 16 bits each in a 64-bit word (a class holds
    // at most 4096 elements of a tile, so no field overflows).
    __device__ static __forceinline__ uint32_t field(uint64_t x, uint32_t c) {
        return static_cast<uint32_t>(x >> (16 * c)) & 0xFFFFu;
    }

    // Ranks inside this wave's run.  Per row, the counts of every class but
    // the last are packed 9 bits each into 32 bits (a row of a wave holds at
    // most 256 elements) and scanned over the lanes by DPP (all lanes take
    // part); the rank of a last-class element is its position minus the earlier elements of
    // the other classes (the valid elements of a run form a prefix).
    __device__ static __forceinline__ uint32_t onehot9(uint32_t c, bool ok) {
        return (ok && c < static_cast<uint32_t>(V - 1)) ? (1u << (9 * c)) : 0u;
    }
    __device__ __forceinline__ void wave_ranks(int lane) {
        uint64_t acc = 0;   // packed 16-bit counts of the earlier rows (uniform)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            uint32_t mine = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) mine += onehot9(cls(r, q), valid(r, q));
            const uint32_t inc = wave_scan_u32(mine);
            uint32_t run = inc - mine;
            const uint32_t pos0 = static_cast<uint32_t>(r * kWave * 4 + lane * 4);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t c = cls(r, q);
                uint32_t others = 0;   // earlier elements of the classes before the last
#pragma unroll
                for (int k = 0; k < V - 1; ++k) others += field(acc, k) + ((run >> (9 * k)) & 0x1FFu);
                const uint32_t mine_c = c < static_cast<uint32_t>(V - 1)
                                            ? field(acc, c) + ((run >> (9 * c)) & 0x1FFu)
                                            : pos0 + q - others;
                rank[r][q] = mine_c;
                run += onehot9(c, valid(r, q));
            }
            const uint32_t row = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), kWave - 1));
#pragma unroll
            for (int k = 0; k < V - 1; ++k) acc += static_cast<uint64_t>((row >> (9 * k)) & 0x1FFu) << (16 * k);
        }
        // the last class of the run: valid elements minus the others
        uint32_t nvalid = static_cast<uint32_t>(__builtin_popcount(vbits));
        nvalid = wave_sum_u32(nvalid);
        uint32_t others = 0;
#pragma unroll
        for (int k = 0; k < V - 1; ++k) others += field(acc, k);
        wtotal = acc + (static_cast<uint64_t>(nvalid - others) << (16 * (V - 1)));
    }

    // Adds each wave's per-class offset to its ranks; returns the tile's
    // packed class sizes.
    __device__ __forceinline__ uint64_t block_ranks(uint64_t *wt, int wave, int lane) {
        if (lane == 0) wt[wave] = wtotal;
        __syncthreads();
        uint64_t before = 0, tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint64_t x = wt[w];
            before += w < wave ? x : 0ull;
            tot += x;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) rank[r][q] += field(before, cls(r, q));
        return tot;
    }
};

struct VArgs {
    const uint32_t *keys;
    int64_t n;
    uint32_t *out_keys;
    void *out_idx;
    int64_t *counts;          // [v] class sizes (output)
    uint64_t *desc;           // [num_tiles][4] per-class prefix of the tile inside its run
    int64_t *wsum;            // [3][kVCountWaves] run totals, then run prefixes
    int64_t num_tiles;
    int64_t tiles_per_wave;
    int32_t need_keys;
};

// Adds to cum[k] the elements of class <= k of one ballot's worth of elements.
template <int V, class Cls>
__device__ __forceinline__ void count_upto(const Cls &cl, uint32_t key, uint8_t byte, bool ok, uint32_t (&cum)[V - 1]) {
    cum[0] += static_cast<uint32_t>(__builtin_popcountll(ballot(ok && cl.template upto<0>(key, byte))));
    if constexpr (V > 2)
        cum[1] += static_cast<uint32_t>(__builtin_popcountll(ballot(ok && cl.template upto<1>(key, byte))));
    if constexpr (V > 3)
        cum[2] += static_cast<uint32_t>(__builtin_popcountll(ballot(ok && cl.template upto<2>(key, byte))));
}

// cum[k] = elements of class <= k among [lo, lo + kRows 64 x 4) before n, by one
// wave; all its loads in flight at once where the stretch is whole.
template <int V, int kRows, bool NT, class Cls>
__device__ __forceinline__ void wave_upto(const VArgs &a, const Cls &cl, int64_t lo, int lane, uint32_t (&cum)[V - 1]) {
#pragma unroll
    for (int k = 0; k < V - 1; ++k) cum[k] = 0;
    if (lo + kRows * kWave * 4 <= a.n) {
        uint32_t key[kRows][4];
        uint8_t byte[kRows][4];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t p = lo + r * (kWave * 4) + lane * 4;
            if constexpr (Cls::kUsesBytes) load_flags<4, NT>(cl.cls + p, byte[r]);
            else load_group<4, NT>(a.keys + p, key[r]);
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                count_upto<V>(cl, Cls::kUsesBytes ? 0u : key[r][q], Cls::kUsesBytes ? byte[r][q] : uint8_t{0}, true, cum);
    } else {
        const int64_t hi = lo + kRows * kWave * 4 < a.n ? lo + kRows * kWave * 4 : a.n;
        for (int64_t p = lo + lane; p - lane < hi; p += kWave) {
            const bool ok = p < hi;
            uint32_t key = 0;
            uint8_t byte = 0;
            if constexpr (Cls::kUsesBytes) byte = ok ? cl.cls[p] : 0;
            else key = ok ? a.keys[p] : 0u;
            count_upto<V>(cl, key, byte, ok, cum);
        }
    }
}

// One wave per contiguous run of tiles, a whole tile per batch of loads.  The
// classes are counted cumulatively (class <= k), one comparison and one scalar
// popcount per element row and class: packed one-hot counters took a dozen
// vector instructions an element and held the registers of half the batch
// (5 10^7 keys in 3 classes 42 -> 35 us, 2 10^8 by modulus 182 -> 132).
template <int V, class Cls, bool NT>
__global__ __launch_bounds__(256) void flatv_count_kernel(VArgs a, Cls cl) {
    constexpr int kTile = kVBlockThreads * kVRows * 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t w = static_cast<int64_t>(blockIdx.x) * (256 / kWave) + wave_id();
    const int64_t t0 = w * a.tiles_per_wave;
    const int64_t t1 = t0 + a.tiles_per_wave < a.num_tiles ? t0 + a.tiles_per_wave : a.num_tiles;
    uint64_t run[V - 1];
#pragma unroll
    for (int k = 0; k < V - 1; ++k) run[k] = 0;
    for (int64_t t = t0; t < t1; ++t) {
        uint32_t cum[V - 1];
        wave_upto<V, kTile / (kWave * 4), NT>(a, cl, t * kTile, lane, cum);
        if (lane < V - 1) {
            uint64_t mine = run[0];
#pragma unroll
            for (int k = 1; k < V - 1; ++k) mine = lane == k ? run[k] : mine;
            a.desc[t * 4 + lane] = mine;
        }
#pragma unroll
        for (int k = 0; k < V - 1; ++k) run[k] += cum[k] - (k > 0 ? cum[k - 1] : 0u);
    }
    if (lane < V - 1 && w < kVCountWaves) {
        uint64_t mine = run[0];
#pragma unroll
        for (int k = 1; k < V - 1; ++k) mine = lane == k ? run[k] : mine;
        a.wsum[lane * kVCountWaves + w] = static_cast<int64_t>(mine);
    }
}

// The same where a run is one tile: a workgroup per tile, a wave per quarter
// (one wave a tile leaves most of the chip idle).
template <int V, class Cls, bool NT>
__global__ __launch_bounds__(256) void flatv_count_small_kernel(VArgs a, Cls cl) {
    constexpr int kQuarter = kVBlockThreads * kVRows;
    __shared__ uint32_t sh[4][V - 1];
    const int lane = threadIdx.x & (kWave - 1), wave = wave_id();
    const int64_t t = blockIdx.x;
    uint32_t cum[V - 1];
    wave_upto<V, kQuarter / (kWave * 4), NT>(a, cl, (4 * t + wave) * kQuarter, lane, cum);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < V - 1; ++k) sh[wave][k] = cum[k] - (k > 0 ? cum[k - 1] : 0u);
    }
    __syncthreads();
    if (threadIdx.x < V - 1) {
        const int k = threadIdx.x;
        a.desc[t * 4 + k] = 0;
        a.wsum[k * kVCountWaves + t] = static_cast<int64_t>(sh[0][k]) + sh[1][k] + sh[2][k] + sh[3][k];
    }
}

// One workgroup: for every class but the last, the tiles' totals become
// exclusive prefixes (a wave takes 8 rows of 64 consecutive entries, LDS across
// the waves; the classes side by side, so that their loads and barriers are
// shared); the class sizes go to counts[0..v).  Bound by one CU's loads: with 8
// consecutive entries to a thread a load touches 64 lines; so, 8 rows of 64, the
// 3-way partition of 5e7 keys took 130.6 us with it, now 125.6, the 4-way one
// 142 us, now 134.
template <int V>
__global__ __launch_bounds__(1024) void flatv_scan_kernel(int64_t *wsum, int64_t nw, int64_t n, int64_t *counts) {
    constexpr int kPer = 8;
    static_assert(kPer * 1024 >= kVCountWaves, "scan capacity");
    __shared__ int64_t wtot[V - 1][16];
    const int tid = threadIdx.x;
    const int wave = wave_id();
    const int64_t i0 = static_cast<int64_t>(wave) * kPer * kWave + (tid & (kWave - 1));
    int64_t v[V - 1][kPer];
#pragma unroll
    for (int k = 0; k < V - 1; ++k) {
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            v[k][j] = i0 + j * kWave < nw ? wsum[k * kVCountWaves + i0 + j * kWave] : 0;
    }
#pragma unroll
    for (int k = 0; k < V - 1; ++k) {
        const int64_t run = wave_rows_prefix(v[k], ceil_div(nw, kWave) - wave * kPer);
        if ((tid & (kWave - 1)) == 0) wtot[k][wave] = run;
    }
    __syncthreads();
    int64_t rest = n;
#pragma unroll
    for (int k = 0; k < V - 1; ++k) {
        int64_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int64_t x = wtot[k][w];
            before += w < wave ? x : 0;
            total += x;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (i0 + j * kWave < nw) wsum[k * kVCountWaves + i0 + j * kWave] = before + v[k][j];
        if (tid == 0) counts[k] = total;
        rest -= total;
    }
    if (tid == 0) counts[V - 1] = rest;
}

template <int V, class Cls, class Idx, bool NT>
__global__ __launch_bounds__(kVBlockThreads) void flatv_scatter_kernel(VArgs a, Cls cl) {
    using T = TileV<kVBlockThreads, kVRows, V>;
    constexpr int kTile = T::kSize;
    __shared__ uint32_t stage[kTile];
    __shared__ uint64_t wt[T::kWaves];

    const int tid = threadIdx.x;
    const int wave = wave_id();
    const int lane = tid & (kWave - 1);
    const int64_t t = blockIdx.x;   // (the XCD-aware order of the 2-way scatter measured 1 % slower here)
    const int64_t lo = t * kTile;
    const int64_t hi = lo + kTile < a.n ? lo + kTile : a.n;

    // destination of the tile's first element of each class:
    // B_c (classes before c) + elements of class c before the tile
    int64_t dst[V];
    {
        int64_t before_tile = 0, base = 0;
#pragma unroll
        for (int k = 0; k < V - 1; ++k) {
            const int64_t e = static_cast<int64_t>(a.desc[t * 4 + k]) +
                              a.wsum[k * kVCountWaves + t / a.tiles_per_wave];
            dst[k] = base + e;
            before_tile += e;
            base += a.counts[k];
        }
        dst[V - 1] = base + (lo - before_tile);
    }

    T tile;
    tile.template load<NT>(a.keys, a.n, lo, lo, hi, cl, a.need_keys != 0, wave, lane);
    tile.wave_ranks(lane);
    const uint64_t ptot = tile.block_ranks(wt, wave, lane);
    uint32_t tot[V], sbase[V];   // class sizes and stage offsets inside the tile
#pragma unroll
    for (int k = 0; k < V; ++k) {
        tot[k] = T::field(ptot, k);
        sbase[k] = k == 0 ? 0u : sbase[k - 1] + tot[k - 1];
    }

    Idx *out_idx = static_cast<Idx *>(a.out_idx);
    const Picker<V, int64_t> dst_of(dst);
    const Picker<V, uint32_t> sbase_of(sbase);
#pragma unroll
    for (int r = 0; r < kVRows; ++r) {
        const int64_t p0 = T::pos(lo, wave, r, lane);
        Idx v[4];
        uint32_t vm = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t c = tile.cls(r, q);
            const bool ok = tile.valid(r, q);
            vm |= static_cast<uint32_t>(ok) << q;
            v[q] = static_cast<Idx>(dst_of(c) + tile.rank[r][q]);
            if (a.out_keys && ok) stage[sbase_of(c) + tile.rank[r][q]] = tile.key[r][q];
        }
        if (out_idx && vm) store_idx_group<4, Idx>(out_idx, p0, v, vm);
    }
    if (a.out_keys) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < V; ++k) write_run<kVBlockThreads>(stage, sbase[k], tot[k], dst[k], a.out_keys, a.n, tid);
    }
}

template <int V, class Cls, bool NT>
int launch_passes(VArgs a, const Cls &cl, int idx_t, hipStream_t st) {
    constexpr int64_t kTile = kVBlockThreads * kVRows * 4;
    a.num_tiles = ceil_div(a.n, kTile);
    const int64_t nt = a.num_tiles;
    int64_t nw = 0;
    if (nt > 0) {
        a.tiles_per_wave = ceil_div(nt, kVCountWaves);
        nw = ceil_div(nt, a.tiles_per_wave);
        if (a.tiles_per_wave == 1)
            IXP_LAUNCH("flatv_count", (flatv_count_small_kernel<V, Cls, NT>), dim3(static_cast<uint32_t>(nt)),
                       dim3(256), 0, st, a, cl);
        else
            IXP_LAUNCH("flatv_count", (flatv_count_kernel<V, Cls, NT>), dim3(static_cast<uint32_t>(ceil_div(nw, 4))),
                       dim3(256), 0, st, a, cl);
    }
    IXP_LAUNCH("flatv_scan", flatv_scan_kernel<V>, dim3(1), dim3(1024), 0, st, a.wsum, nw, a.n, a.counts);
    if (nt == 0) return launch_status();
    const dim3 grid(static_cast<uint32_t>(nt));
    if (idx_t == IXP_I32)
        IXP_LAUNCH("flatv_scatter", (flatv_scatter_kernel<V, Cls, int32_t, NT>), grid, dim3(kVBlockThreads), 0, st, a,
                   cl);
    else
        IXP_LAUNCH("flatv_scatter", (flatv_scatter_kernel<V, Cls, int64_t, NT>), grid, dim3(kVBlockThreads), 0, st, a,
                   cl);
    return launch_status();
}

// Plain loads in both passes where the Infinity Cache (256 MB) still holds part
// of the keys when the scatter comes.  Nontemporal / plain, 3 classes by
// threshold, 32-bit indices: 8 10^6 30.7 / 28.9 us, 2 10^7 64.3 / 62.2, 5 10^7 149 / 130,
// 8 10^7 229 / 223, 10^8 286 / 306; by modulus, 64-bit indices: 5 10^7 276 / 258, 8 10^7
// 439 / 421, 10^8 547 / 557.
template <int V, class Cls>
int launch_v(const VArgs &a, const Cls &cl, int idx_t, hipStream_t st) {
    const bool keep = a.n >= (int64_t{1} << 22) && a.n <= int64_t{5} << 24;
    return keep ? launch_passes<V, Cls, false>(a, cl, idx_t, st) : launch_passes<V, Cls, true>(a, cl, idx_t, st);
}

template <int V>
int dispatch_v(const VArgs &a, const ixp_classes &c, int idx_t, hipStream_t st) {
    switch (c.kind) {
    case IXP_CLASS_MOD: {
        return launch_v<V>(a, ClassMod<V>{}, idx_t, st);
    }
    case IXP_CLASS_THRESH: {
        ClassThresh<V> cl{c.s[0], c.s[1], c.s[2]};
        return launch_v<V>(a, cl, idx_t, st);
    }
    default: {
        ClassBytes<V> cl{c.classes};
        return launch_v<V>(a, cl, idx_t, st);
    }
    }
}

}  // namespace
}  // namespace ixp

using namespace ixp;

extern "C" size_t ixp_partition_v_workspace(int64_t n) {
    if (n < 0) return 0;
    const int64_t nt = ceil_div(n, static_cast<int64_t>(kVBlockThreads) * kVRows * 4);
    return kVHeader + 3 * kVCountWaves * sizeof(int64_t) + static_cast<size_t>(nt) * 4 * sizeof(uint64_t);
}

extern "C" int ixp_partition_v(const void *keys, int32_t key_t, int64_t n, const ixp_classes *cls,
                               void *out_keys, void *out_idx, int32_t idx_t, int64_t *d_counts, void *ws,
                               size_t ws_bytes, void *stream) {
    if (n < 0 || !cls || !d_counts) return IXP_EINVAL;
    const int v = cls->v;
    if (v < 2 || v > 4) return IXP_EINVAL;
    if (idx_t != IXP_I32 && idx_t != IXP_I64) return IXP_EINVAL;
    if (idx_t == IXP_I32 && n > 0x7FFFFFFFll) return IXP_EINVAL;
    switch (cls->kind) {
    case IXP_CLASS_MOD:
        if (key_t != IXP_I32) return IXP_EINVAL;
        break;
    case IXP_CLASS_THRESH:
        if (key_t != IXP_F32) return IXP_EINVAL;
        for (int h = 1; h < v - 1; ++h)
            if (!(cls->s[h - 1] <= cls->s[h])) return IXP_EINVAL;
        break;
    case IXP_CLASS_BYTES:
        if (key_t != IXP_I32 && key_t != IXP_F32) return IXP_EINVAL;
        if (n > 0 && !cls->classes) return IXP_EINVAL;
        break;
    default:
        return IXP_EINVAL;
    }
    const bool need_keys = cls->kind != IXP_CLASS_BYTES || out_keys != nullptr;
    if (n > 0 && need_keys && !keys) return IXP_EINVAL;
    if (!ws || ws_bytes < ixp_partition_v_workspace(n)) return IXP_EWORKSPACE;
    const size_t isz = idx_t == IXP_I32 ? 4 : 8;
    if (!aligned(keys, 16) || !aligned(out_keys, 4) || !aligned(out_idx, 4 * isz) || !aligned(d_counts, 8) ||
        !aligned(ws, 8) || !aligned(cls->classes, 4))
        return IXP_EINVAL;
    char *w = static_cast<char *>(ws);
    VArgs a;
    a.keys = static_cast<const uint32_t *>(keys);
    a.n = n;
    a.out_keys = static_cast<uint32_t *>(out_keys);
    a.out_idx = out_idx;
    a.counts = d_counts;
    a.wsum = reinterpret_cast<int64_t *>(w + kVHeader);
    a.desc = reinterpret_cast<uint64_t *>(w + kVHeader + 3 * kVCountWaves * sizeof(int64_t));
    a.num_tiles = 0;
    a.tiles_per_wave = 1;
    a.need_keys = need_keys ? 1 : 0;
    hipStream_t st = as_stream(stream);
    switch (v) {
    case 2: return dispatch_v<2>(a, *cls, idx_t, st);
    case 3: return dispatch_v<3>(a, *cls, idx_t, st);
    default: return dispatch_v<4>(a, *cls, idx_t, st);
    }
}
