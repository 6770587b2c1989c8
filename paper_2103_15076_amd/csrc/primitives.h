// primitives.h -- wave64 device primitives for gfx950: block scans, a stable
// LSD radix sort (upsweep / row scan / downsweep per digit pass) and a
// flag-compaction "scan" built from two kernels.  No kernel here waits on
// another workgroup: all cross-workgroup ordering is by kernel boundaries.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include <stdint.h>

namespace prim {

typedef unsigned long long u64;
typedef uint32_t u32;

constexpr int BLOCK = 256;  // 4 wavefronts of 64 lanes
constexpr int WAVES = BLOCK / 64;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }
__device__ __forceinline__ int wave_id() { return (int)(threadIdx.x >> 6); }
__device__ __forceinline__ u64 lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// (the builtin: HIP's __ballot takes an int, which costs two vector instructions more)
__device__ __forceinline__ u64 ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// lanes of the mask below this one
__device__ __forceinline__ u32 mask_below(u64 m) {
    return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
}

// Inclusive prefix sums over the lanes of a wave, all of which must be active: rows of 16 by shifts, then each row's last lane into the
// rows behind it (six additions with the lane moves in them, where shuffles take about 40 instructions and six trips to LDS).
__device__ __forceinline__ u32 wave_inclusive_scan(u32 v) {
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// The lanes with `ok` of a wave that hold the same digit `d`, worked out
// for the first WAVE_DIGIT_PEEL distinct digits among the wave's lanes; a lane whose digit comes after
// those is left alone.  Keys in mesh order mostly bring one to
// three distinct leading digits into a wave, so one LDS atomic per digit (by the lane with below = 0,
// adding the count) replaces up to 64 atomics on the same address.  By all lanes.
constexpr int WAVE_DIGIT_PEEL = 4;
struct SameDigit {
    u32 below, count;  // lanes with the digit in front of this one, and all of them
    int lead;          // the first of them
};
__device__ __forceinline__ SameDigit wave_same_digit(bool ok, u32 d) {
    SameDigit r{0u, 1u, lane_id()};
    u64 rem = ballot(ok);
#pragma unroll
    for (int j = 0; j < WAVE_DIGIT_PEEL; ++j) {
        if (rem == 0) break;
        const int lead = (int)__builtin_ctzll(rem);
        const bool in = ok && d == (u32)__builtin_amdgcn_readlane((int)d, lead);
        const u64 m = ballot(in);
        if (in) {
            r.below = mask_below(m);
            r.count = (u32)__popcll(m);
            r.lead = lead;
        }
        rem &= ~m;
    }
    return r;
}

// Workgroups are dealt out to the 8 XCDs in turn; so that neighbouring tiles of a list share an XCD's L2 (they refer to
// the same vertices), an XCD takes one eighth of the n items' tiles in a row.  The tile of this workgroup; a workgroup too many gets the
// number of tiles.  The grid: xcd_grid of the tiles at most.
__device__ __forceinline__ int xcd_item(int block, int tiles) {
    const int per = (tiles + 7) >> 3, j = block >> 3;
    return j < per ? min((block & 7) * per + j, tiles) : tiles;
}
__device__ __forceinline__ int xcd_tile(long long n, int tile_items) {
    return xcd_item((int)blockIdx.x, (int)((n + tile_items - 1) / tile_items));
}
inline int xcd_grid(int tiles) { return (tiles + 7) / 8 * 8; }

// Reads a count that lives either on the device (n_ptr) or in the launch arguments.
__device__ __forceinline__ int load_count(const int* n_ptr, int n_host) { return n_ptr ? *n_ptr : n_host; }

// Exclusive prefix sum of one value per thread over a 256-thread block.
// `total` receives the block sum.  smem must hold WAVES words.  Contains barriers.
__device__ __forceinline__ u32 block_exclusive_scan(u32 v, u32* smem, u32& total) {
    const int lane = lane_id(), w = wave_id();
    const u32 incl = wave_inclusive_scan(v);
    __syncthreads();  // smem may still be in use by a previous call
    if (lane == 63) smem[w] = incl;
    __syncthreads();
    u32 woff = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        u32 s = smem[i];
        if (i < w) woff += s;
        tot += s;
    }
    total = tot;
    return woff + incl - v;
}

__device__ __forceinline__ u32 block_sum(u32 v, u32* smem) {
    const int lane = lane_id(), w = wave_id();
    v = wave_inclusive_scan(v);
    __syncthreads();
    if (lane == 63) smem[w] = v;
    __syncthreads();
    u32 tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) tot += smem[i];
    return tot;
}

// ---------------------------------------------------------------------------
// Radix sort.  Tile = 4096 keys per workgroup.  Within a tile the order of the
// keys is (wave, item, lane), which equals their index order, so ranking by
// (digit, that order) keeps the sort stable.
// ---------------------------------------------------------------------------
// Keys per lane: 16 for large inputs, 4 when the input is small enough that
// 4096-key tiles would leave most compute units without a workgroup.
constexpr int SORT_ITEMS_BIG = 16;
constexpr int SORT_ITEMS_SMALL = 4;
constexpr int SORT_SMALL_MAX_TILES = 2048;

template <typename K>
__device__ __forceinline__ u32 digit_of(K k, int shift, u32 mask) {
    return (u32)(k >> shift) & mask;
}

// Stable ranks of a wave's keys among the wave's keys with the same digit.  digit[i] is the
// digit of the lane's i-th key (keys are ordered by (item, lane)); wrow[d] accumulates this
// wave's count of digit d and must be zero on entry.  On return rank[i] = number of the wave's
// earlier keys with the same digit.  Lanes that hold one digit are found with ballots; the first
// of them adds their number to wrow[d] with one LDS atomic, whose return value (the count left by
// the earlier items: LDS operations of a wave complete in order) it then hands to the others.
// Four items go through together so that four atomics are in flight instead of one.
constexpr int WAVE_RANK_MAX_BITS = 9;  // widest digit wave_rank_digits takes

template <int ITEMS>
__device__ __forceinline__ void wave_rank_digits(const u32 (&digit)[ITEMS], int items, int bits, u32* wrow,
                                                 u32 (&rank)[ITEMS]) {
    constexpr int GROUP = ITEMS < 4 ? ITEMS : 4;
    const u64 lt = lanemask_lt();
#pragma unroll
    for (int i0 = 0; i0 < ITEMS; i0 += GROUP) {
        if (i0 >= items) break;
        u32 below[GROUP], old[GROUP];
        int leader[GROUP];
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            old[j] = 0;
            if (i0 + j < items) {
                const u32 d = digit[i0 + j];
                // lanes whose digit differs from this lane's in some bit: per bit, the ballot of the
                // bit XOR this lane's own bit spread over a word (unrolled; `bits` is wave-uniform)
                u32 dlo = 0, dhi = 0;
#pragma unroll
                for (int b = 0; b < WAVE_RANK_MAX_BITS; ++b) {
                    if (b < bits) {
                        const int own = (int)(d << (31 - b)) >> 31;  // 0 or -1
                        const u64 bal = ballot(own != 0);
                        dlo |= (u32)bal ^ (u32)own;
                        dhi |= (u32)(bal >> 32) ^ (u32)own;
                    }
                }
                const u64 m = ~(((u64)dhi << 32) | dlo);  // lanes of this wave holding the same digit
                below[j] = (u32)__popcll(m & lt);
                leader[j] = __ffsll((long long)m) - 1;
                if (below[j] == 0) old[j] = atomicAdd(&wrow[d], (u32)__popcll(m));
            }
        }
#pragma unroll
        for (int j = 0; j < GROUP; ++j)
            if (i0 + j < items) rank[i0 + j] = (u32)__shfl((int)old[j], leader[j], 64) + below[j];
    }
}

// table[d * T + tile] = number of keys of this tile whose digit is d
template <typename K, int SORT_ITEMS>
__global__ __launch_bounds__(BLOCK) void radix_upsweep_kernel(const K* __restrict__ kin, const int* n_ptr, int n_host,
                                                              int T, u32* __restrict__ table, int shift, int bits) {
    constexpr int SORT_TILE = BLOCK * SORT_ITEMS;
    __shared__ u32 hist[WAVES][256];
    const int n = load_count(n_ptr, n_host);
    const int tile = blockIdx.x;
    const long long base = (long long)tile * SORT_TILE;
    if (base >= n) return;
    const int t = threadIdx.x, w = wave_id();
    const u32 R = 1u << bits, dmask = R - 1;
    for (int i = t; i < WAVES * 256; i += BLOCK) (&hist[0][0])[i] = 0;
    __syncthreads();
    // a digit narrower than 8 bits leaves room for 256/R copies of the histogram per wave:
    // lanes spread over the copies, so fewer of them meet on one LDS word
    const u32 copy = ((u32)lane_id() & ((256u >> bits) - 1u)) << bits;
#pragma unroll 4
    for (int i = 0; i < SORT_ITEMS; ++i) {
        long long idx = base + (long long)i * BLOCK + t;
        if (idx < n) atomicAdd(&hist[w][copy | digit_of<K>(kin[idx], shift, dmask)], 1u);
    }
    __syncthreads();
    if ((u32)t < R) {
        u32 sum = 0;
        for (u32 c = (u32)t; c < 256u; c += R) sum += hist[0][c] + hist[1][c] + hist[2][c] + hist[3][c];
        table[(size_t)t * T + tile] = sum;
    }
}

// One workgroup per digit: exclusive scan of its table row over the tiles in
// use; totals[d] = number of keys with digit d.
__global__ __launch_bounds__(BLOCK) void radix_scan_kernel(u32* __restrict__ table, u32* __restrict__ totals,
                                                           const int* n_ptr, int n_host, int T, int tile_keys) {
    __shared__ u32 smem[WAVES];
    const int n = load_count(n_ptr, n_host);
    const int tiles = (int)(((long long)n + tile_keys - 1) / tile_keys);
    u32* row = table + (size_t)blockIdx.x * T;
    const int t = threadIdx.x;
    u32 carry = 0;
    for (int c = 0; c < tiles; c += BLOCK) {
        const int i = c + t;
        u32 v = (i < tiles) ? row[i] : 0u;
        u32 tot;
        u32 ex = block_exclusive_scan(v, smem, tot);
        if (i < tiles) row[i] = carry + ex;
        carry += tot;
    }
    if (t == 0) totals[blockIdx.x] = carry;
}

template <typename K, bool HAS_VAL, int SORT_ITEMS>
__global__ __launch_bounds__(BLOCK) void radix_downsweep_kernel(const K* __restrict__ kin, K* __restrict__ kout,
                                                                const u32* __restrict__ vin, u32* __restrict__ vout,
                                                                const int* n_ptr, int n_host, int T,
                                                                const u32* __restrict__ table,
                                                                const u32* __restrict__ totals, int shift, int bits) {
    constexpr int SORT_TILE = BLOCK * SORT_ITEMS;
    __shared__ u32 wcnt[WAVES][256];
    __shared__ u32 tstart[256];
    __shared__ u32 gbase[256];
    __shared__ u32 smem[WAVES];
    __shared__ K skey[SORT_TILE];
    __shared__ u32 sval[HAS_VAL ? SORT_TILE : 1];

    const int n = load_count(n_ptr, n_host);
    const int tile = blockIdx.x;
    const long long base = (long long)tile * SORT_TILE;
    if (base >= n) return;
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();
    const u32 R = 1u << bits, dmask = R - 1;

    for (int i = t; i < WAVES * 256; i += BLOCK) (&wcnt[0][0])[i] = 0;

    K key[SORT_ITEMS];
    u32 val[SORT_ITEMS];
    u32 rank[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        long long idx = base + (long long)w * (64 * SORT_ITEMS) + i * 64 + lane;
        bool ok = idx < n;
        key[i] = ok ? kin[idx] : (K) ~(K)0;  // padding sorts last within the tile
        if (HAS_VAL) val[i] = ok ? vin[idx] : 0u;
    }
    __syncthreads();

    {
        u32 digit[SORT_ITEMS];
#pragma unroll
        for (int i = 0; i < SORT_ITEMS; ++i) digit[i] = digit_of<K>(key[i], shift, dmask);
        wave_rank_digits<SORT_ITEMS>(digit, SORT_ITEMS, bits, wcnt[w], rank);
    }
    __syncthreads();

    // per digit: wave counts -> exclusive offsets over waves, tile histogram
    u32 tot = 0;
    if ((u32)t < R) {
        u32 c0 = wcnt[0][t], c1 = wcnt[1][t], c2 = wcnt[2][t], c3 = wcnt[3][t];
        wcnt[0][t] = 0;
        wcnt[1][t] = c0;
        wcnt[2][t] = c0 + c1;
        wcnt[3][t] = c0 + c1 + c2;
        tot = c0 + c1 + c2 + c3;
    }
    u32 dummy;
    const u32 ex = block_exclusive_scan(tot, smem, dummy);
    const u32 gtot = ((u32)t < R) ? totals[t] : 0u;
    const u32 dbase = block_exclusive_scan(gtot, smem, dummy);
    if ((u32)t < R) {
        tstart[t] = ex;
        gbase[t] = dbase + table[(size_t)t * T + tile] - ex;
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const u32 d = digit_of<K>(key[i], shift, dmask);
        const u32 p = tstart[d] + wcnt[w][d] + rank[i];
        skey[p] = key[i];
        if (HAS_VAL) sval[p] = val[i];
    }
    __syncthreads();

    const long long rem = (long long)n - base;
    const int nvalid = rem < SORT_TILE ? (int)rem : SORT_TILE;
    for (int q = t; q < nvalid; q += BLOCK) {
        const K k = skey[q];
        const u32 o = gbase[digit_of<K>(k, shift, dmask)] + (u32)q;
        kout[o] = k;
        if (HAS_VAL) vout[o] = sval[q];
    }
}

struct SortScratch {
    u32* table;   // [256 * T]
    u32* totals;  // [256]
    int T;        // row stride = tiles at capacity
};

// Optional hipEvent bracket around the launch of key_sort's main streaming
// kernel (the per-bucket sort), for
// the roofline measurement of the benchmark; `tag` travels to the record.
struct LaunchTimer {
    hipEvent_t* pool = nullptr;
    int cap = 0, used = 0;
    struct Rec { int e0, e1, tag; };
    Rec* recs = nullptr;
    int nrec = 0;
    bool begin(hipStream_t s, int tag) {
        if (!pool || used + 2 > cap) return false;
        recs[nrec] = Rec{used, used + 1, tag};
        (void)hipEventRecord(pool[used], s);
        used += 2;
        return true;
    }
    void end(hipStream_t s) {
        (void)hipEventRecord(pool[recs[nrec].e1], s);
        ++nrec;
    }
};

inline int sort_items_for(long long n_max) {
    return (n_max + BLOCK * SORT_ITEMS_SMALL - 1) / (BLOCK * SORT_ITEMS_SMALL) <= SORT_SMALL_MAX_TILES ? SORT_ITEMS_SMALL
                                                                                                      : SORT_ITEMS_BIG;
}
inline int sort_tiles(long long n, int items) { return (int)((n + (long long)BLOCK * items - 1) / ((long long)BLOCK * items)); }
// row stride of the tile table for inputs of up to n_cap keys
inline int sort_table_stride(long long n_cap) {
    const int big = sort_tiles(n_cap, SORT_ITEMS_BIG);
    return big > SORT_SMALL_MAX_TILES ? big : SORT_SMALL_MAX_TILES;
}

template <typename K, bool HAS_VAL, int ITEMS>
inline int radix_sort_impl(hipStream_t s, K* k0, K* k1, u32* v0, u32* v1, const int* n_ptr, int n_max, int key_bits,
                           const SortScratch& sc) {
    const int passes = (key_bits + 7) / 8;
    const int per = (key_bits + passes - 1) / passes;
    const int tiles = sort_tiles(n_max, ITEMS);
    int cur = 0, shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int bits = (key_bits - shift) < per ? (key_bits - shift) : per;
        K* kin = cur ? k1 : k0;
        K* kout = cur ? k0 : k1;
        u32* vin = cur ? v1 : v0;
        u32* vout = cur ? v0 : v1;
        radix_upsweep_kernel<K, ITEMS><<<tiles, BLOCK, 0, s>>>(kin, n_ptr, n_max, sc.T, sc.table, shift, bits);
        radix_scan_kernel<<<1 << bits, BLOCK, 0, s>>>(sc.table, sc.totals, n_ptr, n_max, sc.T, BLOCK * ITEMS);
        radix_downsweep_kernel<K, HAS_VAL, ITEMS>
            <<<tiles, BLOCK, 0, s>>>(kin, kout, vin, vout, n_ptr, n_max, sc.T, sc.table, sc.totals, shift, bits);
        shift += bits;
        cur ^= 1;
    }
    if (hipGetLastError() != hipSuccess) return -1;
    return cur;
}

// Sorts on key bits [0, key_bits).  Data ping-pongs between (k0,v0) and
// (k1,v1); returns 0 if the result is in (k0,v0), 1 if in (k1,v1), <0 on a
// launch error.  n_max bounds the device-side count for the grid size.
template <typename K, bool HAS_VAL>
inline int radix_sort(hipStream_t s, K* k0, K* k1, u32* v0, u32* v1, const int* n_ptr, int n_max, int key_bits,
                      const SortScratch& sc) {
    if (n_max <= 0 || key_bits <= 0) return 0;
    if (sort_items_for(n_max) == SORT_ITEMS_SMALL)
        return radix_sort_impl<K, HAS_VAL, SORT_ITEMS_SMALL>(s, k0, k1, v0, v1, n_ptr, n_max, key_bits, sc);
    return radix_sort_impl<K, HAS_VAL, SORT_ITEMS_BIG>(s, k0, k1, v0, v1, n_ptr, n_max, key_bits, sc);
}

// ---------------------------------------------------------------------------
// Bucket sort for inputs of up to BUCKET_SORT_MAX_KEYS keys whose leading bits
// are spread evenly (vertex ids): one stable radix pass on the TOP 8 bits
// splits the keys into 256 buckets, then each bucket is sorted on the
// remaining bits by one workgroup entirely in LDS (register-staged LSD passes
// over a single LDS array).  Two sweeps over memory instead of one per 8 bits,
// and 4 launches instead of 3 per 8 bits.  A bucket that does not fit in LDS
// (a very uneven key distribution) is sorted by the same workgroup with a slow
// pass-by-pass LSD over global memory, so the result is always correct.
// ---------------------------------------------------------------------------
constexpr int BUCKET_THREADS_256 = 1024;  // 256 buckets: 8 keys per lane, up to 8192 keys of a bucket held in LDS
constexpr int BUCKET_THREADS_4096 = 512;  // 4096 buckets: up to 4096 keys (8 per lane), or 8192 key-value
                                          // pairs (16 per lane: vertex incidences run to ~6 per vertex and
                                          // vertex ids need not fill their bit range, so those buckets run fuller)
// keys without values (bucket_keys_kernel): lanes and keys per lane of a bucket's workgroup
constexpr int BUCKET_KEYS_THREADS = 256, BUCKET_KEYS_ITEMS = 16;  // up to 4096 keys in LDS
// Half as many lanes (and keys in LDS) where vertices or the like are made from the groups of buckets that hold this many keys or less on average: then
// a lane has a group, and more buckets fit a compute unit (10.2 M vertices, 128 and 765 keys to a bucket: 421 -> 354 us).  Not where most rows have no item
// (KeySort::crowded): then a few buckets hold nearly all keys, many times the average, and one workgroup sorts each through memory (3.6 k vertices
// with facets and 300 k without: 549 us by 128 lanes, 264 by 256; lists of their corners, whole calls, 450 and 234).
constexpr int BUCKET_FEW_KEYS = 1024;
constexpr int BUCKET_MSD_BITS = 8, NARROW_BITS_MAX = 10;  // (bits of a narrow digit: 8 to 10)
constexpr long long BUCKET_SORT_MAX_KEYS = 1ll << 20;  // average bucket <= half of what LDS holds

template <int NW>
__device__ __forceinline__ u32 wide_block_exclusive_scan(u32 v, u32* smem, u32& total) {
    const int lane = lane_id(), w = wave_id();
    const u32 incl = wave_inclusive_scan(v);
    __syncthreads();
    if (lane == 63) smem[w] = incl;
    __syncthreads();
    u32 woff = 0, tot = 0;
    for (int i = 0; i < NW; ++i) {
        u32 x = smem[i];
        if (i < w) woff += x;
        tot += x;
    }
    total = tot;
    return woff + incl - v;
}

template <typename K>
__device__ __forceinline__ K coherent_load(const K* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Slow path for a bucket larger than BUCKET_CAP: stable LSD over global memory
// by this workgroup alone; wave 0 places the keys 64 at a time in order.
template <typename K, bool HAS_VAL, int BUCKET_THREADS>
__device__ void bucket_sort_oversize(K* a, K* b, u32* va, u32* vb, int cnt, int low_bits, u32* hist /*[256]*/,
                                     u32* smem) {
    constexpr int BUCKET_WAVES = BUCKET_THREADS / 64, PER = BUCKET_THREADS < 256 ? 256 / BUCKET_THREADS : 1;  // counters of a thread
    // data starts in b (the partition pass wrote it there) and must end in a
    K* src = b;
    K* dst = a;
    u32* vsrc = vb;
    u32* vdst = va;
    const int passes = (low_bits + 7) / 8;
    const int per = (low_bits + passes - 1) / passes;
    const int t = threadIdx.x, lane = lane_id();
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int bits = (low_bits - shift) < per ? (low_bits - shift) : per;
        const u32 R = 1u << bits, dmask = R - 1;
        for (int i = t; i < 256; i += BUCKET_THREADS) hist[i] = 0;
        __syncthreads();
        for (int i = t; i < cnt; i += BUCKET_THREADS) atomicAdd(&hist[digit_of<K>(coherent_load(&src[i]), shift, dmask)], 1u);
        __syncthreads();
        u32 tot, c[PER], sum = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const u32 d = (u32)(t * PER + j);
            c[j] = d < R ? hist[d] : 0u;
            sum += c[j];
        }
        u32 ex = wide_block_exclusive_scan<BUCKET_WAVES>(sum, smem, tot);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {  // running output position of each digit
            if (t * PER + j < 256) hist[t * PER + j] = ex;
            ex += c[j];
        }
        __syncthreads();
        if (t < 64) {
            for (int base = 0; base < cnt; base += 64) {
                const int i = base + lane;
                const bool ok = i < cnt;
                const K k = ok ? coherent_load(&src[i]) : (K)0;
                const u32 d = ok ? digit_of<K>(k, shift, dmask) : 0xFFFFFFFFu;
                u64 m = ballot(ok);
                for (int bb = 0; bb < bits; ++bb) {
                    const bool bit = (d >> bb) & 1u;
                    const u64 bal = ballot(bit);
                    m &= bit ? bal : ~bal;
                }
                if (ok) {
                    const u32 below = (u32)__popcll(m & lanemask_lt());
                    const u32 old = hist[d];
                    __builtin_amdgcn_wave_barrier();
                    if (below == 0) hist[d] = old + (u32)__popcll(m);
                    __builtin_amdgcn_wave_barrier();
                    dst[old + below] = k;
                    if (HAS_VAL) vdst[old + below] = coherent_load(&vsrc[i]);
                }
            }
        }
        __threadfence();
        __syncthreads();
        K* tk = src; src = dst; dst = tk;
        u32* tv = vsrc; vsrc = vdst; vdst = tv;
        shift += bits;
    }
    if (src != a) {  // an even number of passes left the result in b
        for (int i = t; i < cnt; i += BUCKET_THREADS) {
            a[i] = coherent_load(&src[i]);
            if (HAS_VAL) va[i] = coherent_load(&vsrc[i]);
        }
    }
}

// One workgroup per bucket.  kin/vin hold the keys partitioned by their top
// digit (bucket d occupies [start_d, start_d + totals[d])); the sorted bucket is
// written to the same range of kout/vout.  low_bits = key bits below the digit.
//
// The bucket is held in LDS.  One stable radix pass on the TOP (up to) 9 of the
// low bits splits it into up to 512 groups of keys that agree on all bits
// sorted so far; with vertex-pair keys a group is the handful of half-edges of
// one lower vertex.  Each group is then finished by one lane with a stable
// sort on the whole key (by counting ranks in registers for up to 16 keys,
// by insertion in place beyond), which for such groups costs far less than
// the two or three more radix passes over every key that the remaining bits
// would take (a radix pass spends one wave-wide ballot per key and bit).  If
// some group is long (keys crowded on few values of those 9 bits), the
// workgroup runs plain LSD radix passes over all the low bits instead.
constexpr int BUCKET_GROUP_BITS = 9;
constexpr int BUCKET_GROUP_MAX = 64;  // longest group the insertion sort is allowed

// Stable sort of the g <= G keys at [gs, gs + g) of an LDS array by one lane: the keys are read into
// registers together, each key's place is the number of keys that must precede it (G x G
// comparisons, none of which waits for memory), and the keys are written back to their places.
template <typename K, bool HAS_VAL, int G>
__device__ __forceinline__ void group_rank_sort(K* skey, u32* sval, int gs, int g) {
    K k[G];
    u32 v[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        k[j] = j < g ? skey[gs + j] : (K)0;
        v[j] = (HAS_VAL && j < g) ? sval[gs + j] : 0u;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (i < g) {
            int r = 0;
#pragma unroll
            for (int j = 0; j < G; ++j) r += (j < g && (k[j] < k[i] || (k[j] == k[i] && j < i))) ? 1 : 0;
            skey[gs + r] = k[i];
            if (HAS_VAL) sval[gs + r] = v[i];
        }
    }
}

// The same for keys without values (so that equal keys need no order among themselves): a bitonic
// sorting network over G registers, G a power of two, empty places filled with the largest key.
template <typename K, int G>
__device__ __forceinline__ void group_network_sort(K* skey, int gs, int g) {
    K k[G];
#pragma unroll
    for (int j = 0; j < G; ++j) k[j] = j < g ? skey[gs + j] : (K) ~(K)0;
#pragma unroll
    for (int size = 2; size <= G; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int l = i ^ stride;
                if (l > i) {
                    const bool up = (i & size) == 0;
                    const K a = k[i], b = k[l];
                    const bool swap = up ? (a > b) : (a < b);
                    k[i] = swap ? b : a;
                    k[l] = swap ? a : b;
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < G; ++j)
        if (j < g) skey[gs + j] = k[j];
}

// LK = type of the keys while they are in LDS and registers.  All keys of a bucket agree above
// their low_bits bits, so 64-bit keys with low_bits <= 32 are kept as their low 32 bits (LK = u32:
// half the LDS, registers and comparison work) and get their common upper part back, bucket <<
// low_bits, on the way out.
template <typename K, bool HAS_VAL, int BUCKET_THREADS, int BUCKET_ITEMS, typename LK = K>
__device__ __forceinline__ void bucket_sort_one(const int bkt, K* __restrict__ kin, K* __restrict__ kout,
                                                u32* __restrict__ vin, u32* __restrict__ vout,
                                                const u32* __restrict__ totals, const u32* __restrict__ starts,
                                                int low_bits) {
    constexpr int BUCKET_WAVES = BUCKET_THREADS / 64;
    constexpr int BUCKET_CAP = BUCKET_THREADS * BUCKET_ITEMS;  // keys of one bucket held in LDS
    constexpr int RMAX = 1 << BUCKET_GROUP_BITS;
    static_assert(RMAX <= BUCKET_THREADS, "one thread per digit in the scans below");
    __shared__ LK skey[BUCKET_CAP];
    __shared__ u32 sval[HAS_VAL ? BUCKET_CAP : 1];
    __shared__ u32 wcnt[BUCKET_WAVES][RMAX];
    __shared__ u32 tstart[RMAX];
    __shared__ u32 smem[BUCKET_WAVES];
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();

    // start of this bucket = sum of the counts of the buckets before it (given, or summed here)
    const int cnt = (int)totals[bkt];
    if (cnt == 0) return;
    u32 start;
    if (starts) {  // (the partition kernel has left them)
        start = starts[bkt];
    } else {
        u32 part = 0;
        for (int j = t; j < bkt; j += BUCKET_THREADS) part += totals[j];
        (void)wide_block_exclusive_scan<BUCKET_WAVES>(part, smem, start);
        __syncthreads();
    }
    if (cnt > BUCKET_CAP) {
        bucket_sort_oversize<K, HAS_VAL, BUCKET_THREADS>(kout + start, kin + start, HAS_VAL ? vout + start : nullptr,
                                         HAS_VAL ? vin + start : nullptr, cnt, low_bits, tstart, smem);
        return;
    }
    if (low_bits <= 0) {
        for (int i = t; i < cnt; i += BUCKET_THREADS) {
            kout[start + i] = kin[start + i];
            if (HAS_VAL) vout[start + i] = vin[start + i];
        }
        return;
    }
    kin += start;
    kout += start;
    if (HAS_VAL) {
        vin += start;
        vout += start;
    }

    const int items = (cnt + BUCKET_THREADS - 1) / BUCKET_THREADS;  // <= BUCKET_ITEMS, same for the whole workgroup

    // One stable pass on key bits [shift, shift + bits): the keys come from memory (FROM_MEMORY) or
    // from skey, in index order = (wave, item, lane), and land in skey/sval; tstart[d] = first
    // position of digit d afterwards.
    auto radix_pass = [&](auto from_memory, int shift, int bits) {
        constexpr bool FROM_MEMORY = decltype(from_memory)::value;
        const u32 R = 1u << bits, dmask = R - 1;
        for (int i = t; i < BUCKET_WAVES * RMAX; i += BUCKET_THREADS)
            if ((u32)(i & (RMAX - 1)) < R) (&wcnt[0][0])[i] = 0;
        LK key[BUCKET_ITEMS];
        u32 val[BUCKET_ITEMS];
        u32 rank[BUCKET_ITEMS];
        u32 digit[BUCKET_ITEMS];
#pragma unroll
        for (int i = 0; i < BUCKET_ITEMS; ++i) {
            key[i] = (LK) ~(LK)0;  // padding ranks last and is dropped
            val[i] = 0u;
            if (i < items) {
                const int idx = w * (64 * items) + i * 64 + lane;
                if (idx < cnt) {
                    key[i] = FROM_MEMORY ? (LK)kin[idx] : skey[idx];
                    if (HAS_VAL) val[i] = FROM_MEMORY ? vin[idx] : sval[idx];
                }
            }
            digit[i] = digit_of<LK>(key[i], shift, dmask);
        }
        __syncthreads();
        wave_rank_digits<BUCKET_ITEMS>(digit, items, bits, wcnt[w], rank);
        __syncthreads();
        u32 dtot = 0;
        if ((u32)t < R) {
            u32 run = 0;
            for (int ww = 0; ww < BUCKET_WAVES; ++ww) {
                const u32 c = wcnt[ww][t];
                wcnt[ww][t] = run;
                run += c;
            }
            dtot = run;
        }
        u32 dummy;
        const u32 dex = wide_block_exclusive_scan<BUCKET_WAVES>(dtot, smem, dummy);
        if ((u32)t < R) tstart[t] = dex;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < BUCKET_ITEMS; ++i) {
            if (i < items) {
                const u32 pos = tstart[digit[i]] + wcnt[w][digit[i]] + rank[i];
                if (pos < (u32)cnt) {
                    skey[pos] = key[i];
                    if (HAS_VAL) sval[pos] = val[i];
                }
            }
        }
        __syncthreads();
    };

    const int gbits = low_bits < BUCKET_GROUP_BITS ? low_bits : BUCKET_GROUP_BITS;
    const int rest = low_bits - gbits;
    radix_pass(std::true_type{}, rest, gbits);
    if (rest > 0) {
        // groups: positions [tstart[d], tstart[d + 1]) (the last one ends at cnt)
        const int ngroups = 1 << gbits;
        int gs = 0, ge = 0;
        if (t < ngroups) {
            gs = (int)tstart[t];
            ge = t + 1 < ngroups ? (int)tstart[t + 1] : cnt;
            if (ge > cnt) ge = cnt;
        }
        if (!__syncthreads_or(ge - gs > BUCKET_GROUP_MAX)) {
            const int g = ge - gs;
            if (g > 16) {  // one lane, in place: every step waits for LDS, so only for the rare long group
                for (int i = gs + 1; i < ge; ++i) {
                    const LK k = skey[i];
                    const u32 v = HAS_VAL ? sval[i] : 0u;
                    int j = i;
                    while (j > gs && skey[j - 1] > k) {
                        skey[j] = skey[j - 1];
                        if (HAS_VAL) sval[j] = sval[j - 1];
                        --j;
                    }
                    skey[j] = k;
                    if (HAS_VAL) sval[j] = v;
                }
            } else if (g > 8) {
                if constexpr (HAS_VAL) group_rank_sort<LK, true, 16>(skey, sval, gs, g);
                else group_network_sort<LK, 16>(skey, gs, g);
            } else if (g > 4) {
                if constexpr (HAS_VAL) group_rank_sort<LK, true, 8>(skey, sval, gs, g);
                else group_network_sort<LK, 8>(skey, gs, g);
            } else if (g > 1) {
                if constexpr (HAS_VAL) group_rank_sort<LK, true, 4>(skey, sval, gs, g);
                else group_network_sort<LK, 4>(skey, gs, g);
            }
            __syncthreads();
        } else {
            const int passes = (low_bits + 7) / 8;
            const int per = (low_bits + passes - 1) / passes;
            int shift = 0;
            for (int p = 0; p < passes; ++p) {
                const int bits = (low_bits - shift) < per ? (low_bits - shift) : per;
                radix_pass(std::false_type{}, shift, bits);
                shift += bits;
            }
        }
    }
    K upper = 0;
    if constexpr (sizeof(LK) < sizeof(K)) upper = (K)(u32)bkt << low_bits;
    for (int i = t; i < cnt; i += BUCKET_THREADS) {
        kout[i] = upper | (K)skey[i];
        if (HAS_VAL) vout[i] = sval[i];
    }
}

template <typename K, bool HAS_VAL, int BUCKET_THREADS, int BUCKET_ITEMS, typename LK = K>
__global__ __launch_bounds__(BUCKET_THREADS) void bucket_sort_kernel(K* __restrict__ kin, K* __restrict__ kout,
                                                                     u32* __restrict__ vin, u32* __restrict__ vout,
                                                                     const u32* __restrict__ totals, int nbuckets,
                                                                     int low_bits, const u32* __restrict__ starts = nullptr) {
    (void)nbuckets;
    bucket_sort_one<K, HAS_VAL, BUCKET_THREADS, BUCKET_ITEMS, LK>((int)blockIdx.x, kin, kout, vin, vout, totals, starts,
                                                                  low_bits);
}

// A sort of keys WITHOUT values by partition on their top digit and a sort of each bucket (key_sort).
template <typename K>
struct KeySort {
    K* k0 = nullptr;  // receives the sorted keys (PlainKeys), or is scratch for buckets that do not fit LDS
    K* k1 = nullptr;  // receives the partitioned keys
    const int* n_ptr = nullptr;
    int n = 0;        // items of the source (at *n_ptr, where that is given, and n at most)
    int key_bits = 0, digit_bits = 0;
    int buckets = 0;     // digits that occur are below this
    int group_bits = BUCKET_GROUP_BITS;  // bits below the digit that make a group (see sort_bucket)
    bool crowded = false;  // fewer items than rows: some buckets may hold many times the average
    // Behind the partition the keys are 32-bit words (in k1, and in k0 where that is scratch): their low 32 bits, which hold
    // all that a bucket's keys differ in.  Half the bytes of three sweeps.
    bool half = false;
    // One array each of a word per digit.  Which route a sort takes (narrow: msd_scatter_kernel, wide: key_starts_kernel and
    // xl_scatter_kernel) goes by the first sort of a launch, so a sort of few digits can take the wide one beside a sort of many.
    //            in front of the sort                         behind it
    //   hist     keys per digit                               zero (what the next count of digits of up to 12 bits starts from)
    //   taken    zero; narrow: part of each range in use      zero (the digits without keys have not been touched)
    //   cursor   anything; wide: next free position           anything
    //   starts   anything; first position of each range       that
    // taken and cursor are two arrays because key_starts_kernel stores a position for every digit: left where a narrow sort looks for
    // zeros, those of digits that no bucket has would send its keys to other places.
    u32* hist = nullptr;
    u32* taken = nullptr;  // (null where the digits are always wide)
    u32* cursor = nullptr;
    u32* starts = nullptr;
    u32* zero = nullptr;    // n_zero words that the per-bucket kernel adds to: cleared by the kernel in front of it
    int n_zero = 0;
    int* total = nullptr;   // receives the number of keys (those that the source keeps)
    int low_bits() const { return key_bits - digit_bits; }
    bool fits_half() const { return sizeof(K) == 8 && low_bits() <= 32; }
};

// ---------------------------------------------------------------------------
// The per-bucket kernel for keys WITHOUT values (incidence keys, edge keys, lists of items per row).  Equal keys are
// indistinguishable, so nothing has to be stable:
//   1. the keys of the bucket are read once; each takes its place in its group (the keys that agree
//      on the top group_bits, 9 at most, of the bucket's low bits: the half-edges of one lower
//      vertex, the items of one row) from one returning LDS atomic on the group's counter;
//   2. one scan of the (up to 512) group counters gives the groups' first positions;
//   3. one lane per group sorts its group on the whole key in registers with a sorting network of
//      minimal size for 4, 6, 8, 12 or 16 keys (a wave runs every size that occurs among its 64
//      groups, so the sizes are graded finely), by ranks up to 64 keys;
//   4. what the sort is for is made of the sorted keys while they are in LDS (`Out`: distinct keys, sums over rows, lists of
//      rows), so that the sorted keys themselves are written nowhere.
// A bucket with a group of more than 64 keys (a vertex of very high degree) is sorted as a whole by
// a bitonic network over the LDS array.  A bucket beyond the LDS capacity (uneven vertex numbering:
// up to 16 times the capacity) is sorted in parts, runs of whole groups that fit, each read out of the
// bucket by the workgroup and written to k0; if it also has a group of more than 64 keys, or is larger still, it
// takes the slow global-memory route of bucket_sort_oversize.  Out then gets the keys from there.  Workgroups are small (256
// lanes) so that several of them share a compute unit and cover each other's barriers.
// Bound by vector issue (three quarters of its time at 10.2 M vertices), so: lane counts and prefix sums by the instructions that
// make them, no 64-bit arithmetic on 32-bit keys, groups that are the rows (not every other one empty), no workgroups for
// digits that cannot occur.  First round of 10.2 M vertices, 61 M incidence and 61 M edge keys: 611 us for the sorts, 472 for the
// quadrics by a launch that read the sorted keys again, 437 for costs with the search for distinct edges; now 616 and 392.  1.2 M:
// 53 + 65 + 68 -> 63 + 52; 115 k: 12.5 + 10.4 + 14.4 -> 13.3 + 10.4; lists of 5.7 M corners 22.9 + 15.0 -> 19.7.
// ---------------------------------------------------------------------------
#define PRIM_CE(a, b)                       \
    {                                       \
        const K x_ = k[a], y_ = k[b];       \
        const bool s_ = y_ < x_;            \
        k[a] = s_ ? y_ : x_;                \
        k[b] = s_ ? x_ : y_;                \
    }

// Sorting networks of 5, 12, 19, 39 and 60 comparators (the smallest known for these sizes; each was
// checked on all 2^G inputs of zeros and ones).
template <typename K, int G>
__device__ __forceinline__ void network_sort_regs(K (&k)[G]) {
    if constexpr (G == 4) {
        PRIM_CE(0, 2) PRIM_CE(1, 3) PRIM_CE(0, 1) PRIM_CE(2, 3) PRIM_CE(1, 2)
    } else if constexpr (G == 6) {
        PRIM_CE(0, 5) PRIM_CE(1, 3) PRIM_CE(2, 4) PRIM_CE(1, 2) PRIM_CE(3, 4) PRIM_CE(0, 3) PRIM_CE(2, 5) PRIM_CE(0, 1)
        PRIM_CE(2, 3) PRIM_CE(4, 5) PRIM_CE(1, 2) PRIM_CE(3, 4)
    } else if constexpr (G == 8) {
        PRIM_CE(0, 2) PRIM_CE(1, 3) PRIM_CE(4, 6) PRIM_CE(5, 7) PRIM_CE(0, 4) PRIM_CE(1, 5) PRIM_CE(2, 6) PRIM_CE(3, 7)
        PRIM_CE(0, 1) PRIM_CE(2, 3) PRIM_CE(4, 5) PRIM_CE(6, 7) PRIM_CE(2, 4) PRIM_CE(3, 5) PRIM_CE(1, 4) PRIM_CE(3, 6)
        PRIM_CE(1, 2) PRIM_CE(3, 4) PRIM_CE(5, 6)
    } else if constexpr (G == 12) {
        PRIM_CE(0, 8) PRIM_CE(1, 7) PRIM_CE(2, 6) PRIM_CE(3, 11) PRIM_CE(4, 10) PRIM_CE(5, 9) PRIM_CE(0, 1) PRIM_CE(2, 5)
        PRIM_CE(3, 4) PRIM_CE(6, 9) PRIM_CE(7, 8) PRIM_CE(10, 11) PRIM_CE(0, 2) PRIM_CE(1, 6) PRIM_CE(5, 10) PRIM_CE(9, 11)
        PRIM_CE(0, 3) PRIM_CE(1, 2) PRIM_CE(4, 6) PRIM_CE(5, 7) PRIM_CE(8, 11) PRIM_CE(9, 10) PRIM_CE(1, 4) PRIM_CE(3, 5)
        PRIM_CE(6, 8) PRIM_CE(7, 10) PRIM_CE(1, 3) PRIM_CE(2, 5) PRIM_CE(6, 9) PRIM_CE(8, 10) PRIM_CE(2, 3) PRIM_CE(4, 5)
        PRIM_CE(6, 7) PRIM_CE(8, 9) PRIM_CE(4, 6) PRIM_CE(5, 7) PRIM_CE(3, 4) PRIM_CE(5, 6) PRIM_CE(7, 8)
    } else {
        static_assert(G == 16, "network sizes: 4, 6, 8, 12, 16");
        PRIM_CE(0, 13) PRIM_CE(1, 12) PRIM_CE(2, 15) PRIM_CE(3, 14) PRIM_CE(4, 8) PRIM_CE(5, 6) PRIM_CE(7, 11) PRIM_CE(9, 10)
        PRIM_CE(0, 5) PRIM_CE(1, 7) PRIM_CE(2, 9) PRIM_CE(3, 4) PRIM_CE(6, 13) PRIM_CE(8, 14) PRIM_CE(10, 15) PRIM_CE(11, 12)
        PRIM_CE(0, 1) PRIM_CE(2, 3) PRIM_CE(4, 5) PRIM_CE(6, 8) PRIM_CE(7, 9) PRIM_CE(10, 11) PRIM_CE(12, 13) PRIM_CE(14, 15)
        PRIM_CE(0, 2) PRIM_CE(1, 3) PRIM_CE(4, 10) PRIM_CE(5, 11) PRIM_CE(6, 7) PRIM_CE(8, 9) PRIM_CE(12, 14) PRIM_CE(13, 15)
        PRIM_CE(1, 2) PRIM_CE(3, 12) PRIM_CE(4, 6) PRIM_CE(5, 7) PRIM_CE(8, 10) PRIM_CE(9, 11) PRIM_CE(13, 14) PRIM_CE(1, 4)
        PRIM_CE(2, 6) PRIM_CE(5, 8) PRIM_CE(7, 10) PRIM_CE(9, 13) PRIM_CE(11, 14) PRIM_CE(2, 4) PRIM_CE(3, 6) PRIM_CE(9, 12)
        PRIM_CE(11, 13) PRIM_CE(3, 5) PRIM_CE(6, 8) PRIM_CE(7, 9) PRIM_CE(10, 12) PRIM_CE(3, 4) PRIM_CE(5, 6) PRIM_CE(7, 8)
        PRIM_CE(9, 10) PRIM_CE(11, 12) PRIM_CE(6, 7) PRIM_CE(8, 9)
    }
}
#undef PRIM_CE

// The g <= G keys at [gs, gs + g) of an LDS array sorted by one lane (empty places hold the largest key).
template <typename K, int G>
__device__ __forceinline__ void group_sort_lds(K* skey, int gs, int g) {
    K k[G];
#pragma unroll
    for (int j = 0; j < G; ++j) k[j] = j < g ? skey[gs + j] : (K) ~(K)0;
    network_sort_regs<K, G>(k);
#pragma unroll
    for (int j = 0; j < G; ++j)
        if (j < g) skey[gs + j] = k[j];
}


// ... and of g <= 64 keys by a wave, one lane per key: a key's place is the number of keys of the group that go before it (every lane reads the
// same address, one read after the other with nothing waiting in between, where an insertion sort by one lane would wait for
// LDS at every step).
template <typename K>
__device__ __forceinline__ void rank_group_lds(K* key, int g) {
    const int lane = lane_id();
    const K k = lane < g ? key[lane] : (K)0;
    int r = 0;
    for (int i = 0; i < g; ++i) {
        const K o = key[i];
        r += (o < k || (o == k && i < lane)) ? 1 : 0;
    }
    __builtin_amdgcn_wave_barrier();  // (a wave's LDS operations complete in order)
    if (lane < g) key[r] = k;
    __builtin_amdgcn_wave_barrier();
}

template <typename LK, int THREADS, int ITEMS>
struct BucketLds {
    static constexpr int NW = THREADS / 64, CAP = THREADS * ITEMS, RMAX = 1 << BUCKET_GROUP_BITS;
    LK skey[CAP];
    u32 gcnt[RMAX];
    u32 gstart[RMAX + 1];
    u32 smem[NW];
    u32 nlong;
};

// The cnt keys at kin sorted on their low_bits low bits by one workgroup; then emit(key_at), key_at(i) = the i-th of them (from LDS, or,
// where they did not fit, from kout).  For cnt = 0 only emit is called.  Where the keys are in LDS by groups, none of which is longer than
// the lanes and waves sort, groups(R, false) is asked first whether it makes what is wanted from the R groups as they are, not sorted, and groups(R,
// true) when each has been sorted.
template <typename LK, int THREADS, int ITEMS, class Groups, class Emit>
__device__ __forceinline__ void sort_bucket(BucketLds<LK, THREADS, ITEMS>& L, LK* kin, LK* kout, const int cnt,
                                            const int low_bits, const int group_bits, Groups groups, Emit emit) {
    constexpr int NW = THREADS / 64;
    constexpr int CAP = THREADS * ITEMS;
    constexpr int RMAX = 1 << BUCKET_GROUP_BITS;
    constexpr int PER = RMAX / THREADS > 0 ? RMAX / THREADS : 1;  // group counters per thread in the scan
    static_assert((CAP & (CAP - 1)) == 0, "the whole-bucket network pads to a power of two within the LDS array");
    static_assert(THREADS >= 64 && THREADS % 64 == 0 && (THREADS >= RMAX || RMAX % THREADS == 0), "whole counters per thread");
    LK* skey = L.skey;
    u32* gcnt = L.gcnt;
    u32* gstart = L.gstart;
    const int t = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(wave_id());  // (in a scalar register: what follows from it is computed once per wave)
    const int gbits = min(group_bits, max(low_bits, 0));
    const int rest = low_bits > gbits ? low_bits - gbits : 0;
    const u32 R = 1u << gbits, dmask = R - 1;

    // The groups g0 .. g1 - 1, whose keys lie at [gstart[g] - gstart[g0], ...) of the LDS array, each sorted on
    // the whole key: one lane per group of up to 16 keys (a sorting network), then a wave per longer group.
    // By the whole workgroup; no group may exceed 64 keys; uses gcnt (as the list of long groups) and nlong.
    auto sort_groups = [&](int g0, int g1) {
        const int lds0 = (int)gstart[g0];
        if (t == 0) L.nlong = 0;
        __syncthreads();
        for (int gi = g0 + t; gi < g1; gi += THREADS) {
            const int gs = (int)gstart[gi] - lds0;
            const int g = (int)gstart[gi + 1] - (int)gstart[gi];
            if (g > 16) {  // listed for the waves (the counters are no longer needed: the list goes there)
                gcnt[atomicAdd(&L.nlong, 1u)] = (u32)gi;
            } else if (g > 12) {
                group_sort_lds<LK, 16>(skey, gs, g);
            } else if (g > 8) {
                group_sort_lds<LK, 12>(skey, gs, g);
            } else if (g > 6) {
                group_sort_lds<LK, 8>(skey, gs, g);
            } else if (g > 4) {
                group_sort_lds<LK, 6>(skey, gs, g);
            } else if (g > 1) {
                group_sort_lds<LK, 4>(skey, gs, g);
            }
        }
        __syncthreads();
        // groups of 17 to 64 keys: a wave takes a group
        const int n_long = (int)L.nlong;
        if (n_long > 0) {
            for (int li = w; li < n_long; li += NW) {
                const int gi = (int)gcnt[li];
                const int gs = (int)gstart[gi] - lds0;
                const int g = (int)gstart[gi + 1] - (int)gstart[gi];
                rank_group_lds(skey + gs, g);
            }
            __syncthreads();
        }
    };
    // the groups' first positions from their counters; is any group longer than the lanes and waves sort?  By the whole workgroup.
    auto scan_groups = [&]() -> bool {
        u32 c[PER], sum = 0, tot;
        int too_long = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const u32 d = (u32)(t * PER + j);
            c[j] = d < R ? gcnt[d] : 0u;
            sum += c[j];
            too_long |= c[j] > (u32)BUCKET_GROUP_MAX ? 1 : 0;
        }
        u32 run = wide_block_exclusive_scan<NW>(sum, L.smem, tot);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const u32 d = (u32)(t * PER + j);
            if (d < R) gstart[d] = run;
            run += c[j];
        }
        if (t == 0) gstart[R] = (u32)cnt;
        return __syncthreads_or(too_long) != 0;
    };

    if (cnt > CAP) {
        // More keys than the LDS array holds.  If no group is long, the bucket is sorted in parts: runs of
        // whole groups of at most CAP keys each, every part fetched from the bucket (which is read once per
        // part, and once more for the groups' sizes) and sorted like a bucket that fits.
        bool done = false;
        if (rest > 0 && cnt <= 16 * CAP) {
            for (int i = t; i < (int)R; i += THREADS) gcnt[i] = 0;
            __syncthreads();
            // fn(key) for every key of the bucket; a thread's loads go out ITEMS at a time, so that a pass over
            // the bucket waits for memory once per CAP keys and not once per key of the thread
            auto for_each_key = [&](auto fn) {
                for (int base = 0; base < cnt; base += CAP) {
                    LK kreg[ITEMS];
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) {
                        const int idx = base + i * THREADS + t;
                        kreg[i] = idx < cnt ? kin[idx] : (LK)0;
                    }
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i)
                        if (base + i * THREADS + t < cnt) fn(kreg[i]);
                }
            };
            for_each_key([&](LK k) { atomicAdd(&gcnt[digit_of<LK>(k, rest, dmask)], 1u); });
            __syncthreads();
            if (!scan_groups()) {
                for (int g0 = 0; g0 < (int)R;) {
                    // the longest run of whole groups from g0 on with at most CAP keys (a group has at most 64
                    // keys, so at least one fits): gstart ascends, the run's end is found by bisection
                    int g1 = g0 + 1, g_hi = (int)R;
                    const u32 part_end = gstart[g0] + (u32)CAP;
                    while (g1 < g_hi) {
                        const int mid = (g1 + g_hi + 1) >> 1;
                        if (gstart[mid] <= part_end) g1 = mid;
                        else g_hi = mid - 1;
                    }
                    const int part0 = (int)gstart[g0], part_n = (int)gstart[g1] - part0;
                    if (part_n > 0) {
                        for (int i = g0 + t; i < g1; i += THREADS) gcnt[i] = 0;
                        __syncthreads();
                        for_each_key([&](LK k) {
                            const int d = (int)digit_of<LK>(k, rest, dmask);
                            if (d >= g0 && d < g1) skey[gstart[d] - (u32)part0 + atomicAdd(&gcnt[d], 1u)] = k;
                        });
                        __syncthreads();
                        sort_groups(g0, g1);
                        for (int i = t; i < part_n; i += THREADS) kout[part0 + i] = skey[i];
                        __syncthreads();
                    }
                    g0 = g1;
                }
                done = true;
            }
            __syncthreads();
        }
        if (!done)  // ... else pass by pass through global memory
            bucket_sort_oversize<LK, false, THREADS>(kout, kin, nullptr, nullptr, cnt, low_bits, gcnt, L.smem);
        __threadfence();
        __syncthreads();
        emit([&](int i) { return coherent_load(&kout[i]); });
        return;
    }

    if (cnt > 0) {
        for (int i = t; i < (int)R; i += THREADS) gcnt[i] = 0;
        const int items = (cnt + THREADS - 1) / THREADS;  // <= ITEMS, the same in every thread
        LK key[ITEMS];
        u32 pos[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            key[i] = (LK)0;
            pos[i] = 0;
            if (i < items) {
                const int idx = i * THREADS + t;
                key[i] = kin[min(idx, cnt - 1)];  // (unconditional: all in flight together)
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i < items && i * THREADS + t < cnt) pos[i] = atomicAdd(&gcnt[digit_of<LK>(key[i], rest, dmask)], 1u);
        __syncthreads();
        const bool any_long = scan_groups();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i < items && i * THREADS + t < cnt) skey[gstart[digit_of<LK>(key[i], rest, dmask)] + pos[i]] = key[i];
        __syncthreads();
        if (rest > 0 && !any_long) {
            if (groups((int)R, false)) return;
            sort_groups(0, (int)R);
            if (groups((int)R, true)) return;
        } else if (rest > 0) {
            // some group is longer still: the whole bucket through a bitonic network, padded to a power of two
            int P = 64;
            while (P < cnt) P <<= 1;
            for (int i = cnt + t; i < P; i += THREADS) skey[i] = (LK) ~(LK)0;
            __syncthreads();
            for (int size = 2; size <= P; size <<= 1) {
                for (int stride = size >> 1; stride > 0; stride >>= 1) {
                    for (int q = t; q < P / 2; q += THREADS) {
                        const int i = 2 * q - (q & (stride - 1)), l = i + stride;
                        const bool up = (i & size) == 0;
                        const LK a = skey[i], b = skey[l];
                        if ((a > b) == up) {
                            skey[i] = b;
                            skey[l] = a;
                        }
                    }
                    __syncthreads();
                }
            }
        }
    }
    emit([&](int i) { return skey[i]; });
}

// What a workgroup makes of its bucket's sorted keys goes by an Out: emit(LDS, bucket, key_at) by the whole workgroup.
struct Bucket {
    int number, cnt, low_bits;
    u32 start;  // position of its first key among all keys
    // Keys are (row << shift) | item.  Of a key of this bucket: its item; its row; its row where only differences count.
    template <typename LK>
    __device__ __forceinline__ u32 item(LK k, int shift) const {
        return (u32)k & (u32)((1ull << shift) - 1ull);
    }
    template <typename LK>
    __device__ __forceinline__ u32 row_in(LK k, int shift) const {
        return (u32)(k >> shift);
    }
    template <typename LK>
    __device__ __forceinline__ int row(LK k, int shift) const {
        if constexpr (sizeof(LK) == 8) return (int)(k >> shift);
        const int within = low_bits - shift;  // 0 to 31: bits of the row below the bucket's number
        return (int)(((u32)number << within) | ((u32)(k >> shift) & ((1u << within) - 1u)));
    }
    template <typename LK>
    __device__ __forceinline__ u64 whole(LK k) const {
        if constexpr (sizeof(LK) == 8) return k;
        return ((u64)(u32)number << low_bits) | (u64)(low_bits >= 32 ? (u32)k : (u32)k & ((1u << low_bits) - 1u));
    }
};

// ... or, if it has emit_groups(LDS, bucket, R) and rows_are_groups(second, bucket, R) agrees, from the R groups of a bucket in LDS (BucketLds), which are
// sorted first or not (GROUPS_SORTED).
template <class Out, class = void>
struct TakesGroups : std::false_type {};
template <class Out>
struct TakesGroups<Out, std::void_t<decltype(&Out::rows_are_groups)>> : std::true_type {};

// ... and says for how many waves of a SIMD there are to be registers (MIN_WAVES; of keys whose workgroups LDS holds enough of).
template <class Out, class = void>
struct MinWaves : std::integral_constant<int, 1> {};
template <class Out>
struct MinWaves<Out, std::void_t<decltype(Out::MIN_WAVES)>> : std::integral_constant<int, Out::MIN_WAVES> {};

template <typename K, typename LK, int THREADS, int ITEMS, class Out>
__global__ __launch_bounds__(THREADS, sizeof(LK) == 4 ? MinWaves<Out>::value : 1) void bucket_keys_kernel(KeySort<K> first_sort, KeySort<K> second_sort, int blocks_first, Out out) {
    __shared__ BucketLds<LK, THREADS, ITEMS> L;
    __shared__ typename Out::template Lds<THREADS, ITEMS> O;
    const bool second = (int)blockIdx.x >= blocks_first;
    const KeySort<K>& S = second ? second_sort : first_sort;
    Bucket b;
    b.number = xcd_item((int)blockIdx.x - (second ? blocks_first : 0), S.buckets);
    if (b.number >= S.buckets) return;  // (a workgroup too many)
    b.cnt = (int)S.hist[b.number];
    b.start = S.starts[b.number];
    b.low_bits = S.key_bits - S.digit_bits;
    LK* kin = reinterpret_cast<LK*>(S.k1) + b.start;
    LK* kout = reinterpret_cast<LK*>(S.k0) + b.start;
    auto reset = [&] {  // (every thread has read its count: barriers lie between)
        if (threadIdx.x == 0 && b.cnt > 0) {
            S.hist[b.number] = 0;
            if (S.taken) S.taken[b.number] = 0;
        }
    };
    auto groups = [&](int R, bool sorted) -> bool {
        if constexpr (TakesGroups<Out>::value) {
            if (sorted != Out::GROUPS_SORTED || !out.rows_are_groups(second, b, R)) return false;
            reset();
            out.template emit_groups<THREADS, ITEMS>(L, b, R);
            return true;
        }
        return false;
    };
    sort_bucket<LK, THREADS, ITEMS>(L, kin, kout, b.cnt, b.low_bits, S.group_bits, groups, [&](auto key_at) {
        reset();
        out.template emit<THREADS, ITEMS>(second, O, b, kin, kout, key_at);
    });
}

// The sorted keys themselves (LK = K: what does not fit LDS is in its place already).
template <typename K>
struct PlainKeys {
    template <int THREADS, int ITEMS>
    struct Lds {};
    template <int THREADS, int ITEMS, class L, typename LK, class KeyAt>
    __device__ __forceinline__ void emit(bool, L&, const Bucket& b, LK*, LK* kout, KeyAt key_at) const {
        if (b.cnt <= THREADS * ITEMS)
            for (int i = threadIdx.x; i < b.cnt; i += THREADS) kout[i] = key_at(i);
    }
};

// The distinct keys, in order, at the front of the bucket's range of the partitioned array (whose keys have all been read),
// and how many they are: per bucket and, for whoever wants the number in front of a bucket, per UNIQUE_GROUP buckets (zero beforehand;
// a cache line each: a line takes an atomic every 11 to 14 ns, and 4,096 of them on the line of 16 such counters took 45 us).
constexpr int UNIQUE_GROUP = 256, UNIQUE_PAD = 32;
struct DistinctKeys {
    u32* per_bucket;
    u32* per_group;
    template <int THREADS, int ITEMS>
    struct Lds {
        u32 wave[THREADS / 64];
    };
    // A wave takes 64 * ITEMS keys in a row, so that one barrier does for the whole bucket.
    template <int THREADS, int ITEMS, class L, typename LK, class KeyAt>
    __device__ __forceinline__ void emit(bool, L& lds, const Bucket& b, LK* kin, LK*, KeyAt key_at) const {
        constexpr int NW = THREADS / 64;
        const int lane = lane_id(), w = wave_id();
        u32 total = 0;
        for (int base = 0; base < b.cnt; base += THREADS * ITEMS) {  // (once where the bucket is in LDS)
            const int n = min(b.cnt - base, THREADS * ITEMS);
            const int items = (n + THREADS - 1) / THREADS, i0 = base + w * 64 * items;
            u32 firsts = 0, cnt = 0;  // bit i: the lane's key i is the first of its kind
            for (int i = 0; i < items; ++i) {
                const int idx = i0 + i * 64 + lane, at = min(idx, b.cnt - 1);
                const bool first = idx < base + n && (idx == 0 || key_at(at) != key_at(max(at - 1, 0)));
                cnt += (u32)__popcll(ballot(first));
                firsts |= first ? 1u << i : 0u;
            }
            __syncthreads();
            if (lane == 0) lds.wave[w] = cnt;
            __syncthreads();
            u32 run = total;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const u32 c = lds.wave[j];
                if (j < w) run += c;
                total += c;
            }
            for (int i = 0; i < items; ++i) {
                const bool first = (firsts >> i & 1u) != 0;
                const u64 bal = ballot(first);
                if (first) kin[run + mask_below(bal)] = key_at(i0 + i * 64 + lane);
                run += (u32)__popcll(bal);
            }
        }
        if (threadIdx.x == 0) {
            per_bucket[b.number] = total;
            if (total) atomicAdd(&per_group[(b.number / UNIQUE_GROUP) * UNIQUE_PAD], total);
        }
    }
};

// Distinct keys in front of a bucket, by a whole workgroup.  smem: WAVES words.
__device__ __forceinline__ u32 distinct_in_front(const u32* __restrict__ per_bucket, const u32* __restrict__ per_group, int bucket, u32* smem) {
    const int group = bucket / UNIQUE_GROUP;
    u32 part = 0;
    for (int j = threadIdx.x; j < group; j += BLOCK) part += per_group[j * UNIQUE_PAD];
    for (int j = group * UNIQUE_GROUP + (int)threadIdx.x; j < bucket; j += BLOCK) part += per_bucket[j];
    return block_sum(part, smem);
}

// Two sorts in one launch (the second one's groups are not taken).
template <class A, class B>
struct TwoOuts {
    A a;
    B b;
    static constexpr bool GROUPS_SORTED = A::GROUPS_SORTED;
    __device__ bool rows_are_groups(bool second, const Bucket& bk, int R) const { return !second && a.rows_are_groups(false, bk, R); }
    template <int THREADS, int ITEMS, class L>
    __device__ __forceinline__ void emit_groups(L& lds, const Bucket& bk, int R) const {
        a.template emit_groups<THREADS, ITEMS>(lds, bk, R);
    }
    template <int THREADS, int ITEMS>
    union Lds {
        typename A::template Lds<THREADS, ITEMS> a;
        typename B::template Lds<THREADS, ITEMS> b;
    };
    template <int THREADS, int ITEMS, class L, typename LK, class KeyAt>
    __device__ __forceinline__ void emit(bool second, L& lds, const Bucket& bk, LK* kin, LK* kout, KeyAt key_at) const {
        if (second) b.template emit<THREADS, ITEMS>(second, lds.b, bk, kin, kout, key_at);
        else a.template emit<THREADS, ITEMS>(second, lds.a, bk, kin, kout, key_at);
    }
};

// Histogram of the top RBITS-bit digit (bits [shift, shift + RBITS)) over the whole input, added
// to `hist` (which starts at zero); tiles of BLOCK * ITEMS keys.
template <typename K, int RBITS, int ITEMS>
__global__ __launch_bounds__(BLOCK) void msd_histogram_kernel(const K* __restrict__ kin, const int* n_ptr, int n_host,
                                                              u32* __restrict__ hist, int shift) {
    constexpr int R = 1 << RBITS;
    constexpr int TILE = BLOCK * ITEMS;
    __shared__ u32 h[R];
    const int n = load_count(n_ptr, n_host);
    const long long base = (long long)blockIdx.x * TILE;
    if (base >= n) return;
    const int t = threadIdx.x;
    for (int i = t; i < R; i += BLOCK) h[i] = 0;
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < ITEMS; ++i) {
        const long long idx = base + (long long)i * BLOCK + t;
        if (idx < n) atomicAdd(&h[digit_of<K>(kin[idx], shift, R - 1)], 1u);
    }
    __syncthreads();
    for (int i = t; i < R; i += BLOCK) {
        const u32 c = h[i];
        if (c) atomicAdd(&hist[i], c);
    }
}

// A key source gives the keys of item i of the input, PER of them: an array (PER = 1), or a functor that makes the keys on the fly (so
// that keys which are a cheap function of other data need not be written out and read back): load(i) fetches what they are made of,
// without conditions, so that all of a lane's loads are in flight together; key(raw, i, c) is the c-th.  A key that the source
// does not keep is left out (and is not in the histogram): the output is as many keys shorter.
// Two sorts may share their launches (`second`: of the second one), where their inputs are there at the same time.
template <typename K>
struct ArrayKeys {
    const K* p;
    static constexpr int PER = 1;
    typedef K Raw;
    __device__ __forceinline__ K load(int i) const { return p[i]; }
    __device__ __forceinline__ K key(K raw, int, int) const { return raw; }
    __device__ __forceinline__ bool keep(K) const { return true; }
};
template <class A>
struct OneSource {
    A a;
    static constexpr int PER = A::PER;
    typedef typename A::Raw Raw;
    __device__ __forceinline__ Raw load(int i) const { return a.load(i); }
    __device__ __forceinline__ auto key(bool, const Raw& raw, int i, int c) const { return a.key(raw, i, c); }
    template <typename K>
    __device__ __forceinline__ bool keep(bool, K k) const { return a.keep(k); }
};
// (of the same items)
template <class A, class B>
struct TwoSources {
    A a;
    B b;
    static constexpr int PER = A::PER;
    typedef typename A::Raw Raw;
    __device__ __forceinline__ Raw load(int i) const { return a.load(i); }
    __device__ __forceinline__ auto key(bool second, const Raw& raw, int i, int c) const { return second ? b.key(raw, i, c) : a.key(raw, i, c); }
    template <typename K>
    __device__ __forceinline__ bool keep(bool second, K k) const { return second ? b.keep(k) : a.keep(k); }
};

// Partition of keys WITHOUT values by their top digit, of 8 to 10 bits (2^(BITS - 8) digits to a thread), in one pass.  hist[d] = number of keys with digit d over the whole input (so digit d owns the output range
// that starts at the sum of the counts before it; the first tile also writes these first
// positions to `starts`); taken[d] = how much of that range is in use, zero at the start.  Every tile counts its keys per digit in LDS, takes its share of each
// digit's range with one returning atomic per digit it holds, and writes its keys there.  The
// order of the keys inside a digit's range depends on the order in which tiles arrive, so this is
// for sorts that then order each range on the whole key; with equal keys indistinguishable the
// final result does not depend on it.  The lanes of a wave whose keys share a digit (keys led by
// mesh indices bring few distinct digits into a wave) rank themselves with one LDS atomic.
template <typename K, typename LK, int BITS, int ITEMS, class Src>
__global__ __launch_bounds__(BLOCK) void msd_scatter_kernel(KeySort<K> first_sort, KeySort<K> second_sort, int tiles_first, Src src) {
    constexpr int R = 1 << BITS, DIGITS = R / BLOCK, PER = Src::PER, KEYS = ITEMS * PER;
    static_assert(DIGITS * BLOCK == R, "whole digits per thread");
    constexpr int TILE = BLOCK * ITEMS;
    __shared__ u32 h[R];  // per digit: this tile's count, then where the tile's keys of that digit go
    __shared__ u32 smem[WAVES];
    const bool second = (int)blockIdx.x >= tiles_first;
    const KeySort<K>& S = second ? second_sort : first_sort;
    const int tile = (int)blockIdx.x - (second ? tiles_first : 0), tiles = second ? (int)gridDim.x - tiles_first : tiles_first;
    const int shift = S.key_bits - S.digit_bits;
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();
    // (an array that the kernel after this one adds to: zeroed here, by all workgroups together)
    for (int i = tile * BLOCK + t; i < S.n_zero; i += tiles * BLOCK) S.zero[i] = 0;
    const int n = load_count(S.n_ptr, S.n);
    const int base = tile * TILE + w * (64 * ITEMS) + lane;
    if (tile * TILE >= n) return;
    typename Src::Raw raw[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) raw[i] = src.load(min(base + i * 64, n - 1));
    u32 first[DIGITS], sum = 0, tot;  // first position of the ranges of the digits DIGITS * t ..
#pragma unroll
    for (int j = 0; j < DIGITS; ++j) {
        first[j] = S.hist[DIGITS * t + j];
        h[DIGITS * t + j] = 0;
    }
#pragma unroll
    for (int j = 0; j < DIGITS; ++j) {
        const u32 c = first[j];
        first[j] = sum;
        sum += c;
    }
    const u32 in_front = block_exclusive_scan(sum, smem, tot);
#pragma unroll
    for (int j = 0; j < DIGITS; ++j) {
        first[j] += in_front;
        if (tile == 0) S.starts[DIGITS * t + j] = first[j];  // for the kernel that sorts the ranges
    }
    if (tile == 0 && S.total && t == 0) *S.total = (int)tot;
    K key[KEYS];
    u32 rk[KEYS];
    bool has[KEYS];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        const int item = base + i / PER * 64;
        key[i] = src.key(second, raw[i / PER], item, i % PER);
        has[i] = item < n && src.keep(second, key[i]);
        const u32 d = digit_of<K>(key[i], shift, R - 1);
        // the lanes that share a digit rank themselves with one returning atomic, by the first of them
        const SameDigit same = wave_same_digit(has[i], d);
        u32 b = 0;
        if (has[i] && same.below == 0) b = atomicAdd(&h[d], same.count);
        rk[i] = (u32)__shfl((int)b, same.lead, 64) + same.below;
    }
    __syncthreads();
    u32 c[DIGITS];
#pragma unroll
    for (int j = 0; j < DIGITS; ++j) {
        c[j] = h[DIGITS * t + j];
        if (c[j]) first[j] += atomicAdd(&S.taken[DIGITS * t + j], c[j]);
    }
#pragma unroll
    for (int j = 0; j < DIGITS; ++j)
        if (c[j]) h[DIGITS * t + j] = first[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        if (has[i]) {
            const u32 pos = h[digit_of<K>(key[i], shift, R - 1)] + rk[i];
            if (pos < (u32)n * PER) reinterpret_cast<LK*>(S.k1)[pos] = (LK)key[i];  // (always, when hist and taken are as described)
        }
    }
}

// Words of each of a sort's arrays (KeySort) for digits of up to 12 bits, and the arrays: hist, taken, cursor, starts, in a row.  The
// first MSD_ZERO_WORDS are zero between sorts.
constexpr int MSD_HIST_WORDS = 4096, MSD_WORDS = 4 * MSD_HIST_WORDS, MSD_ZERO_WORDS = 2 * MSD_HIST_WORDS;
template <typename K>
inline void use_arrays(KeySort<K>& S, u32* arrays) {
    S.hist = arrays;
    S.taken = arrays + MSD_HIST_WORDS;
    S.cursor = arrays + 2 * MSD_HIST_WORDS;
    S.starts = arrays + 3 * MSD_HIST_WORDS;
}
inline int bucket_sort_msd_bits(int key_bits) { return key_bits < BUCKET_MSD_BITS ? key_bits : BUCKET_MSD_BITS; }

__global__ __launch_bounds__(BLOCK) void fill_u32_kernel(u32* __restrict__ p, int n, u32 v) {
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < n) p[i] = v;
}

template <typename K, bool HAS_VAL>
inline int bucket_sort(hipStream_t s, K* k0, K* k1, u32* v0, u32* v1, const int* n_ptr, int n_max, int key_bits,
                       const SortScratch& sc) {
    if (n_max <= 0 || key_bits <= 0) return 0;
    const int msd = bucket_sort_msd_bits(key_bits);
    const int low = key_bits - msd;
    const int tiles = sort_tiles(n_max, SORT_ITEMS_SMALL);
    radix_upsweep_kernel<K, SORT_ITEMS_SMALL><<<tiles, BLOCK, 0, s>>>(k0, n_ptr, n_max, sc.T, sc.table, low, msd);
    radix_scan_kernel<<<1 << msd, BLOCK, 0, s>>>(sc.table, sc.totals, n_ptr, n_max, sc.T, BLOCK * SORT_ITEMS_SMALL);
    radix_downsweep_kernel<K, HAS_VAL, SORT_ITEMS_SMALL>
        <<<tiles, BLOCK, 0, s>>>(k0, k1, v0, v1, n_ptr, n_max, sc.T, sc.table, sc.totals, low, msd);
    bucket_sort_kernel<K, HAS_VAL, BUCKET_THREADS_256, 8>
        <<<1 << msd, BUCKET_THREADS_256, 0, s>>>(k1, k0, v1, v0, sc.totals, 1 << msd, low);
    if (hipGetLastError() != hipSuccess) return -1;
    return 0;
}

// Larger inputs (up to BUCKET_SORT_LARGE_MAX_KEYS): 4096 buckets on the top 12
// bits.  A single 12-bit partition pass would scatter about one key per digit
// and tile, so the partition is done as two stable 6-bit passes (low half
// first), and the bucket sizes come from a 12-bit histogram taken up front.
constexpr int BUCKET_LARGE_MSD_BITS = 12;
constexpr long long BUCKET_SORT_LARGE_MAX_KEYS = 1ll << 23;

// Histogram of the top 12-bit digit over the whole input (added to `hist`, which starts at zero),
// and from the same read of the keys the first partition pass's per-tile counts of the digit's
// low 6 bits (table[d6 * T + tile], what radix_upsweep_kernel would compute for bits
// [shift, shift + 6)).  Keys made from mesh indices often share their leading bits across a
// whole wave; such a wave counts itself with a single LDS atomic.
template <typename K>
__global__ __launch_bounds__(BLOCK) void top_digit_histogram_kernel(const K* __restrict__ kin, const int* n_ptr,
                                                                    int n_host, u32* __restrict__ hist, int shift, int T,
                                                                    u32* __restrict__ table) {
    constexpr int R = 1 << BUCKET_LARGE_MSD_BITS;
    constexpr int TILE = BLOCK * SORT_ITEMS_BIG;
    __shared__ u32 h[R];
    const int n = load_count(n_ptr, n_host);
    const long long base = (long long)blockIdx.x * TILE;
    if (base >= n) return;
    const int t = threadIdx.x;
    for (int i = t; i < R; i += BLOCK) h[i] = 0;
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < SORT_ITEMS_BIG; ++i) {
        const long long idx = base + (long long)i * BLOCK + t;
        const bool ok = idx < n;
        const u32 d = ok ? digit_of<K>(kin[idx], shift, R - 1) : 0u;
        const u64 on = ballot(ok);
        if (on == 0) continue;
        const u32 d0 = (u32)__builtin_amdgcn_readfirstlane((int)d);  // (of the first lane with a key)
        if (ballot(ok && d == d0) == on) {
            if (ok && (on & lanemask_lt()) == 0) atomicAdd(&h[d0], (u32)__popcll(on));
        } else if (ok) {
            atomicAdd(&h[d], 1u);
        }
    }
    __syncthreads();
    for (int i = t; i < R; i += BLOCK) {
        const u32 c = h[i];
        if (c) atomicAdd(&hist[i], c);
    }
    if (t < 64) {
        u32 sum = 0;
        for (int hi = 0; hi < 64; ++hi) sum += h[(hi << 6) | t];
        table[(size_t)t * T + blockIdx.x] = sum;
    }
}

// Keys with values.  Result is in (k1, v1): returns 1; <0 on a launch error.  hist12 holds MSD_HIST_WORDS words.
template <typename K>
inline int bucket_sort_large(hipStream_t s, K* k0, K* k1, u32* v0, u32* v1, const int* n_ptr, int n_max, int key_bits,
                             const SortScratch& sc, u32* hist12) {
    constexpr int R = 1 << BUCKET_LARGE_MSD_BITS;
    const int low = key_bits - BUCKET_LARGE_MSD_BITS;
    const int tiles = sort_tiles(n_max, SORT_ITEMS_BIG);
    fill_u32_kernel<<<R / BLOCK, BLOCK, 0, s>>>(hist12, R, 0u);
    top_digit_histogram_kernel<K><<<tiles, BLOCK, 0, s>>>(k0, n_ptr, n_max, hist12, low, sc.T, sc.table);
    K* kin = k0;
    K* kout = k1;
    u32* vin = v0;
    u32* vout = v1;
    for (int half = 0; half < 2; ++half) {
        const int shift = low + 6 * half;
        if (half == 1)  // (the histogram kernel has left the first pass's counts)
            radix_upsweep_kernel<K, SORT_ITEMS_BIG><<<tiles, BLOCK, 0, s>>>(kin, n_ptr, n_max, sc.T, sc.table, shift, 6);
        radix_scan_kernel<<<64, BLOCK, 0, s>>>(sc.table, sc.totals, n_ptr, n_max, sc.T, BLOCK * SORT_ITEMS_BIG);
        radix_downsweep_kernel<K, true, SORT_ITEMS_BIG>
            <<<tiles, BLOCK, 0, s>>>(kin, kout, vin, vout, n_ptr, n_max, sc.T, sc.table, sc.totals, shift, 6);
        K* tk = kin; kin = kout; kout = tk;
        u32* tv = vin; vin = vout; vout = tv;
    }
    // after two passes the partitioned keys are back in (k0, v0)
    bucket_sort_kernel<K, true, BUCKET_THREADS_4096, 16>
        <<<R, BUCKET_THREADS_4096, 0, s>>>(k0, k1, v0, v1, hist12, R, low);
    if (hipGetLastError() != hipSuccess) return -1;
    return 1;
}

// ---------------------------------------------------------------------------
// Keys without values beyond BUCKET_SORT_MAX_KEYS: the same two sweeps (partition on a top digit, then one workgroup
// per bucket), with a digit of 11 or 12 bits, beyond BUCKET_SORT_LARGE_MAX_KEYS as wide as the input needs for buckets of
// BUCKET_KEYS_AIM keys at most, half of that at least.  Arrays with one word per digit then do not fit LDS, or fill it; a tile of mesh keys holds few
// distinct digits, though, so it counts them in a small hash table.  Bound by memory: 8 bytes read and 8 written per key and sweep
// (less 4 read where keys are made on the fly), where plain radix passes read every key twice and wrote it once for
// every 8 bits (61 M keys of 48 bits: 6 passes, 2.9 ms; this way 0.5 ms).
// ---------------------------------------------------------------------------
constexpr int XL_BITS_MIN = 13, XL_BITS_MAX = 22;
// Keys per bucket, over all that there can be, at most: 1,000 to 2,000 from 2^22 keys on, 500 to 2,000 from 2^20.  Ids that fill
// little more than half of their bit range leave almost half of the buckets empty, and the others hold up to twice that.  A workgroup's own
// part (counters, their prefix sums, what is made of the keys) costs as much as 700 keys do (33 M keys of the second round of 10.2 M
// vertices: 711 to a bucket 230 us, 1,422 to a bucket 140).
constexpr long long BUCKET_KEYS_AIM = 2048;
// Below 2^20 keys the chip also has to be filled.  Partition and bucket sorts of the first round of lattices, us with 8 / 9 / 10 bits: 64 k
// keys 12.0 / 13.4 / 14.4, 147 k 13.0 / 14.3 / 16.8, 220 k 15.6 / 14.9 / 14.7, 368 k 18.2 / 17.6 / 19.7, 500 k 20.7 / 19.7 / 18.4, 682 k
// 21.8 / 20.0 / 22.0, 740 k 22.4 / 20.3 / 23.0, 790 k 75 / 24.1 / 21.0, 920 k 80 / 27.8 / 25.0, 1 M 85 / 29.1 / 24.6 (eight bits from 786 k on: buckets
// beyond what LDS holds).  So 9 bits end where 10 are better; 8 bits could go to about 180 k, for a microsecond.
constexpr long long NARROW_8_BITS_MAX_KEYS = 1 << 16, NARROW_9_BITS_MAX_KEYS = 3 << 18;
inline int xl_bits_for(long long n) {
    int b = XL_BITS_MIN;
    while (b < XL_BITS_MAX - 2 && (BUCKET_KEYS_AIM << b) < n) ++b;
    return b;
}
// Up to two bits more where the bits below the digit then fit the 32 that the per-bucket kernel keeps in LDS.
inline int xl_digit_bits(long long n, int key_bits) {
    const int b = xl_bits_for(n), want = key_bits - 32;
    return want > b && want <= b + 2 ? want : b;
}
// words of the count, first-position and cursor arrays for inputs of up to n_cap keys
inline size_t xl_hist_words(long long n_cap) { return (size_t)1 << (xl_bits_for(n_cap) + 2); }

struct XlScratch {
    u32* hist = nullptr;    // keys per digit
    u32* starts = nullptr;  // first position of every digit's range
    u32* cursor = nullptr;  // next free position in it
};

// Bits of the digit that up to n keys of key_bits bits are partitioned on, and how many bits a key must have for it.
inline int key_digit_bits(long long n, int key_bits) {
    if (n <= BUCKET_SORT_MAX_KEYS) return n <= NARROW_8_BITS_MAX_KEYS ? 8 : (n <= NARROW_9_BITS_MAX_KEYS ? 9 : 10);
    if (n <= BUCKET_KEYS_AIM << (BUCKET_LARGE_MSD_BITS - 1)) return BUCKET_LARGE_MSD_BITS - 1;
    return n <= BUCKET_SORT_LARGE_MAX_KEYS ? BUCKET_LARGE_MSD_BITS : xl_digit_bits(n, key_bits);
}
// buckets of inputs of up to n_cap keys, at most
inline size_t bucket_capacity(long long n_cap) {
    const size_t narrow = (size_t)1 << BUCKET_LARGE_MSD_BITS;
    return n_cap <= BUCKET_SORT_LARGE_MAX_KEYS ? narrow : xl_hist_words(n_cap);
}
inline int key_bits_wanted(long long n) {
    if (n <= BUCKET_SORT_MAX_KEYS) return NARROW_BITS_MAX + 2;
    return n <= BUCKET_SORT_LARGE_MAX_KEYS ? BUCKET_LARGE_MSD_BITS + 2 : XL_BITS_MAX + 2;
}

// A workgroup's counts of wide digits: a small hash table in LDS, as a tile of mesh keys holds few distinct digits.  clear,
// add and flush by the whole workgroup, with barriers between them.  (Straight to memory, with an atomic per wave and digit,
// counting took 270-400 us of a round of 61 M half-edges.)
constexpr int XL_SLOTS = 512, XL_PROBES = 8;
constexpr u32 XL_NONE = 0xFFFFFFFFu;
struct DigitTable {
    u32 digit[XL_SLOTS];
    u32 count[XL_SLOTS];
    __device__ __forceinline__ void clear() {
        for (int i = threadIdx.x; i < XL_SLOTS; i += BLOCK) {
            digit[i] = XL_NONE;
            count[i] = 0;
        }
    }
    // the digit's slot, or XL_NONE where it finds no place
    __device__ __forceinline__ u32 slot_of(u32 d) {
        u32 h = (d * 0x9E3779B1u) >> 23;  // 9 bits
        for (int p = 0; p < XL_PROBES; ++p) {
            const u32 old = atomicCAS(&digit[h], XL_NONE, d);
            if (old == XL_NONE || old == d) return h;
            h = (h + 1) & (XL_SLOTS - 1);
        }
        return XL_NONE;
    }
    // one key for every lane with `ok`: the lanes of a wave that share a digit by the first of them
    __device__ __forceinline__ void add(u32* __restrict__ hist, bool ok, u32 d) {
        const SameDigit same = wave_same_digit(ok, d);
        if (ok && same.below == 0) {
            const u32 s = slot_of(d);
            atomicAdd(s != XL_NONE ? &count[s] : &hist[d], same.count);
        }
    }
    __device__ __forceinline__ void flush(u32* __restrict__ hist) {
        for (int i = threadIdx.x; i < XL_SLOTS; i += BLOCK)
            if (digit[i] != XL_NONE) atomicAdd(&hist[digit[i]], count[i]);
    }
};

template <typename K>
__global__ __launch_bounds__(BLOCK) void xl_count_kernel(const K* __restrict__ kin, const int* n_ptr, int n_host, int shift, u32 mask,
                                                         u32* __restrict__ hist) {
    constexpr int ITEMS = 4;
    __shared__ DigitTable table;
    const int n = load_count(n_ptr, n_host);
    const long long base = (long long)blockIdx.x * (BLOCK * ITEMS);
    if (base >= n) return;
    table.clear();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const long long idx = base + (long long)i * BLOCK + threadIdx.x;
        table.add(hist, idx < n, digit_of<K>(idx < n ? kin[idx] : (K)0, shift, mask));
    }
    __syncthreads();
    table.flush(hist);
}

// starts = cursor = exclusive prefix sums of hist[0, 2^digit_bits), a multiple of KEY_SCAN_DIGITS: every workgroup adds up what lies
// in front of its digits by itself.
constexpr int KEY_SCAN_THREADS = 1024, KEY_SCAN_ITEMS = 4, KEY_SCAN_DIGITS = KEY_SCAN_THREADS * KEY_SCAN_ITEMS;
template <typename K>
__global__ __launch_bounds__(KEY_SCAN_THREADS) void key_starts_kernel(KeySort<K> first_sort, KeySort<K> second_sort, int blocks_first) {
    __shared__ u32 smem[KEY_SCAN_THREADS / 64];
    const bool second = (int)blockIdx.x >= blocks_first;
    const KeySort<K>& S = second ? second_sort : first_sort;
    const int block = (int)blockIdx.x - (second ? blocks_first : 0), blocks = second ? (int)gridDim.x - blocks_first : blocks_first;
    const int t = threadIdx.x, d0 = block * KEY_SCAN_DIGITS;
    for (int i = block * KEY_SCAN_THREADS + t; i < S.n_zero; i += blocks * KEY_SCAN_THREADS) S.zero[i] = 0;
    const uint4* h4 = reinterpret_cast<const uint4*>(S.hist);
    const uint4 c = h4[d0 / 4 + t];
    u32 before = 0, in_front, tot;
#pragma unroll 8
    for (int i = t; i < d0 / 4; i += KEY_SCAN_THREADS) {
        const uint4 q = h4[i];
        before += (q.x + q.y) + (q.z + q.w);
    }
    wide_block_exclusive_scan<KEY_SCAN_THREADS / 64>(before, smem, in_front);
    const u32 sum = (c.x + c.y) + (c.z + c.w);
    const u32 at = in_front + wide_block_exclusive_scan<KEY_SCAN_THREADS / 64>(sum, smem, tot);
    const uint4 o = make_uint4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
    reinterpret_cast<uint4*>(S.starts)[d0 / 4 + t] = o;
    reinterpret_cast<uint4*>(S.cursor)[d0 / 4 + t] = o;
    if (S.total && block == blocks - 1 && t == KEY_SCAN_THREADS - 1) *S.total = (int)(at + sum);
}

// The partition: a tile's distinct digits are entered into a hash table in LDS (the lanes of a wave that share a digit
// by the first of them), which counts their keys and so ranks them; each digit then takes its share of
// its range with one returning atomic.  A digit that finds no place within XL_PROBES steps (a tile without locality)
// takes its places right away.  The order of the keys inside a range does not matter (see msd_scatter_kernel).
// Bound by the chain of a workgroup (keys, ranks, shares, stores) and by vector issue, so 8 or 9 keys per lane (with 16 half as many
// workgroups fit a compute unit, at 1.5 times the time), the three keys of a facet from one load of it, and every load of a lane in flight
// before the first key is made (a branch around each had them wait for one another).  Both sorts of 10.2 M vertices, 123 M keys: 401 -> 224 us;
// 1.2 M: 44 -> 38; with the narrow digits (msd_scatter_kernel) 115 k: 9.6 -> 7.9, 4 k: 6.0 -> 4.5.
constexpr int xl_items(int per) { return per == 3 ? 3 : 8; }
template <typename K, typename LK, class Src>
__global__ __launch_bounds__(BLOCK) void xl_scatter_kernel(KeySort<K> first_sort, KeySort<K> second_sort, int tiles_first, Src src) {
    constexpr int PER = Src::PER, ITEMS = xl_items(PER), KEYS = PER * ITEMS, TILE = BLOCK * ITEMS;
    static_assert(BLOCK * KEYS <= 0xFFFF && XL_SLOTS <= 0x7FFF, "a slot and a rank in one word");
    __shared__ DigitTable T;  // (count: keys of the tile with that digit, then where they go)
    const bool second = (int)blockIdx.x >= tiles_first;
    const KeySort<K>& S = second ? second_sort : first_sort;
    const int n = load_count(S.n_ptr, S.n);
    const int tile = (int)blockIdx.x - (second ? tiles_first : 0);
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();
    const int base = tile * TILE + w * (64 * ITEMS) + lane;
    if (tile * TILE >= n) return;
    typename Src::Raw raw[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) raw[i] = src.load(min(base + i * 64, n - 1));
    const int shift = S.key_bits - S.digit_bits;
    const u32 mask = (1u << S.digit_bits) - 1u;
    u32* __restrict__ cursor = S.cursor;
    T.clear();
    K key[KEYS];
    u32 at[KEYS];  // slot and rank within the tile's keys of the digit, or its place (then slot XL_NONE)
    bool has[KEYS], alone[KEYS];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        const int item = base + i / PER * 64;
        key[i] = src.key(second, raw[i / PER], item, i % PER);
        has[i] = item < n && src.keep(second, key[i]);
        const u32 d = digit_of<K>(key[i], shift, mask);
        const SameDigit same = wave_same_digit(has[i], d);
        u32 b = 0, place = 0;
        if (has[i] && same.below == 0) {
            const u32 slot = T.slot_of(d);
            if (slot != XL_NONE) b = (slot << 16) | atomicAdd(&T.count[slot], same.count);
            else {
                b = XL_NONE;
                place = atomicAdd(&cursor[d], same.count);
            }
        }
        b = (u32)__shfl((int)b, same.lead, 64);
        alone[i] = b == XL_NONE;
        if (__any(alone[i])) place = (u32)__shfl((int)place, same.lead, 64);
        at[i] = (alone[i] ? place : b) + same.below;
    }
    __syncthreads();
    u32 share[XL_SLOTS / BLOCK];  // (all of a thread's atomics in flight together)
#pragma unroll
    for (int j = 0; j < XL_SLOTS / BLOCK; ++j) {
        const u32 d = T.digit[j * BLOCK + t];
        share[j] = d != XL_NONE ? atomicAdd(&cursor[d], T.count[j * BLOCK + t]) : 0u;
    }
#pragma unroll
    for (int j = 0; j < XL_SLOTS / BLOCK; ++j) T.count[j * BLOCK + t] = share[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        if (has[i]) {
            const u32 pos = alone[i] ? at[i] : T.count[at[i] >> 16] + (at[i] & 0xFFFFu);
            if (pos < (u32)n * PER) reinterpret_cast<LK*>(S.k1)[pos] = (LK)key[i];  // (always, when hist and cursor are as described)
        }
    }
}

// Sorts the keys of `src` (whose digits are in a.hist) for `out`; with b, a second sort of the same kind in the same launches
// (both with 32-bit keys behind the partition, or neither).  false on a launch error.  `lt`: brackets the launch of the partition
// (part_tag >= 0) and of the per-bucket kernel.
template <typename K, class Src, class Out>
inline bool key_sort(hipStream_t s, const KeySort<K>& a, const KeySort<K>* b_or_null, const Src& src, const Out& out,
                     LaunchTimer* lt = nullptr, int tag = 0, int part_tag = -1) {
    const KeySort<K> none{};
    const KeySort<K>& b = b_or_null ? *b_or_null : none;
    const int digits_a = 1 << a.digit_bits, digits_b = b_or_null ? 1 << b.digit_bits : 0;
    const int blocks_sort_a = xcd_grid(a.buckets), blocks_sort_b = xcd_grid(b.buckets);
    constexpr int NARROW_ITEMS = Src::PER == 3 ? 1 : SORT_ITEMS_SMALL;
    const bool narrow = a.digit_bits <= NARROW_BITS_MAX;
    auto launch = [&](auto lk) {
        using LK = decltype(lk);
        bool timed = lt && part_tag >= 0 && lt->begin(s, part_tag);
        if (narrow) {
            const int tiles_a = sort_tiles(a.n, NARROW_ITEMS), tiles_b = b_or_null ? sort_tiles(b.n, NARROW_ITEMS) : 0;
            if (a.digit_bits == 8) msd_scatter_kernel<K, LK, 8, NARROW_ITEMS, Src><<<tiles_a + tiles_b, BLOCK, 0, s>>>(a, b, tiles_a, src);
            else if (a.digit_bits == 9) msd_scatter_kernel<K, LK, 9, NARROW_ITEMS, Src><<<tiles_a + tiles_b, BLOCK, 0, s>>>(a, b, tiles_a, src);
            else msd_scatter_kernel<K, LK, 10, NARROW_ITEMS, Src><<<tiles_a + tiles_b, BLOCK, 0, s>>>(a, b, tiles_a, src);
        } else {
            // (arrays of the narrower digits have KEY_SCAN_DIGITS words)
            const int blocks_a = (digits_a + KEY_SCAN_DIGITS - 1) / KEY_SCAN_DIGITS, blocks_b = (digits_b + KEY_SCAN_DIGITS - 1) / KEY_SCAN_DIGITS;
            key_starts_kernel<K><<<blocks_a + blocks_b, KEY_SCAN_THREADS, 0, s>>>(a, b, blocks_a);
            const int tiles_a = sort_tiles(a.n, xl_items(Src::PER)), tiles_b = b_or_null ? sort_tiles(b.n, xl_items(Src::PER)) : 0;
            xl_scatter_kernel<K, LK, Src><<<tiles_a + tiles_b, BLOCK, 0, s>>>(a, b, tiles_a, src);
        }
        if (timed) lt->end(s);
        timed = lt && lt->begin(s, tag);
        const int blocks = blocks_sort_a + blocks_sort_b;
        if (TakesGroups<Out>::value && !b_or_null && !a.crowded && (long long)a.n * Src::PER <= (long long)BUCKET_FEW_KEYS * a.buckets)
            bucket_keys_kernel<K, LK, BUCKET_KEYS_THREADS / 2, BUCKET_KEYS_ITEMS, Out><<<blocks, BUCKET_KEYS_THREADS / 2, 0, s>>>(a, b, blocks_sort_a, out);
        else
            bucket_keys_kernel<K, LK, BUCKET_KEYS_THREADS, BUCKET_KEYS_ITEMS, Out><<<blocks, BUCKET_KEYS_THREADS, 0, s>>>(a, b, blocks_sort_a, out);
        if (timed) lt->end(s);
    };
    if constexpr (std::is_same<Out, PlainKeys<K>>::value) launch(K{});
    else if (a.half) launch(u32{});
    else launch(K{});
    return hipGetLastError() == hipSuccess;
}

// The same for keys in a.k0 that have not been counted.
template <typename K>
inline bool key_sort_array(hipStream_t s, const KeySort<K>& a) {
    const int low = a.key_bits - a.digit_bits, buckets = 1 << a.digit_bits;
    fill_u32_kernel<<<(buckets + BLOCK - 1) / BLOCK, BLOCK, 0, s>>>(a.hist, buckets, 0u);
    if (a.digit_bits <= NARROW_BITS_MAX) {
        fill_u32_kernel<<<(buckets + BLOCK - 1) / BLOCK, BLOCK, 0, s>>>(a.taken, buckets, 0u);
        msd_histogram_kernel<K, NARROW_BITS_MAX, SORT_ITEMS_SMALL><<<sort_tiles(a.n, SORT_ITEMS_SMALL), BLOCK, 0, s>>>(a.k0, a.n_ptr, a.n, a.hist, low);
    } else if (a.digit_bits == BUCKET_LARGE_MSD_BITS) {
        msd_histogram_kernel<K, BUCKET_LARGE_MSD_BITS, SORT_ITEMS_BIG><<<sort_tiles(a.n, SORT_ITEMS_BIG), BLOCK, 0, s>>>(a.k0, a.n_ptr, a.n, a.hist, low);
    } else {
        xl_count_kernel<K><<<sort_tiles(a.n, 4), BLOCK, 0, s>>>(a.k0, a.n_ptr, a.n, low, (u32)buckets - 1u, a.hist);
    }
    return key_sort(s, a, (const KeySort<K>*)nullptr, OneSource<ArrayKeys<K>>{{a.k0}}, PlainKeys<K>{});
}

// ---------------------------------------------------------------------------
// Flag compaction.  count kernel: tilesum[tile] = number of i in the tile with
// pred(i).  scatter kernel: calls out(i, rank) for every flagged i, rank = its
// position among flagged items in index order; writes the grand total.
// Tile = 256 x CHUNKS items (CHUNKS = 1, 4 or 16 per lane); wave w of a workgroup
// owns items [w * 64 * CHUNKS, (w + 1) * 64 * CHUNKS) of the tile.  As few items per
// lane as the tile limit allows: with one item per lane nothing in a lane waits
// for the item before it (measured: a limit of 8192 tiles instead of 2048 took
// 9 us off room115k, 29 us off scene1p2m, 21 us off the 16-mesh batch; 16384
// costs scene1p2m 30 us again, every workgroup of the scatter kernel adding up
// the sums of the tiles in front of it).
// ---------------------------------------------------------------------------
constexpr int COMPACT_MAX_SUMMED_TILES = 8192;  // beyond this the tile sums are scanned by a kernel of their own

inline int compact_chunks_for(long long n_max) {
    if ((n_max + BLOCK - 1) / BLOCK <= COMPACT_MAX_SUMMED_TILES) return 1;
    if ((n_max + 4 * BLOCK - 1) / (4 * BLOCK) <= COMPACT_MAX_SUMMED_TILES) return 4;
    return 16;
}
inline int compact_tiles(long long n, int chunks) {
    return (int)((n + (long long)BLOCK * chunks - 1) / ((long long)BLOCK * chunks));
}
// capacity of the tile-sum array for inputs of up to n_cap items
inline int compact_tilesum_capacity(long long n_cap) {
    const int big = compact_tiles(n_cap, 16);
    return (big > COMPACT_MAX_SUMMED_TILES ? big : COMPACT_MAX_SUMMED_TILES) + 1;
}

// A counting predicate may provide `void on_start() const`: one thread of the count kernel calls it
// before anything else, whatever the number of items (used to tell the host that the kernels in
// front of this one on the stream are done).
template <class P, class = void>
struct pred_has_on_start : std::false_type {};
template <class P>
struct pred_has_on_start<P, std::void_t<decltype(std::declval<const P&>().on_start())>> : std::true_type {};

template <class Pred, int CHUNKS>
__global__ __launch_bounds__(BLOCK) void tile_count_kernel(Pred pred, const int* n_ptr, int n_host,
                                                           int* __restrict__ tilesum) {
    constexpr int CTILE = BLOCK * CHUNKS;
    __shared__ u32 smem[WAVES];
    if constexpr (pred_has_on_start<Pred>::value) {
        if (blockIdx.x == 0 && threadIdx.x == 0) pred.on_start();
    }
    const int n = load_count(n_ptr, n_host);
    const long long base = (long long)blockIdx.x * CTILE;
    if (base >= n) return;
    const int w = wave_id(), lane = lane_id();
    u32 cnt = 0;
    for (int c = 0; c < CHUNKS; ++c) {
        const long long i = base + (long long)w * (64 * CHUNKS) + c * 64 + lane;
        const bool f = (i < n) && pred((int)i);
        cnt += (u32)__popcll(ballot(f));
    }
    if (lane == 0) smem[w] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) tilesum[blockIdx.x] = (int)(smem[0] + smem[1] + smem[2] + smem[3]);
}

// In-place exclusive scan of a[0..T) by one workgroup (used when there are many tiles): 8 consecutive sums per thread
// and step, the next step's loads issued before the scan of this one.  (15,000 tiles: 36 us with one sum per thread.)
constexpr int SCAN_TILES_THREADS = 1024, SCAN_TILES_ITEMS = 8;
__global__ __launch_bounds__(SCAN_TILES_THREADS) void scan_tilesums_kernel(int* __restrict__ a, const int* n_ptr, int n_host,
                                                                           int tile_items) {
    constexpr int ITEMS = SCAN_TILES_ITEMS, STEP = SCAN_TILES_THREADS * ITEMS;
    __shared__ u32 smem[SCAN_TILES_THREADS / 64];
    const int n = load_count(n_ptr, n_host);
    const int T = (int)(((long long)n + tile_items - 1) / tile_items);
    const int t = threadIdx.x;
    u32 v[ITEMS], next[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) next[j] = t * ITEMS + j < T ? (u32)a[t * ITEMS + j] : 0u;
    u32 carry = 0;
    for (int c = 0; c < T; c += STEP) {
        u32 sum = 0, tot;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            v[j] = next[j];
            sum += v[j];
            const int i = c + STEP + t * ITEMS + j;
            next[j] = i < T ? (u32)a[i] : 0u;
        }
        u32 run = carry + wide_block_exclusive_scan<SCAN_TILES_THREADS / 64>(sum, smem, tot);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int i = c + t * ITEMS + j;
            if (i < T) a[i] = (int)run;
            run += v[j];
        }
        carry += tot;
    }
}

// An output functor may declare `static constexpr bool WAVE_WIDE = true` and provide
// wave(i, in_range, flagged, pos), which all 64 lanes of a wave call together (so it may use
// cross-lane operations), in place of operator()(i, pos) called by the flagged lanes only.
template <class Out, class = void>
struct out_is_wave_wide : std::false_type {};
template <class Out>
struct out_is_wave_wide<Out, std::enable_if_t<Out::WAVE_WIDE>> : std::true_type {};

template <class Pred, class Out, int CHUNKS>
__global__ __launch_bounds__(BLOCK) void tile_scatter_kernel(Pred pred, Out out, const int* n_ptr, int n_host,
                                                             const int* __restrict__ tilesum, int prefixed,
                                                             int* __restrict__ total_out) {
    constexpr int CTILE = BLOCK * CHUNKS;
    __shared__ u32 smem[WAVES];
    const int n = load_count(n_ptr, n_host);
    if (n <= 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0 && total_out) *total_out = 0;
        return;
    }
    const int tile = blockIdx.x;
    const long long base = (long long)tile * CTILE;
    if (base >= n) return;
    const int t = threadIdx.x, w = wave_id(), lane = lane_id();

    u32 tileoff;
    if (prefixed) {
        tileoff = (u32)tilesum[tile];
    } else {
        u32 part = 0;
        for (int j = t; j < tile; j += BLOCK) part += (u32)tilesum[j];
        tileoff = block_sum(part, smem);
    }

    u64 bal[CHUNKS];
    u32 cnt = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const long long i = base + (long long)w * (64 * CHUNKS) + c * 64 + lane;
        const bool f = (i < n) && pred((int)i);
        bal[c] = ballot(f);
        cnt += (u32)__popcll(bal[c]);
    }
    __syncthreads();
    if (lane == 0) smem[w] = cnt;
    __syncthreads();
    u32 woff = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        if (i < w) woff += smem[i];
        tot += smem[i];
    }
    u32 run = tileoff + woff;
    const u64 lt = lanemask_lt();
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const long long i = base + (long long)w * (64 * CHUNKS) + c * 64 + lane;
        const bool f = ((bal[c] >> lane) & 1ull) != 0;
        const int pos = (int)(run + (u32)__popcll(bal[c] & lt));
        if constexpr (out_is_wave_wide<Out>::value) {
            out.wave((int)i, i < n, f, pos);  // every lane of the wave calls it
        } else {
            if (f) out((int)i, pos);
        }
        run += (u32)__popcll(bal[c]);
    }
    if (base + CTILE >= n && t == 0 && total_out) *total_out = (int)(tileoff + tot);
}

template <class PredCount, class PredScatter, class Out, int CHUNKS>
inline void compact_impl(hipStream_t s, PredCount pc, PredScatter ps, Out out, const int* n_ptr, int n_max,
                         int* tilesum, int* total_out) {
    const int tiles = compact_tiles(n_max > 0 ? n_max : 1, CHUNKS);
    tile_count_kernel<PredCount, CHUNKS><<<tiles, BLOCK, 0, s>>>(pc, n_ptr, n_max, tilesum);
    const int prefixed = tiles > COMPACT_MAX_SUMMED_TILES;
    if (prefixed) scan_tilesums_kernel<<<1, SCAN_TILES_THREADS, 0, s>>>(tilesum, n_ptr, n_max, BLOCK * CHUNKS);
    tile_scatter_kernel<PredScatter, Out, CHUNKS>
        <<<tiles, BLOCK, 0, s>>>(ps, out, n_ptr, n_max, tilesum, prefixed, total_out);
}

// What follows the count where the counts were made otherwise: the scan of the tile sums, where there are many (the kernels that use
// them add up the sums in front of a tile themselves otherwise: `prefixed`).
inline void compact_scan_sums(hipStream_t s, const int* n_ptr, int n_max, int* tilesum) {
    const int chunks = compact_chunks_for(n_max);
    if (compact_tiles(n_max > 0 ? n_max : 1, chunks) > COMPACT_MAX_SUMMED_TILES)
        scan_tilesums_kernel<<<1, SCAN_TILES_THREADS, 0, s>>>(tilesum, n_ptr, n_max, BLOCK * chunks);
}

// The first half of compact() on its own, for kernels that find their own places from the tile sums.
template <class PredCount>
inline void compact_count(hipStream_t s, PredCount pc, const int* n_ptr, int n_max, int* tilesum) {
    const int tiles = compact_tiles(n_max > 0 ? n_max : 1, compact_chunks_for(n_max));
    switch (compact_chunks_for(n_max)) {
        case 1: tile_count_kernel<PredCount, 1><<<tiles, BLOCK, 0, s>>>(pc, n_ptr, n_max, tilesum); break;
        case 4: tile_count_kernel<PredCount, 4><<<tiles, BLOCK, 0, s>>>(pc, n_ptr, n_max, tilesum); break;
        default: tile_count_kernel<PredCount, 16><<<tiles, BLOCK, 0, s>>>(pc, n_ptr, n_max, tilesum);
    }
    compact_scan_sums(s, n_ptr, n_max, tilesum);
}

// count pass may use a different functor (e.g. one that also stores the flag)
template <class PredCount, class PredScatter, class Out>
inline void compact(hipStream_t s, PredCount pc, PredScatter ps, Out out, const int* n_ptr, int n_max, int* tilesum,
                    int* total_out) {
    switch (compact_chunks_for(n_max)) {
        case 1: compact_impl<PredCount, PredScatter, Out, 1>(s, pc, ps, out, n_ptr, n_max, tilesum, total_out); break;
        case 4: compact_impl<PredCount, PredScatter, Out, 4>(s, pc, ps, out, n_ptr, n_max, tilesum, total_out); break;
        default: compact_impl<PredCount, PredScatter, Out, 16>(s, pc, ps, out, n_ptr, n_max, tilesum, total_out);
    }
}

}  // namespace prim
