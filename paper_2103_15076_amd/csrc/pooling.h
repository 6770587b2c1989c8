// pooling.h -- pooling and unpooling over the vertex clusters recorded by the
// decimation (Picasso paper, Sec. 3, paragraph "Pooling and unpooling").
//
// Features are fp32 [N, C] row-major.  A cluster's members are visited in
// ascending vertex order (CSR built by a stable sort of (cluster_id, vertex)),
// every sum is a left-to-right fp32 sum in that order and there are no fp
// atomics, so results do not depend on scheduling.  One lane owns four
// consecutive channels of one cluster (or of one vertex), so neighbouring
// lanes read neighbouring addresses of the same feature row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#pragma clang fp contract(off)

namespace pool {

constexpr int BLOCK = 256;
enum Mode { AVG = 0, MAX = 1, WEIGHTED = 2, SUM = 3 };

// Four consecutive channels of a feature row.  Loads and stores need 4-byte alignment only (the hardware takes
// 16-byte accesses at any such address), so every channel count and address goes this way.
struct Pack {
    float v[4];
};
struct __attribute__((packed, aligned(4))) PackedFloat4 {
    float v[4];
};
struct __attribute__((packed, aligned(4))) PackedInt4 {
    int v[4];
};

// How the rows of a call are addressed, the same for all its arrays whose rows the call knows (row_kind):
//   ROW_EVEN  the channel count is a multiple of 4, and every array's byte offsets (rows of up to `width` values) fit 32 bits and its row numbers
//             24: an address is one 24-bit multiply-add on top of a base in scalar registers;
//   ROW_TAIL  the same, with a last pack of `left` < 4 channels per row (the others read as 0);
//   ROW_ANY   any size (64-bit offsets) and channel count.
// (With 64-bit offsets everywhere the address arithmetic alone took as many vector instructions as the
// convolutions' sums.)
enum RowKind { ROW_EVEN, ROW_TAIL, ROW_ANY };
inline RowKind row_kind(int C, int width, long long max_rows) {
    const bool fits = max_rows < (1ll << 24) && 4ll * width < (1ll << 24) && 4ll * width * max_rows < (1ll << 32) && max_rows * 64 < (1ll << 32);
    return !fits ? ROW_ANY : (C % 4 == 0 ? ROW_EVEN : ROW_TAIL);
}

// p + i elements
template <int KIND, typename T>
__device__ __forceinline__ T* at(T* p, int i) {
    if constexpr (KIND == ROW_ANY) return p + (size_t)i;
    using Bytes = std::conditional_t<std::is_const_v<T>, const char, char>;
    return reinterpret_cast<T*>(reinterpret_cast<Bytes*>(p) + (uint32_t)i * (uint32_t)sizeof(T));
}
// channel c0 of row i
template <int KIND, typename T>
__device__ __forceinline__ T* row_at(T* p, int i, int C, int c0) {
    if constexpr (KIND == ROW_ANY) return p + ((size_t)i * C + c0);
    using Bytes = std::conditional_t<std::is_const_v<T>, const char, char>;
    return reinterpret_cast<T*>(reinterpret_cast<Bytes*>(p) + (__umul24((uint32_t)i, 4u * (uint32_t)C) + 4u * (uint32_t)c0));
}

template <int KIND>
__device__ __forceinline__ Pack load_row(const float* __restrict__ p, int left) {
    Pack r;
    if (KIND == ROW_EVEN || left >= 4) {
        const PackedFloat4 t = *reinterpret_cast<const PackedFloat4*>(p);
#pragma unroll
        for (int k = 0; k < 4; ++k) r.v[k] = t.v[k];
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) r.v[k] = k < left ? p[k] : 0.0f;
    }
    return r;
}

// The values are in registers from here on.  Used on a batch of loads in front of the code that takes them one
// by one under conditions: the compiler otherwise moves each load to its use, and none are in flight together.
__device__ __forceinline__ void arrived(float& a) { asm volatile("" : "+v"(a)); }
__device__ __forceinline__ void arrived(Pack& p) {
    asm volatile("" : "+v"(p.v[0]), "+v"(p.v[1]), "+v"(p.v[2]), "+v"(p.v[3]));
}

template <int KIND>
__device__ __forceinline__ void store_row(float* __restrict__ p, const Pack& r, int left) {
    if (KIND == ROW_EVEN || left >= 4) {
        PackedFloat4 t;
#pragma unroll
        for (int k = 0; k < 4; ++k) t.v[k] = r.v[k];
        *reinterpret_cast<PackedFloat4*>(p) = t;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < left) p[k] = r.v[k];
    }
}

// How a wave's lanes share out rows of C channels: Q = ceil(C / 4) packs per row, dealt to `parts` waves (blockIdx.y)
// of qc lanes per row, and 64 / qc rows side by side in a wave.  A lane finds its row with one multiplication
// instead of dividing a flat index by Q (a 64-bit division per lane took longer than the lane's loads).
struct RowMap {
    int Q, qc, rw, inv;  // rw = rows per wave and step; inv = ceil(65536 / qc)
};
inline int row_parts(const RowMap& m) { return (m.Q + m.qc - 1) / m.qc; }
// One wave per row where a wave's lanes hold at least two rows (Q <= 32): dealt to several waves, a row's parts end within lines, each
// wave fetches the row's indices again, and what that costs grows with the rows, while lanes without a pack cost next to nothing
// (fewer idle lanes by 2 or 3 parts against one: vertex2facet of 720 k facets, 24 channels 36 -> 19 us, 52: 68 -> 42, 100: 184 -> 136;
// max pooling of 360 k vertices, 100 channels 88 -> 53; the passes over the vertices' facets 97 -> 54, 145 -> 93, 268 -> 178).  From 33 packs
// on a wave holds one row, and up to half of its lanes may be idle: two parts where they use a fifth more of them (120 k facets, 132
// channels: facet2vertex 42 -> 32 us, vertex2facet's backward pass 42 -> 45, pooling the same).  Beyond 64, as few idle lanes as can be.
// one_wave: all lanes of a row in one wave, Q <= 64 (for sums across a row's lanes).
// lines: rows of whole 128-byte lines may go in parts of whole lines, which leave nothing between two waves: three parts of 96 or of 192
// channels (32, 64, 128, 160 and 256 go as they would anyhow).  In one part | in three, us: 192 channels, 115 k vertices, vertex2facet 64 | 54,
// facet2vertex (6 components) 101 | 64, average pooling 21.1 | 20.0, max pooling's backward pass 27.9 | 24.7; 400 k vertices 268 | 218, 305 | 266, 91 | 88, 129 | 107;
// 96 channels, 115 k vertices, facet2vertex 44 | 39, pooling 12.8 | 11.6.  Not in vertex2facet of 96 channels, either way, as long as the rows fit the
// Infinity Cache (beyond_cache): 120 k facets 14 | 20, but 720 k 119 | 106, 1.28 M 185 | 169; the backward pass 60 k vertices 29.2 | 32.0, 360 k 199 | 170 (192
// channels 30 k 29.8 | 28.6, 60 k 48.9 | 50.3, 122 k 107 | 100, 360 k 384 | 353).  Parts that end within lines stay slow beyond it as well (95 channels,
// 1.28 M facets: 334 | 526).  facet2vertex's backward pass, where a part more is a set of partial sums more: beyond the cache, 192 channels only (30 k vertices
// 31.1 | 34.9, 122 k 119 | 109, 360 k 365 | 346; 96 channels 177 | 182).
// odd: rows of no whole number of packs (their loads cross lines whichever way they are dealt) in the passes that walk the vertices' corners
// (facet2vertex, vertex2facet's backward pass), where a wave holds two of them or one: parts by the lanes at work, a tenth of them to be brought by
// each.  In one part | in two, 85 to 95 channels: facet2vertex 30 k vertices 21.2 | 18.9 us, 122 k 68 | 56, 360 k 204 | 208, vertex2facet's backward
// pass 28.0 | 25.9, 75 | 66, 301 | 230; in one | in three, 169 to 191 channels: 33.6 | 31.8, 141 | 112, 392 | 389 and 39.4 | 37.0, 167 | 148, 569 | 441.
inline RowMap row_map(int C, bool one_wave = false, bool lines = false, bool odd = false) {
    RowMap best{}, m;
    double best_use = -1.0;
    m.Q = (C + 3) / 4;
    const int least = (m.Q + 63) / 64;
    lines = lines && C % 32 == 0;
    odd = odd && C % 4 != 0 && m.Q > 21;
    const int most = one_wave || (m.Q <= 32 && !lines && !odd) ? least : least + 3;
    for (int parts = least; parts <= most && parts <= m.Q; ++parts) {
        m.qc = (m.Q + parts - 1) / parts;
        const bool whole = lines && m.qc % 8 == 0;
        if (m.Q <= 32 && parts > 1 && !whole && !odd) continue;
        // share of the lanes that a further part has to bring to work
        const double a_part = m.Q > 64 ? 0.04 : m.Q > 32 && !whole && !odd ? 0.2 : 0.1;
        m.rw = 64 / m.qc;
        m.inv = (65536 + m.qc - 1) / m.qc;
        const double use = (double)m.rw * m.Q / (64.0 * row_parts(m)) - a_part * (parts - least);  // lanes at work
        if (use > best_use) {
            best_use = use;
            best = m;
        }
    }
    return best;
}
inline bool beyond_cache(int C, long long rows) { return 4ll * C * rows > (256ll << 20); }
// workgroups so that every wave takes `steps` x rw rows
inline dim3 row_grid(const RowMap& m, int rows, int steps = 1) {
    const long long per_block = (long long)m.rw * steps * (BLOCK / 64);
    return dim3((unsigned)((rows + per_block - 1) / per_block), (unsigned)row_parts(m));
}

struct RowLane {
    int r, q;  // row within the wave's rows, channel pack of the row
    bool on;
};
__device__ __forceinline__ RowLane row_lane(const RowMap& m, int part) {
    const int u = (int)threadIdx.x & 63;
    RowLane l;
    l.r = (u * m.inv) >> 16;  // u / qc (exact for u, qc <= 64)
    l.q = u - l.r * m.qc + part * m.qc;
    l.on = l.r < m.rw && l.q < m.Q;
    return l;
}
// first of the wave's rows, one step per wave
__device__ __forceinline__ int wave_row(const RowMap& m, int block) {
    return (block * (BLOCK / 64) + ((int)threadIdx.x >> 6)) * m.rw;
}

// y[c] = pooled feature of cluster c.  MAX also writes the first member that attains the maximum.
template <int MODE, int KIND>
__global__ __launch_bounds__(BLOCK) void pool_forward_kernel(const float* __restrict__ x, int C,
                                                             const int* __restrict__ off,
                                                             const int* __restrict__ mem, int n_out,
                                                             const float* __restrict__ w, float* __restrict__ y,
                                                             int* __restrict__ argmax, RowMap map) {
    const RowLane l = row_lane(map, blockIdx.y);
    const int c = wave_row(map, blockIdx.x) + l.r;
    if (!l.on || c >= n_out) return;
    const int c0 = 4 * l.q, left = C - c0;
    const int s = *at<KIND>(off, c), e = *at<KIND>(off, c + 1);
    Pack acc;
    int arg[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        acc.v[k] = 0.0f;
        arg[k] = -1;
    }
    float wsum = 0.0f;
    for (int m = s; m < e; ++m) {
        const int v = *at<KIND>(mem, m);
        const Pack xv = load_row<KIND>(row_at<KIND>(x, v, C, c0), left);
        if (MODE == MAX) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (m == s || xv.v[k] > acc.v[k]) {
                    acc.v[k] = xv.v[k];
                    arg[k] = v;
                }
        } else if (MODE == WEIGHTED) {
            const float wv = *at<KIND>(w, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc.v[k] = acc.v[k] + wv * xv.v[k];
            wsum = wsum + wv;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) acc.v[k] = acc.v[k] + xv.v[k];
        }
    }
    if (MODE == AVG) {
        const float n = (float)(e - s);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc.v[k] = (e > s) ? acc.v[k] / n : 0.0f;
    }
    if (MODE == WEIGHTED) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc.v[k] = (wsum != 0.0f) ? acc.v[k] / wsum : 0.0f;
    }
    store_row<KIND>(row_at<KIND>(y, c, C, c0), acc, left);
    if (MODE == MAX && argmax) {
        int* a = row_at<KIND>(argmax, c, C, c0);
        if (KIND == ROW_EVEN || left >= 4) {
            *reinterpret_cast<PackedInt4*>(a) = PackedInt4{{arg[0], arg[1], arg[2], arg[3]}};
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < left) a[k] = arg[k];
        }
    }
}

// gx[v] = adjoint of the pooling applied to gy, for the features (weights are constants); zeros for a vertex in no cluster (id -1)
template <int MODE, int KIND>
__global__ __launch_bounds__(BLOCK) void pool_backward_kernel(const float* __restrict__ gy, int n_in, int C,
                                                              const int* __restrict__ cid,
                                                              const int* __restrict__ off,
                                                              const int* __restrict__ mem,
                                                              const float* __restrict__ w,
                                                              const int* __restrict__ argmax,
                                                              float* __restrict__ gx, RowMap map) {
    const RowLane l = row_lane(map, blockIdx.y);
    const int v = wave_row(map, blockIdx.x) + l.r;
    if (!l.on || v >= n_in) return;
    const int c0 = 4 * l.q, left = C - c0;
    const int c = *at<KIND>(cid, v);
    if (c < 0) {
        store_row<KIND>(row_at<KIND>(gx, v, C, c0), Pack{}, left);
        return;
    }
    Pack g = load_row<KIND>(row_at<KIND>(gy, c, C, c0), left);
    if (MODE == AVG) {
        const float n = (float)(off[c + 1] - off[c]);
#pragma unroll
        for (int k = 0; k < 4; ++k) g.v[k] = g.v[k] / n;
    } else if (MODE == MAX) {
        const int* a = row_at<KIND>(argmax, c, C, c0);
        PackedInt4 arg;
        if (KIND == ROW_EVEN || left >= 4) {
            arg = *reinterpret_cast<const PackedInt4*>(a);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) arg.v[k] = k < left ? a[k] : v;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (arg.v[k] != v) g.v[k] = 0.0f;
    } else if (MODE == WEIGHTED) {
        float wsum = 0.0f;
        for (int m = off[c]; m < off[c + 1]; ++m) wsum = wsum + w[mem[m]];
        const float wv = w[v];
#pragma unroll
        for (int k = 0; k < 4; ++k) g.v[k] = (wsum != 0.0f) ? (g.v[k] * wv) / wsum : 0.0f;
    }
    store_row<KIND>(row_at<KIND>(gx, v, C, c0), g, left);
}

// Unpooling: every vertex takes its cluster's feature (zeros where its cluster was dropped, id -1).  KIND is that of x alone: how many rows y has the call does not know,
// so those are addressed with 64 bits (one multiplication more per lane).
template <int KIND>
__global__ __launch_bounds__(BLOCK) void unpool_forward_kernel(const float* __restrict__ y, int n_in, int C,
                                                               const int* __restrict__ cid, float* __restrict__ x,
                                                               RowMap map) {
    const RowLane l = row_lane(map, blockIdx.y);
    const int v = wave_row(map, blockIdx.x) + l.r;
    if (!l.on || v >= n_in) return;
    const int c0 = 4 * l.q, left = C - c0, c = *at<KIND>(cid, v);
    store_row<KIND>(row_at<KIND>(x, v, C, c0), c >= 0 ? load_row<KIND>(row_at<ROW_ANY>(y, c, C, c0), left) : Pack{}, left);
}

// The two per-input-vertex tensors of Alg. 2's output list from cluster_id: first[c] = smallest
// member of cluster c (first pass, atomicMin: the result does not depend on order), then
// replace[v] = first[cluster_id[v]] and mapping[v] = cluster_id[v] for that member, -1 otherwise.
__global__ __launch_bounds__(BLOCK) void cluster_first_kernel(const int* __restrict__ cid, int n_in, int n_out,
                                                              int* __restrict__ first, int* __restrict__ err) {
    const int v = blockIdx.x * BLOCK + threadIdx.x;
    if (v >= n_in) return;
    const int c = cid[v];
    if (c == -1) return;  // (the vertex's cluster was dropped: nothing represents it)
    if (c < 0 || c >= n_out) {
        atomicOr(err, 1);
        return;
    }
    atomicMin(&first[c], v);
}

__global__ __launch_bounds__(BLOCK) void replace_mapping_kernel(const int* __restrict__ cid, int n_in, int n_out,
                                                                const int* __restrict__ first,
                                                                int* __restrict__ replace, int* __restrict__ mapping) {
    const int v = blockIdx.x * BLOCK + threadIdx.x;
    if (v >= n_in) return;
    const int c = cid[v];
    if (c < -1 || c >= n_out) return;  // (flagged by the first pass; the call reports it)
    const int r = c >= 0 ? first[c] : -1;
    replace[v] = r;
    mapping[v] = (c >= 0 && r == v) ? c : -1;
}

// The two kernels in front of and behind cluster_first_kernel when the table of first members is the
// library's static array (picasso_replace_mapping_static): the fill, which also clears the flag, and
// replace_mapping_kernel's work plus the status word for the caller.
__global__ __launch_bounds__(BLOCK) void static_begin_kernel(int* __restrict__ first, int n_out, int* __restrict__ flag) {
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < n_out) first[i] = 0x7FFFFFFF;
    if (i == 0) *flag = 0;
}

__global__ __launch_bounds__(BLOCK) void replace_mapping_status_kernel(const int* __restrict__ cid, int n_in, int n_out,
                                                                       const int* __restrict__ first,
                                                                       const int* __restrict__ flag,
                                                                       int* __restrict__ replace, int* __restrict__ mapping,
                                                                       int* __restrict__ status, int ok, int bad) {
    const int v = blockIdx.x * BLOCK + threadIdx.x;
    if (v == 0) *status = (*flag != 0) ? bad : ok;
    if (v >= n_in) return;
    const int c = cid[v];
    if (c < -1 || c >= n_out) return;
    const int r = c >= 0 ? first[c] : -1;
    replace[v] = r;
    mapping[v] = (c >= 0 && r == v) ? c : -1;
}

inline int grid_for(long long n) { return (int)((n + BLOCK - 1) / BLOCK > 0 ? (n + BLOCK - 1) / BLOCK : 1); }

template <int KIND>
inline void launch_pool_forward(hipStream_t s, int mode, const float* x, int C, const int* off, const int* mem,
                                int n_out, const float* w, float* y, int* argmax) {
    const RowMap m = row_map(C, false, true);
    const dim3 g = row_grid(m, n_out);
    switch (mode) {
        case AVG: pool_forward_kernel<AVG, KIND><<<g, BLOCK, 0, s>>>(x, C, off, mem, n_out, w, y, argmax, m); break;
        case MAX: pool_forward_kernel<MAX, KIND><<<g, BLOCK, 0, s>>>(x, C, off, mem, n_out, w, y, argmax, m); break;
        case WEIGHTED: pool_forward_kernel<WEIGHTED, KIND><<<g, BLOCK, 0, s>>>(x, C, off, mem, n_out, w, y, argmax, m); break;
        default: pool_forward_kernel<SUM, KIND><<<g, BLOCK, 0, s>>>(x, C, off, mem, n_out, w, y, argmax, m); break;
    }
}

template <int KIND>
inline void launch_pool_backward(hipStream_t s, int mode, const float* gy, int n_in, int C, const int* cid,
                                 const int* off, const int* mem, const float* w, const int* argmax, float* gx) {
    const RowMap m = row_map(C, false, true);
    const dim3 g = row_grid(m, n_in);
    switch (mode) {
        case AVG: pool_backward_kernel<AVG, KIND><<<g, BLOCK, 0, s>>>(gy, n_in, C, cid, off, mem, w, argmax, gx, m); break;
        case MAX: pool_backward_kernel<MAX, KIND><<<g, BLOCK, 0, s>>>(gy, n_in, C, cid, off, mem, w, argmax, gx, m); break;
        case WEIGHTED: pool_backward_kernel<WEIGHTED, KIND><<<g, BLOCK, 0, s>>>(gy, n_in, C, cid, off, mem, w, argmax, gx, m); break;
        default: pool_backward_kernel<SUM, KIND><<<g, BLOCK, 0, s>>>(gy, n_in, C, cid, off, mem, w, argmax, gx, m); break;
    }
}

}  // namespace pool
