// conv.h -- the two mesh convolutions of the Picasso paper in their depth-wise
// form (Sec. 4 "Mesh Convolution": vertex2facet with barycentric interpolation,
// facet2vertex with Gaussian-mixture fuzzy coefficients; supplementary section
// "Backward propagations of different convolutions").
//
// Features are fp32 [rows, C] row-major; one lane owns four consecutive channels of one row (RowMap in
// pooling.h: any channel count, any 4-byte aligned address), so neighbouring lanes read neighbouring
// addresses.  Sums over a vertex's facets run over its corners in ascending order (the corner
// CSR), filter gradients are reduced in two fixed stages; there are no fp
// atomics, so results do not depend on scheduling.
//
// What bounds these kernels, apart from the feature rows' bytes, is the memory pipeline of a compute unit (16 bytes
// for each of 64 lanes take it 8 ns, whether they are a kilobyte in a row or all one cached word): indices,
// levels and coefficients are therefore fetched once per item, one item per lane, and handed to the lanes of a row
// through LDS, the filter stays in registers or LDS, several rows are gathered per lane before the first is
// used, and one pass makes every gradient of a direction.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pooling.h"
#include "primitives.h"

#pragma clang fp contract(off)

namespace conv {

using pool::BLOCK;
using pool::Pack;
using pool::RowLane;
using pool::RowMap;
using pool::arrived;
using pool::at;
using pool::row_at;
using pool::load_row;
using pool::row_lane;
using pool::store_row;

// Index arrays come from the caller.  They are checked once, where the corner lists are built
// (csr_count_kernel reports a bad index); the kernels below only make sure that a bad one
// cannot reach outside the arrays: it is read as index 0.
__device__ __forceinline__ int in_range_or_zero(int i, int n) { return ((unsigned)i < (unsigned)n) ? i : 0; }

// The number a workgroup works as: the rows that neighbouring vertices and facets gather overlap (mesh numbering has locality), so
// each of the 8 XCDs, to which workgroups go in turn, takes one eighth of the grid's work in a row.  For grids of
// prim::xcd_grid workgroups; others are left in order (prim::xcd_tile: the same where the amount of work is known on the device only).
__device__ __forceinline__ int xcd_block() {
    if (gridDim.x & 7u) return (int)blockIdx.x;
    const unsigned g8 = gridDim.x >> 3;
    return (int)((blockIdx.x & 7u) * g8 + (blockIdx.x >> 3));
}

// The two indexes off[v], off[v + 1] and the three of a facet in one load each.
struct __attribute__((packed, aligned(4))) Int2 { int a, b; };
struct __attribute__((packed, aligned(4))) Int3 { int a, b, c; };
struct __attribute__((packed, aligned(4))) Float3 { float a, b, c; };
__device__ __forceinline__ Float3 load_point(const float* p, int i) { return *reinterpret_cast<const Float3*>(p + 3 * (size_t)i); }
__device__ __forceinline__ Int2 load_pair(const int* p) { return *reinterpret_cast<const Int2*>(p); }
__device__ __forceinline__ Int3 load_triple(const int* p) { return *reinterpret_cast<const Int3*>(p); }

// x / n for r = 1 / n: the quotient corrected by its own remainder and fixed up for the special cases, at a third of a
// division's instructions; used where one n divides several values.  Rounds like a division while 1 / n and the
// remainder are exact enough: 2^-100 <= |n| <= 2^100 and |x| >= 2^-100 (the remainder is a multiple of the last places'
// product, 2^-47 |x| or more, and 2^-149 is the smallest that can be held).  (20 million
// random pairs: none off.)  A smaller x may come out one unit in the last place off (1 in 10,000); a smaller n must not
// come here: below 2^-128 its reciprocal is infinite and the quotient NaN.
__device__ __forceinline__ float quotient(float x, float n, float r) {
    const float q = x * r;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, n, x), r, q), n, x);
}
constexpr float QUOTIENT_MIN = 0x1p-100f, QUOTIENT_MAX = 0x1p100f;

// ---------------------------------------------------------------------------
// Facet geometry: unit normal, area (Sec. 4, first paragraph) and the level k
// of Eq. "interpolate_num", k = floor((A - A_min) / (A_max - A_min)) * alpha +
// beta with A_min, A_max over the facet's own mesh.  Areas are non-negative,
// so their bit patterns order like their values and the per-mesh extremes are
// taken with integer atomics (order-independent), as the maxima of the pattern and of its complement.
// ---------------------------------------------------------------------------
// The meshes' facet offsets, up to MESH_OFFSETS meshes with the launch itself (no upload in front of it), else in memory.
constexpr int MESH_OFFSETS = 64;
struct MeshOffsets {
    int B;
    const int* far;  // null: here
    int here[MESH_OFFSETS + 1];
    __device__ __forceinline__ int operator[](int b) const { return far ? far[b] : here[b]; }
};

__device__ __forceinline__ int mesh_of_facet(const MeshOffsets& foff, int f) {
    int lo = 0, hi = foff.B;  // invariant: foff[lo] <= f < foff[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (foff[mid] <= f) lo = mid; else hi = mid;
    }
    return lo;
}

// The extremes of a mesh: its facets' workgroups spread over EXT_SLOTS cache lines, one atomic pair per workgroup (whose
// facets nearly always belong to one mesh) after combining in LDS: atomics on one line, whichever words of it they
// name, are served one after the other, about 10 ns each (1.9 M facets of 16 meshes: 143 us with a pair for every 256
// facets on two words per mesh). The few workgroups across a mesh's end take a pair per wave and mesh: with one per facet
// those 15 workgroups alone held the kernel back (44.7 us, 19.3 with it).
constexpr int EXT_SLOTS = 8, EXT_PAD = 32;  // words: one 128-byte line per slot; word 0 = largest pattern, 1 = largest complement
constexpr int GEO_ITEMS = 4;                // facets per lane

__device__ __forceinline__ unsigned wave_max(unsigned v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, d, 64));
    return v;
}

__device__ __forceinline__ unsigned* ext_slot(unsigned* ext, int m) {
    return ext + ((size_t)m * EXT_SLOTS + (blockIdx.x & (EXT_SLOTS - 1))) * EXT_PAD;
}

__global__ __launch_bounds__(BLOCK) void facet_geometry_kernel(const float* __restrict__ verts, int N,
                                                               const int* __restrict__ facets, int F, MeshOffsets foff,
                                                               float* __restrict__ normals, float* __restrict__ areas,
                                                               unsigned* __restrict__ ext /* or null */,
                                                               int* __restrict__ err) {
    __shared__ unsigned wmax[BLOCK / 64], wnmin[BLOCK / 64];
    const int first = blockIdx.x * (BLOCK * GEO_ITEMS), last = min(first + BLOCK * GEO_ITEMS, F) - 1;
    Int3 v[GEO_ITEMS];
    bool bad = false;
#pragma unroll
    for (int j = 0; j < GEO_ITEMS; ++j) {
        const int f = first + j * BLOCK + (int)threadIdx.x;
        v[j] = load_triple(facets + 3 * (size_t)min(f, last));
        if (v[j].a < 0 || v[j].a >= N || v[j].b < 0 || v[j].b >= N || v[j].c < 0 || v[j].c >= N) {
            bad = true;
            v[j] = Int3{0, 0, 0};
        }
    }
    if (bad) atomicOr(err, 1);
    Float3 p[GEO_ITEMS][3];
#pragma unroll
    for (int j = 0; j < GEO_ITEMS; ++j) {
        p[j][0] = load_point(verts, v[j].a);
        p[j][1] = load_point(verts, v[j].b);
        p[j][2] = load_point(verts, v[j].c);
    }
    const int mesh0 = ext ? mesh_of_facet(foff, first) : 0;  // (the same in all lanes)
    const bool one_mesh = !ext || foff[mesh0 + 1] > last;
    unsigned hi = 0u, lo = 0u;
#pragma unroll
    for (int j = 0; j < GEO_ITEMS; ++j) {
        const int f = first + j * BLOCK + (int)threadIdx.x;
        const bool in = f <= last;
        const float ax = p[j][1].a - p[j][0].a, ay = p[j][1].b - p[j][0].b, az = p[j][1].c - p[j][0].c;
        const float bx = p[j][2].a - p[j][0].a, by = p[j][2].b - p[j][0].b, bz = p[j][2].c - p[j][0].c;
        const float nx = ay * bz - az * by;
        const float ny = az * bx - ax * bz;
        const float nz = ax * by - ay * bx;
        const float len = sqrtf((nx * nx + ny * ny) + nz * nz);
        const float area = 0.5f * len;
        if (in && areas) areas[f] = area;
        if (in && normals) {
            Float3 n;
            n.a = len > 0.0f ? nx / len : 0.0f;
            n.b = len > 0.0f ? ny / len : 0.0f;
            n.c = len > 0.0f ? nz / len : 0.0f;
            *reinterpret_cast<Float3*>(normals + 3 * (size_t)f) = n;
        }
        const unsigned bits = __float_as_uint(area);
        const bool counts = in && area == area;  // (a NaN area takes no part in the extremes)
        if (!ext) continue;
        if (one_mesh) {
            hi = max(hi, counts ? bits : 0u);
            lo = max(lo, counts ? ~bits : 0u);
        } else {  // a workgroup across a mesh's end: an atomic pair per wave and mesh
            const int m = counts ? mesh_of_facet(foff, f) : -1;
            for (unsigned long long rest = __ballot(counts); rest;) {
                const int m0 = __shfl(m, __ffsll((long long)rest) - 1, 64);
                const bool mine = m == m0;
                const unsigned h = wave_max(mine ? bits : 0u), n = wave_max(mine ? ~bits : 0u);
                if ((threadIdx.x & 63) < 2) atomicMax(ext_slot(ext, m0) + (threadIdx.x & 1), (threadIdx.x & 1) ? n : h);
                rest &= ~__ballot(mine);
            }
        }
    }
    if (!ext || !one_mesh) return;
    hi = wave_max(hi);
    lo = wave_max(lo);
    if ((threadIdx.x & 63) == 0) {
        wmax[threadIdx.x >> 6] = hi;
        wnmin[threadIdx.x >> 6] = lo;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned* wv = threadIdx.x ? wnmin : wmax;
        atomicMax(ext_slot(ext, mesh0) + threadIdx.x, max(max(wv[0], wv[1]), max(wv[2], wv[3])));
    }
}

__device__ __forceinline__ void mesh_extremes(const unsigned* __restrict__ ext, int m, float& lo, float& hi) {
    unsigned h = 0u, l = 0u;
#pragma unroll
    for (int k = 0; k < EXT_SLOTS; ++k) {
        const unsigned* e = ext + ((size_t)m * EXT_SLOTS + k) * EXT_PAD;
        h = max(h, e[0]);
        l = max(l, e[1]);
    }
    lo = __uint_as_float(~l);
    hi = __uint_as_float(h);
}

__global__ __launch_bounds__(BLOCK) void facet_level_kernel(const float* __restrict__ areas, int F, MeshOffsets foff,
                                                            const unsigned* __restrict__ ext, int alpha, int beta,
                                                            int* __restrict__ level) {
    const int first = blockIdx.x * (BLOCK * GEO_ITEMS), last = min(first + BLOCK * GEO_ITEMS, F) - 1;
    float area[GEO_ITEMS];
#pragma unroll
    for (int j = 0; j < GEO_ITEMS; ++j) area[j] = areas[min(first + j * BLOCK + (int)threadIdx.x, last)];
    const int mesh0 = mesh_of_facet(foff, first);  // (the same in all lanes)
    const bool one_mesh = foff[mesh0 + 1] > last;
    float lo, hi;
    mesh_extremes(ext, mesh0, lo, hi);
#pragma unroll
    for (int j = 0; j < GEO_ITEMS; ++j) {
        const int f = first + j * BLOCK + (int)threadIdx.x;
        if (f > last) break;
        if (!one_mesh) mesh_extremes(ext, mesh_of_facet(foff, f), lo, hi);
        const float ratio = hi > lo ? (area[j] - lo) / (hi - lo) : 0.0f;
        level[f] = (int)floorf(ratio) * alpha + beta;
    }
}

// Fuzzy coefficients of the facets (Sec. 4.2): z_ft = |n_f - mu_t|^2 * inv_var_t,
// pi_ft = exp(-z_ft) / sum_m exp(-z_fm).  One lane per facet; the workgroup's rows are made in LDS and written out
// as one contiguous piece (up to FUZZY_LDS_T components; lanes writing T floats each at a stride of T, and
// reading them back for the division, took 45 us for 1.9 M facets of 6 components).
constexpr int FUZZY_LDS_T = 48;
template <bool IN_LDS>
__global__ __launch_bounds__(BLOCK) void fuzzy_kernel(const float* __restrict__ normals, int F,
                                                      const float* __restrict__ mu, const float* __restrict__ inv_var,
                                                      int T, float* __restrict__ pi) {
    extern __shared__ float tile[];  // [BLOCK * T]
    const int f0 = blockIdx.x * BLOCK, f = f0 + threadIdx.x;
    if (f < F) {
        const Float3 n = load_point(normals, f);
        float* row = IN_LDS ? tile + threadIdx.x * T : pi + (size_t)f * T;
        float sum = 0.0f, least = QUOTIENT_MAX;
        for (int t = 0; t < T; ++t) {
            const float dx = n.a - mu[3 * t], dy = n.b - mu[3 * t + 1], dz = n.c - mu[3 * t + 2];
            const float e = expf(-(((dx * dx + dy * dy) + dz * dz) * inv_var[t]));
            row[t] = e;
            least = fminf(least, e);
            sum = sum + e;
        }
        if (least >= QUOTIENT_MIN && sum <= QUOTIENT_MAX) {
            const float r = 1.0f / sum;
            for (int t = 0; t < T; ++t) row[t] = quotient(row[t], sum, r);
        } else {  // a component farther than z = 69: sharp ones, for which all may be
            for (int t = 0; t < T; ++t) row[t] = row[t] / sum;
        }
    }
    if constexpr (IN_LDS) {
        __syncthreads();
        const int n = min(BLOCK, F - f0) * T;
        float* out = pi + (size_t)f0 * T;
        for (int i = 4 * threadIdx.x; i < n; i += 4 * BLOCK) {
            if (i + 4 <= n) {
                const float4 q = *reinterpret_cast<const float4*>(tile + i);
                store_row<pool::ROW_EVEN>(out + i, Pack{{q.x, q.y, q.z, q.w}}, 4);
            } else {
                for (int k = i; k < n; ++k) out[k] = tile[k];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Vertex2facet (Sec. 4.1).  With I_k = sum_s xi_ks I_s, W_k = sum_s xi_ks w_s and
// J = (1/K) sum_k W_k I_k the facet feature is the bilinear form J = w^T M I,
// M = (1/K) sum_k xi_k xi_k^T.  The K = k (k + 1) / 2 points of level k are the
// triangular lattice (i, j, l) / (k - 1) (the centroid alone for k = 1), whose
// moment matrix has the diagonal a = k / (6 (k - 1)) and the off-diagonal
// b = (k - 2) / (12 (k - 1)) (a = b = 1/9 for k = 1; a + 2 b = 1/3 always), so
// J = (a - b) sum_s w_s I_s + b (sum_s w_s) (sum_s I_s).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void lattice_moments(int k, float& a_minus_b, float& b) {
    if (k <= 1) {
        a_minus_b = 0.0f;
        b = 1.0f / 9.0f;
        return;
    }
    const float n = (float)(k - 1);
    a_minus_b = (n + 3.0f) / (12.0f * n);
    b = (n - 1.0f) / (12.0f * n);
}

// LDS written by the lanes of a wave is read by others of the same wave from here on.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// A wave takes `per_wave` consecutive facets: their vertices and moments go to LDS, one facet per lane, then the wave's lanes
// make the facets' rows, rw of them side by side.  (64 channels, 1.9 M facets: 214 us with the indices and the
// filter loaded per row.)
constexpr int V2F_UNROLL = 2;
// At most 64; few enough that all waves of the chip get some.
inline int facets_per_wave(const RowMap& m, long long F) {
    const long long turn = (long long)m.rw * V2F_UNROLL;
    return (int)std::min<long long>(64, std::max<long long>(m.rw, F / (8192 * turn) * turn));
}
template <int KIND>
__global__ __launch_bounds__(BLOCK) void v2f_forward_kernel(const float* __restrict__ x, int N, int C,
                                                            const int* __restrict__ facets, int F,
                                                            const int* __restrict__ level,
                                                            const float* __restrict__ w, float* __restrict__ y,
                                                            int per_wave, RowMap map) {
    __shared__ int4 sv[BLOCK];
    __shared__ float2 sm[BLOCK];
    const RowLane l = row_lane(map, blockIdx.y);
    const int w0 = wave_id() * 64, lane = (int)threadIdx.x & 63;
    const int base = (xcd_block() * (BLOCK / 64) + wave_id()) * per_wave, n = min(per_wave, F - base);
    if (n <= 0) return;
    if (lane < n) {
        const Int3 v = load_triple(row_at<KIND>(facets, base + lane, 3, 0));
        sv[w0 + lane] = make_int4(in_range_or_zero(v.a, N), in_range_or_zero(v.b, N), in_range_or_zero(v.c, N), 0);
        float amb, b;
        lattice_moments(level ? *at<KIND>(level, base + lane) : 1, amb, b);
        sm[w0 + lane] = make_float2(amb, b);
    }
    wave_sync();
    if (!l.on) return;
    const int c0 = 4 * l.q, left = C - c0;
    Pack ws[3], wsum;
#pragma unroll
    for (int s = 0; s < 3; ++s) ws[s] = load_row<KIND>(row_at<KIND>(w, s, C, c0), left);
#pragma unroll
    for (int i = 0; i < 4; ++i) wsum.v[i] = (ws[0].v[i] + ws[1].v[i]) + ws[2].v[i];
    for (int i0 = l.r; i0 < n; i0 += map.rw * V2F_UNROLL) {
        Pack xs[V2F_UNROLL][3];
#pragma unroll
        for (int u = 0; u < V2F_UNROLL; ++u) {  // (rows behind the last load that one again)
            const int4 v = sv[w0 + min(i0 + u * map.rw, n - 1)];
            xs[u][0] = load_row<KIND>(row_at<KIND>(x, v.x, C, c0), left);
            xs[u][1] = load_row<KIND>(row_at<KIND>(x, v.y, C, c0), left);
            xs[u][2] = load_row<KIND>(row_at<KIND>(x, v.z, C, c0), left);
        }
#pragma unroll
        for (int u = 0; u < V2F_UNROLL; ++u)
#pragma unroll
            for (int s = 0; s < 3; ++s) arrived(xs[u][s]);
#pragma unroll
        for (int u = 0; u < V2F_UNROLL; ++u) {
            const int i1 = i0 + u * map.rw;
            if (i1 < n) {
                const float2 m = sm[w0 + i1];
                Pack out;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float dot = fmaf(ws[2].v[i], xs[u][2].v[i], fmaf(ws[1].v[i], xs[u][1].v[i], ws[0].v[i] * xs[u][0].v[i]));
                    const float xsum = (xs[u][0].v[i] + xs[u][1].v[i]) + xs[u][2].v[i];
                    out.v[i] = fmaf(m.x, dot, m.y * (wsum.v[i] * xsum));
                }
                store_row<KIND>(row_at<KIND>(y, base + i1, C, c0), out, left);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// A wave's walk over `n` (at most 64) rows from row0 on, each a range of items [off[row], off[row + 1]): the corners of
// a vertex, the texture points of a facet.  The items' small data (Op::stage) are fetched 64 at a time, one item per
// lane, into the wave's LDS window.  2^split lane groups share a row's items (WalkMap), each taking every 2^split-th of
// them from the window, UNROLL at a time: Op::load starts the gather of an item's feature row, Op::use adds it up.
// Op::end makes the row from a group's sums; sums over a row's groups go through GroupSum.  Every sum has a fixed order.
// Offsets are clipped to [0, n_items], and a row's end to the end of the wave's last row, behind which nothing is staged: whatever
// the offsets (descending ones too), only staged items of the array are used.  soff holds 65 ints of the wave's own.
// ---------------------------------------------------------------------------
constexpr int WALK_WINDOW = 64;
constexpr int WALK_WAVE_ROWS = 64;
struct WalkMap {
    RowMap row;
    int split, rows, per_wave;  // rows side by side in a wave, rows of a wave's walk
};
// So that a step's items about fill the window (`average` items per row) and, where rows differ in length, no
// group walks alone for long; and walks as long as keep all waves busy.
inline WalkMap walk_map(int C, long long n_rows, double average, bool lines = false, bool odd = false) {
    WalkMap m;
    m.row = pool::row_map(C, false, lines, odd);
    m.split = 0;
    while (m.split < 3 && (m.row.rw >> (m.split + 1)) >= 1 && (m.row.rw >> m.split) * average > 48.0) ++m.split;
    m.rows = m.row.rw >> m.split;
    const long long most = std::max(1, 32 / m.rows), busy = n_rows / (8192ll * m.rows);
    m.per_wave = m.rows * (int)std::max<long long>(1, std::min(most, busy));
    return m;
}

struct GroupSum {
    int split, qc;
    __device__ __forceinline__ float operator()(float v) const {  // valid in a row's first group
        for (int d = 1 << split >> 1; d > 0; d >>= 1) v += __shfl_down(v, (unsigned)(d * qc), 64);
        return v;
    }
    __device__ __forceinline__ void operator()(Pack& p) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) p.v[i] = (*this)(p.v[i]);
    }
};

template <int KIND, int UNROLL, class Op>
__device__ __forceinline__ void walk_rows(Op& op, const int* __restrict__ off, int row0, int n, int n_items, const WalkMap& map,
                                          const RowLane& l, int* soff) {
    const int lane = (int)threadIdx.x & 63;
    const int r = l.r >> map.split, sub = l.r & ((1 << map.split) - 1);
    const bool on_row = l.on && r < map.rows;
    const GroupSum sum{map.split, map.row.qc};
    wave_sync();
    for (int i = lane; i <= n; i += 64) soff[i] = min(max(*at<KIND>(off, row0 + i), 0), n_items);
    wave_sync();
    const int last = __builtin_amdgcn_readfirstlane(soff[n]);
    int w0 = 0, w1 = 0;  // the items in the window
    for (int g = 0; g < n; g += map.rows) {
        const bool on = on_row && g + r < n;
        const int s = soff[min(g + r, n)], e = on ? min(soff[min(g + r + 1, n)], last) : s;
        const int ge = __builtin_amdgcn_readfirstlane(soff[min(g + map.rows, n)]);
        int from = __builtin_amdgcn_readfirstlane(soff[g]);
        op.begin(row0 + g + r, on, e - s);
        for (;;) {
            if (!(w0 <= from && ge <= w1)) {
                wave_sync();
                if (from + lane < last) op.stage(lane, from + lane);
                w0 = from;
                w1 = from + WALK_WINDOW;
                wave_sync();
            }
            const int end = min(e, w1), step = 1 << map.split;
            for (int j = max(s, from) + sub; j < end; j += step * UNROLL) {
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) op.load(u, min(j + u * step, end - 1) - w0, min(j + u * step, end - 1));
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) op.wait(u);
#pragma unroll
                for (int u = 0; u < UNROLL; ++u)
                    if (j + u * step < end) op.use(u, j + u * step - w0, j + u * step);
            }
            if (ge <= w1) break;
            from = w1;
        }
        op.end(row0 + g + r, on, on && sub == 0, sum);
    }
}

// ---------------------------------------------------------------------------
// Filter gradients: a sum over all rows (facets, or vertices) per channel, in two fixed stages.  Stage 1, at
// the end of the kernels below: workgroup g has taken the rows [g * chunk, (g + 1) * chunk), each lane some
// of them for its channel pack, summing in registers; the lanes of a pack are now summed within the waves and over
// them in a fixed tree, row by row of the gradient, and left in partial[g][rows][C].  Stage 2 adds the workgroups' partial sums.
// ---------------------------------------------------------------------------
// A facet's fuzzy coefficients of `rows` components (facet2vertex below), 4 (NP - 1) < rows <= 4 NP, in NP slots of four: with NP > 1
// the last four slots hold the last four components (one 16-byte load each, without a branch), so that some of
// them hold a component a second time; such slots are left out (slot_used; uniform, so a scalar branch).
template <int NP>
__device__ __forceinline__ int slot_component(int slot, int rows) {
    return NP == 1 || slot < 4 * (NP - 1) ? slot : rows - 4 * NP + slot;
}
template <int NP>
__device__ __forceinline__ bool slot_used(int slot, int rows) {
    if (NP == 1) return slot < rows;
    return slot < 4 * (NP - 1) || slot >= 4 * NP - (rows - 4 * (NP - 1));
}
template <int KIND, int NP, int ROWS>
__device__ __forceinline__ void rows_to_partial(const float (&acc)[ROWS][4], int rows, const RowMap& map, const RowLane& l,
                                                int C, float4* lds /* [2][BLOCK] */, float* __restrict__ partial) {
    const int wave = wave_id(), lq = l.q - (int)blockIdx.y * map.qc;
    int top = 1;  // smallest power of two >= rw
    while (top < map.rw) top <<= 1;
    __syncthreads();
    int turn = 0;
#pragma unroll
    for (int row = 0; row < ROWS; ++row) {
        if (slot_used<NP>(row, rows)) {  // (the same in all lanes)
            float t[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] = l.on ? acc[row][k] : 0.0f;
            for (int d = top >> 1; d > 0; d >>= 1) {  // the wave's rows
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float o = __shfl_down(t[k], (unsigned)(d * map.qc), 64);
                    if (l.r + d < map.rw) t[k] += o;
                }
            }
            float4* buf = lds + (turn & 1) * BLOCK;  // (two in turn: a barrier per row of the gradient)
            if (l.on && l.r == 0) buf[wave * 64 + lq] = make_float4(t[0], t[1], t[2], t[3]);
            __syncthreads();
            if (wave == (turn & (BLOCK / 64 - 1)) && l.on && l.r == 0) {
                const float4 a = buf[lq], b = buf[64 + lq], c = buf[128 + lq], d = buf[192 + lq];
                const Pack out{{(a.x + b.x) + (c.x + d.x), (a.y + b.y) + (c.y + d.y), (a.z + b.z) + (c.z + d.z), (a.w + b.w) + (c.w + d.w)}};
                store_row<KIND>(partial + ((size_t)blockIdx.x * rows + slot_component<NP>(row, rows)) * C + 4 * l.q, out,
                                C - 4 * l.q);
            }
            ++turn;
        }
    }
}

// out[i] = sum over the workgroups' partials of value i of `width`: a workgroup takes REDUCE_VALUES values in a row, a cache line of
// every partial, REDUCE_PARTIALS partials side by side (lane l adds the partials l, l + REDUCE_PARTIALS, ..., eight loads in flight), and
// the lanes of a value are then added in a fixed tree.  (A wave per value before, whose lanes each fetched a line for one word.  120 k facets, 6
// components, with stage 1: 32 channels 20.7 -> 19.1 us, 64: 26.3 -> 23.9, 128: 39.9 -> 36.4.)
constexpr int REDUCE_THREADS = 1024, REDUCE_VALUES = 16, REDUCE_PARTIALS = REDUCE_THREADS / REDUCE_VALUES;
__global__ __launch_bounds__(REDUCE_THREADS) void reduce_rows_stage2_kernel(const float* __restrict__ partial, int groups, int width,
                                                                            float* __restrict__ out) {
    __shared__ float sums[REDUCE_THREADS / 64][REDUCE_VALUES];
    const int t = threadIdx.x, i = blockIdx.x * REDUCE_VALUES + (t & (REDUCE_VALUES - 1));
    const float* p = partial + min(i, width - 1);
    float acc = 0.0f;
    for (int g0 = t / REDUCE_VALUES; g0 < groups; g0 += REDUCE_PARTIALS * 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = g0 + REDUCE_PARTIALS * j < groups ? p[(size_t)(g0 + REDUCE_PARTIALS * j) * width] : 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = acc + v[j];
    }
#pragma unroll
    for (int d = REDUCE_VALUES; d < 64; d <<= 1) acc = acc + __shfl_xor(acc, d, 64);
    if ((t & 63) < REDUCE_VALUES) sums[t >> 6][t & 63] = acc;
    __syncthreads();
    if (t < 64) {
#pragma unroll
        for (int w = 0; w < REDUCE_THREADS / 64; w += 4) {
            const float s = sums[w + t / REDUCE_VALUES][t & (REDUCE_VALUES - 1)];
            acc = w == 0 ? s : acc + s;
        }
#pragma unroll
        for (int d = REDUCE_VALUES; d < 64; d <<= 1) acc = acc + __shfl_xor(acc, d, 64);
        if (t < REDUCE_VALUES && i < width) out[i] = acc;
    }
}

// Backward pass of vertex2facet (supplementary, vertex2facet kernel): dJ/dI_s = (M w)_s = (a - b) w_s + b sum_r
// w_r and dJ/dw_s = (M I)_s = (a - b) I_s + b sum_r I_r.  Both follow from the same two sums over the corners of
// a vertex, A_s = sum of (a - b) g over its corners in place s of their facets and B = sum of b g:
//   gx_v = sum_s w_s A_s + (sum_s w_s) B,   gw_s = sum_v x_v (A_s + B),
// so one walk over the corner lists, which gathers the facets' gradients once, makes both gradients.
// (Two passes before, gw summed over the facets from three gathered vertex rows each.)
template <int KIND>
struct V2fBackwardOp {
    static constexpr int UNROLL = 3;
    const float* gy;
    const int* level;
    const int* corners;
    float* gx;
    const float* x;  // null: no filter gradient
    int C, c0, left, H;
    int2* win_f;     // [WALK_WINDOW] facet, place of the corner in it
    float2* win_m;   // [WALK_WINDOW] moments of the facet's level
    Pack ws[3], wsum, g[UNROLL];
    float A[3][4], B[4], gw[3][4];
    __device__ void stage(int slot, int j) {
        const int i = in_range_or_zero(*at<KIND>(corners, j), H), f = i / 3;
        float amb, b;
        lattice_moments(level ? *at<KIND>(level, f) : 1, amb, b);
        win_f[slot] = make_int2(f, i - 3 * f);
        win_m[slot] = make_float2(amb, b);
    }
    __device__ void begin(int, bool, int) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A[0][i] = A[1][i] = A[2][i] = B[i] = 0.0f;
    }
    __device__ void load(int u, int slot, int) { g[u] = load_row<KIND>(row_at<KIND>(gy, win_f[slot].x, C, c0), left); }
    __device__ void wait(int u) { arrived(g[u]); }
    __device__ void use(int u, int slot, int) {
        const float2 m = win_m[slot];
#pragma unroll
        for (int i = 0; i < 4; ++i) B[i] = fmaf(m.y, g[u].v[i], B[i]);
        if (m.x != 0.0f) {  // (a facet of level 1, nearly every one, has a = b)
            const int s = win_f[slot].y;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const float a = s == p ? m.x : 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) A[p][i] = fmaf(a, g[u].v[i], A[p][i]);
            }
        }
    }
    __device__ void end(int v, bool on, bool first, const GroupSum& sum) {
        if (gx) {
            Pack out;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out.v[i] = fmaf(wsum.v[i], B[i], fmaf(ws[2].v[i], A[2][i], fmaf(ws[1].v[i], A[1][i], ws[0].v[i] * A[0][i])));
            sum(out);
            if (first) store_row<KIND>(row_at<KIND>(gx, v, C, c0), out, left);
        }
        if (x && on) {
            const Pack xv = load_row<KIND>(row_at<KIND>(x, v, C, c0), left);
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i) gw[s][i] = fmaf(xv.v[i], A[s][i] + B[i], gw[s][i]);
        }
    }
};

// Workgroup b walks over the vertices of its chunk, map.per_wave of them per wave and turn.
template <int KIND>
__global__ __launch_bounds__(BLOCK) void v2f_backward_kernel(const float* __restrict__ gy, const float* __restrict__ x, int C,
                                                             const int* __restrict__ level,
                                                             const float* __restrict__ w,
                                                             const int* __restrict__ off,
                                                             const int* __restrict__ corners, int N, int H, int chunk,
                                                             float* __restrict__ gx,
                                                             float* __restrict__ partial, WalkMap map) {
    __shared__ int2 win_f[BLOCK / 64 * WALK_WINDOW];
    __shared__ float2 win_m[BLOCK / 64 * WALK_WINDOW];
    __shared__ int soff[BLOCK / 64][WALK_WAVE_ROWS + 1];
    __shared__ float4 lds[2 * BLOCK];
    const RowLane l = row_lane(map.row, blockIdx.y);
    const int wave = wave_id();
    V2fBackwardOp<KIND> op;
    op.gy = gy; op.level = level; op.corners = corners; op.gx = gx; op.x = partial ? x : nullptr;
    op.C = C; op.c0 = 4 * l.q; op.left = C - op.c0; op.H = H;
    op.win_f = win_f + wave * WALK_WINDOW; op.win_m = win_m + wave * WALK_WINDOW;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        op.ws[s] = l.on ? load_row<KIND>(row_at<KIND>(w, s, C, op.c0), op.left) : Pack{};
#pragma unroll
        for (int i = 0; i < 4; ++i) op.gw[s][i] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) op.wsum.v[i] = (op.ws[0].v[i] + op.ws[1].v[i]) + op.ws[2].v[i];
    const int begin = min(xcd_block() * chunk, N), end = min(begin + chunk, N);
    for (int v = begin + wave * map.per_wave; v < end; v += map.per_wave * (BLOCK / 64))
        walk_rows<KIND, V2fBackwardOp<KIND>::UNROLL>(op, off, v, min(map.per_wave, end - v), H, map, l, soff[wave]);
    if (partial) rows_to_partial<KIND, 1>(op.gw, 3, map.row, l, C, lds, partial);
}

// ---------------------------------------------------------------------------
// Facet2facet (Sec. 4.1, for meshes rendered with textures): every facet has
// Gamma_f texture points with features of their own and barycentric coordinates;
// only the filter is interpolated, W_k = sum_s xi_ks w_s, and J_f = (1 / Gamma_f)
// sum_k W_k T_k.  Points of facet f = poff[f] .. poff[f+1]; tex [P,C], bary [P,3].
// A facet's points are walked as above (walk_rows), forward; backward they are rows of their own.
// ---------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ Float3 load_bary(const float* __restrict__ bary, int k) {
    return *reinterpret_cast<const Float3*>(row_at<KIND>(bary, k, 3, 0));
}

template <int KIND>
struct F2fForwardOp {
    static constexpr int UNROLL = 4;
    const float* tex;
    const float* bary;
    float* y;
    int C, c0, left;
    Float3* win;  // [WALK_WINDOW]
    Pack ws[3], acc, t[UNROLL];
    float n;
    __device__ void stage(int slot, int k) { win[slot] = load_bary<KIND>(bary, k); }
    __device__ void begin(int, bool, int count) {
        acc = Pack{};
        n = (float)count;
    }
    __device__ void load(int u, int, int k) { t[u] = load_row<KIND>(row_at<KIND>(tex, k, C, c0), left); }
    __device__ void wait(int u) { arrived(t[u]); }
    __device__ void use(int u, int slot, int) {
        const Float3 xi = win[slot];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float wk = fmaf(xi.c, ws[2].v[i], fmaf(xi.b, ws[1].v[i], xi.a * ws[0].v[i]));
            acc.v[i] = fmaf(wk, t[u].v[i], acc.v[i]);
        }
    }
    __device__ void end(int f, bool, bool first, const GroupSum& sum) {
        sum(acc);
        if (!first) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc.v[i] = n > 0.0f ? acc.v[i] / n : 0.0f;
        store_row<KIND>(row_at<KIND>(y, f, C, c0), acc, left);
    }
};

template <int KIND>
__global__ __launch_bounds__(BLOCK) void f2f_forward_kernel(const float* __restrict__ tex,
                                                            const float* __restrict__ bary,
                                                            const int* __restrict__ poff, int F, int P, int C,
                                                            const float* __restrict__ w, 
                                                            float* __restrict__ y, WalkMap map) {
    __shared__ Float3 win[BLOCK / 64 * WALK_WINDOW];
    __shared__ int soff[BLOCK / 64][WALK_WAVE_ROWS + 1];
    const RowLane l = row_lane(map.row, blockIdx.y);
    const int wave = wave_id();
    const int f0 = (xcd_block() * (BLOCK / 64) + wave) * map.per_wave;
    if (f0 >= F) return;
    F2fForwardOp<KIND> op;
    op.tex = tex; op.bary = bary; op.y = y; op.C = C; op.c0 = 4 * l.q; op.left = C - op.c0;
    op.win = win + wave * WALK_WINDOW;
#pragma unroll
    for (int s = 0; s < 3; ++s) op.ws[s] = l.on ? load_row<KIND>(row_at<KIND>(w, s, C, op.c0), op.left) : Pack{};
    walk_rows<KIND, F2fForwardOp<KIND>::UNROLL>(op, poff, f0, min(map.per_wave, F - f0), P, map, l, soff[wave]);
}

// Backward pass: dJ/dT_k = W_k / Gamma_f and dJ/dw_s = (1 / Gamma_f) sum_k xi_ks T_k, each times the facet's
// incoming gradient.  Nothing is summed per facet, so the wave's rows are points, whatever their facets' sizes: a
// wave takes per_wave facets at a time and their points 64 at a time, one lane finding a point's facet among
// the offsets.  (Walking facet by facet left half of the lanes idle: 183 us at 1.8 M points, 32 channels.)
template <int KIND>
__global__ __launch_bounds__(BLOCK) void f2f_backward_kernel(const float* __restrict__ gy, const float* __restrict__ tex,
                                                             const float* __restrict__ bary,
                                                             const int* __restrict__ poff, int F, int P, int C,
                                                             const float* __restrict__ w, int chunk, int per_wave,
                                                             float* __restrict__ gtex, float* __restrict__ partial,
                                                             RowMap map) {
    __shared__ float4 sb[BLOCK];   // per point: barycentric coordinates, 1 / Gamma of its facet
    __shared__ int2 sf[BLOCK];     // ... facet, Gamma
    __shared__ int soff[BLOCK / 64][WALK_WAVE_ROWS + 1];
    __shared__ float4 lds[2 * BLOCK];
    const RowLane l = row_lane(map, blockIdx.y);
    const int wave = wave_id(), w0 = wave * 64, lane = (int)threadIdx.x & 63;
    const int c0 = 4 * l.q, left = C - c0;
    Pack ws[3];
    float gw[3][4] = {};
#pragma unroll
    for (int s = 0; s < 3; ++s) ws[s] = l.on ? load_row<KIND>(row_at<KIND>(w, s, C, c0), left) : Pack{};
    const int begin = min(xcd_block() * chunk, F), end = min(begin + chunk, F);
    for (int f0 = begin + wave * per_wave; f0 < end; f0 += per_wave * (BLOCK / 64)) {
        const int n = min(per_wave, end - f0);
        wave_sync();
        for (int i = lane; i <= n; i += 64) soff[wave][i] = min(max(*at<KIND>(poff, f0 + i), 0), P);
        wave_sync();
        const int p_end = __builtin_amdgcn_readfirstlane(soff[wave][n]);
        for (int p0 = __builtin_amdgcn_readfirstlane(soff[wave][0]); p0 < p_end; p0 += 64) {
            const int np = min(64, p_end - p0);
            wave_sync();
            if (lane < np) {
                int lo = 0, hi = n;  // soff[lo] <= p0 + lane < soff[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (soff[wave][mid] <= p0 + lane) lo = mid; else hi = mid;
                }
                const int count = soff[wave][lo + 1] - soff[wave][lo];
                const Float3 xi = load_bary<KIND>(bary, p0 + lane);
                sb[w0 + lane] = make_float4(xi.a, xi.b, xi.c, 1.0f / (float)count);
                sf[w0 + lane] = make_int2(f0 + lo, count);
            }
            wave_sync();
            for (int i = l.r; l.on && i < np; i += map.rw) {
                const float4 xi = sb[w0 + i];
                const int2 fc = sf[w0 + i];
                const Pack g = load_row<KIND>(row_at<KIND>(gy, fc.x, C, c0), left);
                const Pack t = partial ? load_row<KIND>(row_at<KIND>(tex, p0 + i, C, c0), left) : Pack{};
                const float count = (float)fc.y;
                Pack out;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float gn = quotient(g.v[k], count, xi.w), gt = gn * t.v[k];
                    out.v[k] = gn * fmaf(xi.z, ws[2].v[k], fmaf(xi.y, ws[1].v[k], xi.x * ws[0].v[k]));
                    gw[0][k] = fmaf(xi.x, gt, gw[0][k]);
                    gw[1][k] = fmaf(xi.y, gt, gw[1][k]);
                    gw[2][k] = fmaf(xi.z, gt, gw[2][k]);
                }
                if (gtex) store_row<KIND>(row_at<KIND>(gtex, p0 + i, C, c0), out, left);
            }
        }
    }
    if (partial) rows_to_partial<KIND, 1>(gw, 3, map, l, C, lds, partial);
}

// Zeroes the rows of gtex that belong to no facet (in front of the kernel above): every row from poff[0] to below
// poff[F] is between two consecutive offsets, so these are the rows in front of the first and behind the last.
__global__ __launch_bounds__(BLOCK) void f2f_clear_kernel(const int* __restrict__ poff, int F, int P, int C,
                                                          float* __restrict__ gtex) {
    long long head = (long long)min(max(poff[0], 0), P) * C;
    const long long tail = (long long)min(max(poff[F], 0), P) * C;
    const long long n = (long long)P * C, stride = (long long)gridDim.x * BLOCK, g = (long long)blockIdx.x * BLOCK + threadIdx.x;
    if (tail < head) head = n;  // (offsets that descend: any row may belong to no facet)
    for (long long i = g; i < head; i += stride) gtex[i] = 0.0f;
    for (long long i = tail + g; i < n; i += stride) gtex[i] = 0.0f;
}

// ---------------------------------------------------------------------------
// Facet2vertex (Sec. 4.2): I_v = (1 / |N(v)|) sum_{f in N(v)} (sum_t pi_ft w_t) J_f,
// N(v) = the corners at v in ascending order.
// ---------------------------------------------------------------------------
template <int NP>
__device__ __forceinline__ void load_coefficients(float (&p)[4 * NP], const float* __restrict__ pi, int rows) {
    if constexpr (NP == 1) {
#pragma unroll
        for (int t = 0; t < 4; ++t) p[t] = pi[min(t, rows - 1)];
    } else {
#pragma unroll
        for (int g = 0; g < NP; ++g) {
            const Pack q = load_row<pool::ROW_EVEN>(g + 1 < NP ? pi + 4 * g : pi + (rows - 4), 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) p[4 * g + i] = q.v[i];
        }
    }
}

// Up to 16 components: one running sum sum_f pi_ft J_f per component and channel in registers, the filter applied
// once per vertex at the end (a sixth of the filter reads of applying it per corner).
template <int NP, int KIND>
struct F2vForwardOp {
    static constexpr int UNROLL = NP <= 2 ? 3 : 2, TT = 4 * NP;  // (registers)
    const float* y;
    const float* pi;
    const int* corners;
    float* x;
    int C, c0, left, H, T, lq;
    int* win_f;      // [WALK_WINDOW] facet
    float4* win_p;   // [NP][WALK_WINDOW] its coefficients
    const float4* wl;  // [TT][64] filter
    Pack yf[UNROLL];
    float acc[TT][4], n;
    __device__ void stage(int slot, int j) {
        const int f = in_range_or_zero(*at<KIND>(corners, j), H) / 3;
        win_f[slot] = f;
        float p[TT];
        load_coefficients<NP>(p, row_at<KIND>(pi, f, T, 0), T);
#pragma unroll
        for (int g = 0; g < NP; ++g) win_p[g * WALK_WINDOW + slot] = make_float4(p[4 * g], p[4 * g + 1], p[4 * g + 2], p[4 * g + 3]);
    }
    __device__ void begin(int, bool, int count) {
        n = (float)count;
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[t][i] = 0.0f;
    }
    __device__ void load(int u, int slot, int) { yf[u] = load_row<KIND>(row_at<KIND>(y, win_f[slot], C, c0), left); }
    __device__ void wait(int u) { arrived(yf[u]); }
    __device__ void use(int u, int slot, int) {
#pragma unroll
        for (int g = 0; g < NP; ++g) {
            const float4 p4 = win_p[g * WALK_WINDOW + slot];
            const float p[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (slot_used<NP>(4 * g + t, T))
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[4 * g + t][i] = fmaf(p[t], yf[u].v[i], acc[4 * g + t][i]);
        }
    }
    __device__ void end(int v, bool, bool first, const GroupSum& sum) {
        Pack out{};
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (slot_used<NP>(t, T)) {
                const float4 wt = wl[t * 64 + lq];
                out.v[0] = fmaf(wt.x, acc[t][0], out.v[0]); out.v[1] = fmaf(wt.y, acc[t][1], out.v[1]);
                out.v[2] = fmaf(wt.z, acc[t][2], out.v[2]); out.v[3] = fmaf(wt.w, acc[t][3], out.v[3]);
            }
        sum(out);
        if (!first) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) out.v[i] = n > 0.0f ? out.v[i] / n : 0.0f;
        store_row<KIND>(row_at<KIND>(x, v, C, c0), out, left);
    }
};

// The filter rows t0 .. t0 + rows - 1 of the channels this workgroup works on, in slots as above, to LDS.  By all
// its threads; ends with a barrier.
template <int NP, int KIND>
__device__ __forceinline__ void filter_to_lds(float4* wl /* [4 NP][64] */, const float* __restrict__ w, int t0, int rows, int C,
                                              const RowMap& map) {
    const int q0 = blockIdx.y * map.qc, qn = min(map.qc, map.Q - q0);
    for (int i = threadIdx.x; i < 4 * NP * 64; i += BLOCK) {
        const int t = i >> 6, q = i & 63;
        if (q >= qn || !slot_used<NP>(t, rows)) continue;
        const Pack p = load_row<KIND>(w + (size_t)(t0 + slot_component<NP>(t, rows)) * C + 4 * (q0 + q), C - 4 * (q0 + q));
        wl[i] = make_float4(p.v[0], p.v[1], p.v[2], p.v[3]);
    }
    __syncthreads();
}

template <int NP, int KIND>
__global__ __launch_bounds__(BLOCK) void f2v_forward_kernel(const float* __restrict__ y, int C,
                                                            const float* __restrict__ pi, int T,
                                                            const float* __restrict__ w,
                                                            const int* __restrict__ off,
                                                            const int* __restrict__ corners, int N, int H, 
                                                            float* __restrict__ x, WalkMap map) {
    __shared__ float4 wl[4 * NP * 64];
    __shared__ float4 win_p[BLOCK / 64 * NP * WALK_WINDOW];
    __shared__ int win_f[BLOCK / 64 * WALK_WINDOW];
    __shared__ int soff[BLOCK / 64][WALK_WAVE_ROWS + 1];
    const RowLane l = row_lane(map.row, blockIdx.y);
    const int wave = wave_id();
    filter_to_lds<NP, KIND>(wl, w, 0, T, C, map.row);
    const int v0 = (xcd_block() * (BLOCK / 64) + wave) * map.per_wave;
    if (v0 >= N) return;
    F2vForwardOp<NP, KIND> op;
    op.y = y; op.pi = pi; op.corners = corners; op.x = x;
    op.C = C; op.c0 = 4 * l.q; op.left = C - op.c0; op.H = H; op.T = T; op.lq = l.q - (int)blockIdx.y * map.row.qc;
    op.win_f = win_f + wave * WALK_WINDOW; op.win_p = win_p + wave * NP * WALK_WINDOW; op.wl = wl;
    walk_rows<KIND, F2vForwardOp<NP, KIND>::UNROLL>(op, off, v0, min(map.per_wave, N - v0), H, map, l, soff[wave]);
}

// sum_t pi_ft w_t of four channels, any number of components
template <int KIND>
__device__ __forceinline__ Pack fuzzy_filter(const float* __restrict__ pi, const float* __restrict__ w, int t0, int T, int C,
                                             int c0, Pack coef) {
    for (int t = t0; t < T; ++t) {
        const float p = pi[t];
        const Pack wt = load_row<KIND>(row_at<KIND>(w, t, C, c0), C - c0);
#pragma unroll
        for (int i = 0; i < 4; ++i) coef.v[i] = fmaf(p, wt.v[i], coef.v[i]);
    }
    return coef;
}

// More components than the registers of the kernel above hold: the filter is applied per corner.
template <int KIND>
__global__ __launch_bounds__(BLOCK) void f2v_forward_many_kernel(const float* __restrict__ y, int C,
                                                                 const float* __restrict__ pi, int T,
                                                                 const float* __restrict__ w,
                                                                 const int* __restrict__ off,
                                                                 const int* __restrict__ corners, int N, int H,
                                                                 float* __restrict__ x, RowMap map) {
    const RowLane l = row_lane(map, blockIdx.y);
    const int v = pool::wave_row(map, xcd_block()) + l.r;
    if (!l.on || v >= N) return;
    const int c0 = 4 * l.q, left = C - c0;
    const int s = max(off[v], 0), e = min(off[v + 1], H);
    Pack acc{};
    for (int j = s; j < e; ++j) {
        const int f = in_range_or_zero(corners[j], H) / 3;
        const Pack yf = load_row<KIND>(row_at<KIND>(y, f, C, c0), left);
        const Pack coef = fuzzy_filter<KIND>(row_at<KIND>(pi, f, T, 0), w, 0, T, C, c0, Pack{});
#pragma unroll
        for (int i = 0; i < 4; ++i) acc.v[i] = fmaf(coef.v[i], yf.v[i], acc.v[i]);
    }
    const float n = (float)(e - s);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc.v[i] = (e > s) ? acc.v[i] / n : 0.0f;
    store_row<KIND>(row_at<KIND>(x, v, C, c0), acc, left);
}

// Sum over the lanes of one row (neighbours within a wave, at places 0 .. n - 1; this lane at place q of them),
// valid in the row's first lane.
__device__ __forceinline__ float row_sum(float v, int q, int n) {
    for (int d = 1; d < n; d <<= 1) {
        const float o = __shfl_down(v, d, 64);
        if (q + d < n) v += o;
    }
    return v;
}

// V such sums at once, for rows of Q = 2 d lanes, a power of two (such rows begin at multiples of Q).  A step halves the values: a lane keeps
// the half that its bit d of q names and gives the other away; then, one value left, the further bits are summed as they are.  V - 1
// shuffles or fewer and one for each further bit, where one by one they take V for every bit.  Lane q holds, in front of v, the sums
// q V / Q up to (q + 1) V / Q (V >= Q), or the sum q V / Q rounded down (V < Q).
template <int V>
__device__ __forceinline__ void shared_row_sums(float (&v)[V], int q, int d) {
    if (d == 0) return;
    if constexpr (V == 1) {
        for (; d > 0; d >>= 1) v[0] = v[0] + __shfl_xor(v[0], d, 64);
    } else {
        const bool up = (q & d) != 0;
        float half[V / 2];
#pragma unroll
        for (int i = 0; i < V / 2; ++i) half[i] = (up ? v[i + V / 2] : v[i]) + __shfl_xor(up ? v[i] : v[i + V / 2], d, 64);
        shared_row_sums<V / 2>(half, q, d >> 1);
#pragma unroll
        for (int i = 0; i < V / 2; ++i) v[i] = half[i];
    }
}

// Backward pass of facet2vertex (supplementary, facet2vertex kernel).  With G = the incoming gradients of a
// facet's three vertices, each divided by its |N(v)|, summed:
//   gy_f = (sum_t pi_ft w_t) G,   gw_t = sum_f pi_ft (J_f G),   gpi_ft = sum over channels of w_t (J_f G),
// so one pass over the facets, which gathers the vertices' gradients once, makes all three (one pass for each
// before).  It takes the filter rows t0 .. t0 + rows - 1, rows <= 4 NP (slots as above); gy is made by the pass with t0 = 0, whose caller leaves
// it null in the others.  GPI: a row's lanes lie in one wave (row_map's one_wave) and each component's product is summed across them.  Bound by
// those shuffles, log2(Q) for a component, where they are taken one by one (GPI_ANY).  Rows of 2^k lanes sum 4 or 8 components together
// (GPI_POW2): with Q = 16, eight components take 8 shuffles for 32.  The pass with all three results, 240 k vertices, 16 / 32 / 64 / 128 channels,
// T = 6: 34.5 / 57.7 / 130.9 / 274.5 -> 30.8 / 43.9 / 88.6 / 170.3 us; T = 10: 62.7 / 120.3 / 177.7 / 388.6 -> 51.7 / 80.9 / 117.5 / 229.6; T = 1 by 1 to
// 5 % less.  Not with 13 to 16 components (NP = 4): the products kept back take 203 registers for 166 and so one of three waves; 360 k
// vertices, T = 13, 16 / 32 channels: 71 / 152 us one by one, 86 / 170 together.  A wave
// takes per_wave facets at a time, whose indices, counts and coefficients it brings to LDS, one facet per lane.
enum { GPI_NONE, GPI_ANY, GPI_POW2 };
template <int NP, int KIND, int GPI>
__global__ __launch_bounds__(BLOCK) void f2v_backward_kernel(const float* __restrict__ gx, const float* __restrict__ y, int C,
                                                             const float* __restrict__ pi, int T, int t0, int rows,
                                                             const float* __restrict__ w,
                                                             const int* __restrict__ facets, int F,
                                                             const int* __restrict__ off, int N, int chunk, int per_wave,
                                                             float* __restrict__ gy, float* __restrict__ partial,
                                                             float* __restrict__ gpi, RowMap map) {
    constexpr int TT = 4 * NP, SHARED = NP == 2 ? 8 : 4;  // SHARED: components summed together
    __shared__ float4 wl[TT * 64 > 2 * BLOCK ? TT * 64 : 2 * BLOCK];
    __shared__ int4 sv[BLOCK];         // per facet of the waves' batches: its vertices,
    __shared__ float4 sn[BLOCK], sr[BLOCK];  // ... their |N(v)| and the reciprocals,
    __shared__ float4 sp[NP * BLOCK];  // ... its coefficients
    const RowLane l = row_lane(map, blockIdx.y);
    const int c0 = 4 * l.q, left = C - c0, lq = l.q - (int)blockIdx.y * map.qc;
    const int w0 = wave_id() * 64, lane = (int)threadIdx.x & 63;
    filter_to_lds<NP, KIND>(wl, w, t0, rows, C, map);
    float gw[TT][4] = {};
    const int begin = min(xcd_block() * chunk, F), end = min(begin + chunk, F);
    for (int base = begin + wave_id() * per_wave; base < end; base += per_wave * (BLOCK / 64)) {
        const int n = min(per_wave, end - base);
        wave_sync();
        if (lane < n) {
            const int f = base + lane;
            const Int3 v = load_triple(row_at<KIND>(facets, f, 3, 0));
            const int a = in_range_or_zero(v.a, N), b = in_range_or_zero(v.b, N), c = in_range_or_zero(v.c, N);
            float p[TT];
            load_coefficients<NP>(p, row_at<KIND>(pi, f, T, t0), rows);
            const Int2 oa = load_pair(at<KIND>(off, a)), ob = load_pair(at<KIND>(off, b)), oc = load_pair(at<KIND>(off, c));
            const float na = (float)(oa.b - oa.a), nb = (float)(ob.b - ob.a), nc = (float)(oc.b - oc.a);
            sv[w0 + lane] = make_int4(a, b, c, 0);
            sn[w0 + lane] = make_float4(na, nb, nc, 0.0f);
            sr[w0 + lane] = make_float4(1.0f / na, 1.0f / nb, 1.0f / nc, 0.0f);
#pragma unroll
            for (int g = 0; g < NP; ++g) sp[g * BLOCK + w0 + lane] = make_float4(p[4 * g], p[4 * g + 1], p[4 * g + 2], p[4 * g + 3]);
        }
        wave_sync();
        // (with GPI every lane runs every step, for the sums across a row's lanes)
        for (int i0 = 0; i0 < n; i0 += map.rw) {
            const int i = i0 + l.r, f = base + i, at_i = w0 + min(i, n - 1);
            const bool on = l.on && i < n;
            if (GPI == GPI_NONE && !on) break;
            Pack gv[3] = {}, yf{};
            if (GPI == GPI_NONE || on) {
                const int4 v = sv[at_i];
                gv[0] = load_row<KIND>(row_at<KIND>(gx, v.x, C, c0), left);
                gv[1] = load_row<KIND>(row_at<KIND>(gx, v.y, C, c0), left);
                gv[2] = load_row<KIND>(row_at<KIND>(gx, v.z, C, c0), left);
                yf = load_row<KIND>(row_at<KIND>(y, f, C, c0), left);
            }
            const float4 nn = sn[at_i], rr = sr[at_i];
            Pack g, h, coef{};
            float dots[SHARED] = {};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                g.v[k] = (quotient(gv[0].v[k], nn.x, rr.x) + quotient(gv[1].v[k], nn.y, rr.y)) + quotient(gv[2].v[k], nn.z, rr.z);
                h.v[k] = on ? yf.v[k] * g.v[k] : 0.0f;
            }
#pragma unroll
            for (int gq = 0; gq < NP; ++gq) {
                const float4 p4 = sp[gq * BLOCK + at_i];
                const float p[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
                for (int tq = 0; tq < 4; ++tq) {
                    const int t = 4 * gq + tq;
                    if (slot_used<NP>(t, rows)) {
                        const float4 wt = wl[t * 64 + lq];
                        coef.v[0] = fmaf(p[tq], wt.x, coef.v[0]); coef.v[1] = fmaf(p[tq], wt.y, coef.v[1]);
                        coef.v[2] = fmaf(p[tq], wt.z, coef.v[2]); coef.v[3] = fmaf(p[tq], wt.w, coef.v[3]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) gw[t][k] = fmaf(p[tq], h.v[k], gw[t][k]);
                        if constexpr (GPI != GPI_NONE) {
                            float d = fmaf(wt.w, h.v[3], fmaf(wt.z, h.v[2], fmaf(wt.y, h.v[1], wt.x * h.v[0])));
                            if constexpr (GPI == GPI_POW2) {
                                dots[t % SHARED] = d;
                            } else {
                                d = row_sum(d, lq, map.Q);
                                if (on && lq == 0) gpi[(size_t)f * T + t0 + slot_component<NP>(t, rows)] = d;
                            }
                        }
                    }
                }
                if constexpr (GPI == GPI_POW2) {
                    if ((4 * gq + 4) % SHARED == 0) {
                        shared_row_sums<SHARED>(dots, lq, map.Q >> 1);
                        const int each = max(SHARED / map.Q, 1), way = max(map.Q / SHARED, 1);  // sums to a lane, lanes to a sum
                        const int first = lq / way * each, t1 = 4 * gq + 4 - SHARED + first;
#pragma unroll
                        for (int i = 0; i < SHARED; ++i)
                            if (on && lq % way == 0 && i < each && slot_used<NP>(t1 + i, rows)) gpi[(size_t)f * T + t0 + slot_component<NP>(t1 + i, rows)] = dots[i];
                    }
                }
            }
            if (gy && on) {
                if (T > rows) coef = fuzzy_filter<KIND>(row_at<KIND>(pi, f, T, 0), w, rows, T, C, c0, coef);
#pragma unroll
                for (int k = 0; k < 4; ++k) coef.v[k] = coef.v[k] * g.v[k];
                store_row<KIND>(row_at<KIND>(gy, f, C, c0), coef, left);
            }
        }
    }
    if (partial) rows_to_partial<KIND, NP>(gw, rows, map, l, C, wl, partial);
}

// gpi alone, where a row has more channels than a wave's lanes take at once: a wave per facet.
template <int KIND>
__global__ __launch_bounds__(BLOCK) void f2v_backward_pi_kernel(const float* __restrict__ gx, const float* __restrict__ y,
                                                                int C, int T, const float* __restrict__ w,
                                                                const int* __restrict__ facets, int F,
                                                                const int* __restrict__ off, int N,
                                                                float* __restrict__ gpi) {
    constexpr int TT = 8;
    const int lane = threadIdx.x & 63;
    const int f = blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
    if (f >= F) return;  // (whole waves leave together)
    const Int3 v = load_triple(row_at<KIND>(facets, f, 3, 0));
    const int vs[3] = {in_range_or_zero(v.a, N), in_range_or_zero(v.b, N), in_range_or_zero(v.c, N)};
    float n[3], r[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const Int2 o = load_pair(at<KIND>(off, vs[s]));
        n[s] = (float)(o.b - o.a);
        r[s] = 1.0f / n[s];
    }
    for (int t0 = 0; t0 < T; t0 += TT) {
        float d[TT] = {};
        for (int c0 = 4 * lane; c0 < C; c0 += 256) {
            const Pack yf = load_row<KIND>(row_at<KIND>(y, f, C, c0), C - c0);
            Pack h{};
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const Pack gv = load_row<KIND>(row_at<KIND>(gx, vs[s], C, c0), C - c0);
#pragma unroll
                for (int i = 0; i < 4; ++i) h.v[i] = h.v[i] + quotient(gv.v[i], n[s], r[s]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) h.v[i] = yf.v[i] * h.v[i];
#pragma unroll
            for (int t = 0; t < TT; ++t)
                if (t0 + t < T) {
                    const Pack wt = load_row<KIND>(row_at<KIND>(w, (t0 + t), C, c0), C - c0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[t] = fmaf(wt.v[i], h.v[i], d[t]);
                }
        }
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (t0 + t < T) {
                const float sum = row_sum(d[t], lane, 64);
                if (lane == 0) gpi[(size_t)f * T + t0 + t] = sum;
            }
    }
}

// ---------------------------------------------------------------------------
// Narrow rows, up to NARROW_C channels: a lane has a whole row (vertex, or facet in facet2vertex's backward pass), all channels in
// registers.  The kernels above give such rows a lane for four channels of every second to eighth item and fetch 64 items at a time
// through LDS, so that a wave walks 8 to 32 rows in steps of two trips to memory each; here 64 rows take three (offsets, corners, rows),
// four items in flight.  Facet2vertex's components need no sum across lanes for the coefficients' gradients, and the
// filter comes from scalar registers.  A row of more than NARROW_LONG items goes to all lanes of the wave.  By the kernels above / here,
// 720 k facets, 6 components, us: 3 channels facet2vertex 30 / 11, its backward pass 23 / 13, vertex2facet's 39 / 12; 6 channels 35 / 15, 29 / 18,
// 49 / 21; 8 channels 29 / 18, 26 / 21, 39 / 24 (120 k facets, 6 channels: 10 / 5, 17 / 9, 15 / 9).  The line at 8 channels is where registers run
// out: a row of vertex2facet's backward pass takes 10 values per channel besides the four rows in flight.
// ---------------------------------------------------------------------------
constexpr int NARROW_C = 8, NARROW_LONG = 64, NARROW_VALUES = 64;  // NARROW_VALUES: of a filter's gradient, in registers
template <int C>
struct NarrowRow {
    float v[C];
};
template <int C, typename T>
__device__ __forceinline__ T* narrow_at(T* p, int i) {
    return row_at<pool::ROW_TAIL>(p, i, C, 0);
}
template <int C>
__device__ __forceinline__ NarrowRow<C> load_narrow(const float* p, int i) {
    return *reinterpret_cast<const NarrowRow<C>*>(narrow_at<C>(p, i));
}
template <int C>
__device__ __forceinline__ void store_narrow(float* p, int i, const float (&v)[C]) {
    NarrowRow<C> r;
#pragma unroll
    for (int c = 0; c < C; ++c) r.v[c] = v[c];
    *reinterpret_cast<NarrowRow<C>*>(narrow_at<C>(p, i)) = r;
}

template <int C>
__device__ __forceinline__ void arrived(float (&v)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) pool::arrived(v[c]);
}

constexpr int pow2_at_least(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}
// The sums over a wave's lanes of V values each: halves of what a lane still holds are exchanged until it holds one
// (V - 1 shuffles, not 6 V), in a fixed tree.  Lane l gets the sum of value l * P / 64, P = V filled up to a power of two.
template <int P, int D>
__device__ __forceinline__ void exchange_halves(float (&v)[P]) {
    if constexpr (P > 1) {
        const bool up = ((int)threadIdx.x & D) != 0;
        float half[P / 2];
#pragma unroll
        for (int i = 0; i < P / 2; ++i) half[i] = (up ? v[i + P / 2] : v[i]) + __shfl_xor(up ? v[i] : v[i + P / 2], D, 64);
        exchange_halves<P / 2, D / 2>(half);
        v[0] = half[0];
    } else if constexpr (D > 0) {
        v[0] = v[0] + __shfl_xor(v[0], D, 64);
        exchange_halves<1, D / 2>(v);
    }
}
template <int V>
__device__ __forceinline__ float wave_sums(const float (&in)[V]) {
    constexpr int P = pow2_at_least(V);
    static_assert(P <= 64, "a value per lane");
    float v[P];
#pragma unroll
    for (int i = 0; i < P; ++i) v[i] = i < V ? in[i] : 0.0f;
    exchange_halves<P, 32>(v);
    return v[0];
}
// A workgroup's sums of V values per lane: value i to at(i).
template <int V, class At>
__device__ __forceinline__ void narrow_partial(const float (&in)[V], float (*lds)[64] /* [BLOCK / 64] */, At at_value) {
    constexpr int LANES = 64 / pow2_at_least(V);  // of a value
    const float mine = wave_sums<V>(in);
    const int lane = (int)threadIdx.x & 63;
    if (lane % LANES == 0) lds[wave_id()][lane / LANES] = mine;
    __syncthreads();
    const int i = threadIdx.x;
    if (i < V) {
        float* out = at_value(i);
        if (out) *out = (lds[0][i] + lds[1][i]) + (lds[2][i] + lds[3][i]);
    }
}

// The items [s, e) of the lane's row, in order, U of them at a time: items(j, n) with n <= U of them from j on in use.  Longer rows, by all lanes of the wave:
// every lane makes the sums of every 64th item (acc: V of them, zero at first), which are added up in a fixed tree and handed to the row's lane.
template <int U, int V, class Items>
__device__ __forceinline__ void narrow_walk(int s, int e, float (&acc)[V], Items items) {
    const bool is_long = e - s > NARROW_LONG;
    if (!is_long)
        for (int j = s; j < e; j += U) items(j, min(U, e - j), 1, acc);
    for (unsigned long long rest = __ballot(is_long); rest; rest &= rest - 1) {
        const int owner = __ffsll((long long)rest) - 1, lane = (int)threadIdx.x & 63;
        const int s0 = __shfl(s, owner, 64), e0 = __shfl(e, owner, 64);
        float part[V] = {};
        for (int j = s0 + lane; j < e0; j += 64 * U) items(j, min(U, (e0 - j + 63) / 64), 64, part);
#pragma unroll
        for (int i = 0; i < V; ++i) {
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) part[i] = part[i] + __shfl_xor(part[i], d, 64);
            if (lane == owner) acc[i] = part[i];
        }
    }
}

// See V2fBackwardOp.  Workgroup b takes the vertices of its chunk, one per lane and turn.
template <int C>
__global__ __launch_bounds__(BLOCK) void v2f_backward_narrow_kernel(const float* __restrict__ gy, const float* __restrict__ x,
                                                                    const int* __restrict__ level, const float* __restrict__ w,
                                                                    const int* __restrict__ off, const int* __restrict__ corners,
                                                                    int N, int H, int chunk, float* __restrict__ gx,
                                                                    float* __restrict__ partial) {
    constexpr int U = 4;
    __shared__ float lds[BLOCK / 64][64];
    float gw[3 * C] = {};
    const int begin = min(xcd_block() * chunk, N), end = min(begin + chunk, N);
    for (int v0 = begin; v0 < end; v0 += BLOCK) {  // (whole waves, for the long rows)
        const int v = v0 + (int)threadIdx.x;
        const bool on = v < end;
        const Int2 o = load_pair(at<pool::ROW_TAIL>(off, on ? v : begin));
        const int s = min(max(o.a, 0), H), e = on ? min(max(o.b, s), H) : s;
        const NarrowRow<C> xv = partial ? load_narrow<C>(x, on ? v : begin) : NarrowRow<C>{};
        float acc[4 * C] = {};  // A_0, A_1, A_2, B
        narrow_walk<U>(s, e, acc, [&](int j, int n, int step, float (&sum)[4 * C]) {
            int f[U], place[U], lv[U];
            NarrowRow<C> g[U];
#pragma unroll
            for (int u = 0; u < U; ++u) place[u] = in_range_or_zero(*at<pool::ROW_TAIL>(corners, j + min(u, n - 1) * step), H);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f[u] = place[u] / 3;
                place[u] -= 3 * f[u];
                lv[u] = level ? *at<pool::ROW_TAIL>(level, f[u]) : 1;
                g[u] = load_narrow<C>(gy, f[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) arrived(g[u].v);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < n) {
                    float amb, b;
                    lattice_moments(lv[u], amb, b);
#pragma unroll
                    for (int c = 0; c < C; ++c) sum[3 * C + c] = fmaf(b, g[u].v[c], sum[3 * C + c]);
                    if (amb != 0.0f) {  // (a facet of level 1, nearly every one, has a = b)
#pragma unroll
                        for (int p = 0; p < 3; ++p) {
                            const float a = place[u] == p ? amb : 0.0f;
#pragma unroll
                            for (int c = 0; c < C; ++c) sum[p * C + c] = fmaf(a, g[u].v[c], sum[p * C + c]);
                        }
                    }
                }
        });
        if (gx && on) {
            float out[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float w0 = w[c], w1 = w[C + c], w2 = w[2 * C + c];
                out[c] = fmaf((w0 + w1) + w2, acc[3 * C + c], fmaf(w2, acc[2 * C + c], fmaf(w1, acc[C + c], w0 * acc[c])));
            }
            store_narrow<C>(gx, v, out);
        }
        if (on)
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int c = 0; c < C; ++c) gw[p * C + c] = fmaf(xv.v[c], acc[p * C + c] + acc[3 * C + c], gw[p * C + c]);
    }
    if (partial) narrow_partial<3 * C>(gw, lds, [&](int i) { return partial + (size_t)blockIdx.x * (3 * C) + i; });
}

// Facet2vertex forward (T <= 4 NP components): the filter is put together per corner.
template <int C, int NP>
__global__ __launch_bounds__(BLOCK) void f2v_forward_narrow_kernel(const float* __restrict__ y, const float* __restrict__ pi, int T,
                                                                   const float* __restrict__ w, const int* __restrict__ off,
                                                                   const int* __restrict__ corners, int N, int H,
                                                                   float* __restrict__ x) {
    constexpr int TT = 4 * NP, U = NP <= 2 ? 4 : 2;
    const int v = xcd_block() * BLOCK + (int)threadIdx.x;
    const bool on = v < N;
    const Int2 o = load_pair(at<pool::ROW_TAIL>(off, on ? v : 0));
    const int s = min(max(o.a, 0), H), e = on ? min(max(o.b, s), H) : s;
    float acc[C] = {};
    narrow_walk<U>(s, e, acc, [&](int j, int n, int step, float (&sum)[C]) {
        int f[U];
        NarrowRow<C> yf[U];
        float p[U][TT];
#pragma unroll
        for (int u = 0; u < U; ++u) f[u] = in_range_or_zero(*at<pool::ROW_TAIL>(corners, j + min(u, n - 1) * step), H) / 3;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            yf[u] = load_narrow<C>(y, f[u]);
            load_coefficients<NP>(p[u], row_at<pool::ROW_TAIL>(pi, f[u], T, 0), T);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) arrived(yf[u].v);
        float coef[U][C] = {};
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (slot_used<NP>(t, T)) {
                const float* wt = w + slot_component<NP>(t, T) * C;  // (the same in all lanes)
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int u = 0; u < U; ++u) coef[u][c] = fmaf(p[u][t], wt[c], coef[u][c]);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < n)
#pragma unroll
                for (int c = 0; c < C; ++c) sum[c] = fmaf(coef[u][c], yf[u].v[c], sum[c]);
    });
    if (!on) return;
    const float n = (float)(e - s);
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = n > 0.0f ? acc[c] / n : 0.0f;
    store_narrow<C>(x, v, acc);
}

// See f2v_backward_kernel; T <= 4 NP components, 4 NP C <= NARROW_VALUES.
template <int C, int NP>
__global__ __launch_bounds__(BLOCK) void f2v_backward_narrow_kernel(const float* __restrict__ gx, const float* __restrict__ y,
                                                                    const float* __restrict__ pi, int T, const float* __restrict__ w,
                                                                    const int* __restrict__ facets, int F, const int* __restrict__ off,
                                                                    int N, int chunk, float* __restrict__ gy,
                                                                    float* __restrict__ partial, float* __restrict__ gpi) {
    constexpr int TT = 4 * NP;
    __shared__ float lds[BLOCK / 64][64];
    float gw[TT * C] = {};
    const int begin = min(xcd_block() * chunk, F), end = min(begin + chunk, F);
    for (int f = begin + (int)threadIdx.x; f < end; f += BLOCK) {
        const Int3 v = load_triple(row_at<pool::ROW_TAIL>(facets, f, 3, 0));
        float p[TT];
        load_coefficients<NP>(p, row_at<pool::ROW_TAIL>(pi, f, T, 0), T);
        const NarrowRow<C> yf = load_narrow<C>(y, f);
        const int at_v[3] = {in_range_or_zero(v.a, N), in_range_or_zero(v.b, N), in_range_or_zero(v.c, N)};
        Int2 o[3];
        NarrowRow<C> gv[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            o[s] = load_pair(at<pool::ROW_TAIL>(off, at_v[s]));
            gv[s] = load_narrow<C>(gx, at_v[s]);
        }
        float g[C], h[C], coef[C] = {};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const float n = (float)(o[s].b - o[s].a), r = 1.0f / n;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float q = quotient(gv[s].v[c], n, r);
                g[c] = s == 0 ? q : g[c] + q;
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) h[c] = yf.v[c] * g[c];
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (slot_used<NP>(t, T)) {
                const float* wt = w + slot_component<NP>(t, T) * C;  // (the same in all lanes)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    coef[c] = fmaf(p[t], wt[c], coef[c]);
                    gw[t * C + c] = fmaf(p[t], h[c], gw[t * C + c]);
                }
            }
        if (gpi) {
            float* out = row_at<pool::ROW_TAIL>(gpi, f, T, 0);
#pragma unroll
            for (int g0 = 0; g0 < TT; g0 += 4) {  // (four slots, four components in a row)
                Pack d{};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float* wt = w + min(slot_component<NP>(g0 + k, T), T - 1) * C;
#pragma unroll
                    for (int c = 0; c < C; ++c) d.v[k] = fmaf(wt[c], h[c], d.v[k]);
                }
                if constexpr (NP > 1) store_row<pool::ROW_EVEN>(out + slot_component<NP>(g0, T), d, 4);
                else store_row<pool::ROW_TAIL>(out, d, T);
            }
        }
        if (gy) {
#pragma unroll
            for (int c = 0; c < C; ++c) coef[c] = coef[c] * g[c];
            store_narrow<C>(gy, f, coef);
        }
    }
    if (partial)
        narrow_partial<TT * C>(gw, lds, [&](int i) -> float* {
            const int t = i / C;
            return slot_used<NP>(t, T) ? partial + ((size_t)blockIdx.x * T + slot_component<NP>(t, T)) * C + (i - t * C) : nullptr;
        });
}

}  // namespace conv
