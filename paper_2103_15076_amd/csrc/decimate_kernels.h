// decimate_kernels.h -- device side of the round-based QEM mesh decimation for
// gfx950: Algorithm 2 of the Picasso paper (Sec. 3) and the quadric equations of
// its supplementary section "Quadric error computation".  The greedy grouping
// that the paper leaves on the CPU (Alg. 2 lines 3-10) is done on the GPU by a
// parallel construction of the same matching.  Host side: picasso.hip.
//
// All fp32 arithmetic is written as single IEEE operations in a fixed order
// and compiled without contraction, so that results are reproducible to the bit.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "primitives.h"

#pragma clang fp contract(off)

using prim::u32;
using prim::u64;

namespace {

constexpr int BLOCK = prim::BLOCK;
constexpr u64 VMIN_NONE = ~0ull;
constexpr int ERR_BIT_BAD_INDEX = 1, ERR_BIT_NONFINITE = 2, ERR_BIT_INTERNAL = 4;  // State::err

// ---------------------------------------------------------------------------
// Device-resident bookkeeping
// ---------------------------------------------------------------------------
struct State {
    int err;       // bit0: bad facet index, bit1: non-finite coordinate, bit2: a kernel was launched for sizes it does not take
    int nv[2];     // vertex count, ping-pong by round parity
    int nf;        // facets that go out
    int nh;        // half-edge keys of the current round: 3 for every facet that has not collapsed
    int ne;        // distinct edges of the current round
    int live[3];   // worklist lengths of the selection sub-rounds (rotating)
    int sel_k;     // sub-round index the selection has reached (buffer rotation phase)
    int absorb_n;  // edges through which an un-paired vertex would join a pair's cluster (Alg. 2 line 11)
    int nv_kept;   // output vertices that some output facet refers to (option: degenerated vertices dropped)
    int wide;      // rounds by rings: this round goes by facets (most vertices of the input are no surface's, or there was no place left for a vertex's facets)
    int row_words;   // ... facets of the round's rings in rows: the sum of RingRows::taken
    int longest[2];  // ... of the longest one of more than 64, by the round's parity
    int missed;    // ... the budget's last pair is not among those that budget_range_kernel has listed
    // Written by every selection tail for kernels that the host queued behind it before looking
    // (they run only if the tail finished the matching): 1 / nv of the round then, else zeros.
    int go, guard_nv;
};

// One vertex = 64 bytes: position and the 10 quadric coefficients.
struct __attribute__((aligned(16))) VRec {
    float x, y, z, w0;
    float a00, a01, a02, a11;
    float a12, a22, b0, b1;
    float b2, c, w1, w2;
};

constexpr int MATCH_SLOTS = 32;
constexpr int MATCH_PAD = 32;  // ints: one 128-byte line per slot

struct MeshTab {       // per-mesh tables, all device pointers, B entries (+1 for offsets)
    int B;
    const int* voff;   // [B+1] current vertex offsets
    const int* target; // [B]
    const int* active; // [B] mesh takes part in this round
    const int* nrem;   // [B] pairs still to contract (budget of Alg. 2 line 4)
    int* matched;      // [B] pairs formed this round
    int* mslots;       // [B][MATCH_SLOTS][MATCH_PAD] partial pair counts, spread over cache lines so that
                       // the counting atomics of thousands of waves do not queue on one address
};

__device__ __forceinline__ int mesh_of(const int* __restrict__ voff, int B, int v) {
    if (B <= 1) return 0;
    int lo = 0, hi = B;  // invariant: voff[lo] <= v < voff[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (voff[mid] <= v) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ u32 cost_key(float c) {
    u32 u = __float_as_uint(c);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Order among pairs of equal cost (Alg. 2 line 3; Sec. 3, footnote on the shuffle inserted into the
// sorting): by edge index, or with a seed by a seeded bijection of the 32-bit integers applied to
// the edge index, so that flat regions are clustered differently from epoch to epoch.  Every step
// of enc() is invertible (xor with a constant, multiplication by an odd number, xor with a right
// shift of itself, addition of a constant); dec() undoes them in reverse.
constexpr u32 inverse_mod_2_32(u32 a) {
    u32 x = a;  // correct to 3 bits for odd a; each step doubles the number of correct bits
    for (int i = 0; i < 5; ++i) x *= 2u - a * x;
    return x;
}
constexpr u32 TIE_M1 = 0x9E3779B1u, TIE_M2 = 0x85EBCA77u;
constexpr u32 TIE_M1_INV = inverse_mod_2_32(TIE_M1), TIE_M2_INV = inverse_mod_2_32(TIE_M2);
static_assert(TIE_M1 * TIE_M1_INV == 1u && TIE_M2 * TIE_M2_INV == 1u, "modular inverses");

struct TieBreak {
    u32 on, s0, s1;
    __device__ __forceinline__ u32 enc(u32 e) const {
        if (!on) return e;
        u32 x = e ^ s0;
        x *= TIE_M1;
        x ^= x >> 15;
        x *= TIE_M2;
        x ^= x >> 13;
        return x + s1;
    }
    __device__ __forceinline__ u32 dec(u32 x) const {
        if (!on) return x;
        x -= s1;
        x ^= x >> 13;
        x ^= x >> 26;
        x *= TIE_M2_INV;
        x ^= x >> 15;
        x ^= x >> 30;
        x *= TIE_M1_INV;
        return x ^ s0;
    }
    __device__ __forceinline__ u64 priority(u32 cost_key_, int e) const { return ((u64)cost_key_ << 32) | enc((u32)e); }
};

// An edge's bid on one of its ends: among the edges at one vertex, the order by edge index is the order by their other
// ends (those below the vertex come first in both), so without shuffle the bid names that end instead: the best
// bid on a vertex then tells its partner without a look at the edge.
template <bool SHUFFLE>
__device__ __forceinline__ u64 edge_bid(const TieBreak& tb, u32 cost_key_, int e, int other) {
    if constexpr (SHUFFLE) return tb.priority(cost_key_, e);
    return ((u64)cost_key_ << 32) | (u32)other;
}

// ---------------------------------------------------------------------------
// Round set-up
// ---------------------------------------------------------------------------
struct RoundTab {
    int B;
    const int* voff;
    const int* target;
    int* active;
    const int* was_active;  // in the round before
    int* stuck;
    int* nrem;
    const int* matched;     // ... pairs formed then
    int* mslots;
    int* live_n;  // see SelArgs
    int first_round;
};

// A mesh takes part in a round if it has more vertices than it is to keep, unless it formed no pair in a round before.  (Said by the
// workgroups of a round's first kernel, each for itself, while one of them writes it down: none of what they read changes but `stuck`,
// which that one sets where this says so anyway.)
__device__ __forceinline__ bool mesh_stuck(const RoundTab& R, int b) {
    return R.stuck[b] != 0 || (!R.first_round && R.was_active[b] != 0 && R.matched[b] == 0);
}
__device__ __forceinline__ bool mesh_active(const RoundTab& R, int b) {
    return R.voff[b + 1] - R.voff[b] > R.target[b] && !mesh_stuck(R, b);
}

// Per-mesh budgets and the round's counters, by one workgroup.
__device__ __forceinline__ void round_begin_block(const RoundTab& R, State* st) {
    for (int i = threadIdx.x; i < R.B * MATCH_SLOTS; i += blockDim.x) R.mslots[(size_t)i * MATCH_PAD] = 0;
    if (threadIdx.x < 32) R.live_n[threadIdx.x * MATCH_PAD] = 0;
    for (int b = threadIdx.x; b < R.B; b += blockDim.x) {
        const int nvb = R.voff[b + 1] - R.voff[b];
        const int act = mesh_active(R, b);
        if (mesh_stuck(R, b)) R.stuck[b] = 1;
        R.active[b] = act;
        R.nrem[b] = act ? nvb - R.target[b] : 0;
    }
    if (threadIdx.x == 0) {
        st->nh = 0;
        st->ne = 0;
        st->live[0] = 0;
        st->live[1] = 0;
        st->live[2] = 0;
        st->sel_k = 0;
        st->absorb_n = 0;
    }
}

// ---------------------------------------------------------------------------
// S0: vertex quadrics (supplementary: facet quadric Q=(nn^T, dn, d^2); vertex
// quadric = sum over adjacent facets, here in ascending facet order)
// ---------------------------------------------------------------------------

// Validates and copies the inputs into the workspace; emits the (vertex,
// incidence) pairs whose stable sort is the vertex->facet CSR.
enum { COUNT_NONE = 0, COUNT_SMALL = 1, COUNT_LARGE = 2, COUNT_XL = 3 };

struct Corners {
    int a, b, c;
};
__device__ __forceinline__ Corners load_corners(const int* __restrict__ facets, size_t f) {
    return Corners{facets[3 * f], facets[3 * f + 1], facets[3 * f + 2]};
}
__device__ __forceinline__ int corner(const Corners& q, int c) { return c == 0 ? q.a : (c == 1 ? q.b : q.c); }

// The same of facets as the caller gives them, where no copy of them is made (rounds by rings): an index that is out of range, of which the host has yet to hear, counts as 0.
__device__ __forceinline__ int given_vertex(int v, int n_verts) { return (u32)v < (u32)n_verts ? v : 0; }
__device__ __forceinline__ Corners load_given(const int* __restrict__ facets, size_t f, int n_verts) {
    const Corners q = load_corners(facets, f);
    return Corners{given_vertex(q.a, n_verts), given_vertex(q.b, n_verts), given_vertex(q.c, n_verts)};
}

// Incidence keys of a facet, one per corner: (vertex << fbits) | facet.
struct IncidenceKeys {
    const int* facets;
    int fbits, n_verts;
    static constexpr int PER = 3;
    typedef Corners Raw;
    __device__ __forceinline__ Corners load(int f) const { return load_given(facets, (size_t)f, n_verts); }
    __device__ __forceinline__ u64 key(const Corners& q, int f, int c) const { return ((u64)(u32)corner(q, c) << fbits) | (u64)(u32)f; }
    __device__ __forceinline__ bool keep(u64) const { return true; }
};

// Edge keys of a facet: the sides from its corners to the next ones as
// (lower vertex << vbits) | higher vertex; a side with equal ends, as all three of a collapsed facet (-1, -1, -1) are,
// has none: it gets the all-ones key, which no sort keeps.
__host__ __device__ __forceinline__ u64 edge_sentinel(int vbits) { return vbits >= 32 ? ~0ull : ((1ull << (2 * vbits)) - 1ull); }
__device__ __forceinline__ u64 edge_key(int a, int b, int vbits) {
    const int lo = min(a, b), hi = max(a, b);
    return lo == hi ? edge_sentinel(vbits) : (((u64)(u32)lo << vbits) | (u64)(u32)hi);
}

struct EdgeKeys {
    const int* fcur;
    int vbits;
    static constexpr int PER = 3;
    typedef Corners Raw;
    __device__ __forceinline__ Corners load(int f) const { return load_corners(fcur, (size_t)f); }
    __device__ __forceinline__ u64 key(const Corners& q, int, int c) const { return edge_key(corner(q, c), corner(q, c == 2 ? 0 : c + 1), vbits); }
    __device__ __forceinline__ bool keep(u64 k) const { return k != edge_sentinel(vbits); }
};

// Plane of a facet as (unit normal, d) with n . x + d = 0 (supplementary, facet quadric equation);
// a facet of zero area or with a repeated index gets the zero plane, hence the zero quadric.
// Positions come from the caller's packed [N,3] array.
__device__ __forceinline__ float4 facet_plane(const float* __restrict__ verts, int i0, int i1, int i2) {
    const float4 none = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (i0 == i1 || i1 == i2 || i0 == i2) return none;
    const float3 p0 = make_float3(verts[3 * (size_t)i0], verts[3 * (size_t)i0 + 1], verts[3 * (size_t)i0 + 2]);
    const float3 p1 = make_float3(verts[3 * (size_t)i1], verts[3 * (size_t)i1 + 1], verts[3 * (size_t)i1 + 2]);
    const float3 p2 = make_float3(verts[3 * (size_t)i2], verts[3 * (size_t)i2 + 1], verts[3 * (size_t)i2 + 2]);
    float ax = p1.x - p0.x, ay = p1.y - p0.y, az = p1.z - p0.z;
    float bx = p2.x - p0.x, by = p2.y - p0.y, bz = p2.z - p0.z;
    float nx = ay * bz - az * by;
    float ny = az * bx - ax * bz;
    float nz = ax * by - ay * bx;
    float len = sqrtf((nx * nx + ny * ny) + nz * nz);
    if (len == 0.0f) return none;
    nx = nx / len;
    ny = ny / len;
    nz = nz / len;
    const float d = -((nx * p0.x + ny * p0.y) + nz * p0.z);
    return make_float4(nx, ny, nz, d);
}

// The header (State and the per-mesh tables) of up to HEADER_MESHES meshes is written by init_kernel itself instead of
// a copy from the host in front of it (6 us of a call): everything zero except the counts, the meshes' vertex and
// facet ranges and their targets, which come with the launch.  State::err is left alone (other workgroups of the same kernel flag
// errors there): it is zero between calls.  hdr == nullptr: the header has been uploaded.
constexpr int HEADER_MESHES = 32;
struct HeaderInit {
    int* hdr;
    int total;                           // ints in the header
    int at_voff0, at_foff, at_target;    // where the tables start
};
struct OneMesh {  // (no tables in the launch: 400 bytes of arguments cost a microsecond in front of the first kernel)
    int target;
};
struct FewMeshes {
    int voff[HEADER_MESHES + 1], foff[HEADER_MESHES + 1], target[HEADER_MESHES];
};

// Incidence keys for S0: (vertex << fbits) | facet, one per facet corner, so that sorting the keys
// alone lists every vertex's facets in ascending facet order; edge keys for the first round (see edge_keys_kernel, which is
// the first kernel of the others).  With COUNT_SMALL (digits of 8 to 10 bits) and COUNT_LARGE (11 and 12) the
// kernel also adds both keys' top digits to the histograms that the sorts start from (zero on entry; left so
// by the sorts); the sorts make the keys again from the validated facets, so they are
// written nowhere.  COUNT_XL: digits as wide as the masks say, counted in memory.  COUNT_NONE: no round follows.  edges: the
// round's set-up is made; SORTED (EDGES_SORTED): the edges' digits are wanted as well.
struct DigitCount {
    u32* hist;
    int shift;
    u32 mask;
};
// A workgroup's counts of one sort's digits, in LDS: an array of all digits, kept until the workgroup ends, or (COUNT_XL) a
// table of those that a tile holds.  The lanes of a wave that share a digit, as the keys of neighbouring facets mostly do,
// are counted with a single atomic.  clear, count and flush by whole workgroups, with barriers between them.
template <int COUNT>
struct DigitTally {
    static constexpr int RADIX = COUNT == COUNT_LARGE ? (1 << prim::BUCKET_LARGE_MSD_BITS) : (1 << prim::NARROW_BITS_MAX);
    u32 hist[RADIX];
    __device__ __forceinline__ void clear(const DigitCount& D) {
        for (int i = threadIdx.x; i <= (int)D.mask; i += BLOCK) hist[i] = 0;
    }
    __device__ __forceinline__ void count(const DigitCount& D, bool ok, u64 k) {
        const u32 d = (u32)(k >> D.shift) & D.mask;
        const prim::SameDigit same = prim::wave_same_digit(ok, d);
        if (ok && same.below == 0) atomicAdd(&hist[d], same.count);
    }
    __device__ __forceinline__ void flush(const DigitCount& D) {
        for (int i = threadIdx.x; i <= (int)D.mask; i += BLOCK) {
            const u32 c = hist[i];
            if (c) atomicAdd(&D.hist[i], c);
        }
    }
};
template <>
struct DigitTally<COUNT_XL> {
    prim::DigitTable table;
    __device__ __forceinline__ void clear(const DigitCount&) { table.clear(); }
    __device__ __forceinline__ void count(const DigitCount& D, bool ok, u64 k) {
        table.add(D.hist, ok, (u32)(k >> D.shift) & D.mask);
    }
    __device__ __forceinline__ void flush(const DigitCount& D) { table.flush(D.hist); }
};
template <>
struct DigitTally<COUNT_NONE> {
    __device__ __forceinline__ void clear(const DigitCount&) {}
    __device__ __forceinline__ void count(const DigitCount&, bool, u64) {}
    __device__ __forceinline__ void flush(const DigitCount&) {}
};

constexpr int RINGS_TAKEN = 2 * 33 * MATCH_PAD;  // counters of the rings' rows (RingRows): two sets of rings
enum { EDGES_NONE = 0, EDGES_BY_FACETS = 1, EDGES_SORTED = 2 };
template <int COUNT, bool SORTED, class Tables>
__global__ __launch_bounds__(BLOCK) void init_kernel(const float* __restrict__ verts, int N,
                                                     const int* __restrict__ facets, int F, int B,
                                                     const int* __restrict__ voff, const int* __restrict__ foff,
                                                     VRec* __restrict__ vrec, int* __restrict__ cid,
                                                     int* __restrict__ fcur /* or null */, int fbits, DigitCount inc, DigitCount edge,
                                                     int edges, int vbits, State* st, HeaderInit init, Tables tables,
                                                     float4* __restrict__ planes, int* __restrict__ htab, int n_clear,
                                                     u64* __restrict__ vmin0, u64* __restrict__ vmin1,
                                                     int* __restrict__ mate, u32* __restrict__ pcost, RoundTab R,
                                                     int* __restrict__ taken /* RINGS_TAKEN words, or null */) {
    __shared__ DigitTally<COUNT> corners;
    __shared__ DigitTally<SORTED ? COUNT : COUNT_NONE> sides;
    const int stride = gridDim.x * BLOCK;
    const int g = blockIdx.x * BLOCK + threadIdx.x;
    constexpr bool ONE = std::is_same<Tables, OneMesh>::value;
    const bool here = init.hdr != nullptr;  // (the tables in memory are then not to be read: this kernel writes them)
    if (here && blockIdx.x == 0) {
        constexpr int ERR = (int)(offsetof(State, err) / sizeof(int));
        constexpr int NV0 = (int)(offsetof(State, nv) / sizeof(int));
        for (int i = threadIdx.x; i < init.total; i += BLOCK) {
            if (i == ERR) continue;
            int v = 0;
            if constexpr (ONE) {
                if (i == NV0 || i == init.at_voff0 + 1) v = N;
                else if (i == init.at_foff + 1) v = F;
                else if (i == init.at_target) v = tables.target;
            } else {
                if (i == NV0) v = N;
                else if (i >= init.at_voff0 && i <= init.at_voff0 + B) v = tables.voff[i - init.at_voff0];
                else if (i >= init.at_foff && i <= init.at_foff + B) v = tables.foff[i - init.at_foff];
                else if (i >= init.at_target && i < init.at_target + B) v = tables.target[i - init.at_target];
            }
            init.hdr[i] = v;
        }
    }
    if (edges != EDGES_NONE && blockIdx.x == 0) {
        __syncthreads();  // (the header, where this workgroup has written it)
        round_begin_block(R, st);
    }
    for (int i = g; i < n_clear; i += stride) htab[i] = -1;  // (see final_facets_kernel)
    if (taken && blockIdx.x == 0)
        for (int i = threadIdx.x; i < RINGS_TAKEN; i += BLOCK) taken[i] = 0;
    corners.clear(inc);
    if (SORTED) sides.clear(edge);
    __syncthreads();
    int err = 0;
    for (int w = g; w < N; w += stride) {
        float x = verts[3 * (size_t)w], y = verts[3 * (size_t)w + 1], z = verts[3 * (size_t)w + 2];
        if (!(isfinite(x) && isfinite(y) && isfinite(z))) err |= 2;
        if (COUNT == COUNT_NONE || F == 0) {  // (else QuadricRows writes the whole record)
            VRec r;
            r.x = x; r.y = y; r.z = z; r.w0 = 0.f;
            r.a00 = r.a01 = r.a02 = r.a11 = r.a12 = r.a22 = r.b0 = r.b1 = r.b2 = r.c = r.w1 = r.w2 = 0.f;
            vrec[w] = r;
        }
        if (cid) cid[w] = w;
        if (edges != EDGES_NONE) {
            vmin0[w] = VMIN_NONE;
            if (vmin1) vmin1[w] = VMIN_NONE;
        }
        if (SORTED) {
            mate[w] = -1;
            pcost[w] = ~0u;
        }
    }
    for (int f0 = blockIdx.x * BLOCK; f0 < F; f0 += stride) {  // (whole waves, for the ballots below)
        const int f = f0 + threadIdx.x;
        const bool ok = f < F;
        int lo = 0, hi = 0;
        if (ok) {
            if constexpr (ONE) {
                hi = N;
            } else if (here) {
                const int m = mesh_of(tables.foff, B, f);
                lo = tables.voff[m];
                hi = tables.voff[m + 1];
            } else {
                const int m = mesh_of(foff, B, f);
                lo = voff[m];
                hi = voff[m + 1];
            }
        }
        const Corners given = load_corners(facets, (size_t)(ok ? f : 0));
        int at[3] = {given.a, given.b, given.c};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bool bad = ok && (at[c] < lo || at[c] >= hi);
            if (bad) err |= 1;
            if (bad || !ok) at[c] = fcur ? lo : given_vertex(at[c], N);
            if (ok && fcur) fcur[3 * (size_t)f + c] = at[c];
        }
        // the facet's plane, once per facet, for the vertex quadrics that S0 sums from it
        if (planes && ok) planes[f] = facet_plane(verts, at[0], at[1], at[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) corners.count(inc, ok, ((u64)(u32)at[c] << fbits) | (u64)(u32)f);
        if (SORTED) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int a = at[c], b = at[c == 2 ? 0 : c + 1];
                sides.count(edge, ok && a != b, edge_key(a, b, vbits));
            }
        }
        if constexpr (COUNT == COUNT_XL) {
            __syncthreads();
            corners.flush(inc);
            if (SORTED) sides.flush(edge);
            __syncthreads();
            corners.clear(inc);
            if (SORTED) sides.clear(edge);
            __syncthreads();
        }
    }
    if constexpr (COUNT != COUNT_XL) {
        __syncthreads();
        corners.flush(inc);
        if (SORTED) sides.flush(edge);
    }
    if (err) atomicOr(&st->err, err);
}

// ---------------------------------------------------------------------------
// Lists of items per row (corners of a vertex, members of a cluster) from an array that names every item's row:
// the keys (row << ibits) | item are counted by their top digit and sorted (the partition makes them from the array again; the
// per-bucket kernel writes the lists).  Four launches with the one that tells the host, a fifth for wide digits.
// ---------------------------------------------------------------------------
struct RowKeys {
    const int* row_of;  // [n]
    int n_rows, ibits;
    static constexpr int PER = 1;
    typedef int Raw;
    __device__ __forceinline__ int load(int i) const { return row_of[i]; }
    __device__ __forceinline__ u64 key(int r, int i, int) const {
        return ((u64)((u32)r < (u32)n_rows ? (u32)r : 0u) << ibits) | (u64)(u32)i;  // (a bad row counts as row 0 here)
    }
    __device__ __forceinline__ bool keep(u64) const { return true; }
};

// Adds the keys' digits to the sort's histogram (COUNT as in init_kernel) and flags rows out of range.
constexpr int CSR_COUNT_ITEMS = 4;
template <int COUNT>
__global__ __launch_bounds__(BLOCK) void csr_count_kernel(RowKeys src, int n, DigitCount rows, int* __restrict__ err) {
    constexpr int ITEMS = COUNT == COUNT_LARGE ? 16 : CSR_COUNT_ITEMS;
    __shared__ DigitTally<COUNT> digits;
    digits.clear(rows);
    __syncthreads();
    bool bad = false;
    int row[ITEMS];
    const int base = (int)blockIdx.x * (ITEMS * BLOCK) + (int)threadIdx.x;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) row[j] = src.load(min(base + j * BLOCK, n - 1));
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        bad |= (u32)row[j] >= (u32)src.n_rows;
        digits.count(rows, base + j * BLOCK < n, src.key(row[j], base + j * BLOCK, 0));
    }
    __syncthreads();
    digits.flush(rows);
    if (bad) atomicOr(err, ERR_BIT_BAD_INDEX);
}

// off[r] = first position of row r, items[i] = item at position i: made by the sort's per-bucket kernel from the keys in LDS.  Where
// the digit ends within the row's bits a bucket holds whole rows, of which it writes the offsets, also of those without items;
// where it takes in bits of the item (fewer rows than buckets) a row starts with its first bucket.
// (With the sorted keys written out and taken apart by a launch of its own: 16 bytes per item more.)
struct RowLists {
    int* off;
    int* items;
    int n, n_rows, ibits, digit_bits;
    template <int THREADS, int ITEMS>
    struct Lds {};
    // Where a group of the sort is a row, its first position is the row's.  (Found among the keys, a key and the one in front of it at a
    // time, before: lists of 5.7 M corners of 960 k vertices 19.9 us, now 17.0; of 115 k members of 41 k clusters 6.2 and 5.2.)
    static constexpr bool GROUPS_SORTED = true;
    __device__ bool rows_are_groups(bool, const prim::Bucket& b, int R) const { return b.low_bits > ibits && (1 << (b.low_bits - ibits)) == R; }
    template <int THREADS, int ITEMS, class L>
    __device__ __forceinline__ void emit_groups(L& lds, const prim::Bucket& b, int R) const {
        const int t = threadIdx.x, start = (int)b.start, lo = b.number * R, rows = min(R, n_rows - lo);
        if (b.number == 0 && t == 0) off[n_rows] = n;
        for (int i = t; i < b.cnt; i += THREADS) items[start + i] = (int)b.item(lds.skey[i], ibits);
        for (int r = t; r < rows; r += THREADS) off[lo + r] = start + (int)lds.gstart[r];
    }
    template <int THREADS, int ITEMS, class L, typename LK, class KeyAt>
    __device__ __forceinline__ void emit(bool, L&, const prim::Bucket& b, LK*, LK*, KeyAt key_at) const {
        const int t = threadIdx.x, start = (int)b.start;
        if (b.number == 0 && t == 0) off[n_rows] = n;
        if (b.low_bits < ibits) {
            const int within = ibits - b.low_bits, r = b.number >> within;
            if (t == 0 && r < n_rows && (b.number & ((1 << within) - 1)) == 0) off[r] = start;
            for (int i = t; i < b.cnt; i += THREADS) items[start + i] = (int)(b.whole(key_at(i)) & ((1ull << ibits) - 1ull));
            return;
        }
        const int per = b.low_bits - ibits;
        const long long lo64 = (long long)b.number << per;
        if (lo64 >= n_rows) return;
        const int lo = (int)lo64, hi = (int)min(lo64 + (1ll << per), (long long)n_rows);  // the bucket's rows
        for (int i = t; i < b.cnt; i += THREADS) {
            const auto key = key_at(i), prev = key_at(max(i - 1, 0));
            items[start + i] = (int)b.item(key, ibits);
            if (i == 0 || b.row_in(key, ibits) != b.row_in(prev, ibits)) {
                const int k = b.row(key, ibits);
                for (int r = i ? b.row(prev, ibits) + 1 : lo; r <= k; ++r) off[r] = start + i;
            }
        }
        const int last = b.cnt > 0 ? b.row(key_at(b.cnt - 1), ibits) : lo - 1;
        for (int r = last + 1 + t; r < hi; r += THREADS) off[r] = start + b.cnt;
    }
};

// Ordered segmented reduction over the sorted incidence keys (vertex << fbits | facet), by the sort's per-bucket kernel from
// the keys in LDS (a bucket holds whole vertices): the keys of one vertex are consecutive and ascend in facet index, which is the
// order of the sum.  A wave lists where the vertices start in QR_WINDOW keys at a time; every such row goes to one lane, which
// fetches the facets' planes (computed once per facet by init_kernel), eight in flight, adds up their quadrics
// Q = (n n^T, d n, d^2) left to right and writes the vertex's whole 64-byte record, position
// included.  Vertices without any facet appear in no key: the row of the next
// vertex that has one notes the run of them in front of it (a bucket's last row also the run behind it),
// and the workgroup writes their records (zero quadric) together.
constexpr int QR_CHUNKS = 4, QR_WINDOW = 64 * QR_CHUNKS;
constexpr int QR_GAPS = 64;  // runs of facet-less vertices a bucket lists (further ones are written by the lane that meets them)

__device__ __forceinline__ void write_vertex_record(VRec* __restrict__ vrec, const float* __restrict__ verts, int v,
                                                    const float (&acc)[10]) {
    float4* r = reinterpret_cast<float4*>(&vrec[v]);
    r[0] = make_float4(verts[3 * (size_t)v], verts[3 * (size_t)v + 1], verts[3 * (size_t)v + 2], 0.f);
    r[1] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    r[2] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    r[3] = make_float4(acc[8], acc[9], 0.f, 0.f);
}

// acc += the quadric of the plane (n, d), coefficient by coefficient
__device__ __forceinline__ void add_plane_quadric(float (&acc)[10], const float4 pl) {
    const float q0 = pl.x * pl.x, q1 = pl.x * pl.y, q2 = pl.x * pl.z, q3 = pl.y * pl.y, q4 = pl.y * pl.z;
    const float q5 = pl.z * pl.z, q6 = pl.w * pl.x, q7 = pl.w * pl.y, q8 = pl.w * pl.z, q9 = pl.w * pl.w;
    acc[0] = acc[0] + q0; acc[1] = acc[1] + q1; acc[2] = acc[2] + q2; acc[3] = acc[3] + q3;
    acc[4] = acc[4] + q4; acc[5] = acc[5] + q5; acc[6] = acc[6] + q6; acc[7] = acc[7] + q7;
    acc[8] = acc[8] + q8; acc[9] = acc[9] + q9;
}

// The rings of rounds by rings (see ring_costs_kernel): per vertex the facets that have it, each as its other two corners.  Of up to RING_MAX facets that name up to
// RING_MAX vertices, as nearly always, these vertices are noted, RING_ROW of them in a row of 32 bytes (`ids`), the others beside (`more`): facet i's first corner is the i-th of
// them, its second one that of the number that info gives.  (A ring is found from its vertex alone, most of them in one access.)  Other rings are noted facet by facet (first
// corner | second corner << 32), one behind the other, in `rows`: those of the input where their incidences lie among all, so that there is a place for each, later ones where
// counters say.  Scanned surfaces have 0 % of vertices with more than 8 facets at first and 3 % once they have been decimated, 0.1 % with more than 10: with eight at most a
// ladder of four levels of 16 meshes took 1,099 us.
// info: vertices | facets << 4 | numbers, four bits each, << 8; of other rings RING_ROWS | facets << 4 | where in `rows` << 32.
// The neighbours' costs lie the same way: of short rings in `ids` and `more`, of others beside the facets (first corner's | second corner's << 32, PAIR_NONE where the second one is
// a facet's first).  info of the neighbours, for up to ROW_SMALL facets: how many of them may have a second corner's cost (none or all) | facets << 8.
constexpr int RING_VERTICES = 1 << 28;  // (rounds by rings take fewer vertices)
constexpr int RING_MAX = 10, RING_ROW = 8, RING_MORE = RING_MAX - RING_ROW;
constexpr u32 RING_ROWS = 15;
constexpr int ROW_LINE = 8, ROW_SMALL = 16;  // (up to ROW_SMALL facets are a pair of lanes' and a quarter of a wave's work, more a wave's)
__device__ __forceinline__ u64 rows_info(int n, u32 at) { return (u64)(RING_ROWS | ((u32)n << 4)) | ((u64)at << 32); }
__device__ __forceinline__ int rows_length(u64 info) { return (int)((u32)info >> 4); }
__device__ __forceinline__ u32 rows_at(u64 info) { return (u32)(info >> 32); }
__device__ __forceinline__ u64 ring_info(int vertices, int facets, u64 numbers) { return (u64)((u32)vertices | ((u32)facets << 4)) | (numbers << 8); }
__device__ __forceinline__ bool ring_in_rows(u64 info) { return ((u32)info & 15u) == RING_ROWS; }
__device__ __forceinline__ int ring_ids(u64 info) { return (int)((u32)info & 15u); }  // (of a short ring)
__device__ __forceinline__ int ring_facets(u64 info) { return ring_in_rows(info) ? rows_length(info) : (int)((u32)info >> 4 & 15u); }
__device__ __forceinline__ int ring_second(u64 info, int i) { return (int)((u32)(info >> (8 + 4 * i)) & 15u); }
// Places in rows are handed out in parts, each with a counter in a cache line of its own (a line takes an atomic every 11 ns); those that are too long for a part come from the
// rest, as do those that find no room in a few parts.
constexpr int ROW_ARENAS = 32, ROW_TRIES = 4;
static_assert(RINGS_TAKEN == 2 * (ROW_ARENAS + 1) * MATCH_PAD, "a counter each");
struct RingRows {
    u32* ids;
    u32* more;
    u64* info;
    u64* rows;   // as many as the input has corners
    int* taken;  // [ROW_ARENAS + 1][MATCH_PAD]: words in use of each part, then of the rest
    u32 arena_words, rest_words;
    int* wide;   // set where there is no place
    // By one lane: a place of that many words, ~0u where there is none; asked for first, then looked at, so that the atomic's trip need not be waited for in between.
    __device__ __forceinline__ u32 ask(u32 words) const {
        const u32 part = words <= arena_words ? blockIdx.x & (ROW_ARENAS - 1) : (u32)ROW_ARENAS;
        return (u32)atomicAdd(&taken[part * MATCH_PAD], (int)words);
    }
    __device__ __forceinline__ u32 take(u32 words, u32 asked) const {
        u32 at = asked;
        if (words <= arena_words) {
            for (int k = 0;; ++k) {
                const u32 arena = (blockIdx.x + k) & (ROW_ARENAS - 1);
                if (k > 0) at = (u32)atomicAdd(&taken[arena * MATCH_PAD], (int)words);
                if ((u64)at + words <= arena_words) return arena * arena_words + at;
                if (k + 1 == ROW_TRIES) break;
            }
            at = (u32)atomicAdd(&taken[ROW_ARENAS * MATCH_PAD], (int)words);
        }
        if ((u64)at + words <= rest_words) return ROW_ARENAS * arena_words + at;
        *wide = 1;
        return ~0u;
    }
    // n: how many there are (of a row the first RING_ROW are fetched whatever n is)
    __device__ __forceinline__ void load_ids(int v, u32 (&x)[RING_MAX], int n) const {
        const uint4* r = reinterpret_cast<const uint4*>(ids + (size_t)v * RING_ROW);
        const uint4 a = r[0], b = r[1];
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        x[8] = x[9] = 0;
        if (n > RING_ROW) {
            const uint2 c = *reinterpret_cast<const uint2*>(more + (size_t)v * RING_MORE);
            x[8] = c.x; x[9] = c.y;
        }
    }
    __device__ __forceinline__ void store_ids(int v, const u32 (&x)[RING_MAX], int n) const {
        uint4* r = reinterpret_cast<uint4*>(ids + (size_t)v * RING_ROW);
        r[0] = make_uint4(x[0], x[1], x[2], x[3]);
        r[1] = make_uint4(x[4], x[5], x[6], x[7]);
        if (n > RING_ROW) *reinterpret_cast<uint2*>(more + (size_t)v * RING_MORE) = make_uint2(x[8], x[9]);
    }
    __device__ __forceinline__ u32* place(int v, int i) const {
        return i < RING_ROW ? ids + (size_t)v * RING_ROW + i : more + (size_t)v * RING_MORE + (i - RING_ROW);
    }
    // facet i of v's ring
    __device__ __forceinline__ void load_facet(int v, u64 info_, int i, u32& a, u32& b) const {
        const u32 *p, *q;
        if (ring_in_rows(info_)) {
            p = reinterpret_cast<const u32*>(rows + rows_at(info_) + i);
            q = p + 1;
        } else {
            p = place(v, i);
            q = place(v, ring_second(info_, i));
        }
        a = *p;
        b = *q;
    }
};
static_assert(RING_MORE == 2, "two beside the row");
// A facet of a ring.
__device__ __forceinline__ u64 ring_entry(int next, int prev) { return ((u64)(u32)prev << 32) | (u32)next; }
__device__ __forceinline__ u64 ring_entry_of(const Corners& q, int v) {
    return q.a == v ? ring_entry(q.b, q.c) : q.b == v ? ring_entry(q.c, q.a) : ring_entry(q.a, q.b);
}
// The short ring of the first n of these facets, or rows_info(0, 0) where it takes more than RING_MAX vertices.  (On a surface the second corners are the first ones in
// another order, but for open edges and facets wound the other way round.)
template <int N>
__device__ __forceinline__ u64 make_ring(const u64 (&e)[N], int n, u32 (&id)[RING_MAX]) {
#pragma unroll
    for (int k = 0; k < RING_MAX; ++k) id[k] = k < N && k < n ? (u32)e[k < N ? k : 0] : ~0u;
    u64 seconds = 0;
    u32 missing = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const u32 q = (u32)(e[i] >> 32);
        u32 at = RING_MAX;
#pragma unroll
        for (int k = N - 1; k >= 0; --k) at = id[k] == q ? (u32)k : at;
        missing |= i < n && at == RING_MAX ? 1u << i : 0u;
        seconds |= (u64)at << (4 * i);
    }
    int m = n;
    while (missing != 0 && m < RING_MAX) {
        u32 q = 0;
#pragma unroll
        for (int i = N - 1; i >= 0; --i) q = missing >> i & 1u ? (u32)(e[i] >> 32) : q;
#pragma unroll
        for (int k = 0; k < RING_MAX; ++k) id[k] = k == m ? q : id[k];
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((missing >> i & 1u) && (u32)(e[i] >> 32) == q) {
                seconds = (seconds & ~(15ull << (4 * i))) | ((u64)(u32)m << (4 * i));
                missing &= ~(1u << i);
            }
        ++m;
    }
    return missing != 0 ? rows_info(0, 0) : ring_info(m, n, seconds);
}

// RINGS: the vertex's ring (see ring_costs_kernel) is left as well, from the corners of the facets.
template <bool RINGS>
struct QuadricRows {
    VRec* vrec;
    const float* verts;
    const float4* planes;
    int N, fbits;
    const int* facets;
    RingRows ring;
    int* unfit;       // [ROW_ARENAS][MATCH_PAD]: vertices of few facets with more neighbours than a short ring has, as where facets are any three vertices; zero at the start
    int unfit_limit;  // ... of a part, beyond which the call goes by facets
    int most_facets;  // ... as it does with a vertex of more
    template <int THREADS, int ITEMS>
    struct Lds {
        unsigned short start[THREADS / 64][QR_WINDOW];  // (within the window)
        int gap[2 * QR_GAPS];  // runs [first, end) of vertices without facets
        int n_gaps;
    };
    // Mostly a group of the sort is a vertex: a lane then sorts its vertex's keys in registers and goes on with them (up to
    // GROUP_LANE keys; a wave sorts more).  (With the groups sorted in LDS and the vertices found again among the keys 115 k vertices took 12.3 us, now 9.6, 1.2 M
    // 49 and 42.5, 10.2 M 450 and 421.)
    // (With the rings the compiler takes 118 registers, for four waves: 1.2 M vertices 69 us, with 96 for five 63; of a decimated mesh of 384 k 34 and 28.  With 80 for six it spills:
    // as long there, but 16 spheres with poles of 128 facets, whose buckets are sorted whole, 73 us for 63.)
    static constexpr int MIN_WAVES = RINGS ? 5 : 1;
    static constexpr bool GROUPS_SORTED = false;
    static constexpr int GROUP_SHORT = 8, GROUP_LANE = 16;  // (sizes of a lane's sort)
    __device__ bool rows_are_groups(bool, const prim::Bucket& b, int R) const { return (1 << (b.low_bits - fbits)) == R && b.low_bits > fbits; }
    template <int G, typename LK>
    __device__ __forceinline__ void add_group(float (&acc)[10], const prim::Bucket& b, const LK* key, int g) const {
        LK k[G];
#pragma unroll
        for (int j = 0; j < G; ++j) k[j] = j < g ? key[j] : (LK) ~(LK)0;
        prim::network_sort_regs<LK, G>(k);
#pragma unroll
        for (int j0 = 0; j0 < G; j0 += 8) {  // (eight planes in flight)
            float4 p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j0 + j < g) p[j] = planes[b.item(k[j0 + j], fbits)];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j0 + j < g) add_plane_quadric(acc, p[j]);
        }
    }
    // The ring of a group that a lane has sorted, in any order of its facets, the first of which is the bucket's incidence `start`.  (By itself, behind the quadrics of all groups:
    // together they take 140 registers.)
    template <int G, typename LK>
    __device__ __forceinline__ u64 ring_of_group(const prim::Bucket& b, const LK* key, int g, int v, const u32* start) const {
        if constexpr (G <= RING_MAX) {
            u64 e[G];
#pragma unroll
            for (int j = 0; j < G; ++j) e[j] = j < g ? ring_entry_of(load_given(facets, b.item(key[j], fbits), N), v) : 0ull;
            return leave_ring(v, e, g, [&] { return b.start + *start; });
        } else {
            const u32 at = b.start + *start;
            u64* const row = ring.rows + at;
#pragma unroll 8
            for (int j = 0; j < g; ++j) row[j] = ring_entry_of(load_given(facets, b.item(key[j], fbits), N), v);
            return rows_info(g, at);
        }
    }
    // the ring of up to N facets
    template <int N, class At>
    __device__ __forceinline__ u64 leave_ring(int v, const u64 (&e)[N], int g, At where) const {
        u32 id[RING_MAX];
        const u64 info = make_ring(e, g, id);
        if (!ring_in_rows(info)) {
            ring.store_ids(v, id, ring_ids(info));
            return info;
        }
        const u32 at = where();
        u64* const row = ring.rows + at;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j < g) row[j] = e[j];
        return rows_info(g, at);
    }
    __device__ __forceinline__ void write(int v, const float (&acc)[10], u64 info) const {
        write_vertex_record(vrec, verts, v, acc);
        if constexpr (RINGS) ring.info[v] = info;
    }
    template <int THREADS, int ITEMS, class L>
    __device__ __forceinline__ void emit_groups(L& lds, const prim::Bucket& b, int R) const {
        const int t = threadIdx.x, lane = prim::lane_id(), lo = b.number * R, n = min(R, N - lo);
        if (t == 0) lds.nlong = 0;
        __syncthreads();
        for (int gi = t; gi < n; gi += THREADS) {
            const int gs = (int)lds.gstart[gi], g = (int)lds.gstart[gi + 1] - gs;
            float acc[10] = {};
            if (g > GROUP_LANE) {
                lds.gcnt[atomicAdd(&lds.nlong, 1u)] = (u32)gi;
                continue;
            }
            if (__any(g > GROUP_SHORT)) add_group<GROUP_LANE>(acc, b, lds.skey + gs, g);  // (one of the two for the wave, not one after the other)
            else add_group<GROUP_SHORT>(acc, b, lds.skey + gs, g);
            write_vertex_record(vrec, verts, lo + gi, acc);
        }
        if constexpr (RINGS) {
            int n_unfit = 0;
            for (int gi = t; gi < n; gi += THREADS) {
                const int gs = (int)lds.gstart[gi], g = (int)lds.gstart[gi + 1] - gs;
                if (g > GROUP_LANE) continue;
                u64 info;
                if (g > RING_MAX) info = ring_of_group<GROUP_LANE>(b, lds.skey + gs, g, lo + gi, &lds.gstart[gi]);
                else if (__any(g > GROUP_SHORT)) info = ring_of_group<RING_MAX>(b, lds.skey + gs, g, lo + gi, &lds.gstart[gi]);
                else info = ring_of_group<GROUP_SHORT>(b, lds.skey + gs, g, lo + gi, &lds.gstart[gi]);
                ring.info[lo + gi] = info;
                n_unfit += g <= RING_MAX && ring_in_rows(info) ? 1 : 0;
            }
            if (__any(n_unfit)) {
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) n_unfit += __shfl_xor(n_unfit, d, 64);
                if (lane == 0 && atomicAdd(&unfit[(b.number & (ROW_ARENAS - 1)) * MATCH_PAD], n_unfit) > unfit_limit) *ring.wide = 1;
            }
        }
        __syncthreads();
        for (int li = prim::wave_id(); li < (int)lds.nlong; li += THREADS / 64) {
            const int gi = (int)lds.gcnt[li], gs = (int)lds.gstart[gi], g = (int)lds.gstart[gi + 1] - gs;
            prim::rank_group_lds(lds.skey + gs, g);
            if constexpr (RINGS)
                for (int j = lane; j < g; j += 64)
                    ring.rows[b.start + (u32)(gs + j)] = ring_entry_of(load_given(facets, b.item(lds.skey[gs + j], fbits), N), lo + gi);
            if (lane == 0) {
                float acc[10] = {};
                for (int j0 = 0; j0 < g; j0 += 8) {
                    float4 p[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (j0 + j < g) p[j] = planes[b.item(lds.skey[gs + j0 + j], fbits)];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (j0 + j < g) add_plane_quadric(acc, p[j]);
                }
                write(lo + gi, acc, rows_info(g, b.start + (u32)gs));
            }
        }
    }
    template <int THREADS, int ITEMS, class L, typename LK, class KeyAt>
    __device__ __forceinline__ void emit(bool, L& lds, const prim::Bucket& b, LK*, LK*, KeyAt key_at) const {
        const int t = threadIdx.x, lane = prim::lane_id(), w = prim::wave_id(), n = b.cnt;
        const int per = b.low_bits - fbits;
        const long long lo64 = (long long)b.number << per;
        if (lo64 >= N) return;
        const int lo = (int)lo64, hi = (int)min(lo64 + (1ll << per), (long long)N);  // the bucket's vertices
        const float zero[10] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (n == 0) {
            for (int v = lo + t; v < hi; v += THREADS) write(v, zero, 0);
            return;
        }
        if (t == 0) lds.n_gaps = 0;
        __syncthreads();
        auto vertex_at = [&](int i) { return b.row(key_at(i), fbits); };
        auto row_at = [&](int i) { return b.row_in(key_at(i), fbits); };
        auto note_gap = [&](int first, int end) {
            const int slot = atomicAdd(&lds.n_gaps, 1);
            if (slot < QR_GAPS) {
                lds.gap[2 * slot] = first;
                lds.gap[2 * slot + 1] = end;
            } else {
                for (int g = first; g < end; ++g) write(g, zero, 0);
            }
        };
        unsigned short* list = lds.start[w];
        for (int base = w * QR_WINDOW; base < n; base += (THREADS / 64) * QR_WINDOW) {
            int m = 0;
#pragma unroll
            for (int c = 0; c < QR_CHUNKS; ++c) {
                const int i = base + c * 64 + lane;
                const int at = min(i, n - 1);
                const bool head = i < n && (i == 0 || row_at(at) != row_at(max(at - 1, 0)));
                const u64 bal = prim::ballot(head);
                if (head) list[m + (int)prim::mask_below(bal)] = (unsigned short)(c * 64 + lane);
                m += (int)__popcll(bal);
            }
            __builtin_amdgcn_wave_barrier();  // (a wave's LDS operations complete in order)
            for (int r0 = 0; r0 < m; r0 += 64) {
                const int r = r0 + lane;
                int hp = 0, end = 0, v = 0;
                if (r < m) {
                    hp = base + (int)list[r];
                    v = vertex_at(hp);
                    if (r + 1 < m) {
                        end = base + (int)list[r + 1];
                    } else {
                        end = min(base + QR_WINDOW, n);
                        while (end < n && vertex_at(end) == v) ++end;
                    }
                    const int pv = hp > 0 ? vertex_at(hp - 1) : lo - 1;
                    if (pv + 1 < v) note_gap(pv + 1, v);
                    float acc[10];
#pragma unroll
                    for (int k = 0; k < 10; ++k) acc[k] = 0.0f;
                    for (int j0 = hp; j0 < end; j0 += 8) {
                        float4 p[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (j0 + j < end) p[j] = planes[b.item(key_at(j0 + j), fbits)];
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (j0 + j < end) add_plane_quadric(acc, p[j]);
                    }
                    write_vertex_record(vrec, verts, v, acc);
                    if (end == n && v + 1 < hi) note_gap(v + 1, hi);
                    if constexpr (RINGS)
                        if (end - hp <= RING_MAX) {
                            u64 e[RING_MAX];
#pragma unroll
                            for (int j = 0; j < RING_MAX; ++j)
                                e[j] = j < end - hp ? ring_entry_of(load_given(facets, b.item(key_at(hp + j), fbits), N), v) : 0ull;
                            ring.info[v] = leave_ring(v, e, end - hp, [&] { return b.start + (u32)hp; });
                        } else {
                            ring.info[v] = rows_info(end - hp, b.start + (u32)hp);
                            if (end - hp > most_facets) *ring.wide = 1;
                        }
                }
                if constexpr (RINGS)  // (the facets of the others, one after the other by all lanes)
                    for (u64 todo = prim::ballot(end - hp > RING_MAX); todo != 0; todo &= todo - 1) {
                        const int from = __ffsll((long long)todo) - 1, first = __shfl(hp, from, 64), last = __shfl(end, from, 64), its = __shfl(v, from, 64);
#pragma unroll 4
                        for (int j = first + lane; j < last; j += 64)
                            ring.rows[b.start + (u32)j] = ring_entry_of(load_given(facets, b.item(key_at(j), fbits), N), its);
                    }
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        const int ng = min(lds.n_gaps, QR_GAPS);
        for (int i = 0; i < ng; ++i)
            for (int g = lds.gap[2 * i] + t; g < lds.gap[2 * i + 1]; g += THREADS) write(g, zero, 0);
    }
};

// ---------------------------------------------------------------------------
// S1: candidate pairs = distinct mesh edges (Alg. 2 line 1)
//
// First kernel of every round but the first (whose part init_kernel takes): the round's set-up (block 0), the per-vertex selection state, and the digits of the
// 64-bit keys (lower vertex, higher vertex), one per half-edge: the kernel adds the keys' top digits (8 to 10 bits with
// COUNT_SMALL, 11 or 12 with COUNT_LARGE, as xl_digit_bits says with COUNT_XL) to the histogram that the sort of the keys starts from
// (zeroed beforehand); the sort makes the keys again from the facets, so they are not written.
//
// The round before has contracted pairs and the facets still name its vertices: they are taken to
// the new numbering in place (S5).  A facet that has collapsed is marked (-1, -1, -1) and stays where it is: facets keep
// their places until the end of the call (a compaction each round read and wrote every facet twice more, in two
// launches; 1.2 M vertices: 58 us of the rounds' facet work).  Facets that have become equal to another stay too:
// they change no edge and no cost, are a few in ten thousand, and go at the end (final_facets_kernel).  Cluster labels follow
// the numbering.  A lane takes FACETS facets at a time, all of whose loads are in flight together.
// ---------------------------------------------------------------------------
// A facet whose corners have met is dropped if its mesh has been contracted; a mesh that no round took part in
// keeps its facets as they came.
__device__ __forceinline__ bool facet_collapsed(const Corners& q, const int* __restrict__ voff, int B,
                                                const int* __restrict__ done) {
    return (q.a == q.b || q.b == q.c || q.a == q.c) && done[mesh_of(voff, B, q.a)] != 0;
}

template <int COUNT>
__global__ __launch_bounds__(BLOCK) void edge_keys_kernel(int* __restrict__ fcur, int F, State* st, int cur, int vbits,
                                                          u64* __restrict__ vmin0, u64* __restrict__ vmin1,
                                                          int* __restrict__ mate, u32* __restrict__ pcost, RoundTab R,
                                                          DigitCount edge,
                                                          const int* __restrict__ vmap, const int* __restrict__ done,
                                                          int* __restrict__ cid, int n_orig) {
    constexpr int FACETS = COUNT == COUNT_SMALL ? 1 : 4;
    __shared__ DigitTally<COUNT> sides;
    const int nv = st->nv[cur];
    const int stride = gridDim.x * BLOCK;
    const int t = threadIdx.x, g = blockIdx.x * BLOCK + t;
    for (int w = g; w < nv; w += stride) {
        vmin0[w] = VMIN_NONE;
        vmin1[w] = VMIN_NONE;
        mate[w] = -1;
        pcost[w] = ~0u;
    }
    if (blockIdx.x == 0) round_begin_block(R, st);
    sides.clear(edge);
    __syncthreads();
    for (long long base = (long long)blockIdx.x * (BLOCK * FACETS); base < F; base += (long long)stride * FACETS) {
        Corners q[FACETS];
        bool ok[FACETS];
#pragma unroll
        for (int j = 0; j < FACETS; ++j) {
            const long long f = base + j * BLOCK + t;
            ok[j] = f < F;
            q[j] = load_corners(fcur, (size_t)(ok[j] ? f : 0));
        }
        Corners m[FACETS];
#pragma unroll
        for (int j = 0; j < FACETS; ++j) {
            ok[j] = ok[j] && q[j].a >= 0;
            m[j] = Corners{vmap[max(q[j].a, 0)], vmap[max(q[j].b, 0)], vmap[max(q[j].c, 0)]};
        }
#pragma unroll
        for (int j = 0; j < FACETS; ++j) {
            if (!ok[j]) continue;
            q[j] = m[j];
            if (facet_collapsed(q[j], R.voff, R.B, done)) q[j] = Corners{-1, -1, -1};
            int* o = fcur + 3 * (size_t)(base + j * BLOCK + t);
            o[0] = q[j].a; o[1] = q[j].b; o[2] = q[j].c;
        }
#pragma unroll
        for (int j = 0; j < FACETS; ++j) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int a = corner(q[j], c), b = corner(q[j], c == 2 ? 0 : c + 1);
                sides.count(edge, ok[j] && a != b, edge_key(a, b, vbits));
            }
        }
        if constexpr (COUNT == COUNT_XL) {
            __syncthreads();
            sides.flush(edge);
            __syncthreads();
            sides.clear(edge);
            __syncthreads();
        }
    }
    for (int o = g; o < n_orig; o += stride) cid[o] = vmap[cid[o]];
    if constexpr (COUNT != COUNT_XL) {
        __syncthreads();
        sides.flush(edge);
    }
}

// Where a pair is contracted to.
enum { PLACE_MEAN = 0, PLACE_INVERSE = 1 };

// Point of least quadric error, the solution of A x = -b (supplementary,
// inverse placement equation), for a positive semi-definite A = sum of n n^T.
// The three axes are eliminated in the order of the largest remaining diagonal
// entry (P A P^T = L D L^T); A counts as of full rank when all three pivots are
// positive and the last exceeds rcond_min times the first, their ratio standing
// for the reciprocal condition number.  Returns false, leaving (x, y, z) as
// they are, when A is not of full rank or the solution is not finite.
__device__ __forceinline__ bool quadric_minimiser(float a00, float a01, float a02, float a11, float a12, float a22,
                                                  float b0, float b1, float b2, float rcond_min, float& x, float& y,
                                                  float& z) {
    float r0 = -b0, r1 = -b1, r2 = -b2, t;
    int first = 0;
    float top = a00;
    if (a11 > top) { first = 1; top = a11; }
    if (a22 > top) { first = 2; top = a22; }
    if (first == 1) {  // axes 0 and 1 change places
        t = a00; a00 = a11; a11 = t;
        t = a02; a02 = a12; a12 = t;
        t = r0; r0 = r1; r1 = t;
    } else if (first == 2) {  // axes 0 and 2 change places
        t = a00; a00 = a22; a22 = t;
        t = a01; a01 = a12; a12 = t;
        t = r0; r0 = r2; r2 = t;
    }
    const float d1 = a00;
    if (!(d1 > 0.0f)) return false;
    float l1 = a01 / d1, l2 = a02 / d1;
    float s11 = a11 - (a01 * a01) / d1;
    const float s12 = a12 - (a01 * a02) / d1;
    float s22 = a22 - (a02 * a02) / d1;
    const bool flip = s22 > s11;  // the larger entry of the remaining block goes next
    if (flip) {
        t = s11; s11 = s22; s22 = t;
        t = l1; l1 = l2; l2 = t;
        t = r1; r1 = r2; r2 = t;
    }
    const float d2 = s11;
    if (!(d2 > 0.0f)) return false;
    const float l3 = s12 / d2;
    const float d3 = s22 - l3 * s12;
    if (!(d3 > 0.0f) || !(d3 > rcond_min * d1)) return false;
    const float y1 = r1 - l1 * r0;
    const float y2 = (r2 - l2 * r0) - l3 * y1;
    float w2 = y2 / d3;
    float w1 = y1 / d2 - l3 * w2;
    float w0 = (r0 / d1 - l1 * w1) - l2 * w2;
    if (flip) { t = w1; w1 = w2; w2 = t; }
    if (first == 1) { t = w0; w0 = w1; w1 = t; }
    else if (first == 2) { t = w0; w0 = w2; w2 = t; }
    if (!isfinite(w0) || !isfinite(w1) || !isfinite(w2)) return false;
    x = w0; y = w1; z = w2;
    return true;
}

// S2: cost of a pair = quadric error of the summed quadric at the point the
// pair would be contracted to: the pair's mean, or with PLACE_INVERSE the point
// of least error where the quadric has one (Alg. 2 line 2; supplementary
// Q(x) = x^T A x + 2 b^T x + c and the two placement equations).
struct VertexWords {
    float4 w[4];
};
__device__ __forceinline__ VertexWords load_vertex(const VRec* __restrict__ vrec, int v) {
    const float4* r = reinterpret_cast<const float4*>(&vrec[v]);
    return VertexWords{{r[0], r[1], r[2], r[3]}};
}
// (The same to the bit with its ends exchanged: every step in which they meet is a sum of two.)
template <int PLACE>
__device__ __forceinline__ float pair_cost(const VertexWords& U, const VertexWords& V, float rcond_min) {
    const float4 u0 = U.w[0], u1 = U.w[1], u2 = U.w[2], u3 = U.w[3];
    const float4 v0 = V.w[0], v1 = V.w[1], v2 = V.w[2], v3 = V.w[3];
    const float a00 = u1.x + v1.x, a01 = u1.y + v1.y, a02 = u1.z + v1.z, a11 = u1.w + v1.w;
    const float a12 = u2.x + v2.x, a22 = u2.y + v2.y, b0 = u2.z + v2.z, b1 = u2.w + v2.w;
    const float b2 = u3.x + v3.x, c = u3.y + v3.y;
    float mx = (u0.x + v0.x) * 0.5f;
    float my = (u0.y + v0.y) * 0.5f;
    float mz = (u0.z + v0.z) * 0.5f;
    if (PLACE == PLACE_INVERSE) quadric_minimiser(a00, a01, a02, a11, a12, a22, b0, b1, b2, rcond_min, mx, my, mz);
    const float t0 = (a00 * mx + a01 * my) + a02 * mz;
    const float t1 = (a01 * mx + a11 * my) + a12 * mz;
    const float t2 = (a02 * mx + a12 * my) + a22 * mz;
    const float xAx = (mx * t0 + my * t1) + mz * t2;
    const float bx = (b0 * mx + b1 * my) + b2 * mz;
    return (xAx + 2.0f * bx) + c;
}

// A workgroup's bids, put together in LDS before they go to memory.  Atomics are carried out at the memory side: of 64-bit minima
// the whole chip does 27 lines of 64 bytes (8 vertices) per nanosecond, in 1 MB as in 256 MB and with 8 lanes of a wave on a line's 8
// words (24) as with one, but lanes of a wave that name the same word take a request each (1.7 lines with 8 lanes per word).  The edges of a workgroup touch few vertices, and those lie in few lines, so the table
// holds lines: each goes out as one request.  A line that finds no place (a mesh numbered without locality) goes out
// by itself.  1.2 M vertices, first round: costs and bids 106 -> 83 us, sub-round 0 59 -> 51.
template <int LINES, int THREADS = BLOCK>
struct BidTable {
    static constexpr int PROBES = 4;
    int line[LINES];
    u64 bid[8 * LINES];
    __device__ __forceinline__ void clear() {
        for (int i = threadIdx.x; i < LINES; i += THREADS) line[i] = -1;
        for (int i = threadIdx.x; i < 8 * LINES; i += THREADS) bid[i] = VMIN_NONE;
    }
    // A bid p on vertex v.  rst: an array whose word of every vertex that is bid on is cleared (or null).
    __device__ __forceinline__ void put(u64* __restrict__ vmin, u64* __restrict__ rst, int v, u64 p) {
        const int l = v >> 3;
        u32 h = ((u32)l * 0x9E3779B1u >> 16) & (u32)(LINES - 1);
        for (int j = 0; j < PROBES; ++j) {
            int old = *(volatile int*)&line[h];
            if (old == -1) old = atomicCAS(&line[h], -1, l);
            if (old == -1 || old == l) {
                atomicMin(&bid[8 * h + (u32)(v & 7)], p);
                return;
            }
            h = (h + 1) & (u32)(LINES - 1);
        }
        atomicMin(&vmin[v], p);
        if (rst) rst[v] = VMIN_NONE;
    }
    __device__ __forceinline__ void flush(u64* __restrict__ vmin, u64* __restrict__ rst) {
        for (int i = threadIdx.x; i < 8 * LINES; i += THREADS) {
            const u64 b = bid[i];
            if (b == VMIN_NONE) continue;
            const size_t v = 8 * (size_t)line[i >> 3] + (size_t)(i & 7);
            atomicMin(&vmin[v], b);
            if (rst) rst[v] = VMIN_NONE;
        }
    }
};

// The distinct keys of an edge sort, as its per-bucket kernel has left them (DistinctKeys): per bucket at the front of its range of `keys`.
struct EdgeList {
    const void* keys;  // 32-bit (low bits) or 64-bit words
    const u32* starts;
    const u32* per_bucket;
    const u32* per_group;
    int buckets, low_bits;
    int split_shift, join_shift;  // 2^split_shift workgroups share a bucket, or a workgroup takes 2^join_shift buckets in a row
};

// Writes the distinct edges, their cost keys, and places each edge's first bid
// (sub-round 0 of the selection) on both of its vertices.  Bound by the two vertex records gathered per edge and what a workgroup does
// besides (numbering, its table of bids): a workgroup has 384 edges where there are few, for the chip's sake, and up to 1,536, with twice
// the table, where there are many (10.2 M vertices, 31 M edges: 384 edges 510 us, 1,536 392; workgroups are dealt to the XCDs in eighths
// of the buckets in use, so that the far ends' records are found in their L2).
constexpr int UNIQUE_EDGES_MIN = 384, UNIQUE_EDGES_MAX = 1536, UNIQUE_EDGES_NARROW = 1000;  // edges of a workgroup (about)
constexpr int UNIQUE_GROUPS_MIN = 4096;
constexpr int UNIQUE_JOIN_MAX = 2;
template <int PLACE, bool SHUFFLE, typename LK, int LINES>
__global__ __launch_bounds__(BLOCK) void unique_cost_kernel(EdgeList E, u64* __restrict__ ekey, u32* __restrict__ ecost,
                                                            unsigned char* __restrict__ estate, const VRec* __restrict__ vrec,
                                                            u64* __restrict__ vmin0, int vbits, MeshTab mt, float rcond_min,
                                                            TieBreak tb, int* __restrict__ ne_out) {
    __shared__ u32 smem[prim::WAVES];
    __shared__ BidTable<LINES> bids;
    const int t = threadIdx.x;
    if (E.buckets == 0) {  // no facets
        if (t == 0) *ne_out = 0;
        return;
    }
    const int item = prim::xcd_tile(((((long long)E.buckets - 1) >> E.join_shift) + 1) << E.split_shift, 1);
    const int first = item >> E.split_shift << E.join_shift, part = item & ((1 << E.split_shift) - 1), joined = 1 << E.join_shift;
    if (first >= E.buckets) return;  // (a workgroup too many)
    // distinct edges of the workgroup's buckets, up to and including each
    int upto[1 << UNIQUE_JOIN_MAX], n = 0;
#pragma unroll
    for (int j = 0; j < 1 << UNIQUE_JOIN_MAX; ++j) upto[j] = n += j < joined && first + j < E.buckets ? (int)E.per_bucket[first + j] : 0;
    const bool last = first + joined >= E.buckets && part == 0;
    if (part * BLOCK >= n && !last) return;
    const LK* __restrict__ keys = reinterpret_cast<const LK*>(E.keys);
    bids.clear();
    const int before = (int)prim::distinct_in_front(E.per_bucket, E.per_group, first, smem);  // (barriers)
    if (last && t == 0) *ne_out = before + n;
    const u64 vmask = (1ull << vbits) - 1ull;
    for (int q = part * BLOCK + t; q < n; q += BLOCK << E.split_shift) {
        prim::Bucket b;
        b.number = first;
        b.low_bits = E.low_bits;
        int at = q;
#pragma unroll
        for (int j = 0; j + 1 < 1 << UNIQUE_JOIN_MAX; ++j)
            if (q >= upto[j]) {  // (beyond the joined ones upto is n)
                b.number = first + j + 1;
                at = q - upto[j];
            }
        const u64 k = b.whole(keys[E.starts[b.number] + (u32)at]);
        const int u = (int)(k >> vbits), v = (int)(k & vmask), e = before + q;
        const u32 ck = cost_key(pair_cost<PLACE>(load_vertex(vrec, u), load_vertex(vrec, v), rcond_min));
        const bool act = mt.active[mesh_of(mt.voff, mt.B, u)] != 0;
        ekey[e] = k;
        ecost[e] = ck;
        if (estate) estate[e] = act ? 0 : 1;
        if (act) {
            bids.put(vmin0, nullptr, u, edge_bid<SHUFFLE>(tb, ck, e, v));
            bids.put(vmin0, nullptr, v, edge_bid<SHUFFLE>(tb, ck, e, u));
        }
    }
    __syncthreads();
    bids.flush(vmin0, nullptr);
}

// ---------------------------------------------------------------------------
// S3: greedy disjoint grouping of Alg. 2 lines 3-10, computed in parallel.
//
// Priority of edge e = (cost key, e) packed in 64 bits; the sequential loop of
// the paper visits edges in ascending priority.  An edge is LIVE while neither
// end is paired.  A live edge whose priority is the minimum among the live
// edges at BOTH ends is exactly one the sequential loop accepts, so every
// sub-round accepts all such edges at once, retires the edges touching newly
// paired vertices, and lets the survivors bid again.  vmin buffers rotate:
// sub-round k reads bids in vmin[k%3], places the survivors' bids in
// vmin[(k+1)%3] and clears their slots in vmin[(k+2)%3].
// ---------------------------------------------------------------------------
constexpr int TAIL_THREADS = 1024;
constexpr int TAIL_MAX = 3584;  // live edges the single-workgroup tail takes over (sized by its LDS state)

// A word in the context's pinned host memory and the number to store there: the last kernel
// before a look of the host stores it once its results are written, so that the host may watch
// that word instead of waiting for the stream.
struct HostSignal {
    int* word;
    int seq;
};

// By every thread of the (single) workgroup, as its last act: the workgroup's stores to host
// memory are complete before one thread stores the sequence number.  `wrote`: this thread has
// stored something the host will read (only those threads need the fence, which is not cheap).
__device__ __forceinline__ void signal_host(const HostSignal& h, int tid, bool wrote) {
    if (wrote) __threadfence_system();
    __syncthreads();
    if (tid == 0) __hip_atomic_store(h.word, h.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

constexpr u32 PAIR_NONE = 0xFFFFFFFFu;  // (no finite cost has this key)

// A live edge for the tail.
struct __attribute__((aligned(16))) LiveEdge {
    u64 key;
    u32 cost;
    int e;
};
constexpr int LIVE_SEGS = 32;  // (as the pair counters: the appending waves' atomics spread over cache lines)

struct SelArgs {
    const u64* ekey;
    const u32* ecost;
    u64* vmin[3];
    int* mate;
    u32* pcost;             // per pair, at its lower vertex: its cost key (PAIR_NONE at every other vertex),
    u32* ptie;              // ... and with shuffle its tie-break value: what the budget step goes by
    LiveEdge* live;         // the edges that the last grid-wide sub-round leaves live, for the tail: LIVE_SEGS segments of
    int live_cap;           // ... live_cap places each,
    int* live_n;            // ... filled up to live_n[segment * MATCH_PAD] (or fuller than full)
    unsigned char* estate;  // per edge: 0 = live, 1 = retired (paired, or an end was paired); in listed rounds only before sub-round 0,
                            // of one mesh, all of whose edges are live then, not at all (null: the kernels of a call of 10.2 M vertices 5,431 -> 5,384 us)
    int bound;              // edges of this round at most (no less than 1)
    u64* lkey;              // listed rounds: the live edges (key, cost key, with shuffle their numbers), see select_listed_kernel
    u32* lcost;
    int* lidx;
    int* lcount;
    int list_tile;          // ... places of the lists' tiles,
    int list_tiles;         // ... how many (0: as the round's edges fill)
    const int* fcur;        // rounds by facets (see facet_costs_kernel): the facets,
    const u32* fcost;       // ... their sides' cost keys, n_facets of each side
    const int* fcount;      // ... per tile how many of its places are taken (null: all),
    int n_facets, parts;    // ... the places, the workgroups' parts of facets and vertices,
    int nv;                 // ... vertices
    const int* nf_slots;    // ... facets that have not collapsed (null: State says so), in MATCH_SLOTS parts
    State* st;
    MeshTab mt;
    int vbits;
    int* host_img;     // pinned host memory, device view: the tail leaves [State][matched] there
    int publish_ints;  // for the host, which then needs no copy of its own before it looks
    int* host_check;   // ... and, behind them, the number that the kernel after it will store in the
    int host_seq;      // sequence word (the host compares the two before it trusts what it reads)
    TieBreak tb;       // order among edges of equal cost
    int cur;           // which of the ping-pong vertex / facet counts belong to this round
};

// N edges of one lane in one sub-round.  on: the edge is live (its ends' bids are then those of live edges); what the others hold is not looked
// at.  alive: it stays live, sel: it is accepted (both ends noted).  The best live edge at an end is accepted in this sub-round iff it
// is also the best at its other end.  Without branches: all lanes' loads of a step are in flight together.
template <bool SHUFFLE>
struct JudgedEdge {
    u64 key;
    u32 cost;
    int e, u, v;
    bool on, alive, sel;
    u64 pu, pv;  // its bids on its ends
};
template <bool SHUFFLE, int N>
__device__ __forceinline__ void judge_edges(const SelArgs& A, const u64* __restrict__ cur, JudgedEdge<SHUFFLE> (&E)[N]) {
    const u64 vmask = (1ull << A.vbits) - 1ull;
    u64 mu[N], mv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        E[j].u = E[j].on ? (int)(E[j].key >> A.vbits) : 0;
        E[j].v = E[j].on ? (int)(E[j].key & vmask) : 0;
        mu[j] = cur[E[j].u];
        mv[j] = cur[E[j].v];
    }
    int au[N], av[N];  // the ends' best edges' other ends
    if constexpr (SHUFFLE) {
        u64 ku[N], kv[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ku[j] = A.ekey[E[j].on && mu[j] != VMIN_NONE ? A.tb.dec((u32)mu[j]) : 0u];
            kv[j] = A.ekey[E[j].on && mv[j] != VMIN_NONE ? A.tb.dec((u32)mv[j]) : 0u];
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int a = (int)(ku[j] >> A.vbits), b = (int)(kv[j] >> A.vbits);
            au[j] = E[j].on ? (a == E[j].u ? (int)(ku[j] & vmask) : a) : 0;
            av[j] = E[j].on ? (b == E[j].v ? (int)(kv[j] & vmask) : b) : 0;
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            au[j] = E[j].on && mu[j] != VMIN_NONE ? (int)(u32)mu[j] : 0;
            av[j] = E[j].on && mv[j] != VMIN_NONE ? (int)(u32)mv[j] : 0;
        }
    }
    u64 bu[N], bv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        bu[j] = cur[au[j]];
        bv[j] = cur[av[j]];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        JudgedEdge<SHUFFLE>& x = E[j];
        x.pu = edge_bid<SHUFFLE>(A.tb, x.cost, x.e, x.v);
        x.pv = edge_bid<SHUFFLE>(A.tb, x.cost, x.e, x.u);
        x.sel = x.on && mu[j] == x.pu && mv[j] == x.pv;
        const bool gone_u = SHUFFLE ? bu[j] == mu[j] : bu[j] == ((mu[j] & 0xFFFFFFFF00000000ull) | (u32)x.u);
        const bool gone_v = SHUFFLE ? bv[j] == mv[j] : bv[j] == ((mv[j] & 0xFFFFFFFF00000000ull) | (u32)x.v);
        x.alive = x.on && !x.sel && !gone_u && !gone_v;
        if (x.sel) {
            A.mate[x.u] = x.v;
            A.mate[x.v] = x.u;
            A.pcost[x.u] = x.cost;
            if constexpr (SHUFFLE) A.ptie[x.u] = (u32)x.pu;
        }
    }
}

// pairs formed, counted per mesh: one atomic per wave and mesh
__device__ __forceinline__ void count_pairs(const SelArgs& A, bool sel, int m) {
    const int lane = prim::lane_id();
    u64 sb = prim::ballot(sel);
    while (sb) {
        const int leader = __ffsll((long long)sb) - 1;
        const int m0 = __shfl(m, leader, 64);
        const u64 same = prim::ballot(sel && m == m0);
        if (lane == leader)
            atomicAdd(&A.mt.mslots[((size_t)m0 * MATCH_SLOTS + (blockIdx.x & (MATCH_SLOTS - 1))) * MATCH_PAD],
                      (int)__popcll(same));
        sb &= ~same;
    }
}

// The same for a workgroup whose pairs nearly all belong to one mesh (edges are in mesh order): that mesh's are put together in LDS
// and added by one atomic in the end.  (The counters of a mesh lie in MATCH_SLOTS lines, and a line takes an atomic every
// 11 to 14 ns: with one per wave they took longer than the rest of a sub-round, 150 of 420 us at 30 M edges.)
struct PairTally {
    int mesh, first, end_v, pairs;  // the mesh and its vertices
    // by one thread; v = a vertex of the mesh
    __device__ __forceinline__ void begin(const SelArgs& A, int v) {
        mesh = mesh_of(A.mt.voff, A.mt.B, v);
        first = A.mt.B <= 1 ? 0 : A.mt.voff[mesh];
        end_v = A.mt.B <= 1 ? 0x7FFFFFFF : A.mt.voff[mesh + 1];
        pairs = 0;
    }
    // by all lanes of a wave; u = an end of the pair
    __device__ __forceinline__ void count(const SelArgs& A, bool sel, int u) {
        const bool here = u >= first && u < end_v;
        const u64 mine = prim::ballot(sel && here);
        if (mine && prim::lane_id() == 0) atomicAdd(&pairs, (int)__popcll(mine));
        if (A.mt.B > 1 && __any(sel && !here)) count_pairs(A, sel && !here, sel && !here ? mesh_of(A.mt.voff, A.mt.B, u) : 0);
    }
    // by one thread, behind a barrier
    __device__ __forceinline__ void end(const SelArgs& A) const {
        if (pairs) atomicAdd(&A.mt.mslots[((size_t)mesh * MATCH_SLOTS + (blockIdx.x & (MATCH_SLOTS - 1))) * MATCH_PAD], pairs);
    }
};

// The lanes' live edges appended to their workgroup's segment of the tail's list.  By all lanes of a wave.
__device__ __forceinline__ void append_live(const SelArgs& A, bool alive, u64 key, u32 cost, int e) {
    const u64 b = prim::ballot(alive);
    if (b == 0) return;
    const int seg = blockIdx.x & (LIVE_SEGS - 1), first = __ffsll((long long)b) - 1;
    int at = 0;
    if (prim::lane_id() == first) at = atomicAdd(&A.live_n[seg * MATCH_PAD], (int)__popcll(b));
    at = __shfl(at, first, 64) + (int)__popcll(b & prim::lanemask_lt());
    if (alive && at < A.live_cap) A.live[(size_t)seg * A.live_cap + at] = LiveEdge{key, cost, e};
}

// The same for the small rounds: one mesh's pairs put together in LDS, a batch's counted in memory by one atomic per wave and mesh; the
// meshes' first vertices are fetched beforehand, as the search among them is a chain of loads.
constexpr int TALLY_MESHES = 64;
struct SmallTally {
    int pairs, voff[TALLY_MESHES + 1];
    // by the workgroup, in front of a barrier
    __device__ __forceinline__ void begin(const SelArgs& A) {
        const int t = threadIdx.x;
        if (t == 0) pairs = 0;
        if (A.mt.B > 1 && A.mt.B <= TALLY_MESHES && t <= A.mt.B) voff[t] = A.mt.voff[t];
    }
    // by all lanes of a wave; u = an end of the pair
    __device__ __forceinline__ void count(const SelArgs& A, bool sel, int u) {
        const u64 mine = prim::ballot(sel);
        if (mine == 0) return;
        if (A.mt.B == 1) {
            if (prim::lane_id() == 0) atomicAdd(&pairs, (int)__popcll(mine));
        } else {
            int m = 0;
            if (sel) m = A.mt.B <= TALLY_MESHES ? mesh_of(voff, A.mt.B, u) : mesh_of(A.mt.voff, A.mt.B, u);
            count_pairs(A, sel, m);
        }
    }
    // by one thread, behind a barrier
    __device__ __forceinline__ void end(const SelArgs& A) const {
        if (pairs) atomicAdd(&A.mt.mslots[(size_t)(blockIdx.x & (MATCH_SLOTS - 1)) * MATCH_PAD], pairs);
    }
};

// Grid-wide sub-round over ALL edges of a round of less than LISTED_MIN_EDGES; retired edges are skipped by
// their state byte.  The last one before the tail (APPEND), which leaves a few thousand edges live, lists them for it.
// Bound by the launch and the chain of loads (count, key, cost and state; the ends' bids; their best edges' other ends' bids): each is
// asked for without waiting for the one in front of it where it can be (115 k: the eight of them 54 -> 45 us).
constexpr int SUBROUND_LINES = 128;
template <bool SHUFFLE, bool APPEND>
__global__ __launch_bounds__(BLOCK) void select_subround_kernel(SelArgs A, int k) {
    const u64* __restrict__ cur = A.vmin[k % 3];
    u64* __restrict__ nxt = A.vmin[(k + 1) % 3];
    u64* __restrict__ rst = A.vmin[(k + 2) % 3];
    __shared__ BidTable<SUBROUND_LINES> bids;
    __shared__ SmallTally tally;
    const int i = (int)blockIdx.x * BLOCK + (int)threadIdx.x, at = min(i, A.bound - 1);  // (the grid covers the bound)
    const u64 key = A.ekey[at];  // (not yet known to be an edge: the loads do not wait for one another)
    const u32 cost = A.ecost[at];
    const bool retired = A.estate[at] != 0;
    const int n = A.st->ne;
    if (i == 0) A.st->sel_k = k + 1;
    if ((int)blockIdx.x * BLOCK >= n) return;
    bids.clear();
    tally.begin(A);
    JudgedEdge<SHUFFLE> E[1];
    E[0].key = key;
    E[0].cost = cost;
    E[0].e = i;
    E[0].on = i < n && !retired;
    judge_edges<SHUFFLE, 1>(A, cur, E);
    const JudgedEdge<SHUFFLE>& x = E[0];
    __syncthreads();
    tally.count(A, x.sel, x.u);
    if (x.alive) {
        bids.put(nxt, rst, x.u, x.pu);
        bids.put(nxt, rst, x.v, x.pv);
    } else if (x.on) {
        A.estate[i] = 1;
    }
    if (APPEND) append_live(A, x.alive, key, cost, i);
    __syncthreads();
    bids.flush(nxt, rst);
    if (threadIdx.x == 0) tally.end(A);
}

// Large rounds: every sub-round lists the edges it leaves live (key, cost key, number) for the next, so that each reads
// 16 bytes per live edge in a row, where a walk over all edges' states fetched the keys and costs of a few per cent of them
// line by line.  A workgroup has a part of the edges to itself, its part of the lists is the same places of lkey, lcost and lidx, and
// it leaves their number in lcount: no counter is shared.  Sub-round 0 takes all edges, LISTED_TILE to a workgroup; a
// later one takes `group` parts of 2^part_shift tiles together and joins what is left of them (in place: a live
// edge's new place is never behind its old one).  Bound by memory and by the bids' atomics; sub-round 0 has four edges per lane in
// flight, the others two.  10.2 M vertices, 31 M edges: the first round's seven sub-rounds 967 -> 740 us, all three rounds' 1,800 -> 1,380;
// 1.2 M: 117 -> 95 and 253 -> 205.  Bids put together in LDS in the first three sub-rounds, while several live edges share a line of vertices
// (the third: 126 -> 122 us, 1.2 M 16.1 -> 13.9; the fourth no faster).
constexpr int LISTED_MIN_EDGES = 1 << 20;  // below this the sub-rounds are at their launch floor anyway
constexpr int LISTED_TILE_SHIFT = 10, LISTED_TILE = 1 << LISTED_TILE_SHIFT, LISTED_PER_LANE = LISTED_TILE / BLOCK;
constexpr int LISTED_GROUP_MAX = 4;
constexpr int LISTED_LINES = 256;
// How many parts sub-round k >= 1 joins, and how many tiles a part is (bits), of `tiles` tiles: a workgroup has a few hundred live edges every time
// where these get fewer as on surfaces of varied costs.  Where they hardly do (ties: on a flat lattice of 200 x 200 vertices a round takes 299
// sub-rounds), joining on would leave the whole chip's work to a few workgroups (five there, 230 us a sub-round), so that at
// least LISTED_GROUPS_MIN workgroups are left, one for every compute unit.  (With 512 flat lattices of 115 k and 400 k vertices, to a quarter, take
// 10.9 and 27.8 ms for 11.4 and 37.0, but those with varied costs 241 us for 235, 2 M 1,028 for 1,021, 16 meshes of 60 k 581 for 577.)
constexpr int LISTED_GROUPS_MIN = 256;
inline int listed_group_shift(int k, int part_shift, int tiles) {
    int shift = k <= 3 ? 1 : 2;
    while (shift > 0 && ((tiles - 1) >> (part_shift + shift)) + 1 < LISTED_GROUPS_MIN) --shift;
    return shift;
}
inline int listed_part_shift(int k, int tiles) {
    int shift = 0;
    for (int j = 1; j < k; ++j) {
        const int more = listed_group_shift(j, shift, tiles);
        if (more == 0) break;  // (and none from here on)
        shift += more;
    }
    return shift;
}

// Places of the lanes' live edges among the workgroup's (N per lane, wave by wave); total = their number.  Contains barriers.
template <int N, int NWAVES = prim::WAVES>
__device__ __forceinline__ void live_places(const bool (&alive)[N], u32* smem, int (&place)[N], int& total) {
    const int w = prim::wave_id();
    u32 run = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const u64 b = prim::ballot(alive[j]);
        place[j] = (int)(run + prim::mask_below(b));
        run += (u32)__popcll(b);
    }
    __syncthreads();
    if (prim::lane_id() == 0) smem[w] = run;
    __syncthreads();
    u32 before = 0, all = 0;
#pragma unroll
    for (int j = 0; j < NWAVES; ++j) {
        const u32 c = smem[j];
        if (j < w) before += c;
        all += c;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) place[j] += (int)before;
    total = (int)all;
}

template <bool SHUFFLE, bool APPEND>
__global__ __launch_bounds__(BLOCK) void select_first_kernel(SelArgs A) {
    constexpr int N = LISTED_PER_LANE;
    const u64* __restrict__ cur = A.vmin[0];
    u64* __restrict__ nxt = A.vmin[1];
    u64* __restrict__ rst = A.vmin[2];
    __shared__ BidTable<LISTED_LINES> bids;
    __shared__ PairTally tally;
    __shared__ u32 smem[prim::WAVES];
    const int n = A.st->ne;
    if (blockIdx.x == 0 && threadIdx.x == 0) A.st->sel_k = 1;
    const int tile = prim::xcd_tile(n, LISTED_TILE);
    const long long base = (long long)tile << LISTED_TILE_SHIFT;
    if (base >= n) return;
    const int i0 = (int)base + prim::wave_id() * (64 * N) + prim::lane_id();
    JudgedEdge<SHUFFLE> E[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int i = i0 + j * 64, at = min(i, n - 1);
        E[j].e = i;
        E[j].key = A.ekey[at];
        E[j].cost = A.ecost[at];
        E[j].on = i < n;
    }
    if (A.estate)
#pragma unroll
        for (int j = 0; j < N; ++j) E[j].on = A.estate[min(i0 + j * 64, n - 1)] == 0 && E[j].on;
    bids.clear();
    if (threadIdx.x == 0) tally.begin(A, (int)(E[0].key >> A.vbits));
    judge_edges<SHUFFLE, N>(A, cur, E);
    bool alive[N];
    int place[N], total;
#pragma unroll
    for (int j = 0; j < N; ++j) alive[j] = E[j].alive;
    live_places<N>(alive, smem, place, total);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const JudgedEdge<SHUFFLE>& x = E[j];
        tally.count(A, x.sel, x.u);
        if (x.alive) {
            const size_t p = (size_t)base + (size_t)place[j];
            A.lkey[p] = x.key;
            A.lcost[p] = x.cost;
            if constexpr (SHUFFLE) A.lidx[p] = x.e;
            bids.put(nxt, rst, x.u, x.pu);
            bids.put(nxt, rst, x.v, x.pv);
        }
        if (APPEND) append_live(A, x.alive, x.key, x.cost, x.e);
    }
    __syncthreads();
    bids.flush(nxt, rst);
    if (threadIdx.x == 0) {
        A.lcount[tile] = total;
        tally.end(A);
    }
}

// ---------------------------------------------------------------------------
// Rounds by facets: S1, S2 and the first bids without a list of the distinct edges.
//
// Where nothing needs the edges' numbers (ties that go by the shuffle, line 11, the statistics) an edge may as well be met once per facet that has
// it: its cost is the same to the bit each time, and bids are minima.  So one kernel takes the facets to the round's numbering, as
// edge_keys_kernel does, fetches each facet's three vertex records, and leaves the cost keys of its three sides and the better of a vertex's
// two bids; the sort of the half-edges (partition and per-bucket kernel) and unique_cost_kernel, which number the distinct
// ones, do not run.  Facets that have collapsed leave their tile, so that each round reads what the one before has left.
// Bound by memory: the first round's launch moves 1.55 GB of 10.2 M vertices / 20 M facets in 353 us (4.4 TB/s), later ones wait
// for a chain of gathers (346 and 285 us; six waves a SIMD, hence the bound on registers (409 and 321 without), and workgroups as small as can be:
// tiles of 1,024 facets by 256 lanes took 343 and 299, by 512 lanes 429 and 366, tiles of 512 by 128 lanes with twice the table 361 and 315).
// Rounds 2 and 3 of that mesh took 686 and 565 us up to the first bids with the sort, 227 k facets 32 us of round 2, now 9; whole calls with the
// sort / by facets: 4 k vertices 178 / 155 us, 115 k 213 / 189, 1.2 M 848 / 702, 10.2 M 5,400 / 4,720.
// ---------------------------------------------------------------------------
// What a workgroup wants to know of the meshes: of up to TALLY_MESHES from LDS, as a search is a chain of loads.
struct MeshFlags {
    int voff[TALLY_MESHES + 1];
    unsigned char active[TALLY_MESHES], done[TALLY_MESHES];
    // by the workgroup, in front of a barrier
    __device__ __forceinline__ void begin(const RoundTab& R, const int* __restrict__ done_) {
        const int t = threadIdx.x;
        if (R.B > TALLY_MESHES) return;
        if (t <= R.B) voff[t] = R.voff[t];
        if (t < R.B) {
            active[t] = mesh_active(R, t) ? 1 : 0;
            done[t] = done_ && done_[t] != 0 ? 1 : 0;
        }
    }
    __device__ __forceinline__ bool is_active(const RoundTab& R, int v) const {
        return R.B <= TALLY_MESHES ? active[mesh_of(voff, R.B, v)] != 0 : mesh_active(R, mesh_of(R.voff, R.B, v));
    }
    __device__ __forceinline__ bool is_done(const RoundTab& R, const int* __restrict__ done_, int v) const {
        return R.B <= TALLY_MESHES ? done[mesh_of(voff, R.B, v)] != 0 : done_[mesh_of(R.voff, R.B, v)] != 0;
    }
};

// The facets stand in tiles of THREADS * PER places, each with its own at the front, in order, `fcount` of them (null: all places
// are taken): a collapsed facet leaves its tile.
template <int PLACE, int THREADS, int PER, bool FIRST>
__global__ __launch_bounds__(THREADS, FIRST ? 1 : 6) void facet_costs_kernel(int* __restrict__ fcur, int F, State* st, int cur,
                                                              const VRec* __restrict__ vrec, u64* __restrict__ vmin0,
                                                              u64* __restrict__ vmin1, u32* __restrict__ fcost, RoundTab R,
                                                              const int* __restrict__ vmap, const int* __restrict__ done,
                                                              int* __restrict__ cid, int n_orig, float rcond_min,
                                                              const int* fcount, int* fcount_out, int* __restrict__ nf_slots,
                                                              int* __restrict__ nf_next) {
    constexpr int TILE = THREADS * PER, WAVES = THREADS / 64;
    __shared__ BidTable<!FIRST && THREADS == 128 ? 64 : 128, THREADS> bids;
    __shared__ MeshFlags M;
    __shared__ int at[FIRST ? 1 : 3][FIRST ? 1 : TILE];  // the corners of those left
    __shared__ int left[PER][WAVES];
    const int t = threadIdx.x, stride = gridDim.x * THREADS, g = blockIdx.x * THREADS + t;
    const int tile = prim::xcd_tile(F, TILE);
    const long long f0 = (long long)tile * TILE;
    int n = (int)max(min((long long)F - f0, (long long)TILE), 0ll);
    Corners q[PER];
    int label = 0;
    if constexpr (FIRST) {
#pragma unroll
        for (int j = 0; j < PER; ++j) q[j] = load_corners(fcur, (size_t)(j * THREADS + t < n ? f0 + j * THREADS + t : 0));
    } else {
        // (not yet known to be one; within the tile, as the others' workgroups rewrite theirs)
        if (PER == 1 && t < n) q[0] = load_corners(fcur, (size_t)(f0 + t));
        if (g < n_orig) label = cid[g];
        const int nv = st->nv[cur];
        if (fcount && n > 0) n = fcount[tile];
        if (PER > 1)
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (j * THREADS + t < n) q[j] = load_corners(fcur, (size_t)(f0 + j * THREADS + t));
        for (int w = g; w < nv; w += stride) vmin1[w] = VMIN_NONE;
        if (blockIdx.x == 0) round_begin_block(R, st);
    }
    if (blockIdx.x == 0 && t < MATCH_SLOTS) nf_next[t * MATCH_PAD] = 0;
    bids.clear();
    M.begin(R, FIRST ? nullptr : done);
    __syncthreads();
    if constexpr (!FIRST) {
        bool ok[PER];
        Corners m[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            ok[j] = j * THREADS + t < n && q[j].a >= 0;
            if (PER == 1 || ok[j]) m[j] = Corners{vmap[ok[j] ? q[j].a : 0], vmap[ok[j] ? q[j].b : 0], vmap[ok[j] ? q[j].c : 0]};
        }
        if (g < n_orig) cid[g] = vmap[label];
        u64 bal[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (ok[j] && (m[j].a == m[j].b || m[j].b == m[j].c || m[j].a == m[j].c)) ok[j] = !M.is_done(R, done, m[j].a);
            bal[j] = prim::ballot(ok[j]);
            if (prim::lane_id() == 0) left[j][prim::wave_id()] = (int)__popcll(bal[j]);
        }
        __syncthreads();  // (behind it all of the tile has been read, too)
        int before = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            int mine = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                if (w == prim::wave_id()) mine = before;
                before += left[j][w];
            }
            if (ok[j]) {
                const int p = mine + (int)prim::mask_below(bal[j]);
                at[0][p] = m[j].a; at[1][p] = m[j].b; at[2][p] = m[j].c;
                int* o = fcur + 3 * (size_t)(f0 + p);
                o[0] = m[j].a; o[1] = m[j].b; o[2] = m[j].c;
            }
        }
        if (t == 0 && n > 0) fcount_out[tile] = before;
        n = before;
        __syncthreads();
    }
    auto facet = [&](size_t f, const Corners& p) {
        if (R.B > 1 && !M.is_active(R, p.a)) return;
        const VertexWords A = load_vertex(vrec, p.a), B = load_vertex(vrec, p.b), C = load_vertex(vrec, p.c);
        const u32 ab = cost_key(pair_cost<PLACE>(A, B, rcond_min)), bc = cost_key(pair_cost<PLACE>(B, C, rcond_min)),
                  ca = cost_key(pair_cost<PLACE>(C, A, rcond_min));
        fcost[f] = ab;
        fcost[(size_t)F + f] = bc;
        fcost[2 * (size_t)F + f] = ca;
        auto bid = [&](int u, int v, u32 cost) -> u64 { return u == v ? VMIN_NONE : ((u64)cost << 32) | (u32)v; };
        auto put = [&](int v, u64 x, u64 y) {
            const u64 best = x < y ? x : y;
            if (best != VMIN_NONE) bids.put(vmin0, nullptr, v, best);
        };
        put(p.a, bid(p.a, p.b, ab), bid(p.a, p.c, ca));
        put(p.b, bid(p.b, p.c, bc), bid(p.b, p.a, ab));
        put(p.c, bid(p.c, p.a, ca), bid(p.c, p.b, bc));
    };
    if constexpr (FIRST) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (j * THREADS + t < n) facet((size_t)(f0 + j * THREADS + t), q[j]);
    } else {
#pragma unroll 1
        for (int i = t; i < n; i += THREADS) facet((size_t)(f0 + i), Corners{at[0][i], at[1][i], at[2][i]});
    }
    if constexpr (!FIRST)
        for (int o = g + stride; o < n_orig; o += stride) cid[o] = vmap[cid[o]];
    __syncthreads();
    bids.flush(vmin0, nullptr);
    if (!FIRST && t == 0 && n > 0) atomicAdd(&nf_slots[(blockIdx.x & (MATCH_SLOTS - 1)) * MATCH_PAD], n);
}

// The distinct edges of such a round, for the statistics: the sides of the facets entered into a set (open addressing over `slots` >= 6 F slots,
// all EDGE_NONE beforehand, so that at least half stay free), those that were not there yet counted.
constexpr u64 EDGE_NONE = ~0ull;
__global__ __launch_bounds__(BLOCK) void count_edges_kernel(const int* __restrict__ fcur, int F, const int* __restrict__ fcount,
                                                            int tile_shift, u64* __restrict__ set, u64 slots, int* __restrict__ ne) {
    int fresh = 0;
    for (long long f = (long long)blockIdx.x * BLOCK + threadIdx.x; f < F; f += (long long)gridDim.x * BLOCK) {
        if (fcount && (int)(f & ((1 << tile_shift) - 1)) >= fcount[f >> tile_shift]) continue;
        const Corners q = load_corners(fcur, (size_t)f);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int a = corner(q, c), b = corner(q, c == 2 ? 0 : c + 1);
            if (a == b) continue;
            const u64 key = ((u64)(u32)min(a, b) << 32) | (u64)(u32)max(a, b);
            for (u64 h = __umul64hi(key * 0x9E3779B97F4A7C15ull, slots);; h = h + 1 == slots ? 0 : h + 1) {
                const u64 there = atomicCAS(&set[h], EDGE_NONE, key);
                fresh += there == EDGE_NONE ? 1 : 0;
                if (there == EDGE_NONE || there == key) break;
            }
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) fresh += __shfl_xor(fresh, d, 64);
    if (prim::lane_id() == 0 && fresh) atomicAdd(ne, fresh);
}

// The pairs formed so far, counted by their lower vertices, COUNT_VERTICES to a workgroup.  A vertex is paired if it has a partner already, or if
// in the sub-round of this launch (whose bids are `cur`) the best bid on it names a vertex whose best bid names it; its partner is then being
// written by other workgroups.  Old bids do no harm: an edge of which both ends hold the bid bid on both in one sub-round, in which it was accepted.
constexpr int COUNT_VERTICES = 4 * BLOCK;
__device__ __forceinline__ void count_paired(const SelArgs& A, const u64* __restrict__ cur, PairTally& tally, int part) {
    const int nv = A.st->nv[A.cur], t = threadIdx.x;
    const long long v0 = (long long)part * COUNT_VERTICES;
    if (v0 >= nv) return;
    int m[4];
    u64 b[4], back[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int w = (int)min(v0 + j * BLOCK + t, (long long)nv - 1);
        m[j] = A.mate[w];
        b[j] = cur[w];
    }
    if (t == 0) tally.begin(A, (int)v0);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) back[j] = cur[m[j] < 0 && b[j] != VMIN_NONE ? (int)(u32)b[j] : 0];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const long long w = v0 + j * BLOCK + t;
        const bool now = b[j] != VMIN_NONE && back[j] == ((b[j] & 0xFFFFFFFF00000000ull) | (u32)w);
        const int p = m[j] >= 0 ? m[j] : now ? (int)(u32)b[j] : -1;
        tally.count(A, w < nv && p > w, (int)w);
    }
    __syncthreads();
    if (t == 0) tally.end(A);
}

// Sub-round 0 of such a round.  A vertex is paired if the best bid on it names a vertex whose best bid names it: said by the vertices
// (which also start the pairs' arrays).  A facet's side stays live if neither of its ends is paired; the workgroup leaves its
// live sides as a list, as select_listed_kernel takes them, without those that it also has the other way round (a table of
// the sides from the lower to the higher end, in which one may take another's place: copies do no harm).
template <int THREADS, int PER, bool APPEND>
__global__ __launch_bounds__(THREADS) void select_facets_kernel(SelArgs A) {
    constexpr int TILE = THREADS * PER, N = 3 * PER, SIDES = PER == 1 ? 1024 : 4 * THREADS;
    const u64* __restrict__ cur = A.vmin[0];
    u64* __restrict__ nxt = A.vmin[1];
    __shared__ BidTable<PER == 1 ? 128 : THREADS / 2, THREADS> bids;
    __shared__ u64 side[SIDES];
    __shared__ PairTally tally;
    __shared__ u32 smem[THREADS / 64];
    const int t = threadIdx.x;
    if (blockIdx.x == 0 && t == 0) A.st->sel_k = 1;
    const int part = prim::xcd_item((int)blockIdx.x, A.parts);
    if (part >= A.parts) return;
    const long long f0 = (long long)part * TILE;
    int n = (int)max(min(A.n_facets - f0, (long long)TILE), 0ll);
    const int nv = A.st->nv[A.cur];
    Corners q[PER];
    u32 cost[PER][3];
    auto load = [&](int j) {
        const size_t f = (size_t)(j * THREADS + t < n ? f0 + j * THREADS + t : 0);
        q[j] = load_corners(A.fcur, f);
#pragma unroll
        for (int c = 0; c < 3; ++c) cost[j][c] = A.fcost[(size_t)c * A.n_facets + f];
    };
    if (PER == 1) load(0);  // (not yet known to be one)
    if (A.fcount && n > 0) n = A.fcount[part];
    if (PER > 1)
#pragma unroll
        for (int j = 0; j < PER; ++j) load(j);
    const int per = ((nv - 1) / A.parts + 64) & ~63, v0 = (int)min((long long)part * per, (long long)nv), v1 = min(v0 + per, nv);
    auto vertex_bid = [&](int w) -> u64 { return w < v1 ? cur[w] : VMIN_NONE; };
    auto partner_bid = [&](u64 m) -> u64 { return cur[m != VMIN_NONE ? (int)(u32)m : 0]; };
    auto vertex = [&](int w, u64 m, u64 back) {
        const int p = (int)(u32)m;
        const bool paired = m != VMIN_NONE && back == ((m & 0xFFFFFFFF00000000ull) | (u32)w);
        if (w < v1) {
            A.mate[w] = paired ? p : -1;
            A.pcost[w] = paired && w < p ? (u32)(m >> 32) : PAIR_NONE;
            A.vmin[2][w] = VMIN_NONE;
        }
        if (APPEND) tally.count(A, paired && w < p, w);
    };
    const u64 m0 = vertex_bid(v0 + t);
    bids.clear();
    for (int i = t; i < SIDES; i += THREADS) side[i] = 0;  // (no side's key)
    if (APPEND && t == 0) tally.begin(A, min(v0, nv - 1));
    u64 best[PER][3], back[PER][3];
    bool ok[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        ok[j] = j * THREADS + t < n && q[j].a >= 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) best[j][c] = cur[ok[j] ? corner(q[j], c) : 0];
    }
    const u64 back0 = partner_bid(m0);
#pragma unroll
    for (int j = 0; j < PER; ++j)
#pragma unroll
        for (int c = 0; c < 3; ++c) back[j][c] = partner_bid(best[j][c]);
    __syncthreads();
    vertex(v0 + t, m0, back0);
    for (int w0 = v0 + THREADS; w0 < v1; w0 += THREADS) {  // (few facets)
        const u64 m = vertex_bid(w0 + t);
        vertex(w0 + t, m, partner_bid(m));
    }
    bool alive[N], up[N];
    u64 key[N];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        bool open[3];
        u64 bid_out[3], bid_in[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            open[c] = ok[j] && best[j][c] != VMIN_NONE && back[j][c] != ((best[j][c] & 0xFFFFFFFF00000000ull) | (u32)corner(q[j], c));
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int d = c == 2 ? 0 : c + 1, a = corner(q[j], c), b = corner(q[j], d);
            const bool on = open[c] && open[d] && a != b;
            alive[3 * j + c] = on;
            up[3 * j + c] = a < b;
            key[3 * j + c] = ((u64)(u32)min(a, b) << A.vbits) | (u64)(u32)max(a, b);
            bid_out[c] = on ? ((u64)cost[j][c] << 32) | (u32)b : VMIN_NONE;  // on its start, on its end
            bid_in[d] = on ? ((u64)cost[j][c] << 32) | (u32)a : VMIN_NONE;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const u64 b = bid_out[c] < bid_in[c] ? bid_out[c] : bid_in[c];
            if (b != VMIN_NONE) bids.put(nxt, nullptr, corner(q[j], c), b);
        }
    }
    auto place_of = [&](u64 k) -> u32 { return (((u32)k ^ (u32)(k >> 32)) * 0x9E3779B1u >> 16) & (u32)(SIDES - 1); };
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (alive[i] && up[i]) side[place_of(key[i])] = key[i];
    __syncthreads();
    bool emit[N];
    int place[N], total;
#pragma unroll
    for (int i = 0; i < N; ++i) emit[i] = alive[i] && (up[i] || side[place_of(key[i])] != key[i]);
    live_places<N, THREADS / 64>(emit, smem, place, total);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (emit[i]) {
            const size_t p = (size_t)part * (3 * TILE) + (size_t)place[i];
            A.lkey[p] = key[i];
            A.lcost[p] = cost[i / 3][i % 3];
        }
        if (APPEND) append_live(A, emit[i], key[i], cost[i / 3][i % 3], 0);
    }
    bids.flush(nxt, nullptr);
    if (t == 0) {
        if (part == 0 || f0 < A.n_facets) A.lcount[part] = total;
        if (APPEND) tally.end(A);
    }
}

// COPIES: an edge may be listed more than once (rounds by facets), so pairs are not counted edge by edge: the last sub-round, which lists for
// the tail, has workgroups beside those with edges (list_groups of them) that count them vertex by vertex.
template <bool SHUFFLE, bool COPIES, bool APPEND, bool TABLE>
__global__ __launch_bounds__(BLOCK) void select_listed_kernel(SelArgs A, int k, int part_shift, int group, int list_groups) {
    constexpr int N = 2;
    constexpr bool COUNT = !COPIES;
    const u64* __restrict__ cur = A.vmin[k % 3];
    u64* __restrict__ nxt = A.vmin[(k + 1) % 3];
    u64* __restrict__ rst = A.vmin[(k + 2) % 3];
    __shared__ BidTable<TABLE ? LISTED_LINES : 1> bids;
    __shared__ PairTally tally;
    __shared__ u32 smem[prim::WAVES];
    const int t = threadIdx.x;
    if (COPIES && APPEND && (int)blockIdx.x >= list_groups) {
        count_paired(A, cur, tally, (int)blockIdx.x - list_groups);
        return;
    }
    const int tiles = COPIES ? A.list_tiles : (A.st->ne + LISTED_TILE - 1) / LISTED_TILE;
    const int cap = COPIES ? A.list_tile : LISTED_TILE;
    if (blockIdx.x == 0 && t == 0) A.st->sel_k = k + 1;
    const int parts = (tiles + (1 << part_shift) - 1) >> part_shift;
    const int first = prim::xcd_tile(parts, group) * group;  // (the first of the workgroup's parts)
    if (first >= parts) return;
    const size_t part_size = (size_t)cap << part_shift, base = (size_t)first * part_size;
    int* const count = A.lcount + ((size_t)first << part_shift);
    int upto[LISTED_GROUP_MAX], n_live = 0;
#pragma unroll
    for (int g = 0; g < LISTED_GROUP_MAX; ++g)
        upto[g] = n_live += g < group && first + g < parts ? count[(size_t)g << part_shift] : 0;
    if (n_live == 0) {
        if (t == 0) *count = 0;
        return;
    }
    if (TABLE) bids.clear();
    int left = 0;
    for (int q0 = 0; q0 < n_live; q0 += N * BLOCK) {
        JudgedEdge<SHUFFLE> E[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int q = q0 + j * BLOCK + t, at = min(q, n_live - 1);
            size_t p = base + (size_t)at;
#pragma unroll
            for (int g = 0; g + 1 < LISTED_GROUP_MAX; ++g)
                if (at >= upto[g]) p = base + (size_t)(g + 1) * part_size + (size_t)(at - upto[g]);
            E[j].key = A.lkey[p];
            E[j].cost = A.lcost[p];
            E[j].e = SHUFFLE ? A.lidx[p] : 0;
            E[j].on = q < n_live;
        }
        if (COUNT && q0 == 0 && t == 0) tally.begin(A, (int)(E[0].key >> A.vbits));
        judge_edges<SHUFFLE, N>(A, cur, E);
        bool alive[N];
        int place[N], total;
#pragma unroll
        for (int j = 0; j < N; ++j) alive[j] = E[j].alive;
        live_places<N>(alive, smem, place, total);  // (behind its barriers all of this turn's edges have been read)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const JudgedEdge<SHUFFLE>& x = E[j];
            if (COUNT) tally.count(A, x.sel, x.u);
            if (x.alive) {
                const size_t p = base + (size_t)(left + place[j]);
                A.lkey[p] = x.key;
                A.lcost[p] = x.cost;
                if constexpr (SHUFFLE) A.lidx[p] = x.e;
                if (TABLE) {
                    bids.put(nxt, rst, x.u, x.pu);
                    bids.put(nxt, rst, x.v, x.pv);
                } else {
                    atomicMin(&nxt[x.u], x.pu);
                    atomicMin(&nxt[x.v], x.pv);
                    rst[x.u] = VMIN_NONE;
                    rst[x.v] = VMIN_NONE;
                }
            }
            if (APPEND) append_live(A, x.alive, x.key, x.cost, x.e);
        }
        left += total;
    }
    __syncthreads();
    if (TABLE) bids.flush(nxt, rst);
    if (t == 0) {
        *count = left;
        if (COUNT) tally.end(A);
    }
}

// Tail: once few edges are live, one workgroup finishes the matching with all
// of its state in LDS: the live edges' priorities, a hash map from the (at
// most 2 x TAIL_MAX) vertices they touch to LDS slots, and one 64-bit bid per
// slot.  A sub-round then costs three workgroup barriers instead of a kernel
// launch and several trips to memory, and none once one wave holds the edges that are left.  The live count falls in every
// sub-round (the best live edge is always accepted), so the loop ends.  The bid of a slot whose vertex has been paired is TAIL_PAIRED from then on;
// a batch's pairs, of which there can be as many as edges came in, are marked and counted by mesh at the end (mesh by mesh in the loop the
// tails of 16 meshes took 13-22 us, now 9-15).
// (With six barriers, the list gathered by a launch of its own, and the loads of the end not started at the beginning:
// 14-19 us of every round of one mesh, now 9-16.  What is left is about 2 us per sub-round: the trips to LDS and the issue of 16 waves.
// Edges in registers instead of lists, and stores to memory kept out of the loop, measured the same.)
constexpr int TAIL_SLOTS = 8192;  // power of two, >= 2 * TAIL_MAX
constexpr int TAIL_LDS_MESHES = 1024;
constexpr int TAIL_FREE = -1;
constexpr u64 TAIL_PAIRED = 0;  // (less than any bid; also the priority of an edge that has been accepted, which is not looked at again)

struct TailLds {
    u64 prio[TAIL_MAX];
    u64 bid[TAIL_SLOTS];
    int vkey[TAIL_SLOTS];
    unsigned short su[TAIL_MAX], sv[TAIL_MAX];
    unsigned short lst[2][TAIL_MAX];
    int cnt[3];                  // live edges of the sub-round, of the next, of the one after that, in turn
    int seg_at[LIVE_SEGS + 1];   // first place of each segment's edges
    int nh;
    int pairs[TAIL_LDS_MESHES];  // pairs this kernel formed, per mesh (batches of up to this many meshes)
};
static_assert(sizeof(TailLds) <= 160 * 1024, "one workgroup's LDS");

__device__ __forceinline__ int tail_slot(int* vkey, int v) {
    u32 h = ((u32)v * 0x9E3779B1u) >> 19;  // 13 bits
    for (;;) {
        const int old = atomicCAS(&vkey[h], TAIL_FREE, v);
        if (old == TAIL_FREE || old == v) return (int)h;
        h = (h + 1) & (TAIL_SLOTS - 1);
    }
}

// A word for the host: stored at system scope (not left in a cache of the device), so that it is in
// host memory when the kernel has ended.
__device__ __forceinline__ void host_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// By every thread of the tail, after its last store for the host: once all of them are issued, the
// copy of the sequence number follows them.
__device__ __forceinline__ void tail_mark_published(const SelArgs& A, int tid) {
    __syncthreads();
    if (tid == 0) host_store(A.host_check, A.host_seq);
}

// The round's counters and pair counts, written straight into the host's pinned memory (read at
// the L2, where this kernel's own stores to them already are).
__device__ __forceinline__ void tail_publish(const SelArgs& A, int tid) {
    const int* hdr = reinterpret_cast<const int*>(A.st);
    constexpr int GO0 = (int)(offsetof(State, go) / sizeof(int)), STATE_INTS = (int)(sizeof(State) / sizeof(int));
    for (int i = tid; i < A.publish_ints; i += TAIL_THREADS)
        if (i < GO0 || i >= STATE_INTS)  // (the guard fields are for the device only; the tail is writing them)
            host_store(&A.host_img[i], __hip_atomic_load(&hdr[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// What the kernels queued behind the tail go by (see State).
__device__ __forceinline__ void tail_set_guard(const SelArgs& A, bool finished) {
    A.st->go = finished ? 1 : 0;
    A.st->guard_nv = finished ? A.st->nv[A.cur] : 0;
}

__global__ __launch_bounds__(TAIL_THREADS) void select_tail_kernel(SelArgs A) {
    __shared__ TailLds L;
    constexpr int NW = TAIL_THREADS / 64;
    const int tid = threadIdx.x, lane = prim::lane_id(), w = prim::wave_id();
    // what earlier kernels have left: asked for now, used at the end
    constexpr int LIVE0 = (int)(offsetof(State, live) / sizeof(int)), GO0 = (int)(offsetof(State, go) / sizeof(int));
    static_assert(GO0 <= TAIL_THREADS, "one thread per word");
    int hdr_word = tid < GO0 ? reinterpret_cast<const int*>(A.st)[tid] : 0;
    constexpr int NH = (int)(offsetof(State, nh) / sizeof(int));
    const int slot_pairs = tid < A.mt.B * MATCH_SLOTS ? A.mt.mslots[(size_t)tid * MATCH_PAD] : 0;
    if (A.nf_slots && w == 1) {  // (rounds by facets: half-edges there are)
        int n = lane < MATCH_SLOTS ? A.nf_slots[lane * MATCH_PAD] : 0;
#pragma unroll
        for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
        if (lane == 0) L.nh = 3 * n;
    }
    if (w == 0) {  // the segments' places
        const int c = lane < LIVE_SEGS ? A.live_n[lane * MATCH_PAD] : 0;
        const bool full = __any(c > A.live_cap);
        int incl = c;
#pragma unroll
        for (int d = 1; d < LIVE_SEGS; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        if (lane < LIVE_SEGS) L.seg_at[lane + 1] = incl;
        if (lane == 0) L.seg_at[0] = 0;
        if (lane == LIVE_SEGS - 1) L.cnt[0] = full ? max(incl, TAIL_MAX + 1) : incl;
    }
    if (tid == 0) L.cnt[1] = 0;
    for (int h = tid; h < TAIL_SLOTS / 4; h += TAIL_THREADS)
        reinterpret_cast<int4*>(L.vkey)[h] = make_int4(TAIL_FREE, TAIL_FREE, TAIL_FREE, TAIL_FREE);
    // Up to TAIL_LDS_MESHES meshes, the pairs formed here are tallied in LDS and added to the earlier
    // kernels' counters at the end; that way nothing this kernel writes to memory is read back by
    // it, and it needs no device-wide fence (which costs several microseconds here).
    const bool lds_pairs = A.mt.B <= TAIL_LDS_MESHES;
    if (lds_pairs)
        for (int b = tid; b < A.mt.B; b += TAIL_THREADS) L.pairs[b] = 0;
    __syncthreads();
    if (A.nf_slots && tid == NH) hdr_word = L.nh;
    int n = L.cnt[0];
    if (n > TAIL_MAX) {  // too many: the host runs more grid-wide sub-rounds, the last of which lists again
        if (tid < LIVE_SEGS) A.live_n[tid * MATCH_PAD] = 0;
        if (A.fcur)  // (rounds by facets: the last of them counts all pairs again)
            for (int i = tid; i < A.mt.B * MATCH_SLOTS; i += TAIL_THREADS) A.mt.mslots[(size_t)i * MATCH_PAD] = 0;
        if (tid == 0) {
            A.st->live[0] = n;
            tail_set_guard(A, false);
        }
        if (tid < GO0 && tid < A.publish_ints) host_store(&A.host_img[tid], tid == LIVE0 ? n : hdr_word);
        tail_mark_published(A, tid);
        return;
    }
    const int n_in = n;
    const u64 lt = prim::lanemask_lt();
    const u64 vmask = (1ull << A.vbits) - 1ull;
    for (int seg = w; seg < LIVE_SEGS; seg += NW) {
        const int s0 = L.seg_at[seg], m = L.seg_at[seg + 1] - s0;
        for (int j = lane; j < m; j += 64) {
            const LiveEdge E = A.live[(size_t)seg * A.live_cap + j];
            const int i = s0 + j, su = tail_slot(L.vkey, (int)(E.key >> A.vbits)), sv = tail_slot(L.vkey, (int)(E.key & vmask));
            L.prio[i] = A.tb.on ? A.tb.priority(E.cost, E.e) : (u64)E.cost << 32;
            L.su[i] = (unsigned short)su;
            L.sv[i] = (unsigned short)sv;
            L.lst[0][i] = (unsigned short)i;
            L.bid[su] = VMIN_NONE;
            L.bid[sv] = VMIN_NONE;
        }
    }
    __syncthreads();

    // the bids of an edge of priority p between the vertices u and v
    auto bid_on_u = [&](u64 p, int v) -> u64 { return A.tb.on ? p : p | (u32)v; };
    auto bid_on_v = [&](u64 p, int u) -> u64 { return A.tb.on ? p : p | (u32)u; };
    // an edge that holds the best bid at both ends is accepted; of several copies of it one is told so
    auto accept = [&](int i, int su, int sv, int u, int v, u64 p, bool& sel) {
        sel = L.bid[su] == bid_on_u(p, v) && L.bid[sv] == bid_on_v(p, u);
        if (sel) {
            A.mate[u] = v;
            A.mate[v] = u;
            A.pcost[min(u, v)] = (u32)(p >> 32);
            if (A.tb.on) A.ptie[min(u, v)] = (u32)p;
            sel = atomicExch(&L.bid[su], TAIL_PAIRED) != TAIL_PAIRED;  // (any other edge's bid differs from both values)
            L.bid[sv] = TAIL_PAIRED;
            if (A.mt.B > 1 && sel) L.prio[i] = TAIL_PAIRED;
        }
    };
    int wave_pairs = 0;  // (one mesh)
    // by all lanes of a wave (very many meshes: counted in memory)
    auto tally = [&](bool sel, int u) {
        if (A.mt.B == 1) wave_pairs += (int)__popcll(prim::ballot(sel));
        else if (!lds_pairs) count_pairs(A, sel, sel ? mesh_of(A.mt.voff, A.mt.B, u) : 0);
    };
    int side = 0, now = 0;  // cnt[now] = live edges, in lst[side]
    while (n > 64) {
        const int nxt = now == 2 ? 0 : now + 1, after = nxt == 2 ? 0 : nxt + 1;
        const int padded = (n + 63) & ~63;  // whole waves run each step so that the ballots are uniform
        if (tid == 0) L.cnt[after] = 0;
        for (int j = tid; j < n; j += TAIL_THREADS) {
            const int i = L.lst[side][j], su = L.su[i], sv = L.sv[i];
            const u64 p = L.prio[i];
            atomicMin(&L.bid[su], bid_on_u(p, L.vkey[sv]));
            atomicMin(&L.bid[sv], bid_on_v(p, L.vkey[su]));
        }
        __syncthreads();
        for (int j = tid; j < padded; j += TAIL_THREADS) {
            bool sel = false;
            int u = 0;
            if (j < n) {
                const int i = L.lst[side][j], su = L.su[i], sv = L.sv[i];
                u = L.vkey[su];
                accept(i, su, sv, u, L.vkey[sv], L.prio[i], sel);
            }
            tally(sel, u);
        }
        __syncthreads();
        // keep the edges whose ends are both still free, and clear those ends' bids
        for (int j = tid; j < padded; j += TAIL_THREADS) {
            bool alive = false;
            int i = 0;
            if (j < n) {
                i = L.lst[side][j];
                const int su = L.su[i], sv = L.sv[i];
                alive = L.bid[su] != TAIL_PAIRED && L.bid[sv] != TAIL_PAIRED;
                if (alive) L.bid[su] = L.bid[sv] = VMIN_NONE;
            }
            const u64 ab = prim::ballot(alive);
            if (ab) {
                int wbase = 0;
                if (lane == 0) wbase = atomicAdd(&L.cnt[nxt], (int)__popcll(ab));
                wbase = __shfl(wbase, 0, 64);
                if (alive) L.lst[side ^ 1][wbase + (int)__popcll(ab & lt)] = (unsigned short)i;
            }
        }
        __syncthreads();
        side ^= 1;
        now = nxt;
        n = L.cnt[now];
    }
    if (w == 0 && n > 0) {  // (a wave's LDS operations complete in order)
        bool alive = lane < n;
        const int i = alive ? L.lst[side][lane] : 0;
        const u64 p = alive ? L.prio[i] : 0;
        const int su = alive ? L.su[i] : 0, sv = alive ? L.sv[i] : 0, u = alive ? L.vkey[su] : 0, v = alive ? L.vkey[sv] : 0;
        while (__any(alive)) {
            if (alive) {
                atomicMin(&L.bid[su], bid_on_u(p, v));
                atomicMin(&L.bid[sv], bid_on_v(p, u));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
            bool sel = false;
            if (alive) accept(i, su, sv, u, v, p, sel);
            tally(sel, u);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
            alive = alive && L.bid[su] != TAIL_PAIRED && L.bid[sv] != TAIL_PAIRED;
            if (alive) L.bid[su] = L.bid[sv] = VMIN_NONE;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();

    static_assert(MATCH_SLOTS == 32, "a mesh's slots fill half a wave");
    constexpr int STATE_INTS = (int)(sizeof(State) / sizeof(int));
    if (A.mt.B == 1) {
        if (lane == 0 && wave_pairs) atomicAdd(&L.pairs[0], wave_pairs);
    } else if (lds_pairs) {
        for (int i = tid; i < n_in; i += TAIL_THREADS)
            if (L.prio[i] == TAIL_PAIRED) atomicAdd(&L.pairs[mesh_of(A.mt.voff, A.mt.B, L.vkey[L.su[i]])], 1);
    } else {
        __threadfence();  // the pair counts added above are at the L2 before they are summed
    }
    __syncthreads();
    // one lane per counter slot (a mesh's MATCH_SLOTS slots sit in neighbouring lanes), so that the
    // loads are in flight together; whole waves run each step for the shuffles
    for (int base = 0; base < A.mt.B * MATCH_SLOTS; base += TAIL_THREADS) {
        const int idx = base + tid;
        const bool ok = idx < A.mt.B * MATCH_SLOTS;
        int sum = 0;
        if (ok)  // (only this kernel's own additions, in memory where there are many meshes, came after the first load)
            sum = base == 0 && lds_pairs ? slot_pairs
                                         : __hip_atomic_load(&A.mt.mslots[(size_t)idx * MATCH_PAD], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if (ok && (idx & (MATCH_SLOTS - 1)) == 0) {
            const int b = idx / MATCH_SLOTS;
            if (lds_pairs) sum += L.pairs[b];
            A.mt.matched[b] = sum;
            if (lds_pairs && STATE_INTS + b < A.publish_ints) host_store(&A.host_img[STATE_INTS + b], sum);
        }
    }
    if (tid == 0) {
        A.st->live[0] = 0;
        if (A.nf_slots) A.st->nh = L.nh;
        tail_set_guard(A, true);
    }
    if (lds_pairs) {
        // the host's copy of the counters: everything but live[0] was written by earlier kernels
        if (tid < GO0 && tid < A.publish_ints) host_store(&A.host_img[tid], (tid == LIVE0) ? 0 : hdr_word);
    } else {
        __threadfence();
        __syncthreads();
        tail_publish(A, tid);
    }
    tail_mark_published(A, tid);
}

// The selection tail does not tell the host itself (a system-scope fence inside it, with the pairs it
// has just written still in the cache, costs more than a launch): the kernel after it on the stream
// does, as its first act, with a release store at system scope: what the kernels before that one
// have written is visible to it when it starts, so the release carries those writes along (there
// is next to nothing left in the cache to write back then, so it costs nothing measurable).  Either the first of the kernels queued ahead of the host's
// look (through the counting predicate's on_start) ...
__device__ __forceinline__ void tell_host(const HostSignal& done) {  // by one thread
    if (done.word) __hip_atomic_store(done.word, done.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <class Pred>
struct SignalingPred {
    Pred pred;
    HostSignal done;
    __device__ void on_start() const { tell_host(done); }
    __device__ bool operator()(int i) const { return pred(i); }
};
// ... or a kernel of its own.
__global__ void signal_kernel(HostSignal done) {
    if (threadIdx.x == 0) tell_host(done);
}

// ---------------------------------------------------------------------------
// Rounds by rings: S1 to S3 without a list of the edges, and the whole matching in one launch.
//
// A vertex's ring is the facets that have it, each as its other two corners (RingRows).  The quadrics' kernel leaves the rings of the input; a contraction's
// vertex takes over the rings of the two it was made of, in the new numbering, without the facets whose corners have met.  So no round after the first reads
// a facet, and every vertex has its edges at hand: ring_costs_kernel evaluates them once from either end (the same to the bit) and leaves the neighbours with
// their costs.
//
// The matching (Alg. 2 lines 3-10) is the one in which pairs are accepted in the order of (cost, edge); it is unique, and the edges at a vertex compare by
// (cost, other end).  suitor_kernel makes it the way of Manne and Halappanavar ("New effective multithreaded matching algorithms", IPDPS 2014): every vertex
// bids on its best neighbour; of two bids on a vertex the better one stays, the other's vertex goes on to its next best neighbour, whose bid it betters, and
// so on.  Bids only improve, so a neighbour that has refused a vertex once need not be asked again, no vertex waits for another, and what is left when all
// have ended does not depend on the order.  In the end two vertices are a pair if each holds the other's bid.
// ---------------------------------------------------------------------------
constexpr int RING_THREADS = 128;
constexpr u64 BID_COST = 0xFFFFFFFF00000000ull;  // the cost key of a bid or a neighbour's entry; below it a vertex

// what the other lane of a pair holds
__device__ __forceinline__ u32 of_pair(u32 x) { return (u32)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true); }  // (quad_perm 1, 0, 3, 2)
__device__ __forceinline__ u64 of_pair(u64 x) { return ((u64)of_pair((u32)(x >> 32)) << 32) | of_pair((u32)x); }

// ... and the next one of a row of 16, or the first one
__device__ __forceinline__ u32 next_in_row(u32 x) { return (u32)__builtin_amdgcn_mov_dpp((int)x, 0x12F, 0xF, 0xF, true); }  // (row_ror 15)

constexpr int RING_TILE = RING_THREADS / 2;    // vertices of a workgroup
constexpr int RING_LABELS = 4 * RING_THREADS;  // labels of one of the workgroups behind those of the vertices

// Two lanes a vertex: each takes over the ring of one of the two that the vertex was made of, then evaluates every other neighbour.  Rings that stay in rows of up to ROW_SMALL facets
// are made the same way and evaluated four at a time, a facet a lane; longer ones by the whole wave, 128 facets a turn, one ring after the other.  (Hubs of the input by workgroups of
// their own: a cone of 4,000 facets 1,604 us for 1,650, but every first round 1 us longer.  A vertex of more than a thousand sends the call to rounds by facets.)  With the rows of 11 to 64 facets made and evaluated in one turn of four after the other and a longer one given up for rounds by facets, spheres of segments and
// rings (us a call to a quarter, by facets | then | now): 4 k vertices with poles of 48 facets 159 | 199 | 153, of 128 166 | 188 | 174, 115 k 279 | 304 | 236, 1.2 M 1,153 | 1,211 | 1,052;
// 20 k vertices of a lattice of two sides among 159 k 257 | 298 | 229.
// Bound by the trips from vertex to ring to records, and where rows are rare by the fetching of their code: every step of them that was unrolled, or done twice for few and for
// many, took the 30 % of a decimated mesh's waves that have a row 2 to 4 us longer.  Four waves a SIMD: with five 10 M vertices take 482 us in the first round, 469 with four (the parts' lines push each
// other out of the L2).
template <int PLACE, bool FIRST>
__global__ __launch_bounds__(RING_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) void ring_costs_kernel(State* st, int round, int nv, const VRec* __restrict__ vrec, RingRows in, RingRows out,
                                                                  RingRows adj, u64* __restrict__ first, u64* __restrict__ bids, RoundTab R,
                                                                  const int2* __restrict__ from, const ulonglong2* __restrict__ from_info,
                                                                  const int* __restrict__ vmap, int* __restrict__ cid, int n_labels, float rcond_min,
                                                                  int* __restrict__ facet_slots, int* __restrict__ facet_next) {
    __shared__ MeshFlags M;
    constexpr int HALF = RING_MAX / 2;
    static_assert(32 * ROW_SMALL <= 64 * RING_MAX, "rows of pairs fit the wave's part");
    __shared__ u64 stages[RING_THREADS / 64][64 * RING_MAX];  // a wave's part: its lanes' vertices, then their pairs' facets
    __shared__ int facets;
    const int t = threadIdx.x, lane = prim::lane_id(), half = lane & 1;
    if constexpr (!FIRST) {  // (the labels follow the last contraction)
        const int part = (int)blockIdx.x - (((nv + RING_TILE - 1) / RING_TILE + 7) & ~7);
        if (part >= 0) {
            int c[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const long long o = (long long)part * RING_LABELS + j * RING_THREADS + t;
                c[j] = o < n_labels ? cid[o] : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) c[j] = vmap[c[j]];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const long long o = (long long)part * RING_LABELS + j * RING_THREADS + t;
                if (o < n_labels) cid[o] = c[j];
            }
            return;
        }
    }
    auto neighbour = [&](int u, const VertexWords& U, int x, const VertexWords& X) -> u32 {
        return u == x ? PAIR_NONE : cost_key(pair_cost<PLACE>(U, X, rcond_min));
    };
    const int tiles = (nv + RING_TILE - 1) / RING_TILE, w = prim::xcd_item((int)blockIdx.x, tiles) * RING_TILE + t / 2, v = min(w, nv - 1);
    const bool here = w < nv, lead = here && half == 0;
    u64* const stage = stages[prim::wave_id()];
    u64* const facet_of_pair = stage + lane / 2;  // (in rows of 32)
    auto in_order = [] {  // (a wave's LDS operations complete in order: what is to be kept in order is the compiler)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    };
    u64 info;
    u32 id[RING_MAX];
    int k = 0;             // the facets of its ring, where they are in the pair's place or in a row
    bool is_long = false;  // ... more than ROW_SMALL
    int2 two = make_int2(0, -1);
    ulonglong2 two_info = make_ulonglong2(0, 0);
    VertexWords own;
    if constexpr (!FIRST) {
        two = from[v];
        two_info = from_info[v];
        if (blockIdx.x == 0) round_begin_block(R, st);
        if (t == 0) facets = 0;
    }
    if (blockIdx.x == 0 && t < MATCH_SLOTS) facet_next[t * MATCH_PAD] = 0;
    if (R.B > 1) M.begin(R, nullptr);
    const int hopeless = FIRST ? st->wide : 0;  // (the round goes by facets, and this launch has nothing to do)
    own = load_vertex(vrec, v);
    u64 first_info = 0;
    if constexpr (FIRST) {
        info = first_info = in.info[v];
        in.load_ids(v, id, ring_in_rows(info) ? 0 : ring_ids(info));
        k = ring_in_rows(info) ? rows_length(info) : 0;
        is_long = here && k > ROW_SMALL;
    }
    if (FIRST && hopeless) return;  // (all workgroups)
    u32 x[RING_MAX], y[RING_MAX], kept = 0;  // a short ring's first and second corners; of its facets or a row's, those that stay
    bool backwards = false;
    if constexpr (!FIRST) {
        // the facets of the two it was made of, in the new numbering, without those whose corners have met
        const u64 mine = half ? two_info.y : two_info.x;
        const bool is_short = !ring_in_rows(mine);
        in.load_ids(half ? max(two.y, 0) : two.x, x, ring_in_rows(mine) ? 0 : ring_ids(mine));
        // Rings go either way round; where the vertex that follows the other one is the same in both, the second is taken backwards (else first corners are met twice).
        const u32 other = (u32)(half ? two.x : two.y);
        u32 follows = x[0], at = 0;
#pragma unroll
        for (int j = 1; j < RING_MAX; ++j) at = x[j] == other && j < ring_facets(mine) ? (u32)j : at;
        at = (u32)ring_second(mine, (int)at);
#pragma unroll
        for (int j = 1; j < RING_MAX; ++j) follows = at == (u32)j ? x[j] : follows;
        const u32 they_follow = of_pair(follows);
        backwards = half != 0 && they_follow == follows;
        const int n_ids = is_short ? ring_ids(mine) : 0, n_mine = is_short ? ring_facets(mine) : 0;
#pragma unroll
        for (int j = 0; j < RING_MAX; ++j)
            if (j < RING_ROW || j < n_ids) x[j] = (u32)vmap[j < n_ids ? x[j] : 0u];
        u32* const ids = reinterpret_cast<u32*>(stage) + lane;
#pragma unroll
        for (int j = 0; j < RING_MAX; ++j) ids[j * 64] = x[j];
        in_order();
#pragma unroll
        for (int j = 0; j < RING_MAX; ++j) y[j] = ids[min(ring_second(mine, j), RING_MAX - 1) * 64];  // (of facets it has not: any number)
        in_order();
        u32 ok = 0;
#pragma unroll
        for (int j = 0; j < RING_MAX; ++j) ok |= x[j] != (u32)w && y[j] != (u32)w && x[j] != y[j] ? 1u << j : 0u;
        ok &= (1u << n_mine) - 1u;
        kept = ok;
        info = rows_info(0, 0);
    }
    // The facets that come from rows, up to ROW_SMALL of them.
    const u64 row = FIRST ? info : half ? two_info.y : two_info.x;
    const bool open = here && (ring_in_rows(row) || (!FIRST && (ring_in_rows(two_info.x) || ring_in_rows(two_info.y))));
    const bool any_open = __any(open);
    u64 e[FIRST ? 1 : ROW_SMALL];
    if (any_open) {
        const int length = open && ring_in_rows(row) ? rows_length(row) : 0;
        is_long = max(length, (int)of_pair((u32)length)) > ROW_SMALL;
        constexpr int EACH = ROW_SMALL / 2;
        if constexpr (FIRST) {
#pragma unroll
            for (int j = 0; j < EACH; ++j)
                if (!is_long && 2 * j + half < length) facet_of_pair[(2 * j + half) * 32] = in.rows[rows_at(row) + (u32)(2 * j + half)];
            in_order();
        } else {
#pragma unroll
            for (int j = 0; j < ROW_SMALL; ++j) e[j] = !is_long && j < length ? in.rows[rows_at(row) + (u32)j] : 0ull;
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {  // (all at once take 250 registers; in the end each is in its place again)
                u32 a[EACH], b[EACH];
#pragma unroll
                for (int j = 0; j < EACH; ++j) {
                    a[j] = (u32)vmap[(u32)e[j]];
                    b[j] = (u32)vmap[(u32)(e[j] >> 32)];
                }
#pragma unroll
                for (int j = 0; j < EACH; ++j) {
                    e[j] = e[j + EACH];
                    e[j + EACH] = ring_entry((int)a[j], (int)b[j]);
                    if (!is_long && h * EACH + j < length && a[j] != (u32)w && b[j] != (u32)w && a[j] != b[j]) kept |= 1u << (h * EACH + j);
                }
            }
        }
    }
    // The facets in the pair's place, the one lane's in front of the other's.
    if constexpr (!FIRST) {
        const int n_kept = __popc(kept), n_theirs = (int)of_pair((u32)n_kept), front = half ? n_theirs : 0;
        k = n_kept + n_theirs;
        is_long = is_long || (here && k > ROW_SMALL);
#pragma unroll
        for (int j = 0; j < RING_MAX; ++j) {
            const int place = front + __popc(kept & ((1u << j) - 1u));
            if (!ring_in_rows(row) && (kept >> j & 1u) && place < ROW_SMALL)
                facet_of_pair[place * 32] = ring_entry((int)(backwards ? y[j] : x[j]), (int)(backwards ? x[j] : y[j]));
        }
        if (any_open) {
#pragma unroll
            for (int j = 0; j < ROW_SMALL; ++j) {
                const int place = front + __popc(kept & ((1u << j) - 1u));
                if (ring_in_rows(row) && (kept >> j & 1u) && place < ROW_SMALL) facet_of_pair[place * 32] = e[j];
            }
        }
        in_order();
    }
    const bool made = here && !is_long && (!FIRST || open);  // the ring of the facets in the place
    if constexpr (FIRST)
        if (__any(made && k > RING_MAX)) {
            // Where they are more than a short ring has, those that are there already (of the same two corners: a surface of two sides, say) are left out.  (Later rounds' rings
            // are made of such.)
            constexpr int EACH = ROW_SMALL / 2;
            u64 e[EACH], corners[EACH];
            u32 left = 0;
#pragma unroll
            for (int j = 0; j < EACH; ++j) {
                const int i = 2 * j + half;
                const bool there = made && i < k;
                e[j] = facet_of_pair[i * 32];
                const u32 p = (u32)e[j], q = (u32)(e[j] >> 32);
                corners[j] = there ? ring_entry((int)min(p, q), (int)max(p, q)) : ~0ull;
                left |= there ? 1u << j : 0u;
            }
            in_order();
#pragma unroll
            for (int i = 0; i < EACH; ++i) {
                const u64 theirs = of_pair(corners[i]);
                if (half && corners[i] == theirs) left &= ~(1u << i);
#pragma unroll
                for (int j = i + 1; j < EACH; ++j)
                    if (corners[j] == theirs || corners[j] == corners[i]) left &= ~(1u << j);
            }
            const int n_left = __popc(left), n_theirs = (int)of_pair((u32)n_left);
            if (made) {
                k = n_left + n_theirs;
#pragma unroll
                for (int j = 0; j < EACH; ++j)
                    if (left >> j & 1u) facet_of_pair[((half ? n_theirs : 0) + __popc(left & ((1u << j) - 1u))) * 32] = e[j];
            }
            in_order();
        }
    if (FIRST ? __any(made && k <= RING_MAX) : true) {
        auto make = [&](auto size) {
            constexpr int N = decltype(size)::value;
            u64 e[N];
#pragma unroll
            for (int j = 0; j < N; ++j) e[j] = facet_of_pair[j * 32];
            info = make_ring(e, k, id);
        };
        if (made && k <= RING_MAX) {
            if (FIRST || __any(k > RING_ROW)) make(std::integral_constant<int, RING_MAX>());  // (one of the two for the wave, not one after the other)
            else make(std::integral_constant<int, RING_ROW>());
            if (lead && !ring_in_rows(info)) {
                out.store_ids(w, id, ring_ids(info));
                out.info[w] = info;
            }
        }
    }
    if (!FIRST || R.B > 1) __syncthreads();
    const bool active = here && (R.B <= 1 || M.is_active(R, v)), in_rows = here && ring_in_rows(info);
    auto bid = [&](int u, u64 best) {  // the first one, on the best neighbour
        first[u] = best;
        if (best != VMIN_NONE) atomicMin(&bids[(u32)best], (best & BID_COST) | (u32)u);
    };
    const int n = active && !in_rows ? ring_ids(info) : 0;
    if (n > 0) {
        u32 x[HALF], cost[HALF];  // every other neighbour
        u64 best = VMIN_NONE;
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            x[j] = 2 * j + half < n ? id[2 * j + half] : (u32)v;
            cost[j] = PAIR_NONE;
        }
        auto evaluate = [&](auto from_j, auto to_j) {  // (their records in flight together)
            constexpr int J0 = decltype(from_j)::value, J1 = decltype(to_j)::value;
            VertexWords X[J1 - J0];
#pragma unroll
            for (int j = J0; j < J1; ++j) X[j - J0] = load_vertex(vrec, (int)x[j]);
#pragma unroll
            for (int j = J0; j < J1; ++j) {
                cost[j] = neighbour(v, own, (int)x[j], X[j - J0]);
                const u64 key = x[j] == (u32)v ? VMIN_NONE : ((u64)cost[j] << 32) | x[j];
                best = key < best ? key : best;
            }
        };
        evaluate(std::integral_constant<int, 0>(), std::integral_constant<int, 3>());  // (a surface's vertices have six)
        if (n > 6) evaluate(std::integral_constant<int, 3>(), std::integral_constant<int, HALF>());
        const u64 others = of_pair(best);
        best = others < best ? others : best;
        // the costs in the order of the neighbours: each lane writes half of them
        static_assert(RING_ROW == 8 && HALF == 5, "two costs of each lane to a half of the row, one beside it");
        const u32 s0 = of_pair(half ? cost[0] : cost[2]), s1 = of_pair(half ? cost[1] : cost[3]);
        uint4* const row = reinterpret_cast<uint4*>(adj.ids + (size_t)v * RING_ROW) + half;
        *row = half ? make_uint4(s0, cost[2], s1, cost[3]) : make_uint4(cost[0], s0, cost[1], s1);
        if (n > RING_ROW) adj.more[(size_t)v * RING_MORE + half] = cost[HALF - 1];
        if (lead) bid(v, best);
    } else if (lead && !in_rows) {
        first[v] = VMIN_NONE;
    }
    int n_facets = lead && !in_rows ? ring_facets(info) : 0;
    // Rings in rows of up to ROW_SMALL facets, a facet a lane, several rings at a time.
    const u32 was_at = FIRST ? rows_at(first_info) : 0u;
    const bool in_place = in_rows && !is_long;
    u64 todo = prim::ballot(lead && in_place);
    if (todo != 0) {
        u32 at = was_at, place = 0;  // (all rings' places together)
        int words = 0;
        if constexpr (!FIRST) {
            const int mine = lead && in_place ? k : 0;
            words = mine;  // with those of the lanes in front
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int x = __shfl_up(words, d, 64);
                words += lane >= d ? x : 0;
            }
            at = (u32)(words - mine);
            if (lane == 63) place = out.ask((u32)words);
        }
        if (lead && in_place) n_facets = k;
        const int sub = lane & (ROW_SMALL - 1), group = lane / ROW_SMALL;
        for (bool first_turn = true; todo != 0; first_turn = false) {
            int owner = -1;
#pragma unroll
            for (int j = 0; j < 64 / ROW_SMALL; ++j) {
                if (j == group && todo) owner = __ffsll((long long)todo) - 1;
                todo &= todo - 1;
            }
            const int from_lane = max(owner, 0), u = __shfl(v, from_lane, 64), n_its = __shfl(k, from_lane, 64);
            const bool ok = owner >= 0 && sub < n_its, counts = __shfl(active ? 1 : 0, from_lane, 64) != 0;
            const u64 e = ok ? stage[sub * 32 + from_lane / 2] : ring_entry(u, u);
            const u32 a = (u32)e, b = (u32)(e >> 32);
            const VertexWords U = load_vertex(vrec, u), P = load_vertex(vrec, (int)a);
            bool alone = ok && b != (u32)u;  // the second corner is no facet's first one
            u32 other = a;
#pragma unroll
            for (int j = 0; j < ROW_SMALL; ++j) {
                alone = alone && b != other;
                other = next_in_row(other);
            }
            const u64 alone_in_group = prim::ballot(alone) >> (group * ROW_SMALL) & ((1ull << ROW_SMALL) - 1ull);
            if constexpr (!FIRST)
                if (first_turn) {
                    if (lane == 63) place = out.take((u32)words, place);
                    place = (u32)__builtin_amdgcn_readlane((int)place, 63);
                }
            const u32 its_at = place + (u32)__shfl((int)at, from_lane, 64);
            u32 cost_a = neighbour(u, U, (int)a, P), cost_b = PAIR_NONE;
            if (__any(alone)) {
                const VertexWords Q = load_vertex(vrec, alone ? (int)b : u);
                cost_b = neighbour(u, U, alone ? (int)b : u, Q);
            }
            if (ok && place != ~0u) {  // (where there is no place the round will be done again by facets)
                out.rows[its_at + (u32)sub] = e;
                adj.rows[its_at + (u32)sub] = ((u64)cost_b << 32) | cost_a;
            }
            u64 best = a != (u32)u ? ((u64)cost_a << 32) | a : VMIN_NONE;
            const u64 key_b = alone ? ((u64)cost_b << 32) | b : VMIN_NONE;
            best = key_b < best ? key_b : best;
#pragma unroll
            for (int d = ROW_SMALL / 2; d > 0; d >>= 1) {
                const u64 x = __shfl_xor(best, d, 64);
                best = x < best ? x : best;
            }
            if (owner >= 0 && sub == 0) {
                out.info[u] = rows_info(n_its, its_at);
                adj.info[u] = (u64)(u32)((alone_in_group ? n_its : 0) | n_its << 8);
                bid(u, counts ? best : VMIN_NONE);
            }
        }
    }
    // ... and of more, a facet a lane, one ring after the other.
    for (todo = prim::ballot(lead && in_rows && is_long); todo != 0; todo &= todo - 1) {
        const int from_lane = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
        const int u = __builtin_amdgcn_readlane(v, from_lane), counts = __builtin_amdgcn_readlane(active ? 1 : 0, from_lane);
        auto word = [&](u64 x) -> u64 {
            return ((u64)(u32)__builtin_amdgcn_readlane((int)(x >> 32), from_lane) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)x, from_lane);
        };
        int source[2] = {0, 0}, count[2] = {0, 0};
        u64 source_info[2] = {0, 0};
        u32 at = 0;
        if constexpr (FIRST) {
            at = (u32)__builtin_amdgcn_readlane((int)was_at, from_lane);
            count[0] = __builtin_amdgcn_readlane(k, from_lane);
        } else {
            source[0] = __builtin_amdgcn_readlane(two.x, from_lane);
            source[1] = __builtin_amdgcn_readlane(two.y, from_lane);
            source_info[0] = word(two_info.x);
            source_info[1] = word(two_info.y);
            count[0] = ring_facets(source_info[0]);
            count[1] = source[1] >= 0 ? ring_facets(source_info[1]) : 0;
            if (lane == 0) at = out.ask((u32)(count[0] + count[1]));
        }
        const VertexWords U = load_vertex(vrec, u);
        const int n_from = count[0] + count[1];
        int n_kept = 0;
        u64 best = VMIN_NONE;
        constexpr int AHEAD = 4;  // facets of a lane that are fetched together
        u32 begin = (u32)u;       // the first corner of the first
        bool any_alone = false;
#pragma unroll 1
        for (int i0 = 0; i0 < n_from; i0 += AHEAD * 64) {
            u32 as[AHEAD], bs[AHEAD];
#pragma unroll
            for (int c = 0; c < AHEAD; ++c) {
                const int i = i0 + c * 64 + lane;
                as[c] = bs[c] = FIRST ? (u32)u : 0u;
                if (i < n_from) {
                    if constexpr (FIRST) {
                        const u64 e = in.rows[at + (u32)i];
                        as[c] = (u32)e;
                        bs[c] = (u32)(e >> 32);
                    } else {
                        const bool second = i >= count[0];
                        in.load_facet(second ? source[1] : source[0], second ? source_info[1] : source_info[0], second ? i - count[0] : i, as[c], bs[c]);
                    }
                }
            }
            if constexpr (!FIRST)
#pragma unroll
                for (int c = 0; c < AHEAD; ++c) {
                    as[c] = (u32)vmap[as[c]];
                    bs[c] = (u32)vmap[bs[c]];
                }
#pragma unroll 1
            for (int c0 = 0; c0 < AHEAD && i0 + c0 * 64 < n_from; c0 += 2) {  // (two records in flight together)
                u32 a[2], b[2], cost_a[2], cost_b[2] = {PAIR_NONE, PAIR_NONE};
                u64 all[2];
                VertexWords X[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    a[h] = as[h];
                    b[h] = bs[h];
#pragma unroll
                    for (int j = h + 2; j < AHEAD; j += 2) {
                        as[j - 2] = as[j];
                        bs[j - 2] = bs[j];
                    }
                    const bool ok = i0 + (c0 + h) * 64 + lane < n_from && (FIRST || (a[h] != (u32)u && b[h] != (u32)u && a[h] != b[h]));
                    if (!ok) a[h] = b[h] = (u32)u;
                    all[h] = prim::ballot(ok);
                    X[h] = load_vertex(vrec, (int)a[h]);
                }
                if (i0 == 0 && c0 == 0) begin = (u32)__builtin_amdgcn_readlane((int)a[0], all[0] ? __ffsll((long long)all[0]) - 1 : 0);
#pragma unroll
                for (int h = 0; h < 2; ++h) cost_a[h] = neighbour(u, U, (int)a[h], X[h]);
                // second corners that the next facet does not begin with (behind the last one the first may follow)
                bool alone[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u64 behind = all[h] & ~((2ull << lane) - 1ull);
                    u32 next = (u32)__shfl((int)a[h], behind ? __ffsll((long long)behind) - 1 : lane, 64);
                    const u32 next_chunk = h == 0 && all[1] != 0 ? (u32)__builtin_amdgcn_readlane((int)a[1], __ffsll((long long)all[1]) - 1) : begin;
                    next = behind ? next : next_chunk;
                    alone[h] = (all[h] >> lane & 1u) != 0 && next != b[h] && b[h] != (u32)u;
                }
                if (__any(alone[0] || alone[1])) {
                    any_alone = true;
#pragma unroll
                    for (int h = 0; h < 2; ++h) X[h] = load_vertex(vrec, alone[h] ? (int)b[h] : u);
#pragma unroll
                    for (int h = 0; h < 2; ++h) cost_b[h] = neighbour(u, U, alone[h] ? (int)b[h] : u, X[h]);
                }
                if constexpr (!FIRST)
                    if (i0 == 0 && c0 == 0) {
                        if (lane == 0) at = out.take((u32)n_from, at);
                        at = (u32)__builtin_amdgcn_readfirstlane((int)at);
                    }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u64 key_a = a[h] != (u32)u ? ((u64)cost_a[h] << 32) | a[h] : VMIN_NONE, key_b = alone[h] ? ((u64)cost_b[h] << 32) | b[h] : VMIN_NONE;
                    best = key_a < best ? key_a : best;
                    best = key_b < best ? key_b : best;
                    if ((all[h] >> lane & 1u) != 0 && at != ~0u) {  // (where there is no place the round will be done again by facets)
                        const u32 place = at + (u32)n_kept + prim::mask_below(all[h]);
                        adj.rows[place] = ((u64)cost_b[h] << 32) | cost_a[h];
                        if constexpr (!FIRST) out.rows[place] = ring_entry((int)a[h], (int)b[h]);
                    }
                    n_kept += (int)__popcll(all[h]);
                }
            }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const u64 other = __shfl_xor(best, d, 64);
            best = other < best ? other : best;
        }
        if (lane == 0) {
            if constexpr (!FIRST) out.info[u] = rows_info(n_kept, at);
            if (n_kept <= ROW_SMALL) adj.info[u] = (u64)(u32)((any_alone ? n_kept : 0) | n_kept << 8);
            if (n_kept > 64) atomicMax(&st->longest[round & 1], n_kept);
            n_facets += n_kept;
            bid(u, counts ? best : VMIN_NONE);
        }
    }
    if constexpr (FIRST) {  // (the places of the others have been counted when they were given out)
        if (__any(in_rows)) {
            int words = lead && in_rows ? k : 0;
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) words += __shfl_xor(words, d, 64);
            if (lane == 0) atomicAdd(&out.taken[(blockIdx.x & (ROW_ARENAS - 1)) * MATCH_PAD], words);
        }
    }
    if constexpr (!FIRST) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) n_facets += __shfl_xor(n_facets, d, 64);
        if (lane == 0 && n_facets) atomicAdd(&facets, n_facets);
        __syncthreads();
        if (t == 0 && facets) atomicAdd(&facet_slots[(blockIdx.x & (MATCH_SLOTS - 1)) * MATCH_PAD], facets);
    }
}

// The matching from the first bids (on every vertex's best neighbour) on.  A wave has `per` vertices in a row to itself: it lists whose bids have been bettered, so many at a
// time; its lanes take one after the other, and with it whoever their bids drive out in turn.  Several lanes may come to go on for a vertex (one that finds its bid
// gone, and the one that drove it out): they ask the same neighbours in the same order, and the one that finds the vertex's own bid there ends.
constexpr int SUITOR_LOOK = 4;  // vertices of a lane that are looked at together
constexpr int SUITOR_FEW = 4;   // rings in rows of a wave that all its lanes read together
__global__ __launch_bounds__(BLOCK) void suitor_kernel(int nv, int per, int round, State* st, RingRows ring, RingRows adj, const u64* __restrict__ first, u64* bids,
                                                       int* __restrict__ taken_next) {
    __shared__ u64 tried[prim::WAVES][64 * SUITOR_LOOK];  // the neighbour (with its cost) that has refused the vertex
    __shared__ int lost[prim::WAVES][64 * SUITOR_LOOK];
    const int t = threadIdx.x, lane = prim::lane_id(), w = prim::wave_id();
    if (blockIdx.x == 0 && t <= ROW_ARENAS) taken_next[t * MATCH_PAD] = 0;  // (of the next round)
    if (blockIdx.x == 0 && t == 0) st->longest[(round & 1) ^ 1] = 0;
    // The sum is made here, beside the matching: publish_pairs, which the host waits for, would take 1 us longer for it (16 meshes of 60 k vertices over four levels 1,070 us for 1,063).
    if (blockIdx.x == 0 && w == prim::WAVES - 1) {
        int words = lane <= ROW_ARENAS ? ring.taken[lane * MATCH_PAD] : 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) words += __shfl_xor(words, d, 64);
        if (lane == 0) st->row_words = words;
    }
    if (st->wide) return;
    const long long from = (long long)prim::xcd_item((int)blockIdx.x, (nv - 1) / (per * prim::WAVES) + 1) * prim::WAVES + w;
    long long at = from * per;  // the next vertex to look at
    const long long end = min(at + per, (long long)nv);
    int listed = 0, taken = 0;
    bool busy = false, fetch = false;
    int u = 0, m = 0, k = 0, k_both = 0;  // a short ring's vertices; the facets of one in rows that have costs, and how many of them have two; they lie
    u32 there_at = 0;                     // ... here
    u64 last = 0, row[ROW_LINE];
#pragma unroll
    for (int j = 0; j < ROW_LINE; ++j) row[j] = VMIN_NONE;
    for (;;) {
        while (taken == listed && at < end && __any(!busy)) {
            u64 k[SUITOR_LOOK], b[SUITOR_LOOK];
#pragma unroll
            for (int j = 0; j < SUITOR_LOOK; ++j) k[j] = at + j * 64 + lane < end ? first[at + j * 64 + lane] : VMIN_NONE;
#pragma unroll
            for (int j = 0; j < SUITOR_LOOK; ++j) b[j] = bids[k[j] != VMIN_NONE ? (u32)k[j] : 0u];
            listed = taken = 0;
#pragma unroll
            for (int j = 0; j < SUITOR_LOOK; ++j) {
                const int v = (int)at + j * 64 + lane;
                const bool gone = k[j] != VMIN_NONE && b[j] != ((k[j] & BID_COST) | (u32)v);
                const u64 all = prim::ballot(gone);
                if (gone) {
                    tried[w][listed + (int)prim::mask_below(all)] = k[j];
                    lost[w][listed + (int)prim::mask_below(all)] = v;
                }
                listed += (int)__popcll(all);
            }
            at += 64 * SUITOR_LOOK;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
        const u64 idle = prim::ballot(!busy);
        if (taken < listed) {
            const int i = taken + (int)prim::mask_below(idle);
            if (!busy && i < listed) {
                u = lost[w][i];
                last = tried[w][i];
                busy = fetch = true;
            }
            taken = min(listed, taken + (int)__popcll(idle));
        }
        if (!__any(busy)) break;
        if (fetch) {
            const u64 info = ring.info[u];
            u32 id[RING_MAX], cost[RING_MAX];
            ring.load_ids(u, id, 0);
            adj.load_ids(u, cost, 0);
            const bool in_rows = ring_in_rows(info);
            m = in_rows ? 0 : ring_ids(info);
            k = in_rows ? rows_length(info) : 0;
            there_at = rows_at(info);
            k_both = k;
            if (k > 0 && k <= ROW_SMALL) {
                const u32 with = (u32)adj.info[u];
                k_both = (int)(with & 255u);
                k = (int)(with >> 8);
            }
#pragma unroll
            for (int j = 0; j < ROW_LINE; ++j) row[j] = ((u64)cost[j] << 32) | id[j];
            fetch = false;
        }
        // the best neighbour behind `last` whose bid u's betters or is (what others have bid meanwhile only makes it fewer)
        u64 want = VMIN_NONE;
        auto consider = [&](const auto& x, int n) {
            constexpr int N = (int)(sizeof(x) / sizeof(x[0]));
            u64 there[N];
            bool open[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                open[j] = busy && j < n && x[j] > last && (u32)(x[j] >> 32) != PAIR_NONE;
                if (open[j]) there[j] = bids[(u32)x[j]];
            }
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (open[j] && there[j] >= ((x[j] & BID_COST) | (u32)u) && x[j] < want) want = x[j];
        };
        consider(row, m);
        if (__any(busy && m > ROW_LINE)) {
            u64 x[2] = {VMIN_NONE, VMIN_NONE};
            if (busy && m > ROW_LINE) {
                const uint2 id = *reinterpret_cast<const uint2*>(ring.more + (size_t)u * RING_MORE);
                const uint2 cost = *reinterpret_cast<const uint2*>(adj.more + (size_t)u * RING_MORE);
                x[0] = ((u64)cost.x << 32) | id.x;
                x[1] = ((u64)cost.y << 32) | id.y;
            }
            consider(x, m - ROW_LINE);
        }
        if (__any(busy && k > 0)) {
            // Rings in rows: each lane its own, four facets at a time; the long ones, and all where only a few lanes have more than eight neighbours so, all lanes together, one ring
            // after the other.
            constexpr int LINE = ROW_LINE / 2;
            const bool small = busy && k > 0 && k <= ROW_SMALL, wide = small && (k > ROW_LINE || k_both > 0);
            const bool alone = small && !(wide && __popcll(prim::ballot(wide)) <= SUITOR_FEW);
            const int lines = (k + LINE - 1) / LINE, n_lines = alone ? lines + (k_both + LINE - 1) / LINE : 0;
#pragma unroll 1
            for (int l = 0; __any(l < n_lines); ++l) {
                u64 x[LINE];
                const bool second = l >= lines;
                const int i0 = (second ? l - lines : l) * LINE, n = l >= n_lines ? 0 : second ? k_both : k;
#pragma unroll
                for (int j = 0; j < LINE; ++j) {
                    x[j] = VMIN_NONE;
                    if (i0 + j < n) {
                        const u64 facet = ring.rows[there_at + (u32)(i0 + j)], cost = adj.rows[there_at + (u32)(i0 + j)];
                        x[j] = second ? (cost & BID_COST) | (facet >> 32) : (cost << 32) | (u32)facet;
                    }
                }
                consider(x, LINE);
            }
            for (u64 todo = prim::ballot(busy && k > 0 && !alone); todo != 0; todo &= todo - 1) {
                const int from_lane = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
                const int its = __builtin_amdgcn_readlane(u, from_lane), n = __builtin_amdgcn_readlane(k, from_lane);
                const u32 its_at = (u32)__builtin_amdgcn_readlane((int)there_at, from_lane);
                const u64 behind = ((u64)(u32)__builtin_amdgcn_readlane((int)(last >> 32), from_lane) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)last, from_lane);
                u64 its_want = VMIN_NONE;
#pragma unroll 1
                for (int i = lane; i < n; i += 64) {
                    const u64 e = ring.rows[its_at + (u32)i], cost = adj.rows[its_at + (u32)i];
                    const u64 x[2] = {(cost << 32) | (u32)e, (cost & BID_COST) | (e >> 32)};
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        if (x[j] > behind && (u32)(x[j] >> 32) != PAIR_NONE && bids[(u32)x[j]] >= ((x[j] & BID_COST) | (u32)its) && x[j] < its_want) its_want = x[j];
                }
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) {
                    const u64 other = __shfl_xor(its_want, d, 64);
                    its_want = other < its_want ? other : its_want;
                }
                if (lane == from_lane) want = its_want;
            }
        }
        if (busy) {
            if (want == VMIN_NONE) {
                busy = false;  // (nobody is left: u stays alone)
            } else {
                const u64 mine = (want & BID_COST) | (u32)u;
                const u64 old = atomicMin(&bids[(u32)want], mine);
                if (old > mine) {
                    busy = fetch = old != VMIN_NONE;
                    if (busy) {  // whose bid was there goes on behind this vertex
                        last = (old & BID_COST) | (u32)want;
                        u = (int)(u32)old;
                    }
                } else {
                    busy = old != mine;
                    last = want;
                }
            }
        }
    }
}

// Pairs that may be the budget's last one, as (cost - lo << 32) | lower vertex, for the two kernels of the budget step of a single mesh (see budget_range_kernel).
constexpr int BUDGET_THREADS = 1024, BUDGET_LIST = 32 * BUDGET_THREADS;
struct BudgetList {
    u64 counts;  // pairs in front of the listed range (<< 32), listed ones (the list may hold less)
    u32 lo, hi;  // the range
    u64 entry[BUDGET_LIST];  // (of which there is room for all pairs of the mesh where these are fewer)
};

// The pairs that the bids come to: partners and costs by vertex, how many there are of each mesh, and per tile the vertices that survive them (as a
// compaction's count pass does).
template <int CHUNKS>
__global__ __launch_bounds__(BLOCK) void pairs_kernel(SelArgs A, const u64* __restrict__ bids, int* __restrict__ tilesum, BudgetList* __restrict__ budget) {
    __shared__ PairTally tally;
    __shared__ u32 smem[prim::WAVES];
    const int nv = A.nv, wave = prim::wave_id(), lane = prim::lane_id(), t = threadIdx.x;
    const bool wide = A.st->wide != 0;
    if (blockIdx.x == 0 && t == 0) {  // (what the kernels queued behind this one go by)
        A.st->go = wide ? 0 : 1;
        A.st->guard_nv = wide ? 0 : nv;
        if (budget) budget->counts = 0;
    }
    if (wide) return;
    const long long base = (long long)blockIdx.x * (BLOCK * CHUNKS), i0 = base + wave * (64 * CHUNKS) + lane;
    u64 b[CHUNKS], back[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) b[c] = i0 + c * 64 < nv ? bids[i0 + c * 64] : VMIN_NONE;
    if (t == 0) tally.begin(A, (int)base);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) back[c] = bids[b[c] != VMIN_NONE ? (u32)b[c] : 0u];
    __syncthreads();
    u32 stay = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const long long i = i0 + c * 64;
        const int w = (int)i, p = (int)(u32)b[c];
        const bool paired = b[c] != VMIN_NONE && back[c] == ((b[c] & BID_COST) | (u32)w), lower = paired && w < p;
        if (i < nv) {
            A.mate[w] = paired ? p : -1;
            A.pcost[w] = lower ? (u32)(b[c] >> 32) : PAIR_NONE;
        }
        tally.count(A, lower, w);
        stay += (u32)__popcll(prim::ballot(i < nv && (!paired || lower)));
    }
    if (lane == 0) smem[wave] = stay;
    __syncthreads();
    if (t == 0) {
        tilesum[blockIdx.x] = (int)(smem[0] + smem[1] + smem[2] + smem[3]);
        tally.end(A);
    }
}

// The round's pair counts and State for the host, by one workgroup of a kernel behind pairs_kernel (the number `at`, which does nothing else).
struct PairPublish {
    int at;  // -1: published already
    State* st;
    const int* mslots;
    int* matched;
    int* done;  // (or null) meshes with pairs are marked
    int B;
    const int* facet_slots;  // (or null: all facets are left)
    int* host_img;
    int publish_ints;
    HostSignal tell;
};
__device__ __forceinline__ void publish_pairs(const PairPublish& P, bool missed = false) {
    constexpr int STATE_INTS = (int)(sizeof(State) / sizeof(int)), GO0 = (int)(offsetof(State, go) / sizeof(int)), NH = (int)(offsetof(State, nh) / sizeof(int)),
                  MISSED = (int)(offsetof(State, missed) / sizeof(int));
    static_assert(MATCH_SLOTS == 32, "a mesh's slots fill half a wave");
    const int t = threadIdx.x, n = blockDim.x;
    const bool wide = P.st->wide != 0;
    auto slots_sum = [](int x) {
#pragma unroll
        for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
        return x;
    };
    const int corners = slots_sum(P.facet_slots ? P.facet_slots[(t & (MATCH_SLOTS - 1)) * MATCH_PAD] : 0);
    constexpr int TOGETHER = 8;
    const int n_slots = P.B * MATCH_SLOTS;
    for (int i0 = t; i0 < n_slots; i0 += TOGETHER * n) {  // (whole half waves)
        int x[TOGETHER];
#pragma unroll
        for (int j = 0; j < TOGETHER; ++j) x[j] = i0 + j * n < n_slots ? P.mslots[(size_t)(i0 + j * n) * MATCH_PAD] : 0;
#pragma unroll
        for (int j = 0; j < TOGETHER; ++j) {
            const int i = i0 + j * n, b = i / MATCH_SLOTS;
            if (i >= n_slots) break;
            const int sum = slots_sum(x[j]);
            if ((i & (MATCH_SLOTS - 1)) == 0 && !wide) {
                P.matched[b] = sum;
                if (P.done && sum > 0) P.done[b] = 1;
                if (STATE_INTS + b < P.publish_ints) host_store(&P.host_img[STATE_INTS + b], sum);
            }
        }
    }
    for (int i = t; i < GO0 && i < P.publish_ints; i += n) host_store(&P.host_img[i], i == NH ? corners : i == MISSED ? (missed ? 1 : 0) : reinterpret_cast<const int*>(P.st)[i]);
    signal_host(P.tell, t, true);
}
__global__ __launch_bounds__(BLOCK) void publish_pairs_kernel(PairPublish P) { publish_pairs(P); }

// ---------------------------------------------------------------------------
// The budget step of a single mesh in a round by rings, of more pairs than one compute unit walks in little time, by two launches that know nothing of the host and
// leave the partners and the tiles' counts of survivors as the contraction takes them.
// In the first every workgroup finds in a sample of the costs, the same for all, the range in which the budget's last pair lies (counts of 14 bits, 32 digits an
// octave; six standard deviations of a rank in the middle); the pairs in it are listed, those in front of it counted.
// In the second every workgroup finds the last pair among the listed ones, dissolves what lies beyond it among its own vertices and counts who survives.  Where the
// sample has misled, or too many costs are equal, nothing is contracted, and the host, which is told, takes the general way.  (Costs are few values: 165 k pairs of a lattice have 3,000, one of
// them 13 k of the pairs, so the list has two of them in it now and then: 10 to 23 thousand of 165 thousand pairs, with 16 thousand places too many at every third budget.)
// Bound by chains: a sample's trip, its counts in LDS and their scan in the first; two trips and up to three counts of 12 bits in the second (many of a scanned wall's costs
// are equal, so that the vertices decide).  115 k vertices (a second round of 62 k, 28 k pairs): the search by one workgroup took 22 us and the count of the survivors with the
// release 5, these two 7 and 12; 1.2 M (350 k, 160 k pairs), where the whole chip's histogram passes behind a look of the host took 46 in eight launches, 15 and 19.
// (The second by one workgroup, which then dissolves the listed ones itself: 24 and 42, most of it scattered stores.)
// ---------------------------------------------------------------------------
constexpr int BUDGET_BITS = 14, BUDGET_DIGITS = 1 << BUDGET_BITS, BUDGET_TILES = BUDGET_THREADS / BLOCK;
constexpr int BUDGET_SAMPLES = 4;  // vertices of a place
constexpr int BUDGET_FEW = 1 << 16;  // vertices up to which a lane samples one place, beyond four

// Pairs of the mesh, by the lanes of a whole half wave.
__device__ __forceinline__ int pairs_of_mesh(const int* __restrict__ mslots) {
    int n = mslots[(threadIdx.x & (MATCH_SLOTS - 1)) * MATCH_PAD];
#pragma unroll
    for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
    return n;
}

// Counts a digit of each lane with `on`.  Costs are equal in many pairs of scanned walls, and lanes that name one word take turns: those with the first one's digit go together.
// (Of the sample, whose costs are of many digits, it takes longer: 15 us of the launch above, 19.)
__device__ __forceinline__ void count_digit(u32* hist, bool on, u32 d) {
    const u64 all = prim::ballot(on);
    if (all == 0) return;
    const int lead = __ffsll((long long)all) - 1;
    const u32 first = (u32)__builtin_amdgcn_readlane((int)d, lead);
    const u64 same = prim::ballot(on && d == first);
    if (prim::lane_id() == lead) atomicAdd(&hist[first], (u32)__popcll(same));
    else if (on && d != first) atomicAdd(&hist[d], 1u);
}

__global__ __launch_bounds__(BUDGET_THREADS) void budget_range_kernel(const u32* __restrict__ pcost, int nv, const State* __restrict__ st,
                                                                      const int* __restrict__ mslots, const int* __restrict__ budget,
                                                                      BudgetList* __restrict__ L) {
    constexpr int N_WAVES = BUDGET_THREADS / 64, DIGITS_EACH = BUDGET_DIGITS / BUDGET_THREADS;
    constexpr u32 HIGHEST = 0xFFFFFFFEu, IN_DIGIT = (1u << (32 - BUDGET_BITS)) - 1u;
    __shared__ u32 hist[BUDGET_DIGITS + BUDGET_THREADS];  // (a word between the lanes' digits: they read them at a stride that meets all banks)
    __shared__ u32 smem[N_WAVES], found[2], n_listed, n_below;
    __shared__ u64 list_at;
    const int t = threadIdx.x, lane = prim::lane_id(), w = (int)blockIdx.x * BUDGET_THREADS + t;
    const bool here = w < nv;
    const int go = st->go, keep = budget[0], n = pairs_of_mesh(mslots);
    const u32 own = here ? pcost[w] : PAIR_NONE;  // (of a pair's lower vertex)
    uint4 sample[BUDGET_SAMPLES];
    int place[BUDGET_SAMPLES];
#pragma unroll
    for (int q = 0; q < BUDGET_SAMPLES; ++q) {
        const bool on = q == 0 || nv > BUDGET_FEW;
        place[q] = (int)(((long long)nv * (nv > BUDGET_FEW ? q * BUDGET_THREADS + t : t)) >> (nv > BUDGET_FEW ? 12 : 10)) & ~3;
        sample[q] = on ? *reinterpret_cast<const uint4*>(pcost + place[q]) : make_uint4(PAIR_NONE, PAIR_NONE, PAIR_NONE, PAIR_NONE);
    }
    if (go == 0 || n <= keep) return;
    for (int i = t; i < BUDGET_DIGITS + BUDGET_THREADS; i += BUDGET_THREADS) hist[i] = 0;
    if (t < 2) found[t] = 0;
    if (t == 0) n_listed = n_below = 0;
    __syncthreads();
    auto note = [&](u32 c, int v) {
        const u32 d = c >> (32 - BUDGET_BITS);
        if (c != PAIR_NONE && v < nv) atomicAdd(&hist[d + d / DIGITS_EACH], 1u);
    };
#pragma unroll
    for (int q = 0; q < BUDGET_SAMPLES; ++q) {
        note(sample[q].x, place[q]);
        note(sample[q].y, place[q] + 1);
        note(sample[q].z, place[q] + 2);
        note(sample[q].w, place[q] + 3);
    }
    __syncthreads();
    u32 c[DIGITS_EACH], sum = 0;
#pragma unroll
    for (int j = 0; j < DIGITS_EACH; ++j) {
        c[j] = hist[t * (DIGITS_EACH + 1) + j];
        sum += c[j];
    }
    u32 all, run = prim::wide_block_exclusive_scan<N_WAVES>(sum, smem, all);
    const float rank = (float)all * (float)keep / (float)n, margin = 3.0f * sqrtf((float)all) + 4.0f;
    const u32 from = rank > margin ? (u32)(rank - margin) : 0u, to = min((u32)(rank + margin), all + 1u);
#pragma unroll
    for (int j = 0; j < DIGITS_EACH; ++j) {
        if (run < from && from <= run + c[j]) found[0] = (u32)(t * DIGITS_EACH + j);
        if (run < to && to <= run + c[j]) found[1] = (u32)(t * DIGITS_EACH + j);
        run += c[j];
    }
    __syncthreads();
    const u32 lo = from > 0 ? found[0] << (32 - BUDGET_BITS) : 0u;
    const u32 hi = to > 0 && to <= all ? min(HIGHEST, (found[1] << (32 - BUDGET_BITS)) | IN_DIGIT) : HIGHEST;
    if (blockIdx.x == 0 && t == 0) {
        L->lo = lo;
        L->hi = hi;
    }
    const bool lists = own != PAIR_NONE && own >= lo && own <= hi, below = own < lo;
    const u64 listed = prim::ballot(lists), in_front = prim::ballot(below);
    u32 at = 0;
    if (lane == 0) {
        if (in_front) atomicAdd(&n_below, (u32)__popcll(in_front));
        if (listed) at = atomicAdd(&n_listed, (u32)__popcll(listed));
    }
    __syncthreads();
    if (t == 0) list_at = n_listed || n_below ? atomicAdd(&L->counts, ((u64)n_below << 32) | n_listed) : 0ull;
    __syncthreads();
    at = (u32)list_at + (u32)__shfl((int)at, 0, 64) + prim::mask_below(listed);
    if (lists && at < (u32)BUDGET_LIST) L->entry[at] = ((u64)(own - lo) << 32) | (u32)w;
}

__global__ __launch_bounds__(BUDGET_THREADS) void budget_release_kernel(const u32* __restrict__ pcost, int* __restrict__ mate, int nv, State* st,
                                                                        const int* __restrict__ mslots, const int* __restrict__ budget, int* __restrict__ tilesum,
                                                                        const BudgetList* __restrict__ L, PairPublish publish) {
    constexpr int N_WAVES = BUDGET_THREADS / 64, EACH = 16, AGAIN = 8, BITS = 12;  // keys that a lane keeps, and of what the list has beyond that, how many it fetches together in every turn
    static_assert(BLOCK == 4 * 64, "four waves a tile");
    static_assert(1 << BITS == 4 * BUDGET_THREADS, "four digits a lane");
    __shared__ uint4 hist4[BUDGET_THREADS];
    __shared__ u32 smem[N_WAVES], found[3], n_few;
    __shared__ u64 few[64], last;
    u32* const hist = reinterpret_cast<u32*>(hist4);
    const int t = threadIdx.x, lane = prim::lane_id();
    int w = (int)blockIdx.x * BUDGET_THREADS + t;
    const u64 counts = L->counts;
    const u32 lo = L->lo, hi = L->hi;
    const int go = st->go, keep = budget[0], n = pairs_of_mesh(mslots);
    int m = w < nv ? mate[w] : -1;
    const u32 n_below = (u32)(counts >> 32), listed = (u32)counts;
    const bool binds = go != 0 && n > keep, found_it = (int)n_below < keep && keep <= (int)(n_below + listed) && listed <= (u32)BUDGET_LIST;
    if ((int)blockIdx.x == publish.at) {
        __syncthreads();  // (all have read it)
        if (t == 0 && binds && !found_it) st->go = 0;
        publish_pairs(publish, binds && !found_it);
        return;
    }
    if (!binds || !found_it) return;
    auto pair_key = [&]() { return m >= 0 ? ((u64)pcost[min(w, m)] << 32) | (u32)min(w, m) : 0ull; };
    u64 own = pair_key();
    u64 key[EACH];
    const int each = (int)((listed + BUDGET_THREADS - 1) / BUDGET_THREADS);
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
        const u32 i = (u32)(j * BUDGET_THREADS + t);
        key[j] = i < listed ? L->entry[i] : ~0ull;
    }
    auto each_key = [&](auto fn) {
#pragma unroll
        for (int j = 0; j < EACH; ++j)
            if (j < each) fn(key[j]);
#pragma unroll 1
        for (int j0 = EACH; j0 < each; j0 += AGAIN) {
            u64 more[AGAIN];
#pragma unroll
            for (int j = 0; j < AGAIN; ++j) {
                const u32 i = (u32)((j0 + j) * BUDGET_THREADS + t);
                more[j] = i < listed ? L->entry[i] : ~0ull;
            }
#pragma unroll
            for (int j = 0; j < AGAIN; ++j) fn(more[j]);
        }
    };
    // by counts of 12 bits a time, of the costs from the highest bit that there is, then of the vertices, until 64 or less are left, which one wave ranks
    u32 want = (u32)keep - n_below, equal = listed;
    int undecided = hi == lo ? 32 - __clz(nv) : 64 - __clz((int)(hi - lo));
    u64 decided = undecided >= 64 ? 0ull : ~0ull << undecided, prefix = 0;
    if (t == 0) n_few = 0;
    hist4[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    while (equal > 64u && undecided > 0) {
        const int nb = min(BITS, undecided > 32 ? undecided - 32 : undecided), shift = undecided - nb;
        each_key([&](u64 k) { count_digit(hist, k != ~0ull && (k & decided) == prefix, (u32)(k >> shift) & ((1u << nb) - 1u)); });
        __syncthreads();
        const uint4 c4 = hist4[t];
        hist4[t] = make_uint4(0, 0, 0, 0);  // (for the next turn, behind the barriers that follow)
        const u32 c[4] = {c4.x, c4.y, c4.z, c4.w};
        u32 all, run = prim::wide_block_exclusive_scan<N_WAVES>((c[0] + c[1]) + (c[2] + c[3]), smem, all);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (run < want && want <= run + c[j]) {  // (in one thread)
                found[0] = (u32)(4 * t + j);
                found[1] = run;
                found[2] = c[j];
            }
            run += c[j];
        }
        __syncthreads();
        prefix |= (u64)found[0] << shift;
        want -= found[1];
        equal = found[2];
        undecided = shift == 32 ? 32 - __clz(nv) : shift;
        decided = ~0ull << undecided;
    }
    each_key([&](u64 k) {
        if (k != ~0ull && (k & decided) == prefix) {
            const u32 p = atomicAdd(&n_few, 1u);
            if (p < 64u) few[p] = k;
        }
    });
    __syncthreads();
    if (t < 64) {
        const int c = (int)min(n_few, 64u);
        const u64 k = few[min(t, c - 1)];
        u32 below = 0;
        for (int i = 0; i < c; ++i) below += few[i] < k ? 1u : 0u;
        if (t < c && below + 1u == want) last = k;
    }
    __syncthreads();
    const u64 limit = last + ((u64)lo << 32);
    for (;;) {
        const bool released = m >= 0 && own > limit;  // (each end by its own lane)
        if (released) mate[w] = -1;
        const u64 stays = prim::ballot(w < nv && (m < 0 || released || m > w));
        if (lane == 0) smem[t / 64] = (u32)__popcll(stays);
        __syncthreads();
        const int tile = w / BUDGET_THREADS * BUDGET_TILES + t;
        if (t < BUDGET_TILES && tile < (nv + BLOCK - 1) / BLOCK)
            tilesum[tile] = (int)((smem[4 * t] + smem[4 * t + 1]) + (smem[4 * t + 2] + smem[4 * t + 3]));
        w += ((int)gridDim.x - 1) * BUDGET_THREADS;
        if (w - t >= nv) break;
        m = w < nv ? mate[w] : -1;
        own = pair_key();
        __syncthreads();
    }
}

// Where rounds by rings end before the call does: what the round by facets that follows takes (the facets, no bids, no count of facets), and the labels in the present numbering,
// where a contraction's map is still to be applied to them (vmap, or null).  A copy and three fills instead took 10 us longer at 1.2 M vertices, 1 to 7 at 115 k and as long at 4 k.
__global__ __launch_bounds__(BLOCK) void facets_again_kernel(const int* __restrict__ facets, int F, int* __restrict__ fcur, int nv, u64* __restrict__ vmin0,
                                                             u64* __restrict__ vmin1, int* __restrict__ facet_slots, int* __restrict__ cid,
                                                             const int* __restrict__ vmap, int n_labels) {
    const int g = blockIdx.x * BLOCK + threadIdx.x, stride = gridDim.x * BLOCK;
    if (g < MATCH_SLOTS) facet_slots[g * MATCH_PAD] = 0;
    for (long long f = g; f < F; f += stride) {
        const Corners q = load_corners(facets, (size_t)f);
        fcur[3 * f] = q.a;
        fcur[3 * f + 1] = q.b;
        fcur[3 * f + 2] = q.c;
    }
    for (long long v = g; v < nv; v += stride) vmin0[v] = vmin1[v] = VMIN_NONE;
    if (vmap)
        for (long long o = g; o < n_labels; o += stride) cid[o] = vmap[cid[o]];
}

constexpr u64 ABID_NONE = ~0ull;

// The end of an edge that line 11 of Alg. 2 could add to the other end's cluster: the un-paired
// one when exactly one end is paired, else -1.
__device__ __forceinline__ int joining_end(const int* __restrict__ mate, int u, int v) {
    const bool pu = mate[u] >= 0, pv = mate[v] >= 0;
    return pu == pv ? -1 : (pu ? v : u);
}

// ---------------------------------------------------------------------------
// S2b + budget (Alg. 2 lines 3-4, 6): when a mesh formed more pairs than it may
// remove, only its n_rem pairs of smallest (cost key, tie-break) stay.  A pair stands at its lower vertex (PairKeys):
// among equal costs the order by edge index is the order by that vertex.  The step for the vertices that join clusters
// (line 11) is the same with the candidate vertices in place of pairs (JoinKeys).  So both walk the mesh's vertices, four bytes
// each, and neither the edges nor a gathered list: where the pairs were gathered from the edges, searched and released, that
// took four launches and 41 us for a mesh of 29 k pairs, 22 us for one of 550, and eleven launches for a longer run; now two
// and 40, one and 13, and seven.
// ---------------------------------------------------------------------------
template <bool SHUFFLE>
struct PairKeys {
    const u32* pcost;
    const u32* ptie;
    int* mate;
    static constexpr bool TIE_BY_VERTEX = !SHUFFLE;
    typedef u32 Raw;
    static constexpr Raw NONE = PAIR_NONE;
    __device__ __forceinline__ Raw load(int w) const { return pcost[w]; }
    __device__ __forceinline__ void load4(int w, Raw* r) const {  // (w: a multiple of 4)
        const uint4 q = *reinterpret_cast<const uint4*>(pcost + w);
        r[0] = q.x; r[1] = q.y; r[2] = q.z; r[3] = q.w;
    }
    __device__ __forceinline__ bool has(Raw r) const { return r != PAIR_NONE; }
    __device__ __forceinline__ u32 cost(Raw r) const { return r; }
    __device__ __forceinline__ u32 tie(int w, int v0) const { return SHUFFLE ? ptie[w] : (u32)(w - v0); }
    __device__ __forceinline__ int partner(int w) const { return mate[w]; }
    // the pair is dissolved
    __device__ __forceinline__ void release(int w, int m) const {
        mate[w] = -1;
        mate[m] = -1;
    }
};

struct JoinKeys {
    u64* abid;
    static constexpr bool TIE_BY_VERTEX = false;
    typedef u64 Raw;
    static constexpr Raw NONE = ABID_NONE;
    __device__ __forceinline__ Raw load(int w) const { return abid[w]; }
    __device__ __forceinline__ void load4(int w, Raw* r) const {
        const ulonglong2* q = reinterpret_cast<const ulonglong2*>(abid + w);
        const ulonglong2 a = q[0], b = q[1];
        r[0] = a.x; r[1] = a.y; r[2] = b.x; r[3] = b.y;
    }
    __device__ __forceinline__ bool has(Raw r) const { return r != ABID_NONE; }
    __device__ __forceinline__ u32 cost(Raw r) const { return (u32)(r >> 32); }
    __device__ __forceinline__ u32 tie(int w, int) const { return (u32)abid[w]; }
    // the vertex that would have joined stays on its own: its bid is withdrawn
    __device__ __forceinline__ int partner(int) const { return -1; }
    __device__ __forceinline__ void release(int w, int) const { abid[w] = ABID_NONE; }
};

// Meshes with at most `longer_than` keys (<= cap where any has more): one workgroup per mesh finds the budget's last key, ordered by
// (cost key, tie-break value).  What may be it is listed in LDS in any order: all keys of up to TRUNC_DIRECT, of more those whose costs
// lie about where a sample of 4,096 vertices has the budget's last one; should the sample mislead, or too many costs be equal, the
// range is narrowed by counts of all keys instead, 12 bits a walk.  Of the list, counts of 12 bits a time from the highest bit
// in which its costs can differ leave 64 or less, which one wave ranks.  What lies beyond is released by the kernel that counts the survivors
// (ReleasingPred), or, where something else reads the pairs before it, by trunc_release_kernel or (few keys) here.
// Bound by the issue of one compute unit (a vector instruction per vertex is 0.4 us for 62 k of them; the walk itself takes 3.4, 16 bytes a
// load, the next step's ahead) and by LDS atomics of clustered costs, which take turns: hence a walk that only compares, and counts
// of the listed keys alone.  115 k vertices (62 k and 28 k pairs in the last round): 35 us with counts of all keys, the others and the ties
// listed by walks of their own, and 5 for the release; now 21.  4 k vertices (550 pairs): 12.7, now 5.8; 16 meshes of 32 k vertices: 24 + 5, now 17.
//
// Up to TRUNC_BLOCK_CAP keys a mesh goes this way, because its search, one launch that knows nothing of the host, can be queued
// ahead of the host's look; the whole chip's (below) takes seven or eight.  Whole calls of one round with three quarters of the pairs
// staying, this way / the other: one mesh of 539 pairs 92 / 116 us, 2,139 100 / 129, 8,576 119 / 147, 17,022 134 / 156; eight meshes of
// 2,139 pairs 133 / 162, of 17,022 283 / 301.  Beyond the cap the keys of a mesh may not fit LDS.
constexpr int TRUNC_THREADS = 1024;
constexpr int TRUNC_BLOCK_CAP = 32 * TRUNC_THREADS;
constexpr int TRUNC_SMALL_CAP = 4 * TRUNC_THREADS;  // up to here the release is made here, where the count does not make it
constexpr int TRUNC_LIST = 16 * TRUNC_THREADS, TRUNC_DIRECT = 2 * TRUNC_THREADS;

// What stays of a mesh's keys: those below `cost`, and at it those with tie-break values up to `tie`, or all of them.
struct KeyLimit {
    u32 cost, tie;
    int over;  // 0: every key stays; 1: see above; 3: none stays
};
template <class Keys>
__device__ __forceinline__ bool beyond(const Keys& K, const KeyLimit& L, u32 cost, int w, int v0) {
    return L.over == 3 || cost > L.cost || (cost == L.cost && K.tie(w, v0) > L.tie);
}

template <class Keys>
__global__ __launch_bounds__(TRUNC_THREADS) void trunc_mesh_kernel(Keys K, const int* __restrict__ voff,
                                                                   const int* __restrict__ counts,
                                                                   const int* __restrict__ budgets, int cap, int longer_than,
                                                                   const int* __restrict__ guard, State* st, HostSignal tell,
                                                                   KeyLimit* __restrict__ limits, PairPublish publish) {
    constexpr int Q = 16, STEP = Q * TRUNC_THREADS, WALK_BITS = 12;
    static_assert(1 << WALK_BITS == 4 * TRUNC_THREADS, "four digits per thread");
    __shared__ u64 list[TRUNC_LIST];
    __shared__ uint4 hist4[TRUNC_THREADS];  // counts per digit
    __shared__ u32 smem[TRUNC_THREADS / 64];
    __shared__ u64 found_key, few[64];
    __shared__ u32 found[4];
    __shared__ u32 n_list, n_below;
    u32* hist = reinterpret_cast<u32*>(hist4);
    const int b = blockIdx.x, tid = threadIdx.x, lane = prim::lane_id();
    if (b == publish.at) {
        publish_pairs(publish);
        return;
    }
    if (b == 0 && tid == 0) tell_host(tell);
    // (all of these loads are in flight together)
    const int go = guard ? *guard : 1, keep = budgets[b], v0 = voff[b], v1 = voff[b + 1];
    int n = publish.at >= 0 ? publish.mslots[((size_t)b * MATCH_SLOTS + (tid & (MATCH_SLOTS - 1))) * MATCH_PAD] : counts[b];
    if (publish.at >= 0)
#pragma unroll
        for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
    if (limits && tid == 0) limits[b] = KeyLimit{0u, 0u, 0};
    if (go == 0) return;  // queued ahead of the host's look, and the selection was not finished
    if (n <= keep) return;
    if (n > longer_than) return;  // another kernel for these follows
    if (n > cap) {
        // More keys than this instance holds: the host never launches it so.
        // Nothing is released, and the call is made to fail instead of returning a budget that was not applied.
        if (tid == 0) atomicOr(&st->err, ERR_BIT_INTERNAL);
        return;
    }
    typedef typename Keys::Raw Raw;
    const int first = v0 & ~3;
    const int at = 4 * tid;
    auto vertex_of = [&](int q) { return (q >> 2) * (4 * TRUNC_THREADS) + at + (q & 3); };
    // fn(first vertex, keys of the vertices first + vertex_of(q), Keys::NONE outside the mesh) step by step, by whole waves; the next step's
    // keys are fetched meanwhile
    auto each_step = [&](auto fn) {
        Raw next[Q];
        auto fetch = [&](int base) {
#pragma unroll
            for (int q = 0; q < Q; q += 4) K.load4(min(base + vertex_of(q), (v1 - 1) & ~3), &next[q]);
        };
        fetch(first);
        for (int base = first; base < v1; base += STEP) {
            Raw raw[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) raw[q] = next[q];
            if (base + STEP < v1) fetch(base + STEP);
            if (base < v0 || base + STEP > v1) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int w = base + vertex_of(q);
                    if (w < v0 || w >= v1) raw[q] = Keys::NONE;
                }
            }
            fn(base, raw);
        }
    };
    // Lists (cost key << 32) | vertex of the costs from lo to hi; n_list of them (the list may hold less), n_below in front of lo.
    auto list_range = [&](u32 lo, u32 hi) {
        if (tid == 0) n_list = n_below = 0;
        __syncthreads();
        u32 less = 0;
        each_step([&](int base, const Raw (&raw)[Q]) {
            u32 mine = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const u32 cost = K.cost(raw[q]);  // (of Keys::NONE: above every hi)
                less += cost < lo ? 1u : 0u;
                mine += cost - lo <= hi - lo ? 1u : 0u;
            }
            if (!__any(mine != 0)) return;
            const u32 incl = prim::wave_inclusive_scan(mine);
            u32 p = 0;
            if (lane == 63) p = atomicAdd(&n_list, incl);
            p = (u32)__builtin_amdgcn_readlane((int)p, 63) + incl - mine;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const u32 cost = K.cost(raw[q]);
                if (cost - lo <= hi - lo) {
                    if (p < (u32)TRUNC_LIST) list[p] = ((u64)cost << 32) | (u32)(base + vertex_of(q));
                    ++p;
                }
            }
        });
        less = prim::wave_inclusive_scan(less);
        if (lane == 63 && less) atomicAdd(&n_below, less);
        __syncthreads();
    };
    // From the counts, the digits of 12 bits in which the want-th and the want2-th of those counted lie, want and want2 from the number
    // of all: found[0] (found[1] in front of it, found[2] in it) and found[3].
    auto pick = [&](auto wants) {
        const uint4 c4 = hist4[tid];
        const u32 c[4] = {c4.x, c4.y, c4.z, c4.w};
        u32 tot, run = prim::wide_block_exclusive_scan<TRUNC_THREADS / 64>((c[0] + c[1]) + (c[2] + c[3]), smem, tot);
        u32 want, want2;
        wants(tot, want, want2);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (run < want && want <= run + c[j]) {  // (in one thread)
                found[0] = (u32)(tid * 4 + j);
                found[1] = run;
                found[2] = c[j];
            }
            if (run < want2 && want2 <= run + c[j]) found[3] = (u32)(tid * 4 + j);
            run += c[j];
        }
        __syncthreads();
        return tot;
    };
    auto clear_counts = [&]() {
        hist4[tid] = make_uint4(0, 0, 0, 0);
        __syncthreads();
    };
    u64 last = 0;  // the last key that stays
    const bool none = keep <= 0;
    if (!none) {
        constexpr u32 HIGHEST = 0xFFFFFFFEu;  // (a key has a finite cost)
        u32 lo = 0, hi = HIGHEST;
        if (n > TRUNC_DIRECT) {
            Raw some[4];  // four vertices in a row per lane, evenly over the mesh
            const int w0 = (int)(((long long)(v1 - first) * tid) >> 10) / 4 * 4 + first;
            K.load4(w0, some);
            clear_counts();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (w0 + q >= v0 && w0 + q < v1 && K.has(some[q])) atomicAdd(&hist[K.cost(some[q]) >> (32 - WALK_BITS)], 1u);
            __syncthreads();
            // (six standard deviations of a rank in the middle of a sample of `all`: neighbours are alike)
            u32 r0 = 0, r1 = 0;
            const u32 all = pick([&](u32 all, u32& want, u32& want2) {
                const float rank = (float)all * (float)keep / (float)n, margin = 3.0f * sqrtf((float)all) + 4.0f;
                r0 = want = rank > margin ? (u32)(rank - margin) : 0u;
                r1 = want2 = min((u32)(rank + margin), all + 1u);
            });
            if (r0 > 0) lo = found[0] << (32 - WALK_BITS);
            if (r1 > 0 && r1 <= all) hi = min(HIGHEST, (found[3] << (32 - WALK_BITS)) | ((1u << (32 - WALK_BITS)) - 1u));
            __syncthreads();
        }
        list_range(lo, hi);
        int bit = 32 - __clz((int)(lo ^ hi));  // bits of the listed costs from here on are the same (-1 .. : none differ)
        u32 tie_prefix = 0;  // what their tie-break values share from tie_bit on, where one cost is listed
        int tie_bit = Keys::TIE_BY_VERTEX ? 32 - __clz(v1 - v0) : 32;
        if (!(n_below < (u32)keep && (u32)keep <= n_below + n_list && n_list <= (u32)TRUNC_LIST)) {
            // digit by digit by counts of all keys: of the cost key, then of the tie-break values at that cost
            u32 cost = 0, tie = 0, below = 0;
            int undecided = 64;
            for (;;) {
                const int nb = undecided == 40 || undecided == 8 ? 8 : WALK_BITS;  // (12, 12 and 8 bits of either)
                undecided -= nb;
                __syncthreads();
                clear_counts();
                each_step([&](int base, const Raw (&raw)[Q]) {
#pragma unroll 4
                    for (int q = 0; q < Q; ++q) {
                        if (!K.has(raw[q])) continue;
                        u32 k = K.cost(raw[q]), decided = cost;
                        int above = undecided + nb - 32;
                        if (undecided < 32) {
                            if (k != cost) continue;
                            k = K.tie(base + vertex_of(q), v0);
                            decided = tie;
                            above += 32;
                        }
                        if (above < 32 && k >> above != decided >> above) continue;
                        atomicAdd(&hist[(k >> (above - nb)) & ((1u << nb) - 1u)], 1u);
                    }
                });
                __syncthreads();
                pick([&](u32, u32& want, u32& want2) {
                    want = (u32)keep - below;
                    want2 = 0;
                });
                if (undecided >= 32) cost |= found[0] << (undecided - 32);
                else tie |= found[0] << undecided;
                below += found[1];
                if (found[2] <= (u32)TRUNC_LIST) break;
            }
            __syncthreads();
            lo = cost;
            hi = undecided > 32 ? cost | ((1u << (undecided - 32)) - 1u) : cost;
            bit = undecided > 32 ? undecided - 32 : 0;
            if (undecided >= 32) {
                list_range(lo, hi);
            } else {  // at that cost only the ones with the tie-break values' leading digits
                tie_prefix = tie;
                tie_bit = undecided;
                if (tid == 0) {
                    n_list = 0;
                    n_below = below;
                }
                __syncthreads();
                each_step([&](int base, const Raw (&raw)[Q]) {
#pragma unroll 4
                    for (int q = 0; q < Q; ++q) {
                        const int w = base + vertex_of(q);
                        if (!K.has(raw[q]) || K.cost(raw[q]) != cost || K.tie(w, v0) >> tie_bit != tie >> tie_bit) continue;
                        const u32 place = atomicAdd(&n_list, 1u);
                        if (place < (u32)TRUNC_LIST) list[place] = ((u64)cost << 32) | (u32)w;
                    }
                });
                __syncthreads();
            }
        }
        const int m = (int)min(n_list, (u32)TRUNC_LIST);
        u32 want = (u32)keep - n_below;
        u32* half = reinterpret_cast<u32*>(list);  // (tie-break value or vertex, cost) of entry i at 2 i
        for (int i = tid; i < m; i += TRUNC_THREADS) half[2 * i] = K.tie((int)half[2 * i], v0);
        __syncthreads();
        // of the list, by the costs and then the tie-break values: until 64 or less are left, which one wave ranks
        u32 equal = (u32)m, prefix[2] = {0, 0};
        int from[2] = {32, 32};  // the word's bits from here on are decided
#pragma unroll
        for (int word = 1; word >= 0; --word) {
            from[word] = word == 1 ? bit : tie_bit;
            if (word == 1) prefix[1] = bit >= 32 ? 0u : lo & (~0u << bit);
            else prefix[0] = tie_prefix;
            while (equal > 64u && from[word] > 0) {
                const int nb = min(WALK_BITS, from[word]), shift = from[word] - nb;
                const u32 decided = from[word] >= 32 ? 0u : ~0u << from[word];
                clear_counts();
                for (int i = tid; i < m; i += TRUNC_THREADS) {
                    const u32 k = half[2 * i + word];
                    if ((k & decided) == prefix[word] && (word == 1 || half[2 * i + 1] == prefix[1]))
                        atomicAdd(&hist[(k >> shift) & ((1u << nb) - 1u)], 1u);
                }
                __syncthreads();
                pick([&](u32, u32& first_want, u32& second_want) {
                    first_want = want;
                    second_want = 0;
                });
                prefix[word] |= found[0] << shift;
                want -= found[1];
                equal = found[2];
                from[word] = shift;
                __syncthreads();
            }
        }
        if (tid == 0) n_list = 0;
        __syncthreads();
        const u32 d1 = from[1] >= 32 ? 0u : ~0u << from[1], d0 = from[0] >= 32 ? 0u : ~0u << from[0];
        for (int i = tid; i < m; i += TRUNC_THREADS)
            if ((half[2 * i + 1] & d1) == prefix[1] && (half[2 * i] & d0) == prefix[0]) {
                const u32 p = atomicAdd(&n_list, 1u);
                if (p < 64u) few[p] = list[i];
            }
        __syncthreads();
        if (tid < 64) {
            const int c = (int)min(n_list, 64u);
            const u64 k = few[min(tid, c - 1)];
            u32 rank = 0;
            for (int i = 0; i < c; ++i) rank += few[i] < k ? 1u : 0u;
            if (tid < c && rank + 1u == want) found_key = k;
        }
        __syncthreads();
        last = found_key;
    }
    const KeyLimit limit{(u32)(last >> 32), (u32)last, none ? 3 : 1};
    if (limits) {
        if (tid == 0) limits[b] = limit;
        return;
    }
    each_step([&](int base, const Raw (&raw)[Q]) {
        u32 out = 0;
        int with[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int w = base + vertex_of(q);
            if (K.has(raw[q]) && beyond(K, limit, K.cost(raw[q]), w, v0)) out |= 1u << q;
            with[q] = K.partner(max(min(w, v1 - 1), v0));
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (out >> q & 1u) K.release(base + vertex_of(q), with[q]);
    });
}

// The release by the whole chip, where the search leaves it to this (the stores of 29 k pairs take one compute unit 20 us).
template <class Keys>
__global__ __launch_bounds__(BLOCK) void trunc_release_kernel(Keys K, int nv, const int* __restrict__ voff, int B,
                                                              const KeyLimit* __restrict__ limits) {
    const int w = blockIdx.x * BLOCK + threadIdx.x;
    if (w >= nv) return;
    const int b = mesh_of(voff, B, w);
    const KeyLimit limit = limits[b];
    if (limit.over == 0) return;
    const typename Keys::Raw raw = K.load(w);
    const int with = K.partner(w);
    if (K.has(raw) && beyond(K, limit, K.cost(raw), w, voff[b])) K.release(w, with);
}

// Longer runs: the same search by histogram passes over the mesh's vertices with the whole chip (blockIdx.y = mesh, from b0 on), three of
// 12, 12 and 8 bits for the cost key and as many as the tie-break values have digits.  A pass's workgroups each pick the digit
// that the pass before has decided from its counts (16 KB read from L2, no launch in between).
constexpr int SELECT_BITS = 12, SELECT_BINS = 1 << SELECT_BITS, SELECT_COST_PASSES = 3, SELECT_PASSES = 6;
struct SelectSlot {
    u32 hist[SELECT_PASSES][SELECT_BINS];  // (zero before the first pass)
    // as picked by the pass: what is decided of the cost key, keys below it; the same of the tie-break value; stay = how many
    // of the keys at the decided cost key stay; all = they all do
    struct {
        u32 cost, below, tie, tie_below, stay, all;
    } at[SELECT_PASSES + 1];
};
// A mesh's slot.  A key stands at a vertex of its own (a pair at its lower one, a vertex that could join at itself), so meshes of
// more than 2^SELECT_SLOT_BITS keys start more than 2^SELECT_SLOT_BITS vertices apart: they go by their starts, and no two share
// a slot.  Where shorter runs come here too (the option that lowers the limit) the meshes take turns, SELECT_MESHES of
// them at a time (98 KB a slot).
constexpr int SELECT_SLOT_BITS = 15, SELECT_MESHES = 8;
constexpr int SELECT_GRID_MESHES = 1 << 15;  // meshes of a launch (a grid has at most 65,535 rows)
static_assert(1 << SELECT_SLOT_BITS == TRUNC_BLOCK_CAP, "by default only meshes of more than TRUNC_BLOCK_CAP keys come here");
inline int select_slots_by_start(int B, long long n_verts) { return B > 1 ? (int)(n_verts >> SELECT_SLOT_BITS) + 1 : 1; }
__device__ __forceinline__ int select_slot(const int* voff, int by_start, int b) {
    return by_start ? voff[b] >> SELECT_SLOT_BITS : (int)blockIdx.y;
}
__device__ __forceinline__ int select_shift(int j, int bits) { return max(0, bits - SELECT_BITS * (j + 1)); }
__device__ __forceinline__ int select_width(int j, int bits) { return min(SELECT_BITS, bits - SELECT_BITS * j); }

// The state before pass `pass` (by a whole workgroup): from the pass before, its counts and the state before it.
__device__ __forceinline__ auto select_pick(const SelectSlot& S, int pass, u32 keep, int tie_bits, u32* smem, u32* out /* [3] */) {
    auto a = S.at[0];
    a.cost = a.below = a.tie = a.tie_below = a.stay = a.all = 0;
    if (pass == 0) return a;
    constexpr int PER = SELECT_BINS / BLOCK;
    if (pass > 1) a = S.at[pass - 1];
    const int t = threadIdx.x;
    const bool tie = pass - 1 >= SELECT_COST_PASSES;
    const u32 need = tie ? a.stay - a.tie_below : keep - a.below;  // >= 1: the key sought is among those counted
    u32 c[PER], sum = 0, tot;
#pragma unroll
    for (int j = 0; j < PER; ++j) sum += c[j] = S.hist[pass - 1][t * PER + j];
    u32 run = prim::block_exclusive_scan(sum, smem, tot);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (run < need && need <= run + c[j]) {  // (in one thread)
            out[0] = (u32)(t * PER + j);
            out[1] = run;
            out[2] = c[j];
        }
        run += c[j];
    }
    __syncthreads();
    if (tie) {
        if (!a.all) {
            a.tie = (a.tie << select_width(pass - 1 - SELECT_COST_PASSES, tie_bits)) | out[0];
            a.tie_below += out[1];
        }
    } else {
        a.cost = (a.cost << select_width(pass - 1, 32)) | out[0];
        a.below += out[1];
        if (pass == SELECT_COST_PASSES) {
            a.stay = keep - a.below;
            a.all = out[2] <= a.stay ? 1u : 0u;
        }
    }
    return a;
}

constexpr int SELECT_ITEMS = 8;
template <class Keys>
__global__ __launch_bounds__(BLOCK) void select_pass_kernel(Keys K, const int* __restrict__ voff,
                                                            const int* __restrict__ counts, const int* __restrict__ budgets,
                                                            int longer_than, SelectSlot* __restrict__ slots, int by_start, int b0, int pass,
                                                            int tie_bits) {
    __shared__ u32 h[SELECT_BINS];
    __shared__ u32 smem[prim::WAVES], picked[3];
    const int b = b0 + (int)blockIdx.y, n = counts[b], keep = budgets[b];
    if (n <= keep || n <= longer_than || keep <= 0) return;
    const int v0 = voff[b], v1 = voff[b + 1], t = threadIdx.x;
    const long long base = (long long)v0 + (long long)blockIdx.x * (BLOCK * SELECT_ITEMS);
    if (base >= v1) return;
    SelectSlot& S = slots[select_slot(voff, by_start, b)];
    const auto a = select_pick(S, pass, (u32)keep, tie_bits, smem, picked);
    if (blockIdx.x == 0 && t == 0) S.at[pass] = a;
    const bool tie = pass >= SELECT_COST_PASSES;
    if (tie && a.all) return;
    const int j = tie ? pass - SELECT_COST_PASSES : pass, bits = tie ? tie_bits : 32, shift = select_shift(j, bits), width = select_width(j, bits);
    for (int i = t; i < SELECT_BINS; i += BLOCK) h[i] = 0;
    typename Keys::Raw raw[SELECT_ITEMS];
#pragma unroll
    for (int i = 0; i < SELECT_ITEMS; ++i) raw[i] = K.load((int)min(base + i * BLOCK + t, (long long)v1 - 1));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SELECT_ITEMS; ++i) {  // (whole waves run every step, for the ballots)
        bool ok = base + i * BLOCK + t < v1 && K.has(raw[i]);
        u32 k = K.cost(raw[i]);
        if (tie) {
            ok = ok && k == a.cost;
            k = ok ? K.tie((int)(base + i * BLOCK + t), v0) : 0u;
        }
        // keys that share the digits decided so far; cost keys cluster, so the lanes of a wave that hold
        // one digit count themselves with a single LDS atomic
        ok = ok && (j == 0 || (k >> (shift + width)) == (tie ? a.tie : a.cost));
        const u32 d = (k >> shift) & ((1u << width) - 1u);
        const prim::SameDigit same = prim::wave_same_digit(ok, d);
        if (ok && same.below == 0) atomicAdd(&h[d], same.count);
    }
    __syncthreads();
    for (int i = t; i < SELECT_BINS; i += BLOCK) {
        const u32 c = h[i];
        if (c) atomicAdd(&S.hist[pass][i], c);
    }
}

// ... and the release: `passes` = passes made.
template <class Keys>
__global__ __launch_bounds__(BLOCK) void select_release_kernel(Keys K, const int* __restrict__ voff,
                                                               const int* __restrict__ counts, const int* __restrict__ budgets,
                                                               int longer_than, const SelectSlot* __restrict__ slots, int by_start, int b0,
                                                               int passes, int tie_bits) {
    __shared__ u32 smem[prim::WAVES], picked[3];
    const int b = b0 + (int)blockIdx.y, n = counts[b], keep = budgets[b];
    if (n <= keep || n <= longer_than) return;
    const int v0 = voff[b], v1 = voff[b + 1];
    const long long base = (long long)v0 + (long long)blockIdx.x * (BLOCK * SELECT_ITEMS);
    if (base >= v1) return;
    const bool none = keep <= 0;
    const SelectSlot& S = slots[select_slot(voff, by_start, b)];
    const auto a = select_pick(S, none ? 0 : passes, (u32)keep, tie_bits, smem, picked);
#pragma unroll
    for (int i = 0; i < SELECT_ITEMS; ++i) {
        const long long w = base + i * BLOCK + threadIdx.x;
        if (w >= v1) continue;
        const typename Keys::Raw raw = K.load((int)w);
        const u32 cost = K.cost(raw);
        if (K.has(raw) &&
            (none || cost > a.cost || (cost == a.cost && !a.all && K.tie((int)w, v0) > a.tie)))
            K.release((int)w, K.partner((int)w));
    }
}

// ---------------------------------------------------------------------------
// Alg. 2 line 11 (option), under the vertex budget: after the pairs are final,
// an un-paired vertex next to a paired one joins that pair's cluster through
// its cheapest such edge (cost key, edge index) -- the first the sequential
// walk over the sorted pairs would reach.  Every joining vertex has its own
// edge, so the priorities are distinct; where a mesh has more candidates than
// budget left, the cheapest stay (the same machinery as for the pairs).  Only
// the two founders of a cluster attract: a vertex that joined pulls in nobody.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void absorb_begin_kernel(u64* __restrict__ abid, int* __restrict__ arep,
                                                             const State* st, int cur, int B,
                                                             const int* __restrict__ nrem,
                                                             const int* __restrict__ matched, int* __restrict__ arem,
                                                             int* __restrict__ acand) {
    const int nv = st->nv[cur];
    const int stride = gridDim.x * BLOCK;
    const int g = blockIdx.x * BLOCK + threadIdx.x;
    for (int w = g; w < nv; w += stride) {
        abid[w] = ABID_NONE;
        arep[w] = -1;
    }
    for (int b = g; b < B; b += stride) {
        const int left = nrem[b] - matched[b];
        arem[b] = (matched[b] > 0 && left > 0) ? left : 0;  // budget left once the pairs are formed
        acand[b] = 0;
    }
}

__global__ __launch_bounds__(BLOCK) void absorb_bid_kernel(const u64* __restrict__ ekey, const u32* __restrict__ ecost,
                                                           const State* st, int vbits, const int* __restrict__ mate,
                                                           MeshTab mt, const int* __restrict__ arem,
                                                           u64* __restrict__ abid, TieBreak tb) {
    const int n = st->ne;
    for (int e = blockIdx.x * BLOCK + threadIdx.x; e < n; e += gridDim.x * BLOCK) {
        const u64 k = ekey[e];
        const int u = (int)(k >> vbits), v = (int)(k & ((1ull << vbits) - 1ull));
        const int w = joining_end(mate, u, v);
        if (w >= 0 && arem[mesh_of(mt.voff, mt.B, w)] > 0) atomicMin(&abid[w], tb.priority(ecost[e], e));
    }
}

// Edge e is the one through which its un-paired end joins (its bid stands at that vertex).
struct JoinPred {
    const u64* ekey;
    const u32* ecost;
    const int* mate;
    const u64* abid;
    int vbits;
    TieBreak tb;
    __device__ bool operator()(int e) const {
        const u64 k = ekey[e];
        const int w = joining_end(mate, (int)(k >> vbits), (int)(k & ((1ull << vbits) - 1ull)));
        return w >= 0 && abid[w] == tb.priority(ecost[e], e);
    }
};

struct JoinListOut {
    int* list;
    __device__ void operator()(int e, int pos) const { list[pos] = e; }
};

// The joining edges are listed in edge order, hence by mesh: acand[b] = how many belong to mesh b.
// Also written to host memory (`host_out`), which the host reads once `done` tells it to.
// One workgroup; ABSORB_WAYS lanes look for a mesh's end in the list together, so that a step, two loads one behind the other, leaves a
// 16th of it.  (8 meshes, 13,000 listed edges: 11.2 us with a lane that halved the list for either end of its mesh, now 5.1.)
constexpr int ABSORB_COUNT_THREADS = 1024, ABSORB_WAYS = 16, ABSORB_ENDS = ABSORB_COUNT_THREADS / ABSORB_WAYS;
__global__ __launch_bounds__(ABSORB_COUNT_THREADS) void absorb_count_kernel(const int* __restrict__ list, const State* st,
                                                                            const u64* __restrict__ ekey, int vbits, int B,
                                                                            const int* __restrict__ voff, int* __restrict__ acand,
                                                                            int* __restrict__ host_out, HostSignal done) {
    __shared__ int ends[ABSORB_ENDS + 1];  // [0]: the end of the mesh in front
    const int n = st->absorb_n, t = threadIdx.x, way = t % ABSORB_WAYS, mine = t / ABSORB_WAYS;
    const int group_at = prim::lane_id() - way;  // the group's first lane
    if (t == 0) ends[0] = 0;
    for (int b0 = 0; b0 < B; b0 += ABSORB_ENDS) {
        const int b = b0 + mine;
        const int v1 = b < B ? voff[b + 1] : 0;
        int lo = b + 1 < B ? 0 : n, hi = n;  // the first listed edge whose lower vertex is at or past v1 (the last mesh's end needs no search)
        while (prim::ballot(lo < hi)) {
            const int step = (hi - lo + ABSORB_WAYS - 1) / ABSORB_WAYS, at = lo + way * step;
            const bool in_front = at < hi && (int)(ekey[list[at]] >> vbits) < v1;
            const int c = __popc((u32)(prim::ballot(in_front) >> group_at) & ((1u << ABSORB_WAYS) - 1u));
            hi = c == 0 ? lo : min(lo + c * step, hi);
            lo = c == 0 ? lo : lo + (c - 1) * step + 1;
        }
        if (way == 0) ends[mine + 1] = lo;
        __syncthreads();
        if (t < ABSORB_ENDS && b0 + t < B) {
            const int count = ends[t + 1] - ends[t];
            acand[b0 + t] = count;
            host_out[b0 + t] = count;
        }
        const int last = ends[ABSORB_ENDS];  // (in front of the barrier: behind it the next turn's ends are stored)
        __syncthreads();
        if (t == 0) ends[0] = last;  // (read by this thread only)
    }
    signal_host(done, t, t < min(B, ABSORB_ENDS));
}

// For every listed edge that still stands: the joining vertex records its cluster's representative
// (the founding pair's smaller index) and leaves the key (representative, vertex), whose digit is counted; withdrawn ones
// leave the all-ones key, which the sort does not keep.
__global__ __launch_bounds__(BLOCK) void absorb_keys_kernel(const int* __restrict__ list, const State* st,
                                                            const u64* __restrict__ ekey,
                                                            const u32* __restrict__ ecost, int vbits,
                                                            const int* __restrict__ mate, const u64* __restrict__ abid,
                                                            int* __restrict__ arep, u64* __restrict__ akey, DigitCount digits,
                                                            TieBreak tb) {
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    u64 out = edge_sentinel(vbits);
    if (i < st->absorb_n) {
        const int e = list[i];
        const u64 k = ekey[e];
        const int u = (int)(k >> vbits), v = (int)(k & ((1ull << vbits) - 1ull));
        const int w = joining_end(mate, u, v);
        if (w >= 0 && abid[w] == tb.priority(ecost[e], e)) {
            const int o = (w == u) ? v : u;
            const int mo = mate[o];
            const int r = o < mo ? o : mo;
            arep[w] = r;
            out = ((u64)(u32)r << vbits) | (u64)(u32)w;
        }
        akey[i] = out;
    }
    const bool joins = out != edge_sentinel(vbits);
    const u32 d = (u32)(out >> digits.shift) & digits.mask;
    const prim::SameDigit same = prim::wave_same_digit(joins, d);
    if (joins && same.below == 0) atomicAdd(&digits.hist[d], same.count);
}
// ... and the source of their sort, whose lists (RowLists) are what joins every representative's cluster.
struct JoinedKeys {
    const u64* p;
    u64 none;
    static constexpr int PER = 1;
    typedef u64 Raw;
    __device__ __forceinline__ u64 load(int i) const { return p[i]; }
    __device__ __forceinline__ u64 key(u64 raw, int, int) const { return raw; }
    __device__ __forceinline__ bool keep(u64 k) const { return k != none; }
};

// ---------------------------------------------------------------------------
// S4 + S6: contraction (Alg. 2 lines 12-16) and survivor renumbering
// ---------------------------------------------------------------------------
template <bool ABSORB>
struct AlivePredT {
    const int* mate;
    const int* arep;
    __device__ bool operator()(int w) const {
        const int m = mate[w];
        if (m >= 0 && m < w) return false;  // the larger index of a pair is replaced by the smaller
        return !(ABSORB && arep[w] >= 0);   // as is a vertex that joined a pair's cluster
    }
};

// The same where a budget step has left the meshes' limits: a pair beyond its mesh's is dissolved on the way, each end by its own lane.
template <bool SHUFFLE>
struct ReleasingPred {
    PairKeys<SHUFFLE> K;
    const int* voff;
    int B;
    const KeyLimit* limits;
    __device__ bool operator()(int w) const {
        const int m = K.mate[w];
        if (m < 0) return true;
        const int b = mesh_of(voff, B, w), lo = min(m, w);
        const KeyLimit limit = limits[b];
        if (limit.over != 0 && beyond(K, limit, K.cost(K.load(lo)), lo, voff[b])) {
            K.mate[w] = -1;
            return true;
        }
        return m > w;
    }
};

// For every offset at[0..B] into a list of flagged and other items, how many flagged items lie in front of it: by every lane of the
// waves that walk the list, whose lanes hold the items i0 + lane; incl = flagged items up to and including the lane's.
__device__ __forceinline__ void flagged_before(const int* __restrict__ at, int B, long long i0, u32 incl, int* __restrict__ out) {
    for (int b0 = 0; b0 <= B; b0 += 64) {
        const int b = b0 + prim::lane_id();
        const int p = b <= B ? at[b] : -1;
        const bool here = p > i0 && p <= i0 + 64;
        const u32 v = (u32)__shfl((int)incl, here ? (int)(p - 1 - i0) : 0, 64);
        if (here) out[b] = (int)v;
        else if (p == 0 && i0 == 0) out[b] = 0;
    }
}

// Survivors get their new number (the count pass of a compaction, AlivePredT, has left the survivors per tile of
// BLOCK * chunks vertices) and move to their new slot; a pair's representative takes the summed
// quadric and the pair's target position (the mean; with PLACE_INVERSE the
// point of least error where there is one).  With ABSORB a cluster may have
// more members than its pair: alist[aoff[w]] .. lists, in ascending order, the vertices that joined
// representative w, and quadric and position are
// summed over all members in ascending index order, the position sum divided
// by their number.  vmap[w] = output slot of w's cluster, written by its representative's lane for all its
// members (numbering and contraction were two launches and an array between them; in one they cost what contracting did).
//
// COUNTS: no count pass has run; a workgroup counts the survivors in front of its tile (chunks = 1) itself, all of them, and tells the
// host what the count pass would have told it.  What it reads grows with the vertices, what it saves is a launch: 4 k vertices 8.4 -> 5.4 us
// (both launches before), 115 k 10.7 -> 21.5; on a straight line between them the two meet at 28 k.
constexpr int CONTRACT_COUNTS_MAX = 1 << 14;
template <int PLACE, bool ABSORB, bool COUNTS>
__global__ __launch_bounds__(BLOCK) void contract_kernel(const VRec* __restrict__ vin, VRec* __restrict__ vout,
                                                         const int* __restrict__ mate, int* __restrict__ vmap, State* st,
                                                         int cur, int chunks, const int* __restrict__ tilesum, int prefixed,
                                                         int B, const int* __restrict__ voff_cur, int* __restrict__ voff_nxt,
                                                         const int* __restrict__ matched, int* __restrict__ done,
                                                         int* __restrict__ htab, int n_clear, u64* __restrict__ vmin0,
                                                         float rcond_min, const int* __restrict__ arep,
                                                         const int* __restrict__ aoff, const int* __restrict__ alist,
                                                         const int* __restrict__ guard, HostSignal tell, PairPublish publish,
                                                         int2* __restrict__ from, ulonglong2* __restrict__ from_info,
                                                         const u64* __restrict__ rings) {
    if (COUNTS && blockIdx.x == 0 && threadIdx.x == 0) tell_host(tell);
    if ((int)blockIdx.x == publish.at) {
        publish_pairs(publish);
        return;
    }
    if (guard && *guard == 0) return;  // queued ahead of the host's look, and the selection was not finished
    __shared__ u32 smem[prim::WAVES];
    const int nv = st->nv[cur];
    const int stride = gridDim.x * BLOCK;
    const int g = blockIdx.x * BLOCK + threadIdx.x;
    for (int i = g; i < n_clear; i += stride) htab[i] = -1;  // (see final_facets_kernel)
    if (publish.at < 0)
        for (int b = g; b < B; b += stride)
            if (matched[b] > 0) done[b] = 1;  // (a mesh without a pair is as it was, whatever the others do)
    const int t = threadIdx.x, w64 = prim::wave_id(), lane = prim::lane_id();
    const int tile = blockIdx.x;
    const long long base = (long long)tile * BLOCK * chunks;
    if (base >= nv) return;
    u32 before = 0;  // survivors in front of this tile
    if (COUNTS) {
        u32 part = 0;
#pragma unroll 4
        for (int j = 4 * t; j < (int)base; j += 4 * BLOCK) {
            const int4 m = *reinterpret_cast<const int4*>(mate + j);
            part += (m.x < 0 || m.x > j) + (m.y < 0 || m.y > j + 1) + (m.z < 0 || m.z > j + 2) + (m.w < 0 || m.w > j + 3);
        }
        before = prim::block_sum(part, smem);
    } else if (prefixed) {
        before = (u32)tilesum[tile];
    } else {
        u32 part = 0;
        for (int j = t; j < tile; j += BLOCK) part += (u32)tilesum[j];
        before = prim::block_sum(part, smem);
    }
    const AlivePredT<ABSORB> survives{mate, arep};
    const long long i0 = base + (long long)w64 * (64 * chunks);  // this wave's part of the tile
    u32 cnt = 0;
    for (int c = 0; c < chunks; ++c) {
        const long long i = i0 + c * 64 + lane;
        cnt += (u32)__popcll(prim::ballot(i < nv && survives((int)i)));
    }
    __syncthreads();
    if (lane == 0) smem[w64] = cnt;
    __syncthreads();
    u32 run = before, tot = 0;
#pragma unroll
    for (int j = 0; j < prim::WAVES; ++j) {
        if (j < w64) run += smem[j];
        tot += smem[j];
    }
    if (base + (long long)BLOCK * chunks >= nv && t == 0) st->nv[cur ^ 1] = (int)(before + tot);
    for (int c = 0; c < chunks; ++c) {
        const long long i = i0 + c * 64 + lane;
        const bool alive = i < nv && survives((int)i);
        const u64 bal = prim::ballot(alive);
        const u32 incl = run + (u32)__popcll(bal & (prim::lanemask_lt() | (1ull << lane)));
        flagged_before(voff_cur, B, i0 + c * 64, incl, voff_nxt);  // a mesh starts behind the survivors of those in front of it
        run += (u32)__popcll(bal);
        if (!alive) continue;
        const int w = (int)i, nw = (int)incl - 1, m = mate[w];
        vmap[w] = nw;
        if (vmin0) vmin0[nw] = VMIN_NONE;  // (the next round's first bids, see facet_costs_kernel)
        const float4* a = reinterpret_cast<const float4*>(&vin[w]);
        float4 r0 = a[0], r1 = a[1], r2 = a[2], r3 = a[3];
        if (from) {  // (rounds by rings, see ring_costs_kernel)
            from[nw] = make_int2(w, m);
            from_info[nw] = make_ulonglong2(rings[w], m >= 0 ? rings[m] : 0ull);
        }
        if (m >= 0) {
            vmap[m] = nw;
            const int j0 = ABSORB ? aoff[w] : 0, jend = ABSORB ? aoff[w + 1] : 0;  // this cluster's part of alist (a pair's lower vertex is not the last one)
            if (!ABSORB || j0 == jend) {
                const float4* b = reinterpret_cast<const float4*>(&vin[m]);
                const float4 s0 = b[0], s1 = b[1], s2 = b[2], s3 = b[3];
                r0.x = (r0.x + s0.x) * 0.5f; r0.y = (r0.y + s0.y) * 0.5f; r0.z = (r0.z + s0.z) * 0.5f;
                r1.x = r1.x + s1.x; r1.y = r1.y + s1.y; r1.z = r1.z + s1.z; r1.w = r1.w + s1.w;
                r2.x = r2.x + s2.x; r2.y = r2.y + s2.y; r2.z = r2.z + s2.z; r2.w = r2.w + s2.w;
                r3.x = r3.x + s3.x; r3.y = r3.y + s3.y;
            } else {
                // merge w < m with the ascending list of joined vertices
                bool done_w = false, done_m = false;
                int cnt_in = 0, j = j0;
                while (!done_w || !done_m || j < jend) {
                    int x = 0x7FFFFFFF, from = -1;
                    if (!done_w) { x = w; from = 0; }
                    else if (!done_m) { x = m; from = 1; }
                    if (j < jend) {
                        const int y = alist[j];
                        if (y < x) { x = y; from = 2; }
                    }
                    if (from == 0) {
                        done_w = true;
                    } else if (from == 1) {
                        done_m = true;
                    } else {
                        vmap[x] = nw;
                        ++j;
                    }
                    const float4* b = reinterpret_cast<const float4*>(&vin[x]);
                    const float4 s0 = b[0], s1 = b[1], s2 = b[2], s3 = b[3];
                    if (cnt_in == 0) {
                        r0 = s0; r1 = s1; r2 = s2; r3 = s3;
                    } else {
                        r0.x = r0.x + s0.x; r0.y = r0.y + s0.y; r0.z = r0.z + s0.z;
                        r1.x = r1.x + s1.x; r1.y = r1.y + s1.y; r1.z = r1.z + s1.z; r1.w = r1.w + s1.w;
                        r2.x = r2.x + s2.x; r2.y = r2.y + s2.y; r2.z = r2.z + s2.z; r2.w = r2.w + s2.w;
                        r3.x = r3.x + s3.x; r3.y = r3.y + s3.y;
                    }
                    ++cnt_in;
                }
                const float k = (float)cnt_in;
                r0.x = r0.x / k; r0.y = r0.y / k; r0.z = r0.z / k;
                r0.w = 0.f; r3.z = 0.f; r3.w = 0.f;
            }
            if (PLACE == PLACE_INVERSE)
                quadric_minimiser(r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z, r2.w, r3.x, rcond_min, r0.x, r0.y, r0.z);
        }
        float4* o = reinterpret_cast<float4*>(&vout[nw]);
        o[0] = r0; o[1] = r1; o[2] = r2; o[3] = r3;
    }
}

// ---------------------------------------------------------------------------
// End of the call: last re-indexing (S5), removal of collapsed and repeated facets, results out
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sort3(int& a, int& b, int& c) {
    int t;
    if (a > b) { t = a; a = b; b = t; }
    if (b > c) { t = b; b = c; c = t; }
    if (a > b) { t = a; a = b; b = t; }
}

__device__ __forceinline__ u32 hash3(int a, int b, int c) {
    u32 h = (u32)a * 0x9E3779B1u;
    h ^= (u32)b * 0x85EBCA77u + (h << 6) + (h >> 2);
    h ^= (u32)c * 0xC2B2AE3Du + (h << 6) + (h >> 2);
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    return h;
}

// Where a triple's search of the table starts: the table follows the vertex numbering (the triple's
// smallest vertex x, scaled from the round's new vertex count to the number of slots; the same x always
// gives the same place, which is all the table needs), plus a few bits of the triple's hash.
// Facets that are neighbours in the mesh are neighbours in the facet list and have nearby smallest
// vertices, so the lanes that handle them meet in the same cache lines of the table, where a uniform
// hash would fetch, and later write back, a whole line for nearly every facet (and the keep test
// that follows reads the table the same way).  Measured at 1.2 M vertices: 3 hash bits are best; with
// none the facets of one vertex collide, with 6 or 9 the lines are shared by fewer facets.  Fewer than 8 slots per vertex
// are worse (4: 5 times the time, collisions), atomics being served at 27 lines of 64 bytes per nanosecond.
constexpr int FACET_HOME_WINDOW_BITS = 3;
constexpr int FACET_HOME_PROBES = 8;
__device__ __forceinline__ u32 facet_home(int x, u32 hx, float slots_per_vertex) {
    const float at = (float)x * slots_per_vertex;  // (below 2^32: x is below the vertex count)
    return (u32)at + (hx & ((1u << FACET_HOME_WINDOW_BITS) - 1u));
}
// ... and by how much its steps grow when FACET_HOME_PROBES places along the line were taken: it goes on from a place that the whole triple decides, by
// one, two, three, ... of these strides.  A vertex may have very many facets, and where vertices are numbered in no order the smallest of a
// facet's three is a low one, so that much of the table's low end is full.  A search must not walk through that: calls that keep 99 % of such
// vertices took 45 ms of 130 k and 270 ms of 500 k with steps along the line from the new place on.  Nor must it try the same crowded stretch from one
// multiple of its stride to the next, or eight places of it in a row: the longest of 20 k random facets on 1 k vertices took 73 trips so (counted on the CPU), now
// 17, and its call, to 95 %, 260 us, now 155.  The strides are odd and the sizes powers of two: every slot is met once, so that a search ends.
__device__ __forceinline__ u32 facet_stride(u32 hx) { return ((hx << 16 | hx >> 16) * 0x9E3779B1u) | 1u; }

// A slot of the table: the facet's index in its low `fbits` bits (all ones are no facet's index), bits of its triple's hash above: facets
// whose bits differ have different triples, so that a search passes the slots of others without a look at their corners (a facet and three
// gathers, one after the other, for every fourth facet), and among equal triples the smaller word is the smaller index.
__host__ __device__ __forceinline__ int facet_index_bits(int F) {
    int bits = 1;
    while (bits < 31 && (1ll << bits) - 1 < (long long)F) ++bits;
    return bits;
}
constexpr u32 FACET_SLOT_FREE = ~0u;
__device__ __forceinline__ u32 facet_slot_word(u32 hx, int f, int fbits) { return (hx >> fbits << fbits) | (u32)f; }
__device__ __forceinline__ u32 facet_slot_index(u32 word, int fbits) { return word & ((1u << fbits) - 1u); }

// Re-indexes every facet through vmap (null: they are up to date) and enters the
// ones of contracted meshes that have not collapsed into an open-
// addressing table keyed by the unordered vertex triple.  A slot stores a
// facet index; the slot's identity is that facet's triple, and among equal
// triples the slot converges to the smallest facet index (atomicMin), so the
// survivor does not depend on the order in which lanes arrive.  The table has been cleared to -1.  Once per call: what of
// equal facets remains is the first of them, in whichever round they became equal.
// The output vertices' positions and the final labels go out on the way.
//
// Bound by the table: 27 lines of 64 bytes per nanosecond for its atomics, and the trips of a search, one after the other.  20 M facets
// (6.7 M left of them): 287 us, 390 without the bits of the hash in the slots, with a branch around the gathers of vmap and an entry
// written per facet; 2.4 M: 43 -> 37; 226 k: 13.6 -> 10.2.  Several facets, or a facet and a vertex, per lane and turn take longer
// (445-500 us): the parts' lines push each other out of the L2.
//
// The facets that may remain are listed: a wave takes segments of 64 * SEG facets and leaves what it enters of each, in order, at
// the segment's start (FacetList), so that the two kernels behind this one read those alone, densely.  (With an entry per facet, dead
// or not, those two took 209 us of 20 M facets and 29 of 2.4 M, now 96 and 21.)  Longer segments are denser but make fewer waves:
// 2.4 M facets took 64, 59 and 59 us in all three kernels with segments of 64, 128 and 256 facets; of 20 M, 256 leave 4 for each wave.
// Tiles of 256 facets up to 2^19 of them, 1,024 beyond: a tile adds up the sums of all in front of it (1.9 M facets in 7,365 tiles: 23 us
// for the last kernel, 10 in 1,842).
constexpr int FSLOT_KEEP = -1;  // no slot decides about the facet: it stays
constexpr int facet_segment(int chunks) { return chunks == 1 ? 1 : chunks == 4 ? 2 : 4; }
inline int facet_chunks_for(int F) { return F <= 1 << 19 ? 1 : std::max(4, prim::compact_chunks_for(F)); }
struct FacetList {
    int* corners;          // the facet's corners,
    int* slot;             // the table slot that decides about it (it survives iff the slot ends up holding it) or FSLOT_KEEP,
    int* facet;            // the facet,
    unsigned char* keep;   // whether it survives;
    int* n;                // per segment: its entries
    int* wave_n;           // per wave of the two kernels' tiles: its survivors
};

template <int SEG>
__global__ __launch_bounds__(BLOCK) void final_facets_kernel(const int* __restrict__ fcur, int F, const int* __restrict__ fcount,
                                                             int tile_shift, FacetList L, int* __restrict__ mslots,
                                                             const int* __restrict__ before, const int* __restrict__ vmap, const State* st, int cur,
                                                             u32* __restrict__ htab, u32 hmask, int fbits, int B,
                                                             const int* __restrict__ voff, const int* __restrict__ done,
                                                             const int* cid_in, int* cid_out,
                                                             int n_orig, const VRec* __restrict__ vrec,
                                                             float* __restrict__ verts_out /* or null */) {
    const int stride = gridDim.x * BLOCK;
    const int g = blockIdx.x * BLOCK + threadIdx.x, lane = prim::lane_id();
    const int nv = st->nv[cur];
    const float slots_per_vertex = ((float)hmask + 1.0f) / (float)(nv > 0 ? nv : 1);
    auto renumbered = [&](Corners q) -> Corners {  // (a collapsed facet's corners are -1)
        if (before) q = Corners{before[q.a], before[q.b], before[q.c]};
        if (!vmap) return q;
        const Corners m{vmap[max(q.a, 0)], vmap[max(q.b, 0)], vmap[max(q.c, 0)]};
        return q.a >= 0 ? m : q;
    };
    auto enter = [&](int f, Corners q, int& slot) -> bool {
        if (q.a < 0) return false;
        slot = FSLOT_KEEP;
        if (!done[mesh_of(voff, B, q.a)]) return true;  // the mesh contracted in no round: facets kept as they are
        if (q.a == q.b || q.b == q.c || q.a == q.c) return false;
        sort3(q.a, q.b, q.c);
        const u32 hx = hash3(q.a, q.b, q.c), mine = facet_slot_word(hx, f, fbits);
        u32 h = facet_home(q.a, hx, slots_per_vertex) & hmask, step = 0;
        for (int probe = 1;; ++probe) {
            const u32 old = atomicCAS(&htab[h], FACET_SLOT_FREE, mine);
            if (old == FACET_SLOT_FREE) break;
            if ((old ^ mine) >> fbits == 0) {
                Corners o = renumbered(load_corners(fcur, facet_slot_index(old, fbits)));
                sort3(o.a, o.b, o.c);
                if (o.a == q.a && o.b == q.b && o.c == q.c) {
                    atomicMin(&htab[h], mine);
                    break;
                }
            }
            // a few steps along the line, then (a crowded stretch) all over the table
            if (probe < FACET_HOME_PROBES) {
                h = (h + 1u) & hmask;
            } else {
                h = (probe == FACET_HOME_PROBES ? hx : h + step) & hmask;
                step += facet_stride(hx);
            }
        }
        slot = (int)h;
        return true;
    };
    if (B > 1)
        for (int i = g; i < B * MATCH_SLOTS; i += stride) mslots[(size_t)i * MATCH_PAD] = 0;
    const int wave = __builtin_amdgcn_readfirstlane(g >> 6);
    for (long long s0 = (long long)wave * (64 * SEG); s0 < F; s0 += (long long)stride * SEG) {
        int n = 0;
        const long long tile = s0 >> tile_shift;  // (facets stand at the front of their tiles, see facet_costs_kernel)
        const long long end = fcount ? min((tile << tile_shift) + fcount[tile], (long long)F) : (long long)F;
        for (int c = 0; c < SEG && s0 + c * 64 < end; ++c) {
            const long long f = s0 + c * 64 + lane;
            Corners q{-1, -1, -1};
            if (f < end) q = renumbered(load_corners(fcur, (size_t)f));
            int slot = 0;
            const bool in = enter((int)f, q, slot);
            const u64 all = prim::ballot(in);
            if (in) {
                const size_t p = (size_t)s0 + n + prim::mask_below(all);
                L.corners[3 * p] = q.a;
                L.corners[3 * p + 1] = q.b;
                L.corners[3 * p + 2] = q.c;
                L.slot[p] = slot;
                L.facet[p] = (int)f;
            }
            n += (int)__popcll(all);
        }
        if (lane == 0) L.n[s0 / (64 * SEG)] = n;
    }
    if (cid_out)
        for (int o = g; o < n_orig; o += stride) {
            const int c = cid_in ? cid_in[o] : o;
            cid_out[o] = vmap ? vmap[c] : c;
        }
    if (verts_out)
        for (int w = g; w < nv; w += stride) {
            const float4 p = *reinterpret_cast<const float4*>(&vrec[w]);
            verts_out[3 * (size_t)w] = p.x;
            verts_out[3 * (size_t)w + 1] = p.y;
            verts_out[3 * (size_t)w + 2] = p.z;
        }
}

// The final labels by themselves, in front of that kernel, where there are so many facets that it is better for them to go by these than by both maps, one after the other.
constexpr int LABELS_APART_MIN = 1 << 20;  // vertices of the input
constexpr int LABELS_ITEMS = 4;
__global__ __launch_bounds__(BLOCK) void final_labels_kernel(const int* __restrict__ cid_in, const int* __restrict__ vmap, int* __restrict__ cid_out, int n) {
    const long long o0 = (long long)blockIdx.x * (BLOCK * LABELS_ITEMS) + threadIdx.x;
    int c[LABELS_ITEMS];
#pragma unroll
    for (int j = 0; j < LABELS_ITEMS; ++j) c[j] = o0 + j * BLOCK < n ? cid_in[o0 + j * BLOCK] : 0;
#pragma unroll
    for (int j = 0; j < LABELS_ITEMS; ++j) c[j] = vmap[c[j]];
#pragma unroll
    for (int j = 0; j < LABELS_ITEMS; ++j)
        if (o0 + j * BLOCK < n) cid_out[o0 + j * BLOCK] = c[j];
}

// The survivors among the listed facets, counted per mesh (in its slots; the next kernel adds them up), per tile of BLOCK * CHUNKS facets (as a compaction's count pass does) and wave of it:
// a facet survives if it is the first of its triple, the one that its slot holds.
template <int CHUNKS>
__global__ __launch_bounds__(BLOCK) void count_facets_kernel(FacetList L, int F, const u32* __restrict__ htab, int fbits,
                                                             int* __restrict__ tilesum, int B, const int* __restrict__ voff,
                                                             int* __restrict__ mslots) {
    constexpr int SEG = facet_segment(CHUNKS), SEGS = CHUNKS / SEG, SPAN = 64 * SEG;
    __shared__ u32 smem[prim::WAVES];
    const int w = prim::wave_id(), lane = prim::lane_id();
    const long long at = (long long)blockIdx.x * (BLOCK * CHUNKS) + (long long)w * (64 * CHUNKS);
    int n[SEGS];
#pragma unroll
    for (int j = 0; j < SEGS; ++j) n[j] = at + j * SPAN < F ? L.n[at / SPAN + j] : 0;
    u32 kept = 0;
    int mesh = -1, of_mesh = 0;  // of the wave's survivors, how many are of the mesh it is at
    auto add_to_mesh = [&] {
        if (of_mesh && lane == 0) atomicAdd(&mslots[((size_t)mesh * MATCH_SLOTS + (blockIdx.x & (MATCH_SLOTS - 1))) * MATCH_PAD], of_mesh);
    };
#pragma unroll
    for (int j = 0; j < SEGS; ++j)
        for (int i0 = 0; i0 < SPAN && (i0 == 0 || i0 < n[j]); i0 += 64) {  // (the first entries are asked for together with their number)
            const long long p = min(at + j * SPAN + i0 + lane, (long long)F - 1);
            const int h = L.slot[p], f = L.facet[p];
            bool k = false;
            if (i0 + lane < n[j]) {
                k = h == FSLOT_KEEP || facet_slot_index(htab[max(h, 0)], fbits) == (u32)f;
                L.keep[p] = k ? 1 : 0;
            }
            u64 all = prim::ballot(k);
            kept += (u32)__popcll(all);
            if (B > 1) {
                const int m = k ? mesh_of(voff, B, L.corners[3 * p]) : -1;
                while (all) {  // a mesh after the other
                    const int first = __shfl(m, __ffsll((long long)all) - 1, 64);
                    const u64 same = prim::ballot(m == first);
                    if (first != mesh) {
                        add_to_mesh();
                        mesh = first;
                        of_mesh = 0;
                    }
                    of_mesh += (int)__popcll(same);
                    all &= ~same;
                }
            }
        }
    if (B > 1) add_to_mesh();
    if (lane == 0) {
        smem[w] = kept;
        L.wave_n[blockIdx.x * prim::WAVES + w] = (int)kept;
    }
    __syncthreads();
    if (threadIdx.x == 0) tilesum[blockIdx.x] = (int)(smem[0] + smem[1] + smem[2] + smem[3]);
}

// ... and written out, in order.
template <int CHUNKS>
__global__ __launch_bounds__(BLOCK) void facets_out_kernel(FacetList L, int F, const int* __restrict__ tilesum, int prefixed,
                                                           int B, int* __restrict__ out, const int* __restrict__ mslots,
                                                           int* __restrict__ mesh_facets, int* __restrict__ nf_out) {
    constexpr int SEG = facet_segment(CHUNKS), SEGS = CHUNKS / SEG, SPAN = 64 * SEG;
    __shared__ u32 smem[prim::WAVES];
    const int t = threadIdx.x, w = prim::wave_id(), lane = prim::lane_id(), tile = blockIdx.x;
    const long long at = (long long)tile * (BLOCK * CHUNKS) + (long long)w * (64 * CHUNKS);
    int n[SEGS];
#pragma unroll
    for (int j = 0; j < SEGS; ++j) n[j] = at + j * SPAN < F ? L.n[at / SPAN + j] : 0;
    const int4 waves = reinterpret_cast<const int4*>(L.wave_n)[tile];
    u32 run;
    if (prefixed) {
        run = (u32)tilesum[tile];
    } else {
        u32 part = 0;
        for (int j = t; j < tile; j += BLOCK) part += (u32)tilesum[j];
        run = prim::block_sum(part, smem);
    }
    if (tile == (int)gridDim.x - 1 && t == 0) {
        const int all = (int)run + ((waves.x + waves.y) + (waves.z + waves.w));
        *nf_out = all;
        if (B == 1) mesh_facets[0] = all;
    }
    if (B > 1)
        for (int i = tile * BLOCK + t; i < B * MATCH_SLOTS; i += (int)gridDim.x * BLOCK) {  // (a mesh's slots in half a wave)
            int n_b = mslots[(size_t)i * MATCH_PAD];
#pragma unroll
            for (int d = MATCH_SLOTS / 2; d > 0; d >>= 1) n_b += __shfl_xor(n_b, d, 64);
            if ((i & (MATCH_SLOTS - 1)) == 0) mesh_facets[i / MATCH_SLOTS] = n_b;
        }
    run += (u32)((w > 0 ? waves.x : 0) + (w > 1 ? waves.y : 0) + (w > 2 ? waves.z : 0));
#pragma unroll
    for (int j = 0; j < SEGS; ++j) {
        const long long s0 = at + j * SPAN;
        if (s0 >= F) break;
        for (int i0 = 0; i0 < SPAN && (i0 == 0 || i0 < n[j]); i0 += 64) {
            const long long p = min(s0 + i0 + lane, (long long)F - 1);
            const unsigned char flag = L.keep[p];
            const Corners q = load_corners(L.corners, (size_t)p);
            const bool kept = i0 + lane < n[j] && flag != 0;
            const u64 all = prim::ballot(kept);
            if (kept) {
                const size_t o = 3 * ((size_t)run + prim::mask_below(all));
                out[o] = q.a;
                out[o + 1] = q.b;
                out[o + 2] = q.c;
            }
            run += (u32)__popcll(all);
        }
    }
}

// ---------------------------------------------------------------------------
// Results
// ---------------------------------------------------------------------------
// The call's last kernel, one workgroup: the header's first n ints ([State][matched][mesh_facets])
// copied to the host's read-back area, then the host is told.
// zero[i * zero_stride] and the word behind it, i < n_zero: words that their users find zero, cleared on the way.
__global__ __launch_bounds__(BLOCK) void publish_header_kernel(int* __restrict__ hdr, int n,
                                                               int* __restrict__ host_img, HostSignal done,
                                                               u32* __restrict__ zero, int n_zero, int zero_stride) {
    for (int i = threadIdx.x; i < n; i += BLOCK) host_img[i] = hdr[i];
    for (int i = threadIdx.x; i < n_zero; i += BLOCK) zero[(size_t)i * zero_stride] = zero[(size_t)i * zero_stride + 1] = 0;
    // (the error flags are zero between calls: a single mesh's next call does not upload a header)
    if (threadIdx.x == 0) hdr[offsetof(State, err) / sizeof(int)] = 0;
    signal_host(done, threadIdx.x, (int)threadIdx.x < n);
}

// Degenerated vertices (option): ref[v] = 1 for every vertex that a facet of the final mesh refers to
// (ref is cleared beforehand; all writers store the same value).
__global__ __launch_bounds__(BLOCK) void mark_referenced_kernel(const int* __restrict__ fcur, const State* st,
                                                                int* __restrict__ ref) {
    const long long n = 3ll * st->nf;
    for (long long i = (long long)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * BLOCK) ref[fcur[i]] = 1;
}

struct RefPred {
    const int* ref;
    __device__ bool operator()(int v) const { return ref[v] != 0; }
};

// newid[v] = number of referenced vertices in front of v, for EVERY vertex (so that the count in front
// of a mesh's first vertex can be read off as well)
struct RefOut {
    static constexpr bool WAVE_WIDE = true;
    int* newid;
    __device__ void wave(int v, bool in_range, bool flagged, int pos) const {
        (void)flagged;
        if (in_range) newid[v] = pos;
    }
};

// Only the vertices with ref[v] != 0 go out, at newid[v]; facets and cluster ids follow that
// numbering, cluster ids of dropped vertices become -1, and kept_per_mesh[b] receives mesh b's count.
__global__ __launch_bounds__(BLOCK) void drop_out_kernel(const VRec* __restrict__ vrec, const int* __restrict__ fcur,
                                                         const int* __restrict__ cid, const State* st, int cur,
                                                         int n_orig, float* __restrict__ verts_out,
                                                         int* __restrict__ facets_out, int* __restrict__ cid_out,
                                                         int B, const int* __restrict__ voff, const int* __restrict__ ref,
                                                         const int* __restrict__ newid,
                                                         int* __restrict__ kept_per_mesh) {
    const int nv = st->nv[cur], nf = st->nf;
    const int stride = gridDim.x * BLOCK;
    const int g = blockIdx.x * BLOCK + threadIdx.x;
    for (int w = g; w < nv; w += stride) {
        if (!ref[w]) continue;
        const int o = newid[w];
        const float4 p = *reinterpret_cast<const float4*>(&vrec[w]);
        verts_out[3 * (size_t)o] = p.x;
        verts_out[3 * (size_t)o + 1] = p.y;
        verts_out[3 * (size_t)o + 2] = p.z;
    }
    for (long long i = g; i < 3ll * nf; i += stride) facets_out[i] = newid[fcur[i]];
    for (int o = g; o < n_orig; o += stride) {
        const int c = cid[o];
        cid_out[o] = ref[c] ? newid[c] : -1;
    }
    for (int b = g; b < B; b += stride) {
        const int before = voff[b] < nv ? newid[voff[b]] : st->nv_kept;
        const int upto = voff[b + 1] < nv ? newid[voff[b + 1]] : st->nv_kept;
        kept_per_mesh[b] = upto - before;
    }
}

// Plain streaming copy, 16 bytes per lane per step: the yardstick for the
// achievable HBM rate and for calibrating the profiler's byte counters.
__global__ __launch_bounds__(BLOCK) void copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                     size_t n16) {
    const size_t stride = (size_t)gridDim.x * BLOCK;
    for (size_t i = (size_t)blockIdx.x * BLOCK + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(BLOCK) void export_quadrics_kernel(const VRec* __restrict__ vrec, int N,
                                                                float* __restrict__ out) {
    const int w = blockIdx.x * BLOCK + threadIdx.x;
    if (w >= N) return;
    const float4* r = reinterpret_cast<const float4*>(&vrec[w]);
    const float4 r1 = r[1], r2 = r[2], r3 = r[3];
    float* o = out + 10 * (size_t)w;
    o[0] = r1.x; o[1] = r1.y; o[2] = r1.z; o[3] = r1.w;
    o[4] = r2.x; o[5] = r2.y; o[6] = r2.z; o[7] = r2.w;
    o[8] = r3.x; o[9] = r3.y;
}

__global__ __launch_bounds__(BLOCK) void export_edges_kernel(const u64* __restrict__ ekey, const u32* __restrict__ ecost,
                                                             const State* st, int vbits, int* __restrict__ edges,
                                                             float* __restrict__ cost) {
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    if (e >= st->ne) return;
    const u64 k = ekey[e];
    edges[2 * (size_t)e] = (int)(k >> vbits);
    edges[2 * (size_t)e + 1] = (int)(k & ((1ull << vbits) - 1ull));
    const u32 ck = ecost[e];
    cost[e] = __uint_as_float((ck & 0x80000000u) ? (ck & 0x7FFFFFFFu) : ~ck);
}

inline int ceil_log2(long long n) {
    int b = 0;
    while ((1ll << b) < n) ++b;
    return b < 1 ? 1 : b;
}

}  // namespace
