// picasso.hip -- host side of the library behind the C-ABI of include/picasso.h:
// the context and its workspace, the round loop of the decimation (Algorithm 2
// of the Picasso paper, Sec. 3; kernels in decimate_kernels.h), and the entry
// points, including those of pooling (pooling.h) and the mesh convolutions
// (conv.h).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <new>

#include "../../include/picasso.h"
#include "primitives.h"
#include "decimate_kernels.h"
#include "pooling.h"
#include "conv.h"

#pragma clang fp contract(off)

namespace {

inline int grid_for(long long n, int cap = 0x7FFFFFFF) {
    long long g = (n + BLOCK - 1) / BLOCK;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

}  // namespace

// ---------------------------------------------------------------------------
// Context
// ---------------------------------------------------------------------------
constexpr int NF_ROUND_CAP = 64;  // rounds whose facet counts a call notes for the kernel-timing totals
struct StageRec { int round, stage, e0, e1; };

// How a round went: by sorted edges, by rings, by facets, by the call's facets behind rounds by rings.
enum RoundWay : unsigned char { WAY_SORTED, WAY_RINGS, WAY_FACETS, WAY_FACETS_AGAIN };

struct picasso_ctx {
    int device = 0;
    int64_t max_verts = 0, max_facets = 0;
    int32_t max_meshes = 0;
    int64_t opt_max_rounds = -1;
    int64_t opt_stage_timing = 0;
    int64_t opt_subround_batch = 16;
    char hip_err[256] = {0};

    char* ws = nullptr;  // one device allocation, carved below
    size_t ws_bytes = 0;
    int* hdr = nullptr;  // State followed by the per-mesh tables (see carve)
    int cap_b = 1;       // per-mesh capacity the header was laid out for
    State* st = nullptr;
    VRec* vrec[2] = {nullptr, nullptr};
    int* fcur = nullptr;                // the facets, re-indexed in place round by round
    int* fmap = nullptr;                // ... after the last round, before compaction
    int* cid = nullptr;
    char* sort_buf = nullptr;            // the five arrays below in one piece, all of which the filter gradients' partial sums may take
    size_t sort_bytes = 0;
    u64* key64[2] = {nullptr, nullptr};  // sort buffers (3F keys)
    u32* val32 = nullptr;                // ... for the values of the exported sorts
    u64* ekey = nullptr;
    u32* ecost = nullptr;
    u64* vmin[3] = {nullptr, nullptr, nullptr};
    int* mate = nullptr;
    int* newid = nullptr;                               // (free during the rounds: the pairs' cost keys)
    u32* pcost() const { return reinterpret_cast<u32*>(newid); }
    u32* ptie() const { return reinterpret_cast<u32*>(vmap); }  // (vmap is free between a round's first kernel and its contraction)
    int* vmap = nullptr;
    int* list = nullptr;
    int* fcount() const { return list; }  // per tile of facets, how many there are (rounds by facets, which list no edges there)
    unsigned char* estate = nullptr;
    int* htab = nullptr;
    unsigned char* keep = nullptr;
    int* fslot = nullptr;  // per facet: the hash-table slot that decides about it
    int* tilesum = nullptr;
    u32* distinct = nullptr;  // the edge sort's distinct keys per bucket, then per prim::UNIQUE_GROUP buckets
    size_t distinct_cap = 0;  // ... buckets
    prim::SortScratch sort_sc{};
    u32* hist12 = nullptr;  // the key sorts' arrays of a word per digit (prim::KeySort; prim::MSD_WORDS)
    // The vertex->facet sort has buffers and scratch of its own, so that in the first round it can
    // share its launches with the edge-key sort (neither depends on the other).
    u64* s0_key[2] = {nullptr, nullptr};  // incidence keys (vertex, facet) of S0 and their sort's second buffer
    u32* hist12_s0 = nullptr;
    prim::XlScratch xl{}, xl_s0{};  // the same for the sorts of very large inputs
    bool hist_dirty = true;  // hist12's counts may not be zero (the key sorts leave them so)
    int64_t opt_overlap = 1;
    int64_t opt_trunc_block_max = TRUNC_BLOCK_CAP;
    // per-mesh tables
    int* voff[2] = {nullptr, nullptr};
    int* foff = nullptr;
    int* mesh_facets = nullptr;
    int* target = nullptr;
    int* active[2] = {nullptr, nullptr};  // by the round's parity
    int* nf_slots[2] = {nullptr, nullptr};  // facets that have not collapsed, by the round's parity (see facet_costs_kernel)
    int* stuck = nullptr;
    int* done = nullptr;   // mesh has contracted pairs in some round
    int* nrem = nullptr;
    int* matched = nullptr;
    SelectSlot* select_slots = nullptr;  // the budget step's counts (long runs, see budget_step)
    KeyLimit* limits = nullptr;  // per mesh (see budget_step)
    int* mslots = nullptr;
    LiveEdge* live = nullptr;  // the selection tail's list (see SelArgs) and its segments' lengths
    int* live_n = nullptr;
    // pinned host staging
    // pinned host staging: read-back image of the header's front, then the upload image of the whole header
    int* h_pin = nullptr;
    int* h_pin_dev = nullptr;  // the same memory as the device addresses it
    size_t h_up_off = 0;
    size_t h_pin_ints = 0;
    size_t h_seq_off = 0;  // the word that kernels store a sequence number in for the host (a cache line of its own)
    int host_seq = 0;      // the last sequence number handed out
    int64_t opt_poll_us = 20000;  // for how long the host watches that word before it waits for the stream instead (0: not at all)
    int opt_ahead = 1;     // a round's contraction and facet kernels are queued before the host has looked
    int opt_trunc_width = 0;  // test hook: keys per lane that the per-mesh budget search takes (0: as the sizes need)
    int opt_drop_degenerated = 0;  // output vertices that no output facet refers to are dropped
    hipEvent_t ev[2 * PICASSO_STATS_ROUNDS * PICASSO_ST_COUNT + 4];
    int n_ev = 0;
    hipEvent_t ev_total[2];
    // hipEvent brackets around the edge-key sort's main kernel (benchmark roofline)
    int64_t opt_kernel_timing = 0;  // N > 0: events around the kernel in every N-th decimate call
    int opt_placement = PLACE_MEAN;
    float opt_rcond_min = 1e-3f;
    int opt_absorb = 0;
    uint64_t opt_shuffle_seed = 0;  // != 0: pairs of equal cost in the order of the seeded tie-break
    u64* abid = nullptr;   // per vertex: cheapest edge through which it could join a pair's cluster
    int* arep = nullptr;   // per vertex: representative of the cluster it joined, or -1
    int* aoff = nullptr;   // per vertex: the first of those that joined the cluster it represents, in joiners()
    BudgetList* budget_list() const { return reinterpret_cast<BudgetList*>(abid); }  // (of line 11, which rounds by rings do not have)
    int* joiners() const { return reinterpret_cast<int*>(val32); }  // (free between the edges' sort and the next round)
    int* acand = nullptr;  // per mesh: vertices that could join
    int* arem = nullptr;   // per mesh: budget left after the pairs
    RingRows ring[2], adj;  // rounds by rings: the rings, by the round's parity, and the neighbours with their costs (see ring_costs_kernel)
    int* rows_taken = nullptr;  // ... (see RINGS_TAKEN)
    int2* from = nullptr;   // ... per vertex: the two of the round before that it was made of, and their rings' info
    ulonglong2* from_info = nullptr;
    u32* area_ext = nullptr;  // per mesh: largest facet area and largest complement of one (conv::EXT_SLOTS; zero between calls)
    int64_t kt_calls = 0;           // decimate calls since the option was set
    bool kt_this_call = false;
    hipEvent_t kt_pool[512];
    prim::LaunchTimer::Rec kt_recs[256];
    prim::LaunchTimer kt;
    int64_t kt_launches[PICASSO_KERNEL_COUNT] = {0};
    double kt_ms[PICASSO_KERNEL_COUNT] = {0.0}, kt_bytes[PICASSO_KERNEL_COUNT] = {0.0};
    // host mirrors of the per-mesh state of a decimate call (6 x max_meshes ints, allocated with the
    // context: the calls themselves allocate nothing, on the host either)
    int* h_mesh = nullptr;
    int nf_round[NF_ROUND_CAP];  // facets, vertices, distinct edges of each round of the current call
    int nv_round[NF_ROUND_CAP];
    int ne_round[NF_ROUND_CAP];
    unsigned char way_round[NF_ROUND_CAP];  // (see RoundWay)
    int n_rounds_noted = 0;
    StageRec st_recs[PICASSO_STATS_ROUNDS * PICASSO_ST_COUNT + 2];
};

namespace {

constexpr int HDR_STATE_INTS = (int)(sizeof(State) / sizeof(int));
constexpr size_t hdr_ints(size_t b) { return HDR_STATE_INTS + 10 * b + 3; }  // for up to b meshes (see carve)
constexpr int SEQ_CHECK_WORD = 16;  // within the sequence word's 32-int area: the selection tail's copy of the number (a cache line further)

struct Carver {
    size_t off = 0;
    char* base = nullptr;
    template <typename T>
    T* take(size_t count) {
        size_t o = off;
        off = align_up(off + count * sizeof(T));
        return base ? reinterpret_cast<T*>(base + o) : nullptr;
    }
};

size_t next_pow2(size_t x) {
    size_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Slots of the hash set that up to f facets are entered into.
size_t facet_slots(size_t f) { return next_pow2(2 * std::max<size_t>(f, 1)); }

// Lays the workspace out; with base == nullptr only measures it.
size_t carve(picasso_ctx* c, char* base, int64_t N, int64_t F, int32_t B) {
    Carver cv;
    cv.base = base;
    const size_t n = (size_t)std::max<int64_t>(N, 1), f = (size_t)std::max<int64_t>(F, 1), h = 3 * f;
    const size_t b = (size_t)std::max<int32_t>(B, 1);
    picasso_ctx dummy;
    picasso_ctx* x = c ? c : &dummy;
    // header: everything the host uploads or reads back, contiguous so that one copy moves it.
    //   [State][matched B][mesh_facets B+1] | [voff0 B+1][foff B+1][target B][stuck B][active0 B][active1 B][done B]
    //   <-------- read back ----------->
    int* hdr = cv.take<int>(hdr_ints(b));
    x->hdr = hdr;
    x->st = reinterpret_cast<State*>(hdr);
    if (hdr) {
        int* q = hdr + HDR_STATE_INTS;
        x->matched = q; q += b;
        x->mesh_facets = q; q += b + 1;
        x->voff[0] = q; q += b + 1;
        x->foff = q; q += b + 1;
        x->target = q; q += b;
        x->stuck = q; q += b;
        x->active[0] = q; q += b;
        x->active[1] = q; q += b;
        x->done = q; q += b;
    }
    x->vrec[0] = cv.take<VRec>(n);
    x->vrec[1] = cv.take<VRec>(n);
    x->fcur = cv.take<int>(3 * f);
    x->fmap = cv.take<int>(3 * f);  // (right behind: the two are the rows of a set of rings, too)
    x->cid = cv.take<int>(n);
    auto sort_buffers = [&](char* at) {
        Carver in;
        in.base = at;
        x->key64[0] = in.take<u64>(h);
        x->key64[1] = in.take<u64>(h);
        x->val32 = in.take<u32>(h);
        x->ekey = in.take<u64>(h);
        x->ecost = in.take<u32>(h);
        return in.off;
    };
    x->sort_bytes = sort_buffers(nullptr);
    x->sort_buf = cv.take<char>(x->sort_bytes);
    sort_buffers(x->sort_buf);
    for (int i = 0; i < 3; ++i) x->vmin[i] = cv.take<u64>(n);
    x->mate = cv.take<int>(n);
    x->newid = cv.take<int>(n);
    x->vmap = cv.take<int>(n);
    x->list = cv.take<int>(h);
    x->estate = cv.take<unsigned char>(h);
    x->htab = cv.take<int>(facet_slots(f));
    x->keep = cv.take<unsigned char>(f);
    x->fslot = cv.take<int>(f);
    x->tilesum = cv.take<int>((size_t)prim::compact_tilesum_capacity((long long)std::max(h, n)));
    x->distinct_cap = prim::bucket_capacity((long long)h);
    x->distinct = cv.take<u32>(x->distinct_cap + x->distinct_cap / prim::UNIQUE_GROUP * prim::UNIQUE_PAD);
    x->sort_sc.T = prim::sort_table_stride((long long)h);
    x->sort_sc.table = cv.take<u32>((size_t)256 * x->sort_sc.T);
    x->sort_sc.totals = cv.take<u32>(256);
    x->hist12 = cv.take<u32>(prim::MSD_WORDS);
    for (int i = 0; i < 2; ++i) {
        x->s0_key[i] = cv.take<u64>(h);
    }
    x->hist12_s0 = cv.take<u32>(prim::MSD_WORDS);
    if ((long long)h > prim::BUCKET_SORT_LARGE_MAX_KEYS) {
        const size_t words = prim::xl_hist_words((long long)h);
        for (prim::XlScratch* q : {&x->xl, &x->xl_s0}) {
            q->hist = cv.take<u32>(words);
            q->starts = cv.take<u32>(words);
            q->cursor = cv.take<u32>(words);
        }
    }
    x->voff[1] = cv.take<int>(b + 1);
    x->nrem = cv.take<int>(b);
    x->select_slots = cv.take<SelectSlot>((size_t)std::max(std::min((int)b, SELECT_MESHES), select_slots_by_start((int)b, (long long)n)));
    x->limits = cv.take<KeyLimit>(b);
    x->mslots = cv.take<int>(b * MATCH_SLOTS * MATCH_PAD);
    x->live = cv.take<LiveEdge>((size_t)LIVE_SEGS * TAIL_MAX);
    x->live_n = cv.take<int>(LIVE_SEGS * MATCH_PAD);
    for (int i = 0; i < 2; ++i) x->nf_slots[i] = cv.take<int>(MATCH_SLOTS * MATCH_PAD);
    x->abid = cv.take<u64>(n);
    x->arep = cv.take<int>(n);
    x->aoff = cv.take<int>(n + 1);
    x->acand = cv.take<int>(b);
    x->arem = cv.take<int>(b);
    x->area_ext = cv.take<u32>(b * conv::EXT_SLOTS * conv::EXT_PAD);
    // The rings lie in the sorts' buffers, which rounds by rings do not use (the neighbours' where the facets' planes have been), if these are large enough, as they are where
    // vertices have five and a half facets or more.  Rows lie where rounds by facets have the facets and where the incidence keys have been, with a word for every corner of
    // the input: the input's own in the order of the incidences, later ones as RingRows hands places out.
    const size_t ring_bytes = n * (sizeof(u32) * RING_ROW + sizeof(u64)), region = align_up(h * sizeof(u64)), wanted = ring_bytes + 512;
    const bool fits = region >= wanted;
    x->rows_taken = cv.take<int>(RINGS_TAKEN);
    u64* const rows[3] = {reinterpret_cast<u64*>(x->fcur), x->s0_key[0], x->s0_key[1]};
    for (int i = 0; i < 3; ++i) {
        RingRows& r = i < 2 ? x->ring[i] : x->adj;
        char* const own = fits ? nullptr : cv.take<char>(align_up(wanted));
        Carver in;
        in.base = fits ? reinterpret_cast<char*>(i == 0 ? x->key64[0] : i == 1 ? x->key64[1] : x->ekey) : own;
        r.ids = in.take<u32>(n * RING_ROW);
        r.info = in.take<u64>(n);
        r.more = !fits ? cv.take<u32>(n * RING_MORE) : nullptr;
        r.rows = rows[i];
        // (a ring of all facets fits the rest; where there are few words all are the rest, whose one counter is enough then)
        r.arena_words = (u32)(h / 8 * 5 / ROW_ARENAS);
        if (r.arena_words < 512) r.arena_words = 0;
        r.rest_words = (u32)h - ROW_ARENAS * r.arena_words;
        r.taken = x->rows_taken && i < 2 ? x->rows_taken + i * (ROW_ARENAS + 1) * MATCH_PAD : nullptr;
        r.wide = x->st ? &x->st->wide : nullptr;
    }
    if (fits) {
        Carver costs, values;
        values.base = reinterpret_cast<char*>(x->val32);
        x->from = values.take<int2>(n);
        x->ring[0].more = values.take<u32>(n * RING_MORE);
        x->ring[1].more = reinterpret_cast<u32*>(x->vmin[2]);  // (of the selection by sub-rounds, as is the list of its edges)
        x->adj.more = reinterpret_cast<u32*>(x->list);
        costs.base = reinterpret_cast<char*>(x->ecost);
        x->from_info = costs.take<ulonglong2>(n);
    } else {
        x->from = cv.take<int2>(n);
        x->from_info = cv.take<ulonglong2>(n);
    }
    return cv.off;
}

#define HIP_TRY(ctx, expr)                                                                          \
    do {                                                                                            \
        hipError_t e__ = (expr);                                                                    \
        if (e__ != hipSuccess) {                                                                    \
            snprintf((ctx)->hip_err, sizeof((ctx)->hip_err), "%s at %s:%d: %s", #expr, __FILE__, __LINE__, \
                     hipGetErrorString(e__));                                                       \
            return PICASSO_ERR_HIP;                                                                 \
        }                                                                                           \
    } while (0)

struct StageTimer {
    picasso_ctx* c;
    hipStream_t s;
    bool on;
    int n_recs = 0;  // records in c->st_recs
    int open = -1;
    // (stage PICASSO_ST_COUNT: work for the statistics alone, which is no part of the call's time)
    void begin(int round, int stage) {
        constexpr int cap = (int)(sizeof(c->st_recs) / sizeof(c->st_recs[0]));
        if ((!on && stage != PICASSO_ST_COUNT) || n_recs >= cap || c->n_ev + 2 > (int)(sizeof(c->ev) / sizeof(c->ev[0]))) return;
        const StageRec r{round, stage, c->n_ev, c->n_ev + 1};
        c->n_ev += 2;
        (void)hipEventRecord(c->ev[r.e0], s);
        c->st_recs[n_recs] = r;
        open = n_recs++;
    }
    void end() {
        if (open < 0) return;
        (void)hipEventRecord(c->ev[c->st_recs[open].e1], s);
        open = -1;
    }
    void collect(picasso_stats* stats) {
        if (!stats) return;
        for (int i = 0; i < n_recs; ++i) {
            const StageRec& r = c->st_recs[i];
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, c->ev[r.e0], c->ev[r.e1]) != hipSuccess || r.round >= PICASSO_STATS_ROUNDS) continue;
            if (r.stage == PICASSO_ST_COUNT) stats->ms_total -= ms;
            else stats->ms_stage[r.round][r.stage] += ms;
        }
    }
};

// hipEvents around the launches made while this object lives, credited to `kernel` in round `round`
// (only in the calls that PICASSO_OPT_KERNEL_TIMING picks).
struct KernelBracket {
    picasso_ctx* c;
    hipStream_t s;
    bool on;
    KernelBracket(picasso_ctx* c_, hipStream_t s_, int kernel, int round, bool wanted = true) : c(c_), s(s_) {
        on = wanted && c->kt_this_call && round < 0xFF && c->kt.begin(s, (kernel << 8) | round);
    }
    ~KernelBracket() {
        if (on) c->kt.end(s);
    }
    KernelBracket(const KernelBracket&) = delete;
    KernelBracket& operator=(const KernelBracket&) = delete;
};

// Bits of a vertex in the edge keys, of an item in the keys of row lists: what the largest number needs, but enough for as many
// keys to have the top digit that prim::key_sort partitions them on.  Of a vertex in the incidence keys: the digit lies
// within them, so that a bucket holds whole vertices.
inline int edge_vertex_bits(int nv, long long n_keys) { return std::max(ceil_log2(nv), prim::key_bits_wanted(n_keys) / 2); }
inline int item_bits(int n_rows, int n_items, long long n_keys) {
    return std::max(ceil_log2(std::max(n_items, 1)), prim::key_bits_wanted(n_keys) - ceil_log2(n_rows));
}
inline int incidence_fbits(int F) { return ceil_log2(std::max(F, 1)); }
inline int incidence_key_bits(int N, int F) {
    const int vbits = ceil_log2(N), fbits = incidence_fbits(F);
    return std::max(vbits, prim::key_digit_bits(3ll * F, vbits + fbits)) + fbits;
}

// A sort of up to n keys made from `items` items (KeySort), with the context's first or second set of arrays.
// Keys (row << item_bits) | item of n_rows rows: only so many digits occur, and, where rows are short, the bits of the row below
// the digit make the groups that the per-bucket kernel sorts in registers.  (Nine bits always: every other group of a lattice of 10 M
// vertices empty.)
void rows_of(prim::KeySort<u64>& S, int n_rows, int item_bits, long long n) {
    const int within = S.low_bits() - item_bits;  // bits of the row below the digit
    if (within < 0) return;
    S.buckets = (int)(((long long)n_rows + (1ll << within) - 1) >> within);
    if (within >= 1 && within < S.group_bits && n <= 8ll * n_rows) S.group_bits = within;
    S.crowded = n < n_rows;
}

// Kernels that count the keys' digits for it go by COUNT_ (see init_kernel) and its DigitCount.
prim::KeySort<u64> key_sort_for(picasso_ctx* c, bool second_set, long long n, int items, int key_bits) {
    prim::KeySort<u64> S;
    S.k0 = second_set ? c->s0_key[0] : c->key64[0];
    S.k1 = second_set ? c->s0_key[1] : c->key64[1];
    S.n = items;
    S.key_bits = key_bits;
    S.digit_bits = prim::key_digit_bits(n, key_bits);
    S.half = S.fits_half();
    S.buckets = 1 << S.digit_bits;
    if (S.digit_bits > prim::BUCKET_LARGE_MSD_BITS) {
        const prim::XlScratch& x = second_set ? c->xl_s0 : c->xl;
        S.hist = x.hist;
        S.cursor = x.cursor;
        S.starts = x.starts;
    } else {
        prim::use_arrays(S, second_set ? c->hist12_s0 : c->hist12);
    }
    return S;
}
inline int count_kind(const prim::KeySort<u64>& S) {
    return S.digit_bits <= prim::NARROW_BITS_MAX ? COUNT_SMALL : (S.digit_bits <= prim::BUCKET_LARGE_MSD_BITS ? COUNT_LARGE : COUNT_XL);
}
inline DigitCount digit_count(const prim::KeySort<u64>& S) {
    return DigitCount{S.hist, S.key_bits - S.digit_bits, (1u << S.digit_bits) - 1u};
}
// The counts of digits of up to 12 bits are zero between sorts (KeySort); wider ones are cleared by this before their keys are counted.
void clear_wide_counts(hipStream_t s, const prim::KeySort<u64>& S) {
    if (count_kind(S) == COUNT_XL) prim::fill_u32_kernel<<<grid_for(1 << S.digit_bits), BLOCK, 0, s>>>(S.hist, 1 << S.digit_bits, 0u);
}

// Half-edges to expect of a round whose facets have not been counted yet, from the round before: its half-edges and distinct edges,
// and the vertices it has removed.  A removed vertex takes along the facets at its edge, of which there are half_edges / edges,
// three half-edges each; a sixth more, for pairs on open edges.  Ordinary surfaces: 54 to 55 % are left, the figure is 10 to 18 % above what comes.
// (Seven per vertex are the same there, but half of what two-sided surfaces have, and less with more facets to a vertex, whose buckets then do
// not fit LDS.  To a quarter of the vertices: two-sided surfaces of 593 k 894 -> 722 us, 1.12 M 1426 -> 1101; 25 facets to a vertex, any three
// vertices: 20 k 2339 -> 1697, 100 k 5700 -> 3796.)
long long expected_half_edges(long long half_edges, long long edges, long long removed) {
    if (edges <= 0) return half_edges;
    const long long left = std::max(edges - 3 * removed, 0ll);
    return std::min(half_edges, std::max(half_edges / 4, half_edges * left / edges * 7 / 6));
}

// The sort of the edge keys of a round with nvt vertices and at most nfb facets that have not collapsed, of F; about n_keys keys (all
// of the first round's are known).
prim::KeySort<u64> edge_sort(picasso_ctx* c, int nvt, int nfb, int F, long long n_keys) {
    const int H = 3 * nfb, vbits = edge_vertex_bits(nvt, H);
    prim::KeySort<u64> S = key_sort_for(c, false, n_keys, F, 2 * vbits);
    rows_of(S, nvt, vbits, H);
    S.zero = c->distinct + c->distinct_cap;  // (the counts per group of buckets)
    S.n_zero = (1 << S.digit_bits) / prim::UNIQUE_GROUP * prim::UNIQUE_PAD;
    S.total = &c->st->nh;
    return S;
}
prim::DistinctKeys distinct_keys(picasso_ctx* c) { return prim::DistinctKeys{c->distinct, c->distinct + c->distinct_cap}; }
// ... and of the incidence keys.
prim::KeySort<u64> incidence_sort(picasso_ctx* c, int N, int F) {
    prim::KeySort<u64> S = key_sort_for(c, true, 3ll * F, F, incidence_key_bits(N, F));
    rows_of(S, N, incidence_fbits(F), 3ll * F);
    return S;
}

// Where init_kernel leaves the facets' planes for S0: the edge-key array, which nothing else uses
// before the first round's costs are computed (24 bytes per facet there, 16 needed).
inline float4* facet_planes(picasso_ctx* c) { return reinterpret_cast<float4*>(c->ekey); }
// A vertex of the input with more facets than this, and one for so many vertices, is evaluated by one wave for longer than rounds by facets take: cones of 1,000 facets by rings | by facets
// when their quadrics have shown it, us to 70 %, 318 | 318, of 4,000 1,654 | 1,592, of 20,000 8,205 | 7,862.
constexpr int RINGS_MOST = 1024, RINGS_MOST_EACH = 64;
template <bool RINGS>
QuadricRows<RINGS> quadric_rows(picasso_ctx* c, const float* d_verts, const int* facets, int N, int F) {
    return QuadricRows<RINGS>{c->vrec[0], d_verts, facet_planes(c), N, incidence_fbits(F), facets, c->ring[0],
                              c->ring[1].taken, N / (4 * ROW_ARENAS), RINGS_MOST + N / RINGS_MOST_EACH};
}

RoundTab round_tab(picasso_ctx* c, int B, int round_, int cur_) {
    return RoundTab{B, c->voff[cur_], c->target, c->active[round_ & 1], c->active[(round_ & 1) ^ 1], c->stuck, c->nrem, c->matched, c->mslots,
                    c->live_n, round_ == 0};
}

// First kernel of a round after the first: facets and labels follow the last contraction, the edges' digits are counted.
void launch_edge_keys(picasso_ctx* c, hipStream_t s, int B, int round_, int cur_, const prim::KeySort<u64>& S, int N, int F) {
    clear_wide_counts(s, S);
    c->hist_dirty = true;
    const KernelBracket timed(c, s, PICASSO_KERNEL_FACET_INSERT, round_ - 1);
#define PICASSO_EDGE_KEYS(COUNT, GRID)                                                                                        \
    edge_keys_kernel<COUNT><<<GRID, BLOCK, 0, s>>>(c->fcur, F, c->st, cur_, S.key_bits / 2, c->vmin[0], c->vmin[1], c->mate, \
                                                   c->pcost(), round_tab(c, B, round_, cur_), digit_count(S), c->vmap, c->done, c->cid, N)
    // (a workgroup adds its whole histogram to the other's in the end: with 4096 digits it takes several turns)
    switch (count_kind(S)) {
        case COUNT_SMALL: PICASSO_EDGE_KEYS(COUNT_SMALL, grid_for(std::max(F, 1))); break;
        case COUNT_LARGE: PICASSO_EDGE_KEYS(COUNT_LARGE, grid_for((F + 3) / 4, 2048)); break;
        default: PICASSO_EDGE_KEYS(COUNT_XL, grid_for((F + 3) / 4, 8192));
    }
#undef PICASSO_EDGE_KEYS
}

// Sorts the edge keys (whose digits have been counted) and lists the distinct ones (edge_list).
bool sort_edges(picasso_ctx* c, hipStream_t s, const prim::KeySort<u64>& S, int round_) {
    c->hist_dirty = false;
    return prim::key_sort(s, S, (const prim::KeySort<u64>*)nullptr, prim::OneSource<EdgeKeys>{{c->fcur, S.key_bits / 2}}, distinct_keys(c),
                          c->kt_this_call ? &c->kt : nullptr, round_);
}
// Sorts the incidence keys of these facets and sums the vertices' quadrics (RINGS: leaves their rings, too).
template <bool RINGS>
bool sort_incidences(picasso_ctx* c, hipStream_t s, const prim::KeySort<u64>& S, const float* d_verts, const int* facets, int N, int F) {
    return prim::key_sort(s, S, (const prim::KeySort<u64>*)nullptr, prim::OneSource<IncidenceKeys>{{facets, incidence_fbits(F), N}},
                          quadric_rows<RINGS>(c, d_verts, facets, N, F), c->kt_this_call ? &c->kt : nullptr, PICASSO_KERNEL_QUADRIC_ROWS << 8,
                          PICASSO_KERNEL_SORT_INCIDENCE << 8);
}
// Both in the same launches.
bool sort_edges_and_incidences(picasso_ctx* c, hipStream_t s, const prim::KeySort<u64>& E, const prim::KeySort<u64>& I,
                               const float* d_verts, int N, int F) {
    c->hist_dirty = false;
    return prim::key_sort(s, I, &E, prim::TwoSources<IncidenceKeys, EdgeKeys>{{c->fcur, incidence_fbits(F), N}, {c->fcur, E.key_bits / 2}},
                          prim::TwoOuts<QuadricRows<false>, prim::DistinctKeys>{quadric_rows<false>(c, d_verts, c->fcur, N, F), distinct_keys(c)});
}

// Whether a round of one or several meshes, of at most `edges` edges, keeps a state for each.
bool has_edge_states(int B, int edges) { return B > 1 || edges < LISTED_MIN_EDGES; }

// Costs and first bids of the distinct edges that sort E of at most H keys has left.
void launch_unique_cost(picasso_ctx* c, hipStream_t s, const prim::KeySort<u64>& E, int H, const MeshTab& mt, const TieBreak& tb,
                        const VRec* vrec) {
    EdgeList L{E.k1, E.starts, c->distinct, c->distinct + c->distinct_cap, H > 0 ? E.buckets : 0, E.low_bits(), 0, 0};
    // workgroups (edges are about half the keys): few edges each while there are few, for the chip's sake, then as many as their bids' table takes
    const long long wanted = std::max<long long>((long long)H / 2 / UNIQUE_EDGES_MAX, std::min<long long>((long long)H / 2 / UNIQUE_EDGES_MIN, UNIQUE_GROUPS_MIN));
    while (L.split_shift < 6 && (long long)L.buckets << L.split_shift < wanted) ++L.split_shift;
    while (L.split_shift == 0 && L.join_shift < UNIQUE_JOIN_MAX && L.buckets >> (L.join_shift + 1) >= wanted) ++L.join_shift;
    const int grid = L.buckets > 0 ? prim::xcd_grid((((L.buckets - 1) >> L.join_shift) + 1) << L.split_shift) : 1;
    unsigned char* const estate = has_edge_states(mt.B, H) ? c->estate : nullptr;
    const bool wide = (long long)H / 2 > (long long)grid * UNIQUE_EDGES_NARROW;
#define PICASSO_UNIQUE_LINES(PLACE, SHUFFLE, LK, LINES)                                                                       \
    unique_cost_kernel<PLACE, SHUFFLE, LK, LINES><<<grid, BLOCK, 0, s>>>(L, c->ekey, c->ecost, estate, vrec, c->vmin[0],          \
                                                                  E.key_bits / 2, mt, c->opt_rcond_min, tb, &c->st->ne)
#define PICASSO_UNIQUE_LK(PLACE, SHUFFLE, LK)                      \
    do {                                                           \
        if (wide) PICASSO_UNIQUE_LINES(PLACE, SHUFFLE, LK, 256);   \
        else PICASSO_UNIQUE_LINES(PLACE, SHUFFLE, LK, 128);        \
    } while (0)
#define PICASSO_UNIQUE(PLACE, SHUFFLE)                             \
    do {                                                           \
        if (E.half) PICASSO_UNIQUE_LK(PLACE, SHUFFLE, u32);        \
        else PICASSO_UNIQUE_LK(PLACE, SHUFFLE, u64);               \
    } while (0)
    if (c->opt_placement == PLACE_INVERSE) {
        if (tb.on) PICASSO_UNIQUE(PLACE_INVERSE, true);
        else PICASSO_UNIQUE(PLACE_INVERSE, false);
    } else {
        if (tb.on) PICASSO_UNIQUE(PLACE_MEAN, true);
        else PICASSO_UNIQUE(PLACE_MEAN, false);
    }
#undef PICASSO_UNIQUE
#undef PICASSO_UNIQUE_LK
#undef PICASSO_UNIQUE_LINES
}

// Facets to a tile in the rounds by facets: small ones while the workgroups are to fill the chip, large ones (fewer copies of an edge, lists and
// tables per workgroup that serve more) beyond 2^20 facets.  Whole calls with tiles of 256 | 1,024, us: one mesh of 227 k facets 190 | 222, 800 k
// 391 | 408, 1.4 M 503 | 502, 2.4 M 721 | 702, 20 M 5173 | 4720; 16 meshes of 750 k together 315 | 313, 1.13 M 408 | 394, 1.9 M 629 | 567.  Large
// ones of 512 against 1,024 (more and smaller workgroups, whose barriers hold up fewer waves): 2.4 M 698 -> 690, 20 M 4724 -> 4676, a ladder of four
// levels from 1.9 M 1169 -> 1155; joining two such tiles from the third round on, when half of their places are empty, took longer (703 -> 737, 4742 -> 5077).
constexpr int FACET_TILE_SMALL = 256, FACET_TILE_LARGE = 512;
constexpr int FACET_TILE_SMALL_MAX = 1 << 20;
// Lanes of their workgroups: of the rounds' first kernel behind the first round, where tiles are large, half as many.
constexpr int FACET_LANES = 256, FACET_LANES_LARGE = 128;
static_assert((FACET_TILE_SMALL & (FACET_TILE_SMALL - 1)) == 0 && (FACET_TILE_LARGE & (FACET_TILE_LARGE - 1)) == 0, "a facet's tile is found by a shift");
inline int facet_tile(int F) { return F <= FACET_TILE_SMALL_MAX ? FACET_TILE_SMALL : FACET_TILE_LARGE; }
inline int facet_tiles(int F) { return std::max((F + facet_tile(F) - 1) / facet_tile(F), 1); }
// Workgroups of facets and vertices that a round of at most nv vertices has.
inline int facet_parts(int F, int nv) { return std::max(facet_tiles(F), (nv + 1023) / 1024); }
// Where a round's contraction leaves its map of the vertices.  The first round's is the labels of the input vertices at the same time; rounds by
// facets leave it where the labels are.
int* round_map(picasso_ctx* c, bool by_facets, int round_) { return by_facets && round_ == 0 ? c->cid : c->vmap; }
// fresh: the first such round of a call that has had rounds by rings; the facets are the input's, the labels up to date.
void launch_facet_costs(picasso_ctx* c, hipStream_t s, int B, int round_, int cur_, int N, int F, bool fresh) {
    const int grid = prim::xcd_grid(facet_parts(F, N)), par = round_ & 1;
#define PICASSO_FACET_COSTS(PLACE, TILE, THREADS, FIRST)                                                                              \
    do {                                                                                                                                \
        static_assert((TILE) % (THREADS) == 0, "whole tiles");                                                                          \
        facet_costs_kernel<PLACE, THREADS, (TILE) / (THREADS), FIRST><<<grid, THREADS, 0, s>>>(                                         \
            c->fcur, F, c->st, cur_, c->vrec[cur_], c->vmin[0], c->vmin[1], c->ecost, round_tab(c, B, round_, cur_), fresh ? c->cid : round_map(c, true, round_ - 1), c->done, \
            c->cid, round_ > 1 && !fresh ? N : 0, c->opt_rcond_min, round_ > 1 && !fresh ? c->fcount() : nullptr, c->fcount(), c->nf_slots[par], c->nf_slots[par ^ 1]); \
    } while (0)
#define PICASSO_FACET_COSTS_TILE(PLACE, TILE, THREADS)                                \
    do {                                                                              \
        if (round_ == 0) PICASSO_FACET_COSTS(PLACE, TILE, FACET_LANES, true);         \
        else PICASSO_FACET_COSTS(PLACE, TILE, THREADS, false);                        \
    } while (0)
#define PICASSO_FACET_COSTS_PLACE(PLACE)                                                                                             \
    do {                                                                                                                             \
        if (facet_tile(F) == FACET_TILE_SMALL) PICASSO_FACET_COSTS_TILE(PLACE, FACET_TILE_SMALL, FACET_LANES);                       \
        else PICASSO_FACET_COSTS_TILE(PLACE, FACET_TILE_LARGE, FACET_LANES_LARGE);                                                   \
    } while (0)
    if (c->opt_placement == PLACE_INVERSE) PICASSO_FACET_COSTS_PLACE(PLACE_INVERSE);
    else PICASSO_FACET_COSTS_PLACE(PLACE_MEAN);
#undef PICASSO_FACET_COSTS_PLACE
#undef PICASSO_FACET_COSTS_TILE
#undef PICASSO_FACET_COSTS
}

// A round by rings up to its pairs (see ring_costs_kernel); budget: a budget step by budget_range_kernel follows.
constexpr int SUITOR_WAVES = 8192;  // as many as the chip holds
void launch_ring_round(picasso_ctx* c, hipStream_t s, int B, int round_, int cur_, int nv, int N, const SelArgs& sa, BudgetList* budget) {
    const int par = round_ & 1;
    const RingRows in = c->ring[par ^ 1], out = c->ring[par];
    {
        const KernelBracket timed(c, s, PICASSO_KERNEL_UNIQUE_COST, round_);
        const int tiles = (nv + RING_TILE - 1) / RING_TILE, n_labels = round_ > 1 ? N : 0;
        const int grid = prim::xcd_grid(tiles) + (n_labels + RING_LABELS - 1) / RING_LABELS;
#define PICASSO_RING_COSTS(PLACE, FIRST)                                                                                                            \
    ring_costs_kernel<PLACE, FIRST><<<grid, RING_THREADS, 0, s>>>(c->st, round_, nv, c->vrec[cur_], (FIRST) ? out : in, out, c->adj, c->vmin[1], c->vmin[0], \
                                                                  round_tab(c, B, round_, cur_), c->from, c->from_info, round_map(c, true, round_ - 1), c->cid,  \
                                                                  n_labels, c->opt_rcond_min, c->nf_slots[par], c->nf_slots[par ^ 1])
        if (c->opt_placement == PLACE_INVERSE) {
            if (round_ == 0) PICASSO_RING_COSTS(PLACE_INVERSE, true);
            else PICASSO_RING_COSTS(PLACE_INVERSE, false);
        } else {
            if (round_ == 0) PICASSO_RING_COSTS(PLACE_MEAN, true);
            else PICASSO_RING_COSTS(PLACE_MEAN, false);
        }
#undef PICASSO_RING_COSTS
    }
    {
        const KernelBracket timed(c, s, PICASSO_KERNEL_SUBROUND0, round_);
        const int waves = (int)std::min<long long>(((long long)nv + 63) / 64, SUITOR_WAVES), per = (int)(((long long)nv + waves - 1) / waves + 63) / 64 * 64;
        const int grid = prim::xcd_grid((int)(((long long)nv + (long long)per * prim::WAVES - 1) / ((long long)per * prim::WAVES)));
        suitor_kernel<<<grid, BLOCK, 0, s>>>(nv, per, round_, c->st, out, c->adj, c->vmin[1], c->vmin[0], in.taken);
    }
    const int chunks = prim::compact_chunks_for(nv), tiles = prim::compact_tiles(nv, chunks);
    switch (chunks) {
        case 1: pairs_kernel<1><<<tiles, BLOCK, 0, s>>>(sa, c->vmin[0], c->tilesum, budget); break;
        case 4: pairs_kernel<4><<<tiles, BLOCK, 0, s>>>(sa, c->vmin[0], c->tilesum, budget); break;
        default: pairs_kernel<16><<<tiles, BLOCK, 0, s>>>(sa, c->vmin[0], c->tilesum, budget);
    }
    if (tiles > prim::COMPACT_MAX_SUMMED_TILES) prim::compact_scan_sums(s, nullptr, nv, c->tilesum);
}

// Whether a call that has gone by rings goes on by facets, by the rings of the round before: where more than half a facet a vertex lies in rows (surfaces: 0.01 to 0.1; lattices of
// two sides none, whose second side a ring leaves out), or one is so long that its wave outlasts the others.  By rings | by facets from the second round on, us a call to
// a quarter: 500 wheels of 18 spokes 351 | 328, 20 k vertices of triangles of any three 508 | 366, a cone of 1,000 381 | 354; but 16 spheres of 4 k vertices with poles of 128 facets
// 245 | 266, of 1.2 M with poles of 1,024 1,015 | 1,153 (by facets throughout).
constexpr int RINGS_FEW = 2, RINGS_ALWAYS = 512, RINGS_LONG = 256, RINGS_LONG_EACH = 512;
bool by_facets_from_here(const State* st, int nv) {
    return (long long)RINGS_FEW * (st->row_words - RINGS_ALWAYS) > nv || std::max(st->longest[0], st->longest[1]) > RINGS_LONG + nv / RINGS_LONG_EACH;
}

// The distinct edges of a round by facets, for the statistics.  (In front of the selection the sorts' buffers are free but for the costs, which lie
// behind the first two, of 48 bytes a facet.)
void launch_count_edges(picasso_ctx* c, hipStream_t s, int round_, int F) {
    const long long slots = 6ll * F, words = 2 * slots;
    u32* const set = reinterpret_cast<u32*>(c->sort_buf);
    for (long long at = 0; at < words; at += 1 << 30) {
        const int n = (int)std::min(words - at, 1ll << 30);
        prim::fill_u32_kernel<<<grid_for(n), BLOCK, 0, s>>>(set + at, n, ~0u);
    }
    count_edges_kernel<<<grid_for(F, 8192), BLOCK, 0, s>>>(c->fcur, F, round_ > 0 ? c->fcount() : nullptr, ceil_log2(facet_tile(F)),
                                                          reinterpret_cast<u64*>(set), (u64)slots, &c->st->ne);
}

// Up to this many facets the facet set is cleared by the call's first kernel (see launch_init).
constexpr int64_t CLEAR_AHEAD_MAX_FACETS = 1 << 20;

// The validating kernel, instantiated for the sorts its keys go to.  work: rounds (or S0) follow; edges: the first round's
// set-up as well (EDGES_BY_FACETS), and its edges' digits (EDGES_SORTED).
int launch_init(picasso_ctx* c, hipStream_t s, const float* d_verts, int N, const int32_t* d_facets, int F, int B,
                bool work, int edges, const HeaderInit& init = HeaderInit{}, const FewMeshes& tables = FewMeshes{}, bool rings = false) {
    const prim::KeySort<u64> I = incidence_sort(c, N, F), E = edge_sort(c, N, F, F, 3ll * F);
    if (work && c->hist_dirty)  // (a call ended between a count of its edges and their sort)
        prim::fill_u32_kernel<<<prim::MSD_ZERO_WORDS / BLOCK, BLOCK, 0, s>>>(c->hist12, prim::MSD_ZERO_WORDS, 0u);
    if (work) {
        c->hist_dirty = edges == EDGES_SORTED && F > 0;
        clear_wide_counts(s, I);
        if (edges == EDGES_SORTED) clear_wide_counts(s, E);
    }
    float4* planes = work ? facet_planes(c) : nullptr;
    // the facet set that the end of the call uses (larger ones are cleared by the last contraction, when fewer facets are left)
    const int n_clear = F <= CLEAR_AHEAD_MAX_FACETS ? (int)facet_slots((size_t)F) : 0;
#define PICASSO_INIT_TABLES(COUNT, SORTED, TABLES)                                                                             \
    init_kernel<COUNT, SORTED><<<grid_for(std::max(N, F), 4096), BLOCK, 0, s>>>(                                                      \
        d_verts, N, d_facets, F, B, c->voff[0], c->foff, c->vrec[0], edges == EDGES_BY_FACETS ? nullptr : c->cid, rings ? nullptr : c->fcur, incidence_fbits(F), digit_count(I),      \
        digit_count(E), edges, E.key_bits / 2, c->st, init, TABLES, planes, c->htab, n_clear, c->vmin[0], rings ? nullptr : c->vmin[1],   \
        c->mate, c->pcost(), round_tab(c, B, 0, 0), rings ? c->rows_taken : nullptr)
#define PICASSO_INIT_EDGES(COUNT, SORTED)                                           \
    do {                                                                            \
        if (B == 1) PICASSO_INIT_TABLES(COUNT, SORTED, OneMesh{tables.target[0]});  \
        else PICASSO_INIT_TABLES(COUNT, SORTED, tables);                            \
    } while (0)
#define PICASSO_INIT(COUNT)                                             \
    do {                                                                \
        if (edges == EDGES_SORTED) PICASSO_INIT_EDGES(COUNT, true);     \
        else PICASSO_INIT_EDGES(COUNT, false);                          \
    } while (0)
    if (!work) PICASSO_INIT_EDGES(COUNT_NONE, false);
    else if (count_kind(I) == COUNT_SMALL) PICASSO_INIT(COUNT_SMALL);
    else if (count_kind(I) == COUNT_LARGE) PICASSO_INIT(COUNT_LARGE);
    else PICASSO_INIT(COUNT_XL);
#undef PICASSO_INIT
#undef PICASSO_INIT_EDGES
#undef PICASSO_INIT_TABLES
    return hipGetLastError() == hipSuccess ? PICASSO_OK : PICASSO_ERR_HIP;
}

// Fills the pinned image of the header (State + per-mesh tables) and sends it with one copy.
// `by_kernel`: only the image; the first kernel writes the header itself (few meshes, see HeaderInit).
int upload_header(picasso_ctx* c, hipStream_t s, int B, const int32_t* nv_in, const int32_t* nf_in,
                  const int32_t* target, int64_t* N_out, int64_t* F_out, bool by_kernel = false) {
    const int cb = c->cap_b;
    int* img = c->h_pin + c->h_up_off;
    const int total = (int)hdr_ints((size_t)cb);
    memset(img, 0, sizeof(int) * total);
    int* hv = img + (c->voff[0] - c->hdr);
    int* hf = img + (c->foff - c->hdr);
    int* ht = img + (c->target - c->hdr);
    int64_t nacc = 0, facc = 0;
    for (int b = 0; b < B; ++b) {
        if (nv_in[b] < 1 || nf_in[b] < 0 || target[b] < 1) return PICASSO_ERR_INVALID_ARG;
        hv[b] = (int)nacc;
        hf[b] = (int)facc;
        ht[b] = target[b];
        nacc += nv_in[b];
        facc += nf_in[b];
        if (nacc > c->max_verts || facc > c->max_facets) return PICASSO_ERR_WORKSPACE;
    }
    hv[B] = (int)nacc;
    hf[B] = (int)facc;
    State* h = reinterpret_cast<State*>(img);
    h->nv[0] = (int)nacc;
    *N_out = nacc;
    *F_out = facc;
    if (!by_kernel) HIP_TRY(c, hipMemcpyAsync(c->hdr, img, sizeof(int) * total, hipMemcpyHostToDevice, s));
    return PICASSO_OK;
}

// The signal for the next kernel after which the host looks at the read-back area.
// (The number wraps around after 2^32 signals; only equality with the last one stored matters.)
HostSignal next_signal(picasso_ctx* c) {
    c->host_seq = (int)((unsigned)c->host_seq + 1u);
    return HostSignal{c->h_pin_dev + c->h_seq_off, c->host_seq};
}

// Waits until the kernel that was given `sig` has written its results to the pinned read-back
// area.  That kernel stores the sequence number after them (system-scope release), so the host
// watches the word: it sees it some microseconds before a stream synchronisation would return,
// and everything queued on the stream before that kernel is complete by then as well.  Falls back
// to the stream synchronisation when the word has not changed within the context's limit (20 ms
// unless set otherwise; 0 = do not watch at all), which also brings any launch error to light.
hipError_t wait_for_signal(picasso_ctx* c, hipStream_t s, const HostSignal& sig) {
    if (c->opt_poll_us > 0) {
        const int* word = c->h_pin + c->h_seq_off;
        const auto t0 = std::chrono::steady_clock::now();
        const auto limit = std::chrono::microseconds(c->opt_poll_us);
        const long check_every = c->opt_poll_us >= 1000 ? 1023 : 15;  // (the clock is read every so many looks)
        for (long spins = 1;; ++spins) {
            if (__atomic_load_n(word, __ATOMIC_ACQUIRE) == sig.seq) return hipSuccess;
            if ((spins & check_every) == 0 && std::chrono::steady_clock::now() - t0 > limit) break;
#if defined(__x86_64__)
            __builtin_ia32_pause();
#endif
        }
    }
    return hipStreamSynchronize(s);
}

// [State][matched][mesh_facets] brought to the pinned read-back area by a one-workgroup kernel that then
// tells the host; returns when the host has them (and everything queued before has been executed).
int read_header(picasso_ctx* c, hipStream_t s, u32* zero = nullptr, int n_zero = 0) {
    const HostSignal done = next_signal(c);
    publish_header_kernel<<<1, BLOCK, 0, s>>>(c->hdr, HDR_STATE_INTS + 2 * c->cap_b + 1, c->h_pin_dev, done, zero, n_zero,
                                             conv::EXT_PAD);
    HIP_TRY(c, wait_for_signal(c, s, done));
    return PICASSO_OK;
}

int status_from_err_bits(int bits) {
    if (bits & ERR_BIT_INTERNAL) return PICASSO_ERR_INTERNAL;
    if (bits & ERR_BIT_BAD_INDEX) return PICASSO_ERR_BAD_INDEX;
    if (bits & ERR_BIT_NONFINITE) return PICASSO_ERR_NONFINITE;
    return PICASSO_OK;
}

// The budget step of a single mesh in rounds by rings goes by budget_range_kernel between these (pairs there may be at most).  Below the first the search of one workgroup takes
// no longer; up to the second the list holds what the sample points at, at most 18 % of the pairs of lattices and rooms.  In a batch the meshes' searches share the chip already
// (16 meshes of 32 k vertices 18 us).
constexpr int BUDGET_GROUPS = 255;  // workgroups that release, one a compute unit with the one that tells the host
constexpr int BUDGET_CHIP_MIN = 1 << 13, BUDGET_CHIP_MAX = 180000;
static_assert(offsetof(BudgetList, entry) + BUDGET_CHIP_MIN * sizeof(u64) <= 2 * BUDGET_CHIP_MIN * sizeof(u64), "a word for each of its vertices (budget_list): as many entries as it has pairs");
static_assert(offsetof(BudgetList, entry) + BUDGET_LIST * sizeof(u64) <= (2 * BUDGET_LIST + 2) * sizeof(u64), "... or all");
static_assert(2ll * BUDGET_CHIP_MAX <= (long long)BLOCK * prim::COMPACT_MAX_SUMMED_TILES, "tiles of one chunk");

// Budget step: among a mesh's keys (its formed pairs, or the vertices that could join clusters by line 11) where there are more
// of them than it may use (counts[b] > budgets[b]) the budgets[b] first ones in ascending (cost key, tie-break) order stay;
// the others are released.  most = the largest such count; nv_max = all meshes' vertices; least = the smallest.
// `guarded` (most <= the limit of one workgroup per mesh only): queued behind the
// selection tail before the host has looked; the counts are then upper bounds and the
// kernel does nothing unless the tail finished the matching; it stores `tell` first.
// by_count: the kernel that counts the survivors releases what the search of one workgroup per mesh leaves beyond its limits.
template <class Keys>
int budget_step(picasso_ctx* c, hipStream_t s, const Keys& K, int B, const int* voff, int nv_max, int most, int least,
                const int* counts, const int* budgets, bool by_count, bool guarded = false, HostSignal tell = HostSignal{nullptr, 0},
                const PairPublish& publish = PairPublish{-1}) {
    const int limit = (int)c->opt_trunc_block_max;
    const bool longer = most > limit;
    if (guarded && longer) return PICASSO_ERR_INVALID_ARG;
    if (least <= limit) {
        const int* guard = guarded ? &c->st->go : nullptr;
        const int need = std::min(most, limit);
        const int longer_than = longer ? limit : 0x7FFFFFFF;
        int cap = need <= TRUNC_SMALL_CAP ? TRUNC_SMALL_CAP : TRUNC_BLOCK_CAP;
        if (c->opt_trunc_width) cap = c->opt_trunc_width * TRUNC_THREADS;  // (test hook)
        const bool here = cap <= TRUNC_SMALL_CAP && !by_count;  // (few keys: released by the search itself)
        KeyLimit* limits = here ? nullptr : c->limits;
        trunc_mesh_kernel<Keys><<<B + (publish.at >= 0 ? 1 : 0), TRUNC_THREADS, 0, s>>>(K, voff, counts, budgets, cap, longer_than, guard, c->st, tell, limits, publish);
        if (!here && !by_count) trunc_release_kernel<Keys><<<grid_for(nv_max), BLOCK, 0, s>>>(K, nv_max, voff, B, c->limits);
    }
    if (longer) {
        SelectSlot* S = c->select_slots;
        const int by_start = B == 1 || limit == TRUNC_BLOCK_CAP;  // (see select_slot)
        const int slots = by_start ? select_slots_by_start(B, nv_max) : std::min(B, SELECT_MESHES);
        const long long words = (long long)slots * (long long)(sizeof(SelectSlot) / sizeof(u32));
        const int tie_bits = Keys::TIE_BY_VERTEX ? ceil_log2(nv_max) : 32;
        const int passes = SELECT_COST_PASSES + (tie_bits + SELECT_BITS - 1) / SELECT_BITS;
        const int group = by_start ? SELECT_GRID_MESHES : SELECT_MESHES;
        for (int b0 = 0; b0 < B; b0 += group) {
            const dim3 grid((unsigned)((nv_max + BLOCK * SELECT_ITEMS - 1) / (BLOCK * SELECT_ITEMS)), (unsigned)std::min(B - b0, group));
            if (b0 == 0 || !by_start)
                prim::fill_u32_kernel<<<grid_for(words), BLOCK, 0, s>>>(reinterpret_cast<u32*>(S), (int)words, 0u);
            for (int p = 0; p < passes; ++p)
                select_pass_kernel<Keys><<<grid, BLOCK, 0, s>>>(K, voff, counts, budgets, limit, S, by_start, b0, p, tie_bits);
            select_release_kernel<Keys><<<grid, BLOCK, 0, s>>>(K, voff, counts, budgets, limit, S, by_start, b0, passes, tie_bits);
        }
    }
    return hipGetLastError() == hipSuccess ? PICASSO_OK : PICASSO_ERR_HIP;
}
int pair_budget(picasso_ctx* c, hipStream_t s, const TieBreak& tb, int B, const int* voff, int nv_max, int most, int least,
                bool by_count, bool guarded = false, HostSignal tell = HostSignal{nullptr, 0}, const PairPublish& publish = PairPublish{-1}) {
    if (tb.on)
        return budget_step(c, s, PairKeys<true>{c->pcost(), c->ptie(), c->mate}, B, voff, nv_max, most, least, c->matched, c->nrem, by_count, guarded, tell, publish);
    return budget_step(c, s, PairKeys<false>{c->pcost(), nullptr, c->mate}, B, voff, nv_max, most, least, c->matched, c->nrem, by_count, guarded, tell, publish);
}

// Sub-round k of the selection.  last: it lists the edges it leaves live for the tail.
// many: most edges are live still, also beyond the first sub-rounds, so bids are put together in LDS there, too (400 k vertices of one plane,
// to a quarter: 56 -> 28 ms).
void launch_subround(picasso_ctx* c, hipStream_t s, const SelArgs& sa, int k, bool last, bool many, int round) {
    const bool listed = sa.bound >= LISTED_MIN_EDGES;
    const KernelBracket timed(c, s, PICASSO_KERNEL_SUBROUND0, round, k == 0); /* (the first only) */
    const int tiles = sa.fcur ? sa.list_tiles : (sa.bound - 1) / LISTED_TILE + 1;
    const int shift = listed_part_shift(k, tiles), group = 1 << listed_group_shift(k, shift, tiles);
    if (sa.fcur) {
        if (k == 0) {
            const int grid = prim::xcd_grid(sa.parts);
            const bool small = facet_tile(sa.n_facets) == FACET_TILE_SMALL;
            constexpr int PER_SMALL = FACET_TILE_SMALL / FACET_LANES, PER_LARGE = FACET_TILE_LARGE / FACET_LANES;
            if (small && last) select_facets_kernel<FACET_LANES, PER_SMALL, true><<<grid, FACET_LANES, 0, s>>>(sa);
            else if (small) select_facets_kernel<FACET_LANES, PER_SMALL, false><<<grid, FACET_LANES, 0, s>>>(sa);
            else if (last) select_facets_kernel<FACET_LANES, PER_LARGE, true><<<grid, FACET_LANES, 0, s>>>(sa);
            else select_facets_kernel<FACET_LANES, PER_LARGE, false><<<grid, FACET_LANES, 0, s>>>(sa);
            return;
        }
        const int parts = ((tiles - 1) >> shift) + 1, groups = prim::xcd_grid((parts + group - 1) / group);
        const int grid = groups + (last ? (sa.nv + COUNT_VERTICES - 1) / COUNT_VERTICES : 0);
        if (k <= 2 || many) {
            if (last) select_listed_kernel<false, true, true, true><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, groups);
            else select_listed_kernel<false, true, false, true><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, groups);
        } else {
            if (last) select_listed_kernel<false, true, true, false><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, groups);
            else select_listed_kernel<false, true, false, false><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, groups);
        }
        return;
    }
#define PICASSO_SUBROUND(SHUFFLE, APPEND)                                                                                   \
    do {                                                                                                                     \
        if (!listed) {                                                                                                       \
            select_subround_kernel<SHUFFLE, APPEND><<<grid_for(sa.bound), BLOCK, 0, s>>>(sa, k);                             \
        } else if (k == 0) {                                                                                                 \
            select_first_kernel<SHUFFLE, APPEND><<<prim::xcd_grid((sa.bound + LISTED_TILE - 1) / LISTED_TILE), BLOCK, 0, s>>>(sa); \
        } else {                                                                                                             \
            const int parts = ((tiles - 1) >> shift) + 1;                                                                     \
            const int grid = prim::xcd_grid((parts + group - 1) / group);                                                    \
            if (k <= 2 || many) select_listed_kernel<SHUFFLE, false, APPEND, true><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, grid); \
            else select_listed_kernel<SHUFFLE, false, APPEND, false><<<grid, BLOCK, 0, s>>>(sa, k, shift, group, grid);       \
        }                                                                                                                    \
    } while (0)
    if (sa.tb.on) {
        if (last) PICASSO_SUBROUND(true, true);
        else PICASSO_SUBROUND(true, false);
    } else {
        if (last) PICASSO_SUBROUND(false, true);
        else PICASSO_SUBROUND(false, false);
    }
#undef PICASSO_SUBROUND
}

// Alg. 2 line 11 on the device for the round whose pairs are final (see the kernels).  First its candidates, counted per mesh; `counted` is
// told when the counts are in the read-back area.  ne: the round's edges at most.
void list_joiners(picasso_ctx* c, hipStream_t s, int B, int cur, int vbits, int ne, int nv_total, const MeshTab& mt, const TieBreak& tb,
                  const HostSignal& counted) {
    absorb_begin_kernel<<<grid_for(std::max(nv_total, B), 4096), BLOCK, 0, s>>>(c->abid, c->arep, c->st, cur, B, c->nrem,
                                                                              c->matched, c->arem, c->acand);
    absorb_bid_kernel<<<grid_for(std::max(ne, 1), 8192), BLOCK, 0, s>>>(c->ekey, c->ecost, c->st, vbits, c->mate, mt,
                                                                      c->arem, c->abid, tb);
    JoinPred jp{c->ekey, c->ecost, c->mate, c->abid, vbits, tb};
    JoinListOut jl{c->list};
    prim::compact(s, jp, jp, jl, &c->st->ne, ne, c->tilesum, &c->st->absorb_n);
    int* host_counts = c->h_pin_dev + HDR_STATE_INTS + c->cap_b;  // (the offsets' slots of the read-back area: free until the end)
    absorb_count_kernel<<<1, ABSORB_COUNT_THREADS, 0, s>>>(c->list, c->st, c->ekey, vbits, B, c->voff[cur], c->acand, host_counts, counted);
}
// Then, when the host has the counts, what the budgets leave of them.  nrem / h_matched: per-mesh budget and pairs kept (host mirrors);
// h_joined receives the vertices that join per mesh; where any does, aoff and joiners() list them by representative.  (The counts decide
// whether the budget step is needed.)
int run_absorb(picasso_ctx* c, hipStream_t s, int B, int cur, int vbits, int nv_total, const TieBreak& tb, const int* nrem,
               const int* h_matched, int* h_joined) {
    const int* h_cand = c->h_pin + HDR_STATE_INTS + c->cap_b;
    long long n_list = 0;
    int most = 0, least = 0x7FFFFFFF;
    for (int b = 0; b < B; ++b) {
        const int left = (h_matched[b] > 0 && nrem[b] > h_matched[b]) ? nrem[b] - h_matched[b] : 0;
        const int cand = h_cand[b];
        n_list += cand;
        if (cand > left) {
            most = std::max(most, cand);
            least = std::min(least, cand);
        }
        h_joined[b] = std::min(cand, left);
    }
    if (n_list == 0) return PICASSO_OK;
    if (most > 0) {  // the cheapest `left` candidates of each such mesh stay
        const int rc = budget_step(c, s, JoinKeys{c->abid}, B, c->voff[cur], nv_total, most, least, c->acand, c->arem, false);
        if (rc != PICASSO_OK) return rc;
    }
    prim::KeySort<u64> S = key_sort_for(c, false, n_list, (int)n_list, 2 * vbits);
    S.n_ptr = &c->st->absorb_n;
    // (few keys over many representatives: a digit or two more, where a group of a bucket is then one of them)
    const int within = S.low_bits() - vbits, more = within - prim::BUCKET_GROUP_BITS;
    if (more > 0 && S.digit_bits + more <= prim::NARROW_BITS_MAX) {
        S.digit_bits += more;
        S.half = S.fits_half();
    }
    rows_of(S, nv_total, vbits, n_list);
    S.crowded = false;  // (joined vertices lie where the pairs do, all over the mesh)
    clear_wide_counts(s, S);
    absorb_keys_kernel<<<grid_for(n_list), BLOCK, 0, s>>>(c->list, c->st, c->ekey, c->ecost, vbits, c->mate, c->abid,
                                                         c->arep, c->key64[0], digit_count(S), tb);
    const RowLists lists{c->aoff, c->joiners(), (int)n_list, nv_total, vbits, S.digit_bits};
    if (!prim::key_sort(s, S, (const prim::KeySort<u64>*)nullptr, prim::OneSource<JoinedKeys>{{c->key64[0], edge_sentinel(vbits)}}, lists)) return PICASSO_ERR_HIP;
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int decimate_impl(picasso_ctx* c, hipStream_t s, int B, const float* d_verts, const int32_t* d_facets,
                  const int32_t* nv_in, const int32_t* nf_in, const int32_t* target_nv, float* d_verts_out,
                  int32_t* d_facets_out, int32_t* d_cluster_id, int32_t* h_nv_out, int32_t* h_nf_out,
                  picasso_stats* stats) {
    if (!c || !d_verts || !nv_in || !nf_in || !target_nv || !d_verts_out || !d_facets_out || !d_cluster_id ||
        !h_nv_out || !h_nf_out || B < 1)
        return PICASSO_ERR_INVALID_ARG;
    if (B > c->max_meshes) return PICASSO_ERR_WORKSPACE;
    HIP_TRY(c, hipSetDevice(c->device));
    if (stats) memset(stats, 0, sizeof(*stats));

    int64_t N64 = 0, F64 = 0;
    const bool header_by_kernel = B <= HEADER_MESHES;  // few meshes: no copy in front of the first kernel
    int rc = upload_header(c, s, B, nv_in, nf_in, target_nv, &N64, &F64, header_by_kernel);
    if (rc != PICASSO_OK) return rc;
    if (F64 > 0 && !d_facets) return PICASSO_ERR_INVALID_ARG;
    const int N = (int)N64, F = (int)F64;
    HeaderInit hinit{};
    FewMeshes tables{};
    if (header_by_kernel) {
        hinit.hdr = c->hdr;
        hinit.total = (int)hdr_ints((size_t)c->cap_b);
        hinit.at_voff0 = (int)(c->voff[0] - c->hdr);
        hinit.at_foff = (int)(c->foff - c->hdr);
        hinit.at_target = (int)(c->target - c->hdr);
        const int* img = c->h_pin + c->h_up_off;
        memcpy(tables.voff, img + hinit.at_voff0, sizeof(int) * (B + 1));
        memcpy(tables.foff, img + hinit.at_foff, sizeof(int) * (B + 1));
        memcpy(tables.target, img + hinit.at_target, sizeof(int) * B);
    }

    c->n_ev = 0;
    c->kt.pool = c->kt_pool;
    c->kt.cap = (int)(sizeof(c->kt_pool) / sizeof(c->kt_pool[0]));
    c->kt.recs = c->kt_recs;
    c->kt.used = 0;
    c->kt.nrec = 0;
    c->kt_this_call = c->opt_kernel_timing > 0 && (c->kt_calls++ % c->opt_kernel_timing) == 0;
    struct TimingScope {  // (no brackets outside this call, however it ends)
        picasso_ctx* c;
        ~TimingScope() { c->kt_this_call = false; }
    } timing_scope{c};
    c->n_rounds_noted = 0;
    StageTimer tm{c, s, c->opt_stage_timing != 0 && stats != nullptr};
    if (stats) HIP_TRY(c, hipEventRecord(c->ev_total[0], s));  // (an event costs queue time: only when asked for)

    // host mirror of the per-mesh vertex counts
    int* const nvb = c->h_mesh;
    int* const stuck = nvb + c->max_meshes;
    int* const act = stuck + c->max_meshes;
    int* const nrem = act + c->max_meshes;
    int* const h_matched = nrem + c->max_meshes;
    int* const h_joined = h_matched + c->max_meshes;
    for (int b = 0; b < B; ++b) {
        nvb[b] = nv_in[b];
        stuck[b] = act[b] = nrem[b] = h_matched[b] = h_joined[b] = 0;
    }
    auto any_active = [&]() {
        bool any = false;
        for (int b = 0; b < B; ++b) {
            act[b] = (nvb[b] > target_nv[b]) && !stuck[b];
            nrem[b] = act[b] ? nvb[b] - target_nv[b] : 0;
            any |= (act[b] != 0);
        }
        return any;
    };
    bool work = any_active() && c->opt_max_rounds != 0;

    // In the first round the sorts of the incidence keys (S0) and of the edge keys (S1) depend only on the validated
    // input, not on each other: they share their launches.  (Not when stage times are being recorded, to keep them
    // attributable, and in a call whose kernels are bracketed by events: a bracketed kernel then has the chip to itself,
    // and its duration is its own.)
    // The rounds go by facets where nothing needs the edges' numbers (see facet_costs_kernel; a call that gives statistics and
    // brackets its kernels brackets those of the sorts).  By sorted edges | by facets, us: rooms of 115 k vertices to 25 % 279 | 237, to 70 % (one round)
    // 163 | 157, a lattice of 400 k 455 | 359, 260 | 231.  Facets in no order, whose bids find no place in the workgroups' tables, gain where rounds
    // follow the first, and one round of them alone only beyond a million vertices: 115 k to 25 % 434 | 352, to 70 % 247 | 254, an icosphere of 164 k 453 | 420,
    // 233 | 263, 1.2 M 2,550 | 2,091, 1,803 | 1,639.  (The first round could be sorted where the host knew the order; a look at the word in front
    // of a bid's atomic takes longer: 263 -> 287.)
    const bool by_facets = c->opt_shuffle_seed == 0 && !c->opt_absorb && !(stats && c->kt_this_call);
    // ... and of these by rings (see ring_costs_kernel) where the vertices have about six facets, as on a surface; in calls for statistics, which count the edges of
    // the facets, by facets.  By facets | by rings, us: lattices of 20 k vertices to a quarter 184 | 147, of 400 k 381 | 307, an icosphere of 164 k 385 | 249, facets permuted, 115 k
    // 389 | 243, 2.25 M 4,179 | 2,663, vertices as well 407 | 265, 4,928 | 4,106, a flat lattice of 116 k 8,694 | 1,867.  Lattices of two sides (twelve facets a vertex, six
    // neighbours) beside vertices of no facet, or beside a lattice, which pass the rule: 40 k to 70 % 181 | 168, 8 k among 64 k 204 | 182 to a quarter.  20 k vertices with 60 k facets of any three
    // of them 375 | 621.  With 40 k, which pass it, nearly every vertex has more neighbours than a short ring, which the quadrics' kernel finds out, and the call goes by facets after all:
    // 310 | 327 (to 70 %, one round, 123 | 157).
    // Vertices of many facets, which the host cannot see beforehand: see ring_costs_kernel and by_facets_from_here.
    // Rounds by rings read the call's facets to its end, where its last kernels write: outputs laid over them (d_facets_out but for, which is written behind the last read) go by
    // facets, which are copied first.
    auto over_facets = [&](const void* out, size_t bytes) {
        const uintptr_t a = (uintptr_t)out, b = (uintptr_t)d_facets;
        return a < b + sizeof(int32_t) * 3 * (size_t)F && b < a + bytes;
    };
    const bool laid_over = over_facets(d_verts_out, sizeof(float) * 3 * (size_t)N) || over_facets(d_cluster_id, sizeof(int32_t) * (size_t)N);
    bool rings = by_facets && !stats && work && F > 0 && 4ll * F <= 9ll * N && N < RING_VERTICES && !laid_over;
    bool fresh = false;  // (see launch_facet_costs)
    const bool together = work && !by_facets && F > 0 && c->opt_overlap && !tm.on && !c->kt_this_call &&
                          edge_sort(c, N, F, F, 3ll * F).half == incidence_sort(c, N, F).half;
    tm.begin(0, PICASSO_ST_QUADRICS);
    rc = launch_init(c, s, d_verts, N, d_facets, F, B, work, !work ? EDGES_NONE : by_facets ? EDGES_BY_FACETS : EDGES_SORTED, hinit, tables, rings);
    if (rc != PICASSO_OK) return rc;
    if (work) {
        const prim::KeySort<u64> I = incidence_sort(c, N, F);
        if (together) {
            if (!sort_edges_and_incidences(c, s, edge_sort(c, N, F, F, 3ll * F), I, d_verts, N, F)) return PICASSO_ERR_HIP;
        } else if (F > 0) {
            if (!(rings ? sort_incidences<true>(c, s, I, d_verts, d_facets, N, F) : sort_incidences<false>(c, s, I, d_verts, c->fcur, N, F))) return PICASSO_ERR_HIP;
        }
    }
    tm.end();

    State* hst = reinterpret_cast<State*>(c->h_pin);  // read-back area
    const TieBreak tb{c->opt_shuffle_seed != 0 ? 1u : 0u, (u32)c->opt_shuffle_seed, (u32)(c->opt_shuffle_seed >> 32)};

    int cur = 0;        // ping-pong index of vrec / facets / voff / State counts
    int nv_total = N;   // exact (host mirror)
    int nf_bound = F;   // upper bound on the facets that have not collapsed
    size_t slots_clear = F <= CLEAR_AHEAD_MAX_FACETS ? facet_slots((size_t)F) : 0;  // leading slots of the facet set that are clear
    int round = 0;
    int ne_prev = 0, nv_prev = 0;  // edge and vertex counts of the round before
    bool validated = false;
    bool compacted = false;   // collapsed facets have left their tiles
    bool renumbered = false;  // the facets and labels still have the numbers from before the last contraction

    auto facets_again = [&](const int* map) {
        nf_bound = F;  // (rings may hold repeated facets once)
        facets_again_kernel<<<grid_for(std::max(std::max(nv_total, F), map ? N : 0), 4096), BLOCK, 0, s>>>(d_facets, F, c->fcur, nv_total, c->vmin[0], c->vmin[1],
                                                                                                       c->nf_slots[round & 1], c->cid, map, N);
    };

    while (work && (c->opt_max_rounds < 0 || round < c->opt_max_rounds)) {
        const int nrec_before = c->kt.nrec;  // (bracketed launches before this round)
        if (rings && round > 0 && by_facets_from_here(hst, nv_total)) {
            rings = false;
            fresh = true;
            facets_again(round > 1 ? c->vmap : nullptr);
        }
        const int H = 3 * nf_bound;
        const int vbits = edge_vertex_bits(nv_total, H);
        MeshTab mt{B, c->voff[cur], c->target, c->active[round & 1], c->nrem, c->matched, c->mslots};

        // ---- S1 (+S2): edges and costs
        tm.begin(round, PICASSO_ST_EDGES);
        const unsigned char way = rings ? WAY_RINGS : by_facets ? (fresh ? WAY_FACETS_AGAIN : WAY_FACETS) : WAY_SORTED;
        if (rings) {  // (below: with the selection)
        } else if (by_facets) {
            const KernelBracket timed(c, s, PICASSO_KERNEL_UNIQUE_COST, round);
            launch_facet_costs(c, s, B, round, cur, N, F, fresh);
            fresh = false;
            compacted = round > 0;
        } else {
            const prim::KeySort<u64> E = edge_sort(c, nv_total, nf_bound, F, round > 0 ? expected_half_edges(H, ne_prev, nv_prev - nv_total) : H);
            if (round > 0) launch_edge_keys(c, s, B, round, cur, E, N, F);
            if (!(round == 0 && together) && H > 0 && !sort_edges(c, s, E, round)) return PICASSO_ERR_HIP;
            const KernelBracket timed(c, s, PICASSO_KERNEL_UNIQUE_COST, round);
            launch_unique_cost(c, s, E, H, mt, tb, c->vrec[cur]);
        }
        const bool was_renumbered = renumbered;
        renumbered = false;
        tm.end();
        if (by_facets && stats && F > 0 && round < PICASSO_STATS_ROUNDS) {
            tm.begin(round, PICASSO_ST_COUNT);
            launch_count_edges(c, s, round, F);
            tm.end();
        }

        // The contraction.  `guarded`: queued behind the selection tail before the host
        // has looked; it then goes by what the tail leaves in State (go, guard_nv) and does
        // nothing unless it finished the matching.  clear: slots of the facet set to clear on the way.
        // releases: a budget step has left limits that the count applies.
        // counted: the tiles' survivors are there already (see pairs_kernel).
        auto issue_contract = [&](int n_joined, size_t clear, bool releases, bool guarded, HostSignal tell, bool counted = false, PairPublish publish = PairPublish{-1}) {
            const int nxt = cur ^ 1;
            const int* guard = guarded ? &c->st->go : nullptr;
            const int* n_ptr = guarded ? &c->st->guard_nv : nullptr;
            const bool counts = n_joined == 0 && !releases && nv_total <= CONTRACT_COUNTS_MAX && !counted;
            if (counts || counted) {
            } else if (n_joined > 0) {
                prim::compact_count(s, AlivePredT<true>{c->mate, c->arep}, n_ptr, nv_total, c->tilesum);
            } else if (releases && tb.on) {
                const ReleasingPred<true> pred{{c->pcost(), c->ptie(), c->mate}, c->voff[cur], B, c->limits};
                prim::compact_count(s, SignalingPred<ReleasingPred<true>>{pred, tell}, n_ptr, nv_total, c->tilesum);
            } else if (releases) {
                const ReleasingPred<false> pred{{c->pcost(), nullptr, c->mate}, c->voff[cur], B, c->limits};
                prim::compact_count(s, SignalingPred<ReleasingPred<false>>{pred, tell}, n_ptr, nv_total, c->tilesum);
            } else {
                SignalingPred<AlivePredT<false>> first{{c->mate, nullptr}, tell};  // (`tell.word` may be null: nothing to tell)
                prim::compact_count(s, first, n_ptr, nv_total, c->tilesum);
            }
            const int chunks = prim::compact_chunks_for(nv_total), tiles = prim::compact_tiles(nv_total, chunks);
            const int prefixed = tiles > prim::COMPACT_MAX_SUMMED_TILES;
            if (publish.at >= 0) publish.at = tiles;
            const int grid = tiles + (publish.at >= 0 ? 1 : 0);
            static_assert(CONTRACT_COUNTS_MAX <= BLOCK * prim::COMPACT_MAX_SUMMED_TILES, "tiles of one chunk");
#define PICASSO_CONTRACT(PLACE, ABSORB, COUNTS, RCOND)                                                               \
    contract_kernel<PLACE, ABSORB, COUNTS><<<grid, BLOCK, 0, s>>>(c->vrec[cur], c->vrec[nxt], c->mate, round_map(c, by_facets, round), c->st, cur,  \
                                                           chunks, c->tilesum, prefixed, B, c->voff[cur],             \
                                                           c->voff[nxt], c->matched, c->done, c->htab, (int)clear, \
                                                           by_facets ? c->vmin[0] : nullptr, RCOND, c->arep, c->aoff, c->joiners(), guard, tell, publish, \
                                                           rings ? c->from : nullptr, c->from_info, c->ring[round & 1].info)
            if (c->opt_placement == PLACE_INVERSE) {
                if (n_joined > 0) PICASSO_CONTRACT(PLACE_INVERSE, true, false, c->opt_rcond_min);
                else if (counts) PICASSO_CONTRACT(PLACE_INVERSE, false, true, c->opt_rcond_min);
                else PICASSO_CONTRACT(PLACE_INVERSE, false, false, c->opt_rcond_min);
            } else {
                if (n_joined > 0) PICASSO_CONTRACT(PLACE_MEAN, true, false, 0.0f);
                else if (counts) PICASSO_CONTRACT(PLACE_MEAN, false, true, 0.0f);
                else PICASSO_CONTRACT(PLACE_MEAN, false, false, 0.0f);
            }
#undef PICASSO_CONTRACT
        };
        // Where no mesh can form more pairs than its budget allows (a matching pairs at most half the
        // vertices) and nothing else has to be decided after the selection, the contraction is queued
        // right behind the tail: the device does not idle while the host looks.
        // Where the budget will bind (a mesh has to stop below 40 % of its vertices; a matching on these
        // meshes pairs 85-95 % of them) and the per-mesh search can take every such mesh, the budget step
        // is queued there too, in front of it: it finds on the device which meshes are over their
        // budgets, and does nothing where none is.  In between (40-50 %) nothing is queued ahead.
        // (Rounds larger still take long enough for the idling not to count, and then know which contraction is the last, which clears
        // the facet set on its way.)
        constexpr int AHEAD_MAX_FACETS = 1 << 22;
        bool ahead_ok = !c->opt_absorb && !stats && c->opt_ahead && nf_bound <= AHEAD_MAX_FACETS;
        bool ahead_budget = false, chip_budget = false;
        int seg_bound = 0;  // pairs of the largest mesh that may exceed its budget, at most
        if (ahead_ok) {
            bool likely = false;
            for (int b = 0; b < B; ++b)
                if (act[b] && 2ll * nrem[b] < nvb[b]) {
                    seg_bound = std::max(seg_bound, nvb[b] / 2);
                    likely |= 5ll * nrem[b] < 2ll * nvb[b];
                }
            ahead_budget = seg_bound > 0;
            chip_budget = rings && B == 1 && seg_bound > BUDGET_CHIP_MIN && seg_bound <= BUDGET_CHIP_MAX && c->opt_trunc_block_max == TRUNC_BLOCK_CAP && !c->opt_trunc_width;
            if (ahead_budget && !(likely && (chip_budget || seg_bound <= c->opt_trunc_block_max))) ahead_ok = false;
        }
        // Line 11's candidates likewise, where no budget step can come in front of them: one look of the host less (its counts come with the tail's;
        // should the tail hand back, they are made again).  Not in listed rounds, whose lists lie where the candidates go.
        bool joiners_ahead = c->opt_absorb && !stats && c->opt_ahead && std::max(H, 1) < LISTED_MIN_EDGES;
        for (int b = 0; b < B; ++b) joiners_ahead &= !act[b] || 2ll * nrem[b] >= nvb[b];
        bool ahead = false;  // the kernels are queued and the tail has finished the matching

        // ---- S3: selection sub-rounds
        tm.begin(round, PICASSO_ST_SELECT);
        SelArgs sa;
        sa.cur = cur;
        sa.ekey = c->ekey;
        sa.ecost = c->ecost;
        for (int i = 0; i < 3; ++i) sa.vmin[i] = c->vmin[i];
        sa.mate = c->mate;
        sa.pcost = c->pcost();
        sa.ptie = c->ptie();
        sa.live = c->live;
        sa.live_cap = TAIL_MAX;
        sa.live_n = c->live_n;
        sa.estate = has_edge_states(B, H) ? c->estate : nullptr;
        sa.bound = std::max(H, 1);
        sa.lkey = c->key64[0];  // (between the edges' sort and line 11 these four are free)
        sa.lcost = c->val32;
        sa.lidx = c->list;
        sa.lcount = c->fslot;
        sa.list_tile = by_facets ? 3 * facet_tile(F) : LISTED_TILE;
        sa.list_tiles = by_facets ? facet_tiles(F) : 0;
        sa.fcur = by_facets ? c->fcur : nullptr;
        sa.fcost = c->ecost;
        sa.fcount = round > 0 ? c->fcount() : nullptr;
        sa.n_facets = F;
        sa.parts = facet_parts(F, nv_total);
        sa.nv = nv_total;
        sa.nf_slots = by_facets && round > 0 ? c->nf_slots[round & 1] : nullptr;
        sa.st = c->st;
        sa.mt = mt;
        sa.vbits = vbits;
        sa.host_img = c->h_pin_dev;
        sa.publish_ints = HDR_STATE_INTS + B;
        sa.host_check = c->h_pin_dev + c->h_seq_off + SEQ_CHECK_WORD;
        sa.tb = tb;
        int sel_k = 0;
        auto check_errors = [&]() -> int {
            if (!validated) {
                const int st_err = status_from_err_bits(hst->err);
                if (st_err != PICASSO_OK) {  // (the flags go back to zero for the next call, see HeaderInit)
                    prim::fill_u32_kernel<<<1, BLOCK, 0, s>>>(reinterpret_cast<u32*>(&c->st->err), 1, 0u);
                    return st_err;
                }
                validated = true;
            }
            if (hst->err & ERR_BIT_INTERNAL) {  // a kernel of the round before has refused its sizes
                prim::fill_u32_kernel<<<1, BLOCK, 0, s>>>(reinterpret_cast<u32*>(&c->st->err), 1, 0u);
                return PICASSO_ERR_INTERNAL;
            }
            return PICASSO_OK;
        };
        bool recount = true;  // the tiles' survivors are still to be counted when the budget step, if any, is done
        if (rings) {
            BudgetList* const listed = ahead_ok && ahead_budget && chip_budget ? c->budget_list() : nullptr;
            launch_ring_round(c, s, B, round, cur, nv_total, N, sa, listed);
            const HostSignal done = next_signal(c);
            PairPublish publish{0, c->st, c->mslots, c->matched, nullptr, B, round > 0 ? c->nf_slots[round & 1] : nullptr, c->h_pin_dev, HDR_STATE_INTS + B, done};
            const HostSignal nothing{nullptr, 0};
            size_t clear_ahead = 0;
            if (listed) {
                const int parts = (nv_total + BUDGET_THREADS - 1) / BUDGET_THREADS;
                publish.at = std::min(parts, BUDGET_GROUPS);
                budget_range_kernel<<<parts, BUDGET_THREADS, 0, s>>>(c->pcost(), nv_total, c->st, c->mslots, c->nrem, listed);
                budget_release_kernel<<<publish.at + 1, BUDGET_THREADS, 0, s>>>(c->pcost(), c->mate, nv_total, c->st, c->mslots, c->nrem, c->tilesum, listed, publish);
                clear_ahead = slots_clear == 0 ? facet_slots((size_t)nf_bound) : 0;  // (likely the last contraction)
                issue_contract(0, clear_ahead, false, true, nothing, true);
            } else if (ahead_ok && ahead_budget) {
                publish.at = B;
                rc = pair_budget(c, s, tb, B, c->voff[cur], nv_total, seg_bound, 0, true, true, nothing, publish);
                if (rc != PICASSO_OK) return rc;
                clear_ahead = slots_clear == 0 ? facet_slots((size_t)nf_bound) : 0;
                issue_contract(0, clear_ahead, true, true, nothing);
            } else if (ahead_ok) {
                publish.done = c->done;
                issue_contract(0, 0, false, true, nothing, true, publish);
            } else {
                publish_pairs_kernel<<<1, BLOCK, 0, s>>>(publish);
            }
            HIP_TRY(c, wait_for_signal(c, s, done));
            if ((rc = check_errors()) != PICASSO_OK) return rc;
            ahead = ahead_ok;
            recount = false;
            if (listed && hst->missed) ahead = false;  // (nothing has been contracted, nor dissolved)
            else if (!hst->wide) slots_clear = std::max(slots_clear, clear_ahead);
            if (hst->wide) {  // a row did not fit: this round and those behind it by facets
                rings = false;
                fresh = round > 0;
                facets_again(nullptr);
                c->kt.nrec = nrec_before;  // (its launches have done nothing that counts)
                renumbered = was_renumbered;
                continue;
            }
        }
        // Grid-wide sub-rounds while many edges are live (the live count falls about 3x per
        // sub-round), then the live edges are gathered and one workgroup finishes; the host
        // looks once per batch.
        int launched = 0;
        const int ne_bound = H;  // distinct edges <= half-edges
        // edges of this round: about half the half-edges at first, later the previous round's
        // count scaled by the drop in vertices (the facet bound lags one round behind)
        long long live_est = std::max(H / 2, 1);
        if (round > 0 && ne_prev > 0 && nv_prev > 0)
            live_est = std::max<long long>(1, std::min<long long>(H, (long long)ne_prev * nv_total / nv_prev * 21 / 20));
        // (by facets copies of them as well: a third more on surfaces in order, of one side or two, twice as many where the facets are in none)
        if (by_facets) live_est = live_est * 3 / 2;
        // Where many costs are equal the edges can be live for long (a flat lattice of 200 x 200 vertices: 299 sub-rounds, most of which end
        // a few hundred of 119,000 edges): a batch that leaves more than half of its edges live is followed by one of twice
        // its sub-rounds, and nothing is queued ahead behind that, which would do nothing.  That lattice to a quarter, with batches of four sub-rounds
        // each: by sorted edges 4.4 ms, by facets 79 with five workgroups to a sub-round (see listed_group_shift); so 3.8.  With line 11's
        // candidates queued behind each batch 7.6, so 3.0.
        bool slow = false, queued = false;
        int wide_before = 0;
        while (!rings) {
            // live edges fall by about 2.8x, 2.7x, 3.2x, 4x, 5x, ... per sub-round on meshes with varied costs
            static const int decay_x10[] = {28, 27, 32, 40, 50, 60};
            int wide = slow ? 2 * wide_before : 0;
            if (!slow)
                for (long long l = live_est; l > TAIL_MAX; ++wide) l = l * 10 / decay_x10[std::min(wide, 5)];
            wide = std::min<int>(wide, (int)std::max<int64_t>(1, c->opt_subround_batch));
            wide = std::max(wide, 1);  // (the last of them lists what it leaves live for the tail)
            wide_before = wide;
            queued = !slow;
            for (int j = 0; j < wide; ++j) launch_subround(c, s, sa, sel_k + j, j == wide - 1, slow, round);
            sel_k += wide;
            // the kernel behind the tail tells the host that the tail's results are in the read-back area
            const HostSignal tail_done = next_signal(c);
            sa.host_seq = tail_done.seq;
            select_tail_kernel<<<1, TAIL_THREADS, 0, s>>>(sa);
            launched += wide + 1;
            const HostSignal nothing{nullptr, 0};
            if (ahead_ok && queued) {
                if (ahead_budget) {
                    rc = pair_budget(c, s, tb, B, c->voff[cur], nv_total, seg_bound, 0, true, true, tail_done);
                    if (rc != PICASSO_OK) return rc;
                }
                issue_contract(0, 0, ahead_budget, true, ahead_budget ? nothing : tail_done);
            } else if (joiners_ahead && queued) {
                list_joiners(c, s, B, cur, vbits, ne_bound, nv_total, mt, tb, tail_done);
            } else {
                signal_kernel<<<1, 64, 0, s>>>(tail_done);
            }
            HIP_TRY(c, wait_for_signal(c, s, tail_done));  // [State][matched] are in the read-back area
            // The tail stored its counters at system scope and, after them, its own copy of the number
            // that the kernel behind it has just stored; should that copy not be there yet, what the
            // host would read is not to be trusted: wait for the stream, after which everything is.
            if (__atomic_load_n(c->h_pin + c->h_seq_off + SEQ_CHECK_WORD, __ATOMIC_ACQUIRE) != tail_done.seq) {
                HIP_TRY(c, hipStreamSynchronize(s));
                if (c->h_pin[c->h_seq_off + SEQ_CHECK_WORD] != tail_done.seq) {
                    snprintf(c->hip_err, sizeof(c->hip_err), "the selection's results did not reach host memory");
                    return PICASSO_ERR_HIP;
                }
            }
            if ((rc = check_errors()) != PICASSO_OK) return rc;
            sel_k = hst->sel_k;
            const int live = hst->live[0];
            if (live == 0) {
                ahead = ahead_ok && queued;
                break;
            }
            slow = 2ll * live > live_est;
            live_est = live;
        }
        for (int b = 0; b < B; ++b) h_matched[b] = c->h_pin[HDR_STATE_INTS + b];
        const int nf_now = round == 0 ? F : hst->nh / 3;  // (rounds by rings: of the rings' entries)
        const int ne_now = by_facets ? (int)(3ll * nf_now / 2) : hst->ne;  // (about)
        nf_bound = std::min(nf_bound, nf_now);
        if (c->n_rounds_noted < NF_ROUND_CAP) {
            c->nf_round[c->n_rounds_noted] = nf_now;
            c->nv_round[c->n_rounds_noted] = nv_total;
            c->ne_round[c->n_rounds_noted] = ne_now;
            c->way_round[c->n_rounds_noted] = way;
            ++c->n_rounds_noted;
        }
        ne_prev = ne_now;
        nv_prev = nv_total;
        if (stats && round < PICASSO_STATS_ROUNDS) {
            stats->nv[round] = nv_total;
            stats->nf[round] = nf_now;
            stats->ne[round] = hst->ne;
            stats->subrounds[round] = launched;
        }

        // ---- budget truncation (only where a mesh formed more pairs than it may remove)
        int n_sel = 0, seg_max = 0, seg_min = 0x7FFFFFFF;  // pairs; of the meshes over their budgets, the most and the least
        for (int b = 0; b < B; ++b) {
            if (h_matched[b] > nrem[b]) {
                seg_max = std::max(seg_max, h_matched[b]);
                seg_min = std::min(seg_min, h_matched[b]);
                h_matched[b] = nrem[b];
            }
            n_sel += h_matched[b];
        }
        if (seg_max > 0 && ahead && !ahead_budget) return PICASSO_ERR_HIP;  // (cannot happen: a matching pairs at most half the vertices)
        bool releases = false;
        if (seg_max > 0 && !ahead) {
            // (line 11 reads the pairs before they are counted)
            releases = !c->opt_absorb && seg_min <= c->opt_trunc_block_max;
            recount = true;
            rc = pair_budget(c, s, tb, B, c->voff[cur], nv_total, seg_max, seg_min, releases);
            if (rc != PICASSO_OK) return rc;
        }

        // ---- Alg. 2 line 11 (option): un-paired vertices join a neighbouring pair's cluster while budget is left
        int n_joined = 0;
        for (int b = 0; b < B; ++b) h_joined[b] = 0;
        bool budget_left = false;
        for (int b = 0; b < B; ++b) budget_left |= (h_matched[b] > 0 && nrem[b] > h_matched[b]);
        if (c->opt_absorb && budget_left) {
            if (!joiners_ahead || !queued) {
                const HostSignal counted = next_signal(c);
                list_joiners(c, s, B, cur, vbits, hst->ne, nv_total, mt, tb, counted);
                HIP_TRY(c, wait_for_signal(c, s, counted));
            }
            rc = run_absorb(c, s, B, cur, vbits, nv_total, tb, nrem, h_matched, h_joined);
            if (rc != PICASSO_OK) return rc;
            for (int b = 0; b < B; ++b) n_joined += h_joined[b];
        }
        tm.end();
        if (stats && round < PICASSO_STATS_ROUNDS) stats->nsel[round] = n_sel + n_joined;

        // host mirror of the outcome
        for (int b = 0; b < B; ++b) {
            if (act[b] && h_matched[b] == 0) stuck[b] = 1;
            nvb[b] -= h_matched[b] + h_joined[b];
        }
        if (n_sel == 0) {  // nothing contracted anywhere: the meshes are unchanged
            work = any_active();
            break;
        }

        // ---- S4 + S6: contraction and renumbering (already queued behind the tail, and run,
        // where `ahead` is set)
        work = any_active();
        if (!ahead) {
            const bool last = !work || (c->opt_max_rounds >= 0 && round + 1 >= c->opt_max_rounds);
            const size_t clear = last && slots_clear == 0 ? facet_slots((size_t)nf_bound) : 0;
            tm.begin(round, PICASSO_ST_CONTRACT);
            issue_contract(n_joined, clear, releases, false, HostSignal{nullptr, 0}, !recount);
            tm.end();
            slots_clear = std::max(slots_clear, clear);
        }
        nv_total -= n_sel + n_joined;
        cur ^= 1;
        ++round;
        renumbered = true;
    }

    if (!validated) {
        rc = read_header(c, s);
        if (rc != PICASSO_OK) return rc;
        const int st_err = status_from_err_bits(hst->err);
        if (st_err != PICASSO_OK) return st_err;
    }

    // ---- the end: last re-indexing, collapsed and repeated facets out (S5), results
    const size_t slots = facet_slots((size_t)nf_bound);
    if (round > 0 && slots_clear < slots)  // (rounds ended without the contraction that was to be the last)
        prim::fill_u32_kernel<<<grid_for((long long)slots), BLOCK, 0, s>>>(reinterpret_cast<u32*>(c->htab), (int)slots, ~0u);
    const bool drop = c->opt_drop_degenerated != 0;
    u32* const htab = reinterpret_cast<u32*>(c->htab);
    const int fbits = facet_index_bits(F), chunks = facet_chunks_for(F);
    // (the sorts' first buffer is free: 6 ints a facet, and at least 64; 1.1 a facet and up to 11 more are taken)
    int* const spare = reinterpret_cast<int*>(c->key64[0]);
    const size_t wave_at = ((size_t)F + 3) / 4 * 4, n_at = wave_at + prim::WAVES * (size_t)prim::compact_tiles(std::max(F, 1), chunks);
    const FacetList fl{c->fmap, c->fslot, spare, c->keep, spare + n_at, spare + wave_at};
    // (facets of rounds by facets stand at the front of their tiles once a second round has begun)
    const int* const fcount = compacted ? c->fcount() : nullptr;
    const int tile_shift = ceil_log2(facet_tile(F));
    // (null: what a vertex's label is in front of the last contraction is its number; see round_map)
    const int* const labels = by_facets && (round == 0 || (round == 1 && renumbered)) ? nullptr : c->cid;
    // rounds by rings have left the facets as they came: the labels in front of the last contraction take them there
    const int* before = rings && round > 0 ? labels : nullptr;
    int* const labels_out = !drop ? d_cluster_id : before ? c->arep : c->cid;  // (where the labels are still read: beside them)
    const int* last_map = renumbered ? round_map(c, by_facets, round - 1) : nullptr;
    const bool labels_apart = before && last_map && N >= LABELS_APART_MIN;
    if (labels_apart) {
        final_labels_kernel<<<grid_for((N + LABELS_ITEMS - 1) / LABELS_ITEMS), BLOCK, 0, s>>>(labels, last_map, labels_out, N);
        before = nullptr;
        last_map = labels_out;
    }
    tm.begin(std::max(round - 1, 0), PICASSO_ST_FACETS);
    {
        const KernelBracket timed(c, s, PICASSO_KERNEL_FACET_INSERT, round - 1, renumbered);
#define PICASSO_FINAL_FACETS(SEG)                                                                                       \
    final_facets_kernel<SEG><<<grid_for(std::max(N, F), 8192), BLOCK, 0, s>>>(                                          \
        rings ? d_facets : c->fcur, F, fcount, tile_shift, fl, c->mslots, before, last_map, c->st, cur, htab, (u32)(slots - 1), fbits, B, c->voff[cur],     \
        c->done, labels, labels_apart ? nullptr : labels_out, N, c->vrec[cur], drop ? nullptr : d_verts_out)
        switch (facet_segment(chunks)) {
            case 1: PICASSO_FINAL_FACETS(1); break;
            case 2: PICASSO_FINAL_FACETS(2); break;
            default: PICASSO_FINAL_FACETS(4);
        }
#undef PICASSO_FINAL_FACETS
    }
    if (F == 0) prim::fill_u32_kernel<<<grid_for(B), BLOCK, 0, s>>>(reinterpret_cast<u32*>(c->mesh_facets), B, 0u);
    if (F > 0) {
        const int tiles = prim::compact_tiles(F, chunks);
        int* const out = drop ? c->fcur : d_facets_out;
#define PICASSO_FACETS_OUT(CHUNKS)                                                                                      \
    count_facets_kernel<CHUNKS><<<tiles, BLOCK, 0, s>>>(fl, F, htab, fbits, c->tilesum, B, c->voff[cur], c->mslots);         \
    prim::compact_scan_sums(s, nullptr, F, c->tilesum);                                                                 \
    facets_out_kernel<CHUNKS><<<tiles, BLOCK, 0, s>>>(fl, F, c->tilesum, tiles > prim::COMPACT_MAX_SUMMED_TILES,        \
                                                      B, out, c->mslots, c->mesh_facets, &c->st->nf)
        switch (chunks) {
            case 1: PICASSO_FACETS_OUT(1); break;
            case 4: PICASSO_FACETS_OUT(4); break;
            default: PICASSO_FACETS_OUT(16);
        }
#undef PICASSO_FACETS_OUT
    }
    tm.end();
    if (drop) {
        // output vertices that no output facet refers to are dropped: mark, number the others, copy out
        int* ref = c->mate;  // (free once the rounds are over)
        const int out_grid = grid_for(std::max(std::max(N, 3 * nf_bound), 1), 8192);
        prim::fill_u32_kernel<<<grid_for(nv_total), BLOCK, 0, s>>>(reinterpret_cast<u32*>(ref), nv_total, 0u);
        mark_referenced_kernel<<<grid_for(std::max(3 * nf_bound, 1), 8192), BLOCK, 0, s>>>(c->fcur, c->st, ref);
        const RefPred rp{ref};
        const RefOut ro{c->newid};
        prim::compact(s, rp, rp, ro, &c->st->nv[cur], nv_total, c->tilesum, &c->st->nv_kept);
        drop_out_kernel<<<out_grid, BLOCK, 0, s>>>(c->vrec[cur], c->fcur, labels_out, c->st, cur, N, d_verts_out, d_facets_out,
                                                   d_cluster_id, B, c->voff[cur], ref, c->newid, c->matched);
    }
    if (stats) HIP_TRY(c, hipEventRecord(c->ev_total[1], s));
    rc = read_header(c, s);
    if (rc != PICASSO_OK) return rc;
    if (hst->err & ERR_BIT_INTERNAL) return PICASSO_ERR_INTERNAL;  // (the publishing kernel has cleared the flag)
    // the events of the measurement options are read below; all were recorded before the last kernel,
    // so waiting for the last of them returns at once and leaves every one of them readable
    if (stats) HIP_TRY(c, hipEventSynchronize(c->ev_total[1]));
    else if (c->kt.nrec > 0) HIP_TRY(c, hipEventSynchronize(c->kt_pool[c->kt.recs[c->kt.nrec - 1].e1]));
    HIP_TRY(c, hipGetLastError());
    const int* h_nf = c->h_pin + HDR_STATE_INTS + c->cap_b;

    // the bracketed kernels: event times and the algorithmic bytes of their rounds (see picasso_timed_kernel)
    for (int i = 0; i < c->kt.nrec; ++i) {
        const prim::LaunchTimer::Rec& r = c->kt.recs[i];
        const int kernel = r.tag >> 8, rd = r.tag & 0xFF;
        float ms = 0.f;
        if (kernel < PICASSO_KERNEL_COUNT && rd < c->n_rounds_noted &&
            hipEventElapsedTime(&ms, c->kt_pool[r.e0], c->kt_pool[r.e1]) == hipSuccess) {
            const double nv = c->nv_round[rd], nf = c->nf_round[rd], ne = c->ne_round[rd], H = 3.0 * nf;
            double bytes = 0.0;
            switch (kernel) {
                case PICASSO_KERNEL_SORT: bytes = 4.0 * H + 4.0 * ne; break;
                case PICASSO_KERNEL_UNIQUE_COST: {
                    const double nv_before = rd > 0 ? c->nv_round[rd - 1] : 0, nf_before = rd > 0 ? c->nf_round[rd - 1] : 0, labels = rd > 1 ? 8.0 * (double)N : 0.0;
                    switch (c->way_round[rd]) {
                        case WAY_SORTED: bytes = 17.0 * ne + 72.0 * nv; break;
                        case WAY_RINGS: bytes = rd == 0 ? 152.0 * nv : 36.0 * nv_before + 176.0 * nv + labels; break;
                        case WAY_FACETS_AGAIN: bytes = 12.0 * (double)F + 24.0 * nf + 4.0 * (double)N + 80.0 * nv; break;
                        default: bytes = rd == 0 ? 24.0 * nf + 72.0 * nv : 12.0 * nf_before + 24.0 * nf + 4.0 * nv_before + 80.0 * nv + labels;
                    }
                    break;
                }
                case PICASSO_KERNEL_SUBROUND0:
                    bytes = c->way_round[rd] == WAY_RINGS ? 16.0 * nv : c->way_round[rd] == WAY_SORTED ? 14.0 * ne + 24.0 * nv : 24.0 * nf + 32.0 * nv;
                    break;
                case PICASSO_KERNEL_FACET_INSERT:  // (the last round's is another kernel)
                    if (rd + 1 < c->n_rounds_noted) bytes = 24.0 * nf + 4.0 * nv + 8.0 * (double)N + 24.0 * (double)c->nv_round[rd + 1];
                    else bytes = (rings ? 12.0 * (double)F + 16.0 * nf : 28.0 * nf) + 4.0 * nv + 8.0 * (double)N + (drop ? 0.0 : 28.0 * (double)nv_total);
                    break;
                case PICASSO_KERNEL_SORT_INCIDENCE: bytes = 24.0 * (double)F; break;
                default: bytes = 12.0 * (double)F + 16.0 * (double)F + 76.0 * (double)N; break;  // QUADRIC_ROWS
            }
            c->kt_launches[kernel] += 1;
            c->kt_ms[kernel] += ms;
            c->kt_bytes[kernel] += bytes;
        }
    }

    int warn = PICASSO_OK;
    for (int b = 0; b < B; ++b) {
        // (with degenerated vertices dropped, the last kernels have left the meshes' counts where the pair counts were)
        h_nv_out[b] = c->opt_drop_degenerated ? c->h_pin[HDR_STATE_INTS + b] : nvb[b];
        h_nf_out[b] = h_nf[b];
        if (nvb[b] > target_nv[b] && (c->opt_max_rounds < 0 || stuck[b])) warn = PICASSO_WARN_BUDGET_UNMET;
    }
    if (stats) {
        stats->rounds = round;
        stats->nv_out = c->opt_drop_degenerated ? hst->nv_kept : hst->nv[cur];
        stats->nf_out = hst->nf;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->ev_total[0], c->ev_total[1]) == hipSuccess) stats->ms_total = ms;
        tm.collect(stats);
    }
    return warn;
}

// S0 for the entry points that give its results out: behind init_kernel, if that has found nothing wrong.
int checked_vertex_quadrics(picasso_ctx* c, hipStream_t s, const float* d_verts, int N, int F) {
    int rc = read_header(c, s);
    if (rc != PICASSO_OK) return rc;
    rc = status_from_err_bits(reinterpret_cast<State*>(c->h_pin)->err);
    if (rc != PICASSO_OK) {  // S0 will not run: take back the digit counts the validating kernel has added
        prim::fill_u32_kernel<<<prim::MSD_ZERO_WORDS / BLOCK, BLOCK, 0, s>>>(c->hist12_s0, prim::MSD_ZERO_WORDS, 0u);
        return rc;
    }
    const prim::KeySort<u64> I = incidence_sort(c, N, F);
    if (F > 0 && !sort_incidences<false>(c, s, I, d_verts, c->fcur, N, F)) return PICASSO_ERR_HIP;
    return PICASSO_OK;
}

// Filter gradients of the convolutions' backward passes: `rows` x C values summed over n_rows rows in two stages
// (conv::rows_to_partial, conv::reduce_rows_stage2_kernel).  Stage 1's workgroups leave their partial sums in the
// context's sort buffers (sort_buf).  As many workgroups as the chip holds at once (256 compute units; a workgroup takes several
// turns of rows_per_turn rows, keeping their sums in registers), fewer where there are not so many turns or the
// buffer does not hold their partials.  Where rows are dealt to several workgroups in parts that leave a wave several rows (narrow ones, that end
// within cache lines), all parts of a row are counted: those at work on the same rows then find the lines that they share in the caches, and so
// they do not with as many workgroups for each part, of which the chip takes up one part after the other.  In all | for each, us: 60 k vertices, 260
// channels, vertex2facet's backward pass 56 | 73, facet2vertex's (6 components) 98 | 123, 300: 83 | 96, 106 | 127, 132: 38 | 43, 37 | 50; 115 k, 260: 152 | 177,
// 188 | 210, 132: 67 | 83, 97 | 111.  Parts of a row to a wave share a line in sixteen, and stay as they were (115 k, 500 channels: 333 | 293).
struct FilterSplit {
    int groups, chunk;
    float* partial;
};
// CALL(kind) with the addressing that C channels and arrays of up to max_rows rows of up to `width` values take
#define PICASSO_ROW_KINDS(C, width, max_rows, CALL)               \
    do {                                                          \
        switch (pool::row_kind((C), (width), (max_rows))) {       \
            case pool::ROW_EVEN: CALL(pool::ROW_EVEN); break;     \
            case pool::ROW_TAIL: CALL(pool::ROW_TAIL); break;     \
            default: CALL(pool::ROW_ANY);                         \
        }                                                         \
    } while (0)

// Rows narrow enough for a lane each (conv.h); arrays beyond 32-bit offsets go by the kernels for any.
bool narrow_rows(int C, int width, long long max_rows) {
    return C <= conv::NARROW_C && pool::row_kind(C, width, max_rows) != pool::ROW_ANY;
}
#define PICASSO_NARROW(C, CALL)                                       \
    do {                                                              \
        switch (C) {                                                  \
            case 1: CALL(1); break;                                   \
            case 2: CALL(2); break;                                   \
            case 3: CALL(3); break;                                   \
            case 4: CALL(4); break;                                   \
            case 5: CALL(5); break;                                   \
            case 6: CALL(6); break;                                   \
            case 7: CALL(7); break;                                   \
            default: CALL(8);                                         \
        }                                                             \
    } while (0)

// m: how rows are dealt to workgroups (null: to one)
int split_filter_rows(picasso_ctx* c, int n_rows, int rows, int C, const pool::RowMap* m, int rows_per_turn, int blocks_per_cu, bool wanted,
                      FilterSplit* out) {
    // (With the first of the sorts' buffers alone 22 k facets of 200 channels and 6 components left 110
    // workgroups to facet2vertex's backward pass, 56 us; now 440, 23.)
    const size_t h = (size_t)3 * (size_t)c->max_facets;
    const size_t cap = c->sort_bytes / sizeof(float);
    const size_t per_group = (size_t)rows * C;
    if (wanted && per_group > h * sizeof(u64) / sizeof(float)) return PICASSO_ERR_WORKSPACE;
    const long long turns = ((long long)n_rows + rows_per_turn - 1) / rows_per_turn;
    const int parts = m && m->rw > 1 ? pool::row_parts(*m) : 1;
    // (five to a compute unit are as many as gain there: 60 k vertices, 260 channels, one component 88 us, with six 112)
    long long most = parts > 1 ? std::max(256 * std::min(blocks_per_cu, 5) / parts, 1) : 256 * blocks_per_cu;
    if (wanted) most = std::min<long long>(most, (long long)(cap / per_group));
    const long long per_block = (turns + most - 1) / most;  // turns of a workgroup
    long long groups = (turns + per_block - 1) / per_block;
    if (groups >= 8 && (groups + 7) / 8 * 8 <= most) groups = (groups + 7) / 8 * 8;  // (see conv::xcd_block)
    out->chunk = (int)std::min<long long>(per_block * rows_per_turn, 0x7FFFFFFFll / groups);
    out->groups = (int)groups;
    out->partial = wanted ? reinterpret_cast<float*>(c->sort_buf) : nullptr;
    return PICASSO_OK;
}
void sum_filter_rows(hipStream_t s, const FilterSplit& sp, int width, float* d_out) {
    conv::reduce_rows_stage2_kernel<<<(width + conv::REDUCE_VALUES - 1) / conv::REDUCE_VALUES, conv::REDUCE_THREADS, 0, s>>>(sp.partial, sp.groups,
                                                                                                                          width, d_out);
}

// Items 0 .. n - 1 listed per row (d_row_of[i] in [0, n_rows)), ascending: d_off [n_rows + 1], d_items [n].
int build_csr(picasso_ctx* c, hipStream_t s, const int32_t* d_row_of, int n, int n_rows, int32_t* d_off, int32_t* d_items) {
    HIP_TRY(c, hipSetDevice(c->device));
    const int ibits = item_bits(n_rows, n, n);
    const RowKeys src{d_row_of, n_rows, ibits};
    prim::KeySort<u64> S = key_sort_for(c, true, n, n, ibits + ceil_log2(n_rows));
    S.k0 = c->key64[0];
    S.k1 = c->key64[1];
    rows_of(S, n_rows, ibits, n);
    clear_wide_counts(s, S);
    int* err = &c->st->err;
    switch (count_kind(S)) {
        case COUNT_SMALL: csr_count_kernel<COUNT_SMALL><<<prim::sort_tiles(n, CSR_COUNT_ITEMS), BLOCK, 0, s>>>(src, n, digit_count(S), err); break;
        case COUNT_LARGE: csr_count_kernel<COUNT_LARGE><<<prim::sort_tiles(n, 16), BLOCK, 0, s>>>(src, n, digit_count(S), err); break;
        default: csr_count_kernel<COUNT_XL><<<prim::sort_tiles(n, CSR_COUNT_ITEMS), BLOCK, 0, s>>>(src, n, digit_count(S), err);
    }
    const RowLists out{d_off, d_items, n, n_rows, ibits, S.digit_bits};
    if (!prim::key_sort(s, S, (const prim::KeySort<u64>*)nullptr, prim::OneSource<RowKeys>{src}, out)) return PICASSO_ERR_HIP;
    const int rc = read_header(c, s);
    if (rc != PICASSO_OK) return rc;
    HIP_TRY(c, hipGetLastError());
    return (reinterpret_cast<State*>(c->h_pin)->err & ERR_BIT_BAD_INDEX) ? PICASSO_ERR_BAD_INDEX : PICASSO_OK;
}

}  // namespace

// Scratch of picasso_replace_mapping_static (the entry point for callers that cannot allocate):
// the smallest member of every cluster, then (a cache line further) the bad-index flag.  In host
// code this name is only a handle for hipGetSymbolAddress; kernels get the looked-up address.
static __device__ __align__(256) int scratch[PICASSO_STATIC_MAX_CLUSTERS + 64];

namespace {
constexpr int STATIC_MAX_DEVICES = 64;
std::atomic<int*> scratch_ptr[STATIC_MAX_DEVICES];  // per device: where its copy of `scratch` lies (null: not looked up yet)
}  // namespace

// ---------------------------------------------------------------------------
// C-ABI
// ---------------------------------------------------------------------------
extern "C" {

size_t picasso_workspace_bytes(int64_t max_verts, int64_t max_facets, int32_t max_meshes) {
    return carve(nullptr, nullptr, max_verts, max_facets, max_meshes);
}

int picasso_create(picasso_ctx** out, int device, int64_t max_verts, int64_t max_facets, int32_t max_meshes) {
    if (!out || max_verts < 1 || max_facets < 0 || max_meshes < 1) return PICASSO_ERR_INVALID_ARG;
    // 32-bit indices throughout: half-edge slots (3 per facet) and the facet hash table
    // (next power of two above 2 * facets) must fit an int
    if (max_verts > 0x7FFFFFF0ll || max_facets > (1ll << 29)) return PICASSO_ERR_INVALID_ARG;
    picasso_ctx* c = new (std::nothrow) picasso_ctx();
    if (!c) return PICASSO_ERR_HIP;
    c->device = device;
    c->max_verts = max_verts;
    c->max_facets = max_facets;
    c->max_meshes = max_meshes;
    if (hipSetDevice(device) != hipSuccess) { delete c; return PICASSO_ERR_HIP; }
    c->ws_bytes = carve(nullptr, nullptr, max_verts, max_facets, max_meshes);
    if (hipMalloc((void**)&c->ws, c->ws_bytes) != hipSuccess) { delete c; return PICASSO_ERR_HIP; }
    carve(c, c->ws, max_verts, max_facets, max_meshes);
    c->cap_b = max_meshes;
    c->h_mesh = new (std::nothrow) int[6 * (size_t)max_meshes];
    if (!c->h_mesh) {
        (void)hipFree(c->ws);
        delete c;
        return PICASSO_ERR_HIP;
    }
    c->h_up_off = (size_t)HDR_STATE_INTS + 2 * (size_t)max_meshes + 16;
    c->h_seq_off = (c->h_up_off + hdr_ints((size_t)max_meshes) + 13 + 31) / 32 * 32;
    c->h_pin_ints = c->h_seq_off + 32;
    // (mapped into the device's address space and coherent with it: kernels store there what the host reads while they run)
    if (hipHostMalloc((void**)&c->h_pin, c->h_pin_ints * sizeof(int), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipFree(c->ws);
        delete[] c->h_mesh;
        delete c;
        return PICASSO_ERR_HIP;
    }
    memset(c->h_pin, 0, c->h_pin_ints * sizeof(int));
    // the incidence sort's digit counts start at zero; every S0 leaves them at zero again.  So do the
    // header's error flags (see HeaderInit).
    if (hipMemset(c->hist12_s0, 0, sizeof(u32) * prim::MSD_ZERO_WORDS) != hipSuccess ||
        hipMemset(c->area_ext, 0, sizeof(u32) * (size_t)max_meshes * conv::EXT_SLOTS * conv::EXT_PAD) != hipSuccess ||
        hipMemset(c->hdr, 0, sizeof(int) * hdr_ints((size_t)max_meshes)) != hipSuccess) {
        (void)hipHostFree(c->h_pin);
        (void)hipFree(c->ws);
        delete[] c->h_mesh;
        delete c;
        return PICASSO_ERR_HIP;
    }
    if (hipHostGetDevicePointer((void**)&c->h_pin_dev, c->h_pin, 0) != hipSuccess) {
        (void)hipHostFree(c->h_pin);
        (void)hipFree(c->ws);
        delete[] c->h_mesh;
        delete c;
        return PICASSO_ERR_HIP;
    }
    const int nev = (int)(sizeof(c->ev) / sizeof(c->ev[0]));
    for (int i = 0; i < nev; ++i) (void)hipEventCreate(&c->ev[i]);
    (void)hipEventCreate(&c->ev_total[0]);
    (void)hipEventCreate(&c->ev_total[1]);
    for (hipEvent_t& e : c->kt_pool) (void)hipEventCreate(&e);
    *out = c;
    return PICASSO_OK;
}

void picasso_destroy(picasso_ctx* c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    const int nev = (int)(sizeof(c->ev) / sizeof(c->ev[0]));
    for (int i = 0; i < nev; ++i) (void)hipEventDestroy(c->ev[i]);
    (void)hipEventDestroy(c->ev_total[0]);
    (void)hipEventDestroy(c->ev_total[1]);
    for (hipEvent_t& e : c->kt_pool) (void)hipEventDestroy(e);
    if (c->h_pin) (void)hipHostFree(c->h_pin);
    if (c->ws) (void)hipFree(c->ws);
    delete[] c->h_mesh;
    delete c;
}

int picasso_set_option(picasso_ctx* c, int option, int64_t value) {
    if (!c) return PICASSO_ERR_INVALID_ARG;
    switch (option) {
        case PICASSO_OPT_MAX_ROUNDS: c->opt_max_rounds = value; return PICASSO_OK;
        case PICASSO_OPT_STAGE_TIMING: c->opt_stage_timing = value; return PICASSO_OK;
        case PICASSO_OPT_KERNEL_TIMING:
            if (value < 0) return PICASSO_ERR_INVALID_ARG;
            c->opt_kernel_timing = value;
            c->kt_calls = 0;
            return PICASSO_OK;
        case PICASSO_OPT_OVERLAP: c->opt_overlap = value; return PICASSO_OK;
        case PICASSO_OPT_TRUNC_BLOCK_MAX:
            if (value < 0) return PICASSO_ERR_INVALID_ARG;
            c->opt_trunc_block_max = std::min<int64_t>(value, TRUNC_BLOCK_CAP);
            return PICASSO_OK;
        case PICASSO_OPT_SHUFFLE_SEED:
            c->opt_shuffle_seed = (uint64_t)value;
            return PICASSO_OK;
        case PICASSO_OPT_HOST_POLL:
            if (value < 0 || value > 10000000) return PICASSO_ERR_INVALID_ARG;
            c->opt_poll_us = value == 1 ? 20000 : value;
            return PICASSO_OK;
        case PICASSO_OPT_LAUNCH_AHEAD:
            if (value != 0 && value != 1) return PICASSO_ERR_INVALID_ARG;
            c->opt_ahead = (int)value;
            return PICASSO_OK;
        case PICASSO_OPT_DROP_DEGENERATED:
            if (value != 0 && value != 1) return PICASSO_ERR_INVALID_ARG;
            c->opt_drop_degenerated = (int)value;
            return PICASSO_OK;
        case PICASSO_OPT_TRUNC_SELECT:
            return value == 0 || value == 1 ? PICASSO_OK : PICASSO_ERR_INVALID_ARG;  // (one way is left)
        case PICASSO_OPT_TRUNC_WIDTH:
            if (value != 0 && value != 4 && value != 8 && value != 16 && value != 32) return PICASSO_ERR_INVALID_ARG;
            c->opt_trunc_width = (int)value;
            return PICASSO_OK;
        case PICASSO_OPT_ABSORB:
            if (value != 0 && value != 1) return PICASSO_ERR_INVALID_ARG;
            c->opt_absorb = (int)value;
            return PICASSO_OK;
        case PICASSO_OPT_PLACEMENT:
            if (value != PLACE_MEAN && value != PLACE_INVERSE) return PICASSO_ERR_INVALID_ARG;
            c->opt_placement = (int)value;
            return PICASSO_OK;
        case PICASSO_OPT_RCOND_MIN_BITS: {
            if (value < 0 || value > 0xFFFFFFFFll) return PICASSO_ERR_INVALID_ARG;
            const u32 bits = (u32)value;
            float f;
            memcpy(&f, &bits, sizeof f);
            if (!(f >= 0.0f) || !std::isfinite(f)) return PICASSO_ERR_INVALID_ARG;
            c->opt_rcond_min = f;
            return PICASSO_OK;
        }
        case PICASSO_OPT_SUBROUND_BATCH:
            if (value < 1 || value > 1024) return PICASSO_ERR_INVALID_ARG;
            c->opt_subround_batch = value;
            return PICASSO_OK;
        default: return PICASSO_ERR_INVALID_ARG;
    }
}

const char* picasso_strerror(int status) {
    switch (status) {
        case PICASSO_OK: return "ok";
        case PICASSO_WARN_BUDGET_UNMET: return "warning: a mesh ran out of edges before reaching its vertex budget";
        case PICASSO_ERR_INVALID_ARG: return "invalid argument";
        case PICASSO_ERR_BAD_INDEX: return "facet index out of range";
        case PICASSO_ERR_NONFINITE: return "non-finite vertex coordinate";
        case PICASSO_ERR_WORKSPACE: return "input exceeds the capacity the context was created with";
        case PICASSO_ERR_HIP: return "HIP runtime error";
        case PICASSO_ERR_INTERNAL: return "internal error: a kernel met sizes that its launch does not take";
        default: return "unknown status";
    }
}

const char* picasso_last_hip_error(picasso_ctx* c) { return c ? c->hip_err : ""; }

int picasso_kernel_timing(picasso_ctx* c, int kernel, int reset, int64_t* launches, double* ms_total,
                          double* bytes_total) {
    if (!c || kernel < 0 || kernel >= PICASSO_KERNEL_COUNT) return PICASSO_ERR_INVALID_ARG;
    if (launches) *launches = c->kt_launches[kernel];
    if (ms_total) *ms_total = c->kt_ms[kernel];
    if (bytes_total) *bytes_total = c->kt_bytes[kernel];
    if (reset) {
        c->kt_launches[kernel] = 0;
        c->kt_ms[kernel] = 0.0;
        c->kt_bytes[kernel] = 0.0;
    }
    return PICASSO_OK;
}

int picasso_decimate_batch(picasso_ctx* c, void* stream, int32_t B, const float* d_verts, const int32_t* d_facets,
                           const int32_t* h_nv_in, const int32_t* h_nf_in, const int32_t* h_target_nv,
                           float* d_verts_out, int32_t* d_facets_out, int32_t* d_cluster_id, int32_t* h_nv_out,
                           int32_t* h_nf_out, picasso_stats* stats) {
    return decimate_impl(c, (hipStream_t)stream, B, d_verts, d_facets, h_nv_in, h_nf_in, h_target_nv, d_verts_out,
                         d_facets_out, d_cluster_id, h_nv_out, h_nf_out, stats);
}

int picasso_decimate(picasso_ctx* c, void* stream, const float* d_verts, int32_t N, const int32_t* d_facets,
                     int32_t F, int32_t target_nv, float* d_verts_out, int32_t* d_facets_out, int32_t* d_cluster_id,
                     int32_t* h_nv_out, int32_t* h_nf_out, picasso_stats* stats) {
    if (N < 1 || F < 0 || target_nv < 1) return PICASSO_ERR_INVALID_ARG;
    return decimate_impl(c, (hipStream_t)stream, 1, d_verts, d_facets, &N, &F, &target_nv, d_verts_out, d_facets_out,
                         d_cluster_id, h_nv_out, h_nf_out, stats);
}

int picasso_device_copy(void* stream, void* d_dst, const void* d_src, size_t nbytes) {
    if (!d_dst || !d_src || (nbytes & 15) || ((uintptr_t)d_dst & 15) || ((uintptr_t)d_src & 15))
        return PICASSO_ERR_INVALID_ARG;
    if (nbytes == 0) return PICASSO_OK;
    const size_t n16 = nbytes / 16;
    const int g = (int)std::min<size_t>((n16 + BLOCK - 1) / BLOCK, 256 * 32);
    copy_kernel<<<g, BLOCK, 0, (hipStream_t)stream>>>((const float4*)d_src, (float4*)d_dst, n16);
    return hipGetLastError() == hipSuccess ? PICASSO_OK : PICASSO_ERR_HIP;
}

int picasso_vertex_quadrics(picasso_ctx* c, void* stream, const float* d_verts, int32_t N, const int32_t* d_facets,
                            int32_t F, float* d_quadrics_out) {
    if (!c || !d_verts || N < 1 || F < 0 || (F > 0 && !d_facets) || !d_quadrics_out) return PICASSO_ERR_INVALID_ARG;
    if (N > c->max_verts || F > c->max_facets) return PICASSO_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    int32_t big = 0x7FFFFFFF;
    int64_t n64, f64;
    int rc = upload_header(c, s, 1, &N, &F, &big, &n64, &f64);
    if (rc != PICASSO_OK) return rc;
    rc = launch_init(c, s, d_verts, N, d_facets, F, 1, true, EDGES_NONE);
    if (rc != PICASSO_OK) return rc;
    rc = checked_vertex_quadrics(c, s, d_verts, N, F);
    if (rc != PICASSO_OK) return rc;
    export_quadrics_kernel<<<grid_for(N), BLOCK, 0, s>>>(c->vrec[0], N, d_quadrics_out);
    HIP_TRY(c, hipStreamSynchronize(s));
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_edge_costs(picasso_ctx* c, void* stream, const float* d_verts, int32_t N, const int32_t* d_facets,
                       int32_t F, int32_t* d_edges_out, float* d_cost_out, int32_t* h_ne_out) {
    if (!c || !d_verts || N < 1 || F < 0 || (F > 0 && !d_facets) || !d_edges_out || !d_cost_out || !h_ne_out)
        return PICASSO_ERR_INVALID_ARG;
    if (N > c->max_verts || F > c->max_facets) return PICASSO_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    int32_t one = 1;
    int64_t n64, f64;
    int rc = upload_header(c, s, 1, &N, &F, &one, &n64, &f64);
    if (rc != PICASSO_OK) return rc;
    rc = launch_init(c, s, d_verts, N, d_facets, F, 1, true, EDGES_SORTED);
    if (rc != PICASSO_OK) return rc;
    State* hst = reinterpret_cast<State*>(c->h_pin);
    rc = checked_vertex_quadrics(c, s, d_verts, N, F);
    if (rc != PICASSO_OK) return rc;
    const int H = 3 * F, vbits = edge_vertex_bits(N, H);
    MeshTab mt{1, c->voff[0], c->target, c->active[0], c->nrem, c->matched, c->mslots};
    const prim::KeySort<u64> E = edge_sort(c, N, F, F, 3ll * F);
    if (F > 0) {
        if (!sort_edges(c, s, E, 0)) return PICASSO_ERR_HIP;
    }
    launch_unique_cost(c, s, E, H, mt, TieBreak{0u, 0u, 0u}, c->vrec[0]);
    export_edges_kernel<<<grid_for(std::max(H, 1)), BLOCK, 0, s>>>(c->ekey, c->ecost, c->st, vbits, d_edges_out,
                                                                   d_cost_out);
    rc = read_header(c, s);
    if (rc != PICASSO_OK) return rc;
    HIP_TRY(c, hipGetLastError());
    *h_ne_out = hst->ne;
    return PICASSO_OK;
}

// ---- pooling / unpooling over cluster_id (Sec. 3, "Pooling and unpooling")

int picasso_cluster_csr(picasso_ctx* c, void* stream, const int32_t* d_cluster_id, int32_t n_in, int32_t n_out,
                        int32_t* d_offsets, int32_t* d_members) {
    if (!c || !d_cluster_id || n_in < 1 || n_out < 1 || !d_offsets || !d_members) return PICASSO_ERR_INVALID_ARG;
    if (n_in > 3 * c->max_facets || n_out > c->max_verts) return PICASSO_ERR_WORKSPACE;
    return build_csr(c, (hipStream_t)stream, d_cluster_id, n_in, n_out, d_offsets, d_members);
}

// ---- mesh convolutions, depth-wise (Sec. 4 "Mesh Convolution"; supplementary, backward propagations)

int picasso_vertex_corner_csr(picasso_ctx* c, void* stream, const int32_t* d_facets, int32_t F, int32_t N,
                              int32_t* d_offsets, int32_t* d_corners) {
    if (!c || !d_facets || F < 1 || N < 1 || !d_offsets || !d_corners) return PICASSO_ERR_INVALID_ARG;
    if (F > c->max_facets) return PICASSO_ERR_WORKSPACE;
    return build_csr(c, (hipStream_t)stream, d_facets, 3 * F, N, d_offsets, d_corners);
}

int picasso_facet_geometry(picasso_ctx* c, void* stream, const float* d_verts, int32_t N, const int32_t* d_facets,
                           int32_t F, int32_t B, const int32_t* h_nf, int32_t alpha, int32_t beta, float* d_normals,
                           float* d_areas, int32_t* d_level) {
    if (!c || !d_verts || !d_facets || N < 1 || F < 1 || B < 1 || (B > 1 && !h_nf) || alpha < 0 || beta < 1 ||
        (!d_normals && !d_areas && !d_level))
        return PICASSO_ERR_INVALID_ARG;
    if (B > c->max_meshes || (d_level && !d_areas && F > 3 * c->max_facets)) return PICASSO_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    // facet offsets of the meshes: with the launch, or (very many meshes) staged in pinned memory like the decimation's header
    conv::MeshOffsets foff{};
    foff.B = B;
    foff.far = B > conv::MESH_OFFSETS ? c->foff : nullptr;
    int* img = foff.far ? c->h_pin + c->h_up_off : foff.here;
    long long acc = 0;
    for (int b = 0; b < B; ++b) {
        img[b] = (int)acc;
        const long long nb = (B > 1) ? h_nf[b] : F;
        if (nb < 0) return PICASSO_ERR_INVALID_ARG;
        acc += nb;
    }
    img[B] = (int)acc;
    if (acc != F) return PICASSO_ERR_INVALID_ARG;
    if (foff.far) HIP_TRY(c, hipMemcpyAsync(c->foff, img, sizeof(int) * (B + 1), hipMemcpyHostToDevice, s));
    const int geo_grid = (F + pool::BLOCK * conv::GEO_ITEMS - 1) / (pool::BLOCK * conv::GEO_ITEMS);
    float* areas = d_areas ? d_areas : reinterpret_cast<float*>(c->ecost);  // scratch when only levels are wanted
    conv::facet_geometry_kernel<<<geo_grid, pool::BLOCK, 0, s>>>(d_verts, N, d_facets, F, foff, d_normals,
                                                                         (d_areas || d_level) ? areas : nullptr,
                                                                         d_level ? c->area_ext : nullptr, &c->st->err);
    if (d_level)
        conv::facet_level_kernel<<<geo_grid, pool::BLOCK, 0, s>>>(areas, F, foff, c->area_ext, alpha, beta, d_level);
    int rc = read_header(c, s, c->area_ext, d_level ? B * conv::EXT_SLOTS : 0);
    if (rc != PICASSO_OK) return rc;
    HIP_TRY(c, hipGetLastError());
    return (reinterpret_cast<State*>(c->h_pin)->err & 1) ? PICASSO_ERR_BAD_INDEX : PICASSO_OK;
}

int picasso_fuzzy_coefficients(picasso_ctx* c, void* stream, const float* d_normals, int32_t F, const float* d_mu,
                               const float* d_inv_var, int32_t T, float* d_pi) {
    if (!c || !d_normals || F < 1 || !d_mu || !d_inv_var || T < 1 || !d_pi) return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    if (T <= conv::FUZZY_LDS_T)
        conv::fuzzy_kernel<true><<<pool::grid_for(F), pool::BLOCK, sizeof(float) * pool::BLOCK * T, s>>>(d_normals, F, d_mu, d_inv_var, T, d_pi);
    else
        conv::fuzzy_kernel<false><<<pool::grid_for(F), pool::BLOCK, 0, s>>>(d_normals, F, d_mu, d_inv_var, T, d_pi);
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_v2f_forward(picasso_ctx* c, void* stream, const float* d_x, int32_t N, int32_t C, const int32_t* d_facets,
                        int32_t F, const int32_t* d_level, const float* d_w, float* d_y) {
    if (!c || !d_x || N < 1 || C < 1 || !d_facets || F < 1 || !d_w || !d_y) return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const pool::RowMap m = pool::row_map(C, false, C > 128 || pool::beyond_cache(C, (long long)N + F));  // (see there)
    const int per_wave = conv::facets_per_wave(m, F), per_block = per_wave * (pool::BLOCK / 64);
    const dim3 grid(prim::xcd_grid((F + per_block - 1) / per_block), pool::row_parts(m));
#define PICASSO_CALL(K) \
    conv::v2f_forward_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_x, N, C, d_facets, F, d_level, d_w, d_y, per_wave, m)
    PICASSO_ROW_KINDS(C, C, std::max(N, F), PICASSO_CALL);
#undef PICASSO_CALL
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_v2f_backward(picasso_ctx* c, void* stream, const float* d_gy, const float* d_x, int32_t N, int32_t C,
                         const int32_t* d_facets, int32_t F, const int32_t* d_level, const float* d_w,
                         const int32_t* d_offsets, const int32_t* d_corners, float* d_gx, float* d_gw) {
    if (!c || !d_gy || !d_x || N < 1 || C < 1 || !d_facets || F < 1 || !d_w || !d_offsets || !d_corners ||
        (!d_gx && !d_gw))
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    FilterSplit sp;
    if (narrow_rows(C, C, std::max(N, F))) {
        const int rc = split_filter_rows(c, N, 3, C, nullptr, pool::BLOCK, 5, d_gw != nullptr, &sp);
        if (rc != PICASSO_OK) return rc;
#define PICASSO_CALL(CH) \
    conv::v2f_backward_narrow_kernel<CH><<<sp.groups, pool::BLOCK, 0, s>>>(d_gy, d_x, d_level, d_w, d_offsets, d_corners, N, 3 * F, sp.chunk, d_gx, sp.partial)
        PICASSO_NARROW(C, PICASSO_CALL);
#undef PICASSO_CALL
        if (d_gw) sum_filter_rows(s, sp, 3 * C, d_gw);
        HIP_TRY(c, hipGetLastError());
        return PICASSO_OK;
    }
    const conv::WalkMap m = conv::walk_map(C, N, (double)(3ll * F) / N, C > 128 || pool::beyond_cache(C, (long long)N + F), true);  // (see row_map)
    const int rc = split_filter_rows(c, N, 3, C, &m.row, m.per_wave * (pool::BLOCK / 64), 5, d_gw != nullptr, &sp);
    if (rc != PICASSO_OK) return rc;
    const dim3 grid(sp.groups, pool::row_parts(m.row));
#define PICASSO_CALL(K)                                                                                                     \
    conv::v2f_backward_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_gy, d_x, C, d_level, d_w, d_offsets, d_corners, N, 3 * F,     \
                                                              sp.chunk, d_gx, sp.partial, m)
    PICASSO_ROW_KINDS(C, C, std::max(N, F), PICASSO_CALL);
#undef PICASSO_CALL
    if (d_gw) sum_filter_rows(s, sp, 3 * C, d_gw);
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_f2f_forward(picasso_ctx* c, void* stream, const float* d_tex, const float* d_bary, const int32_t* d_poff,
                        int32_t F, int32_t P, int32_t C, const float* d_w, float* d_y) {
    if (!c || !d_tex || !d_bary || !d_poff || F < 1 || P < 0 || C < 1 || !d_w || !d_y) return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const conv::WalkMap m = conv::walk_map(C, F, (double)P / F);
    const int per_block = m.per_wave * (pool::BLOCK / 64);
    const dim3 grid(prim::xcd_grid((F + per_block - 1) / per_block), pool::row_parts(m.row));
#define PICASSO_CALL(K) \
    conv::f2f_forward_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_tex, d_bary, d_poff, F, P, C, d_w, d_y, m)
    PICASSO_ROW_KINDS(C, C, std::max(F, P), PICASSO_CALL);
#undef PICASSO_CALL
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_f2f_backward(picasso_ctx* c, void* stream, const float* d_gy, const float* d_tex, const float* d_bary,
                         const int32_t* d_poff, int32_t F, int32_t P, int32_t C, const float* d_w, float* d_gtex,
                         float* d_gw) {
    if (!c || !d_gy || !d_tex || !d_bary || !d_poff || F < 1 || P < 0 || C < 1 || !d_w || (!d_gtex && !d_gw))
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const pool::RowMap m = pool::row_map(C);
    FilterSplit sp;
    const int per_wave = (int)std::max<long long>(1, std::min<long long>(conv::WALK_WAVE_ROWS / 2, F / 4096));
    const int rc = split_filter_rows(c, F, 3, C, &m, per_wave * (pool::BLOCK / 64), 5, d_gw != nullptr, &sp);
    if (rc != PICASSO_OK) return rc;
    const dim3 grid(sp.groups, pool::row_parts(m));
#define PICASSO_CALL(K)                                                                                                     \
    conv::f2f_backward_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_gy, d_tex, d_bary, d_poff, F, P, C, d_w, sp.chunk, per_wave,    \
                                                              d_gtex, sp.partial, m)
    PICASSO_ROW_KINDS(C, C, std::max(F, P), PICASSO_CALL);
#undef PICASSO_CALL
    if (d_gw) sum_filter_rows(s, sp, 3 * C, d_gw);
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_f2f_clear_unowned(picasso_ctx* c, void* stream, const int32_t* d_poff, int32_t F, int32_t P, int32_t C,
                              float* d_gtex) {
    if (!c || !d_poff || F < 1 || P < 0 || C < 1 || !d_gtex) return PICASSO_ERR_INVALID_ARG;
    HIP_TRY(c, hipSetDevice(c->device));
    conv::f2f_clear_kernel<<<256, pool::BLOCK, 0, (hipStream_t)stream>>>(d_poff, F, P, C, d_gtex);
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_f2v_forward(picasso_ctx* c, void* stream, const float* d_y, int32_t F, int32_t C, const float* d_pi,
                        int32_t T, const float* d_w, const int32_t* d_offsets, const int32_t* d_corners, int32_t N,
                        float* d_x) {
    if (!c || !d_y || F < 1 || C < 1 || !d_pi || T < 1 || !d_w || !d_offsets || !d_corners || N < 1 || !d_x)
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    if (T <= 16 && narrow_rows(C, std::max(C, T), std::max(N, F))) {
        const int grid = prim::xcd_grid((N + pool::BLOCK - 1) / pool::BLOCK);
#define PICASSO_F2V(CH, NP) \
    conv::f2v_forward_narrow_kernel<CH, NP><<<grid, pool::BLOCK, 0, s>>>(d_y, d_pi, T, d_w, d_offsets, d_corners, N, 3 * F, d_x)
#define PICASSO_CALL(CH)                      \
    if (T <= 4) PICASSO_F2V(CH, 1);           \
    else if (T <= 8) PICASSO_F2V(CH, 2);      \
    else if (T <= 12) PICASSO_F2V(CH, 3);     \
    else PICASSO_F2V(CH, 4)
        PICASSO_NARROW(C, PICASSO_CALL);
#undef PICASSO_CALL
#undef PICASSO_F2V
        HIP_TRY(c, hipGetLastError());
        return PICASSO_OK;
    }
    const conv::WalkMap m = conv::walk_map(C, N, (double)(3ll * F) / N, true, true);  // (see row_map)
    const int per_block = (T <= 16 ? m.per_wave : m.row.rw) * (pool::BLOCK / 64);
    const dim3 grid(prim::xcd_grid((N + per_block - 1) / per_block), pool::row_parts(m.row));
#define PICASSO_F2V(NP, K) \
    conv::f2v_forward_kernel<NP, K><<<grid, pool::BLOCK, 0, s>>>(d_y, C, d_pi, T, d_w, d_offsets, d_corners, N, 3 * F, d_x, m)
#define PICASSO_CALL(K)                      \
    if (T <= 4) PICASSO_F2V(1, K);           \
    else if (T <= 8) PICASSO_F2V(2, K);      \
    else if (T <= 12) PICASSO_F2V(3, K);     \
    else if (T <= 16) PICASSO_F2V(4, K);     \
    else conv::f2v_forward_many_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_y, C, d_pi, T, d_w, d_offsets, d_corners, N, 3 * F, d_x, m.row)
    PICASSO_ROW_KINDS(C, std::max(C, T), std::max(N, F), PICASSO_CALL);
#undef PICASSO_CALL
#undef PICASSO_F2V
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_f2v_backward(picasso_ctx* c, void* stream, const float* d_gx, const float* d_y, int32_t F, int32_t C,
                         const float* d_pi, int32_t T, const float* d_w, const int32_t* d_facets,
                         const int32_t* d_offsets, int32_t N, float* d_gy, float* d_gw, float* d_gpi) {
    if (!c || !d_gx || !d_y || F < 1 || C < 1 || !d_pi || T < 1 || !d_w || !d_facets || !d_offsets || N < 1 ||
        (!d_gy && !d_gw && !d_gpi))
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const int np = (T + 3) / 4;
    if (np <= 4 && 4 * np * C <= conv::NARROW_VALUES && narrow_rows(C, std::max(C, T), std::max(N, F))) {
        FilterSplit sp;
        const int rc = split_filter_rows(c, F, T, C, nullptr, pool::BLOCK, 5, d_gw != nullptr, &sp);
        if (rc != PICASSO_OK) return rc;
#define PICASSO_F2V_BACK(CH, NP)                                                                                        \
    do {                                                                                                                \
        if constexpr (4 * (NP) * (CH) <= conv::NARROW_VALUES)                                                           \
            conv::f2v_backward_narrow_kernel<CH, NP><<<sp.groups, pool::BLOCK, 0, s>>>(                                 \
                d_gx, d_y, d_pi, T, d_w, d_facets, F, d_offsets, N, sp.chunk, d_gy, sp.partial, d_gpi);                 \
    } while (0)
#define PICASSO_CALL(CH)                        \
    if (np == 1) PICASSO_F2V_BACK(CH, 1);       \
    else if (np == 2) PICASSO_F2V_BACK(CH, 2);  \
    else if (np == 3) PICASSO_F2V_BACK(CH, 3);  \
    else PICASSO_F2V_BACK(CH, 4)
        PICASSO_NARROW(C, PICASSO_CALL);
#undef PICASSO_CALL
#undef PICASSO_F2V_BACK
        if (d_gw) sum_filter_rows(s, sp, T * C, d_gw);
        HIP_TRY(c, hipGetLastError());
        return PICASSO_OK;
    }
    // one pass per 16 filter rows; gpi with it where a row's lanes fit a wave, else by a kernel of its own
    const bool gpi_fused = d_gpi && C <= 256;
    const pool::RowMap m = pool::row_map(C, gpi_fused, C > 128 && pool::beyond_cache(C, (long long)N + F));
    const int per_wave = conv::facets_per_wave(m, F);
    if (d_gy || d_gw || gpi_fused) {
        for (int t0 = 0; t0 < T; t0 += 16) {
            float* gy = t0 == 0 ? d_gy : nullptr;
            if (!gy && !d_gw && !gpi_fused) break;
            const int rows = std::min(16, T - t0);
            FilterSplit sp;
            const int rc = split_filter_rows(c, F, rows, C, &m, per_wave * (pool::BLOCK / 64), rows <= 4 ? 6 : (rows <= 12 ? 4 : 3), d_gw != nullptr, &sp);
            if (rc != PICASSO_OK) return rc;
            const dim3 grid(sp.groups, pool::row_parts(m));
#define PICASSO_F2V_BACK_GPI(NP, K, GPI)                                                                              \
    conv::f2v_backward_kernel<NP, K, GPI><<<grid, pool::BLOCK, 0, s>>>(                                               \
        d_gx, d_y, C, d_pi, T, t0, rows, d_w, d_facets, F, d_offsets, N, sp.chunk, per_wave, gy, sp.partial, d_gpi, m)
#define PICASSO_F2V_BACK(NP, K)                                                                                       \
    do {                                                                                                              \
        /* (components together where GPI_POW2 is the faster: conv.h) */                                               \
        if (gpi_fused && (m.Q & (m.Q - 1)) == 0) PICASSO_F2V_BACK_GPI(NP, K, NP <= 3 ? conv::GPI_POW2 : conv::GPI_ANY); \
        else if (gpi_fused) PICASSO_F2V_BACK_GPI(NP, K, conv::GPI_ANY);                                               \
        else PICASSO_F2V_BACK_GPI(NP, K, conv::GPI_NONE);                                                             \
    } while (0)
#define PICASSO_CALL(K)                         \
    if (rows <= 4) PICASSO_F2V_BACK(1, K);      \
    else if (rows <= 8) PICASSO_F2V_BACK(2, K); \
    else if (rows <= 12) PICASSO_F2V_BACK(3, K);\
    else PICASSO_F2V_BACK(4, K)
            PICASSO_ROW_KINDS(C, std::max(C, T), std::max(N, F), PICASSO_CALL);
#undef PICASSO_CALL
#undef PICASSO_F2V_BACK
#undef PICASSO_F2V_BACK_GPI
            if (d_gw) sum_filter_rows(s, sp, rows * C, d_gw + (size_t)t0 * C);
        }
    }
    if (d_gpi && !gpi_fused) {
        const int grid = (F + pool::BLOCK / 64 - 1) / (pool::BLOCK / 64);
#define PICASSO_CALL(K) \
    conv::f2v_backward_pi_kernel<K><<<grid, pool::BLOCK, 0, s>>>(d_gx, d_y, C, T, d_w, d_facets, F, d_offsets, N, d_gpi)
        PICASSO_ROW_KINDS(C, std::max(C, T), std::max(N, F), PICASSO_CALL);
#undef PICASSO_CALL
    }
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_replace_mapping(picasso_ctx* c, void* stream, const int32_t* d_cluster_id, int32_t n_in, int32_t n_out,
                            int32_t* d_replace, int32_t* d_mapping) {
    if (!c || !d_cluster_id || n_in < 1 || n_out < 0 || !d_replace || !d_mapping) return PICASSO_ERR_INVALID_ARG;
    if (n_out > c->max_verts) return PICASSO_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    prim::fill_u32_kernel<<<1, BLOCK, 0, s>>>(reinterpret_cast<u32*>(&c->st->err), 1, 0u);
    if (n_out > 0)
        prim::fill_u32_kernel<<<grid_for(n_out), BLOCK, 0, s>>>(reinterpret_cast<u32*>(c->newid), n_out, 0x7FFFFFFFu);
    pool::cluster_first_kernel<<<pool::grid_for(n_in), pool::BLOCK, 0, s>>>(d_cluster_id, n_in, n_out, c->newid,
                                                                            &c->st->err);
    pool::replace_mapping_kernel<<<pool::grid_for(n_in), pool::BLOCK, 0, s>>>(d_cluster_id, n_in, n_out, c->newid,
                                                                              d_replace, d_mapping);
    int rc = read_header(c, s);
    if (rc != PICASSO_OK) return rc;
    HIP_TRY(c, hipGetLastError());
    return (reinterpret_cast<State*>(c->h_pin)->err & 1) ? PICASSO_ERR_BAD_INDEX : PICASSO_OK;
}

int picasso_replace_mapping_static(int device, void* stream, const int32_t* d_cluster_id, int32_t n_in, int32_t n_out,
                                   int32_t* d_replace, int32_t* d_mapping, int32_t* d_status) {
    if (device < 0 || device >= STATIC_MAX_DEVICES || !d_cluster_id || n_in < 1 || n_out < 0 || !d_replace ||
        !d_mapping || !d_status)
        return PICASSO_ERR_INVALID_ARG;
    if (n_out > PICASSO_STATIC_MAX_CLUSTERS) return PICASSO_ERR_WORKSPACE;
    if (hipSetDevice(device) != hipSuccess) return PICASSO_ERR_HIP;
    // every device holds its own copy of the array at its own address: looked up once per device, with
    // that device current; from here on only that address is used, never the array's name
    int* ptr = scratch_ptr[device].load(std::memory_order_acquire);
    if (!ptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PICASSO_ERR_HIP;
        ptr = static_cast<int*>(p);
        scratch_ptr[device].store(ptr, std::memory_order_release);
    }
    hipStream_t s = (hipStream_t)stream;
    int* first = ptr;
    int* flag = ptr + PICASSO_STATIC_MAX_CLUSTERS;
    // the array keeps the last call's contents: what this call reads starts from its own fill
    // (a kernel, not a memset command, so that the call can be recorded into a graph)
    pool::static_begin_kernel<<<pool::grid_for(n_out), pool::BLOCK, 0, s>>>(first, n_out, flag);
    pool::cluster_first_kernel<<<pool::grid_for(n_in), pool::BLOCK, 0, s>>>(d_cluster_id, n_in, n_out, first, flag);
    pool::replace_mapping_status_kernel<<<pool::grid_for(n_in), pool::BLOCK, 0, s>>>(
        d_cluster_id, n_in, n_out, first, flag, d_replace, d_mapping, d_status, PICASSO_OK, PICASSO_ERR_BAD_INDEX);
    return hipGetLastError() == hipSuccess ? PICASSO_OK : PICASSO_ERR_HIP;
}

int picasso_pool_forward(picasso_ctx* c, void* stream, int mode, const float* d_x, int32_t n_in, int32_t C,
                         const int32_t* d_offsets, const int32_t* d_members, int32_t n_out, const float* d_weight,
                         float* d_y, int32_t* d_argmax) {
    if (!c || !d_x || !d_offsets || !d_members || !d_y || n_in < 1 || n_out < 1 || C < 1 || mode < 0 || mode > 3 ||
        (mode == pool::WEIGHTED && !d_weight))
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
#define PICASSO_CALL(K) pool::launch_pool_forward<K>(s, mode, d_x, C, d_offsets, d_members, n_out, d_weight, d_y, d_argmax)
    PICASSO_ROW_KINDS(C, C, std::max(n_in, n_out), PICASSO_CALL);
#undef PICASSO_CALL
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_pool_backward(picasso_ctx* c, void* stream, int mode, const float* d_gy, int32_t n_in, int32_t C,
                          const int32_t* d_cluster_id, const int32_t* d_offsets, const int32_t* d_members,
                          int32_t n_out, const float* d_weight, const int32_t* d_argmax, float* d_gx) {
    if (!c || !d_gy || !d_cluster_id || !d_offsets || !d_members || !d_gx || n_in < 1 || n_out < 1 || C < 1 ||
        mode < 0 || mode > 3 || (mode == pool::WEIGHTED && !d_weight) || (mode == pool::MAX && !d_argmax))
        return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
#define PICASSO_CALL(K) \
    pool::launch_pool_backward<K>(s, mode, d_gy, n_in, C, d_cluster_id, d_offsets, d_members, d_weight, d_argmax, d_gx)
    PICASSO_ROW_KINDS(C, C, std::max(n_in, n_out), PICASSO_CALL);
#undef PICASSO_CALL
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_unpool_forward(picasso_ctx* c, void* stream, const float* d_y, int32_t n_in, int32_t C,
                           const int32_t* d_cluster_id, float* d_x) {
    if (!c || !d_y || !d_cluster_id || !d_x || n_in < 1 || C < 1) return PICASSO_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const pool::RowMap m = pool::row_map(C, false, true);
#define PICASSO_CALL(K) \
    pool::unpool_forward_kernel<K><<<pool::row_grid(m, n_in), pool::BLOCK, 0, s>>>(d_y, n_in, C, d_cluster_id, d_x, m)
    PICASSO_ROW_KINDS(C, C, n_in, PICASSO_CALL);
#undef PICASSO_CALL
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_unpool_backward(picasso_ctx* c, void* stream, const float* d_gx, int32_t n_in, int32_t C,
                            const int32_t* d_offsets, const int32_t* d_members, int32_t n_out, float* d_gy) {
    return picasso_pool_forward(c, stream, pool::SUM, d_gx, n_in, C, d_offsets, d_members, n_out, nullptr, d_gy, nullptr);
}

int picasso_bucket_sort(picasso_ctx* c, void* stream, int key_bytes, void* d_keys, uint32_t* d_vals, int64_t n,
                        int key_bits) {
    if (!c || !d_keys || n < 0 || (key_bytes != 4 && key_bytes != 8) || key_bits < 1 || key_bits > 8 * key_bytes)
        return PICASSO_ERR_INVALID_ARG;
    if (n > 3 * c->max_facets || n > prim::BUCKET_SORT_LARGE_MAX_KEYS) return PICASSO_ERR_WORKSPACE;
    if (n == 0) return PICASSO_OK;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    int rc;
    c->hist_dirty = true;
    auto large_keys = [&](auto* k0, auto* k1) -> int {
        prim::KeySort<std::remove_pointer_t<decltype(k0)>> S;
        S.k0 = k0;
        S.k1 = k1;
        S.n = (int)n;
        S.key_bits = key_bits;
        S.digit_bits = prim::BUCKET_LARGE_MSD_BITS;
        S.buckets = 1 << S.digit_bits;
        prim::use_arrays(S, c->hist12);
        return prim::key_sort_array(s, S) ? 0 : -1;
    };
    const bool large = n > prim::BUCKET_SORT_MAX_KEYS;
    if (large && key_bits <= prim::BUCKET_LARGE_MSD_BITS) return PICASSO_ERR_INVALID_ARG;
    if (key_bytes == 8) {
        u64* k1 = c->key64[1];
        if (large)
            rc = d_vals ? prim::bucket_sort_large<u64>(s, (u64*)d_keys, k1, d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc, c->hist12)
                        : large_keys((u64*)d_keys, k1);
        else
            rc = d_vals ? prim::bucket_sort<u64, true>(s, (u64*)d_keys, k1, d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc)
                        : prim::bucket_sort<u64, false>(s, (u64*)d_keys, k1, nullptr, nullptr, nullptr, (int)n, key_bits, c->sort_sc);
        if (rc == 1) HIP_TRY(c, hipMemcpyAsync(d_keys, k1, sizeof(u64) * n, hipMemcpyDeviceToDevice, s));
    } else {
        u32* k1 = reinterpret_cast<u32*>(c->key64[1]);
        if (large)
            rc = d_vals ? prim::bucket_sort_large<u32>(s, (u32*)d_keys, k1, d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc, c->hist12)
                        : large_keys((u32*)d_keys, k1);
        else
            rc = d_vals ? prim::bucket_sort<u32, true>(s, (u32*)d_keys, k1, d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc)
                        : prim::bucket_sort<u32, false>(s, (u32*)d_keys, k1, nullptr, nullptr, nullptr, (int)n, key_bits, c->sort_sc);
        if (rc == 1) HIP_TRY(c, hipMemcpyAsync(d_keys, k1, sizeof(u32) * n, hipMemcpyDeviceToDevice, s));
    }
    if (rc < 0) return PICASSO_ERR_HIP;
    if (rc == 1 && d_vals) HIP_TRY(c, hipMemcpyAsync(d_vals, c->val32, sizeof(u32) * n, hipMemcpyDeviceToDevice, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

int picasso_radix_sort(picasso_ctx* c, void* stream, int key_bytes, void* d_keys, uint32_t* d_vals, int64_t n,
                       int key_bits) {
    if (!c || !d_keys || n < 0 || (key_bytes != 4 && key_bytes != 8) || key_bits < 1 || key_bits > 8 * key_bytes)
        return PICASSO_ERR_INVALID_ARG;
    if (n > 3 * c->max_facets) return PICASSO_ERR_WORKSPACE;
    if (n == 0) return PICASSO_OK;
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    int where;
    if (key_bytes == 8) {
        u64* k = (u64*)d_keys;
        where = d_vals ? prim::radix_sort<u64, true>(s, k, c->key64[1], d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc)
                       : prim::radix_sort<u64, false>(s, k, c->key64[1], nullptr, nullptr, nullptr, (int)n, key_bits, c->sort_sc);
        if (where < 0) return PICASSO_ERR_HIP;
        if (where == 1) {
            HIP_TRY(c, hipMemcpyAsync(k, c->key64[1], sizeof(u64) * n, hipMemcpyDeviceToDevice, s));
            if (d_vals) HIP_TRY(c, hipMemcpyAsync(d_vals, c->val32, sizeof(u32) * n, hipMemcpyDeviceToDevice, s));
        }
    } else {
        u32* k = (u32*)d_keys;
        u32* k1 = reinterpret_cast<u32*>(c->key64[1]);
        where = d_vals ? prim::radix_sort<u32, true>(s, k, k1, d_vals, c->val32, nullptr, (int)n, key_bits, c->sort_sc)
                       : prim::radix_sort<u32, false>(s, k, k1, nullptr, nullptr, nullptr, (int)n, key_bits, c->sort_sc);
        if (where < 0) return PICASSO_ERR_HIP;
        if (where == 1) {
            HIP_TRY(c, hipMemcpyAsync(k, k1, sizeof(u32) * n, hipMemcpyDeviceToDevice, s));
            if (d_vals) HIP_TRY(c, hipMemcpyAsync(d_vals, c->val32, sizeof(u32) * n, hipMemcpyDeviceToDevice, s));
        }
    }
    HIP_TRY(c, hipStreamSynchronize(s));
    HIP_TRY(c, hipGetLastError());
    return PICASSO_OK;
}

}  // extern "C"
