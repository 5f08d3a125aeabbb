// rb_update_sample in ONE launch for shapes that rb_step_small_kernel does not serve: any candidate and representative
// count, any selection and replacement strategy, any storage form, up to ONE_CLASSES classes, where step_form finds it faster.
// Included by rb.hip only, after rb_kernels_small.h (whose wavefront selection it uses).
#pragma once

#include "rb_device.h"
#include "rb_kernels_small.h"

namespace {

constexpr int ONE_TPB = 512;                        // threads of a workgroup: one workgroup per compute unit
constexpr int ONE_NWAVE = ONE_TPB / WAVE;
constexpr int ONE_PER = RB_MAX_BATCH / ONE_TPB;     // mini-batch positions, candidates and representatives per thread at most
constexpr int ONE_CLASSES = 10240;                  // most classes: their fill counts are kept in LDS
constexpr int ONE_FILL_PER = (ONE_CLASSES / 4 + ONE_TPB - 1) / ONE_TPB;    // vectors of four fill counts per thread
constexpr int ONE_PACE = 64;                        // stores of a tile go out in one burst (paced ones measured 0.4 us slower)
constexpr int ONE_PLANNED = 64;                     // rows a workgroup plans at a time
constexpr int ONE_LIST = 4 * WAVE;                  // the candidate list and the draws are read this many at a time
constexpr int ONE_PARKED = 2 * ONE_TPB;             // mini-batches up to this size have all their labels read into LDS
constexpr int ONE_POS_BITS = 12;                    // candidate list: class << ONE_POS_BITS | mini-batch position
constexpr uint32_t ONE_NO_CLASS = 0xFFFFFFFFu;      // ... of a candidate whose label is outside [0, K), and behind the list's end
static_assert(RB_MAX_BATCH <= 1 << ONE_POS_BITS && ONE_CLASSES < 1 << (31 - ONE_POS_BITS), "class and position in one word");
constexpr int ONE_WORDS = RB_MAX_BATCH / 32;        // words of a bitmap over the mini-batch's positions

struct OneArgs {
    UpdateArgs u;                       // (u.tpr, u.tile_vec, u.tile_rem: tiles of the candidates' rows)
    vec16* out_x;
    int64_t* out_y;
    int32_t r;
    int32_t tpr, tile_vec, tile_rem;    // tiles of the representatives' rows
    int32_t share, cshare;              // work items (row, tile) per workgroup; cshare: of the candidates, 0: as many as make the shares equal
    int32_t nwg;                        // workgroups of the launch
    const int32_t* chunk_old;           // samples per chunk of classes before the step
    int32_t first_cand;                 // workgroups 0 ... first_cand - 1 move representatives (and keep the books), the others candidates
};

// The arguments of rb_step_one_kernel as they lie in memory
struct OneKernelArgs {
    const int64_t* batch_y;
    const int32_t* fill_old;
    const int32_t* chunk_old;
    Seed sd;
    uint32_t b_c, r_nchunks;
    int32_t first_cand;
    OneArgs rest;
};

// LDS words in front of the arrays whose size depends on the shape (see rb_step_one_kernel)
constexpr int ONE_CHUNKS = WAVE;                    // chunk sums: one per lane
static_assert(ONE_CLASSES <= ONE_CHUNKS * CH, "a wavefront holds all chunk sums");
constexpr size_t ONE_MATE_WORDS = ONE_NWAVE * (WAVE / 2 + ONE_WORDS + ONE_WORDS / 2);
__host__ __device__ inline int one_padded(int n) { return (n + ONE_LIST - 1) / ONE_LIST * ONE_LIST; }
inline size_t one_lds_bytes(int b, int cap, int r, int nchunks)
{
    return 4 * ((size_t)nchunks * (CH + CH / 32) + ONE_CHUNKS + ONE_MATE_WORDS + 2 * (size_t)((b + 3) & ~3) + one_padded(cap) + one_padded(cap > r ? cap : r)) +
           ((size_t)cap * 2 + 3) / 4 * 4;
}

// Lane `lane` looks at four consecutive words of every ONE_LIST of the candidate list or the draws (one LDS access): number `bit` of
// its words is this one of the list.
__device__ __forceinline__ int one_entry(int bit, int lane) { return (bit >> 2) * ONE_LIST + 4 * lane + (bit & 3); }

// The candidates of one class in a step, as one wavefront collects them from the workgroup's candidate list.
struct Mates {
    uint64_t hit;         // bit i: candidate one_entry(i, lane) is one of them
    int mine, before;     // how many of them the lane holds, and the lanes before it
    int total;
    int rank;             // ... of them earlier in the mini-batch than position p
};

__device__ __forceinline__ Mates one_mates(const uint32_t* s_kx, int m, int32_t k, int p)
{
    const int lane = threadIdx.x & (WAVE - 1);
    Mates t;
    t.hit = 0;
    int earlier = 0;
    const uint32_t lo = (uint32_t)k << ONE_POS_BITS, mid = lo | (uint32_t)p, hi = lo | (RB_MAX_BATCH - 1);
#pragma unroll 4
    for (int m0 = 0; m0 < m; m0 += ONE_LIST) {
        const uint4 v = *reinterpret_cast<const uint4*>(s_kx + m0 + 4 * lane);
        const uint32_t mate = (v.x >= lo && v.x <= hi ? 1u : 0u) | (v.y >= lo && v.y <= hi ? 2u : 0u) | (v.z >= lo && v.z <= hi ? 4u : 0u) | (v.w >= lo && v.w <= hi ? 8u : 0u);
        t.hit |= (uint64_t)mate << (m0 / WAVE);
        earlier += (v.x >= lo && v.x < mid) + (v.y >= lo && v.y < mid) + (v.z >= lo && v.z < mid) + (v.w >= lo && v.w < mid);
    }
    t.mine = __popcll(t.hit);
    const int incl = wave_scan_incl(t.mine | (earlier << 16));      // both sums are <= 4096
    t.before = (incl & 0xFFFF) - t.mine;
    t.total = lane_read(incl, WAVE - 1) & 0xFFFF;
    t.rank = lane_read(incl, WAVE - 1) >> 16;
    return t;
}

// Up to WAVE class-mates, one lane each: position (-1: lane has none) and rank.
__device__ __forceinline__ void one_mate_lanes(const Mates& t, const uint32_t* s_kx, uint16_t* pend, int& x, int& rank)
{
    const int lane = threadIdx.x & (WAVE - 1);
    int at = t.before;
    for (uint64_t h = t.hit; h != 0; h &= h - 1) pend[at++] = (uint16_t)(s_kx[one_entry(__builtin_ctzll(h), lane)] & (RB_MAX_BATCH - 1));
    wave_lds_wait();
    x = lane < t.total ? pend[lane] : -1;
    rank = 0;
    for (int j = 0; j < t.total; ++j) rank += lane_read(x, j) < x;
}

// More than WAVE class-mates: bitmap of their positions and how many are set before each of its words.
__device__ __forceinline__ void one_mate_map(const Mates& t, const uint32_t* s_kx, uint32_t* cm, uint16_t* cmpre)
{
    const int lane = threadIdx.x & (WAVE - 1);
    static_assert(ONE_WORDS == 2 * WAVE, "two bitmap words per lane");
    cm[2 * lane] = 0u;
    cm[2 * lane + 1] = 0u;
    wave_lds_wait();
    for (uint64_t h = t.hit; h != 0; h &= h - 1) {
        const int x = (int)(s_kx[one_entry(__builtin_ctzll(h), lane)] & (RB_MAX_BATCH - 1));
        atomicOr(&cm[x >> 5], 1u << (x & 31));
    }
    wave_lds_wait();
    const int p0 = __popc(cm[2 * lane]), p1 = __popc(cm[2 * lane + 1]);
    const int before = wave_scan_incl(p0 + p1) - (p0 + p1);
    cmpre[2 * lane] = (uint16_t)before;
    cmpre[2 * lane + 1] = (uint16_t)(before + p0);
    wave_lds_wait();
}

// The last position of class k's candidates that go to `slot` and lie behind position p (ANY: some number >= 0 if there is
// one); -1: there is none.  All lanes call it; cm / cmpre as one_mate_map left them.  Every lane draws for the class-mates it
// holds itself: the candidate list is dealt to the lanes evenly, whatever the positions (64 positions per lane, as in the bitmap,
// leave most lanes idle in a mini-batch of a few hundred: one class of two, 300 + 300 rows, 14.3 -> 10.3 us).
template <bool ANY>
__device__ __forceinline__ int one_last_writer(const UpdateArgs& a, const Mates& t, const uint32_t* s_kx, const uint32_t* cm,
                                               const uint16_t* cmpre, int p, int slot, int64_t fill0, int64_t aux0)
{
    const int lane = threadIdx.x & (WAVE - 1);
    int last = -1;
    for (uint64_t h = t.hit; __ballot(h != 0) != 0; h &= h - 1) {
        const int x = h != 0 ? (int)(s_kx[one_entry(__builtin_ctzll(h), lane)] & (RB_MAX_BATCH - 1)) : -1;
        if (x > p && x > last) {
            const int rank = cmpre[x >> 5] + __popc(cm[x >> 5] & ((1u << (x & 31)) - 1u));
            if (mate_slot(a, x, rank, fill0, aux0) == slot) last = x;
        }
        if (ANY && __ballot(last >= 0) != 0) return 0;
    }
    int found = -1;
    for (uint64_t w = __ballot(last >= 0); w != 0; w &= w - 1) {
        const int x = lane_read(last, __builtin_ctzll(w));
        found = x > found ? x : found;
    }
    return found;
}

// Number (rank among the class's candidates) of the last one that FIFO replacement sends to `slot`; -1: there is none.
// filled: samples before the step plus candidates.
__device__ __forceinline__ int one_fifo_rank(const UpdateArgs& a, int slot, int64_t fill0, int64_t filled, int64_t aux0)
{
    const int64_t over = filled - a.S;                       // overwrites: the slots aux0, aux0 + 1, ... one after the other
    const int64_t first = slot >= aux0 ? slot - aux0 : slot - aux0 + a.S;
    if (first < over) return (int)(a.S + first + (uint32_t)(over - 1 - first) / (uint32_t)a.S * a.S - fill0);
    return slot >= fill0 ? (int)(slot - fill0) : -1;         // appended and not overwritten
}

// Where the candidate at position p of class k (>= 0) is stored: its slot, or -1 if it is not stored (not kept, or a later
// class-mate takes the slot).
__device__ __forceinline__ int one_place(const UpdateArgs& a, const uint32_t* s_kx, int m, int32_t k, int p,
                                         int64_t fill0, int64_t aux0, uint16_t* pend, uint32_t* cm, uint16_t* cmpre)
{
    const Mates t = one_mates(s_kx, m, k, p);
    if (fill0 + t.total <= a.S) return (int)(fill0 + t.rank);                   // all of them append: distinct slots
    if (a.eviction == RB_EVICT_FIFO) {
        // it is itself overwritten in this step if a class-mate comes a whole round of S later
        return fill0 + t.rank + a.S < fill0 + t.total ? -1 : mate_slot(a, p, t.rank, fill0, aux0);
    }
    if (t.total <= WAVE) {
        int x, rank;
        one_mate_lanes(t, s_kx, pend, x, rank);
        const int slot = x >= p ? mate_slot(a, x, rank, fill0, aux0) : -1;       // this candidate and the later ones
        const int own = lane_read(slot, __builtin_ctzll(__ballot(x == p) | (1ull << 63)));
        return own < 0 || __ballot(x > p && slot == own) != 0 ? -1 : own;
    }
    const int own = mate_slot(a, p, t.rank, fill0, aux0);
    if (own < 0) return -1;
    one_mate_map(t, s_kx, cm, cmpre);
    return one_last_writer<true>(a, t, s_kx, cm, cmpre, p, own, fill0, aux0) >= 0 ? -1 : own;
}

// Mini-batch position whose row slot `slot` of class k holds after the step if the step writes it, else -1.
__device__ __forceinline__ int one_writer(const UpdateArgs& a, const uint32_t* s_kx, int m, int32_t k, int slot,
                                          int64_t filled, uint16_t* pend, uint32_t* cm, uint16_t* cmpre)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const Mates t = one_mates(s_kx, m, k, 0);
    if (t.total == 0) return -1;
    const int64_t fill0 = filled - t.total;                                     // filled: count before the step plus candidates
    if (slot < fill0 && filled <= a.S) return -1;                               // held before the step, and nothing is overwritten
    const int64_t aux0 = a.eviction != RB_EVICT_UNIFORM ? a.aux_old[k] : 0;
    const bool fifo = a.eviction == RB_EVICT_FIFO;
    const int want = fifo ? one_fifo_rank(a, slot, fill0, filled, aux0) : -1;
    if (fifo && want < 0) return -1;
    if (t.total <= WAVE) {
        int x, rank;
        one_mate_lanes(t, s_kx, pend, x, rank);
        int at = x >= 0 && (fifo ? rank == want : mate_slot(a, x, rank, fill0, aux0) == slot) ? x : -1;
        for (uint64_t w = __ballot(at >= 0); w != 0; w &= w - 1) {              // the one latest in the mini-batch
            const int xw = lane_read(at, __builtin_ctzll(w));
            at = xw > at ? xw : at;
        }
        return lane_read(at, 0);
    }
    one_mate_map(t, s_kx, cm, cmpre);
    if (fifo) {                                                                 // the lane whose 64 positions hold it
        uint64_t bits = (uint64_t)cm[2 * lane] | ((uint64_t)cm[2 * lane + 1] << 32);
        const int skip = want - cmpre[2 * lane];
        const bool mine = skip >= 0 && skip < __popcll(bits);
        for (int i = 0; mine && i < skip; ++i) bits &= bits - 1;
        const int x = mine ? 64 * lane + __builtin_ctzll(bits) : 0;
        return lane_read(x, __builtin_ctzll(__ballot(mine) | (1ull << 63)));
    }
    return one_last_writer<false>(a, t, s_kx, cm, cmpre, -1, slot, fill0, aux0);
}

// ---------------------------------------------------------------------------
// Update and sampling of one step.
//
// Every workgroup first works out, in LDS, the candidate list (class and position) and, if it moves representatives,
// the fill counts after the update and all sampling draws.  It takes a contiguous share of its side's work items (row, tile
// of at most WAVE * U vectors): its wavefronts plan the share's rows, one row each - with ballots over the candidate list,
// where a candidate goes, resp. which stored sample a representative is and whether this very step writes that slot (then
// the mini-batch row stored there is copied: no workgroup reads a row another one writes) - and then move the tiles.
//
// What bounds it: the chain selection -> labels -> candidate list -> fill counts -> draws -> rows, 0.3 to 1 us a link
// with the counts, on every compute unit at once; the rows themselves take a third of the time or less.  Hence one
// workgroup of 512 threads per compute unit (1024 threads: equal at 1024 + 1024 rows, 0.3 to 0.5 us slower at small
// counts; 256: 2 to 3 us slower; two workgroups per unit: 0.1 to 0.4 us faster for few rows, 6 us slower for 1024 + 1024),
// a row planned once per workgroup and not by every wavefront, one list word per candidate, four words of it per lane and LDS access,
// the samples before a class from the old sums per chunk and the candidates that add to them (summing 10240 counts took 1.4 us),
// the candidates' labels alone of a large mini-batch (2 us), a kernel per kind of selection and arguments read where they are used
// (0.7 to 1 us: what did not fit the scalar registers went to vector lanes and back).  Measured on MI355X, us, before these and now:
// 1024 + 1024 rows of 8 KB of 10000 classes 16.5 -> 13.0; Bernoulli selection with reservoir replacement, 90 + 75 rows of 49 KB kept as
// bfloat16, 9.4 -> 8.0; Bernoulli, 9 + 20 rows of 59 KB kept as bfloat16 7.5 -> 6.4; FIFO, 563 + 150 rows of 1 KB of 2017 classes
// 9.3 -> 8.6; 9 + 7 rows of 99 KB in 8 bits of 1160 classes 7.4 -> 6.6.  (Where the two launches are the faster form: step_form.)
//
// LDS (dynamic): s_fill[nchunks * CH] i32, s_hit[nchunks * CH / 32] u32 (bitmap of the classes with candidates), s_chunk[ONE_CHUNKS] i32,
// per wavefront pend u16[WAVE], cm u32[ONE_WORDS], cmpre u16[ONE_WORDS]; s_lab[b] u32, s_first[b] u32, s_kx[cap] u32,
// s_t[max(cap, r)] u32 (both rounded up to ONE_LIST), s_x[cap] u16.
// ---------------------------------------------------------------------------
template <int U, bool NT, int ST, bool BERNOULLI>
__global__ void __launch_bounds__(ONE_TPB) rb_step_one_kernel(const int64_t* batch_y, const int32_t* fill_old, const int32_t* chunk_old,
                                                              uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi,
                                                              uint32_t b_c, uint32_t r_nchunks, int32_t first_cand, const OneArgs)
{
    const OneArgs& sa = kernel_argument<OneArgs>(offsetof(OneKernelArgs, rest));
    const UpdateArgs& a = sa.u;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int b = (int)(b_c & 0xFFFFu), c = (int)(b_c >> 16);
    const int r = (int)(r_nchunks & 0xFFFFu), nchunks = (int)(r_nchunks >> 16), nfill = nchunks * CH;
    const Seed sd = {seed_lo, seed_hi, step_lo, step_hi};
    const bool gather = (int)blockIdx.x < first_cand;

    // labels of the whole mini-batch and, for the representatives, all fill counts and their sums per chunk: requested now.
    // Of a large mini-batch under the exact selection only the candidates' labels are read, once their positions are known; a load
    // per 64 bytes brings them near until then.  (All 4096 read and parked in LDS cost 2 us more.)
    constexpr int HELD = BERNOULLI ? ONE_PER : ONE_PARKED / ONE_TPB;
    const bool parked = BERNOULLI || b <= ONE_PARKED;
    int64_t yv[HELD], near_label = 0;
#pragma unroll
    for (int u = 0; u < HELD; ++u) {                        // (threads past the end read the last one again)
        yv[u] = 0;
        if (u * ONE_TPB < b && parked) yv[u] = batch_y[min(tid + u * ONE_TPB, b - 1)];
    }
    if (!BERNOULLI) {
        static_assert(RB_MAX_BATCH * sizeof(int64_t) / 64 <= ONE_TPB, "one load per thread");
        near_label = batch_y[min(8 * tid, b - 1)];
    }
    int4 fo[ONE_FILL_PER];
    int chunk_sum = 0;
    if (gather) {
#pragma unroll
        for (int u = 0; u < ONE_FILL_PER; ++u) {
            fo[u] = make_int4(0, 0, 0, 0);
            if (u * 4 * ONE_TPB < nfill) fo[u] = *reinterpret_cast<const int4*>(fill_old + min(4 * (tid + u * ONE_TPB), nfill - 4));
        }
        if (wave == 0 && lane < nchunks) chunk_sum = chunk_old[lane];
    }

    const ArgLines<sizeof(OneKernelArgs)> lines;

    extern __shared__ __align__(16) uint32_t lds[];
    int32_t* s_fill = reinterpret_cast<int32_t*>(lds);
    uint32_t* s_hit = lds + nfill;
    int32_t* s_chunk = reinterpret_cast<int32_t*>(s_hit + nfill / 32);
    uint32_t* mates = reinterpret_cast<uint32_t*>(s_chunk + ONE_CHUNKS);
    uint32_t* cm = mates + wave * ONE_WORDS;
    uint16_t* cmpre = reinterpret_cast<uint16_t*>(mates + ONE_NWAVE * ONE_WORDS) + wave * ONE_WORDS;
    uint16_t* pend = reinterpret_cast<uint16_t*>(mates + ONE_NWAVE * (ONE_WORDS + ONE_WORDS / 2)) + wave * WAVE;
    const int bp = (b + 3) & ~3;
    const int cand_cap = BERNOULLI ? b : c;
    uint32_t* s_lab = mates + ONE_MATE_WORDS;
    uint32_t* s_first = s_lab + bp;
    uint32_t* s_kx = s_first + bp;
    uint32_t* s_t = s_kx + one_padded(cand_cap);
    uint16_t* s_x = reinterpret_cast<uint16_t*>(s_t + one_padded(cand_cap > r ? cand_cap : r));
    __shared__ int s_seg[WAVE];                 // Bernoulli: heads per stretch of WAVE positions
    __shared__ int s_bad;
    __shared__ int s_slot[ONE_PLANNED], s_class[ONE_PLANNED], s_fwd[ONE_PLANNED];    // the rows planned last: slot (-1: not moved), class, writer
    if (tid == 0) s_bad = 0;

    // ---- candidates: positions ----
    int m = c;                                  // number of candidates
    int at[ONE_PER];                            // Bernoulli: list index of position tid + u * ONE_TPB, -1: not selected
    // Sampling draws: thread `sid + u * ONE_TPB` of them.  A draw takes a wavefront twenty multiplications of a quarter of the rate, and the
    // wavefronts of a compute unit share its four units: each makes those it has alone, the last wavefronts the first ones, while the
    // first ones select or flip coins.  (Two each in any case, before the selection's, and the books by the first wavefronts (below): 10 + 4 rows of
    // 1 KB, Bernoulli, 5.92 us, now 5.85; 64 + 26 of 1031 classes, of 5 KB 6.62 : 6.32, of 11 KB 6.67 : 6.36.  Of large
    // mini-batches they are made while the candidates' labels travel: 1024 + 1024 of 8 KB 13.57 : 13.01.)
    const int sid = tid ^ (ONE_TPB - WAVE);
    uint64_t bits[ONE_PER];                     // random bits of sampling draw sid + u * ONE_TPB
    const auto draw_bits = [&]() {
        const int first = __builtin_amdgcn_readfirstlane(sid);
#pragma unroll
        for (int u = 0; u < ONE_PER; u += 2) {              // (two at a time: one draw is a chain of dependent multiplications)
            if (first + u * ONE_TPB >= r) break;
            bits[u] = draw64(sd, PURPOSE_SAMPLE, (uint32_t)(sid + u * ONE_TPB));
            if (first + (u + 1) * ONE_TPB < r) bits[u + 1] = draw64(sd, PURPOSE_SAMPLE, (uint32_t)(sid + (u + 1) * ONE_TPB));
            asm volatile("" : "+v"(bits[u]), "+v"(bits[u + 1]));        // (here, not where they are used)
        }
    };
    if (gather && parked) draw_bits();
    if constexpr (BERNOULLI) {
        uint32_t heads = 0;                     // bit u: the coin of position tid + u * ONE_TPB
#pragma unroll 1
        for (int u = 0; u * ONE_TPB < b; ++u) {
            const int q = tid + u * ONE_TPB;
            const bool head = q < b && (int)below(sd, PURPOSE_COIN, (uint32_t)q, (uint64_t)b) < c;
            heads |= (uint32_t)head << u;
            const int in_seg = __popcll(__ballot(head));
            if (lane == 0) s_seg[u * ONE_NWAVE + wave] = in_seg;
        }
        lds_barrier();
        static_assert(ONE_PER * ONE_NWAVE == WAVE, "one lane per stretch of positions");
        const int segs = (b + ONE_TPB - 1) / ONE_TPB * ONE_NWAVE;
        const int incl = wave_scan_incl(lane < segs ? s_seg[lane] : 0);
        m = lane_read(incl, WAVE - 1);
#pragma unroll
        for (int u = 0; u < ONE_PER; ++u) {
            if (u * ONE_TPB >= b) break;
            const bool mine = (heads >> u) & 1;
            const uint64_t seg_heads = __ballot(mine);
            at[u] = mine ? lane_read(incl, u * ONE_NWAVE + wave) - __popcll(seg_heads >> lane) : -1;       // (this one and the heads behind it)
            if (mine) s_x[at[u]] = (uint16_t)(tid + u * ONE_TPB);
        }
    } else if (c <= WAVE) {
        if (wave == 0) {
            bool active;
            const int x = wave_select(sd, b, c, s_first, active);
            if (active) s_x[lane] = (uint16_t)x;
        }
    } else {
        // Floyd's c-subset, all draws at once (see rb_update_kernel)
        const int base = b - c;
#pragma unroll 1
        for (int i0 = tid; i0 < c; i0 += 2 * ONE_TPB) {
            const int i1 = i0 + ONE_TPB;
            if (__builtin_amdgcn_readfirstlane(i1) < c) {
                const uint64_t d0 = draw64(sd, PURPOSE_SELECT, (uint32_t)i0), d1 = draw64(sd, PURPOSE_SELECT, (uint32_t)i1);
                const uint32_t t0 = reduce32(d0, (uint32_t)(base + i0 + 1)), t1 = reduce32(d1, (uint32_t)(base + i1 + 1));
                s_t[i0] = t0;
                s_first[t0] = 0xFFFFFFFFu;
                if (i1 < c) { s_t[i1] = t1; s_first[t1] = 0xFFFFFFFFu; }
            } else {
                const uint32_t t0 = reduce32(draw64(sd, PURPOSE_SELECT, (uint32_t)i0), (uint32_t)(base + i0 + 1));
                s_t[i0] = t0;
                s_first[t0] = 0xFFFFFFFFu;
            }
        }
        lds_barrier();
        for (int i = tid; i < c; i += ONE_TPB) atomicMin(&s_first[s_t[i]], (uint32_t)i);
        lds_barrier();
        // a draw is replaced iff an earlier one had the same value, or it is base + q for an earlier q that was replaced
#pragma unroll 2
        for (int i = tid; i < c; i += ONE_TPB) {
            const int own = (int)s_t[i];
            bool taken = s_first[own] != (uint32_t)i;
            int cur = i, q = own - base;
            while (!taken && q >= 0 && q < cur) {
                cur = q;
                const int d = (int)s_t[cur];
                taken = s_first[d] != (uint32_t)cur;
                q = d - base;
            }
            s_x[i] = (uint16_t)(taken ? base + i : own);
        }
    }
    lines.arrived();
    lds_barrier();

    // classes of the candidates; ends with a barrier after which the list is complete
    const auto listed = [&](int x, int64_t y) { return (uint64_t)y < (uint64_t)a.K ? ((uint32_t)y << ONE_POS_BITS) | (uint32_t)x : ONE_NO_CLASS; };
    // (meanwhile: done while the labels travel, where they are requested only now)
    const auto classes = [&](auto meanwhile) {
        for (int q = m + tid; q < one_padded(m); q += ONE_TPB) s_kx[q] = ONE_NO_CLASS;
        if constexpr (BERNOULLI) {
#pragma unroll
            for (int u = 0; u < ONE_PER; ++u) {
                if (u * ONE_TPB >= b) break;
                int64_t y = yv[u];
                asm volatile("" : "+v"(y));     // keeps the range test, and so the wait for the label, from moving up
                if (at[u] >= 0) s_kx[at[u]] = listed(tid + u * ONE_TPB, y);
            }
        } else if (parked) {
#pragma unroll
            for (int u = 0; u < ONE_PARKED / ONE_TPB; ++u) {
                if (u * ONE_TPB >= b) break;
                const int q = tid + u * ONE_TPB;
                int64_t y = yv[u];
                asm volatile("" : "+v"(y));
                if (q < b) s_lab[q] = listed(q, y);
            }
            lds_barrier();
            for (int q = tid; q < c; q += ONE_TPB) s_kx[q] = s_lab[s_x[q]];
        } else {
            asm volatile("" : : "v"(near_label));
            // (two at a time, both requested before either is waited for: 1024 + 1024 rows of 8 KB of a mini-batch of 4096 14.05 -> 13.57 us)
            int i0 = 0;
            for (; i0 + ONE_TPB < c; i0 += 2 * ONE_TPB) {
                const int q0 = i0 + tid, q1 = q0 + ONE_TPB;
                const int x0 = s_x[q0], x1 = s_x[min(q1, c - 1)];
                int64_t y0 = batch_y[x0], y1 = batch_y[x1];
                if (i0 == 0) meanwhile();
                asm volatile("" : "+v"(y0), "+v"(y1));      // (the compiler would move the second request into its branch, behind the wait for the first)
                s_kx[q0] = listed(x0, y0);
                if (q1 < c) s_kx[q1] = listed(x1, y1);
            }
            const int x0 = s_x[min(i0 + tid, c - 1)];
            int64_t y0 = 0;
            if (i0 < c) y0 = batch_y[x0];
            if (i0 == 0) meanwhile();
            asm volatile("" : "+v"(y0));
            if (i0 + tid < c) s_kx[i0 + tid] = listed(x0, y0);
        }
        lds_barrier();
    };
    constexpr int WIDE = stored_wide(ST);       // vectors of a mini-batch / output row per vector of a stored row
    int64_t v_lo, v_hi;

    if (!gather) {
        // ---- candidate movers ----
        const int items = m * a.tpr, nwg = sa.nwg - first_cand;
        const int share = sa.cshare != 0 ? sa.cshare : (items + nwg - 1) / nwg;
        const int lo = ((int)blockIdx.x - first_cand) * share, hi = min(lo + share, items);
        if (lo >= hi) return;
        // A row is requested as soon as its position is known, before the labels have arrived (by every wavefront: a load
        // that only some issue would make the wait for the labels a wait for the rows).  Of a large mini-batch the candidates' labels are
        // requested behind the rows, and arrive behind them.
        int it = min(lo + wave, hi - 1);
        Tile<U, NT, WAVE, ONE_PACE, stored_cv(ST, CV_NARROW), true> t;
        {
            const int i = it / a.tpr;
            tile_bounds(it - i * a.tpr, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);
            t.load(a.batch_x + (int64_t)__builtin_amdgcn_readfirstlane(s_x[i]) * a.row_vec * WIDE, v_lo, v_hi);
        }
        classes([]() {});
        it = lo + wave;
        bool loaded = true;
        // (a second round only when the coins of the Bernoulli selection gave many times the candidates the grid was sized for)
        for (int row = lo / a.tpr; row * a.tpr < hi; row += ONE_PLANNED) {
            const int end = min((hi + a.tpr - 1) / a.tpr, row + ONE_PLANNED);
            for (int i = row + wave; i < end; i += ONE_NWAVE) {
                const uint32_t kx = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_kx[i]);
                int slot = -1;
                if (kx != ONE_NO_CLASS) {       // else a label outside [0, K): dropped (the representatives' workgroups flag it)
                    const int32_t ki = (int32_t)(kx >> ONE_POS_BITS);
                    const int64_t fill0 = a.fill_old[ki];
                    const int64_t aux0 = a.eviction != RB_EVICT_UNIFORM ? a.aux_old[ki] : 0;
                    slot = one_place(a, s_kx, m, ki, (int)(kx & (RB_MAX_BATCH - 1)), fill0, aux0, pend, cm, cmpre);
                }
                if (lane == 0) s_slot[i - row] = slot;
            }
            if (a.tpr == 1) wave_lds_wait();        // (the rows a wavefront moves are the ones it planned)
            else lds_barrier();
            for (; it < min(hi, end * a.tpr); it += ONE_NWAVE) {
                const int i = it / a.tpr, tile = it - i * a.tpr;
                const int slot = __builtin_amdgcn_readfirstlane(s_slot[i - row]);
                if (slot >= 0) {
                    const uint32_t kx = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_kx[i]);
                    const int64_t dst_row = (int64_t)(kx >> ONE_POS_BITS) * a.S + slot;
                    if (!loaded) {
                        tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);
                        t.load(a.batch_x + (int64_t)(kx & (RB_MAX_BATCH - 1)) * a.row_vec * WIDE, v_lo, v_hi);
                    }
                    t.store(a.buf_x + dst_row * a.row_vec, v_lo, v_hi);
                    if (tile == 0 && lane == 0) { a.buf_y[dst_row] = (int64_t)(kx >> ONE_POS_BITS); count_moved(a.state); }
                }
                loaded = false;
            }
            if (a.tpr != 1 && end * a.tpr < hi) lds_barrier();
        }
        return;
    }

    // ---- fill counts after the update (not yet cut off at the capacity: step_form keeps S + RB_MAX_BATCH within 32 bits) ----
    for (int i = tid; i < nfill / 32; i += ONE_TPB) s_hit[i] = 0u;
    if (wave == 0) s_chunk[lane] = chunk_sum;
#pragma unroll
    for (int u = 0; u < ONE_FILL_PER; ++u) {
        if (u * 4 * ONE_TPB >= nfill) break;
        if (4 * (tid + u * ONE_TPB) < nfill) *reinterpret_cast<int4*>(s_fill + 4 * (tid + u * ONE_TPB)) = fo[u];
    }
    classes(draw_bits);
    const int32_t cap = (int32_t)a.S;
    for (int q = tid; q < m; q += 2 * ONE_TPB) {
        const uint32_t kx[2] = {s_kx[q], q + ONE_TPB < m ? s_kx[q + ONE_TPB] : ONE_NO_CLASS};
        int held[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (kx[u] != ONE_NO_CLASS) held[u] = atomicAdd(&s_fill[kx[u] >> ONE_POS_BITS], 1);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t k = kx[u] >> ONE_POS_BITS;
            if (kx[u] == ONE_NO_CLASS) {
                if (q + u * ONE_TPB < m) s_bad = 1;
                continue;
            }
            atomicOr(&s_hit[k >> 5], 1u << (k & 31));
            if (held[u] < cap) atomicAdd(&s_chunk[k / CH], 1);      // one more sample of the class
        }
    }
    lds_barrier();
    // stored samples up to and including chunk `lane`
    const int in_chunk = s_chunk[lane], upto = wave_scan_incl(in_chunk);
    const int F = lane_read(upto, WAVE - 1);
    const int n = r < F ? r : F;
    const int base = F - n;
#pragma unroll
    for (int u = 0; u < ONE_PER; ++u) {
        if (u * ONE_TPB >= n) break;
        const int q = sid + u * ONE_TPB;
        if (q < n) s_t[q] = reduce32(bits[u], (uint32_t)(base + q + 1));
    }
    if (blockIdx.x == 0 && tid == 0) {
        a.state->last_n = n;
        if (s_bad) atomicOr(&a.state->flags, RB_FLAG_BAD_LABEL);
    }
    lds_barrier();

    // ---- representative movers ----
    const int lo = (int)blockIdx.x * sa.share, hi = min(lo + sa.share, r * sa.tpr);
    int it = lo + wave;
    // (one round for every count accepted: a share has at most 33 rows.  Written without the loop the same round measured 1 to 2 %
    // slower with few rows: Bernoulli selection, 90 + 75 rows of 49 KB kept as bfloat16, 9.21 -> 9.5 us)
    for (int row = lo / sa.tpr; row * sa.tpr < hi; row += ONE_PLANNED) {
        const int end = min((hi + sa.tpr - 1) / sa.tpr, row + ONE_PLANNED);
        for (int j = row + wave; j < end; j += ONE_NWAVE) {
            if (j >= n) {                      // fewer stored samples than asked for
                if (lane == 0) s_slot[j - row] = -1;
                continue;
            }
            // draw j is replaced by base + j iff an earlier draw had the same value, or it equals
            // base + q for an earlier q whose own draw was replaced
            const int own = __builtin_amdgcn_readfirstlane((int)s_t[j]);
            int cur = j, tc = own;
            bool taken = false;
            for (;;) {
                bool same = false;
#pragma unroll 4
                for (int q0 = 0; q0 < cur; q0 += ONE_LIST) {
                    const uint4 v = *reinterpret_cast<const uint4*>(s_t + q0 + 4 * lane);
                    const int left = cur - q0 - 4 * lane;           // of the lane's words, those before draw `cur`
                    same |= (v.x == (uint32_t)tc && left > 0) | (v.y == (uint32_t)tc && left > 1) | (v.z == (uint32_t)tc && left > 2) | (v.w == (uint32_t)tc && left > 3);
                }
                if (__ballot(same) != 0) { taken = true; break; }
                const int q = tc - base;
                if (q < 0 || q >= cur) break;
                cur = q;
                tc = __builtin_amdgcn_readfirstlane((int)s_t[cur]);
            }
            const int g = taken ? base + j : own;          // class-major number of the sample
            // the chunk of classes that holds it (the number of chunks that end at or before it), then the class
            const int ch = __popcll(__ballot(upto <= g));
            const int4 f = *reinterpret_cast<const int4*>(s_fill + ch * CH + 4 * lane);
            int owner, sub, ps;
            WaveFill(make_int4(min(f.x, cap), min(f.y, cap), min(f.z, cap), min(f.w, cap)))
                .locate(g - (lane_read(upto, ch) - lane_read(in_chunk, ch)), owner, sub, ps);
            const int pk = ch * CH + 4 * owner + sub;
            int fwd = -1;
            if ((__builtin_amdgcn_readfirstlane((int)s_hit[pk >> 5]) >> (pk & 31)) & 1) fwd = one_writer(a, s_kx, m, pk, ps, s_fill[pk], pend, cm, cmpre);
            if (lane == 0) {
                s_slot[j - row] = ps;
                s_class[j - row] = pk;
                s_fwd[j - row] = fwd;
            }
        }
        if (sa.tpr == 1) wave_lds_wait();           // (the rows a wavefront moves are the ones it planned)
        else lds_barrier();
        for (; it < min(hi, end * sa.tpr); it += ONE_NWAVE) {
            const int j = it / sa.tpr, tile = it - j * sa.tpr;
            const int ps = __builtin_amdgcn_readfirstlane(s_slot[j - row]);
            if (ps < 0) {
                if (tile == 0 && lane == 0) sa.out_y[j] = -1;
                continue;
            }
            const int pk = __builtin_amdgcn_readfirstlane(s_class[j - row]), fwd = __builtin_amdgcn_readfirstlane(s_fwd[j - row]);
            tile_bounds(tile, sa.tile_vec, sa.tile_rem, a.row_vec, v_lo, v_hi);
            vec16* dst = sa.out_x + (int64_t)j * a.row_vec * WIDE;
            if (ST != RB_STORE_SAME && fwd >= 0) {
                // from the mini-batch: what the slot will hold is the row in its stored form
                Tile<U, NT, WAVE, ONE_PACE, stored_cv(ST, CV_BOTH)> o;
                o.load(a.batch_x + (int64_t)fwd * a.row_vec * WIDE, v_lo, v_hi);
                o.store(dst, v_lo, v_hi);
            } else {
                const vec16* src = fwd >= 0 ? a.batch_x + (int64_t)fwd * a.row_vec : a.buf_x + ((int64_t)pk * a.S + ps) * a.row_vec;
                Tile<U, NT, WAVE, ONE_PACE, stored_cv(ST, CV_WIDEN)> o;
                o.load(src, v_lo, v_hi);
                o.store(dst, v_lo, v_hi);
            }
            if (tile == 0 && lane == 0) { sa.out_y[j] = pk; count_moved(a.state); }
        }
        if (sa.tpr != 1 && end * sa.tpr < hi) lds_barrier();
    }

    // ---- books: new fill counts, their sums per chunk, the strategy's state (a chunk per wavefront, dealt over the workgroups) ----
    // (by the last wavefronts where there are fewer tiles than wavefronts: they have none to wait for.  FIFO and reservoir replacement, whose
    // state is read first, Bernoulli, 9 + 7 rows of 1.6 KB 5.96 -> 5.66 us; where all have tiles the first ones are done first)
    const int keeper = hi - lo < ONE_NWAVE ? ONE_NWAVE - 1 - wave : wave;
    for (int ch = keeper * first_cand + blockIdx.x; ch < nchunks; ch += first_cand * ONE_NWAVE) {
        const int k0 = ch * CH + 4 * lane;
        const int4 v = *reinterpret_cast<const int4*>(s_fill + k0);
        const int4 f = make_int4(min(v.x, cap), min(v.y, cap), min(v.z, cap), min(v.w, cap));
        *reinterpret_cast<int4*>(a.fill_new + k0) = f;
        if (lane == 0) a.chunk_new[ch] = s_chunk[ch];
        if (a.eviction != RB_EVICT_UNIFORM) {
            const int4 old4 = *reinterpret_cast<const int4*>(a.fill_old + k0);
            const int4 aux4 = *reinterpret_cast<const int4*>(a.aux_old + k0);
            const int4 next = make_int4(next_aux(a, old4.x, aux4.x, v.x - old4.x), next_aux(a, old4.y, aux4.y, v.y - old4.y),
                                        next_aux(a, old4.z, aux4.z, v.z - old4.z), next_aux(a, old4.w, aux4.w, v.w - old4.w));
            *reinterpret_cast<int4*>(a.aux_new + k0) = next;
        }
    }
}

}  // namespace
