// Small-count kernels (at most 64 candidates / representatives): one wavefront of a workgroup selects and places the candidates, one per
// chunk of classes finds the representative; includes the single-launch update + sample kernel.
// Included by rb.hip only, after rb_device.h.
#pragma once

#include "rb_device.h"

namespace {

constexpr int YPRE = 4;    // label loads per thread issued before anything else (covers b <= 1024)

// The first YPRE labels per thread (threads past the end hold the last one again).
__device__ __forceinline__ void request_labels(int64_t (&yv)[YPRE], const int64_t* __restrict__ batch_y, int b)
{
#pragma unroll
    for (int u = 0; u < YPRE; ++u) {
        yv[u] = -1;
        if (u * TPB < b) yv[u] = batch_y[min((int)threadIdx.x + u * TPB, b - 1)];
    }
}

// ... into LDS (LAB_INVALID when outside [0, K)) and (ALL) those beyond them; called by all threads.
template <bool ALL>
__device__ __forceinline__ void park_labels(const int64_t (&yv)[YPRE], const int64_t* __restrict__ batch_y, int b, int K, int32_t* s_y)
{
    const auto parked = [&](int64_t y) { return (uint64_t)y < (uint64_t)K ? (int32_t)y : LAB_INVALID; };
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < YPRE; ++u) {
        if (u * TPB >= b) break;
        const int q = tid + u * TPB;
        int64_t y = yv[u];
        // keeps the compiler from evaluating the range test (and so waiting for the load) any
        // earlier than here; the loads are meant to stay in flight across the code before
        asm volatile("" : "+v"(y));
        if (q < b) s_y[q] = parked(y);
    }
    if (!ALL) return;
    for (int q = tid + YPRE * TPB; q < b; q += TPB) s_y[q] = parked(batch_y[q]);
}

// Of a mini-batch larger than that only the candidates' labels are read, as soon as wavefront 0 has selected them (parking all
// 4096 takes twelve more loads per thread, one after the other: 16 + 16 rows of 12 KB, FIFO, two calls 9.9 -> 8.1 us).
__device__ __forceinline__ int64_t far_label(const UpdateArgs& a, bool active, int x)
{
    return active && x >= YPRE * TPB ? a.batch_y[x] : -1;
}

// Class of the lane's candidate (wavefront 0): parked, or far_label's y.
__device__ __forceinline__ int32_t candidate_class(const UpdateArgs& a, bool active, int x, const int32_t* s_y, int64_t y)
{
    if (!active) return LAB_UNSELECTED;
    if (x < YPRE * TPB) return s_y[x];
    asm volatile("" : "+v"(y));
    return y >= 0 && y < a.K ? (int32_t)y : LAB_INVALID;
}

// ---------------------------------------------------------------------------
// Pieces of the plan shared by the small-count kernels.  Called by wavefront 0
// only, with all of its 64 lanes active.
// ---------------------------------------------------------------------------

// Floyd's c-subset of the b mini-batch positions, all draws at once: lane i < c
// draws t_i uniform in [0, b-c+i]; the sequential algorithm replaces t_i by
// b-c+i when t_i was chosen before, which is the case iff an earlier lane drew
// the same value, or t_i = b-c+q for an earlier q whose own draw was replaced.
// Returns the lane's candidate position (0 for lanes >= c); s_first: b words of LDS.
__device__ __forceinline__ int wave_select(const Seed& sd, int b, int c, uint32_t* s_first, bool& active)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int base = b - c;
    active = lane < c;
    const uint32_t t = active ? (uint32_t)below(sd, PURPOSE_SELECT, (uint32_t)lane, (uint64_t)(base + lane + 1)) : 0u;
    if (active) s_first[t] = 0xFFFFFFFFu;
    if (active) atomicMin(&s_first[t], (uint32_t)lane);
    bool taken = active && s_first[t] != (uint32_t)lane;
    int q = (int)t - base;                       // lane whose replacement value the draw equals
    bool open = active && !taken && q >= 0 && q < lane;
    if (__ballot(open) != 0) {
        const int packed = (int)(t | (taken ? 0x80000000u : 0u));      // t < 4096: bit 31 is free for the flag
        do {
            const int pc = __shfl(packed, open ? q : lane, WAVE);
            if (open) {
                const int further = pc - base;
                if (pc < 0) taken = true;
                open = pc >= 0 && further >= 0 && further < q;
                q = further;
            }
        } while (__ballot(open) != 0);
    }
    return active ? (taken ? base + lane : (int)t) : 0;
}

// Slot of class-mate number `rank` (at mini-batch position x) of a class that held fill0 samples: appended while there is
// room, else what the replacement strategy overwrites; -1: not kept (reservoir).  aux0: the strategy's state of the class.
__device__ __forceinline__ int mate_slot(const UpdateArgs& a, int x, int rank, int64_t fill0, int64_t aux0)
{
    const int64_t at = fill0 + rank;
    if (at < a.S) return (int)at;
    // (aux0 < S and at - S < RB_MAX_BATCH: 32 unsigned bits; a 64-bit remainder is some hundred instructions)
    if (a.eviction == RB_EVICT_FIFO) return (int)((uint32_t)(aux0 + at - a.S) % (uint32_t)a.S);
    const bool reservoir = a.eviction == RB_EVICT_RESERVOIR;
    const int64_t offers = aux0 + rank < INT32_MAX ? aux0 + rank : INT32_MAX;      // to the class, before this one
    const int64_t draw = (int64_t)below(a.sd, PURPOSE_EVICT, (uint32_t)x, reservoir ? (uint64_t)offers + 1 : (uint64_t)a.S);
    return draw < a.S ? (int)draw : -1;
}

// The strategy's state of a class after a step that offers it `count` candidates (old: samples it held, aux: state before).
__device__ __forceinline__ int32_t next_aux(const UpdateArgs& a, int64_t old, int64_t aux, int64_t count)
{
    if (a.eviction == RB_EVICT_FIFO) {
        const int64_t over = old + count > a.S ? old + count - a.S : 0;            // the oldest sample moves on by the overwrites
        return (int32_t)((uint32_t)(aux + over) % (uint32_t)a.S);
    }
    const int64_t seen = aux + count;
    return (int32_t)(seen < INT32_MAX ? seen : INT32_MAX);
}

// For every lane of `mask`: how many other lanes of it hold a smaller x.
__device__ __forceinline__ int rank_among(uint64_t mask, int x)
{
    int rank = 0;
    while (mask != 0) {
        const int m = __builtin_ctzll(mask);
        mask &= mask - 1;
        rank += (int)(__builtin_amdgcn_readlane(x, m) < x);
    }
    return rank;
}

// Where candidate i (mini-batch position p, class ki, fill0 samples of that class stored before
// the step) is stored: row index ki*S + slot, or -1 if it is not stored (label outside [0, K),
// or a later class-mate overwrites its slot).  Lane l holds candidate l: position x, class k, and (uniform
// replacement) the slot it overwrites if its class is full.  AUX: FIFO or reservoir replacement.
template <bool AUX>
__device__ __forceinline__ int64_t wave_place(const UpdateArgs& a, bool active, int x, int32_t k, int draw, int i, int p, int32_t ki, int32_t fill0)
{
    if (ki < 0) return -1;
    const uint32_t S = (uint32_t)a.S;            // (counts and slots are below 2^31: sums with a step's candidates fit 32 unsigned bits)
    // candidates of class ki; in mini-batch order the one with `rank` class-mates
    // before it is insertion number fill0 + rank of the class
    const bool same = active && k == ki;
    const int total = __popcll(__ballot(same));
    const int rank = __popcll(__ballot(same && x < p));
    if ((uint32_t)fill0 + total <= S) return (int64_t)ki * a.S + fill0 + rank;     // all append: distinct slots
    if (AUX && a.eviction == RB_EVICT_FIFO) {
        // it is itself overwritten in this step if a class-mate comes a whole round of S later
        return rank + a.S < total ? -1 : (int64_t)ki * a.S + mate_slot(a, p, rank, fill0, a.aux_old[ki]);
    }
    if (AUX) {
        // a later class-mate may take the slot, or it may not be kept
        const int slot = same ? mate_slot(a, x, rank_among(__ballot(same), x), fill0, a.aux_old[ki]) : -1;
        const int own = lane_read(slot, i);
        return own < 0 || __ballot(same && x > p && slot == own) != 0 ? -1 : (int64_t)ki * a.S + own;
    }
    // Insertions beyond the capacity overwrite a uniformly drawn slot.  This
    // candidate is not stored if a later class-mate overwrites its slot.
    const int own = (uint32_t)fill0 + rank < S ? fill0 + rank : lane_read(draw, i);
    uint64_t rivals = __ballot(same && x > p && draw == own);
    while (rivals != 0) {
        const int m = __builtin_ctzll(rivals);
        rivals &= rivals - 1;
        const int xm = __builtin_amdgcn_readlane(x, m);
        const int rank_m = __popcll(__ballot(same && x < xm));
        if ((uint32_t)fill0 + rank_m >= S) return -1;                  // m does overwrite
    }
    return (int64_t)ki * a.S + own;
}

// Number, among the stored samples class by class, of representative j: lane l holds Floyd draw l (all ones beyond the last),
// `base` is the range of the first draw less one.  Draw j is replaced by base + j iff an earlier draw had the same value, or it
// equals base + q for an earlier q whose own draw was replaced.
__device__ __forceinline__ int wave_sample_number(uint32_t t, int j, int base)
{
    const int lane = threadIdx.x & (WAVE - 1);
    int cur = j;
    for (;;) {
        const uint32_t tc = (uint32_t)lane_read((int)t, cur);
        if (__ballot(lane < cur && t == tc) != 0) return base + j;
        const int q = (int)tc - base;
        if (q < 0 || q >= cur) return lane_read((int)t, j);
        cur = q;
    }
}

// The samples of the classes a wavefront holds, four consecutive ones per lane.
struct WaveFill {
    int4 f;
    int local, incl;      // samples of the lane's classes, and of the lanes up to and including this one

    WaveFill() = default;
    __device__ __forceinline__ explicit WaveFill(int4 counts) : f(counts)
    {
        local = f.x + f.y + f.z + f.w;
        incl = wave_scan_incl(local);
    }
    __device__ __forceinline__ int total() const { return lane_read(incl, WAVE - 1); }
    // Sample number g of them (0 <= g < total(), the same in all lanes): lane and number of its class there, and its slot.
    __device__ __forceinline__ void locate(int g, int& owner, int& sub, int& slot) const
    {
        const int at = g - (incl - local);
        const int f01 = f.x + f.y, f012 = f01 + f.z;
        const int u = (at >= f.x) + (at >= f01) + (at >= f012);
        const int s = at - (u == 0 ? 0 : u == 1 ? f.x : u == 2 ? f01 : f012);
        owner = __builtin_ctzll(__ballot(at >= 0 && at < local) | (1ull << 63));
        sub = lane_read(u, owner);
        slot = lane_read(s, owner);
    }
};

__device__ __forceinline__ int capped_sum(int old, int more, int cap)      // min(old + more, cap), old <= cap
{
    return old + min(more, cap - old);
}

constexpr int DIRECT_CHUNKS = 4;         // up to this many chunks of classes every wavefront of a workgroup reads one chunk's counts

// Fill counts of classes 4 tid ... 4 tid + 3 (nchunks * CH counts exist); zeros beyond.
__device__ __forceinline__ int4 request_fill(const int32_t* fill, int nchunks)
{
    const int first = 4 * (int)threadIdx.x;
    int4 f = make_int4(0, 0, 0, 0);
    if (first < nchunks * CH) f = *reinterpret_cast<const int4*>(fill + first);
    return f;
}

// What the first instructions of these kernels need comes as arguments of its own in front of the structure: the hardware puts the
// first 14 words of a kernel's arguments into scalar registers when it starts a wavefront, so labels and fill counts are requested
// and the selection is drawn without waiting for the arguments' trip from memory (0.3 us of the chain in every launch: 16 + 16 rows
// of 12 KB 4.38 -> 4.12 us, 4 + 4 in two calls 7.11 -> 6.49, 64 + 64 rows of 301 KB in two calls 17.7 -> 16.8).

// ---------------------------------------------------------------------------
// rb_update for c <= WAVE candidates, exact selection, any replacement strategy and storage form: the plan is computed by the first
// wavefront of each workgroup alone, one lane per candidate, with ballots and
// lane reads instead of workgroup scans; the other three wavefronts only move
// data.  Same grid as rb_update_kernel.  Up to DIRECT_CHUNKS chunks of classes the fill counts are requested together with the labels
// (read once the class is known they are one more trip to memory, 0.6 us).
//
// LDS (dynamic): s_first[b] u32 (lowest lane that drew a value), s_y[b] i32
// (label of every mini-batch position below YPRE * TPB, LAB_INVALID when outside [0, K)),
// s_old[DIRECT_CHUNKS * CH] i32 (fill counts before the step, if there are no more classes).
// ---------------------------------------------------------------------------
template <int U, bool NT, int ST, bool AUX, bool STREAM = NT>     // ST: RB_STORE_*, the form binary32 samples are stored in; AUX: FIFO or reservoir replacement; STREAM: streaming stores
__global__ void __launch_bounds__(TPB) rb_update_small_kernel(const int64_t* batch_y, const int32_t* fill_old, uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi,
                                                              uint32_t b_c, int32_t nchunks, const UpdateArgs a)
{
    const int b = (int)(b_c & 0xFFFFu), c = (int)(b_c >> 16);
    const Seed sd = {seed_lo, seed_hi, step_lo, step_hi};
    extern __shared__ uint32_t lds[];
    uint32_t* s_first = lds;                                   // [b]
    int32_t* s_y = reinterpret_cast<int32_t*>(lds + b);        // [b]
    int32_t* s_old = reinterpret_cast<int32_t*>(lds + ((2 * b + 3) & ~3));     // [DIRECT_CHUNKS * CH], 16-byte aligned
    __shared__ int s_wave[NWAVE];
    __shared__ int s_hist[CH];
    __shared__ int s_p[2];          // mini-batch position of the current candidate (double-buffered over rows)
    __shared__ int64_t s_dst[2];    // slot row it is stored to, -1: not stored

    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const bool w0 = tid < WAVE;
    const bool direct = nchunks <= DIRECT_CHUNKS;

    // labels of the mini-batch and fill counts: requested now, parked in LDS once the selection is done
    int64_t yv[YPRE];
    request_labels(yv, batch_y, b);
    int4 fo = make_int4(0, 0, 0, 0);
    if (direct) fo = request_fill(fill_old, nchunks);

    // wavefront 0: lane i computes candidate i of Floyd's emission order
    bool active = false;
    int x = 0;                       // its mini-batch position
    int64_t yx = -1;                 // its label, if it lies beyond the parked ones
    if (w0) {
        x = wave_select(sd, b, c, s_first, active);
        yx = far_label(a, active, x);
    }

    if ((int)blockIdx.x < nchunks) {
        // ---- bookkeeping: fill_new = min(fill_old + candidates of the class, S) ----
        park_labels<false>(yv, batch_y, b, a.K, s_y);
        const int k_lo = blockIdx.x * CH;
        s_hist[tid] = 0;
        __syncthreads();
        if (w0) {
            const int32_t k = candidate_class(a, active, x, s_y, yx);
            if (active && k >= k_lo && k < k_lo + CH) atomicAdd(&s_hist[k - k_lo], 1);
            if (blockIdx.x == 0 && __ballot(active && k == LAB_INVALID) != 0 && lane == 0)
                atomicOr(&a.state->flags, RB_FLAG_BAD_LABEL);
        }
        __syncthreads();
        const int kk = k_lo + tid;
        int32_t nf = 0;
        if (kk < a.K) {
            int64_t v = (int64_t)a.fill_old[kk] + s_hist[tid];
            nf = (int32_t)(v < a.S ? v : a.S);
            a.fill_new[kk] = nf;
            if (AUX) a.aux_new[kk] = next_aux(a, a.fill_old[kk], a.aux_old[kk], s_hist[tid]);
        }
        int total;
        block_scan_excl(nf, total, s_wave);
        if (tid == 0) a.chunk_new[blockIdx.x] = total;
        return;
    }

    // ---- movers ---------------------------------------------------------------
    const int mover = blockIdx.x - nchunks;
    const int group = mover / a.tpr, tile = mover % a.tpr;
    int64_t v_lo, v_hi;
    tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);

    // The first row is handled outside the loop over further rows: the label loads are still in
    // flight here and a loop header would make the compiler wait for them before the barrier.
    int32_t k = LAB_UNSELECTED;      // wavefront 0: class of the lane's candidate
    int draw = -1;                   // ... and (uniform replacement) the slot it overwrites if the class is full
    const auto place = [&](int i, int p) {
        const int32_t ki = lane_read(k, i);
        // One access through a pointer to either memory would wait for the row that has just been requested.  So rows that are converted
        // have a branch for each memory: FIFO and reservoir replacement, more than six workgroups on a compute unit, 60 rows of 464 KB
        // as bfloat16 of 1500 classes 9.7 -> 8.0 us, in 8 bits 9.8 -> 8.3, of 43 classes 9.0 -> 7.7; 16 of 99 KB in 8 bits 3.9 -> 3.8.
        // Plain rows do as well or better with the wait: 64 of 203 KB, FIFO, 7.0 against 7.4, 40 of 301 KB 6.6 : 6.7, 16 of 99 KB 3.38 : 3.36.
        if constexpr (ST != RB_STORE_SAME) {
            if (direct) return wave_place<AUX>(a, active, x, k, draw, i, p, ki, ki < 0 ? 0 : s_old[ki]);
            return wave_place<AUX>(a, active, x, k, draw, i, p, ki, ki < 0 ? 0 : a.fill_old[ki]);
        }
        const int32_t fill0 = ki < 0 ? 0 : direct ? s_old[ki] : a.fill_old[ki];
        return wave_place<AUX>(a, active, x, k, draw, i, p, ki, fill0);
    };
    {
        const int i = group * a.rpb;           // candidate, in Floyd emission order
        if (i >= c) return;
        if (w0) {
            const int pi = lane_read(x, i);
            if (lane == 0) s_p[0] = pi;
        }
        lds_barrier();
        const int p = s_p[0];
        // The row is requested as soon as its position is known: before the labels have
        // arrived, and long before wavefront 0 has worked out where it goes.
        Tile<U, NT, TPB, step_pace(ST, U), stored_cv(ST, CV_NARROW), true, true, STREAM> t;
        t.load(a.batch_x + (int64_t)p * a.row_vec * stored_wide(ST), v_lo, v_hi);
        if (!AUX && w0) draw = (int)below(sd, PURPOSE_EVICT, (uint32_t)x, (uint64_t)a.S);
        park_labels<false>(yv, batch_y, b, a.K, s_y);
        if (direct) *reinterpret_cast<int4*>(s_old + 4 * tid) = fo;
        lds_barrier();
        if (w0) {
            k = candidate_class(a, active, x, s_y, yx);
            const int64_t dst = place(i, p);
            if (lane == 0) s_dst[0] = dst;
        }
        lds_barrier();
        const int64_t dst_row = s_dst[0];
        if (dst_row >= 0) {
            t.store(a.buf_x + dst_row * a.row_vec, v_lo, v_hi);
            if (tile == 0 && tid == 0) { a.buf_y[dst_row] = dst_row / a.S; count_moved(a.state); }
        }
    }
    for (int rr = 1; rr < a.rpb; ++rr) {
        const int i = group * a.rpb + rr;
        if (i >= c) break;
        const int par = rr & 1;
        if (w0) {
            const int pi = lane_read(x, i);
            if (lane == 0) s_p[par] = pi;
        }
        __syncthreads();
        const int p = s_p[par];
        Tile<U, NT, TPB, step_pace(ST, U), stored_cv(ST, CV_NARROW), true, true, STREAM> t;
        t.load(a.batch_x + (int64_t)p * a.row_vec * stored_wide(ST), v_lo, v_hi);
        if (w0) {
            const int64_t dst = place(i, p);
            if (lane == 0) s_dst[par] = dst;
        }
        __syncthreads();
        const int64_t dst_row = s_dst[par];
        if (dst_row >= 0) {
            t.store(a.buf_x + dst_row * a.row_vec, v_lo, v_hi);
            if (tile == 0 && tid == 0) { a.buf_y[dst_row] = dst_row / a.S; count_moved(a.state); }
        }
    }
}

// ---------------------------------------------------------------------------
// rb_sample_augment for r <= WAVE representatives and at most WAVE chunks of
// classes.  Up to DIRECT_CHUNKS chunks each of the four wavefronts reads the counts
// of one chunk (four consecutive classes per lane; as many as there are chunks), the one whose chunk
// holds the wanted sample finds its class; above, wavefront 0 reads the sums of all chunks and
// then the CH counts of the one that holds the sample.  (Four classes per lane are one LDS or memory access without bank conflicts
// and three comparisons; one wavefront with sixteen consecutive classes per lane took 1 us longer.  With rb_update_small_kernel,
// both calls, us before and after: 4 + 4 rows of 12 KB 7.29 -> 6.49, 64 + 64 of 301 KB 17.75 -> 16.85, 31 + 22 of 370 KB 13.2 -> 11.8.)
// ---------------------------------------------------------------------------
template <int U, bool NT, int ST, bool STREAM = NT, int PACE = step_pace(ST, U)>
__global__ void __launch_bounds__(TPB) rb_sample_small_kernel(const int32_t* fill, const int32_t* chunk, uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi,
                                                              int32_t r, int32_t nchunks, const SampleArgs a)
{
    const Seed sd = {seed_lo, seed_hi, step_lo, step_hi};
    __shared__ int s_pick[2][2];    // (class, slot) of the current row, double-buffered over rows
    __shared__ __align__(16) int s_tot[DIRECT_CHUNKS];

    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const bool direct = nchunks <= DIRECT_CHUNKS;
    static_assert(DIRECT_CHUNKS == NWAVE && CH == 4 * WAVE, "a chunk per wavefront, four classes per lane");

    // The wavefronts that plan: one per chunk of classes, or the first alone (no more than that have anything to add, and with three
    // and more workgroups on a compute unit they take issue slots from the others' planners: 40 rows of 301 KB in 8 bits, 1025
    // classes, 5.85 us with four of them and 4.95 with one; 64 of 203 KB, 10 classes, 6.5 and 6.0).
    const bool plans = wave < (direct ? nchunks : 1);
    WaveFill mine;
    uint64_t bits = 0;
    int cs = 0, cincl = 0;          // not direct: samples in chunk `lane`, and up to it
    int F = 0, before = 0;          // stored samples; direct: of the chunks before this wavefront's
    if (plans) {
        // the fill counts are requested first; the random bits do not depend on them
        // (only their reduction to [0, F-n+i] does) and are computed while the loads fly
        int4 fo = make_int4(0, 0, 0, 0);
        if (direct) fo = request_fill(fill, nchunks);
        else if (lane < nchunks) cs = chunk[lane];
        bits = draw64(sd, PURPOSE_SAMPLE, (uint32_t)lane);
        // (keeps the compiler from moving the draw down to its only use, behind the wait for the counts, the scan and the barrier:
        // rb_sample_augment alone, 4 rows of 8 KB 3.1 -> 2.8 us, 16 of 99 KB 3.55 -> 3.3, 7 of 602 KB 4.2 -> 3.9)
        asm volatile("" : "+v"(bits));
        if (direct) mine = WaveFill(fo);
        else cincl = wave_scan_incl(cs);
    }
    if (direct) {
        if (lane == WAVE - 1) s_tot[wave] = plans ? mine.incl : 0;
        lds_barrier();
    }
    int n = 0, base = 0;
    uint32_t t = 0xFFFFFFFFu;       // Floyd draw `lane`
    if (plans) {
        if (direct) {
            const int4 tot = *reinterpret_cast<const int4*>(s_tot);
            before = __builtin_amdgcn_readfirstlane((wave > 0 ? tot.x : 0) + (wave > 1 ? tot.y : 0) + (wave > 2 ? tot.z : 0));
            F = __builtin_amdgcn_readfirstlane(tot.x + tot.y + tot.z + tot.w);
        } else {
            F = lane_read(cincl, WAVE - 1);
        }
        n = r < F ? r : F;
        base = F - n;
        if (lane < n) t = reduce32(bits, (uint32_t)base + lane + 1);
        if (blockIdx.x == 0 && tid == 0) a.state->last_n = n;
    }

    const int group = blockIdx.x / a.tpr, tile = blockIdx.x % a.tpr;
    int64_t v_lo, v_hi;
    tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);

    for (int rr = 0; rr < a.rpb; ++rr) {
        const int j = group * a.rpb + rr;      // output row
        if (j >= r) break;
        const int par = rr & 1;
        if (plans && j < n) {
            int owner, sub, ps;
            const int g = wave_sample_number(t, j, base) - before;
            if (direct) {
                if (g >= 0 && g < mine.total()) {                     // in this wavefront's chunk
                    mine.locate(g, owner, sub, ps);
                    if (lane == 0) { s_pick[par][0] = wave * CH + 4 * owner + sub; s_pick[par][1] = ps; }
                }
            } else {
                // chunk holding it: the number of chunks that end at or before it
                const int ch = __popcll(__ballot(lane < nchunks && cincl <= g));
                const WaveFill in(*reinterpret_cast<const int4*>(fill + (int64_t)ch * CH + 4 * lane));
                in.locate(g - (lane_read(cincl, ch) - lane_read(cs, ch)), owner, sub, ps);
                if (lane == 0) { s_pick[par][0] = ch * CH + 4 * owner + sub; s_pick[par][1] = ps; }
            }
        } else if (tid == 0) {
            s_pick[par][0] = -1;               // fewer stored samples than asked for
        }
        lds_barrier();
        const int pk = __builtin_amdgcn_readfirstlane(s_pick[par][0]), ps = s_pick[par][1];
        if (pk < 0) {
            if (tile == 0 && tid == 0) a.out_y[j] = -1;
            continue;
        }
        Tile<U, NT, TPB, PACE, stored_cv(ST, CV_WIDEN), false, true, STREAM> t2;
        t2.load(a.buf_x + ((int64_t)pk * a.S + ps) * a.row_vec, v_lo, v_hi);
        t2.store(a.out_x + (int64_t)j * a.row_vec * stored_wide(ST), v_lo, v_hi);
        if (tile == 0 && tid == 0) { a.out_y[j] = pk; count_moved(a.state); }
    }
}

// ---------------------------------------------------------------------------
// rb_update_sample, c <= WAVE, r <= WAVE, at most DIRECT_CHUNKS chunks of
// classes, exact selection: update and sampling of one step in ONE launch, with
// any replacement strategy and storage form.  What bounds it is the chain from
// the labels to the rows' addresses and the launch itself, so a second dependent
// launch is the thing to avoid.  Of the 4.1 us that 16 + 16 rows of 12 KB take, 1.2 lie between two launches and 1.8 go by
// before a representative's row is requested: 0.7 for the selection, during which the labels arrive, 0.3 for classes and counts,
// 0.3 for draws, 0.3 to find the sample and whether the step writes it.  Measured on MI355X, this launch against the two of
// the calls: 16 + 16 rows of 12 KB 4.1 : 6.6 us, 14 + 7 of 602 KB 6.9 : 8.8; before one chunk of classes per wavefront took the place of
// one wavefront with sixteen classes per lane: 16 + 16 rows of 12 KB 5.2, 14 + 7 of 602 KB 7.9, 64 + 64 of 301 KB 15.75 (15.25 now),
// 8 + 8 of 602 KB in 8 bits 6.45 (5.2 now).  With binary32 samples stored in fewer bits the vectors
// are converted when they are stored: a conversion at the load would wait for
// the row before its destination is worked out.
//
// Grid: bookkeeping workgroups, then the movers of the c candidate rows
// (exactly as in rb_update_small_kernel: their rows are read while the others plan; representatives
// first: 14 + 7 rows of 602 KB 7.0 -> 7.6 us), then the movers of the r
// representative rows.  A representative mover cannot read the fill counts
// the bookkeeping workgroups of the same launch are writing, so it derives
// them itself: old counts + a histogram of this step's candidates, a chunk of classes
// per wavefront, four consecutive classes per lane.  A
// representative whose slot is written in this very step is copied from the
// mini-batch row that is being stored there ("forwarding"), never from the
// slot, so no workgroup reads a row another one is writing.
//
// LDS (dynamic): s_first[b], s_y[b] as in rb_update_small_kernel, then DIRECT_CHUNKS * CH words:
// candidate movers: fill counts before the step; representative movers: candidates of each class in this step.
// ---------------------------------------------------------------------------

template <int U, bool NT, int ST, bool AUX, bool STREAM = NT>     // STREAM: streaming stores
__global__ void __launch_bounds__(TPB) rb_step_small_kernel(const int64_t* batch_y, const int32_t* fill_old, uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi, uint32_t b_c,
                                                            uint32_t r_nchunks, int32_t tpr, int32_t first_gather, const StepArgs sa)
{
    const UpdateArgs& a = sa.u;
    const int b = (int)(b_c & 0xFFFFu), c = (int)(b_c >> 16), r = (int)(r_nchunks & 0xFFFFu), nchunks = (int)(r_nchunks >> 16);
    const Seed sd = {seed_lo, seed_hi, step_lo, step_hi};
    extern __shared__ uint32_t lds[];
    uint32_t* s_first = lds;                                       // [b]
    int32_t* s_y = reinterpret_cast<int32_t*>(lds + b);            // [b]
    int32_t* s_old = reinterpret_cast<int32_t*>(lds + ((2 * b + 3) & ~3));     // [DIRECT_CHUNKS * CH], 16-byte aligned
    int32_t* s_cnt = s_old;
    __shared__ int s_wave[NWAVE];
    __shared__ int s_hist[CH];
    __shared__ int s_p;             // candidate mover: mini-batch position of the row
    __shared__ int64_t s_dst;       // candidate mover: slot row it is stored to, -1: not stored
    __shared__ int s_x[WAVE];       // representative mover: the candidates' positions
    __shared__ uint64_t s_bits[WAVE];                  // ... random bits of sampling draw i, made by wavefront 1
    __shared__ __align__(16) int s_tot[NWAVE];         // ... samples in each chunk of classes
    __shared__ int s_pick[3];       // ... class, slot, forwarding position (-1: read the slot)

    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const bool gather = (int)blockIdx.x >= first_gather;

    // labels of the mini-batch and fill counts: requested now
    int64_t yv[YPRE];
    request_labels(yv, batch_y, b);
    const int4 fo = request_fill(fill_old, nchunks);

    // wavefront 0 selects the candidates while wavefront 1 makes the random bits of the sampling draws
    bool active = false;
    int x = 0;
    int64_t yx = -1;                // label of the lane's candidate, if it lies beyond the parked ones
    if (wave == 0) {
        x = wave_select(sd, b, c, s_first, active);
        yx = far_label(a, active, x);
    } else if (gather && wave == 1) {
        s_bits[lane] = draw64(sd, PURPOSE_SAMPLE, (uint32_t)lane);
    }

    if ((int)blockIdx.x < nchunks) {
        // ---- bookkeeping: fill_new = min(fill_old + candidates of the class, S) ----
        park_labels<false>(yv, batch_y, b, a.K, s_y);
        const int k_lo = blockIdx.x * CH;
        s_hist[tid] = 0;
        __syncthreads();
        if (wave == 0) {
            const int32_t k = candidate_class(a, active, x, s_y, yx);
            if (active && k >= k_lo && k < k_lo + CH) atomicAdd(&s_hist[k - k_lo], 1);
            if (blockIdx.x == 0 && __ballot(active && k == LAB_INVALID) != 0 && lane == 0)
                atomicOr(&a.state->flags, RB_FLAG_BAD_LABEL);
        }
        __syncthreads();
        const int kk = k_lo + tid;
        int32_t nf = 0;
        if (kk < a.K) {
            int64_t v = (int64_t)a.fill_old[kk] + s_hist[tid];
            nf = (int32_t)(v < a.S ? v : a.S);
            a.fill_new[kk] = nf;
            if (AUX) a.aux_new[kk] = next_aux(a, a.fill_old[kk], a.aux_old[kk], s_hist[tid]);
        }
        int total;
        block_scan_excl(nf, total, s_wave);
        if (tid == 0) a.chunk_new[blockIdx.x] = total;
        return;
    }

    if (!gather) {
        // ---- candidate movers (rows of the mini-batch into their slots) ----------
        const int mover = blockIdx.x - nchunks;
        const int i = mover / tpr, tile = mover % tpr;         // candidate in Floyd emission order, tile of its row
        int64_t v_lo, v_hi;
        tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);
        if (wave == 0) {
            const int pi = lane_read(x, i);
            if (lane == 0) s_p = pi;
        }
        lds_barrier();
        const int p = s_p;
        // requested as soon as the position is known, before the labels have arrived
        Tile<U, NT, TPB, step_pace(ST, U), stored_cv(ST, CV_NARROW), true, true, STREAM> t;
        t.load(a.batch_x + (int64_t)p * a.row_vec * stored_wide(ST), v_lo, v_hi);
        int draw = -1;                                         // (uniform replacement) the slot the lane's candidate overwrites if its class is full
        if (!AUX && wave == 0) draw = (int)below(sd, PURPOSE_EVICT, (uint32_t)x, (uint64_t)a.S);
        park_labels<false>(yv, batch_y, b, a.K, s_y);
        *reinterpret_cast<int4*>(s_old + 4 * tid) = fo;
        lds_barrier();
        if (wave == 0) {
            const int32_t k = candidate_class(a, active, x, s_y, yx);
            const int32_t ki = lane_read(k, i);
            const int64_t dst = wave_place<AUX>(a, active, x, k, draw, i, p, ki, ki < 0 ? 0 : s_old[ki]);
            if (lane == 0) s_dst = dst;
        }
        lds_barrier();
        const int64_t dst_row = s_dst;
        if (dst_row >= 0) {
            t.store(a.buf_x + dst_row * a.row_vec, v_lo, v_hi);
            if (tile == 0 && tid == 0) { a.buf_y[dst_row] = dst_row / a.S; count_moved(a.state); }
        }
        return;
    }

    // ---- representative movers (stored samples into the augmented mini-batch) ---
    const int mover = blockIdx.x - first_gather;
    const int j = mover / tpr, tile = mover % tpr;             // output row, tile of it
    int64_t v_lo, v_hi;
    tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);

    *reinterpret_cast<int4*>(s_cnt + 4 * tid) = make_int4(0, 0, 0, 0);
    park_labels<false>(yv, batch_y, b, a.K, s_y);
    if (wave == 0) {
        s_x[lane] = x;
        if (active && x >= YPRE * TPB) s_y[x] = candidate_class(a, true, x, s_y, yx);      // (the only labels behind the parked ones)
    }
    lds_barrier();
    // every wavefront: the candidates' classes, one lane each, and the new counts of its own chunk
    x = s_x[lane];
    active = lane < c;
    const uint64_t bits = s_bits[lane];
    const int32_t k = active ? s_y[x] : LAB_UNSELECTED;
    const int cap = (int)a.S;
    if (k >= 0 && k / CH == wave) atomicAdd(&s_cnt[k], 1);
    const int4 more = *reinterpret_cast<const int4*>(s_cnt + 4 * tid);
    const WaveFill mine(make_int4(capped_sum(fo.x, more.x, cap), capped_sum(fo.y, more.y, cap), capped_sum(fo.z, more.z, cap), capped_sum(fo.w, more.w, cap)));
    if (lane == WAVE - 1) s_tot[wave] = mine.incl;
    lds_barrier();
    const int4 tot = *reinterpret_cast<const int4*>(s_tot);
    const int before = __builtin_amdgcn_readfirstlane((wave > 0 ? tot.x : 0) + (wave > 1 ? tot.y : 0) + (wave > 2 ? tot.z : 0));
    const int F = __builtin_amdgcn_readfirstlane(tot.x + tot.y + tot.z + tot.w);
    const int n = r < F ? r : F, base = F - n;
    if (mover == 0 && tid == 0) a.state->last_n = n;
    if (j >= n) {                              // fewer stored samples than asked for
        if (tile == 0 && tid == 0) sa.out_y[j] = -1;
        return;
    }
    const uint32_t t = lane < n ? reduce32(bits, (uint32_t)base + lane + 1) : 0xFFFFFFFFu;      // Floyd draw `lane`
    const int g = wave_sample_number(t, j, base) - before;
    if (g >= 0 && g < mine.total()) {          // in this wavefront's chunk
        int owner, sub, ps;
        mine.locate(g, owner, sub, ps);
        const int pk = wave * CH + 4 * owner + sub;
        // Is slot ps of class pk written in this step, and by which candidate?
        const bool same = k == pk;
        const uint64_t same_mask = __ballot(same);
        int fwd = -1;
        if (same_mask != 0) {
            const int fill0 = lane_read(sub == 0 ? fo.x : sub == 1 ? fo.y : sub == 2 ? fo.z : fo.w, owner);
            if (ps >= fill0 || (uint32_t)fill0 + __popcll(same_mask) > (uint32_t)cap) {
                const int my_rank = rank_among(same_mask, x);          // class-mates earlier in the mini-batch
                int slot = -1;
                if (same) slot = mate_slot(a, x, my_rank, fill0, AUX ? a.aux_old[pk] : 0);
                uint64_t writers = __ballot(same && slot == ps);
                while (writers != 0) {                 // the one latest in the mini-batch is what the slot holds
                    const int m = __builtin_ctzll(writers);
                    writers &= writers - 1;
                    const int xm = __builtin_amdgcn_readlane(x, m);
                    fwd = xm > fwd ? xm : fwd;
                }
            }
        }
        if (lane == 0) { s_pick[0] = pk; s_pick[1] = ps; s_pick[2] = fwd; }
    }
    lds_barrier();
    const int pk = s_pick[0], ps = s_pick[1], fwd = s_pick[2];
    vec16* dst = sa.out_x + (int64_t)j * a.row_vec * stored_wide(ST);
    if (ST != RB_STORE_SAME && fwd >= 0) {
        // from the mini-batch: what the slot will hold is the row in its stored form
        Tile<U, NT, TPB, step_pace(ST, U), stored_cv(ST, CV_BOTH)> t;
        t.load(a.batch_x + (int64_t)fwd * a.row_vec * stored_wide(ST), v_lo, v_hi);
        t.store(dst, v_lo, v_hi);
    } else {
        const vec16* src = fwd >= 0 ? a.batch_x + (int64_t)fwd * a.row_vec
                                    : a.buf_x + ((int64_t)pk * a.S + ps) * a.row_vec;
        Tile<U, NT, TPB, step_pace(ST, U), stored_cv(ST, CV_WIDEN), false, true, STREAM> t;
        t.load(src, v_lo, v_hi);
        t.store(dst, v_lo, v_hi);
    }
    if (tile == 0 && tid == 0) { sa.out_y[j] = pk; count_moved(a.state); }
}

}  // namespace
