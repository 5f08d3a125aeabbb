// General kernels: buffer reset, rb_update and rb_sample_augment for any candidate / representative count and any policy variant.
// Included by rb.hip only, after rb_device.h.
#pragma once

#include "rb_device.h"

namespace {

// ---------------------------------------------------------------------------
// Reset: fill counts, partial sums and state words to zero, labels to -1.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(TPB) rb_reset_kernel(uint32_t* __restrict__ ws, int64_t ws_words,
                                                        int64_t* __restrict__ buf_y, int64_t slots)
{
    const int64_t stride = (int64_t)gridDim.x * TPB;
    const int64_t first = (int64_t)blockIdx.x * TPB + threadIdx.x;
    for (int64_t i = first; i < ws_words; i += stride) ws[i] = 0u;
    for (int64_t i = first; i < slots; i += stride) buf_y[i] = -1;
}

// ---------------------------------------------------------------------------
// rb_update: Algorithm 1, any c (used for c > WAVE).
//
// The whole workgroup first computes, once, what every candidate is (its
// mini-batch position and class) into LDS; then each of its four wavefronts
// takes one work item (candidate row, tile of WAVE * U vectors) and works out
// alone, with ballots over the candidate list, where that candidate goes.
//
// LDS (dynamic): s_k[cap] i32 (class per candidate, LAB_INVALID outside [0, K), LAB_UNSELECTED behind the list's end),
// s_x[cap] u16 (candidate positions, Floyd emission order or, with the Bernoulli selection, mini-batch order), both rounded up to GEN_LIST;
// with the exact selection also s_first[b] u32 (lowest candidate index that drew a value) and s_t[cap] u16 (Floyd draws).  cap = c, or b for
// Bernoulli.
//
// What bounds it, beside the rows: one wavefront per unit of a compute unit makes all draws, one chain of dependent multiplications behind the
// other, and every wavefront passes over the whole list.  Hence two draws side by side, the list read four candidates per lane and
// access, coins counted by ballots (a thread that walked its stretch of the mini-batch twice took 16 LDS accesses each time).
//
// Grid: `nchunks` bookkeeping workgroups (new fill counts and chunk sums for CH
// classes each), then ceil(c * tpr / NWAVE) mover workgroups.
// ---------------------------------------------------------------------------

constexpr int GEN_LIST = 4 * WAVE;          // the candidate list and the sampling draws are read this many at a time
__host__ __device__ inline int gen_padded(int n) { return (n + GEN_LIST - 1) / GEN_LIST * GEN_LIST; }
inline size_t gen_update_lds_bytes(int b, int cap, bool bernoulli) { return (size_t)gen_padded(cap) * 6 + (bernoulli ? 0 : (size_t)b * 4 + (size_t)cap * 2); }
inline size_t gen_sample_lds_bytes(int r, int nchunks) { return 4 * (size_t)(nchunks + r > ((r + 3) & ~3) ? nchunks + r : (r + 3) & ~3); }

// Lane `lane` looks at four consecutive candidates of every GEN_LIST: number `bit` of its candidates is this one of the list.
__device__ __forceinline__ int gen_entry(int bit, int lane) { return (bit >> 2) * GEN_LIST + 4 * lane + (bit & 3); }

// A kernel per form of the selection: exact with few candidates (gen_few), exact with more, Bernoulli.  (Two draws side by side and four
// candidates per access: 300 to 500 candidates 3 % faster, 500 to 2048 9 to 12 %, more 30 %, but 65 to 128 2 % slower, 128 to 200 1 %, 200 to 300 equal.
// Coins counted by ballots: mini-batches of 256 to 1024 5 % faster, 1024 to 2048 7 %, more 12 %, smaller ones equal.)
enum { GEN_EXACT_FEW = 0, GEN_EXACT_MANY = 1, GEN_COINS = 2 };
// Few are more when rows are long: the wavefronts of GEN_EXACT_MANY, sooner done with the list, get in each other's way where 300 to 700
// workgroups move rows of 16 KB and more (the same rows with plain stores take as long as before).  Which kernel is ahead changes from shape to
// shape.  Few against many over 16000 shapes of 193 to 512 candidates, rows of 16 KB and more: FIFO replacement, which makes no draws behind the
// list, 1.01 to 1.03 by range and storage form, at most 3 of 100 more than 3 % slower (388 of 83 KB 14.5 : 15.8 us); else plain rows, up to 320 candidates, 1.00 to 1.01
// (3 of 100), beyond 0.98 to 1.01 (up to 30 of 100); converted ones 0.99 to 1.00 (up to 16).
constexpr int GEN_FEW = 192, GEN_FEW_LONG = 320, GEN_FEW_LONG_FIFO = 512;
constexpr int64_t GEN_LONG_VEC = 1024;
inline bool gen_few(int c, int64_t row_vec, bool converted, int eviction)
{
    if (row_vec < GEN_LONG_VEC) return c <= GEN_FEW;
    return c <= (eviction == RB_EVICT_FIFO ? GEN_FEW_LONG_FIFO : converted ? GEN_FEW : GEN_FEW_LONG);
}
// Lists of this many candidates: the later class-mates of a class with many in this step are gathered for their draws.  They are dealt to the lanes
// unevenly, and of 300 candidates of three classes a lane holds up to eight: 283 + 3 classes 10.1 us, 11.1 with a draw per candidate a lane holds
// (which is as fast from about 400 on, where the list's passes count).
constexpr int GEN_GATHERED = 384;

template <int U, bool NT, int NARROW, int FORM>       // NARROW: binary32 mini-batch rows are stored 0 - as they come, 1 - as bfloat16, 2 - in 8 bits per element
__global__ void __launch_bounds__(TPB) rb_update_kernel(const UpdateArgs a)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const int listed = gen_padded(a.cap);
    int32_t* s_k = reinterpret_cast<int32_t*>(lds);                   // [listed]
    uint16_t* s_x = reinterpret_cast<uint16_t*>(lds + listed);        // [listed]
    uint32_t* s_first = lds + listed + listed / 2;                    // [b]
    uint16_t* s_t = reinterpret_cast<uint16_t*>(s_first + a.b);       // [cap]
    __shared__ int s_wave[NWAVE];
    __shared__ int s_hist[CH];
    __shared__ int s_seg[WAVE];                             // Bernoulli: heads per stretch of WAVE positions
    __shared__ uint16_t s_pend[NWAVE][2 * WAVE];            // per wavefront: the class-mates, one per lane, or later ones waiting for their evict draw
    __shared__ uint32_t s_cm[NWAVE][RB_MAX_BATCH / 32];     // per wavefront: bitmap of the class-mates' positions
    __shared__ uint16_t s_cmpre[NWAVE][RB_MAX_BATCH / 32];  // class-mates before each bitmap word

    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int b = a.b, c = a.c;
    int m;      // number of candidates of this step (the same in every workgroup)

    if constexpr (FORM == GEN_COINS) {
        // ---- one coin per sample, heads with probability c/b; candidates in mini-batch order ----
        // All labels are requested first (coalesced, MAX_PER = RB_MAX_BATCH / TPB per thread) so that their memory round trip overlaps
        // the coin draws.
        constexpr int MAX_PER = RB_MAX_BATCH / TPB;
        int64_t yl[MAX_PER];
#pragma unroll
        for (int u = 0; u < MAX_PER; ++u) {
            const int q = tid + u * TPB;
            yl[u] = q < b ? a.batch_y[q] : -1;
        }
        uint32_t heads = 0;                    // bit u: the coin of sample tid + u * TPB
#pragma unroll 1
        for (int u = 0; u * TPB < b; u += 2) {
            const int q0 = tid + u * TPB, q1 = q0 + TPB;
            uint64_t d0, d1 = 0;
            const bool second = (u + 1) * TPB < b;
            if (second) {                      // (two at a time)
                d0 = draw64(a.sd, PURPOSE_COIN, (uint32_t)q0);
                d1 = draw64(a.sd, PURPOSE_COIN, (uint32_t)q1);
            } else {
                d0 = draw64(a.sd, PURPOSE_COIN, (uint32_t)q0);
            }
            const bool head0 = q0 < b && (int)reduce32(d0, (uint32_t)b) < c, head1 = q1 < b && (int)reduce32(d1, (uint32_t)b) < c;
            heads |= (uint32_t)head0 << u | (uint32_t)head1 << (u + 1);
            const int in0 = __popcll(__ballot(head0)), in1 = __popcll(__ballot(head1));
            if (lane == 0) {
                s_seg[u * NWAVE + wave] = in0;
                s_seg[(u + 1) * NWAVE + wave] = in1;
            }
        }
        __syncthreads();
        static_assert(MAX_PER * NWAVE == WAVE && MAX_PER % 2 == 0, "one lane per stretch of positions, pairs of them");
        const int incl = wave_scan_incl(lane < (b + TPB - 1) / TPB * NWAVE ? s_seg[lane] : 0);
        m = lane_read(incl, WAVE - 1);
#pragma unroll
        for (int u = 0; u < MAX_PER; ++u) {
            if (u * TPB >= b) break;
            const bool mine = (heads >> u) & 1;
            const uint64_t seg_heads = __ballot(mine);
            const int at = lane_read(incl, u * NWAVE + __builtin_amdgcn_readfirstlane(wave)) - __popcll(seg_heads >> lane);     // (the sum less this one and the heads behind it)
            if (mine) {
                s_x[at] = (uint16_t)(tid + u * TPB);
                s_k[at] = yl[u] >= 0 && yl[u] < a.K ? (int32_t)yl[u] : LAB_INVALID;
            }
        }
    } else {
        // ---- candidate selection: Floyd's c-subset of [0, b), all draws at once --
        // Draw i is t_i in [0, b-c+i]; it is "taken" iff an earlier draw had the same
        // value, or it equals b-c+q for an earlier q whose own draw was taken; a
        // taken draw is replaced by b-c+i.
        m = c;
        const int base = b - c;
        // s_first[v] = lowest candidate index that drew v: only the entries that are drawn at all
        // are initialised (by every thread that drew them), then minimised
        // (of a large mini-batch the labels are near when the candidates' are asked for: one load per 64 bytes)
        static_assert(RB_MAX_BATCH * sizeof(int64_t) / 64 <= 2 * TPB, "two loads per thread");
        int64_t near0 = 0, near1 = 0;
        if (FORM == GEN_EXACT_MANY && b > 4 * TPB) {
            near0 = a.batch_y[min(8 * tid, b - 1)];
            near1 = a.batch_y[min(8 * (tid + TPB), b - 1)];
        }
        if constexpr (FORM == GEN_EXACT_FEW) {
            for (int i = tid; i < c; i += TPB) {
                uint32_t t = (uint32_t)below(a.sd, PURPOSE_SELECT, (uint32_t)i, (uint64_t)(base + i + 1));
                s_t[i] = (uint16_t)t;
                s_first[t] = 0xFFFFFFFFu;
            }
        } else {
#pragma unroll 1
            for (int i0 = tid; i0 < c; i0 += 2 * TPB) {
                const int i1 = i0 + TPB;
                if (__builtin_amdgcn_readfirstlane(i1) < c) {       // (two at a time)
                    const uint64_t d0 = draw64(a.sd, PURPOSE_SELECT, (uint32_t)i0), d1 = draw64(a.sd, PURPOSE_SELECT, (uint32_t)i1);
                    const uint32_t t0 = reduce32(d0, (uint32_t)(base + i0 + 1)), t1 = reduce32(d1, (uint32_t)(base + i1 + 1));
                    s_t[i0] = (uint16_t)t0;
                    s_first[t0] = 0xFFFFFFFFu;
                    if (i1 < c) { s_t[i1] = (uint16_t)t1; s_first[t1] = 0xFFFFFFFFu; }
                } else {
                    const uint32_t t0 = reduce32(draw64(a.sd, PURPOSE_SELECT, (uint32_t)i0), (uint32_t)(base + i0 + 1));
                    s_t[i0] = (uint16_t)t0;
                    s_first[t0] = 0xFFFFFFFFu;
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < c; i += TPB) atomicMin(&s_first[s_t[i]], (uint32_t)i);
        __syncthreads();
        for (int i = tid; i < c; i += TPB) {
            int cur = i;
            bool taken = false;
            for (;;) {
                int t = s_t[cur];
                if (s_first[t] != (uint32_t)cur) { taken = true; break; }   // an earlier draw had this value
                int q = t - base;                                           // the step whose fallback value is t
                if (q < 0 || q >= cur) break;
                cur = q;                                                    // taken iff that step fell back
            }
            s_x[i] = (uint16_t)(taken ? base + i : (int)s_t[i]);
        }
        // the candidates' labels, four loads in flight per thread
        if (FORM == GEN_EXACT_MANY) asm volatile("" : : "v"(near0), "v"(near1));
        for (int i0 = tid; i0 < c; i0 += 4 * TPB) {
            int64_t y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * TPB;
                y[u] = i < c ? a.batch_y[s_x[i]] : -1;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * TPB;
                if (i < c) s_k[i] = (y[u] >= 0 && y[u] < a.K) ? (int32_t)y[u] : LAB_INVALID;
            }
        }
    }
    if (FORM != GEN_EXACT_FEW)
        for (int q = m + tid; q < gen_padded(m); q += TPB) s_k[q] = LAB_UNSELECTED;
    __syncthreads();

    if ((int)blockIdx.x < a.nchunks) {
        // ---- bookkeeping: fill_new = min(fill_old + candidates of the class, S) ----
        const int k_lo = blockIdx.x * CH;
        s_hist[tid] = 0;
        __syncthreads();
        bool bad = false;
        for (int i = tid; i < m; i += TPB) {
            const int32_t k = s_k[i];
            if (k >= k_lo && k < k_lo + CH) atomicAdd(&s_hist[k - k_lo], 1);
            bad |= (k == LAB_INVALID);
        }
        __syncthreads();
        const int k = k_lo + tid;
        int32_t nf = 0;
        if (k < a.K) {
            const int64_t old = a.fill_old[k];
            const int64_t v = old + s_hist[tid];
            nf = (int32_t)(v < a.S ? v : a.S);
            a.fill_new[k] = nf;
            if (a.eviction == RB_EVICT_FIFO) {
                // the oldest sample moves on by the number of overwrites
                const int64_t over = v > a.S ? v - a.S : 0;
                a.aux_new[k] = (int32_t)(((int64_t)a.aux_old[k] + over) % a.S);
            } else if (a.eviction == RB_EVICT_RESERVOIR) {
                const int64_t seen = (int64_t)a.aux_old[k] + s_hist[tid];
                a.aux_new[k] = (int32_t)(seen < INT32_MAX ? seen : INT32_MAX);
            }
        }
        int total;
        block_scan_excl(nf, total, s_wave);
        if (tid == 0) a.chunk_new[blockIdx.x] = total;
        if (blockIdx.x == 0 && bad) atomicOr(&a.state->flags, RB_FLAG_BAD_LABEL);
        return;
    }

    // ---- movers: one work item per wavefront and round, no workgroup barrier from here on ----
    const int64_t stride = (int64_t)(gridDim.x - a.nchunks) * NWAVE;
    for (int64_t item = (int64_t)(blockIdx.x - a.nchunks) * NWAVE + wave; item < (int64_t)m * a.tpr; item += stride) {
        int i, tile;                           // candidate, tile of its row
        split_item(item, a.tpr, i, tile);
        const int p = s_x[i];                                             // its mini-batch position
        const int32_t ki = s_k[i];
        if (ki < 0) continue;                  // label outside [0, K): dropped (flagged by bookkeeping)
        int64_t v_lo, v_hi;
        tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);

        const int64_t fill0 = a.fill_old[ki];
        const int64_t aux0 = a.eviction != RB_EVICT_UNIFORM ? a.aux_old[ki] : 0;
        // the row is read while the wavefront works out where it goes
        // (8-bit rows are converted when they are stored: at the load the conversion would wait for the row before its place is
        // worked out.  10 + 9 rows of 384 KB, both calls: 14.4 -> 10.8 us; 100 + 90 rows of 602 KB 47.3 -> 34.3 with two vectors
        // per lane.  bfloat16 rows do the same either way and keep half the registers.)
        Tile<U, NT, WAVE, false, NARROW == 2 ? CV_NARROW8 : NARROW ? CV_NARROW : CV_NONE, NARROW == 2> t;
        t.load(a.batch_x + (int64_t)p * a.row_vec * (NARROW == 2 ? 4 : NARROW ? 2 : 1), v_lo, v_hi);

        // Candidates of class ki, in mini-batch order: the one with `rank` class-mates before it is
        // insertion number fill0 + rank of the class.  Each lane looks at four of every GEN_LIST candidates,
        // remembers in a bit mask which of them are class-mates, and the counts are summed over the
        // wavefront once at the end (no ballot, hence no scalar dependency, per round).
        uint64_t hit = 0;                      // bit i: candidate entry(i) is a class-mate (m <= 64 * WAVE)
        int my_rank = 0;
        // (a list of up to two candidates per lane: one of every WAVE, else few lanes hold most class-mates; 72 candidates of 2 classes
        // 5.66 us, 5.95 with four per lane)
        const bool wide = FORM == GEN_EXACT_MANY || (FORM == GEN_COINS && m > 2 * WAVE);
        const auto entry = [&](int bit) { return wide ? gen_entry(bit, lane) : bit * WAVE + lane; };
        if (wide) {
#pragma unroll 2
            for (int m0 = 0; m0 < m; m0 += GEN_LIST) {
                const int4 kq = *reinterpret_cast<const int4*>(s_k + m0 + 4 * lane);
                const ushort4 xq = *reinterpret_cast<const ushort4*>(s_x + m0 + 4 * lane);
                const uint32_t same = (kq.x == ki ? 1u : 0u) | (kq.y == ki ? 2u : 0u) | (kq.z == ki ? 4u : 0u) | (kq.w == ki ? 8u : 0u);
                hit |= (uint64_t)same << (m0 / WAVE);
                my_rank += (kq.x == ki && xq.x < p) + (kq.y == ki && xq.y < p) + (kq.z == ki && xq.z < p) + (kq.w == ki && xq.w < p);
            }
        } else {
            for (int m0 = 0, round = 0; m0 < m; m0 += WAVE, ++round) {
                const int q = m0 + lane;
                const bool same = q < m && s_k[q] == ki;
                const int xq = q < m ? s_x[q] : 0;
                hit |= (uint64_t)same << round;
                my_rank += same && xq < p;
            }
        }
        const int mine = __popcll(hit);
        const int incl = wave_scan_incl(mine | (my_rank << 16));      // both sums are <= 4096
        const int total = lane_read(incl, WAVE - 1) & 0xFFFF, rank = lane_read(incl, WAVE - 1) >> 16;
        int64_t slot;
        if (fill0 + total <= a.S) {
            slot = fill0 + rank;               // all of them append: distinct slots
        } else if (a.eviction == RB_EVICT_FIFO) {
            // insertion number fill0 + rank overwrites the oldest sample once the class is full; it is
            // itself overwritten in this step if a class-mate comes a whole round of S later
            const int64_t at = fill0 + rank;
            if (at + a.S < fill0 + total) continue;
            slot = at < a.S ? at : (aux0 + at - a.S) % a.S;
        } else if (total <= WAVE) {
            // Insertions beyond the capacity overwrite a uniformly drawn slot (or, with reservoir
            // sampling, are kept with probability S / offers).  This candidate is not stored if a
            // later class-mate overwrites its slot.  The usual case: every class-mate gets a lane
            // (in no particular order), which works out its insertion number (class-mates before it)
            // and, if it overwrites, the slot it draws.
            const bool reservoir = a.eviction == RB_EVICT_RESERVOIR;
            uint16_t* pend = s_pend[wave];
            int at = (incl & 0xFFFF) - mine;
            for (uint64_t h = hit; h != 0; h &= h - 1) pend[at++] = s_x[entry(__builtin_ctzll(h))];
            wave_lds_wait();
            const bool has = lane < total;
            const int xl = has ? pend[lane] : 0;
            int rl = 0;
            for (int j = 0; j < total; ++j) rl += lane_read(xl, j) < xl;
            const bool draws = has && xl >= p && fill0 + rl >= a.S;     // this candidate and the later ones
            int dr = -1;
            if (draws) {
                const int64_t offers = aux0 + rl < INT32_MAX ? aux0 + rl : INT32_MAX;   // to the class, before this one
                dr = (int)below(a.sd, PURPOSE_EVICT, (uint32_t)xl, reservoir ? (uint64_t)offers + 1 : (uint64_t)a.S);
            }
            int64_t own = fill0 + rank;
            if (own >= a.S) {
                const int me = __builtin_ctzll(__ballot(has && xl == p) | (1ull << 63));
                own = lane_read(dr, me);
                if (own >= a.S) continue;      // reservoir: not kept
            }
            if (__ballot(draws && xl > p && dr == (int)own) != 0) continue;
            slot = own;
        } else {
            // the same for a class with more than WAVE candidates in this step
            const bool reservoir = a.eviction == RB_EVICT_RESERVOIR;
            int64_t own = fill0 + rank;
            if (own >= a.S) {
                const int64_t offers = aux0 + rank < INT32_MAX ? aux0 + rank : INT32_MAX;   // to the class, before this one
                own = (int64_t)below(a.sd, PURPOSE_EVICT, (uint32_t)p, reservoir ? (uint64_t)offers + 1 : (uint64_t)a.S);
                if (own >= a.S) continue;      // reservoir: not kept
            }
            // bitmap of the class-mates' positions: rank of a position = class-mates below it
            uint32_t* cm = s_cm[wave];
            uint16_t* cmpre = s_cmpre[wave];
            cm[2 * lane] = 0u;
            cm[2 * lane + 1] = 0u;
            wave_lds_wait();                   // (else a lane without class-mates takes its words for the zeros it wrote)
            for (uint64_t h = hit; h != 0; h &= h - 1) {
                const int x = s_x[entry(__builtin_ctzll(h))];
                atomicOr(&cm[x >> 5], 1u << (x & 31));
            }
            wave_lds_wait();
            {
                const int p0 = __popc(cm[2 * lane]), p1 = __popc(cm[2 * lane + 1]);
                const int before = wave_scan_incl(p0 + p1) - (p0 + p1);
                cmpre[2 * lane] = (uint16_t)before;
                cmpre[2 * lane + 1] = (uint16_t)(before + p0);
            }
            wave_lds_wait();
            const auto takes = [&](int x) {    // whether the later class-mate at x overwrites this candidate's slot
                // the rival's insertion number decides whether it overwrites at all, and (reservoir) its odds
                const int rank_r = cmpre[x >> 5] + __popc(cm[x >> 5] & ((1u << (x & 31)) - 1u));
                if (fill0 + rank_r < a.S) return false;
                const int64_t offers = aux0 + rank_r < INT32_MAX ? aux0 + rank_r : INT32_MAX;
                return (int64_t)below(a.sd, PURPOSE_EVICT, (uint32_t)x, reservoir ? (uint64_t)offers + 1 : (uint64_t)a.S) == own;
            };
            bool beaten = false;
            if (FORM == GEN_EXACT_FEW || m <= GEN_GATHERED) {
                // they are gathered WAVE at a time so that their draws are made with full wavefronts
                uint16_t* pend = s_pend[wave];
                int npend = 0;
                for (int m0 = 0; m0 < m + WAVE && !beaten; m0 += WAVE) {
                    if (m0 < m) {
                        const int q = m0 + lane;
                        const int xq = q < m ? s_x[q] : 0;
                        const bool later = q < m && s_k[q] == ki && xq > p;
                        const uint64_t mask = __ballot(later);
                        if (later) pend[npend + __popcll(mask & ((1ull << lane) - 1))] = (uint16_t)xq;
                        npend += __popcll(mask);
                    }
                    if (npend >= WAVE || (m0 >= m && npend > 0)) {
                        wave_lds_wait();
                        const int take = npend < WAVE ? npend : WAVE;
                        beaten = __ballot(lane < take && takes(pend[lane])) != 0;
                        const int rest = lane + take < npend ? pend[lane + take] : 0;    // at most WAVE - 1 left over
                        wave_lds_wait();
                        if (lane + take < npend) pend[lane] = (uint16_t)rest;
                        npend -= take;
                    }
                }
            } else {
                // every lane draws for those it holds: the list is dealt to the lanes evenly
                for (uint64_t h = hit; !beaten && __ballot(h != 0) != 0; h &= h - 1) {
                    const int x = h != 0 ? (int)s_x[entry(__builtin_ctzll(h))] : -1;
                    beaten = __ballot(x > p && takes(x)) != 0;
                }
            }
            if (beaten) continue;
            slot = own;
        }
        const int64_t dst_row = (int64_t)ki * a.S + slot;
        t.store(a.buf_x + dst_row * a.row_vec, v_lo, v_hi);
        if (tile == 0 && lane == 0) { a.buf_y[dst_row] = ki; count_moved(a.state); }
    }
}

// ---------------------------------------------------------------------------
// rb_sample_augment: n = min(r, F) distinct stored samples, uniformly; any r
// and any number of classes (used when r > WAVE or there are more than WAVE
// chunks of classes).
//
// The workgroup computes F, the number of stored samples before every chunk of
// CH classes, and all n Floyd draws into LDS once; then each wavefront takes
// one work item (output row, tile of WAVE * U vectors): it decides whether its
// draw is taken, finds the chunk that holds the wanted sample, reads that
// chunk's CH fill counts (four consecutive classes per lane) and moves its tile.
//
// What bounds it, beside the rows: the draws (up to 16 per thread; of more than BIG_MAX two at a time, the first two while the chunk sums
// travel: 2000 rows of 4 KB of 300 classes 9.8 -> 8.2 us) and the chain draw -> chunk -> fill counts -> row.
//
// LDS (dynamic): s_t[r] u32, s_cpre[nchunks] i32.
// Grid: ceil(r * tpr / NWAVE) workgroups.
// ---------------------------------------------------------------------------

// MANY: of more than BIG_MAX representatives, of as many slots at least (1024 to 2048 7 % faster, more 14 %; up to 256 as fast or 1 % slower; of
// fewer slots most draws are never needed: 747 of 18 slots 6.2 us, 8.7 with the first ones made in front).
template <int U, bool NT, int WIDEN, bool MANY>        // WIDEN: rows are handed out 0 - as stored, 1 - widened from bfloat16, 2 - from 8 bits per element to binary32
__global__ void __launch_bounds__(TPB) rb_sample_kernel(const SampleArgs a)
{
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t* s_t = lds;                                  // [r]
    int32_t* s_cpre = reinterpret_cast<int32_t*>(lds + a.r);    // [nchunks]
    __shared__ int s_wave[NWAVE];

    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = MANY ? __builtin_amdgcn_readfirstlane(tid / WAVE) : tid / WAVE;

    // ---- F and the number of stored samples before every chunk, with many the random bits of the first draws meanwhile ----
    const int cper = (a.nchunks + TPB - 1) / TPB;
    uint64_t bits0 = 0, bits1 = 0;                        // of the draws tid and tid + TPB
    int csum = 0;
    for (int u = 0; u < cper; ++u) {
        int ch = tid * cper + u;
        if (ch < a.nchunks) csum += a.chunk[ch];
    }
    if constexpr (MANY) {
        bits0 = draw64(a.sd, PURPOSE_SAMPLE, (uint32_t)tid);
        bits1 = draw64(a.sd, PURPOSE_SAMPLE, (uint32_t)(tid + TPB));
        asm volatile("" : "+v"(bits0), "+v"(bits1));      // (here, not where they are used)
    }
    int F;
    int cbefore = block_scan_excl(csum, F, s_wave);
    for (int u = 0; u < cper; ++u) {
        int ch = tid * cper + u;
        if (ch < a.nchunks) {
            s_cpre[ch] = cbefore;
            cbefore += a.chunk[ch];
        }
    }
    const int n = a.r < F ? a.r : F;
    if (blockIdx.x == 0 && tid == 0) a.state->last_n = n;

    // ---- Floyd's n-subset of [0, F): all draws ----------------------------------
    const int base = F - n;
    if constexpr (MANY) {
        if (tid < n) s_t[tid] = reduce32(bits0, (uint32_t)base + (uint32_t)tid + 1u);
        if (tid + TPB < n) s_t[tid + TPB] = reduce32(bits1, (uint32_t)(base + tid + TPB) + 1u);
#pragma unroll 1
        for (int u = 2; wave * WAVE + u * TPB < n; u += 2) {
            const int i0 = tid + u * TPB, i1 = i0 + TPB;
            if (wave * WAVE + (u + 1) * TPB < n) {
                const uint64_t d0 = draw64(a.sd, PURPOSE_SAMPLE, (uint32_t)i0), d1 = draw64(a.sd, PURPOSE_SAMPLE, (uint32_t)i1);
                s_t[i0] = reduce32(d0, (uint32_t)base + (uint32_t)i0 + 1u);
                if (i1 < n) s_t[i1] = reduce32(d1, (uint32_t)base + (uint32_t)i1 + 1u);
            } else if (i0 < n) {
                s_t[i0] = reduce32(draw64(a.sd, PURPOSE_SAMPLE, (uint32_t)i0), (uint32_t)base + (uint32_t)i0 + 1u);
            }
        }
    } else {
        for (int i = tid; i < n; i += TPB)
            s_t[i] = (uint32_t)below(a.sd, PURPOSE_SAMPLE, (uint32_t)i, (uint64_t)base + i + 1);
    }
    __syncthreads();

    // ---- one work item per wavefront, no workgroup barrier from here on ---------
    const int64_t item = (int64_t)blockIdx.x * NWAVE + wave;
    if (item >= (int64_t)a.r * a.tpr) return;
    int j, tile;                               // output row, tile of it
    split_item(item, a.tpr, j, tile);
    if (j >= n) {                              // fewer stored samples than asked for
        if (tile == 0 && lane == 0) a.out_y[j] = -1;
        return;
    }
    int64_t v_lo, v_hi;
    tile_bounds(tile, a.tile_vec, a.tile_rem, a.row_vec, v_lo, v_hi);

    // Draw j is replaced by base + j iff an earlier draw had the same value, or it equals
    // base + q for an earlier q whose own draw was replaced.
    int cur = j;
    bool taken = false;
    for (;;) {
        const uint32_t t = s_t[cur];
        bool same = false;
        if constexpr (MANY) {
#pragma unroll 2
            for (int q0 = 0; q0 < cur; q0 += GEN_LIST) {      // (lanes behind the last draw read its words again; none of theirs counts)
                const int at = q0 + 4 * lane, left = cur - at;        // of the lane's words, those before draw `cur`
                const uint4 v = *reinterpret_cast<const uint4*>(s_t + min(at, (n - 1) & ~3));
                same |= (v.x == t && left > 0) | (v.y == t && left > 1) | (v.z == t && left > 2) | (v.w == t && left > 3);
            }
        } else {
            for (int q = lane; q < cur; q += WAVE) same |= (s_t[q] == t);
        }
        if (__ballot(same) != 0) { taken = true; break; }
        const int64_t q = (int64_t)t - base;
        if (q < 0 || q >= cur) break;
        cur = (int)q;
    }
    const int g = taken ? base + j : (int)s_t[j];      // g-th stored sample, class-major

    // chunk holding g: the last one with s_cpre <= g
    int lo = 0, hi = a.nchunks - 1;
    if (MANY && a.nchunks <= WAVE) lo = hi = __popcll(__ballot(lane < a.nchunks && s_cpre[lane] <= g)) - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (s_cpre[mid] <= g) lo = mid; else hi = mid - 1;
    }
    const int gl = g - s_cpre[lo];
    const int4 f = *reinterpret_cast<const int4*>(a.fill + (int64_t)lo * CH + 4 * lane);
    const int local = f.x + f.y + f.z + f.w;
    const int lincl = wave_scan_incl(local);
    int acc = lincl - local;
    const bool mine = gl >= acc && gl < lincl;
    int u = 0;
    if (mine) {
        if (gl >= acc + f.x) { acc += f.x; u = 1;
            if (gl >= acc + f.y) { acc += f.y; u = 2;
                if (gl >= acc + f.z) { acc += f.z; u = 3; } } }
    }
    const int owner = __builtin_ctzll(__ballot(mine) | (1ull << 63));
    const int pk = lane_read(lo * CH + 4 * lane + u, owner);
    const int ps = lane_read(gl - acc, owner);

    Tile<U, NT, WAVE, false, WIDEN == 2 ? CV_WIDEN8 : WIDEN ? CV_WIDEN : CV_NONE> t;
    t.load(a.buf_x + ((int64_t)pk * a.S + ps) * a.row_vec, v_lo, v_hi);
    t.store(a.out_x + (int64_t)j * a.row_vec * (WIDEN == 2 ? 4 : WIDEN ? 2 : 1), v_lo, v_hi);
    if (tile == 0 && lane == 0) { a.out_y[j] = pk; count_moved(a.state); }
}

}  // namespace
