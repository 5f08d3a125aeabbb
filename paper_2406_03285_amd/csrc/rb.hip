// Rehearsal-buffer hot path for gfx950 (MI355X): the C ABI of include/rb.h (host side); the
// kernels are in rb_kernels_small.h (at most 64 candidates / representatives, and the
// single-launch step), rb_kernels_planned.h (the same step with its plan made during the previous
// launch), rb_kernels_one.h (the single launch for any counts), rb_kernels_general.h (two launches, any counts) and
// rb_kernels_aux.h, their common device code in rb_device.h.  Every form serves every replacement strategy and storage form.
//
// One kernel launch per hot call.  Every workgroup first re-derives, in LDS,
// the few integers of the step's plan it needs (which mini-batch positions are
// candidates, which slot a candidate goes to, which stored sample a
// representative is) and then moves its share of one sample row with 16-byte
// vector loads and stores.  The plan is O(b + K) integers while a row is
// hundreds of kilobytes, so recomputing it per workgroup is cheaper than a
// second, dependent launch.  Nothing is staged through LDS: a row is read once
// and written once, so the data path is global -> registers -> global.
// When the labels of the next mini-batch are known in advance (rb_announce_next)
// the plan is not recomputed per workgroup at all: one workgroup of the previous
// launch leaves it as a table in the workspace and the step's launch only moves rows.
// rb_kernels_one.h holds the single launch of the shapes that the small-count kernels do not serve.
//
// Per-class fill counts are kept twice (ping-pong): an update reads the "old"
// copy everywhere and a few bookkeeping workgroups write the "new" one, so no
// workgroup can observe a count another workgroup of the same launch changed.
// The same two copies let a plan made ahead be dropped: the host just points
// back at the copy the planner read.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <new>

#include "rb.h"
#include "rb_device.h"
#include "rb_kernels_general.h"
#include "rb_kernels_small.h"
#include "rb_kernels_planned.h"
#include "rb_kernels_window.h"
#include "rb_kernels_big.h"
#include "rb_kernels_bigwin.h"
#include "rb_kernels_one.h"
#include "rb_kernels_aux.h"

// ===========================================================================
// Host side: the C ABI
// ===========================================================================
struct rb_buffer {
    int64_t K, S;
    int64_t row_bytes;       // bytes of one stored row
    int64_t row_vec;         // 16-byte vectors of one stored row
    int64_t sample_bytes;    // bytes of one sample as the caller hands it in and gets it back
    int32_t dtype;
    int32_t storage;         // RB_STORE_*
    int32_t nchunks;
    // device storage (borrowed)
    void* buf_x;
    int64_t* buf_y;
    char* ws;
    hipStream_t stream;
    bool bound;
    bool host_rows;          // buf_x is host memory the device reaches over the link
    int cur;                 // which of the two fill-count copies is current
    // workspace layout (byte offsets)
    size_t off_fill[2], off_chunk[2], ws_bytes;
    // launch-shape knobs
    int opt_unroll, opt_nt, opt_rpb, opt_fuse, opt_window, opt_planners;
    // policy variant and its per-class state (two copies, like the fill counts)
    int selection, eviction;
    size_t off_aux[2];
    int64_t updates;         // rb_update calls since the last rb_bind
    // plan-ahead form of the single-launch step
    size_t off_tbl[2];       // the two plan tables
    size_t off_wtbl[2];      // the two plan tables of the several-steps-per-launch form (and of the large-count form)
    size_t off_bfwd[2];      // large-count form: the two tables of the slot rows a step writes
    size_t off_bwtbl[2];     // the two plan tables of the several-steps-per-launch form for large counts
    uint32_t bw_number;      // number of the last window planned in that form (its planners' flags are set to it)
    uint32_t bw_table_number[2];   // ... and which window each of the two tables holds
    int tbl_next;            // table the next plan is written to
    int tbl_planned;         // table that holds the pending plan
    bool plan_valid;         // a step has been planned (and the fill counts advanced) but not yet executed
    const int64_t* plan_y;   // ... for these arguments
    int64_t plan_b, plan_c, plan_r;
    uint64_t plan_seed, plan_step;
    const int64_t* next_y;   // announced labels of the next mini-batch, consumed by the next rb_update_sample
    // several steps per launch: labels announced for the call after the next rb_update_sample_many, and the
    // window that the last launch of a call planned for them
    const int64_t* ann_y[WIN_MAX];
    int64_t ann_n;
    bool wplan_valid;        // a window has been planned (and the fill counts advanced) but not yet executed
    const int64_t* wplan_y[WIN_MAX];
    int wplan_form;          // MANY_SMALL or MANY_LARGE: whose table it is in
    int64_t wplan_w, wplan_b, wplan_c, wplan_r;
    uint64_t wplan_seed, wplan_first;
    int wplan_tbl;           // table that holds it
    int64_t wplan_nat;       // size the windows have grown to (the planned one may be shorter: what was left, what was announced)
    uint64_t stream_number;  // how often the handle was given a stream
    hipEvent_t done;         // event that the last launch of the rb_update_sample_many call being made records; null: none, or it has
    int static_dev;          // device whose static scratch array is this handle's workspace, -1: the caller's workspace
};

// Workspace of rb_bind_static: callers that cannot allocate get their workspace from here.  One copy per GPU
// that loads this library, at an address of its own on each; in host code the array's name only stands for the
// symbol (it is no device address), so the address is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[RB_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
void* scratch_ptr[MAX_DEVICES] = {};          // device address of `scratch` on each device, once known
rb_buffer* scratch_holder[MAX_DEVICES] = {};  // the handle that is bound to it

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline bool overlap(const void* p, int64_t p_bytes, const void* q, int64_t q_bytes)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + (uintptr_t)q_bytes && b < a + (uintptr_t)p_bytes;
}
inline bool in_host_memory(const void* p)
{
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) == hipSuccess) return at.type == hipMemoryTypeHost;
    (void)hipGetLastError();                      // memory the runtime does not know: taken for the device's
    return false;
}
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Launches a kernel; the result is this launch's own.  (`<<<>>>` drops it, and hipGetLastError, asked behind it, also tells of calls of
// anybody's that have failed on this thread before: a step that runs would be taken for one that does not.)
template <typename T> struct as_is { using type = T; };
template <typename... P>
hipError_t launch(void (*kernel)(P...), dim3 grid, int threads, size_t lds, hipStream_t st, const typename as_is<P>::type&... arguments)
{
    void* args[] = {const_cast<void*>(static_cast<const void*>(&arguments))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3((unsigned)threads), args, lds, st);
    if (e != hipSuccess) (void)hipGetLastError();       // (nor is it left for others)
    return e;
}

// How rb_update_sample_many carries out a call: step by step, or several steps per launch planned by one workgroup per
// launch (rb_kernels_window.h) or by two per step (rb_kernels_bigwin.h).
enum { MANY_SINGLE = 0, MANY_SMALL = 1, MANY_LARGE = 2 };

struct Shape {
    int unroll, tpr, tile_vec, tile_rem, rpb;
    int64_t groups;
};

// Split `rows` rows of `row_vec` vectors into tiles of at most width * unroll vectors, where `width`
// is the number of threads that share a tile: TPB in the small-count kernels (a workgroup per tile),
// WAVE in the general ones (a wavefront per tile).
// (With 8-bit storage a vector stands for four accesses of a thread, so one may be enough in flight: `few` is the number of
// tiles below which two become one.  Measured on MI355X, one vector per thread against two: update and sampling in one launch,
// 8 + 8 rows of 602 KB (592 and 304 tiles) 6.9 : 6.4 us, 32 + 32 rows of 49 KB (192 and 128 tiles) 6.0 : 6.4, hence `few` = 256
// there; in two launches 32 + 32 rows of 602 KB (1184 and 608 tiles each) 14.7 : 15.7, 64 + 64 26.5 : 23.3; planned one step ahead,
// where nothing precedes the rows, 8 + 8 rows of 602 KB 6.2 : 8.5, 8 + 8 of 192 KB 5.5 : 7.7, 16 + 16 of 49 KB 5.6 : 6.9, 64 + 64 of
// 12 KB 9.4 : 9.5; the same for large counts 100 + 100 rows of 12 KB 6.5 : 8.1, of 49 KB 7.7 : 10.1, 300 + 300 of 49 KB, 1200
// tiles and two vectors either way, 15.4.)
// most: the most vectors per thread the caller's kernel can hold (the converting movers hold several accesses per
// vector); preferred: what the caller's kernel does best with, taken when the option leaves the choice open.
Shape plan_shape(const rb_buffer* rb, int64_t rows, int width, int most = 8, int preferred = 0, int64_t few = 1024)
{
    Shape s;
    const int64_t row_vec = rb->row_vec;
    int u = rb->opt_unroll != 0 ? rb->opt_unroll : preferred;
    if (u == 0) {
        // Largest unroll that still leaves at least 1024 tiles (four workgroups per compute unit in
        // the small-count kernels, four wavefronts in the general ones); never below two vectors in
        // flight per thread (one was slower at every size measured) unless the row is shorter.
        u = 8;
        while (u > 2 && rows * ((row_vec + (int64_t)width * u - 1) / ((int64_t)width * u)) < 1024) u >>= 1;
        if (u == 2 && rb->storage == RB_STORE_U8 && rows * ((row_vec + 2 * width - 1) / (2 * width)) < few) u = 1;
        while (u > 1 && (int64_t)width * (u / 2) >= row_vec) u >>= 1;
    }
    if (u > most) u = most;
    s.unroll = u;
    const int64_t cap = (int64_t)width * u;
    s.tpr = (int)((row_vec + cap - 1) / cap);
    // even split in units of TILE_UNIT vectors: every tile holds nunits / tpr units, the first nunits % tpr one more
    const int64_t nunits = (row_vec + TILE_UNIT - 1) / TILE_UNIT;
    s.tile_vec = (int)(nunits / s.tpr);
    s.tile_rem = (int)(nunits % s.tpr);
    s.rpb = 1;
    if (width == TPB && s.tpr == 1) {
        int r = rb->opt_rpb;
        if (r == 0) {
            r = 1;
            while (r < 16 && (rows + r - 1) / r > 1024) r <<= 1;
        }
        s.rpb = r;
    }
    s.groups = (rows + s.rpb - 1) / s.rpb;
    return s;
}

// Tiles of rb_sample_small_kernel's launch.  Rows that are converted on the way lose a microsecond when a compute unit gets a fourth
// workgroup: bfloat16, more than 1024 classes, two vectors per thread, 760 workgroups 5.3 us, 832 6.3, 1000 7.2; 8 bits, one
// vector, 760 4.95, 832 6.0, 1000 6.6.  From there on the next larger tiles are taken.  bfloat16, two vectors and four: 52 rows of 301 KB 7.15 : 6.7,
// 64 of 250 KB 7.5 : 6.45, 64 of 301 KB 8.05 : 7.15; up to 1024 classes, where a workgroup starts to move later, 64 of 203 KB
// 6.2 : 6.6, 64 of 250 KB 7.35 : 6.8: there two stay.  8 bits, one and two: 64 of 203 KB 6.0 : 5.3, 64 of 301 KB 7.45 : 6.15, 52 of 400 KB
// 7.75 : 6.55, but where two vectors make more than three workgroups per compute unit as well 64 of 450 KB 9.35 : 9.8, 52 of 500 KB 9.2 : 9.15.
// (There, with 1024 workgroups and more, a wait after every second store instead of a burst: 64 of 602 KB, 10 classes, 11.3 : 10.4 us, 1000 classes
// 11.9 : 10.8, 64 of 500 KB, 1025 classes, 10.9 : 10.1, 64 of 2 MB 33.7 : 33.4; with three workgroups 64 of 301 KB 6.15 : 6.6.)
constexpr int64_t THREE_EACH = 3 * 256;           // workgroups
Shape sample_small_shape(const rb_buffer* rb, int64_t r)
{
    const bool u8 = rb->storage == RB_STORE_U8;
    const int most = u8 ? 2 : 8;
    const Shape s = plan_shape(rb, r, TPB, most);
    if (u8 && s.unroll == 1 && r * s.tpr > THREE_EACH && r * ((rb->row_vec + 2 * TPB - 1) / (2 * TPB)) <= THREE_EACH) return plan_shape(rb, r, TPB, most, 2);
    if (rb->storage == RB_STORE_BF16 && rb->nchunks > DIRECT_CHUNKS && s.unroll == 2 && r * s.tpr > THREE_EACH) return plan_shape(rb, r, TPB, most, 4);
    return s;
}

// Whether a one-step launch that moves `rows` plain rows in tiles of eight vectors per thread (33 MB and more, about one round of
// workgroups) does better with ordinary stores behind its streaming loads: what a workgroup writes waits in the die's L2 while
// others read, and what the chip's last cache (256 MB) holds need not reach memory at once.  In megabytes written by the launch, both
// ends of each kind of launch.  rb_step_small_kernel does from the start, us, streaming and ordinary: 64 + 64 rows of 301 KB [38.5 MB] 15.2 : 14.6,
// 64 + 8 of 602 KB [43] 17.1 : 16.1, 48 + 48 [58] 23.2 : 20.3, 64 + 64 [77] 31.7 : 28.7, of 1 MB [128] 50.7 : 45.2, of 2.6 MB [336] 119.0 : 112.8,
// 64 + 16 of 4.2 MB [336] 105.0 : 95.9, but 64 + 64 of 2.9 MB [369] 130.5 : 133.4, of 4.2 MB [537] 184 : 194.  Launches whose rows all move at
// the same time do from about 45 MB on.  Planned one step ahead: 64 + 64 of 301 KB [38.5] 13.8 : 14.2, 48 + 48 of 400 KB [38.4] 13.8 : 14.3,
// 64 + 64 of 400 KB [51] 20.4 : 19.8, of 602 KB [77] 29.1 : 26.8, of 1 MB 47.5 : 42.7, of 2.6 MB [336] 113.7 : 108.1, of 2.9 MB [369] 124.9 : 127.9.
// Two calls: 64 + 64 of 602 KB [38.5 each] 29.3 : 30.0, of 800 KB [51] 41.3 : 38.2, of 1 MB [64] 51.2 : 46.6, of 3.1 MB [201] 145.0 : 141.9,
// of 3.7 MB [235] 167.6 : 170.6, of 4.2 MB [268] 186.7 : 189.7.  Smaller tiles and launches of many steps lose (14 + 7 rows of 602 KB 8.0 : 8.4,
// 64 rows of 301 KB with four vectors 8.9 : 9.4, 20 steps of 64 + 64 rows of 301 KB at once 225 : 253), and so do rows stored in host
// memory, which no cache holds back (one launch, 64 + 64 rows of 301 KB 396 : 474, planned, of 602 KB 785 : 800).
enum { STORES_STEP = 0, STORES_PLANNED = 1, STORES_HALF = 2 };     // update and sample in one launch; by a plan; one of the two calls
bool ordinary_stores(const rb_buffer* rb, int64_t rows, int kind)
{
    const int64_t bytes = rows * rb->row_bytes;
    if (rb->host_rows) return false;
    return bytes >= (kind == STORES_STEP ? 0 : INT64_C(45000000)) && bytes < (kind == STORES_HALF ? INT64_C(210000000) : INT64_C(345000000));
}

// LDS of rb_update_small_kernel and rb_step_small_kernel
size_t small_lds_bytes(int64_t b, int nchunks)
{
    return round_up((size_t)b * 8, 16) + (nchunks <= DIRECT_CHUNKS ? (size_t)DIRECT_CHUNKS * CH * 4 : 0);
}

// The small-count kernels: vectors per thread (8-bit storage: at most two, a thread holds four accesses per vector),
// storage form and whether the replacement strategy keeps per-class state are template parameters.
template <bool NT, int ST, bool AUX>
hipError_t launch_update_small_s(const UpdateArgs& a, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    const auto go = [&](auto kernel) {
        return launch(kernel, grid, TPB, lds, st, a.batch_y, a.fill_old, a.sd.seed_lo, a.sd.seed_hi, a.sd.step_lo, a.sd.step_hi,
                      (uint32_t)(a.b | a.c << 16), a.nchunks, a);
    };
    switch (unroll) {
    case 1: return go(rb_update_small_kernel<1, NT, ST, AUX>);
    case 2: return go(rb_update_small_kernel<2, NT, ST, AUX>);
    default:
        if constexpr (ST == RB_STORE_U8) return hipErrorInvalidValue;
        else if (unroll == 4) return go(rb_update_small_kernel<4, NT, ST, AUX>);
        else if (ST == RB_STORE_SAME && ordinary) return go(rb_update_small_kernel<8, NT, ST, AUX, NT && ST != RB_STORE_SAME>);
        else return go(rb_update_small_kernel<8, NT, ST, AUX>);
    }
}

template <bool NT>
hipError_t launch_update_small(const UpdateArgs& a, int storage, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    const bool aux = a.eviction != RB_EVICT_UNIFORM;
    switch (storage) {
    case RB_STORE_BF16:
        return aux ? launch_update_small_s<NT, RB_STORE_BF16, true>(a, unroll, grid, lds, st, ordinary) : launch_update_small_s<NT, RB_STORE_BF16, false>(a, unroll, grid, lds, st, ordinary);
    case RB_STORE_U8:
        return aux ? launch_update_small_s<NT, RB_STORE_U8, true>(a, unroll, grid, lds, st, ordinary) : launch_update_small_s<NT, RB_STORE_U8, false>(a, unroll, grid, lds, st, ordinary);
    default:
        return aux ? launch_update_small_s<NT, RB_STORE_SAME, true>(a, unroll, grid, lds, st, ordinary) : launch_update_small_s<NT, RB_STORE_SAME, false>(a, unroll, grid, lds, st, ordinary);
    }
}

template <bool NT, int ST>
hipError_t launch_sample_small_s(const SampleArgs& a, int unroll, dim3 grid, hipStream_t st, bool ordinary)
{
    const auto go = [&](auto kernel) {
        return launch(kernel, grid, TPB, 0, st, a.fill, a.chunk, a.sd.seed_lo, a.sd.seed_hi, a.sd.step_lo, a.sd.step_hi, a.r, a.nchunks, a);
    };
    switch (unroll) {
    case 1: return go(rb_sample_small_kernel<1, NT, ST>);
    case 2:
        if (ST == RB_STORE_U8 && grid.x > THREE_EACH) return go(rb_sample_small_kernel<2, NT, ST, NT, ST == RB_STORE_U8 ? 2 : step_pace(ST, 2)>);
        else return go(rb_sample_small_kernel<2, NT, ST>);
    default:
        if constexpr (ST == RB_STORE_U8) return hipErrorInvalidValue;
        else if (unroll == 4) return go(rb_sample_small_kernel<4, NT, ST>);
        else if (ST == RB_STORE_SAME && ordinary) return go(rb_sample_small_kernel<8, NT, ST, NT && ST != RB_STORE_SAME>);
        else return go(rb_sample_small_kernel<8, NT, ST>);
    }
}

template <bool NT>
hipError_t launch_sample_small(const SampleArgs& a, int storage, int unroll, dim3 grid, hipStream_t st, bool ordinary)
{
    switch (storage) {
    case RB_STORE_BF16: return launch_sample_small_s<NT, RB_STORE_BF16>(a, unroll, grid, st, ordinary);
    case RB_STORE_U8: return launch_sample_small_s<NT, RB_STORE_U8>(a, unroll, grid, st, ordinary);
    default: return launch_sample_small_s<NT, RB_STORE_SAME>(a, unroll, grid, st, ordinary);
    }
}

template <bool NT, int FORM>
hipError_t launch_update_f(const UpdateArgs& a, int narrow, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    if (narrow == 2) {                  // 8 bits per element: a lane holds four accesses per vector of the tile (at most four vectors)
        if (unroll == 1) return launch(rb_update_kernel<1, NT, 2, FORM>, grid, TPB, lds, st, a);
        if (unroll == 2) return launch(rb_update_kernel<2, NT, 2, FORM>, grid, TPB, lds, st, a);
        return launch(rb_update_kernel<4, NT, 2, FORM>, grid, TPB, lds, st, a);
    }
    if (narrow == 1) {
        switch (unroll) {
        case 1: return launch(rb_update_kernel<1, NT, 1, FORM>, grid, TPB, lds, st, a);
        case 2: return launch(rb_update_kernel<2, NT, 1, FORM>, grid, TPB, lds, st, a);
        case 4: return launch(rb_update_kernel<4, NT, 1, FORM>, grid, TPB, lds, st, a);
        default: return launch(rb_update_kernel<8, NT, 1, FORM>, grid, TPB, lds, st, a);
        }
    }
    switch (unroll) {
    case 1: return launch(rb_update_kernel<1, NT, 0, FORM>, grid, TPB, lds, st, a);
    case 2: return launch(rb_update_kernel<2, NT, 0, FORM>, grid, TPB, lds, st, a);
    case 4: return launch(rb_update_kernel<4, NT, 0, FORM>, grid, TPB, lds, st, a);
    default: return launch(rb_update_kernel<8, NT, 0, FORM>, grid, TPB, lds, st, a);
    }
}

template <bool NT>
hipError_t launch_update(const UpdateArgs& a, int narrow, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    if (a.selection == RB_SELECT_BERNOULLI) return launch_update_f<NT, GEN_COINS>(a, narrow, unroll, grid, lds, st);
    return gen_few(a.c, a.row_vec, narrow != 0, a.eviction) ? launch_update_f<NT, GEN_EXACT_FEW>(a, narrow, unroll, grid, lds, st) : launch_update_f<NT, GEN_EXACT_MANY>(a, narrow, unroll, grid, lds, st);
}

template <bool NT, bool MANY>
hipError_t launch_sample_f(const SampleArgs& a, int widen, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    if (widen == 2) {
        if (unroll == 1) return launch(rb_sample_kernel<1, NT, 2, MANY>, grid, TPB, lds, st, a);
        return launch(rb_sample_kernel<2, NT, 2, MANY>, grid, TPB, lds, st, a);
    }
    if (widen == 1) {
        if (unroll == 1) return launch(rb_sample_kernel<1, NT, 1, MANY>, grid, TPB, lds, st, a);
        if (unroll == 2) return launch(rb_sample_kernel<2, NT, 1, MANY>, grid, TPB, lds, st, a);
        return launch(rb_sample_kernel<4, NT, 1, MANY>, grid, TPB, lds, st, a);
    }
    switch (unroll) {
    case 1: return launch(rb_sample_kernel<1, NT, 0, MANY>, grid, TPB, lds, st, a);
    case 2: return launch(rb_sample_kernel<2, NT, 0, MANY>, grid, TPB, lds, st, a);
    case 4: return launch(rb_sample_kernel<4, NT, 0, MANY>, grid, TPB, lds, st, a);
    default: return launch(rb_sample_kernel<8, NT, 0, MANY>, grid, TPB, lds, st, a);
    }
}

template <bool NT>
hipError_t launch_sample(const SampleArgs& a, int widen, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    return a.r > BIG_MAX && a.r <= a.K * a.S ? launch_sample_f<NT, true>(a, widen, unroll, grid, lds, st) : launch_sample_f<NT, false>(a, widen, unroll, grid, lds, st);
}

template <bool NT, int ST, bool AUX>
hipError_t launch_step_s(const StepArgs& sa, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    const UpdateArgs& a = sa.u;
    const auto go = [&](auto kernel) {
        return launch(kernel, grid, TPB, lds, st, a.batch_y, a.fill_old, a.sd.seed_lo, a.sd.seed_hi, a.sd.step_lo, a.sd.step_hi,
                      (uint32_t)(a.b | a.c << 16), (uint32_t)(sa.r | a.nchunks << 16), a.tpr, a.nchunks + a.c * a.tpr, sa);
    };
    switch (unroll) {
    case 1: return go(rb_step_small_kernel<1, NT, ST, AUX>);
    case 2: return go(rb_step_small_kernel<2, NT, ST, AUX>);
    default:
        if constexpr (ST == RB_STORE_U8) return hipErrorInvalidValue;
        else if (unroll == 4) return go(rb_step_small_kernel<4, NT, ST, AUX>);
        else if constexpr (ST != RB_STORE_SAME) return hipErrorInvalidValue;
        else if (ordinary) return go(rb_step_small_kernel<8, NT, ST, AUX, false>);
        else return go(rb_step_small_kernel<8, NT, ST, AUX>);
    }
}

template <bool NT>
hipError_t launch_step(const StepArgs& a, int storage, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    const bool aux = a.u.eviction != RB_EVICT_UNIFORM;
    switch (storage) {
    case RB_STORE_BF16:
        return aux ? launch_step_s<NT, RB_STORE_BF16, true>(a, unroll, grid, lds, st, ordinary) : launch_step_s<NT, RB_STORE_BF16, false>(a, unroll, grid, lds, st, ordinary);
    case RB_STORE_U8:
        return aux ? launch_step_s<NT, RB_STORE_U8, true>(a, unroll, grid, lds, st, ordinary) : launch_step_s<NT, RB_STORE_U8, false>(a, unroll, grid, lds, st, ordinary);
    default:
        return aux ? launch_step_s<NT, RB_STORE_SAME, true>(a, unroll, grid, lds, st, ordinary) : launch_step_s<NT, RB_STORE_SAME, false>(a, unroll, grid, lds, st, ordinary);
    }
}

template <bool NT, int PACE>
hipError_t launch_copy(vec16* dst, const vec16* src, int64_t nvec, int unroll, hipStream_t st)
{
    const int64_t cap = (int64_t)TPB * unroll;
    dim3 grid((unsigned)((nvec + cap - 1) / cap));
    switch (unroll) {
    case 1: return launch(rb_copy_kernel<1, NT, PACE>, grid, TPB, 0, st, dst, src, nvec);
    case 2: return launch(rb_copy_kernel<2, NT, PACE>, grid, TPB, 0, st, dst, src, nvec);
    case 4: return launch(rb_copy_kernel<4, NT, PACE>, grid, TPB, 0, st, dst, src, nvec);
    default: return launch(rb_copy_kernel<8, NT, PACE>, grid, TPB, 0, st, dst, src, nvec);
    }
}

Seed make_seed(uint64_t seed, uint64_t step)
{
    Seed s;
    s.seed_lo = (uint32_t)seed;
    s.seed_hi = (uint32_t)(seed >> 32);
    s.step_lo = (uint32_t)step;
    s.step_hi = (uint32_t)(step >> 32);
    return s;
}

template <bool NT, int ST>
hipError_t launch_planned_s(const MoveArgs& m, const PlanArgs& next, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    const auto go = [&](auto kernel) {
        return launch(kernel, grid, TPB, lds, st, m.table, m.batch_x, m.buf_x, m.out_x, m.row_vec, (uint32_t)(m.c | m.r << 16),
                      (uint32_t)m.tpr | (uint32_t)m.plan_next << 31, m.tile_vec, m.tile_rem, m, next);
    };
    switch (unroll) {
    case 1: return go(rb_step_planned_kernel<1, NT, ST>);
    case 2: return go(rb_step_planned_kernel<2, NT, ST>);
    case 4:
        if constexpr (ST == RB_STORE_U8) return hipErrorInvalidValue;    // (at most two vectors per lane: step_planned)
        else return go(rb_step_planned_kernel<4, NT, ST>);
    default:
        if constexpr (ST != RB_STORE_SAME) return hipErrorInvalidValue;  // (bfloat16 rows: at most four)
        else if (ordinary) return go(rb_step_planned_kernel<8, NT, ST, false>);
        else return go(rb_step_planned_kernel<8, NT, ST>);
    }
}

template <bool NT>
hipError_t launch_planned(const MoveArgs& m, const PlanArgs& next, int storage, int unroll, dim3 grid, size_t lds, hipStream_t st, bool ordinary)
{
    switch (storage) {
    case RB_STORE_BF16: return launch_planned_s<NT, RB_STORE_BF16>(m, next, unroll, grid, lds, st, ordinary);
    case RB_STORE_U8: return launch_planned_s<NT, RB_STORE_U8>(m, next, unroll, grid, lds, st, ordinary);
    default: return launch_planned_s<NT, RB_STORE_SAME>(m, next, unroll, grid, lds, st, ordinary);
    }
}

// Called by every entry point other than rb_update_sample.  A step that was planned ahead will not
// be executed as planned: the fill counts go back to the copy the planner read (it only wrote the
// other one).  An announcement that has not been used yet is forgotten as well: it was made for the
// call that should have come next.
void discard_window_plan(rb_buffer* rb)
{
    if (rb->wplan_valid) {
        rb->cur ^= 1;
        rb->wplan_valid = false;
    }
}

// Whether the window that the call before planned ahead (window_plan_kept) is the start of this call: same shape, seed
// and step number, and the very label arrays that were announced.
bool window_plan_matches(const rb_buffer* rb, int form, int64_t n, const int64_t* const* batch_y, int64_t b, int64_t c, int64_t r,
                         uint64_t seed, uint64_t first_step)
{
    bool same = rb->wplan_valid && rb->wplan_form == form && rb->wplan_w <= n && rb->wplan_b == b && rb->wplan_c == c && rb->wplan_r == r &&
                rb->wplan_seed == seed && rb->wplan_first == first_step;
    for (int64_t k = 0; same && k < rb->wplan_w; ++k) same = rb->wplan_y[k] == batch_y[k];
    return same;
}

// The last launch of a call has planned the first w steps of the call that was announced, into table tbl of the given
// form (MANY_SMALL, MANY_LARGE).
void window_plan_kept(rb_buffer* rb, int form, int64_t w, int64_t b, int64_t c, int64_t r, uint64_t seed, uint64_t first_step, int tbl,
                      int64_t nat, const int64_t* const* ann_y)
{
    rb->wplan_valid = true;
    rb->wplan_form = form;
    rb->wplan_w = w; rb->wplan_b = b; rb->wplan_c = c; rb->wplan_r = r;
    rb->wplan_seed = seed; rb->wplan_first = first_step;
    rb->wplan_tbl = tbl;
    rb->wplan_nat = nat;
    for (int64_t k = 0; k < w; ++k) rb->wplan_y[k] = ann_y[k];
}

void discard_plan(rb_buffer* rb)
{
    if (rb->plan_valid) {
        rb->cur ^= 1;
        rb->plan_valid = false;
    }
    discard_window_plan(rb);
    rb->next_y = nullptr;
    rb->ann_n = 0;
}

PlanArgs make_plan(const rb_buffer* rb, const int64_t* batch_y, int64_t b, int64_t c, int64_t r, uint64_t seed, uint64_t step)
{
    PlanArgs p;
    p.batch_y = batch_y;
    p.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    p.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    p.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    p.table = rb->ws + rb->off_tbl[rb->tbl_next];
    p.sd = make_seed(seed, step);
    p.b = (int32_t)b; p.c = (int32_t)c; p.r = (int32_t)r;
    p.K = (int32_t)rb->K; p.nchunks = rb->nchunks;
    p.S = rb->S;
    p.eviction = rb->eviction;
    p.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    p.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    p.selection = rb->selection;
    p.ce = (int32_t)(rb->selection == RB_SELECT_BERNOULLI ? big_coin_entries(b) : c);
    return p;
}

// Host bookkeeping after a plan has been enqueued.
void plan_enqueued(rb_buffer* rb, const int64_t* batch_y, int64_t b, int64_t c, int64_t r, uint64_t seed, uint64_t step)
{
    rb->cur ^= 1;
    rb->tbl_planned = rb->tbl_next;
    rb->tbl_next ^= 1;
    rb->plan_valid = true;
    rb->plan_y = batch_y; rb->plan_b = b; rb->plan_c = c; rb->plan_r = r; rb->plan_seed = seed; rb->plan_step = step;
}

// One step of the plan-ahead form: plan it now unless the previous launch already did, move its
// rows by the table, and let the same launch plan the following step when its labels are known.
int step_planned(rb_buffer* rb, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c, int64_t r,
                 uint64_t seed, uint64_t step, void* out_x, int64_t* out_y, const int64_t* next_y)
{
    if (!rb->plan_valid) {
        const PlanArgs now = make_plan(rb, batch_y, b, c, r, seed, step);
        if (launch(rb_plan_kernel, dim3(1), TPB, (size_t)b * 8, rb->stream, now) != hipSuccess) return RB_EHIP;
        plan_enqueued(rb, batch_y, b, c, r, seed, step);
    }
    // (rows that are converted do better with fewer vectors per thread: 64 + 64 rows of 602 KB in 8 bits 25.6 us with four,
    // 21.0 with two; as bfloat16 25.9 with eight, 23.1 with four)
    const Shape sh = plan_shape(rb, c + r, TPB, rb->storage == RB_STORE_U8 ? 2 : rb->storage == RB_STORE_BF16 ? 4 : 8);
    MoveArgs m;
    m.batch_x = static_cast<const vec16*>(batch_x);
    m.buf_x = static_cast<vec16*>(rb->buf_x);
    m.buf_y = rb->buf_y;
    m.out_x = static_cast<vec16*>(out_x);
    m.out_y = out_y;
    m.table = rb->ws + rb->off_tbl[rb->tbl_planned];
    m.state = reinterpret_cast<DevState*>(rb->ws);
    m.c = (int32_t)c; m.r = (int32_t)r; m.cgrid = (int32_t)c;
    m.S = rb->S;
    m.row_vec = rb->row_vec;
    m.tpr = sh.tpr; m.tile_vec = sh.tile_vec; m.tile_rem = sh.tile_rem;
    const int64_t movers = (c + r) * sh.tpr;
    rb->plan_valid = false;                     // this step is being executed
    m.plan_next = next_y ? 1 : 0;
    PlanArgs next = {};
    if (next_y) next = make_plan(rb, next_y, b, c, r, seed, step + 1);
    const dim3 grid((unsigned)(movers + m.plan_next));
    const size_t lds = next_y ? (size_t)b * 8 : 0;
    const bool ordinary = ordinary_stores(rb, c + r, STORES_PLANNED);
    const hipError_t e = rb->opt_nt ? launch_planned<true>(m, next, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary)
                                    : launch_planned<false>(m, next, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary);
    if (e == hipSuccess && next_y) plan_enqueued(rb, next_y, b, c, r, seed, step + 1);
    if (e != hipSuccess) return RB_EHIP;
    rb->updates += 1;
    return RB_OK;
}

// The 1024-thread kernels ask for more dynamic LDS than a kernel gets by default: allowed once per kernel and device.
template <auto kernel, int bytes = (int)BIG_LDS_BYTES>
hipError_t allow_big_lds()
{
    static bool allowed[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (dev < 0 || dev >= 64 || !allowed[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) allowed[dev] = true;
    }
    return hipSuccess;
}

template <int U, bool NT, int ST>
hipError_t launch_big_u(const MoveArgs& m, const PlanArgs& next, const uint32_t* fwd, uint32_t* fwd_next, dim3 grid, hipStream_t st)
{
    // (the converting movers have to fit the 128 registers per lane of a 1024-thread workgroup: big_shape)
    if constexpr ((ST == RB_STORE_U8 && U > 2) || (ST == RB_STORE_BF16 && U > 8)) {
        return hipErrorInvalidValue;
    } else {
        const size_t lds = m.plan_next ? BIG_LDS_BYTES : 0;
        if (lds != 0) {
            const hipError_t e = allow_big_lds<&rb_step_big_kernel<U, NT, ST>>();
            if (e != hipSuccess) return e;
        }
        return launch(rb_step_big_kernel<U, NT, ST>, grid, BIG_TPB, lds, st, m.table, m.batch_x, m.buf_x, m.out_x, m.row_vec, (uint32_t)(m.cgrid | m.r << 16),
                      (uint32_t)m.tpr | (uint32_t)m.plan_next << 31, m.tile_vec, m.tile_rem, m, next, fwd, fwd_next);
    }
}

template <bool NT, int ST>
hipError_t launch_big_s(const MoveArgs& m, const PlanArgs& next, const uint32_t* fwd, uint32_t* fwd_next, int unroll, dim3 grid,
                        hipStream_t st)
{
    switch (unroll) {
    case 1: return launch_big_u<1, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 2: return launch_big_u<2, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 4: return launch_big_u<4, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 6: return launch_big_u<6, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 8: return launch_big_u<8, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 10: return launch_big_u<10, NT, ST>(m, next, fwd, fwd_next, grid, st);
    case 12: return launch_big_u<12, NT, ST>(m, next, fwd, fwd_next, grid, st);
    default: return hipErrorInvalidValue;
    }
}

template <bool NT>
hipError_t launch_big(const MoveArgs& m, const PlanArgs& next, const uint32_t* fwd, uint32_t* fwd_next, int storage, int unroll,
                      dim3 grid, hipStream_t st)
{
    switch (storage) {
    case RB_STORE_BF16: return launch_big_s<NT, RB_STORE_BF16>(m, next, fwd, fwd_next, unroll, grid, st);
    case RB_STORE_U8: return launch_big_s<NT, RB_STORE_U8>(m, next, fwd, fwd_next, unroll, grid, st);
    default: return launch_big_s<NT, RB_STORE_SAME>(m, next, fwd, fwd_next, unroll, grid, st);
    }
}

// Tiles of the large-count launch.  Its workgroups hold four groups of movers each, and a compute unit holds one such
// workgroup at a time (traced: of 325 workgroups the last 69 start when the first ones end), so a launch of a few
// hundred workgroups runs in rounds of 256, and a round that is nearly empty costs as much as a full one (measured
// on MI355X with a bare mover, 129 rows of 301 056 bytes: 323 workgroups of four 32 KiB tiles 18.9 us, 226
// workgroups of four 42 KiB tiles 14.9 us, 258 workgroups 20.1 us; 256 rows: 640 workgroups 33.6 us, 448
// workgroups 31.4 us; the whole step gains less: 65 candidates and 64 representatives 17.3 -> 16.5 us, 128 and 128
// 33.0 -> 32.0 us).  So, when the rows are long enough (tiles of 12 KiB and more), a row gets as many tiles as keep
// the whole launch, planners included, within one round, or else within two.  Measured and not adopted: at most
// one mover workgroup per compute unit whose groups go round the tiles themselves (5 to 10 % slower than letting
// the second round of workgroups start as the first ones end); for many short rows a wavefront per row, sixteen
// rows per workgroup, so that one round suffices (10000 classes, 1024 + 1024 rows of 8 KiB: no change, the step is
// bound by the planners and the launch itself).
Shape big_shape(const rb_buffer* rb, int64_t rows, int planners)
{
    // (with 8-bit storage a lane holds four accesses per vector, and these workgroups have 128 registers per lane: two vectors)
    // - or one, as long as the tiles of one vector keep the launch within one round (100 + 100 rows of 49 KB 7.7 us with one, 10.1
    // with two; 302 + 85 rows of 51 KB, 387 and 194 workgroups, 12.1 : 10.8)
    if (rb->storage == RB_STORE_U8) {
        const int64_t tiles = rows * ((rb->row_vec + BIG_GROUP - 1) / BIG_GROUP);
        return plan_shape(rb, rows, BIG_GROUP, 2, 0, tiles <= (256 - planners) * (int64_t)BIG_GROUPS ? 1024 : 0);
    }
    Shape s = plan_shape(rb, rows, BIG_GROUP);
    if (rb->opt_unroll != 0) return s;
    constexpr int64_t CUS = 256;
    const int64_t nunits = (rb->row_vec + TILE_UNIT - 1) / TILE_UNIT;
    for (int64_t k = 1; k <= 2; ++k) {
        int64_t tpr = (CUS * k - planners) * BIG_GROUPS / rows;
        if (tpr > nunits) tpr = nunits;
        if (tpr < 1) continue;
        const int64_t tile = (nunits / tpr + (nunits % tpr ? 1 : 0)) * TILE_UNIT;      // vectors of the longest tile
        int u = (int)((tile + BIG_GROUP - 1) / BIG_GROUP);
        if (u > (rb->storage == RB_STORE_BF16 ? 8 : 12)) continue;
        if (u < 4) break;                                                                 // short rows: the plain split
        u = (u + 1) / 2 * 2;                                                              // 4, 6, 8, 10 or 12
        s.unroll = u;
        s.tpr = (int)tpr;
        s.tile_vec = (int)(nunits / tpr);
        s.tile_rem = (int)(nunits % tpr);
        s.rpb = 1;
        s.groups = rows;
        return s;
    }
    return s;
}

// One step of the plan-ahead form for large counts (up to BIG_MAX candidates and representatives, up to
// BIG_CLASSES classes); same bookkeeping as step_planned, the tables are the (larger) ones that the
// several-steps-per-launch form uses for shapes this form does not serve.  Two workgroups plan.
int step_big(rb_buffer* rb, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c, int64_t r,
             uint64_t seed, uint64_t step, void* out_x, int64_t* out_y, const int64_t* next_y)
{
    static_assert(BIG_TABLE_BYTES <= WIN_TABLE_BYTES, "the big plan's table must fit the window table");
    if (!rb->plan_valid) {
        PlanArgs now = make_plan(rb, batch_y, b, c, r, seed, step);
        now.table = rb->ws + rb->off_wtbl[rb->tbl_next];
        if (allow_big_lds<&rb_big_plan_kernel>() != hipSuccess) return RB_EHIP;
        if (launch(rb_big_plan_kernel, dim3(2), BIG_TPB, BIG_LDS_BYTES, rb->stream, now, reinterpret_cast<uint32_t*>(rb->ws + rb->off_bfwd[rb->tbl_next])) != hipSuccess) return RB_EHIP;
        plan_enqueued(rb, batch_y, b, c, r, seed, step);
    }
    // candidate entries of the table, and how many of them the grid covers: all c, or, with the Bernoulli selection
    // (about c of the b positions are selected), c and eight standard deviations (more are served by going round)
    const bool bernoulli = rb->selection == RB_SELECT_BERNOULLI;
    const int64_t ce = bernoulli ? big_coin_entries(b) : c;
    int64_t margin = 16;
    while (margin * margin < 64 * c) ++margin;
    const int64_t cgrid = bernoulli ? std::min(b, c + margin) : c;
    const Shape sh = big_shape(rb, cgrid + r, next_y ? 2 : 0);
    MoveArgs m;
    m.batch_x = static_cast<const vec16*>(batch_x);
    m.buf_x = static_cast<vec16*>(rb->buf_x);
    m.buf_y = rb->buf_y;
    m.out_x = static_cast<vec16*>(out_x);
    m.out_y = out_y;
    m.table = rb->ws + rb->off_wtbl[rb->tbl_planned];
    m.state = reinterpret_cast<DevState*>(rb->ws);
    m.c = (int32_t)ce; m.r = (int32_t)r; m.cgrid = (int32_t)cgrid;
    m.S = rb->S;
    m.row_vec = rb->row_vec;
    m.tpr = sh.tpr; m.tile_vec = sh.tile_vec; m.tile_rem = sh.tile_rem;
    const int64_t items = (cgrid + r) * sh.tpr;
    rb->plan_valid = false;                     // this step is being executed
    m.plan_next = next_y ? 1 : 0;
    PlanArgs next = {};
    if (next_y) {
        next = make_plan(rb, next_y, b, c, r, seed, step + 1);
        next.table = rb->ws + rb->off_wtbl[rb->tbl_next];
    }
    const uint32_t* fwd = reinterpret_cast<const uint32_t*>(rb->ws + rb->off_bfwd[rb->tbl_planned]);
    uint32_t* fwd_next = reinterpret_cast<uint32_t*>(rb->ws + rb->off_bfwd[rb->tbl_next]);
    const dim3 grid((unsigned)((items + BIG_GROUPS - 1) / BIG_GROUPS + 2 * m.plan_next));
    const hipError_t e = rb->opt_nt ? launch_big<true>(m, next, fwd, fwd_next, rb->storage, sh.unroll, grid, rb->stream)
                                    : launch_big<false>(m, next, fwd, fwd_next, rb->storage, sh.unroll, grid, rb->stream);
    if (e == hipSuccess && next_y) plan_enqueued(rb, next_y, b, c, r, seed, step + 1);
    if (e != hipSuccess) return RB_EHIP;
    rb->updates += 1;
    return RB_OK;
}

// A launch that records `done` (null: none) when it ends: its own completion is the event, without a packet of its own behind it in
// the stream.  Two streams that wait for each other's events, 200 us of kernel a round: 237.0 us a round with the event recorded
// behind the kernel, 233.7 so.
template <typename K, typename M, typename P>
hipError_t launch_recorded(K kernel, dim3 grid, int threads, size_t lds, hipStream_t st, hipEvent_t done, const M& m, const P& next)
{
    if (done != nullptr) {
        void* args[] = {const_cast<M*>(&m), const_cast<P*>(&next)};
        const hipError_t e = hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3((unsigned)threads), args, lds, st, nullptr, done, 0);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
    return launch(kernel, grid, threads, lds, st, m, next);
}

// The event of the call being made, if its last launch is the one about to go out.
hipEvent_t take_done(rb_buffer* rb, bool last)
{
    const hipEvent_t e = last ? rb->done : nullptr;
    if (last) rb->done = nullptr;
    return e;
}

template <bool NT, int ST, bool AUX>
hipError_t launch_window_u(const WinMoveArgs& m, const WinPlanArgs& next, int unroll, dim3 grid, hipStream_t st, hipEvent_t done)
{
    const auto go = [&](auto kernel) { return launch_recorded(kernel, grid, TPB, 0, st, done, m, next); };
    switch (unroll) {
    case 1: return go(rb_window_kernel<1, NT, ST, AUX>);
    case 2: return go(rb_window_kernel<2, NT, ST, AUX>);
    case 4: return go(rb_window_kernel<4, NT, ST, AUX>);
    default:
        if constexpr (ST == RB_STORE_U8) return hipErrorInvalidValue;    // (a lane holds four accesses per vector: at most four vectors)
        else return go(rb_window_kernel<8, NT, ST, AUX>);
    }
}

// aux: the replacement strategy keeps per-class state (FIFO, reservoir)
template <bool NT>
hipError_t launch_window(const WinMoveArgs& m, const WinPlanArgs& next, int storage, bool aux, int unroll, dim3 grid, hipStream_t st, hipEvent_t done)
{
    switch (storage) {
    case RB_STORE_BF16:
        return aux ? launch_window_u<NT, RB_STORE_BF16, true>(m, next, unroll, grid, st, done) : launch_window_u<NT, RB_STORE_BF16, false>(m, next, unroll, grid, st, done);
    case RB_STORE_U8:
        return aux ? launch_window_u<NT, RB_STORE_U8, true>(m, next, unroll, grid, st, done) : launch_window_u<NT, RB_STORE_U8, false>(m, next, unroll, grid, st, done);
    default:
        return aux ? launch_window_u<NT, RB_STORE_SAME, true>(m, next, unroll, grid, st, done) : launch_window_u<NT, RB_STORE_SAME, false>(m, next, unroll, grid, st, done);
    }
}

WinPlanArgs window_plan_args(rb_buffer* rb, const int64_t* const* batch_y, int64_t at, int64_t w, int64_t b, int64_t c, int64_t r,
                             uint64_t seed, uint64_t first_step, int table)
{
    WinPlanArgs p = {};
    for (int64_t i = 0; i < w; ++i) p.batch_y[i] = batch_y[at + i];
    p.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    p.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    p.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    p.table = rb->ws + rb->off_wtbl[table];
    p.seed_lo = (uint32_t)seed; p.seed_hi = (uint32_t)(seed >> 32);
    p.first_step = first_step + (uint64_t)at;
    p.w = (int32_t)w;
    p.b = (int32_t)b; p.c = (int32_t)c; p.r = (int32_t)r;
    p.K = (int32_t)rb->K; p.nchunks = rb->nchunks;
    p.S = rb->S;
    p.eviction = rb->eviction;
    p.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    p.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    return p;
}

// `left` steps go into launches of at most `cap` steps: the size of the first of them when they are made as equal
// as possible (20 steps, 16 at most: 10 and 10, not 16 and 4 - a short launch hides little of the next window's plan).
int64_t even_share(int64_t left, int64_t cap)
{
    if (left <= 0) return 0;
    const int64_t launches = (left + cap - 1) / cap;
    return (left + launches - 1) / launches;
}

// Whether rb_update_sample_many puts several steps of this shape into one launch, and how many at most: the option,
// and what the planner's tables hold.  1: one launch (or two) per step.
int64_t window_limit(const rb_buffer* rb, int64_t b, int64_t c, int64_t r)
{
    const bool windowed = c >= 1 && c <= WAVE && r >= 1 && r <= WAVE && rb->nchunks <= DIRECT_CHUNKS && b <= 2048 && rb->opt_fuse &&
                          rb->opt_window >= 2 && rb->selection == RB_SELECT_EXACT;
    if (!windowed) return 1;
    return std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(WIN_MAX, rb->opt_window),
                                                  std::min<int64_t>(WIN_ENTRIES / (c + r), WIN_SLOTS / std::max(c, r))));
}

// n steps as launches of up to WIN_MAX steps each.  Workgroup 0 of every launch plans the next
// window while the others move the rows of this one; the first window is planned by a launch of its
// own and kept short, so that the movers get going early - unless the last launch of the call before
// planned it (ann_y: labels announced for the first ann_n steps of the call after this one).
int steps_windowed(rb_buffer* rb, int64_t n, const void* const* batch_x, const int64_t* const* batch_y, int64_t b, int64_t c,
                   int64_t r, uint64_t seed, uint64_t first_step, void* const* out_x, int64_t* const* out_y,
                   int64_t ann_n, const int64_t* const* ann_y)
{
    static_assert(sizeof(rb_buffer::ann_y) / sizeof(void*) >= WIN_MAX, "announced labels and planned windows are kept for a whole launch");
    const int64_t wmax = window_limit(rb, b, c, r);
    // With thousands of workgroups per launch, and the planner's LDS leaving room for four workgroups per
    // compute unit, tiles of four vectors per thread measured best (1000 classes of 3x224x224 bfloat16 samples,
    // 64 candidates and representatives: 13.1 us per step against 14.1 with two and 14.2 with eight; binary32
    // samples, 8 and 8: 3.9 against 4.1 and 4.1).  With binary32 samples stored as bfloat16 a thread holds twice as
    // many half vectors, and two per thread measured best (8 and 8: 2.6 us against 2.7).
    // With 8-bit storage a thread holds four quarter vectors per vector of the tile (16 bytes of the sample each): one.
    const int unroll_option = rb->opt_unroll;
    Shape sh = plan_shape(rb, wmax * (c + r), TPB, rb->storage == RB_STORE_U8 ? 4 : 8,
                          rb->storage == RB_STORE_U8 ? 1 : rb->storage == RB_STORE_BF16 ? 2 : 4);
    // ... and a third more tiles than that needs, i.e. tiles about three quarters full (most threads hold three vectors):
    // the launch's workgroups come in more and shorter rounds.  Measured with 301 KB rows, 64 + 64 per step: 12.42 us per step
    // with 25 to 28 tiles per row against 12.74 with the 19 that four vectors per thread need, 13.4 with 38; 602 KB rows,
    // 8 + 8 per step: 3.06 with 38 to 46 against 3.07 with 37, 3.12 with 56.
    if (unroll_option == 0 && sh.unroll == 4 && sh.tpr > 1) {
        const int64_t nunits = (rb->row_vec + TILE_UNIT - 1) / TILE_UNIT;
        sh.tpr = (int)((rb->row_vec + (int64_t)TPB * 3 - 1) / ((int64_t)TPB * 3));
        sh.tile_vec = (int)(nunits / sh.tpr);
        sh.tile_rem = (int)(nunits % sh.tpr);
    }
    // Window sizes.  A launch of w steps should not have to wait for the plan of the next window, which the one
    // planner workgroup makes meanwhile; so the windows grow as fast as that allows, and the first one (planned
    // with nothing to hide behind) is the smallest from which they can grow.  Measured on MI355X: rows move at
    // about 5.5 TB/s; a window's plan takes about 3 us more than a launch's own fixed cost, plus 1.6 us and
    // 0.04 us per candidate or representative for every step.
    const double move_us = (double)(c + r) * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;
    const double plan_us = 1.6 + 0.04 * (double)std::max(c, r);
    const auto grown = [&](int64_t w) {
        return std::max<int64_t>(1, std::min<int64_t>(wmax, (int64_t)((move_us * (double)w - 3.0) / plan_us)));
    };
    int64_t w0 = 1;
    while (w0 < wmax && grown(w0) <= w0) ++w0;
    int64_t at = 0, w;
    int tbl;
    const bool resume = window_plan_matches(rb, MANY_SMALL, n, batch_y, b, c, r, seed, first_step);
    int64_t nat;                                // size the windows have grown to, whatever a call's end cut them down to
    if (resume) {
        w = rb->wplan_w;
        tbl = rb->wplan_tbl;
        nat = rb->wplan_nat;
        rb->wplan_valid = false;                // it is being executed
    } else {
        discard_window_plan(rb);
        w = std::min(w0, n);
        nat = w0;
        tbl = 0;
        const WinPlanArgs p = window_plan_args(rb, batch_y, 0, w, b, c, r, seed, first_step, tbl);
        const auto kernel = rb->eviction != RB_EVICT_UNIFORM ? rb_window_plan_kernel<true> : rb_window_plan_kernel<false>;
        if (launch(kernel, dim3(1), TPB, 0, rb->stream, p) != hipSuccess) return RB_EHIP;
        rb->cur ^= 1;
    }
    while (at < n) {
        const int64_t next_at = at + w;
        nat = std::min(wmax, std::max(nat, grown(nat)));
        // the next window: the steps that are left in equal parts rather than full windows and a short one
        int64_t next_w = even_share(n - next_at, nat);
        // the last launch of the call plans the first steps of the call that was announced
        const bool ahead = next_w == 0 && ann_n > 0;
        if (ahead) next_w = even_share(ann_n, nat);
        WinPlanArgs next = {};
        if (ahead) next = window_plan_args(rb, ann_y, 0, next_w, b, c, r, seed, first_step + (uint64_t)n, tbl ^ 1);
        else if (next_w > 0) next = window_plan_args(rb, batch_y, next_at, next_w, b, c, r, seed, first_step, tbl ^ 1);
        WinMoveArgs m = {};
        for (int64_t k = 0; k < w; ++k) {
            m.batch_x[k] = static_cast<const vec16*>(batch_x[at + k]);
            m.out_x[k] = static_cast<vec16*>(out_x[at + k]);
            m.out_y[k] = out_y[at + k];
        }
        m.buf_x = static_cast<vec16*>(rb->buf_x);
        m.buf_y = rb->buf_y;
        m.table = rb->ws + rb->off_wtbl[tbl];
        m.state = reinterpret_cast<DevState*>(rb->ws);
        m.w = (int32_t)w; m.c = (int32_t)c; m.r = (int32_t)r;
        m.S = rb->S;
        m.row_vec = rb->row_vec;
        m.tpr = sh.tpr; m.tile_vec = sh.tile_vec; m.tile_rem = sh.tile_rem;
        const dim3 grid((unsigned)(w * (c + r) * sh.tpr + (next_w > 0 ? 1 : 0)));
        const bool aux = rb->eviction != RB_EVICT_UNIFORM;
        const hipEvent_t done = take_done(rb, next_at >= n);
        const hipError_t e = rb->opt_nt ? launch_window<true>(m, next, rb->storage, aux, sh.unroll, grid, rb->stream, done)
                                        : launch_window<false>(m, next, rb->storage, aux, sh.unroll, grid, rb->stream, done);
        if (e != hipSuccess) return RB_EHIP;
        if (next_w > 0) rb->cur ^= 1;
        if (ahead) window_plan_kept(rb, MANY_SMALL, next_w, b, c, r, seed, first_step + (uint64_t)n, tbl ^ 1, nat, ann_y);
        at = next_at;
        w = ahead ? 0 : next_w;
        tbl ^= 1;
    }
    rb->updates += n;
    return RB_OK;
}

template <int U, int W, bool NT, int ST>
hipError_t launch_bigwin_u(const BwMoveArgs& m, const BwPlanArgs& next, dim3 grid, hipStream_t st, hipEvent_t done)
{
    if constexpr (ST == RB_STORE_U8 && U > 2) {
        return hipErrorInvalidValue;           // (a lane holds four accesses per vector, and these workgroups have 128 registers per lane: bigwin_shape)
    } else {
        const size_t lds = next.w > 0 ? BIG_LDS_BYTES : 0;
        if (lds != 0) {
            const hipError_t e = allow_big_lds<&rb_bigwin_kernel<U, W, NT, ST>>();
            if (e != hipSuccess) return e;
        }
        return launch_recorded(rb_bigwin_kernel<U, W, NT, ST>, grid, BIG_TPB, lds, st, done, m, next);
    }
}

// width: threads per tile (bigwin_width), unroll: vectors per thread
template <bool NT, int ST>
hipError_t launch_bigwin_s(const BwMoveArgs& m, const BwPlanArgs& next, int width, int unroll, dim3 grid, hipStream_t st, hipEvent_t done)
{
    if (width == WAVE) return unroll == 2 ? launch_bigwin_u<2, WAVE, NT, ST>(m, next, grid, st, done) : launch_bigwin_u<8, WAVE, NT, ST>(m, next, grid, st, done);
    if (width == 2 * WAVE) return launch_bigwin_u<8, 2 * WAVE, NT, ST>(m, next, grid, st, done);
    switch (unroll) {
    case 1: return launch_bigwin_u<1, TPB, NT, ST>(m, next, grid, st, done);
    case 2: return launch_bigwin_u<2, TPB, NT, ST>(m, next, grid, st, done);
    case 4: return launch_bigwin_u<4, TPB, NT, ST>(m, next, grid, st, done);
    default: return launch_bigwin_u<8, TPB, NT, ST>(m, next, grid, st, done);
    }
}

template <bool NT>
hipError_t launch_bigwin(const BwMoveArgs& m, const BwPlanArgs& next, int storage, int width, int unroll, dim3 grid, hipStream_t st, hipEvent_t done)
{
    switch (storage) {
    case RB_STORE_BF16: return launch_bigwin_s<NT, RB_STORE_BF16>(m, next, width, unroll, grid, st, done);
    case RB_STORE_U8: return launch_bigwin_s<NT, RB_STORE_U8>(m, next, width, unroll, grid, st, done);
    default: return launch_bigwin_s<NT, RB_STORE_SAME>(m, next, width, unroll, grid, st, done);
    }
}

// Tiles of the several-steps launch for large counts.  A compute unit holds a fixed number of wavefronts, so the bytes it
// has in flight are what a wavefront has in flight: rows of up to 8 KiB are moved by one wavefront each (eight vectors per
// lane), rows of up to 16 KiB by two; longer rows are cut into tiles for 256 threads like everywhere else.
Shape bigwin_shape(const rb_buffer* rb, int64_t rows, int& width)
{
    width = TPB;
    const bool q8 = rb->storage == RB_STORE_U8;        // at most two vectors per lane: a wavefront per row up to 128 vectors
    if (rb->opt_unroll == 0 && rb->row_vec <= (q8 ? WAVE * 2 : 2 * WAVE * 8)) width = rb->row_vec <= WAVE * 8 ? WAVE : 2 * WAVE;
    // (long rows stored as bfloat16: a lane holds two half vectors per vector, four vectors measured best - 1000 classes of
    // 3x224x224 samples, 8 + 8 rows per step: 2.86 us per step against 3.05 with two and 3.39 with eight)
    if (width == TPB) return plan_shape(rb, rows, TPB, q8 ? 2 : 8, rb->storage == RB_STORE_BF16 ? 4 : 0);
    Shape s;
    s.unroll = width == WAVE && rb->row_vec <= WAVE * 2 ? 2 : 8;
    s.tpr = 1;
    const int64_t nunits = (rb->row_vec + TILE_UNIT - 1) / TILE_UNIT;
    s.tile_vec = (int)nunits;
    s.tile_rem = 0;
    s.rpb = 1;
    s.groups = rows;
    return s;
}

// Whether rb_update_sample_many puts several steps of this shape into one launch of the large-count form, and how
// many at most (1: it does not).  Shapes that the small form takes (window_limit) are not meant.  (Bernoulli selection: mini-batches that
// cannot bring more candidates than a planner has threads, so that no step of a window can lose any; the single step's plan is made for
// larger ones as well, big_coins.)
int64_t bigwin_limit(const rb_buffer* rb, int64_t b, int64_t c, int64_t r)
{
    const bool eligible = c >= 1 && c <= BIG_MAX && r >= 1 && r <= BIG_MAX && b <= BIG_BATCH &&
                          rb->K <= BIG_CLASSES && rb->opt_fuse &&
                          rb->opt_window >= 2 && (rb->selection == RB_SELECT_EXACT || b <= BIG_MAX) && rb->K * rb->S <= INT64_C(0x7FFFFFFF) &&
                          rb->S <= INT32_MAX - (int64_t)BW_MAX * RB_MAX_BATCH;
    if (!eligible) return 1;
    return std::min<int64_t>(BW_MAX, rb->opt_window);
}

BwPlanArgs bigwin_plan_args(rb_buffer* rb, const int64_t* const* batch_y, int64_t at, int64_t w, int64_t b, int64_t c, int64_t r,
                            uint64_t seed, uint64_t first_step, int table)
{
    BwPlanArgs p = {};
    for (int64_t i = 0; i < w; ++i) p.batch_y[i] = batch_y[at + i];
    p.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    p.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    p.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    p.table = rb->ws + rb->off_bwtbl[table];
    p.seed_lo = (uint32_t)seed; p.seed_hi = (uint32_t)(seed >> 32);
    p.first_step = first_step + (uint64_t)at;
    p.w = (int32_t)w;
    p.b = (int32_t)b; p.c = (int32_t)c; p.r = (int32_t)r;
    p.K = (int32_t)rb->K; p.nchunks = rb->nchunks;
    p.S = rb->S;
    p.eviction = rb->eviction;
    p.selection = rb->selection;
    p.ce = (int32_t)(rb->selection == RB_SELECT_BERNOULLI ? b : c);     // (b <= BIG_MAX then, bigwin_limit: the tables have room for BIG_MAX a step)
    rb->bw_number += 1;
    if (rb->bw_number == 0) rb->bw_number = 1;          // 0 is what a cleared flag shows
    p.number = rb->bw_number;
    rb->bw_table_number[table] = p.number;
    p.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    p.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    return p;
}

// n steps of the large-count form as launches of up to BW_MAX steps each: the first 2 w' workgroups of every launch
// plan the next window of w' steps (rb_kernels_bigwin.h) while the others move the rows of this one.  Bookkeeping as
// in steps_windowed.  The planners of a window work side by side, so a plan takes about as long whatever the
// window's size: a chain of about fifteen dependent trips to memory (measured on MI355X, 1024 candidates and
// representatives of 10000 classes: 20 to 26 us on an idle chip, 30 to 45 us under the movers' traffic), so the
// windows are of full size from the second launch on; the first window, planned with nothing to hide behind, is
// short, so that rows start to move early.
int steps_bigwin(rb_buffer* rb, int64_t n, const void* const* batch_x, const int64_t* const* batch_y, int64_t b, int64_t c,
                 int64_t r, uint64_t seed, uint64_t first_step, void* const* out_x, int64_t* const* out_y,
                 int64_t ann_n, const int64_t* const* ann_y)
{
    static_assert(BW_MAX <= WIN_MAX, "announced labels and planned windows are kept for at most WIN_MAX steps");
    const int64_t wmax = bigwin_limit(rb, b, c, r);
    // candidate entries of a step in the table, and how many of them the grid covers: all c, or, with the Bernoulli selection
    // (about c of the b positions are selected), c and eight standard deviations (more are served by going round)
    const bool bernoulli = rb->selection == RB_SELECT_BERNOULLI;
    const int64_t ce = bernoulli ? b : c;
    int64_t margin = 16;
    while (margin * margin < 64 * c) ++margin;
    const int64_t cgrid = bernoulli ? std::min(b, c + margin) : c;
    int width;
    const Shape sh = bigwin_shape(rb, wmax * (cgrid + r), width);
    const double move_us = (double)(c + r) * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;
    int64_t w0 = 1;
    while (w0 < wmax && move_us * (double)w0 < 12.0) ++w0;
    if (allow_big_lds<&rb_bigwin_plan_kernel>() != hipSuccess) return RB_EHIP;
    int64_t at = 0, w;
    int tbl;
    const bool resume = window_plan_matches(rb, MANY_LARGE, n, batch_y, b, c, r, seed, first_step);
    if (resume) {
        w = rb->wplan_w;
        tbl = rb->wplan_tbl;
        rb->wplan_valid = false;                // it is being executed
    } else {
        discard_window_plan(rb);
        w = std::min(w0, n);
        tbl = 0;
        const BwPlanArgs p = bigwin_plan_args(rb, batch_y, 0, w, b, c, r, seed, first_step, tbl);
        if (launch(rb_bigwin_plan_kernel, dim3((unsigned)(2 * w)), BIG_TPB, BIG_LDS_BYTES, rb->stream, p) != hipSuccess) return RB_EHIP;
        rb->cur ^= 1;
    }
    while (at < n) {
        const int64_t next_at = at + w;
        int64_t next_w = even_share(n - next_at, wmax);
        // the last launch of the call plans the first steps of the call that was announced
        const bool ahead = next_w == 0 && ann_n > 0;
        if (ahead) next_w = even_share(ann_n, wmax);
        BwMoveArgs m = {};
        for (int64_t k = 0; k < w; ++k) {
            m.batch_x[k] = static_cast<const vec16*>(batch_x[at + k]);
            m.out_x[k] = static_cast<vec16*>(out_x[at + k]);
            m.out_y[k] = out_y[at + k];
        }
        m.buf_x = static_cast<vec16*>(rb->buf_x);
        m.buf_y = rb->buf_y;
        m.table = rb->ws + rb->off_bwtbl[tbl];
        m.state = reinterpret_cast<DevState*>(rb->ws);
        m.w = (int32_t)w; m.c = (int32_t)ce; m.r = (int32_t)r; m.cgrid = (int32_t)cgrid;
        m.number = rb->bw_table_number[tbl];
        m.S = rb->S;
        m.row_vec = rb->row_vec;
        m.tpr = sh.tpr; m.tile_vec = sh.tile_vec; m.tile_rem = sh.tile_rem;
        BwPlanArgs next = {};
        if (ahead) next = bigwin_plan_args(rb, ann_y, 0, next_w, b, c, r, seed, first_step + (uint64_t)n, tbl ^ 1);
        else if (next_w > 0) next = bigwin_plan_args(rb, batch_y, next_at, next_w, b, c, r, seed, first_step, tbl ^ 1);
        const int64_t items = w * (cgrid + r) * sh.tpr;
        const int64_t per_block = BIG_TPB / width;
        const dim3 grid((unsigned)((items + per_block - 1) / per_block + 2 * next_w));
        const hipEvent_t done = take_done(rb, next_at >= n);
        const hipError_t e = rb->opt_nt ? launch_bigwin<true>(m, next, rb->storage, width, sh.unroll, grid, rb->stream, done)
                                        : launch_bigwin<false>(m, next, rb->storage, width, sh.unroll, grid, rb->stream, done);
        if (e != hipSuccess) return RB_EHIP;
        if (next_w > 0) rb->cur ^= 1;
        if (ahead) window_plan_kept(rb, MANY_LARGE, next_w, b, c, r, seed, first_step + (uint64_t)n, tbl ^ 1, wmax, ann_y);
        at = next_at;
        w = ahead ? 0 : next_w;
        tbl ^= 1;
    }
    rb->updates += n;
    return RB_OK;
}

// Which several-steps form serves this shape (MANY_SINGLE: none) and how many steps it puts into one launch at most.
// Where both forms could: the one workgroup that plans a window of the small form does so step after step (about
// 1.6 us + 0.04 us per candidate or representative each, 2.3 to 2.7 us under load), which is hidden as long as the rows
// of a step take longer to move; the two planners per step of the large form work side by side and take as long for
// sixteen steps as for one, but their launch moves long rows about 6 % slower, and rows that are converted on the way
// 15 to 25 % slower.  Measured on MI355X, us per step, small form against large form: 8 + 8 rows of 12 KB 2.7 : 1.05;
// 8 + 8 rows of 301 KB 2.59 : 2.07, 12 + 12 of them 2.88 : 2.86, 16 + 16 3.09 : 3.37; 4 + 4 rows of 602 KB 2.26 : 2.07,
// 6 + 6 2.52 : 2.58, 8 + 8 3.08 : 3.32; 8 + 8 rows of 602 KB stored as bfloat16 2.54 : 3.22, in 8 bits 2.5 : 2.9.  So the
// large form takes a shape when its rows move (at 5.5 TB/s) in less than 1.25 times the small form's nominal plan time,
// in less than 0.8 times when they are converted.  RB_OPT_PLANNERS overrides the choice where the shape allows.
int many_form(const rb_buffer* rb, int64_t b, int64_t c, int64_t r, int64_t& steps)
{
    const int64_t small = window_limit(rb, b, c, r), large = bigwin_limit(rb, b, c, r);
    int form = MANY_SINGLE;
    if (small >= 2 && large >= 2) {
        const double move_us = (double)(c + r) * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;
        const double plan_us = 1.6 + 0.04 * (double)std::max(c, r);
        form = move_us < (rb->storage == RB_STORE_SAME ? 1.25 : 0.8) * plan_us ? MANY_LARGE : MANY_SMALL;
        if (rb->opt_planners != 0) form = rb->opt_planners;
    } else if (small >= 2) {
        form = MANY_SMALL;
    } else if (large >= 2) {
        form = MANY_LARGE;
    }
    steps = form == MANY_SMALL ? small : form == MANY_LARGE ? large : 1;
    return form;
}

template <int U, bool NT, int ST, bool BERNOULLI>
hipError_t launch_one_u(const OneArgs& a, dim3 grid, size_t lds, hipStream_t st)
{
    if constexpr ((ST == RB_STORE_U8 && U > 1) || (ST == RB_STORE_BF16 && U > 2)) {
        return hipErrorInvalidValue;           // (converted rows: step_one)
    } else {
        constexpr int most = 4 * (ONE_CLASSES + ONE_CLASSES / 32 + ONE_CHUNKS + (int)ONE_MATE_WORDS + 4 * RB_MAX_BATCH) + 2 * RB_MAX_BATCH;      // one_lds_bytes at its largest
        static_assert(most <= 156 * 1024, "a compute unit has 160 KB of LDS");
        constexpr auto kernel = &rb_step_one_kernel<U, NT, ST, BERNOULLI>;
        const hipError_t e = allow_big_lds<kernel, most>();
        if (e != hipSuccess) return e;
        const UpdateArgs& u = a.u;
        return launch(kernel, grid, ONE_TPB, lds, st, u.batch_y, u.fill_old, a.chunk_old, u.sd.seed_lo, u.sd.seed_hi, u.sd.step_lo, u.sd.step_hi,
                      (uint32_t)(u.b | u.c << 16), (uint32_t)(a.r | u.nchunks << 16), a.first_cand, a);
    }
}

template <bool NT, int ST, bool BERNOULLI>
hipError_t launch_one_s(const OneArgs& a, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    // (without streaming accesses: one kernel per storage form, the one with the most vectors per lane)
    if constexpr (!NT) return launch_one_u<ST == RB_STORE_U8 ? 1 : ST == RB_STORE_BF16 ? 2 : 8, NT, ST, BERNOULLI>(a, grid, lds, st);
    else switch (unroll) {
    case 1: return launch_one_u<1, NT, ST, BERNOULLI>(a, grid, lds, st);
    case 2: return launch_one_u<2, NT, ST, BERNOULLI>(a, grid, lds, st);
    case 4: return launch_one_u<4, NT, ST, BERNOULLI>(a, grid, lds, st);
    default: return launch_one_u<8, NT, ST, BERNOULLI>(a, grid, lds, st);
    }
}

template <bool NT, bool BERNOULLI>
hipError_t launch_one_f(const OneArgs& a, int storage, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    switch (storage) {
    case RB_STORE_BF16: return launch_one_s<NT, RB_STORE_BF16, BERNOULLI>(a, unroll, grid, lds, st);
    case RB_STORE_U8: return launch_one_s<NT, RB_STORE_U8, BERNOULLI>(a, unroll, grid, lds, st);
    default: return launch_one_s<NT, RB_STORE_SAME, BERNOULLI>(a, unroll, grid, lds, st);
    }
}

template <bool NT>
hipError_t launch_one(const OneArgs& a, int storage, int unroll, dim3 grid, size_t lds, hipStream_t st)
{
    return a.u.selection == RB_SELECT_BERNOULLI ? launch_one_f<NT, true>(a, storage, unroll, grid, lds, st) : launch_one_f<NT, false>(a, storage, unroll, grid, lds, st);
}

// Tiles of `rows` rows for `waves` wavefronts that take one tile after the other: as many tiles per row as make the
// wavefronts' shares equal, with at most `most` vectors per lane.  Returns the vectors per lane they need.
int one_tiles(const rb_buffer* rb, int64_t rows, int64_t waves, int most, int32_t& tpr, int32_t& tile_vec, int32_t& tile_rem)
{
    const int64_t units = (rb->row_vec + TILE_UNIT - 1) / TILE_UNIT;
    int64_t n = (units + most - 1) / most;
    if (rb->opt_unroll == 0) {
        const int64_t rounds = (rows * n + waves - 1) / waves;
        n = std::max(n, std::min(units, rounds * waves / rows));
    }
    tpr = (int32_t)n;
    tile_vec = (int32_t)(units / n);
    tile_rem = (int32_t)(units % n);
    return (int)((units + n - 1) / n);
}

// Shapes whose whole plan one wavefront can make: rb_step_small_kernel, and the plan-ahead step of rb_kernels_planned.h.
bool small_counts(const rb_buffer* rb, int64_t c, int64_t r)
{
    return c >= 1 && c <= WAVE && r >= 1 && r <= WAVE && rb->nchunks <= DIRECT_CHUNKS && rb->opt_fuse && rb->selection == RB_SELECT_EXACT;
}

// How rb_update_sample carries out a step that is not planned ahead: STEP_SMALL (rb_step_small_kernel), STEP_ONE
// (rb_step_one_kernel) or STEP_TWO (the two kernels of rb_update and rb_sample_augment).
// STEP_ONE as long as the fill counts fit LDS, work items and a class's count with a step's candidates on top (not yet cut
// off at the capacity) are counted in 32 bits, and the rows are moved soon enough: with one workgroup of planners and movers per
// compute unit long rows move slower than in the general kernels, rows that are converted most of all, and of those the
// representatives', whose workgroups have the longer plan in front of them.  The lines are drawn by the time the rows take at 5.5 TB/s, all of
// them and the representatives', from 12800 random shapes (2 to 10000 classes, mini-batches of 16 to 4096, rows of 256 bytes to 602 KB, up
// to 45 us of rows, all strategies) measured on MI355X both ways.  Two launches against one, geometric mean of the shapes in a range
// and their 5th percentile, on this and on the far side of the lines:
//   plain, exact           representatives 8 to 14 us   1.06 (0.98)      16 to 20 us   1.01 (0.96)     20 to 30   0.98 (0.91)
//   plain, Bernoulli       12 to 18                     1.09 (1.01)      20 to 30      1.03 (0.98)
//   bfloat16, exact        4 to 6                       1.11 (0.99)      10 to 12      1.02 (0.93)     12 to 14   1.00 (0.94)
//   bfloat16, Bernoulli    6 to 8                       1.16 (1.05)      16 to 20      1.03 (0.93)     20 to 30   0.99 (0.92)
//   8 bits, exact          2 to 3                       1.13 (0.99)      3 to 4        1.05 (0.89)     6 to 8     0.99 (0.89)
//   8 bits, Bernoulli      2 to 3                       1.19 (0.99)      3 to 4        1.08 (0.82)     10 to 12   0.96 (0.84)
// (Long rows, more than 192 KB or 80 KB as bfloat16, exact selection with uniform or FIFO replacement, beyond the lines for few rows below: 553
// shapes 1.04, half of them more than 3 % faster and 1 of 15 more than 3 % slower in one launch; bfloat16 rows beyond 130 KB 1.00.)
// More than 1024 candidates: the two launches' search for class-mates grows with their square (plain rows beyond 14 us 1.54, bfloat16 beyond
// 5.5 us 1.47, 8 bits beyond 4 us 1.40), and the lines lie further out.  Nearer they lie, or none are drawn further than before, for
//   few long rows, up to 128: plain, exact, beyond 14 us 1.01 (0.95), up to 128 candidates 1.03; bfloat16, representatives beyond 3.3 us, up to 64 rows
//     1.04; and up to 64 on either side, exact, when the two launches are those of the small-count kernels, a workgroup per tile: plain 5.5 to 7 us
//     1.04 (0.91), 8 to 10 0.99; bfloat16 5.5 to 7 1.01 (0.94), 7 to 8 0.96; 8 bits 2 to 3 1.04, 3 to 4 1.01 (0.93);
//   more than 1024 representatives of short rows, which the sampling kernel moves as well: rows of up to 13 KB, plain, beyond 14 us 7 of 10 slower
//     in one launch, 8 bits beyond 2.8 us 8 of 10;
//   converted rows of fewer than 32 classes, or more candidates than slots: those of candidates that lose their slot to a later one are read
//     (8 bits, FIFO, 7 classes, 236 + 8 rows of 567 KB 48 : 37 us; more than 1.9 candidates per slot 4 of 5 slower).
constexpr double ONE_MEASURED_US = 45.0;     // most time of rows the two forms were compared with
enum { STEP_TWO = 0, STEP_SMALL = 1, STEP_ONE = 2 };
int step_form(const rb_buffer* rb, int64_t c, int64_t r)
{
    if (small_counts(rb, c, r)) return STEP_SMALL;
    const bool exact = rb->selection == RB_SELECT_EXACT, small_two = exact && c <= WAVE && r <= WAVE, many = c > BIG_MAX;
    const double one_us = (double)(c + r) * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;     // the rows, all and the representatives'
    const double reps_us = (double)r * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;
    const bool further = !small_two && c + r > 2 * WAVE && r <= BIG_MAX && (rb->storage == RB_STORE_SAME || (rb->K >= 32 && c <= rb->K * rb->S));
    double one_most, reps_most;
    switch (rb->storage) {
    case RB_STORE_U8:
        one_most = !further ? 2.0 : many ? ONE_MEASURED_US : exact ? 4.0 : 5.5;
        reps_most = !further ? 2.0 : many ? 8.0 : 3.0;
        break;
    case RB_STORE_BF16:
        one_most = !further ? 5.5 : many ? ONE_MEASURED_US : 20.0;
        reps_most = !further ? 3.3 : many ? 12.0 : exact ? 6.0 : 8.0;
        break;
    default:
        one_most = small_two ? 8.0 : !further || (exact && c <= 2 * WAVE) ? 14.0 : ONE_MEASURED_US;
        reps_most = !further || (exact && !many) ? 14.0 : 18.0;
    }
    if (one_us >= one_most || reps_us >= reps_most) return STEP_TWO;
    // Representatives that cannot exist leave the workgroups they are dealt to idle, and the others, planned by eight wavefronts
    // each, take longer than one wavefront per row of the two launches: 9 + 3754 rows of 128 bytes, 360 slots, 11.9 : 8.6 us;
    // 15 + 2593 of 1.5 KB, 120 slots, 10.6 : 8.2; 9 + 552 of 36 KB, 120 slots, 10.9 : 9.9; 17 + 185 in 8 bits, 160 slots, 10.0 : 9.3.
    if (r > rb->K * rb->S) return STEP_TWO;
    // A representative of a class that overwrites slots in this step searches the step's candidates of that class, in the two
    // launches nobody does.  With few classes, i.e. many candidates of each (labels that occur equally often assumed), that
    // costs more than a launch, sooner with FIFO and reservoir replacement, where the two launches' candidates need no search
    // or mostly none.  One launch against two, rows of 2 KB: uniform replacement, 10 classes 4096 + 4096 [410 candidates per
    // class] 64 : 114 us, 4 classes 2000 + 2000 [500] 32.1 : 30.2, 2 classes 2000 + 2000 [1000] 40 : 33; reservoir, 1 class
    // 150 + 150 9.1 : 9.0 and 600 + 600 14.9 : 11.2, as bfloat16 2 classes 150 + 150 [75] 9.9 : 9.0 and 4 classes 600 + 600
    // [150] 13.2 : 11.9, 10 classes 1000 + 1000 [100] 13.1 : 15.6 and 4096 + 4096 [410] 54.6 : 50.1, 50 classes 4096 + 4096
    // [82] 44.5 : 60.9; FIFO, 1 class 600 + 600 11.8 : 10.6.
    const int64_t mates = rb->eviction == RB_EVICT_UNIFORM ? 448 : std::max<int64_t>(WAVE, 8 * rb->K + 32);
    if (c > mates * rb->K) return STEP_TWO;
    // Every representative's workgroup copies all fill counts into LDS, and summed them as well when this was measured: 0.21 us per 1000
    // classes then, which the second launch does not cost.  What that one costs instead, measured at 2000 classes, where the counts are nearly free, grows with the rows; two
    // launches of the small-count kernels cost least.  One launch against two, rows of 3 KB, at 6000 / 8000 / 10000 classes:
    // as they are 5 + 5 rows 7.5 : 7.3 at 6000; 17 + 7, FIFO, 8.3 : 8.1 at 5076; 30 + 30 7.9 : 8.0 at 6000; 109 + 29 8.2 : 8.5, 9.1 : 8.6 (7832 classes); 200 + 200
    // 8.7 : 9.4 at 6000; 400 + 400 9.7 : 10.7, 10.1 : 10.7, 10.5 : 10.8; 1000 + 1000 13.6 : 16.2 at 10000.  As bfloat16 5 + 5
    // 7.6 : 7.6 at 4000, 8.9 : 7.6 at 10000; 30 + 30 8.3 : 8.4, 8.6 : 8.2; 200 + 200 9.0 : 9.8, 9.5 : 9.9, 9.9 : 9.9.  In 8 bits 5 + 5
    // 8.5 : 8.3 at 4000, 10.1 : 8.3 at 10000; 200 + 200 10.1 : 10.2, 10.5 : 10.1; 1000 + 1000 15.1 : 15.1 at 10000.  Bernoulli
    // selection, as they are, 5 + 5 7.9 : 7.9, 8.4 : 7.9; 109 + 29 8.2 : 8.6, 8.6 : 8.7, 9.0 : 8.9; 200 + 200 9.5 : 10.0 at 10000; in
    // 8 bits 30 + 30 9.3 : 9.5, 9.8 : 9.7, 10.2 : 9.5.  (With the old sums per chunk the counts cost 0.1 us per 1000 classes, and the line is
    // nearer than it need be: beyond it two launches take 1.2 times as long with the general kernels, 1.02 to 1.08 with the small-count ones.)
    const bool u8 = rb->storage == RB_STORE_U8;
    const double rows = (double)(c + r);
    const double second_us = rb->selection == RB_SELECT_BERNOULLI ? (u8 ? 0.72 : 0.82) + 0.004 * rows
                           : small_two ? (rb->storage == RB_STORE_SAME ? 0.4 + 0.0085 * rows : 0.3 + 0.007 * rows)
                           : u8 ? 0.63 + 0.0005 * rows : 0.85 + 0.0019 * rows;
    if (0.21e-3 * (double)(rb->K - 2000) > second_us) return STEP_TWO;
    if (c >= 1 && r >= 1 && rb->K <= ONE_CLASSES && rb->opt_fuse &&
        rb->S <= INT32_MAX - RB_MAX_BATCH && (rb->row_vec + TILE_UNIT - 1) / TILE_UNIT <= INT32_MAX / 2 / RB_MAX_BATCH)
        return STEP_ONE;
    return STEP_TWO;
}

// Whether an announced step with the Bernoulli selection goes through the planners of large counts.  Mini-batches of up to BIG_MAX positions
// always do.  Of larger ones the step that was not announced is the other form: it makes all coins and draws in front of its rows, a plan is
// made beside them, but takes longer than short rows where
//   FIFO or reservoir replacement has the update planner keep the state of many classes, and its threads meet at the counters of classes
//     with many candidates (labels, which the host cannot see), while the other form is a single launch.  What a plan saves and costs there,
//     in us, is fitted to 11300 shapes; 0.3 of the 1.2 are not, they leave shapes that are about equal to the plan;
//   a single class has all candidates: more than 300 of them 0.91, FIFO and reservoir replacement 0.80 times as fast when planned.
// Unannounced steps' time over announced ones' (singly or 16 a call, the worse), random shapes of 1025 to 4096 positions, a quarter each of
// them with labels of three classes, of fifty, skewed and uniform ones:
//   all counts, classes, rows up to 8 us, strategies: 1.29, 1.0 % more than 3 % slower when announced (all of them planned: 1.4 %);
//   FIFO and reservoir, 2500 to 10240 classes, 64 to 512 candidates, rows up to 6 us: 1.12, 11 % (1.10, 21 %);
//   up to 3000 classes, 200 to 512 candidates, rows up to 5 us: 1.25, 7 % (1.24, 8 %).
// The steps that are not planned would be 0.79 to 0.92 times as fast, one in nine of them more than 3 % faster.
bool plans_coins(const rb_buffer* rb, int64_t b, int64_t c, int64_t r)
{
    if (!big_coins(b, c)) return false;
    if (b <= BIG_MAX) return true;
    const double rows_us = (double)(c + r) * (double)(rb->row_bytes + rb->sample_bytes) / 5.5e6;
    if (rb->K == 1) return c <= 300 || rows_us >= 4.0;
    if (rb->eviction == RB_EVICT_UNIFORM || rows_us >= 6.0 || step_form(rb, c, r) != STEP_ONE) return true;
    const double saves_us = 1.2 + 0.22e-3 * (double)b + 2.5e-3 * (double)r + 0.6 * std::max(0.0, rows_us - 1.5);
    const double costs_us = 0.67e-6 * (double)rb->K * (double)(c + 200) + 0.9e-3 * (double)c;
    return saves_us >= costs_us;
}

// Update and sampling of one step in one launch without a plan (rb_kernels_one.h).
int step_one(rb_buffer* rb, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c, int64_t r,
             uint64_t seed, uint64_t step, void* out_x, int64_t* out_y)
{
    OneArgs oa;
    UpdateArgs& a = oa.u;
    a.batch_x = static_cast<const vec16*>(batch_x);
    a.batch_y = batch_y;
    a.buf_x = static_cast<vec16*>(rb->buf_x);
    a.buf_y = rb->buf_y;
    a.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    a.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    a.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    a.state = reinterpret_cast<DevState*>(rb->ws);
    a.sd = make_seed(seed, step);
    a.b = (int32_t)b; a.c = (int32_t)c;
    a.K = (int32_t)rb->K; a.nchunks = rb->nchunks;
    a.S = rb->S;
    a.row_vec = rb->row_vec;
    a.rpb = 1;
    a.selection = rb->selection; a.eviction = rb->eviction;
    a.cap = (int32_t)(rb->selection == RB_SELECT_BERNOULLI ? b : c);
    a.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    a.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    oa.out_x = static_cast<vec16*>(out_x);
    oa.out_y = out_y;
    oa.r = (int32_t)r;
    oa.chunk_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_chunk[rb->cur]);
    // rows the grid is sized for (Bernoulli selection: the mean and about one standard deviation; the movers loop, and a grid
    // sized for more leaves that many more wavefronts without work)
    int64_t rows = c;
    if (rb->selection == RB_SELECT_BERNOULLI) {
        int64_t slack = 0;
        while (slack * slack < c) ++slack;
        rows = std::min(b, c + slack);
    }
    constexpr int64_t CUS = 256;                // one workgroup per compute unit, dealt to the two sides by their rows
    const int64_t most_r = std::min<int64_t>(CUS - 1, std::max<int64_t>(1, (CUS * r + (rows + r) / 2) / (rows + r)));
    // (rows that are converted: small tiles.  612 + 625 rows of 11.5 KB in 8 bits 15.6 us with one vector per lane, 17.8 with two,
    // 20.5 with four; as bfloat16 13.9, 12.9 with two, 14.2)
    int limit = rb->storage == RB_STORE_U8 ? 1 : rb->storage == RB_STORE_BF16 ? 2 : 8;
    if (rb->opt_unroll != 0) limit = std::min(limit, rb->opt_unroll);
    const int uc = one_tiles(rb, rows, (CUS - most_r) * ONE_NWAVE, limit, a.tpr, a.tile_vec, a.tile_rem);
    const int ur = one_tiles(rb, r, most_r * ONE_NWAVE, limit, oa.tpr, oa.tile_vec, oa.tile_rem);
    int unroll = 1;
    while (unroll < std::max(uc, ur)) unroll <<= 1;
    // (the representatives' workgroups keep the books as well: at least as many of them as give every wavefront one chunk of classes.
    // reservoir replacement, Bernoulli selection, 5 + 5 rows of 3 KB of 6000 classes 7.1 -> 6.7 us; with FIFO replacement and 10000 classes
    // one of them took five chunks per wavefront, one behind the other, 9.5 to 9.8 us, against 7.2 to 7.4)
    const int64_t nr = std::max<int64_t>(std::min(most_r, (r * oa.tpr + ONE_NWAVE - 1) / ONE_NWAVE), (rb->nchunks + ONE_NWAVE - 1) / ONE_NWAVE);
    const int64_t nc = std::min(CUS - std::max(most_r, nr), (rows * a.tpr + ONE_NWAVE - 1) / ONE_NWAVE);
    oa.first_cand = (int32_t)nr;
    oa.share = (int32_t)((r * oa.tpr + nr - 1) / nr);
    oa.cshare = rb->selection == RB_SELECT_BERNOULLI ? 0 : (int32_t)((c * a.tpr + nc - 1) / nc);
    oa.nwg = (int32_t)(nr + nc);
    const dim3 grid((unsigned)(nr + nc));
    const size_t lds = one_lds_bytes((int)b, a.cap, (int)r, rb->nchunks);
    const hipError_t e = rb->opt_nt ? launch_one<true>(oa, rb->storage, unroll, grid, lds, rb->stream)
                                    : launch_one<false>(oa, rb->storage, unroll, grid, lds, rb->stream);
    if (e != hipSuccess) return RB_EHIP;
    rb->cur ^= 1;
    rb->updates += 1;
    return RB_OK;
}

// What the host can check of the arguments of one update + sample step.
int check_step(const rb_buffer* rb, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c, int64_t r,
               const void* out_x, const int64_t* out_y)
{
    if (!rb || !batch_x || !batch_y) return RB_EINVAL;
    if (b < 1 || b > RB_MAX_BATCH || c < 0 || c > b) return RB_EINVAL;
    if (!aligned(batch_x, 16) || !aligned(batch_y, 8)) return RB_EINVAL;
    if (r < 0 || r > RB_MAX_BATCH) return RB_EINVAL;
    if (r > 0 && (!out_x || !out_y || !aligned(out_x, 16) || !aligned(out_y, 8))) return RB_EINVAL;
    if (!rb->bound) return RB_ESTATE;
    return RB_OK;
}

}  // namespace

// The asynchronous form of the single primitive: two events order the training stream and the
// buffer's stream against each other.
struct rb_pipeline {
    rb_buffer* rb;
    hipEvent_t ready;     // on the training stream: mini-batch produced, earlier representatives consumed
    hipEvent_t done;      // on the buffer's stream: the latest step's update and sampling are complete
    bool recorded;        // `done` has been recorded behind that step (wait_done)
    int64_t prev_r;       // rows the latest step asked for
    bool started;         // at least one step has been enqueued
    uint64_t stream_number;   // the buffer's stream then (rb_buffer::stream_number)
};

// What a failed operation on streams or events leaves is not left for others either (launch).
static bool succeeded(hipError_t e)
{
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

static bool captured(hipStream_t stream)
{
    hipStreamCaptureStatus status;
    return !succeeded(hipStreamIsCapturing(stream, &status)) || status != hipStreamCaptureStatusNone;       // (no telling: taken for captured)
}

// Makes `train` wait for the latest step.  A call whose training stream is the buffer's own records no event, which nobody may ever wait
// for; then it is recorded here, behind whatever else has gone to that stream (the caller has ordered it behind the stream the step ran on
// if the handle has been given another one since).
static bool wait_done(rb_pipeline* p, hipStream_t train)
{
    if (!p->recorded) {
        if (!succeeded(hipEventRecord(p->done, p->rb->stream))) return false;
        p->recorded = true;
    }
    return succeeded(hipStreamWaitEvent(train, p->done, 0));
}

// The two streams' hand-over before a call's steps: the training stream goes on once the previous call's representatives are complete,
// the buffer's stream starts these steps once the training stream has got this far.  The latter need not wait for the former, which
// the buffer's stream has behind it: after rb_pipeline_drain, when the training stream waits a second time, that wait is not in the
// way of the steps (32 iterations of 8 + 8 rows of 602 KB a call 121.5 -> 116.5 us).  It goes first where the handle has been given
// another stream since, and into a graph that is being captured (it is refused if those representatives come from outside, and
// then nothing has been captured).
static bool hand_over(rb_pipeline* p, hipStream_t train)
{
    const bool first = p->started && (!p->recorded || p->stream_number != p->rb->stream_number || captured(train));
    if (first && !wait_done(p, train)) return false;
    if (!succeeded(hipEventRecord(p->ready, train)) || !succeeded(hipStreamWaitEvent(p->rb->stream, p->ready, 0))) return false;
    return first || !p->started || wait_done(p, train);
}

extern "C" {

int rb_create(rb_buffer** out, int64_t classes, int64_t slots_per_class,
              const int64_t* sample_shape, int32_t ndim, int32_t dtype)
{
    if (!out) return RB_EINVAL;
    *out = nullptr;
    if (!sample_shape || ndim < 1 || ndim > 16) return RB_EINVAL;
    if (classes < 1 || classes > RB_MAX_CLASSES || slots_per_class < 1) return RB_EINVAL;
    if (slots_per_class > RB_MAX_SLOTS / classes) return RB_EINVAL;
    if (dtype != RB_F32 && dtype != RB_BF16) return RB_EINVAL;
    int64_t elems = 1;
    for (int i = 0; i < ndim; ++i) {
        if (sample_shape[i] < 1) return RB_EINVAL;
        if (elems > (INT64_C(1) << 40) / sample_shape[i]) return RB_EINVAL;   // a row of more than 2^40 elements
        elems *= sample_shape[i];
    }
    const int64_t row_bytes = elems * (dtype == RB_F32 ? 4 : 2);
    if (row_bytes % 16 != 0) return RB_EINVAL;
    rb_buffer* rb = new (std::nothrow) rb_buffer();
    if (!rb) return RB_ENOMEM;
    rb->K = classes;
    rb->S = slots_per_class;
    rb->row_bytes = row_bytes;
    rb->row_vec = row_bytes / 16;
    rb->sample_bytes = row_bytes;
    rb->dtype = dtype;
    rb->storage = RB_STORE_SAME;
    rb->nchunks = (int32_t)((classes + CH - 1) / CH);
    rb->buf_x = nullptr; rb->buf_y = nullptr; rb->ws = nullptr; rb->stream = nullptr;
    rb->bound = false;
    rb->host_rows = false;
    rb->static_dev = -1;
    rb->cur = 0;
    size_t off = STATE_BYTES;
    const size_t fill_bytes = round_up((size_t)rb->nchunks * CH * sizeof(int32_t), 256);
    const size_t chunk_bytes = round_up((size_t)rb->nchunks * sizeof(int32_t), 256);
    rb->off_fill[0] = off; off += fill_bytes;
    rb->off_fill[1] = off; off += fill_bytes;
    rb->off_chunk[0] = off; off += chunk_bytes;
    rb->off_chunk[1] = off; off += chunk_bytes;
    rb->off_aux[0] = off; off += fill_bytes;
    rb->off_aux[1] = off; off += fill_bytes;
    rb->off_tbl[0] = off; off += PLAN_BYTES;
    rb->off_tbl[1] = off; off += PLAN_BYTES;
    rb->off_wtbl[0] = off; off += WIN_TABLE_BYTES;
    rb->off_wtbl[1] = off; off += WIN_TABLE_BYTES;
    rb->off_bfwd[0] = off; off += BIG_FWD_BYTES;
    rb->off_bfwd[1] = off; off += BIG_FWD_BYTES;
    rb->off_bwtbl[0] = off; off += BW_TABLE_BYTES;
    rb->off_bwtbl[1] = off; off += BW_TABLE_BYTES;
    rb->bw_number = 0; rb->bw_table_number[0] = 0; rb->bw_table_number[1] = 0;
    rb->ws_bytes = off;
    rb->tbl_next = 0; rb->tbl_planned = 0; rb->plan_valid = false; rb->plan_y = nullptr; rb->next_y = nullptr;
    rb->ann_n = 0; rb->wplan_valid = false; rb->wplan_tbl = 0;
    rb->selection = RB_SELECT_EXACT; rb->eviction = RB_EVICT_UNIFORM; rb->updates = 0;
    rb->opt_unroll = 0; rb->opt_nt = 1; rb->opt_rpb = 0; rb->opt_fuse = 1; rb->opt_window = WIN_MAX; rb->opt_planners = 0;
    *out = rb;
    return RB_OK;
}

int rb_query_sizes(const rb_buffer* rb, size_t* x_bytes, size_t* y_bytes, size_t* workspace_bytes)
{
    if (!rb) return RB_EINVAL;
    if (x_bytes) *x_bytes = (size_t)rb->K * (size_t)rb->S * (size_t)rb->row_bytes;
    if (y_bytes) *y_bytes = (size_t)rb->K * (size_t)rb->S * sizeof(int64_t);
    if (workspace_bytes) *workspace_bytes = rb->ws_bytes;
    return RB_OK;
}

int rb_set_storage(rb_buffer* rb, int32_t storage)
{
    if (!rb) return RB_EINVAL;
    if (storage != RB_STORE_SAME && storage != RB_STORE_BF16 && storage != RB_STORE_U8) return RB_EINVAL;
    if (rb->bound) return RB_ESTATE;                 // the storage the caller bound was sized for the other form
    if (storage == RB_STORE_BF16 && (rb->dtype != RB_F32 || rb->sample_bytes % 32 != 0)) return RB_EINVAL;
    if (storage == RB_STORE_U8 && (rb->dtype != RB_F32 || rb->sample_bytes % 64 != 0)) return RB_EINVAL;
    rb->storage = storage;
    rb->row_bytes = storage == RB_STORE_BF16 ? rb->sample_bytes / 2 : storage == RB_STORE_U8 ? rb->sample_bytes / 4 : rb->sample_bytes;
    rb->row_vec = rb->row_bytes / 16;
    return RB_OK;
}

namespace {
// The handle no longer uses a device's static scratch array.
void release_scratch(rb_buffer* rb)
{
    if (rb->static_dev >= 0 && scratch_holder[rb->static_dev] == rb) scratch_holder[rb->static_dev] = nullptr;
    rb->static_dev = -1;
}
}  // namespace

int rb_bind(rb_buffer* rb, void* buf_x, int64_t* buf_y, void* workspace, void* hip_stream)
{
    if (!rb || !buf_x || !buf_y || !workspace) return RB_EINVAL;
    if (!aligned(buf_x, 16) || !aligned(buf_y, 8) || !aligned(workspace, 256)) return RB_EINVAL;
    if (rb->static_dev >= 0 && workspace != scratch_ptr[rb->static_dev]) release_scratch(rb);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int64_t slots = rb->K * rb->S;
    int64_t blocks = (slots + TPB - 1) / TPB;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (launch(rb_reset_kernel, dim3((unsigned)blocks), TPB, 0, st, static_cast<uint32_t*>(workspace), (int64_t)(rb->ws_bytes / 4), buf_y, slots) != hipSuccess)
        return RB_EHIP;
    rb->buf_x = buf_x;
    rb->buf_y = buf_y;
    rb->ws = static_cast<char*>(workspace);
    rb->stream = st;
    rb->stream_number += 1;
    rb->cur = 0;
    rb->updates = 0;
    rb->plan_valid = false; rb->next_y = nullptr; rb->tbl_next = 0;
    rb->ann_n = 0; rb->wplan_valid = false;
    rb->bw_number = 0; rb->bw_table_number[0] = 0; rb->bw_table_number[1] = 0;     // (the reset clears the planners' flags)
    rb->host_rows = in_host_memory(buf_x);
    rb->bound = true;
    return RB_OK;
}

int rb_bind_static(rb_buffer* rb, void* buf_x, int64_t* buf_y, void* hip_stream)
{
    if (!rb || !buf_x || !buf_y) return RB_EINVAL;
    if (!aligned(buf_x, 16) || !aligned(buf_y, 8)) return RB_EINVAL;
    if (rb->ws_bytes > sizeof scratch) return RB_ELIMIT;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return RB_EHIP;
    if (!scratch_ptr[dev]) {
        // first use on this device (which is current): where this device's copy of the array lives
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return RB_EHIP;
        scratch_ptr[dev] = p;
    }
    rb_buffer* before = scratch_holder[dev];
    if (rb->static_dev >= 0 && rb->static_dev != dev) release_scratch(rb);
    rb->static_dev = dev;                          // (rb_bind keeps the array with this handle)
    const int rc = rb_bind(rb, buf_x, buf_y, scratch_ptr[dev], hip_stream);   // clears what the handle uses of the array, on the stream
    if (rc != RB_OK) {
        if (before != rb) rb->static_dev = -1;
        return rc;
    }
    if (before && before != rb) {                  // the array changes hands: the other handle has no workspace any more
        before->bound = false;
        before->static_dev = -1;
    }
    scratch_holder[dev] = rb;
    return RB_OK;
}

int rb_set_stream(rb_buffer* rb, void* hip_stream)
{
    if (!rb) return RB_EINVAL;
    rb->stream = static_cast<hipStream_t>(hip_stream);
    rb->stream_number += 1;
    return RB_OK;
}

int rb_set_policy(rb_buffer* rb, int32_t selection, int32_t eviction)
{
    if (!rb) return RB_EINVAL;
    if (selection != RB_SELECT_EXACT && selection != RB_SELECT_BERNOULLI) return RB_EINVAL;
    if (eviction != RB_EVICT_UNIFORM && eviction != RB_EVICT_FIFO && eviction != RB_EVICT_RESERVOIR) return RB_EINVAL;
    if (rb->updates != 0) return RB_ESTATE;      // the per-class state of one strategy means nothing to another
    rb->selection = selection;
    rb->eviction = eviction;
    return RB_OK;
}

int rb_update(rb_buffer* rb, const void* batch_x, const int64_t* batch_y,
              int64_t b, int64_t c, uint64_t seed, uint64_t step)
{
    if (!rb || !batch_x || !batch_y) return RB_EINVAL;
    if (b < 1 || b > RB_MAX_BATCH || c < 0 || c > b) return RB_EINVAL;
    if (!aligned(batch_x, 16) || !aligned(batch_y, 8)) return RB_EINVAL;
    if (!rb->bound) return RB_ESTATE;
    discard_plan(rb);
    if (c == 0) return RB_OK;

    const int narrow = rb->storage == RB_STORE_BF16 ? 1 : rb->storage == RB_STORE_U8 ? 2 : 0;
    const bool small = c <= WAVE && rb->selection == RB_SELECT_EXACT;
    // Rows the grid is sized for.  The Bernoulli selection yields a random number of candidates
    // (mean c, at most b); the movers loop over the work items, so any number is handled, and
    // the grid only has to be large enough for the usual case.
    int64_t rows = c;
    if (rb->selection == RB_SELECT_BERNOULLI) {
        int64_t slack = 16;
        while (slack * slack < 36 * c) ++slack;          // about six standard deviations
        rows = c + slack < b ? c + slack : b;
    }
    // (converted rows, general kernel: 100 + 90 bfloat16 rows of 602 KB 40.0 us with eight vectors per lane, 38.1 with four.  Every
    // tile repeats the plan's pass over the candidate list, so from about 770 candidates on rows that have several large tiles
    // keep those.  Both calls, r = 64, large against small tiles: bfloat16 rows of 49 KB 600 candidates 18.5 : 18.5 us,
    // 800 23.1 : 22.9, 900 24.7 : 26.1, 1000 25.4 : 28.1; of 192 KB 600 44.7 : 43.9, 800 55.8 : 57.6, 1000 66.5 : 71.8; 8 bits,
    // 49 KB, 700 21.0 : 20.4, 900 22.9 : 25.1; rows of 12 KB, one large tile, 1024 as bfloat16 15.4 : 14.5, 8 bits 16.5 : 15.2)
    // (Bernoulli selection: a coin per position of the mini-batch in every workgroup, and 6 bytes of LDS for it, so the size of the
    // mini-batch counts as well: large against small tiles, rb_update alone, bfloat16 rows of 602 KB, mini-batch of 512 / 1024 / 2048 / 4096,
    // c = 10 [537 workgroups of small tiles] 6.3 : 5.6, 6.8 : 6.0, 7.7 : 7.0, 9.2 : 10.2, c = 60 [1980] 14.3 : 14.0, 15.1 : 15.4, 17.0 : 19.0,
    // 21.4 : 25.7; of 192 KB, c = 60 [642] 7.0 : 7.2, 7.5 : 7.6, 8.6 : 8.9, 10.2 : 11.4; in 8 bits alike.  The chosen form is within 3 % of
    // the better one at each of 72 shapes, 49 to 602 KB, c = 10, 60 and 200)
    const int64_t small_tiles = (rb->row_vec + WAVE * (narrow == 2 ? 2 : 4) - 1) / (WAVE * (narrow == 2 ? 2 : 4));
    const bool coins = rb->selection == RB_SELECT_BERNOULLI && (b >= 3072 || (b >= 1024 && rows * small_tiles > 1024 * NWAVE));
    const bool many = !small && (c > BIG_MAX || coins || (rows > 768 && rb->row_vec > WAVE * (narrow == 2 ? 4 : 8)));
    const Shape sh = plan_shape(rb, rows, small ? TPB : WAVE, narrow == 2 ? (many ? 4 : 2) : narrow == 1 && !small && !many ? 4 : 8);
    UpdateArgs a;
    a.batch_x = static_cast<const vec16*>(batch_x);
    a.batch_y = batch_y;
    a.buf_x = static_cast<vec16*>(rb->buf_x);
    a.buf_y = rb->buf_y;
    a.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    a.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    a.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    a.state = reinterpret_cast<DevState*>(rb->ws);
    a.sd = make_seed(seed, step);
    a.b = (int32_t)b; a.c = (int32_t)c;
    a.K = (int32_t)rb->K; a.nchunks = rb->nchunks;
    a.S = rb->S;
    a.row_vec = rb->row_vec;
    a.tpr = sh.tpr; a.tile_vec = sh.tile_vec; a.tile_rem = sh.tile_rem; a.rpb = sh.rpb;
    a.selection = rb->selection; a.eviction = rb->eviction;
    a.cap = (int32_t)(rb->selection == RB_SELECT_BERNOULLI ? b : c);
    a.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    a.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    const dim3 grid((unsigned)(rb->nchunks + (small ? sh.groups * sh.tpr : (rows * sh.tpr + NWAVE - 1) / NWAVE)));
    const size_t lds = small ? small_lds_bytes(b, rb->nchunks) : gen_update_lds_bytes((int)b, a.cap, rb->selection == RB_SELECT_BERNOULLI);
    const bool ordinary = ordinary_stores(rb, c, STORES_HALF);
    const hipError_t e = small ? (rb->opt_nt ? launch_update_small<true>(a, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary)
                                             : launch_update_small<false>(a, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary))
                               : (rb->opt_nt ? launch_update<true>(a, narrow, sh.unroll, grid, lds, rb->stream)
                                             : launch_update<false>(a, narrow, sh.unroll, grid, lds, rb->stream));
    if (e != hipSuccess) return RB_EHIP;
    rb->cur ^= 1;
    rb->updates += 1;
    return RB_OK;
}

int rb_sample_augment(rb_buffer* rb, int64_t r, uint64_t seed, uint64_t step, void* out_x, int64_t* out_y)
{
    if (!rb || r < 0 || r > RB_MAX_BATCH) return RB_EINVAL;
    if (r > 0 && (!out_x || !out_y || !aligned(out_x, 16) || !aligned(out_y, 8))) return RB_EINVAL;
    if (!rb->bound) return RB_ESTATE;
    discard_plan(rb);
    if (r == 0) return RB_OK;

    const int widen = rb->storage == RB_STORE_BF16 ? 1 : rb->storage == RB_STORE_U8 ? 2 : 0;
    const bool small = r <= WAVE && rb->nchunks <= WAVE;
    const Shape sh = small ? sample_small_shape(rb, r) : plan_shape(rb, r, WAVE, widen == 2 ? 2 : widen == 1 ? 4 : 8);
    SampleArgs a;
    a.buf_x = static_cast<const vec16*>(rb->buf_x);
    a.out_x = static_cast<vec16*>(out_x);
    a.out_y = out_y;
    a.fill = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    a.chunk = reinterpret_cast<const int32_t*>(rb->ws + rb->off_chunk[rb->cur]);
    a.state = reinterpret_cast<DevState*>(rb->ws);
    a.sd = make_seed(seed, step);
    a.r = (int32_t)r;
    a.K = (int32_t)rb->K; a.nchunks = rb->nchunks;
    a.S = rb->S;
    a.row_vec = rb->row_vec;
    a.tpr = sh.tpr; a.tile_vec = sh.tile_vec; a.tile_rem = sh.tile_rem; a.rpb = sh.rpb;
    const dim3 grid((unsigned)(small ? sh.groups * sh.tpr : (r * sh.tpr + NWAVE - 1) / NWAVE));
    const size_t lds = small ? 0 : gen_sample_lds_bytes((int)r, rb->nchunks);
    const bool ordinary = ordinary_stores(rb, r, STORES_HALF);
    const hipError_t e = small ? (rb->opt_nt ? launch_sample_small<true>(a, rb->storage, sh.unroll, grid, rb->stream, ordinary)
                                             : launch_sample_small<false>(a, rb->storage, sh.unroll, grid, rb->stream, ordinary))
                               : (rb->opt_nt ? launch_sample<true>(a, widen, sh.unroll, grid, lds, rb->stream)
                                             : launch_sample<false>(a, widen, sh.unroll, grid, lds, rb->stream));
    return e == hipSuccess ? RB_OK : RB_EHIP;
}

int rb_update_sample(rb_buffer* rb, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c,
                     int64_t r, uint64_t seed, uint64_t step, void* out_x, int64_t* out_y)
{
    const int bad = check_step(rb, batch_x, batch_y, b, c, r, out_x, out_y);
    if (bad != RB_OK) return bad;
    discard_window_plan(rb);                     // a single step is not what a planned window was made for
    rb->ann_n = 0;

    const bool plannable = small_counts(rb, c, r);
    // larger counts have a plan-ahead form of their own
    // (with the Bernoulli selection, whose number of candidates is only bounded by b, where plans_coins says so)
    const bool big = !plannable && c >= 1 && c <= BIG_MAX && r >= 1 && r <= BIG_MAX && b <= BIG_BATCH &&
                     rb->K <= BIG_CLASSES && rb->opt_fuse && (rb->selection == RB_SELECT_EXACT || plans_coins(rb, b, c, r)) &&
                     rb->K * rb->S <= INT64_C(0x7FFFFFFF) && rb->S <= INT32_MAX - RB_MAX_BATCH;
    const int64_t* next_y = rb->next_y;
    rb->next_y = nullptr;                        // an announcement serves one call
    if (rb->plan_valid && !((plannable || big) && rb->plan_y == batch_y && rb->plan_b == b && rb->plan_c == c && rb->plan_r == r &&
                            rb->plan_seed == seed && rb->plan_step == step))
        discard_plan(rb);
    if (plannable && (rb->plan_valid || next_y))
        return step_planned(rb, batch_x, batch_y, b, c, r, seed, step, out_x, out_y, next_y);
    if (big && (rb->plan_valid || next_y))
        return step_big(rb, batch_x, batch_y, b, c, r, seed, step, out_x, out_y, next_y);
    // (results that lie over the mini-batch: a single launch would write them while it still reads it)
    const int64_t bx = b * rb->sample_bytes, by = b * (int64_t)sizeof(int64_t), ox = r * rb->sample_bytes, oy = r * (int64_t)sizeof(int64_t);
    const bool apart = !overlap(out_y, oy, batch_y, by) && !overlap(out_x, ox, batch_x, bx) && !overlap(out_y, oy, batch_x, bx) &&
                       !overlap(out_x, ox, batch_y, by);
    const int form = apart ? step_form(rb, c, r) : STEP_TWO;
    if (form == STEP_ONE) return step_one(rb, batch_x, batch_y, b, c, r, seed, step, out_x, out_y);
    if (form == STEP_TWO) {
        const int rc = rb_update(rb, batch_x, batch_y, b, c, seed, step);
        if (rc != RB_OK) return rc;
        return rb_sample_augment(rb, r, seed, step, out_x, out_y);
    }
    // (bfloat16 rows: 64 + 64 rows of 602 KB 28.8 us with eight vectors per thread, 25.3 with four)
    const Shape sh = plan_shape(rb, c + r, TPB, rb->storage == RB_STORE_U8 ? 2 : rb->storage == RB_STORE_BF16 ? 4 : 8, 0, 256);
    StepArgs sa;
    UpdateArgs& a = sa.u;
    a.batch_x = static_cast<const vec16*>(batch_x);
    a.batch_y = batch_y;
    a.buf_x = static_cast<vec16*>(rb->buf_x);
    a.buf_y = rb->buf_y;
    a.fill_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_fill[rb->cur]);
    a.fill_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_fill[rb->cur ^ 1]);
    a.chunk_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_chunk[rb->cur ^ 1]);
    a.state = reinterpret_cast<DevState*>(rb->ws);
    a.sd = make_seed(seed, step);
    a.b = (int32_t)b; a.c = (int32_t)c;
    a.K = (int32_t)rb->K; a.nchunks = rb->nchunks;
    a.S = rb->S;
    a.row_vec = rb->row_vec;
    a.tpr = sh.tpr; a.tile_vec = sh.tile_vec; a.tile_rem = sh.tile_rem; a.rpb = 1;
    a.selection = RB_SELECT_EXACT; a.eviction = rb->eviction; a.cap = (int32_t)c;
    a.aux_old = reinterpret_cast<const int32_t*>(rb->ws + rb->off_aux[rb->cur]);
    a.aux_new = reinterpret_cast<int32_t*>(rb->ws + rb->off_aux[rb->cur ^ 1]);
    sa.out_x = static_cast<vec16*>(out_x);
    sa.out_y = out_y;
    sa.r = (int32_t)r;
    const dim3 grid((unsigned)(rb->nchunks + (c + r) * sh.tpr));
    const size_t lds = small_lds_bytes(b, rb->nchunks);
    const bool ordinary = ordinary_stores(rb, c + r, STORES_STEP);
    const hipError_t e = rb->opt_nt ? launch_step<true>(sa, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary)
                                    : launch_step<false>(sa, rb->storage, sh.unroll, grid, lds, rb->stream, ordinary);
    if (e != hipSuccess) return RB_EHIP;
    rb->cur ^= 1;
    rb->updates += 1;
    return RB_OK;
}

int rb_announce_next(rb_buffer* rb, const int64_t* next_batch_y)
{
    if (!rb) return RB_EINVAL;
    if (next_batch_y && !aligned(next_batch_y, 8)) return RB_EINVAL;
    rb->next_y = next_batch_y;
    return RB_OK;
}

int rb_query_steps_per_launch(const rb_buffer* rb, int64_t b, int64_t c, int64_t r, int64_t* steps)
{
    if (!rb || !steps) return RB_EINVAL;
    if (b < 1 || b > RB_MAX_BATCH || c < 0 || c > b || r < 0 || r > RB_MAX_BATCH) return RB_EINVAL;
    (void)many_form(rb, b, c, r, *steps);
    return RB_OK;
}

int rb_query_launches(const rb_buffer* rb, int64_t b, int64_t c, int64_t r, int64_t* launches)
{
    if (!rb || !launches) return RB_EINVAL;
    if (b < 1 || b > RB_MAX_BATCH || c < 0 || c > b || r < 0 || r > RB_MAX_BATCH) return RB_EINVAL;
    *launches = step_form(rb, c, r) != STEP_TWO ? 1 : (c > 0) + (r > 0);
    return RB_OK;
}

int rb_announce_next_many(rb_buffer* rb, int64_t n, const int64_t* const* next_batch_y)
{
    if (!rb || n < 0 || (n > 0 && !next_batch_y)) return RB_EINVAL;
    const int64_t keep = std::min<int64_t>(n, WIN_MAX);        // more than one launch can cover is of no use
    for (int64_t i = 0; i < keep; ++i)
        if (!next_batch_y[i] || !aligned(next_batch_y[i], 8)) return RB_EINVAL;
    for (int64_t i = 0; i < keep; ++i) rb->ann_y[i] = next_batch_y[i];
    rb->ann_n = keep;
    return RB_OK;
}

int rb_update_sample_many(rb_buffer* rb, int64_t n, const void* const* batch_x, const int64_t* const* batch_y,
                          int64_t b, int64_t c, int64_t r, uint64_t seed, uint64_t first_step,
                          void* const* out_x, int64_t* const* out_y)
{
    if (!rb || n < 0 || !batch_x || !batch_y) return RB_EINVAL;
    if (r > 0 && (!out_x || !out_y)) return RB_EINVAL;
    // what was announced is about the call after this one and serves this call only
    const int64_t ann_n = rb->ann_n;
    const int64_t* ann_y[WIN_MAX];
    for (int64_t i = 0; i < ann_n; ++i) ann_y[i] = rb->ann_y[i];
    rb->ann_n = 0;
    for (int64_t i = 0; i < n; ++i) {
        const int bad = check_step(rb, batch_x[i], batch_y[i], b, c, r, r > 0 ? out_x[i] : nullptr, r > 0 ? out_y[i] : nullptr);
        if (bad != RB_OK) return bad;
    }
    int64_t per_launch;
    const int form = n >= 2 ? many_form(rb, b, c, r, per_launch) : MANY_SINGLE;
    if (form != MANY_SINGLE) {
        if (rb->plan_valid) {                    // a single step that was planned ahead is not executed as planned
            rb->cur ^= 1;
            rb->plan_valid = false;
        }
        rb->next_y = nullptr;
        return form == MANY_SMALL ? steps_windowed(rb, n, batch_x, batch_y, b, c, r, seed, first_step, out_x, out_y, ann_n, ann_y)
                                  : steps_bigwin(rb, n, batch_x, batch_y, b, c, r, seed, first_step, out_x, out_y, ann_n, ann_y);
    }
    discard_window_plan(rb);
    for (int64_t i = 0; i < n; ++i) {
        // the next step's labels are known: plan ahead (also across calls when the next call's first labels were announced)
        rb->next_y = i + 1 < n ? batch_y[i + 1] : (ann_n > 0 ? ann_y[0] : nullptr);
        const int rc = rb_update_sample(rb, batch_x[i], batch_y[i], b, c, r, seed, first_step + (uint64_t)i,
                                        r > 0 ? out_x[i] : nullptr, r > 0 ? out_y[i] : nullptr);
        if (rc != RB_OK) return rc;      // only a failed launch can get here
    }
    return RB_OK;
}

int rb_pipeline_create(rb_pipeline** out, rb_buffer* rb)
{
    if (!out) return RB_EINVAL;
    *out = nullptr;
    if (!rb) return RB_EINVAL;
    rb_pipeline* p = new (std::nothrow) rb_pipeline();
    if (!p) return RB_ENOMEM;
    p->rb = rb;
    p->prev_r = 0;
    p->recorded = false;
    p->started = false;
    p->stream_number = 0;
    if (!succeeded(hipEventCreateWithFlags(&p->ready, hipEventDisableTiming))) {
        delete p;
        return RB_EHIP;
    }
    if (!succeeded(hipEventCreateWithFlags(&p->done, hipEventDisableTiming))) {
        (void)hipEventDestroy(p->ready);
        delete p;
        return RB_EHIP;
    }
    *out = p;
    return RB_OK;
}

int rb_pipeline_step(rb_pipeline* p, const void* batch_x, const int64_t* batch_y, int64_t b, int64_t c,
                     int64_t r, uint64_t seed, uint64_t step, void* next_x, int64_t* next_y,
                     void* train_stream, int64_t* ready_rows)
{
    if (!p) return RB_EINVAL;
    rb_buffer* rb = p->rb;
    const int bad = check_step(rb, batch_x, batch_y, b, c, r, next_x, next_y);
    if (bad != RB_OK) return bad;
    hipStream_t train = static_cast<hipStream_t>(train_stream);
    const bool two_streams = train != rb->stream;
    // (1) the training stream may go on once the previous step's representatives are complete
    if (two_streams && !hand_over(p, train)) return RB_EHIP;
    p->recorded = false;                        // (should anything fail from here on, wait_done is for all that the buffer's stream has got)
    // (2) update with this mini-batch, then collect the next representatives
    const int rc = rb_update_sample(rb, batch_x, batch_y, b, c, r, seed, step, next_x, next_y);
    if (rc != RB_OK) return rc;
    if (two_streams && !succeeded(hipEventRecord(p->done, rb->stream))) return RB_EHIP;
    if (ready_rows) *ready_rows = p->started ? p->prev_r : 0;
    p->prev_r = r;
    p->recorded = two_streams;
    p->started = true;
    p->stream_number = rb->stream_number;
    return RB_OK;
}

int rb_pipeline_drain(rb_pipeline* p, void* train_stream, int64_t* ready_rows)
{
    if (!p) return RB_EINVAL;
    hipStream_t train = static_cast<hipStream_t>(train_stream);
    if (p->started && train != p->rb->stream && !wait_done(p, train)) return RB_EHIP;
    if (ready_rows) *ready_rows = p->started ? p->prev_r : 0;
    return RB_OK;
}

int rb_pipeline_step_many(rb_pipeline* p, int64_t n, const void* const* batch_x, const int64_t* const* batch_y,
                          int64_t b, int64_t c, int64_t r, uint64_t seed, uint64_t first_step,
                          void* const* next_x, int64_t* const* next_y, void* train_stream, int64_t* ready_rows)
{
    if (!p || n < 0 || !batch_x || !batch_y) return RB_EINVAL;
    if (r > 0 && (!next_x || !next_y)) return RB_EINVAL;
    rb_buffer* rb = p->rb;
    // everything is checked before the first stream operation, so that an error leaves nothing behind
    for (int64_t i = 0; i < n; ++i) {
        const int bad = check_step(rb, batch_x[i], batch_y[i], b, c, r, r > 0 ? next_x[i] : nullptr, r > 0 ? next_y[i] : nullptr);
        if (bad != RB_OK) return bad;
    }
    if (n == 0) {
        if (ready_rows) *ready_rows = p->started ? p->prev_r : 0;
        return RB_OK;
    }
    hipStream_t train = static_cast<hipStream_t>(train_stream);
    const bool two_streams = train != rb->stream;
    // (1) the training stream may go on once the previous call's representatives are complete
    if (two_streams && !hand_over(p, train)) return RB_EHIP;
    p->recorded = false;                        // (as in rb_pipeline_step)
    // (2) the n updates, each followed by the collection of the next representatives
    // (their last launch records the event, except into a graph that is being captured, and when the steps go out one by one)
    if (two_streams && !captured(rb->stream)) rb->done = p->done;
    const bool asked = rb->done != nullptr;
    const int rc = rb_update_sample_many(rb, n, batch_x, batch_y, b, c, r, seed, first_step, next_x, next_y);
    const bool recorded = asked && rb->done == nullptr;
    rb->done = nullptr;
    if (rc != RB_OK) return rc;
    if (two_streams && !recorded && !succeeded(hipEventRecord(p->done, rb->stream))) return RB_EHIP;
    if (ready_rows) *ready_rows = p->started ? p->prev_r : 0;
    p->prev_r = r;
    p->recorded = two_streams;
    p->started = true;
    p->stream_number = rb->stream_number;
    return RB_OK;
}

int rb_pipeline_destroy(rb_pipeline* p)
{
    if (!p) return RB_EINVAL;
    const bool ok = hipEventDestroy(p->ready) == hipSuccess;
    const bool ok2 = hipEventDestroy(p->done) == hipSuccess;
    delete p;
    return ok && ok2 ? RB_OK : RB_EHIP;
}

int rb_read_state(rb_buffer* rb, int32_t* fill_host, int64_t* last_n_host, uint32_t* flags_host)
{
    if (!rb) return RB_EINVAL;
    if (!rb->bound) return RB_ESTATE;
    discard_plan(rb);
    if (hipStreamSynchronize(rb->stream) != hipSuccess) return RB_EHIP;
    DevState st;
    if (hipMemcpy(&st, rb->ws, sizeof st, hipMemcpyDeviceToHost) != hipSuccess) return RB_EHIP;
    if (fill_host &&
        hipMemcpy(fill_host, rb->ws + rb->off_fill[rb->cur], (size_t)rb->K * sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess)
        return RB_EHIP;
    if (last_n_host) *last_n_host = st.last_n;
    if (flags_host) *flags_host = st.flags;
    return RB_OK;
}

int rb_read_moved_rows(rb_buffer* rb, uint64_t* rows_host)
{
    if (!rb || !rows_host) return RB_EINVAL;
    if (!rb->bound) return RB_ESTATE;
    discard_plan(rb);
    if (hipStreamSynchronize(rb->stream) != hipSuccess) return RB_EHIP;
    static_assert(MOVED_STRIDE % sizeof(uint64_t) == 0, "counters are read as an array of 64-bit words");
    uint64_t words[MOVED_COUNTERS * MOVED_STRIDE / sizeof(uint64_t)];
    if (hipMemcpy(words, rb->ws + STATE_HEAD_BYTES, sizeof words, hipMemcpyDeviceToHost) != hipSuccess) return RB_EHIP;
    uint64_t sum = 0;
    for (int i = 0; i < MOVED_COUNTERS; ++i) sum += words[i * (MOVED_STRIDE / sizeof(uint64_t))];
    *rows_host = sum;
    return RB_OK;
}

int rb_set_option(rb_buffer* rb, int32_t option, int64_t value)
{
    if (!rb) return RB_EINVAL;
    switch (option) {
    case RB_OPT_UNROLL:
        if (value != 0 && value != 1 && value != 2 && value != 4 && value != 8) return RB_EINVAL;
        rb->opt_unroll = (int)value;
        return RB_OK;
    case RB_OPT_NONTEMPORAL:
        if (value != 0 && value != 1) return RB_EINVAL;
        rb->opt_nt = (int)value;
        return RB_OK;
    case RB_OPT_ROWS_PER_BLOCK:
        if (value < 0 || value > 16) return RB_EINVAL;
        rb->opt_rpb = (int)value;
        return RB_OK;
    case RB_OPT_FUSE:
        if (value != 0 && value != 1) return RB_EINVAL;
        rb->opt_fuse = (int)value;
        return RB_OK;
    case RB_OPT_WINDOW:
        if (value < 1 || value > WIN_MAX) return RB_EINVAL;
        rb->opt_window = (int)value;
        return RB_OK;
    case RB_OPT_PLANNERS:
        if (value < 0 || value > 2) return RB_EINVAL;
        rb->opt_planners = (int)value;
        return RB_OK;
    default:
        return RB_EINVAL;
    }
}

int rb_destroy(rb_buffer* rb)
{
    if (rb) release_scratch(rb);
    delete rb;
    return RB_OK;
}

const char* rb_strerror(int status)
{
    switch (status) {
    case RB_OK: return "ok";
    case RB_EINVAL: return "invalid argument";
    case RB_ENOMEM: return "out of host memory";
    case RB_ESTATE: return "buffer is not bound to device storage";
    case RB_EHIP: return "a HIP call failed";
    case RB_ELIMIT: return "the buffer needs more workspace than the library's static scratch array holds";
    default: return "unknown status";
    }
}

int rb_standin_compute(void* hip_stream, float* sink, int64_t blocks, int64_t iters)
{
    if (!sink || blocks < 1 || blocks > (1 << 20) || iters < 0) return RB_EINVAL;
    const hipError_t e = launch(rb_standin_kernel, dim3((unsigned)blocks), TPB, 0, static_cast<hipStream_t>(hip_stream), sink, iters);
    return e == hipSuccess ? RB_OK : RB_EHIP;
}

int rb_copy_bytes(void* hip_stream, void* dst, const void* src, size_t bytes, int32_t unroll, int32_t nontemporal)
{
    if (!dst || !src || bytes == 0 || bytes % 16 != 0 || !aligned(dst, 16) || !aligned(src, 16)) return RB_EINVAL;
    if (unroll != 1 && unroll != 2 && unroll != 4 && unroll != 8) return RB_EINVAL;
    const int64_t nvec = (int64_t)(bytes / 16);
    if ((nvec + (int64_t)TPB * unroll - 1) / ((int64_t)TPB * unroll) > 0x7FFFFFFF) return RB_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    vec16* d = static_cast<vec16*>(dst);
    const vec16* s = static_cast<const vec16*>(src);
    hipError_t e = nontemporal == 2 ? launch_copy<true, 64>(d, s, nvec, unroll, st)
                 : nontemporal      ? launch_copy<true, 1>(d, s, nvec, unroll, st)
                                    : launch_copy<false, 1>(d, s, nvec, unroll, st);
    return e == hipSuccess ? RB_OK : RB_EHIP;
}

}  // extern "C"
