// Seeding and plain-generation kernels for gfx950 (CDNA4, wave64).
//
// init:  one state per work-item, state[g] = H(seed, g) (Listing S4).
// gen:   a persistent loop per lane. The lane loads its states once, then for
//        every iteration k stores them to row k of the iteration-major output
//        and advances them one xorshift step (Listing S5), and finally writes
//        them back. The paper's kernel reads and writes 16 bytes of state per
//        value per launch; here state traffic is 16 bytes per work-item per
//        call, and each value costs only its 8 (or 4) output bytes.
// paced: the same on a persistent grid that keeps to a row schedule, for rows
//        of any alignment (staged through LDS so that whole lines are stored)
//        and, when the rows are too short to fill the device, with the
//        iterations cut into segments that run side by side.
//
// Store layout: a wavefront owns 64 * V consecutive work-items (V = 2*P for
// 64-bit output, 4*P for 32-bit), split into P "chunk columns". In column p,
// lane l owns the 16 bytes at work-items [base + p*64*E + l*E, +E), E = 16 /
// sizeof(T). So every store instruction of the wave writes one contiguous
// 1 KiB line-aligned span (global_store_dwordx4 from all 64 lanes) whenever
// the row starts on a 128-byte line. Only staged rows use LDS per value.
#include <algorithm>
#include <atomic>

#include "device.h"
#include "internal.h"

namespace rngx {
namespace {

typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void init_kernel(uint64_t *__restrict__ state, uint32_t n,
                                                   SeedMix mix)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += stride)
        state[g] = init_state(mix, (uint32_t)g);
}

// The word emitted for state x. The paper's generator emits the state (its
// low half for 32-bit output). The scrambled variant emits the state times
// 2685821657736338717 modulo 2^64 (the xorshift* multiplier of Vigna, 2016),
// its high half for 32-bit output; the state sequence is the same.
constexpr uint64_t kStarMultiplier = 2685821657736338717ull;
template <typename T, bool STAR> __device__ __forceinline__ T emit(uint64_t x);
template <> __device__ __forceinline__ uint64_t emit<uint64_t, false>(uint64_t x) { return x; }
template <> __device__ __forceinline__ uint32_t emit<uint32_t, false>(uint64_t x)
{
    return (uint32_t)x;
}
template <> __device__ __forceinline__ uint64_t emit<uint64_t, true>(uint64_t x)
{
    return x * kStarMultiplier;
}
template <> __device__ __forceinline__ uint32_t emit<uint32_t, true>(uint64_t x)
{
    return (uint32_t)((x * kStarMultiplier) >> 32);
}

template <typename T> struct Vec16;
template <> struct Vec16<uint64_t> {
    static constexpr int E = 2;
    typedef u64x2 type;
    template <bool STAR> __device__ static __forceinline__ type pack(const uint64_t *x)
    {
        return type{emit<uint64_t, STAR>(x[0]), emit<uint64_t, STAR>(x[1])};
    }
};
template <> struct Vec16<uint32_t> {
    static constexpr int E = 4;
    typedef u32x4 type;
    template <bool STAR> __device__ static __forceinline__ type pack(const uint64_t *x)
    {
        return type{emit<uint32_t, STAR>(x[0]), emit<uint32_t, STAR>(x[1]),
                    emit<uint32_t, STAR>(x[2]), emit<uint32_t, STAR>(x[3])};
    }
};

template <bool NT, typename VT> __device__ __forceinline__ void store16(VT *p, VT v)
{
    if (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Output words of one 128-byte line, the unit in which the device's memory
// takes writes whole.
template <typename T> constexpr uint32_t kLine = 128 / sizeof(T);

// One complete wavefront, all iterations, in place, unscheduled: its 64*P*E
// work-items starting at wbase.
template <typename T, int P, bool NT, bool ALIGNED, bool STAR>
__device__ __forceinline__ void full_wave(uint64_t *__restrict__ state, uint32_t n,
                                          uint32_t iters, T *__restrict__ out, uint64_t wbase,
                                          uint32_t lane)
{
    typedef Vec16<T> VT;
    constexpr int E = VT::E;
    uint64_t x[P][E];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
#pragma unroll
        for (int e = 0; e < E; ++e)
            x[p][e] = state[g + e];
    }
    for (uint32_t k = 0; k < iters; ++k) {
        T *row = out + (size_t)k * n;
        const bool al = ALIGNED || ((reinterpret_cast<uintptr_t>(row) & 15u) == 0);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
            if (al) {
                store16<NT>(reinterpret_cast<typename VT::type *>(row + g),
                            VT::template pack<STAR>(x[p]));
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    row[g + e] = emit<T, STAR>(x[p][e]);
            }
#pragma unroll
            for (int e = 0; e < E; ++e)
                x[p][e] = xs_step(x[p][e]);
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
#pragma unroll
        for (int e = 0; e < E; ++e)
            state[g + e] = x[p][e];
    }
}

// The last, partial wavefront: element-wise guarded (the paper's
// gid < nseeds test).
template <typename T, int P, bool STAR>
__device__ __forceinline__ void partial_wave(uint64_t *__restrict__ state, uint32_t n,
                                             uint32_t iters, T *__restrict__ out, uint64_t wbase,
                                             uint32_t lane)
{
    constexpr int E = Vec16<T>::E;
    uint64_t x[P][E];
    uint32_t cnt[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
        cnt[p] = g >= n ? 0u : (uint32_t)((n - g) < (uint64_t)E ? (n - g) : E);
#pragma unroll
        for (int e = 0; e < E; ++e)
            x[p][e] = (uint32_t)e < cnt[p] ? state[g + e] : 0u;
    }
    for (uint32_t k = 0; k < iters; ++k) {
        T *row = out + (size_t)k * n;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if ((uint32_t)e < cnt[p])
                    row[g + e] = emit<T, STAR>(x[p][e]);
        }
        // Apart from the guarded stores, so that lanes with and without a
        // word take their steps together (in one loop with the stores the
        // compiler gave each side its own: 1 x 200 u32 of 4 chunks 102 us, 79).
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int e = 0; e < E; ++e)
                x[p][e] = xs_step(x[p][e]);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((uint32_t)e < cnt[p])
                state[g + e] = x[p][e];
    }
}

// P chunk columns per lane; NT: non-temporal stores; ALIGNED: every row
// start is 16-byte aligned.
template <typename T, int P, bool NT, bool ALIGNED, bool STAR>
__global__ __launch_bounds__(1024) void gen_kernel(uint64_t *__restrict__ state, uint32_t n,
                                                   uint32_t iters, T *__restrict__ out)
{
    constexpr uint64_t WAVE_ITEMS = 64ull * P * Vec16<T>::E;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t wbase = wave * WAVE_ITEMS;
    if (wbase >= n)
        return;
    if (wbase + WAVE_ITEMS <= n)
        full_wave<T, P, NT, ALIGNED, STAR>(state, n, iters, out, wbase, lane);
    else
        partial_wave<T, P, STAR>(state, n, iters, out, wbase, lane);
}

// ---- the scheduled launch --------------------------------------------------

// A persistent grid of gridDim.x blocks, all resident at once, walks strips of
// columns. Every wavefront keeps to one row schedule from its own start t0
// (its first clock reading): its row number j, counted over all its strips, is
// written no earlier than t0 + j * delta256 / 256 clock ticks, so the
// wavefronts write near the same row instead of drifting apart. (Measured on
// MI355X: one start time shared by the whole grid, the first wavefront's, ran
// 3-20 % slower at 2^20-2^24 states and the same at 2^26.) The strips are of
// equal size: a grid as large as fits leaves a last strip of few blocks that
// takes as long as a full one (2,200,000 x 256 u64: 6.9 TB/s, 4.7 so).
//
// Bound by the memory's writes: 2^22 x 256 u64 7.0 TB/s at a schedule of 7,000
// GB/s, where a large fill runs at 6.7. Registers decide whether every block
// the occupancy query promises is resident: all variants stay within 64 vector
// registers (8 wavefronts per SIMD) but those of four 4-byte chunks (80-86),
// and within 80 scalar ones (with 88, of 8 wavefronts per SIMD only 7 were
// resident and a launch took twice its time).
//
// Staged rows (SHIFT). A row that does not start on a 128-byte line has its
// wavefronts' spans end inside lines, which then reach the memory in parts
// (half the rate). Here a wavefront writes the lines that START in its
// columns: it also keeps the kLine states right of them (one per lane, about
// 6 % more steps), puts the row's words into LDS in column order and reads
// them back at the row's line offset, so its stores are whole lines again.
// LDS moves 32 bytes per 16 stored, a quarter of its rate at 7 TB/s.
// 10^6 + 3 states x 256: u64 4.1 -> 6.9 TB/s, u32 4.1 -> 6.6.
//
// Segments (Polys = JumpPolys). A row of n states occupies n / 128 wavefronts
// (u64); below some 500 they cannot have enough stores under way. So the
// iterations are cut into segments, each computed by its own blocks from the
// states jumped ahead by T^(first row) (build_jump, nibble_product); the blocks of
// the last segment write the new states. 4,096 x 10,000 u64: 1,650 -> 55 us
// (0.2 -> 6.0 TB/s), 65,536 x 1,000: 173 -> 80 us.
//
// In both, wavefronts read states that others advance, so the new states go
// to another buffer.
struct PacedArgs {
    const uint64_t *state_in;
    uint64_t *state_out; // state_in itself for an in-place launch
    void *out;
    uint32_t n, iters;
    uint32_t seg_rows;   // iterations per segment (iters: one segment)
    uint32_t col_blocks; // blocks that cover one row
    uint32_t items;      // segments * col_blocks
    uint64_t delta256;   // schedule step, clock ticks * 256 (0: none)
    uint32_t burst;      // rows per schedule step
};

// T^k as a nibble table in LDS for one block: `poly` holds the 64
// coefficients of T^k = sum over i of poly_i T^i. Lane j of the first
// wavefront forms T^k e_j by 64 steps from e_j (about 1 us; no memory);
// entry v of table q is then T^k (v << 4q).
__device__ __forceinline__ void build_jump(uint64_t poly, uint64_t *cols, uint64_t *tab)
{
    __syncthreads(); // the block is done with the previous table
    if (threadIdx.x < 64) {
        uint64_t e = (uint64_t)1 << threadIdx.x, y = 0;
#pragma unroll 8
        for (int i = 0; i < 64; ++i) {
            y ^= e & (0 - ((poly >> i) & 1u));
            e = xs_step(e);
        }
        cols[threadIdx.x] = y;
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < 256; t += blockDim.x) {
        uint64_t y = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            y ^= (t >> b) & 1u ? cols[(t >> 4) * 4 + b] : 0;
        tab[t] = y;
    }
    __syncthreads();
}

// 16 bytes at any word of LDS.
__device__ __forceinline__ u64x2 lds_chunk(const uint64_t *p)
{
    typedef u64x2 u64x2_w __attribute__((aligned(8)));
    return *reinterpret_cast<const u64x2_w *>(p);
}
__device__ __forceinline__ u32x4 lds_chunk(const uint32_t *p)
{
    typedef u32x4 u32x4_w __attribute__((aligned(4)));
    return *reinterpret_cast<const u32x4_w *>(p);
}

constexpr uint32_t kAheadRows = 4;

// Keeps the value's computation before this point.
__device__ __forceinline__ void pin(uint64_t &x) { asm volatile("" : "+v"(x)); }

// Rows of one wavefront's columns, from its states x (and, for staged rows,
// xh: the kLine states right of its columns, one per lane).
// `ahead` is called once, kAheadRows rows before the end (or at the start).
template <typename T, int P, bool NT, bool STAR, bool SHIFT, bool WHOLE, typename Ahead>
__device__ __forceinline__ void paced_rows(uint64_t (&x)[P][Vec16<T>::E], uint64_t xh, T *row,
                                           uint32_t rows, uint64_t n, uint64_t wbase,
                                           uint32_t lane, T *stage, uint64_t t0, uint64_t &sched,
                                           uint64_t delta256, uint32_t burst, const Ahead &ahead)
{
    typedef Vec16<T> VT;
    typedef typename VT::type V16;
    constexpr int E = VT::E;
    constexpr uint32_t W = 64u * P * E, L = kLine<T>;
    // Columns from wbase to the end of the row (all that matter here).
    const uint32_t cols = (uint32_t)(n - wbase < W + L ? n - wbase : W + L);
    uint32_t left = 1;
    const uint32_t ahead_at = rows > kAheadRows ? rows - kAheadRows : 0;
#pragma nounroll
    for (uint32_t k = 0; k < rows; ++k) {
        if (sizeof(T) == 8 && k == ahead_at)
            ahead();
        if (delta256 && --left == 0) {
            wait_until(t0 + (sched >> 8));
            sched += delta256;
            left = burst;
        }
        if (SHIFT) {
            // The wavefront writes the lines that start in its columns.
            const uint32_t d =
                (0u - (uint32_t)(reinterpret_cast<uintptr_t>(row) / sizeof(T))) & (L - 1);
#pragma unroll
            for (int p = 0; p < P; ++p)
                *reinterpret_cast<V16 *>(stage + p * 64 * E + lane * E) =
                    VT::template pack<STAR>(x[p]);
            if (lane < L)
                stage[W + lane] = emit<T, STAR>(xh);
            wave_lds_fence();
            V16 v[P];
#pragma unroll
            for (int p = 0; p < P; ++p)
                v[p] = lds_chunk(stage + d + p * 64 * E + lane * E);
            // The words of the row's first and last, partial lines and
            // chunks: its first d, and those past its last whole chunk.
            const uint32_t lim = WHOLE || d >= cols ? 0 : cols - d;
            const T head = stage[lane];
            T tail = 0;
            if (!WHOLE)
                tail = stage[stage_tail(d, lim, lane, E, W + L)];
            wave_lds_fence();
            // The next states are formed while the LDS answers.
            __builtin_amdgcn_sched_barrier(0);
            xh = xs_step(xh);
            pin(xh);
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    x[p][e] = xs_step(x[p][e]);
                    pin(x[p][e]);
                }
            T *const dst = row + wbase + d;
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (WHOLE || p * 64 + lane < lim / E)
                    store16<NT>(reinterpret_cast<V16 *>(dst + p * 64 * E + lane * E), v[p]);
            if (wbase == 0 && lane < d && lane < n)
                row[lane] = head;
            if (!WHOLE && lane < lim % E && lim < W)
                dst[(lim & ~(E - 1u)) + lane] = tail;
        } else {
            // Every row is a whole number of 16-byte chunks: of lines, or of an
            // output that caches hold, or in place.
            T *const dst = row + wbase;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (WHOLE || (p * 64 + lane) * E < cols)
                    store16<NT>(reinterpret_cast<V16 *>(dst + p * 64 * E + lane * E),
                                VT::template pack<STAR>(x[p]));
#pragma unroll
                for (int e = 0; e < E; ++e)
                    x[p][e] = xs_step(x[p][e]);
            }
        }
        row += n;
    }
}

// The states of a wavefront's columns, 16 bytes at a time where all of them
// exist (whole).
template <int P, int E>
__device__ __forceinline__ void load_states(uint64_t (&x)[P][E], const uint64_t *state, uint64_t n,
                                            uint64_t wbase, uint32_t lane, bool whole)
{
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
        if (whole) {
#pragma unroll
            for (int e = 0; e < E; e += 2) {
                const u64x2 v = *reinterpret_cast<const u64x2 *>(state + g + e);
                x[p][e] = v.x;
                x[p][e + 1] = v.y;
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                x[p][e] = g + e < n ? state[g + e] : 0;
        }
    }
}
template <int P, int E>
__device__ __forceinline__ void store_states(const uint64_t (&x)[P][E], uint64_t *state,
                                             uint64_t n, uint64_t wbase, uint32_t lane, bool whole)
{
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t g = wbase + (uint64_t)p * 64 * E + (uint64_t)lane * E;
        if (whole) {
#pragma unroll
            for (int e = 0; e < E; e += 2)
                *reinterpret_cast<u64x2 *>(state + g + e) = u64x2{x[p][e], x[p][e + 1]};
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (g + e < n)
                    state[g + e] = x[p][e];
        }
    }
}

// A launch without segments takes no polynomials.
struct NoPolys {
};
__device__ __forceinline__ uint64_t poly_of(const NoPolys &, uint32_t) { return 0; }
__device__ __forceinline__ uint64_t poly_of(const JumpPolys &p, uint32_t seg) { return p.c[seg]; }

template <typename T, int P, bool NT, bool STAR, bool SHIFT, typename Polys>
__global__ __launch_bounds__(1024) void
gen_paced_kernel(const PacedArgs a, const Polys polys)
{
    constexpr int E = Vec16<T>::E;
    constexpr uint32_t W = 64u * P * E; // work-items per wavefront
    constexpr uint32_t L = kLine<T>;
    constexpr bool SEG = sizeof(Polys) > sizeof(NoPolys);
    // Whether the next strip's states are loaded during this one's last rows:
    // 1-2.5 % at 10^7-2^26 states x 4-64 u64; nothing, and 2 % lost at 2^26 x
    // 2-8, for 4-byte words, whose states take twice the registers.
    constexpr bool AHEAD = sizeof(T) == 8 && !SEG;
    __shared__ uint64_t jump_cols[SEG ? 64 : 1], jump_tab[SEG ? 256 : 1];
    extern __shared__ __align__(16) unsigned char lds_dyn[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    T *stage = reinterpret_cast<T *>(lds_dyn) + (size_t)wid * (W + L);
    T *const out = static_cast<T *>(a.out);
    const uint64_t n = a.n;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    uint64_t sched = 0;
    uint32_t have = 0; // the segment jump_tab belongs to (0: none)
    // First column of the wavefront's part of a work item, and its states.
    const auto column = [&](uint32_t item) {
        const uint32_t cb = SEG ? item % a.col_blocks : item;
        return ((uint64_t)cb * (blockDim.x >> 6) + wid) * W;
    };
    uint64_t xn[P][E], xhn = 0; // of the next item
    const auto fetch = [&](uint32_t item) {
        const uint64_t at = column(item);
        load_states(xn, a.state_in, n, at, lane, at + W <= n);
        if (SHIFT)
            xhn = lane < L && at + W + lane < n ? a.state_in[at + W + lane] : 0;
    };
    if (AHEAD)
        fetch(blockIdx.x);
    for (uint32_t item = blockIdx.x; item < a.items; item += gridDim.x) {
        const uint32_t seg = SEG ? item / a.col_blocks : 0;
        const uint64_t wbase = column(item);
        if (!SEG && wbase >= n)
            return; // later strips lie further right
        if (!AHEAD)
            fetch(item);
        uint64_t x[P][E], xh = xhn;
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int e = 0; e < E; ++e)
                x[p][e] = xn[p][e];
        if (SEG && seg) { // uniform over the block
            if (seg != have)
                build_jump(poly_of(polys, seg), jump_cols, jump_tab);
            have = seg;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int e = 0; e < E; ++e)
                    x[p][e] = nibble_product(jump_tab, x[p][e]);
            if (SHIFT)
                xh = nibble_product(jump_tab, xh);
        }
        const bool more = a.items - item > gridDim.x;
        const auto ahead = [&] {
            if (AHEAD && more)
                fetch(item + gridDim.x);
        };
        if (SEG && wbase >= n)
            continue; // no columns here (the wavefront still helped with the table)
        const uint32_t k0 = seg * a.seg_rows;
        const uint32_t rows = a.iters - k0 < a.seg_rows ? a.iters - k0 : a.seg_rows;
        T *row = out + (uint64_t)k0 * n;
        if (wbase + W + (SHIFT ? L : 0) <= n)
            paced_rows<T, P, NT, STAR, SHIFT, true>(x, xh, row, rows, n, wbase, lane, stage, t0,
                                                    sched, a.delta256, a.burst, ahead);
        else
            paced_rows<T, P, NT, STAR, SHIFT, false>(x, xh, row, rows, n, wbase, lane, stage, t0,
                                                     sched, a.delta256, a.burst, ahead);
        if (k0 + rows == a.iters)
            store_states(x, a.state_out, n, wbase, lane, wbase + W <= n);
    }
}

template <typename T, int P, bool NT, bool AL, bool STAR>
hipError_t launch_gen_t(uint32_t block, uint64_t *state, uint32_t n, uint32_t iters, T *out,
                        hipStream_t s)
{
    constexpr uint64_t WAVE_ITEMS = 64ull * P * Vec16<T>::E;
    const uint64_t waves = (n + WAVE_ITEMS - 1) / WAVE_ITEMS;
    const uint64_t blocks = (waves * 64 + block - 1) / block;
    return launch_on(s, gen_kernel<T, P, NT, AL, STAR>, (uint32_t)blocks, block, 0, state, n,
                     iters, out);
}

// The scheduled launch: grid = every block that fits on the device at once
// (at most the blocks the work needs); the schedule's step is the time
// the grid's share of a row (blocks x block x 16 x P bytes) takes at
// pace_gbs, in ticks of the device's constant-rate clock, times 256.
template <typename T, int P, bool NT, bool STAR, bool SHIFT, typename Polys>
hipError_t launch_paced_t(const GenPlan &plan, const Polys &polys, uint64_t *state,
                          uint64_t *state_out, uint32_t n, uint32_t iters, void *out,
                          hipStream_t s)
{
    const uint32_t block = plan.cfg.block, pace_gbs = plan.cfg.pace_gbs;
    constexpr uint32_t W = 64u * P * Vec16<T>::E;
    const uint32_t wpb = block / 64;
    const size_t lds = SHIFT ? (size_t)wpb * (W + kLine<T>) * sizeof(T) : 0;
    // Device attributes and this kernel's occupancy at `block`, cached per
    // device (devices beyond the table query every launch).
    constexpr int kDevs = 16;
    static std::atomic<int> cached_occ[kDevs][16] = {};
    static std::atomic<int> cached_cus[kDevs] = {}, cached_khz[kDevs] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    const bool cacheable = dev >= 0 && dev < kDevs;
    const int bi = (int)wpb - 1; // block 64..1024
    int cus = cacheable ? cached_cus[dev].load(std::memory_order_relaxed) : 0;
    int clock_khz = cacheable ? cached_khz[dev].load(std::memory_order_relaxed) : 0;
    int occ = cacheable ? cached_occ[dev][bi].load(std::memory_order_relaxed) : 0;
    if (cus <= 0 || clock_khz <= 0 || occ <= 0) {
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &occ, gen_paced_kernel<T, P, NT, STAR, SHIFT, Polys>, (int)block, lds);
        if (e != hipSuccess)
            return e;
        cus = cus > 0 ? cus : 1;
        clock_khz = clock_khz > 0 ? clock_khz : 100000;
        occ = occ > 0 ? occ : 1;
        if (cacheable) {
            cached_cus[dev].store(cus, std::memory_order_relaxed);
            cached_khz[dev].store(clock_khz, std::memory_order_relaxed);
            cached_occ[dev][bi].store(occ, std::memory_order_relaxed);
        }
    }
    const uint64_t waves = ((uint64_t)n + W - 1) / W;
    const uint64_t col_blocks = (waves + wpb - 1) / wpb;
    const uint64_t items = col_blocks * plan.segs;
    uint64_t grid = (uint64_t)occ * (uint64_t)cus;
    // Strips of equal size.
    const uint64_t strips = (items + grid - 1) / grid;
    grid = (items + strips - 1) / strips;
    // The schedule counts a row's own bytes. A later strip's states are read
    // and an earlier one's written while rows are, 16 bytes per work-item
    // more: where that is traffic to the memory (states beyond the Infinity
    // Cache) the row's time grows by its share, and for 4-byte words, whose
    // share is twice as large, by what exceeds 4.5 %. (2^26 states x 32 u64
    // 5.7 -> 6.3 TB/s, x 64 u32 5.8 -> 6.1; 10^7 x 32 u32 6.1 -> 6.8. Of no
    // use elsewhere: 2^24 x 32 u64 7.3 without, 7.1 with the excess over 3 %.)
    const double share = 16.0 / ((double)sizeof(T) * iters);
    const double states = strips == 1 ? 1.0
                          : (uint64_t)n * 8 > kCacheBytes ? 1.0 + share
                          : sizeof(T) == 4 ? std::max(1.0, (1.0 + share) / 1.045) : 1.0;
    const double row_bytes = (double)grid * block * 16.0 * P * states;
    const double ticks = pace_gbs ? row_bytes / (pace_gbs * 1e9) * clock_khz * 1e3 : 0.0;
    PacedArgs a;
    a.state_in = state;
    a.state_out = state_out;
    a.out = out;
    a.n = n;
    a.iters = iters;
    a.seg_rows = plan.seg_rows;
    a.col_blocks = (uint32_t)col_blocks;
    a.items = (uint32_t)items;
    // Rows between clock readings: about a microsecond of the schedule (a
    // reading costs a wavefront about 0.1 us).
    const double rows_per_us = ticks > 0 ? clock_khz * 1e-3 / ticks : 0.0;
    a.burst = rows_per_us > 8.0 ? 8u : rows_per_us > 1.0 ? (uint32_t)rows_per_us : 1u;
    a.delta256 = (uint64_t)(ticks * 256.0 * a.burst);
    return launch_on(s, gen_paced_kernel<T, P, NT, STAR, SHIFT, Polys>, (uint32_t)grid, block, lds,
                     a, polys);
}

template <typename T, int P, bool STAR, bool SHIFT, typename Polys>
hipError_t launch_paced_nt(const GenPlan &plan, const Polys &polys, uint64_t *state, uint64_t *so,
                           uint32_t n, uint32_t iters, T *out, hipStream_t s)
{
    return plan.cfg.nontemporal
               ? launch_paced_t<T, P, true, STAR, SHIFT>(plan, polys, state, so, n, iters, out, s)
               : launch_paced_t<T, P, false, STAR, SHIFT>(plan, polys, state, so, n, iters, out,
                                                          s);
}

template <typename T, int P, bool STAR>
hipError_t launch_gen_p(const GenPlan &plan, const JumpPolys &polys, uint64_t *state,
                        uint64_t *alt, uint32_t n, uint32_t iters, T *out, hipStream_t s)
{
    if (plan.scheduled) {
        uint64_t *const so = plan.out_of_place() ? alt : state;
        if (plan.segs > 1) // one chunk per lane (plan_gen)
            return plan.shift
                       ? launch_paced_nt<T, 1, STAR, true>(plan, polys, state, so, n, iters, out, s)
                       : launch_paced_nt<T, 1, STAR, false>(plan, polys, state, so, n, iters, out,
                                                            s);
        // Staged rows: at most two chunks (four would stage more than 64 KiB
        // a block).
        constexpr int Q = P < 2 ? P : 2;
        const NoPolys none;
        return plan.shift
                   ? launch_paced_nt<T, Q, STAR, true>(plan, none, state, so, n, iters, out, s)
                   : launch_paced_nt<T, P, STAR, false>(plan, none, state, so, n, iters, out, s);
    }
    const bool nt = plan.cfg.nontemporal != 0;
    const uint32_t block = plan.cfg.block;
    if (nt)
        return plan.aligned16 ? launch_gen_t<T, P, true, true, STAR>(block, state, n, iters, out, s)
                              : launch_gen_t<T, P, true, false, STAR>(block, state, n, iters, out,
                                                                      s);
    return plan.aligned16 ? launch_gen_t<T, P, false, true, STAR>(block, state, n, iters, out, s)
                          : launch_gen_t<T, P, false, false, STAR>(block, state, n, iters, out, s);
}

template <typename T, bool STAR>
hipError_t launch_gen_typed(const GenPlan &plan, const JumpPolys &polys, uint64_t *state,
                            uint64_t *alt, uint32_t n, uint32_t iters, T *out, hipStream_t s)
{
    switch (plan.cfg.chunks) {
    case 1: return launch_gen_p<T, 1, STAR>(plan, polys, state, alt, n, iters, out, s);
    case 2: return launch_gen_p<T, 2, STAR>(plan, polys, state, alt, n, iters, out, s);
    default: return launch_gen_p<T, 4, STAR>(plan, polys, state, alt, n, iters, out, s);
    }
}

} // namespace

hipError_t launch_init(uint64_t *state, uint32_t n, const SeedMix &mix, hipStream_t s)
{
    const uint32_t block = 256;
    uint64_t blocks = ((uint64_t)n + block - 1) / block;
    if (blocks > 65536)
        blocks = 65536;
    return launch_on(s, init_kernel, (uint32_t)blocks, block, 0, state, n, mix);
}

hipError_t launch_gen(const GenPlan &plan, const JumpPolys &polys, bool u32, bool star,
                      uint64_t *state, uint64_t *alt, uint32_t n, uint32_t iters, void *out,
                      hipStream_t s)
{
    uint32_t *o32 = static_cast<uint32_t *>(out);
    uint64_t *o64 = static_cast<uint64_t *>(out);
    if (u32)
        return star ? launch_gen_typed<uint32_t, true>(plan, polys, state, alt, n, iters, o32, s)
                    : launch_gen_typed<uint32_t, false>(plan, polys, state, alt, n, iters, o32, s);
    return star ? launch_gen_typed<uint64_t, true>(plan, polys, state, alt, n, iters, o64, s)
                : launch_gen_typed<uint64_t, false>(plan, polys, state, alt, n, iters, o64, s);
}

} // namespace rngx
