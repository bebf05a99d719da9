// Base projection and adapter update in one matrix-core kernel for gfx950 (bf16 in, fp32 accumulate):
//     y[t] = x[t] . W  +  s_i . v[t] . B_i          v[t] = x[t] . A_i from the shrink kernels
// for the tokens of a batch in one list of rows, those of an adapter next to each other (LinearRows).  The adapter product enters
// as one more slab of the contraction after the k loop over h_in, segment by segment of a block's rows, so the output is written once
// and never read: the separate addition of the adapter result to the base output (paper section 3.1)
// disappears.  This is the variant of the hot path whose roof is the matrix cores, not HBM.
//
// Block = 8 wavefronts on 32 MB rows (192, 256 or 288; figures below: 256) x 256 output columns; wavefront w owns the row half w/4 and the
// column quarter w%4: MB x 4 products of 16 x 16 (v_mfma_f32_16x16x32_bf16, 16 MB accumulator registers).  x rows
// (gathered by token) and Wt rows (Wt[n][k] = W[k][n], the layout a linear layer keeps its weight in) are both
// contiguous along k: a stage is 64 k of both, 64 KB, brought into LDS by global_load_lds_dwordx4 -- the load writes
// LDS itself (at the wavefront's base + 16 bytes x lane; checked on the part), so no registers stage the data.
//
// What bounds the loop is that matrix cores, LDS and the load path each need most of a stage's time (products 0.85 us at
// the peak rate, 192 KB of operand reads, 64 KB of loads): done one after the other by wavefronts in step, with a wait
// for all loads at the stage's end, a stage took 2 us.  So the two wavefronts of a SIMD (w and w + 4) take turns: a
// stage is two phases (the first and the second half of the wavefront's row blocks), a phase a *load section* -- the phase's operand
// reads and the requests for later stages -- and a *product section* of 32 products, with a barrier behind each, and
// wavefronts 4..7 run one section behind wavefronts 0..3.  The requests are counted, not drained: an LDS half (128 rows
// of x or Wt) is requested three phases before it is read, as soon as the phase after its last read has begun, and a
// load section waits only until the eight latest requests are all that is outstanding.  Both sides of the hand-over
// are ordered by the barriers: a section ends with its own reads done (lgkmcnt(0)) and its own part of the half that
// the next phase reads landed (vmcnt(8)), and the other group of wavefronts has passed the same point one barrier
// later, before anybody reads (or overwrites) that half.
// Measured on 4096 x 4096 x 4096 (one round of 256 blocks): 129.5 us with all wavefronts in step, 98.5 us this way;
// 8192 x 8192 x 8192: 934 -> 710 us (1.55 PFLOP/s; the vendor library's product 766 us).  With all units busy the stages take 1.38 us, with 64 of them
// 0.91 us, the products' own time: what the card sustains then bounds the loop, not its schedule.  It is power: the same launches on zeros
// take 485 us at 8192 x 8192 x 8192 (2.27 PFLOP/s; 689 on normal values, same card) and 66 at 4096 x 4096 x 4096 (91).  Four phases of 16 products
// take 107 us, operand reads spread evenly over the phases 98 us, requests from the product section 102 us.
//
// LDS rows are 128 bytes without padding; bank conflicts are avoided by a swizzle instead: 16-byte slot s of row r
// holds piece s ^ ((r/2) % 8) of the row's 64 k, so the 16 rows an operand read touches at once fall into 16
// different bank groups.
// Operand layout of the instruction: A (16 x 32): lane l holds row l%16, k = 8*(l/16) .. +7;
// B (32 x 16): lane l holds column l%16, same k; D: lane l holds column l%16, rows 4*(l/16) .. +3.
// The products are formed transposed -- the W block is the row operand, the x block the column
// operand -- so that a lane's four accumulator registers are four consecutive output columns of one
// token: 8 bytes of bf16, parked in LDS and stored from there in whole 128-byte lines.
// After the k loop the scaled intermediate s.v of the block's rows is staged in LDS as bf16 and every
// wavefront adds, per segment of its rows, the products with that segment's Bp, whose rank-packed layout gives the
// row operand directly from global memory (a lane's 8 ranks are 16 contiguous bytes); rows of other segments keep their sums.
// (Rows without gaps, where every tile had 64 rows of its own: a 13B layer's batch 12 -> 10 row panels, 1936 -> 1804 us for its seven
// projections; eight prompts at 4096 x 4096 19 -> 17 panels, 162 -> 154 us.)
// The adapter term of tokens on the GEMV path is computed by the GEMV kernels beforehand into the workspace or the
// (zeroed) output rows, and this kernel adds it to the accumulators of those rows (LinearList::add0 ..) before the one rounding
// of the stored value.
//
// Block order.  Tiles are counted in groups of four row panels, a group column by column, and every XCD takes a run of
// consecutive ones (block b runs on XCD b % 8): the 32 blocks of an XCD then share 4 row panels and 8 column panels
// through its L2 instead of all row panels (2816 x 13824 x 5120: 363 -> 340 us).
//
// One block fills a CU (its two stages take 128 KB of LDS), so a grid of N tiles runs in ceil(N / CUs) rounds and the
// last round may be nearly empty (288 tiles on 256 CUs: a second round of 32).  The tiles of that last round are
// therefore split along k into up to 8 parts, one block each (linear_split_shape).  The parts of a tile finish it
// together: each owns a share of every wavefront's rows, leaves its fp32 accumulators of the other shares in a scratch
// area (device-scope atomic stores, past the per-XCD L2s), counts itself in, waits until all parts have, adds the other
// parts' sums of its own share and runs the adapter slab and the store for it.  (With the last part to arrive finishing
// the tile alone 384 tiles of 64 stages take 176 us, 160 us this way.)  But a part may wait only for parts that are
// running: others may have no place on the device until this one leaves it, for instance beside a launch of another
// cache that waits the same way.  So the parts count themselves in when they start, and the first to have its sums
// decides: if all parts have started, they share the tile; if not, every part leaves all its sums and ends, and the last
// to arrive finishes the tile alone.  Either way a row block's sums are added in the same order.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lora_device.h"

namespace lora {

namespace {
constexpr int LBM = 256, LBN = 256, LBK = 64;
constexpr int LROW = LBK * 2;                   // bytes per row of a stage in LDS (swizzled, not padded)
constexpr int L_HALF = 128 * LROW;              // 128 rows of x or Wt, 64 k: 16 KB
constexpr int SV_ROW = LORA_MAX_RANK * 2 + 16;  // bytes per row of the staged s.v
// two stages of x half 0, x half 1, Wt half 0, Wt half 1; s.v and the parked outputs (16 MB x 64 of eight wavefronts) use the same memory
template <int MB> constexpr int linear_lds = std::max({2 * (32 * MB + LBN) * LROW, 32 * MB * SV_ROW, 8 * 16 * MB * 128});
static_assert(linear_lds<8> == 128 << 10 && linear_lds<9> <= 160 << 10, "one block to a compute unit");
constexpr int MAX_PARTS = 8;                    // a wavefront's 128 rows are eight blocks of 16
constexpr size_t PART_WORDS = LINEAR_SHARE_BYTES / sizeof(unsigned long long);
}  // namespace

typedef float floatx2 __attribute__((ext_vector_type(2)));

// split of the last round: blocks [0, n_whole) work on whole tiles; block n_whole + parts * j + p on part p of tile n_whole + j
constexpr uint32_t SPLIT_SHARED = 1, SPLIT_LAST = 2;
struct LinearSplit {
    int n_whole, parts;           // parts = 1: no split
    unsigned long long *partial;  // [tile j][part][row block of 16: 8][column block of 16: 4][half 2][thread 512] 8-byte words
    SplitState *state;            // [tile j], zero between launches
    int32_t *fault;
};

// Tile number -> (row panel, column panel): groups of H row panels, column by column
template <int H> __device__ __forceinline__ void linear_tile(int t, int n_mt, int n_nt, int &bm, int &bn)
{
    const int per = H * n_nt, grp = t / per, rem = t - grp * per, height = min(H, n_mt - H * grp);
    bn = rem / height;
    bm = H * grp + (rem - bn * height);
}

// A barrier alone: what must be complete at it has been waited for by count
__device__ __forceinline__ void section_end()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The s.v operand of the adapter product: of the 8 ranks of a lane the first n (what lies behind them was never written).  As masks of
// whole words: a stale NaN must not survive.
__device__ __forceinline__ uint4 rank_mask(int n)
{
    auto word = [&](int j) { return n >= 2 * j + 2 ? 0xffffffffu : (n == 2 * j + 1 ? 0x0000ffffu : 0u); };
    return make_uint4(word(0), word(1), word(2), word(3));
}
__device__ __forceinline__ bf16x8 sv_operand(const uint4 &v, const uint4 &live)
{
    return __builtin_bit_cast(bf16x8, make_uint4(v.x & live.x, v.y & live.y, v.z & live.z, v.w & live.w));
}
// Where a block of 16 rows has rows of several segments, those outside the segment whose products have just been added get back what they had: lane
// (m, g) holds sums of row m alone, and an infinity or NaN in the segment's weights would come through a row of zeros as NaN.
template <int NB> __device__ __forceinline__ void keep_rows_outside(floatx4 (&acc)[NB], const floatx4 (&had)[NB], bool row_in)
{
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[nb][e] = row_in ? acc[nb][e] : had[nb][e];
}

template <int MB>
__global__ __launch_bounds__(512) void linear_tiles_kernel(ApplyArgs a, const __bf16 *__restrict__ Wt,
                                                           LinearList list, int n_mt, int n_nt, LinearSplit sp)
{
    constexpr int BM = 32 * MB, MB0 = (MB + 1) / 2, MB1 = MB / 2;  // rows of the block; row blocks of a wavefront per phase
    constexpr int X0 = 32 * MB0 * LROW, X1 = 32 * MB1 * LROW, BUF = X0 + X1 + 2 * L_HALF;  // bytes of x half 0 and 1, of a stage
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int rh = w >> 2, cq = w & 3;
    int tile_no, part = 0, tail = -1;
    if (MB == 8 && (int)blockIdx.x >= sp.n_whole) {
        tail = __builtin_amdgcn_readfirstlane(((int)blockIdx.x - sp.n_whole) / sp.parts);
        part = ((int)blockIdx.x - sp.n_whole) - tail * sp.parts;
        tile_no = sp.n_whole + tail;
        if (tid == 0) __hip_atomic_fetch_add(&sp.state[tail].started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {  // XCD j takes a run of consecutive tiles
        const int j = (int)blockIdx.x & 7, q = sp.n_whole >> 3, r = sp.n_whole & 7;
        tile_no = j * q + min(j, r) + ((int)blockIdx.x >> 3);
    }
    int bm, bn;
    linear_tile<4>(tile_no, n_mt, n_nt, bm, bn);
    const int n0 = bn * LBN;
    const int row0 = BM * bm, wrow = row0 + 16 * MB * rh;  // the block's first row and the wavefront's
    // the token ids of the block's rows (rows past the end count as the last; they are never stored): from memory while the block starts, later from LDS
    __shared__ int32_t tok_of_row[BM];
    auto token_of = [&](int row) { return list.tok[min(row, list.n_rows - 1)]; };
    if (tid < BM) tok_of_row[tid] = token_of(row0 + tid);

    const __bf16 *x = static_cast<const __bf16 *>(a.x);
    __bf16 *y = static_cast<__bf16 *>(a.y);
    const int n_k = a.h_in / LBK;
    // this block's stages of the k walk
    const int k_lo = tail < 0 ? 0 : n_k * part / sp.parts, k_hi = tail < 0 ? n_k : n_k * (part + 1) / sp.parts;

    // Half h of x holds the rows of phase h, 16 MBh of either row half, half h of Wt columns 64 c + 32 h .. +31 of the four column
    // quarters c.  Loader: a request brings 8 LDS rows x 128 bytes to the wavefront-uniform LDS address of the first, lane l to slot l%8 of row l/8, for
    // which it fetches piece (l%8) ^ ((row/2) % 8) of the row.  Request q of wavefront w brings rows 8 (w + 8 q) .. of a half; where that leaves four
    // wavefronts one request more, they are wavefronts 0..3, and 4..7 for x half 1 if x half 0 gives the others one more already
    constexpr int Q0 = (MB0 + 1) / 2, Q1 = (MB1 + 1) / 2;  // the most requests of a wavefront per x half
    constexpr bool ODD0 = MB0 % 2 != 0, ODD1 = MB1 % 2 != 0;
    const int w1 = ODD0 ? w ^ 4 : w;                       // the wavefront's place among the requests of x half 1
    const bool more0 = !ODD0 || w < 4, more1 = !ODD1 || w1 < 4;  // makes its last request of the half too
    const int lr = lane >> 3, piece = (lane & 7) ^ ((4 * (w & 1) + (lr >> 1)) & 7);
    const __bf16 *xg0[Q0], *xg1[Q1], *wg[2][2];
    {
        int tok0[Q0], tok1[Q1];
#pragma unroll
        for (int q = 0; q < Q0; ++q) {
            const int r = 8 * (w + 8 * q) + lr, half = r >= 16 * MB0;
            tok0[q] = token_of(row0 + 16 * MB * half + r - 16 * MB0 * half);
        }
#pragma unroll
        for (int q = 0; q < Q1; ++q) {
            const int r = 8 * (w1 + 8 * q) + lr, half = r >= 16 * MB1;
            tok1[q] = token_of(row0 + 16 * MB * half + 16 * MB0 + r - 16 * MB1 * half);
        }
#pragma unroll
        for (int q = 0; q < Q0; ++q) xg0[q] = x + (size_t)tok0[q] * a.h_in + piece * 8;
#pragma unroll
        for (int q = 0; q < Q1; ++q) xg1[q] = x + (size_t)tok1[q] * a.h_in + piece * 8;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // h_out is a multiple of 64, so a run of 64 columns is inside or outside as a whole
            const int w_row = min(n0 + 64 * ((w >> 2) + 2 * q), a.h_out - 64) + 32 * h + 8 * (w & 3) + lr;
            wg[h][q] = Wt + (size_t)w_row * a.h_in + piece * 8;
        }
    auto stage_at = [&](int buf) { return lds + buf * BUF; };  // x half 0, x half 1, Wt half 0, Wt half 1
    auto k_of = [&](int kt) { return min(kt, k_hi - 1) * LBK; };  // past the end: the last stage again (nobody reads it)
    auto load_x0 = [&](int kt, int buf) {
        const int k = k_of(kt);
        unsigned char *dst = stage_at(buf) + 8 * w * LROW;
#pragma unroll
        for (int q = 0; q < Q0; ++q)
            if (q < Q0 - 1 || more0) request16(xg0[q] + k, dst + 64 * q * LROW);
    };
    auto load_x1 = [&](int kt, int buf) {
        const int k = k_of(kt);
        unsigned char *dst = stage_at(buf) + X0 + 8 * w1 * LROW;
#pragma unroll
        for (int q = 0; q < Q1; ++q)
            if (q < Q1 - 1 || more1) request16(xg1[q] + k, dst + 64 * q * LROW);
    };
    auto load_w = [&](int kt, int buf) {
        const int k = k_of(kt);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 2; ++q) request16(wg[h][q] + k, stage_at(buf) + X0 + X1 + h * L_HALF + (8 * w + 64 * q) * LROW);
    };
    // Waits until at most the latest stage's worth of requests is outstanding (x half 0 or 1, then the other, and Wt), and for the section's own reads
    constexpr int PER_LOW = MB0 / 2 + MB1 / 2 + 4 + (ODD0 && ODD1);  // of the wavefronts with fewer
    auto wait_section = [&]() {
        if (ODD0 != ODD1 && w < 4) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(PER_LOW + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(PER_LOW) : "memory");
    };

    floatx4 acc[MB][4];  // [block of 16 rows][block of 16 columns]
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mb][nb][e] = 0.f;

    // operand reads: LDS row R, k piece 4ks + g sits in slot (4ks + g) ^ ((R/2) % 8); R/2 % 8 = m/2 for all of a lane's rows
    const int swz = (m >> 1) & 7;
    bf16x8 xo[MB0][2], wo[4][2];  // [block of 16 rows / columns][k step]
    auto read_x = [&](int buf, auto h_tag) {
        constexpr int H = decltype(h_tag)::value, N = H ? MB1 : MB0;
        const unsigned char *s = stage_at(buf) + H * X0 + (16 * N * rh + m) * LROW;
#pragma unroll
        for (int mb = 0; mb < N; ++mb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) xo[mb][ks] = *reinterpret_cast<const bf16x8 *>(s + mb * 16 * LROW + (((4 * ks + g) ^ swz) << 4));
    };
    auto read_w = [&](int buf) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const unsigned char *s = stage_at(buf) + X0 + X1 + (nb >> 1) * L_HALF + (32 * cq + 16 * (nb & 1) + m) * LROW;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) wo[nb][ks] = *reinterpret_cast<const bf16x8 *>(s + (((4 * ks + g) ^ swz) << 4));
        }
    };
    auto products = [&](auto h_tag) {
        constexpr int H = decltype(h_tag)::value, N = H ? MB1 : MB0;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int mb = 0; mb < N; ++mb)
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
                    acc[MB0 * H + mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wo[nb][ks], xo[mb][ks], acc[MB0 * H + mb][nb], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
    };

    // requests in the order of their use: per stage x half 0, Wt half 0, Wt half 1 | x half 1
    load_x0(k_lo, 0);
    load_w(k_lo, 0);
    load_x1(k_lo, 0);
    load_x0(k_lo + 1, 1);
    load_w(k_lo + 1, 1);
    wait_section();
    section_end();
    if (rh == 1) section_end();  // the second group of wavefronts runs one section behind
    for (int kt = k_lo; kt < k_hi; ++kt) {
        const int buf = (kt - k_lo) & 1;
        read_x(buf, std::integral_constant<int, 0>{});
        read_w(buf);
        load_x1(kt + 1, buf ^ 1);  // that half was last read in the phase before
        wait_section();  // x half 1 of this stage is in (a stage's worth of requests came after it)
        section_end();
        products(std::integral_constant<int, 0>{});
        section_end();
        read_x(buf, std::integral_constant<int, 1>{});
        load_x0(kt + 2, buf);
        load_w(kt + 2, buf);
        wait_section();  // x half 0 and Wt of the next stage are in
        section_end();
        products(std::integral_constant<int, 1>{});
        section_end();
    }
    if (rh == 0) section_end();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the requests past the end: LDS is used for other things below
    __syncthreads();

    // ---- a tile split along k.  Row block mb of every wavefront (8 to a part's wavefront) belongs to part
    // ((mb + 1) * parts - 1) / 8; its sum is that part's plus the others' in their order, whoever adds it up
    int own_lo = 0, own_hi = MB;  // the row blocks this block finishes
    if constexpr (MB == 8) if (tail >= 0) {
        SplitState *const st = sp.state + tail;
        unsigned long long *const sums = sp.partial + (size_t)tail * sp.parts * PART_WORDS;
        __shared__ uint32_t said;
        if (tid == 0) {
            const uint32_t all_run = __hip_atomic_load(&st->started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)sp.parts;
            uint32_t way = 0;
            const uint32_t mine = all_run ? SPLIT_SHARED : SPLIT_LAST;
            if (__hip_atomic_compare_exchange_strong(&st->way, &way, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) way = mine;
            said = way;
        }
        __syncthreads();
        const bool shared = said == SPLIT_SHARED;
        if (shared) own_lo = 8 * part / sp.parts, own_hi = 8 * (part + 1) / sp.parts;
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
            if (shared && mb >= own_lo && mb < own_hi) continue;  // uniform
            unsigned long long *const dst = sums + part * PART_WORDS + mb * 8 * 512;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const floatx4 c = acc[mb][nb];
                const floatx2 lo = {c[0], c[1]}, hi = {c[2], c[3]};
                __hip_atomic_store(dst + (nb * 2 + 0) * 512 + (uint32_t)tid, __builtin_bit_cast(unsigned long long, lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(dst + (nb * 2 + 1) * 512 + (uint32_t)tid, __builtin_bit_cast(unsigned long long, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores above have been performed where every XCD sees them
        __syncthreads();
        if (tid == 0) {
            uint32_t n = 1 + __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (shared) {  // (all parts are running, and a part waits for nothing before it has counted itself in)
                for (int spin = 0; spin < (1 << 20) && n < (uint32_t)sp.parts; ++spin) {
                    __builtin_amdgcn_s_sleep(8);
                    n = __hip_atomic_load(&st->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (n < (uint32_t)sp.parts) __hip_atomic_store(sp.fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // pinned host memory
            }
            said = n;
        }
        __syncthreads();
        const bool all_in = said == (uint32_t)sp.parts;
        if (!shared && !all_in) return;  // (the whole block: a part that comes later finishes the tile)
        if (all_in) {
#pragma unroll
            for (int mb = 0; mb < 8; ++mb) {
                if (mb < own_lo || mb >= own_hi) continue;  // uniform
                const int owner = ((mb + 1) * sp.parts - 1) >> 3;
                floatx4 sum[4];
                for (int i = 0; i < sp.parts; ++i) {
                    const int q = i == 0 ? owner : i - 1 + (i - 1 >= owner);
                    floatx4 v[4];
                    if (q == part) {  // uniform
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb) v[nb] = acc[mb][nb];
                    } else {
                        const unsigned long long *const src = sums + q * PART_WORDS + mb * 8 * 512;
                        unsigned long long w8[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) w8[j] = __hip_atomic_load(src + j * 512 + (uint32_t)tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const floatx2 f = __builtin_bit_cast(floatx2, w8[j]);
                            v[j >> 1][2 * (j & 1)] = f[0];
                            v[j >> 1][2 * (j & 1) + 1] = f[1];
                        }
                    }
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[nb][e] = i == 0 ? v[nb][e] : sum[nb][e] + v[nb][e];
                }
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = sum[nb];
            }
        }
        // the last to have read (or the only one) sets the state back for the next launch
        __syncthreads();
        if (tid == 0 && (!shared || __hip_atomic_fetch_add(&st->read, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)sp.parts - 1)) {
            __hip_atomic_store(&st->started, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->way, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->read, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // row blocks (of the wavefront's eight) that this block finishes
    auto owns = [&](int mb) { return mb >= own_lo && mb < own_hi; };

    // ---- the adapter slab, segment by segment of the wavefront's rows.  Bp operands: granule 4ks + g (the 8 ranks a lane's
    // operand holds, contiguous per column; past the stored rank the last granule, which meets zeros of s.v), all four k
    // steps requested at once -- and for the first segment before s.v is staged, so that the requests fly while the staging
    // waits for its own loads.
    bf16x8 bo[4][4];
    auto load_bp = [&](const LinearSeg &t) {
        const __bf16 *Bp = reinterpret_cast<const __bf16 *>(a.proj_base + (int64_t)t.row * a.row_bytes) + (size_t)rank_storage(t.rank) * a.h_in;
        const int rs8 = rank_storage(t.rank) >> 3;
        int own_lane = lane;
        if constexpr (MB > 8) asm volatile("" : "+v"(own_lane));  // (places made anew for every segment: the registers hold none beside the products)
        const int lm = own_lane & 15, lg = own_lane >> 4;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int col = min(n0 + 64 * cq + 16 * nb + lm, a.h_out - 1);
                bo[ks][nb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Bp + ((size_t)min(4 * ks + lg, rs8 - 1) * a.h_out + col) * 8));
            }
    };
    // (rows with an adapter product come first in the list)
    const int wend = min(wrow + 16 * MB, list.n_rows);
    int seg0 = 0, seg1 = 0;  // wavefront-uniform: the segments of the runs its rows lie in, less those that end before or begin behind them
    if (wrow < min(list.add0, wend)) {
        const LinearRows r0 = list.rows[wrow / LORA_TILE_TOKENS], r1 = list.rows[(wend - 1) / LORA_TILE_TOKENS];
        seg0 = r0.first_seg, seg1 = r1.first_seg + r1.n_segs;
        while (seg0 < seg1 && list.segs[seg0].r1 <= wrow) ++seg0;
        while (seg0 < seg1 && list.segs[seg1 - 1].r0 >= wend) --seg1;
    }
    LinearSeg seg = {};
    if (seg0 < seg1) {
        seg = list.segs[seg0];
        load_bp(seg);
    }
    unsigned char *sv = lds;  // s.v of the block's rows as bf16
    if (row0 < list.add0) {
        // chunk tid % 16 (8 ranks) of rows tid / 16 + 32 i: the token ids in one round, then the pieces, four or five rows at a time
        // (unconditional, from addresses inside v; what lies past a row's rank is masked where it is used)
        const int c8 = tid & 15, r0 = tid >> 4;
        int tok[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) tok[i] = tok_of_row[r0 + 32 * i];
#pragma unroll
        for (int i0 = 0; i0 < MB; i0 += MB0) {
            uint4 pc[MB0];
#pragma unroll
            for (int j = 0; j < MB0 && i0 + j < MB; ++j)  // s.v comes as bf16 from the shrink or the reduce (rows of the fp32 pitch)
                pc[j] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const __bf16 *>(a.v) + (size_t)tok[i0 + j] * (2 * a.v_stride) + c8 * 8);
#pragma unroll
            for (int j = 0; j < MB0 && i0 + j < MB; ++j) *reinterpret_cast<uint4 *>(sv + (r0 + 32 * (i0 + j)) * SV_ROW + c8 * 16) = pc[j];
        }
    }
    __syncthreads();
    for (int s = seg0; s < seg1; ++s) {
        if (s > seg0) {
            seg = list.segs[s];
            load_bp(seg);
        }
        const int ks32 = (seg.rank + 31) >> 5;
        const int lo = seg.r0 - wrow, hi = seg.r1 - wrow;  // its rows among the wavefront's
        const unsigned char *svr = sv + (16 * MB * rh + m) * SV_ROW + g * 16;
        int ranks_left = seg.rank - 8 * g;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if constexpr (MB > 8) asm("" : "+v"(ranks_left));  // (the masks made anew for every row block: the registers hold no four of them)
            const int r0 = 16 * mb, r = r0 + m;
            if (!owns(mb) || r0 + 16 <= lo || r0 >= hi) continue;  // uniform
            const bool whole = lo <= r0 && r0 + 16 <= hi;  // uniform
            floatx4 had[4];
            if (!whole) {
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) had[nb] = acc[mb][nb];
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks >= ks32) continue;
                const bf16x8 so = sv_operand(*reinterpret_cast<const uint4 *>(svr + mb * 16 * SV_ROW + ks * 64), rank_mask(ranks_left - 32 * ks));
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bo[ks][nb], so, acc[mb][nb], 0, 0, 0);
            }
            if (!whole) keep_rows_outside<4>(acc[mb], had, lo <= r && r < hi);
        }
    }

    // ---- store.  The products are formed transposed (the W block is the instruction's row operand, the x
    // block its column operand): lane (m, g) holds, in the four registers of block (mb, nb), row 16*mb + m of the
    // wavefront's 16 MB and the four consecutive columns 16*nb + 4g .. of its 64 -- 8 bytes of bf16.  The
    // wavefront parks its 16 MB x 64 outputs in LDS and stores whole 128-byte row pieces, 8 rows per
    // instruction (stored from the registers, an instruction would write 32 bytes to each of 16 rows).
    // Park layout, free of bank conflicts both ways: row r is 128 bytes, its 8-byte cell c sits at
    // c ^ (2 * ((r/2) % 8)), i.e. its 16-byte slot s at s ^ ((r/2) % 8).  Rows of GEMV tokens take their adapter term, computed
    // beforehand, into the accumulators here, so that the sum is formed in fp32 before the one rounding.
    __syncthreads();  // every wavefront is done with the staged s.v
    unsigned char *park = lds + w * (16 * MB * 128);
    const bool live = wrow < list.n_rows && n0 + 64 * cq < a.h_out;  // wavefront-uniform (h_out is a multiple of 64)
    if (!live) return;  // (no barrier follows)
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    int own_tid = tid;
    if constexpr (MB > 8) asm volatile("" : "+v"(own_tid));  // (row numbers of its own: none is kept from before the products)
    const int ln = own_tid & 63, mr = ln & 15, gr = ln >> 4;
    if (wrow < list.add1 && wend > list.add0) {
        // as fp32 at the same place of the workspace, or in y: the token ids in one round, then per row block the four terms
        int tok[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) tok[mb] = tok_of_row[wrow - row0 + 16 * mb + mr];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if (!owns(mb)) continue;
            const int r = wrow + 16 * mb + mr;
            if (r < list.add0 || r >= list.add1) continue;
            const size_t at = (size_t)tok[mb] * a.h_out + n0 + 64 * cq + 4 * gr;
            floatx4 term[4];
            if (a.y32) {
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) term[nb] = *reinterpret_cast<const floatx4 *>(a.y32 + at + 16 * nb);
            } else {
                bf16x4 old[4];
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) old[nb] = *reinterpret_cast<const bf16x4 *>(y + at + 16 * nb);
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) term[nb][e] = (float)old[nb][e];
            }
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[mb][nb][e] += term[nb][e];
        }
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (!owns(mb)) continue;
        const int row = 16 * mb + mr;
        unsigned char *pr = park + row * 128;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const floatx4 c = acc[mb][nb];
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)c[e];
            *reinterpret_cast<bf16x4 *>(pr + (((4 * nb + gr) ^ (((row >> 1) & 7) << 1)) << 3)) = o;
        }
    }
    // the rows' token ids all before the first store (a lookup between two stores makes the second wait for the first)
    const int rl = ln >> 3, sl = ln & 7;
    int tok8[2 * MB];
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) tok8[i] = tok_of_row[wrow - row0 + 8 * i + rl];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // only this wavefront reads what it wrote; its LDS operations execute in order
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
        const int row = 8 * i + rl;
        if (owns(i >> 1) && wrow + row < list.n_rows) {
            const uint4 v = *reinterpret_cast<const uint4 *>(park + row * 128 + ((sl ^ ((row >> 1) & 7)) << 4));
            // (a streaming store: the rows leave the caches as they are written instead of lying there dirty
            // until the next kernel's loads push them out -- the tile shrink that follows runs 2 to 3 us shorter)
            typedef unsigned u32x4_nt __attribute__((ext_vector_type(4)));
            const u32x4_nt vn = {v.x, v.y, v.z, v.w};
            __builtin_nontemporal_store(vn, reinterpret_cast<u32x4_nt *>(y + (size_t)tok8[i] * a.h_out + n0 + 64 * cq + 8 * sl));
        }
    }
}

// ---------------------------------------------------------------------------------------
// The same for launches that tiles of 256 x 256 leave the chip idle with (417 x 2048 x 2048: 16 tiles, split along k into 128 blocks of
// 4 stages whose hand-over took most of 27 us): blocks of 4 wavefronts on 64 RM rows x 64 columns, wavefront w on the row half w / 2
// and the column half w % 2.  Stages of 64 k of both operands travel through a ring of NST, NST - 1 of them on their way (requests counted, as
// above), one barrier per stage; two or three blocks share a compute unit, and one multiplies while another waits.  What bounds it:
// with few blocks the trip to memory, 0.27 us a stage with three on their way; with many what the units take in, 15 to 19 TB/s
// of tiles that are re-read by every row and column of tiles.  Measured, 256 x 256 tiles -> this kernel: 64 x 4096 x 4096 30.9 -> 12.3 us, 417 x 2048 x 2048
// 27.5 -> 12.3, 992 x 1024 x 1024 26.2 -> 8.1, 2283 x 1088 x 1088 28.1 -> 14.4, 1234 x 2048 x 2048 30.3 -> 20.3 (128 rows), 785 x 2560 x 2560
// 32.4 -> 23.3 (128 rows); 1000 x 4096 x 4096 46.7 and 48.2.  Stages of 128 k (whole 256-byte rows) took the same time, tiles of 64 x 128 up to
// a fifth more than 128 x 64, 128 x 128 with four wavefronts half more.
// (The wavefronts per SIMD are those that LDS leaves room for; told of more, the compiler moves the sums between register files in every stage, 785 x 2560 x 2560 29.1 -> 30.3 us.)
// ---------------------------------------------------------------------------------------
template <int RM, int NST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, RM == 1 ? 3 : 2))) void linear_small_kernel(ApplyArgs a, const __bf16 *__restrict__ Wt, LinearList list, int n_mt, int n_nt, LinearSplit sp)
{
    constexpr int BM = 64 * RM, BN = 64, MB = 2 * RM, NB = 2;  // MB, NB: blocks of 16 rows and columns of a wavefront
    constexpr int STAGE = (BM + BN) * LROW, PER = 2 * (RM + 1);  // PER: requests of a wavefront per stage
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int wr = w >> 1, wc = w & 1;
    // XCD j (blocks j, j + 8, ...) takes a run of consecutive (tile, part) pairs
    const int n_pos = n_mt * n_nt * sp.parts, j8 = (int)blockIdx.x & 7, q8 = n_pos >> 3, r8 = n_pos & 7;
    const int pos = j8 * q8 + min(j8, r8) + ((int)blockIdx.x >> 3);
    const int tile_no = pos / sp.parts, part = pos - tile_no * sp.parts;
    int bm, bn;
    linear_tile<16 / RM>(tile_no, n_mt, n_nt, bm, bn);
    const int n0 = bn * BN, row0 = bm * BM;

    LinearRows run[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        run[i] = list.rows[min(RM * bm + i, list.n_rt - 1)];
        if (RM * bm + i >= list.n_rt) run[i].n_tok = run[i].n_segs = 0;
    }
    const int dead_tok = run[0].tok0;
    const __bf16 *x = static_cast<const __bf16 *>(a.x);
    __bf16 *y = static_cast<__bf16 *>(a.y);
    const int n_k = a.h_in / LBK, k_lo = n_k * part / sp.parts, n_st = n_k * (part + 1) / sp.parts - k_lo;

    // Loader: request q of wavefront w brings rows 8 (w + 4 q) + lane / 8 of x, then of Wt: 8 rows x 128 bytes, lane l to slot l % 8, for
    // which it fetches piece (l % 8) ^ ((row / 2) % 8)
    const int lr = lane >> 3, piece = (lane & 7) ^ ((4 * (w & 1) + (lr >> 1)) & 7);
    const __bf16 *src[PER];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int ti[2] = {8 * w + lr, 8 * w + 32 + lr};
        int tok[2];
        tile_tokens_of(list.tok, run[i], ti, dead_tok, tok);
#pragma unroll
        for (int q = 0; q < 2; ++q) src[2 * i + q] = x + (size_t)tok[q] * a.h_in + piece * 8 + (size_t)k_lo * LBK;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) src[2 * RM + q] = Wt + (size_t)(n0 + 32 * q + 8 * w + lr) * a.h_in + piece * 8 + (size_t)k_lo * LBK;  // (h_out is a multiple of 64)
    auto load_stage = [&](int st, int slot) {
        const int k = min(st, n_st - 1) * LBK;
        unsigned char *dst = lds + slot * STAGE + 8 * w * LROW;
#pragma unroll
        for (int q = 0; q < PER; ++q)
            request16(src[q] + k, dst + 32 * q * LROW);
    };

    floatx4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int swz = (m >> 1) & 7;
    auto multiply = [&](int slot) {
        const unsigned char *xs = lds + slot * STAGE + (32 * RM * wr + m) * LROW, *ws = lds + slot * STAGE + (BM + 32 * wc + m) * LROW;
        bf16x8 xo[MB][2], wo[NB][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int at = ((4 * ks + g) ^ swz) << 4;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) xo[mb][ks] = *reinterpret_cast<const bf16x8 *>(xs + mb * 16 * LROW + at);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) wo[nb][ks] = *reinterpret_cast<const bf16x8 *>(ws + nb * 16 * LROW + at);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wo[nb][ks], xo[mb][ks], acc[mb][nb], 0, 0, 0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read when this wavefront is at the next barrier
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) load_stage(s, s);
    int slot = 0, fill = NST - 1;
    for (int st = 0; st < n_st - (NST - 1); ++st) {
        wait_requests<PER *(NST - 2)>();
        section_end();
        load_stage(st + NST - 1, fill);  // the slot read before the barrier
        multiply(slot);
        fill = slot;
        slot = slot + 1 == NST ? 0 : slot + 1;
    }
    // the last stages, with nothing left to request
    auto last = [&](auto left_tag) {
        constexpr int LEFT = decltype(left_tag)::value;  // stages behind this one
        if (n_st <= LEFT) return;
        wait_requests<PER * LEFT>();
        section_end();
        multiply(slot);
        slot = slot + 1 == NST ? 0 : slot + 1;
    };
    if constexpr (NST > 3) last(std::integral_constant<int, 2>{});
    if constexpr (NST > 2) last(std::integral_constant<int, 1>{});
    last(std::integral_constant<int, 0>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // LDS is used for other things below

    // ---- a tile split along k: every part but the last to arrive leaves its sums and ends; nobody waits
    if (sp.parts > 1) {
        SplitState *const st = sp.state + tile_no;
        unsigned long long *const sums = sp.partial + (size_t)tile_no * sp.parts * (BM * BN / 2);
        __shared__ uint32_t said;
        if (tid == 0) said = __hip_atomic_load(&st->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        bool all_in = said == (uint32_t)sp.parts - 1;
        if (!all_in) {  // uniform
            unsigned long long *const dst = sums + (size_t)part * (BM * BN / 2) + tid;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const floatx4 c = acc[mb][nb];
                    const floatx2 lo = {c[0], c[1]}, hi = {c[2], c[3]};
                    __hip_atomic_store(dst + ((mb * NB + nb) * 2 + 0) * 256, __builtin_bit_cast(unsigned long long, lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(dst + ((mb * NB + nb) * 2 + 1) * 256, __builtin_bit_cast(unsigned long long, hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // performed where every XCD sees them
            __syncthreads();
            if (tid == 0) said = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            all_in = said == (uint32_t)sp.parts - 1;
            if (!all_in) return;  // the whole block
        }
        floatx4 sum[MB][NB];  // in the order of the parts, whoever adds them up
        for (int q = 0; q < sp.parts; ++q) {
            floatx4 v[MB][NB];
            if (q == part) {  // uniform
#pragma unroll
                for (int i = 0; i < MB * NB; ++i) v[i / NB][i % NB] = acc[i / NB][i % NB];
            } else {
                const unsigned long long *const from = sums + (size_t)q * (BM * BN / 2) + tid;
                unsigned long long w8[MB * NB * 2];
#pragma unroll
                for (int i = 0; i < MB * NB * 2; ++i) w8[i] = __hip_atomic_load(from + i * 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int i = 0; i < MB * NB * 2; ++i) {
                    const floatx2 f = __builtin_bit_cast(floatx2, w8[i]);
                    v[i / 2 / NB][i / 2 % NB][2 * (i & 1)] = f[0];
                    v[i / 2 / NB][i / 2 % NB][2 * (i & 1) + 1] = f[1];
                }
            }
#pragma unroll
            for (int i = 0; i < MB * NB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[i / NB][i % NB][e] = q == 0 ? v[i / NB][i % NB][e] : sum[i / NB][i % NB][e] + v[i / NB][i % NB][e];
        }
#pragma unroll
        for (int i = 0; i < MB * NB; ++i) acc[i / NB][i % NB] = sum[i / NB][i % NB];
        if (tid == 0) {
            __hip_atomic_store(&st->started, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->way, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->read, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // ---- the adapter slab and the terms of GEMV rows, as above, with the operands straight from memory.  Row block mb of the
    // wavefront: rows 32 RM wr + 16 mb + m of the block
    int tok[MB];
#pragma unroll
    for (int i = 0; i < RM; ++i) {  // (RM 1: row blocks 32 wr .. of the one run; RM 2: run wr)
        if (RM == 2 && i != wr) continue;  // uniform
        int ti[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ti[mb] = (RM == 1 ? 32 * wr : 0) + 16 * mb + m;
        tile_tokens_of(list.tok, run[i], ti, dead_tok, tok);
    }
    const int wrow = row0 + 32 * RM * wr, col0 = n0 + 32 * wc;  // the wavefront's first row and column
    const int seg0 = run[0].first_seg, seg1 = RM == 2 && run[RM - 1].n_segs > 0 ? run[RM - 1].first_seg + run[RM - 1].n_segs : seg0 + run[0].n_segs;
    for (int s = seg0; s < seg1; ++s) {
        const LinearSeg seg = list.segs[s];
        const int lo = seg.r0 - wrow, hi = seg.r1 - wrow;
        if (hi <= 0 || lo >= 32 * RM) continue;  // uniform
        const int rs = rank_storage(seg.rank), rs8 = rs >> 3, ks32 = (seg.rank + 31) >> 5;
        const __bf16 *Bp = reinterpret_cast<const __bf16 *>(a.proj_base + (int64_t)seg.row * a.row_bytes) + (size_t)rs * a.h_in;
#pragma unroll
        for (int k0 = 0; k0 < 4; k0 += 2) {  // two k steps at a time
            if (k0 >= ks32) continue;  // uniform
            bf16x8 bo[2][NB];
            uint4 vo[2][MB];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int gran = 4 * (k0 + ks) + g;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    bo[ks][nb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Bp + ((size_t)min(gran, rs8 - 1) * a.h_out + col0 + 16 * nb + m) * 8));
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    vo[ks][mb] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const __bf16 *>(a.v) + (size_t)tok[mb] * (2 * a.v_stride) + gran * 8);
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int r = 16 * mb + m;
                floatx4 had[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) had[nb] = acc[mb][nb];
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const bf16x8 so = sv_operand(vo[ks][mb], rank_mask(seg.rank - 32 * (k0 + ks) - 8 * g));
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bo[ks][nb], so, acc[mb][nb], 0, 0, 0);
                }
                keep_rows_outside<NB>(acc[mb], had, lo <= r && r < hi);  // (in every block: behind a branch the loads above would be made one block at a time, 28.5 -> 29.3 us at 785 x 2560 x 2560)
            }
        }
    }
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    if (wrow < list.add1 && wrow + 32 * RM > list.add0) {  // uniform
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int r = wrow + 16 * mb + m;
            if (r < list.add0 || r >= list.add1) continue;
            const size_t at = (size_t)tok[mb] * a.h_out + col0 + 4 * g;
            floatx4 term[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if (a.y32) {
                    term[nb] = *reinterpret_cast<const floatx4 *>(a.y32 + at + 16 * nb);
                } else {
                    const bf16x4 old = *reinterpret_cast<const bf16x4 *>(y + at + 16 * nb);
#pragma unroll
                    for (int e = 0; e < 4; ++e) term[nb][e] = (float)old[e];
                }
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[mb][nb][e] += term[nb][e];
        }
    }
    // ---- store: parked in LDS (row r: 16-byte slot s at s ^ ((r / 2) % 8)), then whole rows of the tile
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int row = 32 * RM * wr + 16 * mb + m;
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)acc[mb][nb][e];
            *reinterpret_cast<bf16x4 *>(lds + row * (2 * BN) + (((8 * wc + 4 * nb + g) ^ (((row >> 1) & 7) << 1)) << 3)) = o;
        }
    constexpr int PASSES = 2 * RM;  // 32 rows each, 8 lanes to a row
    const int sl = tid & 7, rl = tid >> 3;
    int tok8[PASSES];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int ti[2] = {rl, rl + 32};
        int tk[2];
        tile_tokens_of(list.tok, run[i], ti, dead_tok, tk);
#pragma unroll
        for (int p = 0; p < 2; ++p) tok8[2 * i + p] = ti[p] < run[i].n_tok ? tk[p] : -1;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int row = 32 * p + rl;
        const uint4 v = *reinterpret_cast<const uint4 *>(lds + row * (2 * BN) + ((sl ^ ((row >> 1) & 7)) << 4));
        typedef unsigned u32x4_nt __attribute__((ext_vector_type(4)));
        const u32x4_nt vn = {v.x, v.y, v.z, v.w};
        if (tok8[p] >= 0) __builtin_nontemporal_store(vn, reinterpret_cast<u32x4_nt *>(y + (size_t)tok8[p] * a.h_out + n0 + 8 * sl));
    }
}

// y[token][0 .. h_out) = 0 for the listed tokens (the rows the GEMV expand then adds its term to)
__global__ __launch_bounds__(256) void zero_rows_kernel(__bf16 *__restrict__ y, const int32_t *__restrict__ toks, int n, int h_out)
{
    const int per_row = h_out / 8;  // 16-byte pieces
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n * per_row; i += gridDim.x * 256) {
        const int r = i / per_row, c = i - r * per_row;
        *reinterpret_cast<uint4 *>(y + (size_t)toks[r] * h_out + c * 8) = make_uint4(0, 0, 0, 0);
    }
}

hipError_t launch_zero_rows(void *y, const int32_t *toks, int n, int h_out, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int blocks = std::min(1024, (n * (h_out / 8) + 255) / 256);
    hipLaunchKernelGGL(zero_rows_kernel, dim3(blocks), dim3(256), 0, st, static_cast<__bf16 *>(y), toks, n, h_out);
    return hipGetLastError();
}

// Parts the tiles of the last round are split into (1: none), and how many tiles that round has.  The number of parts
// is the one with the shortest estimate, in stages of 1.33 us: ceil(tiles * parts / CUs) waves of n_k / parts stages
// and about 8 more for a block's start and end, and the hand-over, whose bytes (512 KB for every part but one, written
// and read past the caches) take 0.09 stages each at the 4.5 TB/s of memory.  (48 tiles of 64 stages behind a whole round: 45 us in five
// parts, estimated 50; 136 tiles of 80 stages: 117 us in three parts, estimated 125, and whole 112, estimated 117.)
// max_shares: what the scratch holds, in accumulator sets of a tile (LINEAR_SHARE_BYTES).
static double linear_split_shape(int n_tiles, int n_k, int n_cu, size_t max_shares, int &parts, int &n_tail)
{
    n_tail = n_tiles % n_cu;
    parts = 1;
    double best = 0;
    for (int p = 1; p <= MAX_PARTS && (p == 1 || (p * 4 <= n_k && (size_t)n_tail * p <= max_shares)); ++p) {
        const double t = (double)((n_tail * p + n_cu - 1) / n_cu) * ((n_k + p - 1) / p + 8) + 0.09 * n_tail * (p - 1);
        if (p == 1 || t < best) best = t, parts = p;
    }
    if (parts == 1) n_tail = 0;
    return 1.33 * (best + (double)(n_tiles / n_cu) * (n_k + 8));
}

// Tiles of 64 RM x 64 (linear_small_kernel), n_k stages: estimated microseconds with the k range in `parts` parts.  4 us for a block's start and end; the
// stages of a block at 0.27 us (64 rows) or 0.38 us (128 rows), or the bytes the units take in, at a rate that falls where an XCD's L2 does not hold
// `l2_bytes`, x and its eighth of Wt (785 x 2560 x 2560, 5.6 MB, 128 rows: 23.3 us; 686 x 3264 x 3264, 7.2 MB: 38.2 us); a split's hand-over.
static double small_estimate(int n_tiles, int n_k, int rm, int parts, double l2_bytes)
{
    const bool fits = l2_bytes < 6.5e6;
    const double stage = rm == 1 ? 0.27 : 0.38, bytes = (double)n_tiles * n_k * 64 * (rm + 1) * LROW, rate = rm == 1 ? (fits ? 16e6 : 14e6) : (fits ? 15e6 : 12e6);
    const double hand_over = parts == 1 ? 0.0 : 1.5 + 0.5 * parts + (double)n_tiles * (parts - 1) * 64 * rm * 64 * 8 / 4.5e6;
    return 4.0 + std::max(stage * ((n_k + parts - 1) / parts), bytes / rate) + hand_over;
}

// Whole tiles of `rows` x 256 with n_k stages, as measured: 10 us for a block's start and end, and stages that take as long as their products at the matrix cores' peak
// while a quarter of the units is busy (0.91 us for 256 rows), and, all units busy, what the card sustains (1.38 us, 1.4 PFLOP/s): 64 tiles of 64 stages take 68 us, 128
// 72, 192 82, 256 98.5.  So a last round with few tiles is not as cheap as its share of the units, but cheaper than a full one.
static double rounds_us(int rows, int n_tiles, double n_k, int n_cu)
{
    const double peak = rows == 192 ? 0.77 : rows == 288 ? 1.02 : 0.906, full = 1.316 * (rows == 192 ? 0.726 : rows == 288 ? 1.104 : 1.0);
    double t = 0;
    for (int left = n_tiles; left > 0; left -= n_cu) {
        const double load = full * std::min(left, n_cu) / n_cu, p2 = peak * peak, l2 = load * load;
        t += 10 + n_k * std::sqrt(std::sqrt(p2 * p2 + l2 * l2));
    }
    return t;
}
// Tiles of 192 and 288 rows, whole ones only, where they fit the units better than tiles of 256 with their last round split.  Measured (us; tiles of 256 as chosen above, of
// 192, of 288): 4300 x 4096 x 4096 125 / 137 / 103 (272 tiles; 368; 240), 4416 132 / 136 / 108, 5809 155 / 151 / 184, 3000 80 / 77 / 87, 3500 x 2560 x 2560 49 / 44 / 53,
// 2560 x 13824 x 5120 273 / 286 / 257, 3000 x 11008 x 4096 219 / 223 / 204; not chosen: 2048 x 4096 x 4096 63 / 65 / 79, 2560 x 5120 x 5120 107 / 163 / 115, 1600 x 4096 x 4096
// 57 / 61 / 76; 160 and 224 rows were the best nowhere (2560 x 5120 x 5120: 168, 105).  The estimate is within 8 % of these, hence the 5 % it has to gain.
// Few stages are no exception.  Of 150 drawn products (500 to 9000 rows, 768 to 11500 columns) 90 of 12 to 35 stages take 1.092 times less in the geometric mean than with
// tiles of 256 alone (the best of the three each time 1.095), 60 of 3 to 11 stages 1.049 (1.070), and none that left 256 got slower: 4396 x 2112 x 4096 82.7 / 78.2 / 61.7,
// 5082 x 1024 x 3584 56.4 / 48.8 / 37.3, 4527 x 1536 x 2496 39.2 / 35.1 / 41.8, 7095 x 576 x 2368 43.3 / 35.6 / 27.5.

template <int RM, int NST> constexpr int small_lds = NST * 64 * (RM + 1) * LROW;

hipError_t prepare_linear_kernels()
{
    hipError_t e = allow_lds(linear_tiles_kernel<8>, linear_lds<8>);
    if (e == hipSuccess) e = allow_lds(linear_tiles_kernel<6>, linear_lds<6>);
    if (e == hipSuccess) e = allow_lds(linear_tiles_kernel<9>, linear_lds<9>);
    if (e == hipSuccess) e = allow_lds(linear_small_kernel<1, 4>, small_lds<1, 4>);
    if (e == hipSuccess) e = allow_lds(linear_small_kernel<1, 3>, small_lds<1, 3>);
    if (e == hipSuccess) e = allow_lds(linear_small_kernel<2, 3>, small_lds<2, 3>);
    return e;
}

template <int RM, int NST>
static hipError_t launch_small(const ApplyArgs &a, const void *Wt, const LinearList &list, int parts, void *split_scratch, SplitState *split_state,
                               hipStream_t st, const KernelTimer *tm, hipEvent_t done)
{
    const int n_mt = (list.n_rt + RM - 1) / RM, n_nt = a.h_out / 64;
    const LinearSplit sp{0, parts, static_cast<unsigned long long *>(split_scratch), split_state, nullptr};
    launch_k(tm, done, LORA_K_LINEAR, linear_small_kernel<RM, NST>, dim3(n_mt * n_nt * parts), dim3(256), small_lds<RM, NST>, st, a, static_cast<const __bf16 *>(Wt), list, n_mt, n_nt, sp);
    return hipGetLastError();
}

LinearShape linear_shape(int n_rows, int h_in, int h_out, size_t split_scratch_bytes, int n_split_state, int n_cu)
{
    const int n_rt = (n_rows + LORA_TILE_TOKENS - 1) / LORA_TILE_TOKENS, n_k = h_in / LBK, n_tiles = (n_rt + 3) / 4 * ((h_out + LBN - 1) / LBN);
    int parts, n_tail;
    // (the estimate reads 15 to 25 % more than 256 x 256 tiles take where the other kernel comes near them)
    const double big = 0.85 * linear_split_shape(n_tiles, n_k, n_cu, split_scratch_bytes / LINEAR_SHARE_BYTES, parts, n_tail);
    const int tiles64 = n_rt * (h_out / 64), tiles128 = (n_rt + 1) / 2 * (h_out / 64);
    const double l2_bytes = 2.0 * h_in * (64.0 * n_rt + h_out / 8);
    int p64 = 1;
    for (int p = 2; p <= MAX_PARTS && tiles64 <= n_split_state && 4 * p <= n_k && (size_t)tiles64 * p * 64 * 64 * 4 <= split_scratch_bytes; ++p)
        if (small_estimate(tiles64, n_k, 1, p, l2_bytes) < small_estimate(tiles64, n_k, 1, p64, l2_bytes)) p64 = p;
    const double t64 = small_estimate(tiles64, n_k, 1, p64, l2_bytes), t128 = small_estimate(tiles128, n_k, 2, 1, l2_bytes);
    // (a ring of four where all blocks fit side by side with it: 992 x 1024 x 1024 8.1 us, 8.8 with three; 2283 x 1088 x 1088 17.0, 14.4 with three)
    if (t64 <= big && t64 <= t128) return {64, tiles64 * p64 <= 2 * n_cu ? 4 : 3, tiles64, p64 > 1 ? tiles64 : 0, p64};
    if (t128 <= big) return {128, 3, tiles128, 0, 1};
    if (n_tail > n_split_state) parts = 1, n_tail = 0;
    const int n_nt = (h_out + LBN - 1) / LBN, whole = n_tiles - n_tail;
    const double now = rounds_us(256, whole, n_k, n_cu) + (parts > 1 ? rounds_us(256, n_tail * parts, (double)n_k / parts, n_cu) + 4.0 + 0.06 * n_tail * (parts - 1) : 0.0);
    const int tiles192 = (n_rows + 191) / 192 * n_nt, tiles288 = (n_rows + 287) / 288 * n_nt;
    const double t192 = rounds_us(192, tiles192, n_k, n_cu), t288 = rounds_us(288, tiles288, n_k, n_cu);
    if (std::min(t192, t288) < 0.95 * now) return t192 < t288 ? LinearShape{192, 2, tiles192, 0, 1} : LinearShape{288, 2, tiles288, 0, 1};
    return {LBM, 2, n_tiles, n_tail, parts};
}

hipError_t launch_linear_tiles(const ApplyArgs &a, const void *Wt, const LinearList &list, void *split_scratch,
                               size_t split_scratch_bytes, SplitState *split_state, int n_split_state, int32_t *fault, int n_cu,
                               hipStream_t st, const KernelTimer *tm, hipEvent_t done)
{
    if (list.n_rt <= 0) return hipSuccess;
    const LinearShape sh = linear_shape(list.n_rows, a.h_in, a.h_out, split_scratch_bytes, n_split_state, n_cu);
    if (sh.rows == 64 && sh.ring == 4) return launch_small<1, 4>(a, Wt, list, sh.parts, split_scratch, split_state, st, tm, done);
    if (sh.rows == 64) return launch_small<1, 3>(a, Wt, list, sh.parts, split_scratch, split_state, st, tm, done);
    if (sh.rows == 128) return launch_small<2, 3>(a, Wt, list, sh.parts, split_scratch, split_state, st, tm, done);
    const LinearSplit sp{sh.tiles - sh.split, sh.parts, static_cast<unsigned long long *>(split_scratch), split_state, fault};
    auto go = [&](auto mb_tag) {
        constexpr int MB = decltype(mb_tag)::value;
        launch_k(tm, done, LORA_K_LINEAR, linear_tiles_kernel<MB>, dim3(sp.n_whole + sh.split * sh.parts), dim3(512), linear_lds<MB>, st, a, static_cast<const __bf16 *>(Wt),
                 list, (list.n_rows + 32 * MB - 1) / (32 * MB), (a.h_out + LBN - 1) / LBN, sp);
    };
    switch (sh.rows) {
    case 192: go(std::integral_constant<int, 6>{}); break;
    case 288: go(std::integral_constant<int, 9>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
    }
    return hipGetLastError();
}

}  // namespace lora
