// Matrix-core path of the batched LoRA apply for gfx950 (bf16 in, fp32 accumulate): tiles of
// up to 64 tokens that share one cache slot -- prompt segments, or the pooled decode tokens
// of a hot adapter.  Built on v_mfma_f32_16x16x32_bf16; operand layout of that instruction:
//   A (16 x 32): lane l holds row l%16,  k = 8*(l/16) .. +7
//   B (32 x 16): lane l holds col l%16,  k = 8*(l/16) .. +7
//   D (16 x 16): lane l holds col l%16,  rows 4*(l/16) .. +3
// Because a contraction does not care about the order of k, both kernels give every lane
// group a k range that makes the lane's global loads contiguous and use the same range for
// both operands.
//
//   shrink:  V[tile][rank] = X[tile][k-range] . At^T        (split over k ranges of h_in)
//   expand:  Y[tile][cols]^T += Bp[cols][rank] . (s.V)^T     (split over column ranges)
//
// (paper section 3.1: the two adapter products and the aggregation into the base output.)
#include <algorithm>
#include <type_traits>

#include "lora_device.h"

namespace lora {

namespace {
constexpr int VS_ROW = LORA_MAX_RANK * 2 + 16;  // bytes per token row of the staged V tile (padded)
}  // namespace

// ---------------------------------------------------------------------------------------
// shrink.  Block = 4 wavefronts on one tile and one k range, walked in stages of 128 k.
//  - x, the HBM stream, goes through an LDS ring of three stages: every thread fetches four
//    16-byte pieces per stage with a wavefront instruction covering 4 token rows x 256
//    contiguous bytes, two stages ahead of the one being multiplied (so two stages of loads are
//    in flight in registers while a third waits ready in LDS), one barrier per stage.  Rows are
//    padded by 16 bytes, which puts the 16 rows of an A-operand read in distinct banks.
//  - At, which comes out of L2 and is shared by all tiles of a segment, is loaded into registers one
//    stage ahead -- the four lanes of a quad on one rank row (64-byte requests; in the operand's own
//    order, with neighbouring lanes in different rows, the same bytes cost the load path 1.7 times
//    as long) -- and put in operand order by a lane permutation before the products.
//  - From 4 rank blocks (of 16) up, wavefront w owns rank blocks w and w+4 for the whole k range
//    and writes its part of V itself.  Below that, the wavefronts split the four MFMA k steps of
//    a stage instead, each covering all rank blocks, and their partials are summed through LDS.
//  - The launch's work -- every tile's k range -- is cut into runs of about equal cost, one block per run
//    (and projection), all blocks resident at once: a block walks the pieces of its run, a piece being a k
//    range of one tile.  A piece that is not a whole tile leaves a partial sum in the scratch slot of its run
//    and mfma_reduce_kernel adds a tile's pieces up.  (With one block per tile and a fixed number of k ranges
//    the launch ended when the XCD with the most or the costliest tiles did: a timeline of the prefill
//    configuration showed half of the blocks done at 15 us and the last at 26 us.)
// Blocks are numbered so that consecutive runs (same tiles, same segment, same At) fall on one XCD (blocks
// b, b + 8, ... run on XCD b % 8).
// One launch serves the projections of a batch; those that read the same x (q, k, v; gate, up) share its fetch.
// ---------------------------------------------------------------------------------------
namespace {
constexpr int SK = SHRINK_STAGE_K;      // k elements per stage
constexpr int XROW = SK * 2 + 16;       // bytes per token row of a stage in LDS
constexpr int NSTAGE = 3;
}  // namespace

// Every global load below is unconditional, from an address clamped into the tensor, and what
// must not count is zeroed where x is written to LDS (zero x rows and zero x tail columns make
// whatever At held there irrelevant).  Loads under a condition would be compiled into branches,
// and the wait counters cannot be tracked across those: every stage would then wait for all
// outstanding loads and the prefetch distance would collapse to nothing.
// token id of row ti (>= 0) of a tile
__device__ __forceinline__ int tile_token(const ApplyArgs &a, const DevItem &it, int ti)
{
    return tile_token_of(a.tok_list, it, ti);
}

// token ids of N rows of a tile at once (rows past the tile's last count as its last)
template <int N>
__device__ __forceinline__ void tile_tokens(const ApplyArgs &a, const DevItem &it, const int (&ti)[N], int (&tok)[N])
{
    tile_tokens_of(a.tok_list, it, ti, it.tok0, tok);
}

template <bool NSPLIT, int NBW>  // NBW: rank blocks (of 16) a wavefront works on
__device__ __forceinline__ void mfma_shrink_body(const ApplyArgs &a, const DevItem &it, int k_begin, int k_end, int phase,
                                                 float *part, unsigned char (*xs)[LORA_TILE_TOKENS * XROW])
{
    constexpr int NKW = NSPLIT ? 4 : 1;  // MFMA k steps of a stage a wavefront works on
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int rs = rank_storage(it.rank);
    const int n_st = (k_end - k_begin + SK - 1) / SK;
    const int k_last = a.h_in - 8;  // last 16-byte piece of a row

    const __bf16 *At = reinterpret_cast<const __bf16 *>(a.proj_base + (int64_t)it.row * a.row_bytes);
    const __bf16 *x = static_cast<const __bf16 *>(a.x);

    // k offset of stage st.  The walk over k starts at a different stage in every block, so that
    // blocks running side by side do not all pull the same column window (rows lie h_in apart)
    auto stage_k = [&](int st) {
        // (the prefetches run up to three stages past the end: they re-read the last stage, which is
        // still in L1/L2 -- wrapped round to the first stages they came from memory again, +43 % of x
        // for a block of seven stages)
        int s = min(st, n_st - 1) + phase;
        s -= s >= n_st ? n_st : 0;
        return k_begin + s * SK;
    };

    // loader: rows 16w + 4i + lane/16, piece lane%16 (8 elements)
    const int lp = lane & 15;
    const __bf16 *xg[4];
    int lds_off[4];
    bool x_ok[4];
    {
        int row[4], tok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = 16 * w + 4 * i + (lane >> 4);
        tile_tokens(a, it, row, tok);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x_ok[i] = row[i] < it.n_tok;
            xg[i] = x + (size_t)tok[i] * a.h_in;
            lds_off[i] = row[i] * XROW + lp * 16;
        }
    }
    // At operands: block slot q -> rank block nbq; rows past the stored rank are clamped (their
    // results are never written)
    // A B operand wants, in lane (m, g), rank row m and k chunk g of the step: 16 rows x 64 bytes per load
    // instruction with neighbouring lanes in different rows, the costliest shape for the load path.  The same
    // 16 x 64 bytes are therefore fetched with the four lanes of a quad on one row (lane l: row l/4, chunk
    // l%4 -- a 64-byte request per quad) and put in operand order by a lane permutation on the way to the
    // products (ds_bpermute: lane (m, g) takes the registers of lane 4m + g).
    int nbq[NBW];
    const __bf16 *ag[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q) {
        nbq[q] = NSPLIT ? w + 4 * q : q;
        ag[q] = At + (size_t)min(16 * nbq[q] + (lane >> 2), rs - 1) * a.h_in;
    }
    const int perm_src = 4 * (4 * m + g);  // byte address of the source lane, as ds_bpermute takes it
    const int ks0 = NSPLIT ? 0 : w;  // first MFMA k step of a stage for this wavefront

    uint4 xr[2][4];
    auto load_x = [&](int st, uint4(&d)[4]) {
        const int k = min(stage_k(st) + lp * 8, k_last);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = *reinterpret_cast<const uint4 *>(xg[i] + k);
    };
    auto store_x = [&](int slot, int st, const uint4(&d)[4]) {
        const bool k_ok = stage_k(st) + lp * 8 < k_end;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<uint4 *>(&xs[slot][lds_off[i]]) = (x_ok[i] && k_ok) ? d[i] : make_uint4(0, 0, 0, 0);
    };
    uint4 br[2][NBW][NKW];
    auto load_at = [&](int st, uint4(&d)[NBW][NKW]) {
        const int k = stage_k(st) + 8 * (lane & 3);
#pragma unroll
        for (int q = 0; q < NBW; ++q)
#pragma unroll
            for (int j = 0; j < NKW; ++j) d[q][j] = *reinterpret_cast<const uint4 *>(ag[q] + min(k + 32 * (ks0 + j), k_last));
    };
    auto operand_of = [&](const uint4 &r) {
        uint4 o;
        o.x = __builtin_amdgcn_ds_bpermute(perm_src, r.x);
        o.y = __builtin_amdgcn_ds_bpermute(perm_src, r.y);
        o.z = __builtin_amdgcn_ds_bpermute(perm_src, r.z);
        o.w = __builtin_amdgcn_ds_bpermute(perm_src, r.w);
        return __builtin_bit_cast(bf16x8, o);
    };

    floatx4 acc[4][NBW];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int q = 0; q < NBW; ++q) acc[mb][q] = floatx4{0.f, 0.f, 0.f, 0.f};

    load_x(0, xr[0]);
    load_x(1, xr[1]);
    load_at(0, br[0]);
    store_x(0, 0, xr[0]);
    load_x(2, xr[0]);
    __syncthreads();

    // one stage; CUR = st % 2 and SLOT = st % 3 are compile-time constants so that the staging
    // arrays stay in registers and the ring slots are fixed addresses
    auto stage = [&](auto cur_tag, auto slot_tag, int st) {
        constexpr int CUR = decltype(cur_tag)::value;
        constexpr int SLOT = decltype(slot_tag)::value;
        load_at(st + 1, br[CUR ^ 1]);  // At of the next stage, then this stage's products
        const unsigned char *xb = xs[SLOT];
        bf16x8 bop[NBW][NKW];
#pragma unroll
        for (int q = 0; q < NBW; ++q)
#pragma unroll
            for (int j = 0; j < NKW; ++j) bop[q][j] = operand_of(br[CUR][q][j]);
#pragma unroll
        for (int j = 0; j < NKW; ++j) {
            const int ks = ks0 + j;
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) {
                const bf16x8 av = *reinterpret_cast<const bf16x8 *>(&xb[(16 * mb + m) * XROW + (4 * ks + g) * 16]);
#pragma unroll
                for (int q = 0; q < NBW; ++q) acc[mb][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bop[q][j], acc[mb][q], 0, 0, 0);
            }
        }
        // stage st+1 goes to LDS (its buffer was last read two barriers ago), stage st+3 is requested
        store_x((SLOT + 1) % NSTAGE, st + 1, xr[CUR ^ 1]);
        load_x(st + 3, xr[CUR ^ 1]);
        __syncthreads();
    };
    // (the walk leaves through a break after its last stage: with every stage under a condition of its own a
    // stage can be reached past a skipped one as far as the compiler can tell, the load counts it merges at
    // such a join are the smallest of both ways, and every wait for x then also waited for the requests of
    // the stage before -- the two-stage lead of x was one)
    for (int st = 0;; st += 6) {
        stage(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, st);
        if (st + 1 >= n_st) break;
        stage(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, st + 1);
        if (st + 2 >= n_st) break;
        stage(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{}, st + 2);
        if (st + 3 >= n_st) break;
        stage(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{}, st + 3);
        if (st + 4 >= n_st) break;
        stage(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, st + 4);
        if (st + 5 >= n_st) break;
        stage(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{}, st + 5);
        if (st + 6 >= n_st) break;
    }

    // Where the rows go.  The tile's whole k range: the result itself, into the rows of v that belong to the
    // tile's tokens; else this piece's partial sum, one row per row of the tile (mfma_reduce_kernel adds the
    // pieces up).  The row numbers are all fetched before the first store: a lookup between two stores makes
    // the second wait for the first to be acknowledged (loads and stores share the counter, which can only
    // be waited down), 0.3 us each -- 10 us for the 32 stores of a rank-128 piece
    float *const out = part ? part : a.v;
    auto rows_of = [&](int mb, int (&rows)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) rows[r] = 16 * mb + 4 * g + r;
        if (part) return;
        const int ti[4] = {rows[0], rows[1], rows[2], rows[3]};
        tile_tokens(a, it, ti, rows);
    };
    // (a whole tile's result goes out as the expand takes it: scaled and rounded to bf16, rows of the same pitch)
    const float s_v = a.scale * it.alpha;
    __bf16 *const out16 = reinterpret_cast<__bf16 *>(a.v);
    auto write_v = [&](int mb, const int (&rows)[4], int q, const floatx4 &val) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ti = 16 * mb + 4 * g + r, jr = 16 * nbq[q] + m;
            if (ti < it.n_tok && jr < it.rank) {
                if (part) out[(size_t)rows[r] * a.v_stride + jr] = val[r];
                else out16[(size_t)rows[r] * (2 * a.v_stride) + jr] = (__bf16)(s_v * val[r]);
            }
        }
    };
    if (NSPLIT) {
        int rows[4][4];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) rows_of(mb, rows[mb]);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int q = 0; q < NBW; ++q) write_v(mb, rows[mb], q, acc[mb][q]);
    } else {
        // the four wavefronts hold partial sums over k: park them in the (now idle) x ring and let
        // wavefront w add up and write token block w
        float *red = reinterpret_cast<float *>(&xs[0][0]);  // [wave][mb][q][r][lane], at most 4*4*3*4*64*4 B = 48 KB
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int q = 0; q < NBW; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(((w * 4 + mb) * NBW + q) * 4 + r) * 64 + lane] = acc[mb][q][r];
        int rows[4];
        rows_of(w, rows);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NBW; ++q) {
            floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int src = 0; src < 4; ++src)
#pragma unroll
                for (int r = 0; r < 4; ++r) sum[r] += red[(((src * 4 + w) * NBW + q) * 4 + r) * 64 + lane];
            write_v(w, rows, q, sum);
        }
    }
}

constexpr int SKD = 64, SROW = SKD * 2;  // k elements of a stage of the kernels below, and the bytes of a row

// the arguments of one projection of the batch
template <int N>
__device__ __forceinline__ ApplyArgs tile_args(const TileBatchArgs<N> &tb, int pj)
{
    const BatchProj &p = tb.p[pj];
    ApplyArgs a;
    a.proj_base = p.proj_base;
    a.row_bytes = (int64_t)(p.h_in + p.h_out) * 2;
    a.tok_list = tb.tok_list;
    a.x = p.x;
    a.y = p.y;
    a.v = tb.v + (size_t)pj * tb.v_set;
    a.h_in = p.h_in;
    a.h_out = p.h_out;
    a.v_stride = tb.v_stride;
    a.scale = tb.scale;
    return a;
}

// Copy (of the three kernels of the shrink): nothing, or the ListCopy of lists that blocks behind the others copy
template <int N, typename... Copy>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_shrink_kernel(const ShrinkCut *__restrict__ cuts, const DevItem *__restrict__ tiles, int runs_per_xcd, int n_proj, int quanta,
                                                                                                        int n_tiles, TileBatchArgs<N> tb, Copy... copy)
{
    if constexpr (sizeof...(Copy) > 0)
        if ((... || (blockIdx.x >= copy.first_block))) return (copy_lists(copy, blockIdx.x, 256), ...);
    // (the scalars in front are fields of tb: leading arguments arrive in registers with the wavefront)
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    unsigned char(*const xs)[LORA_TILE_TOKENS * XROW] = reinterpret_cast<unsigned char(*)[LORA_TILE_TOKENS * XROW]>(ring);
    static_assert(NSTAGE * LORA_TILE_TOKENS * XROW >= 4 * 4 * 3 * 4 * 64 * 4, "the sum over the wavefronts' k parts reuses the x ring");

    // XCD j = blockIdx % 8 works on the runs [j * runs_per_xcd, (j + 1) * runs_per_xcd) of every group, group by group;
    // its i-th block of a group on (run, projection) number i, projection innermost: the blocks that read the same part
    // of x for the projections of a group are neighbours in the dispatch order of one XCD and walk k in the same order,
    // so that x is fetched from memory once and found in L2 by the others
    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    int g0 = 0, gn = n_proj;  // the block's group: first projection and size
    if constexpr (N > GROUP_MAX_PROJS) {
        const uint32_t grp = tb.group[local / runs_per_xcd];  // (indexed by a projection of the group)
        g0 = (int)(grp & 0xffu);
        gn = (int)(grp >> 8);
    }
    const int in_group = local - g0 * runs_per_xcd;
    const int run = xcd * runs_per_xcd + in_group / gn, pj = g0 + in_group % gn;
    const ShrinkCut from = cuts[run], to = cuts[run + 1];
    const ApplyArgs a = tile_args(tb, pj);
    const int last_tile = min(to.part > 0 ? to.tile : to.tile - 1, n_tiles - 1);
    for (int tile = from.tile; tile <= last_tile; ++tile) {
        const int lo = tile == from.tile ? from.part : 0, hi = tile == to.tile ? to.part : quanta;
        if (lo >= hi) continue;  // (an empty run)
        const DevItem it = tiles[tile];
        const int k_begin = shrink_part_stage(lo, quanta, a.h_in, SK) * SK;
        const int k_end = min(a.h_in, shrink_part_stage(hi, quanta, a.h_in, SK) * SK);
        const int n_st = (k_end - k_begin + SK - 1) / SK;
        const int phase = (int)(((unsigned)(run + tile) * 5u) % (unsigned)n_st);
        float *my_part = (lo == 0 && hi == quanta)
                             ? nullptr
                             : tb.part + (size_t)pj * tb.part_set + (size_t)shrink_slot(run, from.tile, tile) * SHRINK_SLOT_ROWS * a.v_stride;
        const int NB = (it.rank + 15) >> 4;
        if (NB > 4) mfma_shrink_body<true, 2>(a, it, k_begin, k_end, phase, my_part, xs);
        else if (NB == 4) mfma_shrink_body<true, 1>(a, it, k_begin, k_end, phase, my_part, xs);
        else if (NB == 3) mfma_shrink_body<false, 3>(a, it, k_begin, k_end, phase, my_part, xs);
        else if (NB == 2) mfma_shrink_body<false, 2>(a, it, k_begin, k_end, phase, my_part, xs);
        else mfma_shrink_body<false, 1>(a, it, k_begin, k_end, phase, my_part, xs);
        __syncthreads();  // the next piece reuses the ring
    }
}

// ---------------------------------------------------------------------------------------
// shrink of a short launch: a block of W wavefronts per (projection, unit of 16 tokens x 16 rank rows), the wavefronts split k.  With the
// kernel above such a launch leaves every tile in pieces of a few stages, 9 to 12 us, and 4 to 6 us more to add them up; what it waits
// for is the trip to memory, so here a wavefront keeps three stages of 64 k of its own on their way in LDS (requests that write LDS
// themselves, waited for by count; 8 rows x 128 bytes each), meets no barrier before the end, and the block writes the result itself.
// x is taken in once per 16 rank rows and At once per 16 tokens: for short launches only.
// LDS rows of a stage as in linear_kernels.hip: 16-byte slot s of row r holds piece s ^ ((r / 2) % 8).
// ---------------------------------------------------------------------------------------
namespace {
constexpr int DK = 64, DROW = DK * 2, DSTAGE = 32 * DROW, DRING = 4;  // 16 rows of x, 16 of At
}  // namespace

template <int N, int W, typename... Copy>
__global__ __launch_bounds__(64 * W) void mfma_shrink_direct_kernel(TileBatchArgs<N> tb, Copy... copy)
{
    if constexpr (sizeof...(Copy) > 0)
        if ((... || (blockIdx.x >= copy.first_block))) return (copy_lists(copy, blockIdx.x, 64 * W), ...);
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    // XCD j (blocks j, j + 8, ...) takes a run of consecutive (projection, unit) pairs
    const int n = tb.n_direct * tb.n, j8 = (int)blockIdx.x & 7, pos = j8 * (n >> 3) + min(j8, n & 7) + ((int)blockIdx.x >> 3);
    const int pj = pos / tb.n_direct;
    const DevItem it = tb.direct[pos - pj * tb.n_direct];
    const ApplyArgs a = tile_args(tb, pj);
    const int rs = rank_storage(it.rank);
    const __bf16 *At = reinterpret_cast<const __bf16 *>(a.proj_base + (int64_t)it.row * a.row_bytes);
    const int n_k = a.h_in / DK, k_lo = n_k * w / W, n_st = n_k * (w + 1) / W - k_lo;

    const int lr = lane >> 3, ls = lane & 7;
    const __bf16 *src[4];
    {
        const int ti[2] = {lr, 8 + lr};
        int tok[2];
        tile_tokens(a, it, ti, tok);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int piece = ls ^ ((4 * q + (lr >> 1)) & 7);
            src[q] = static_cast<const __bf16 *>(a.x) + (size_t)tok[q] * a.h_in + (size_t)k_lo * DK + piece * 8;
            src[2 + q] = At + (size_t)min(it.a + 8 * q + lr, rs - 1) * a.h_in + (size_t)k_lo * DK + piece * 8;  // rows past the stored rank: never written
        }
    }
    unsigned char *const mine = ring + w * (DRING * DSTAGE);
    auto request = [&](int st, int slot) {
#pragma unroll
        for (int q = 0; q < 4; ++q) request16(src[q] + st * DK, mine + slot * DSTAGE + q * 8 * DROW);
    };
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int slot) {
        const unsigned char *s = mine + slot * DSTAGE + m * DROW;
        bf16x8 xo[2], ao[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int at = ((4 * ks + g) ^ ((m >> 1) & 7)) << 4;
            xo[ks] = *reinterpret_cast<const bf16x8 *>(s + at);
            ao[ks] = *reinterpret_cast<const bf16x8 *>(s + 16 * DROW + at);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo[ks], ao[ks], acc, 0, 0, 0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before the slot is requested again
    };
#pragma unroll
    for (int s = 0; s < DRING - 1; ++s)
        if (s < n_st) request(s, s);
    int slot = 0;
    for (int st = 0; st < n_st - (DRING - 1); ++st) {
        request(st + DRING - 1, (slot + DRING - 1) % DRING);
        wait_requests<4 * (DRING - 1)>();
        multiply(slot);
        slot = (slot + 1) % DRING;
    }
    auto last = [&](auto left_tag) {
        constexpr int LEFT = decltype(left_tag)::value;  // stages behind this one
        if (n_st <= LEFT) return;
        wait_requests<4 * LEFT>();
        multiply(slot);
        slot = (slot + 1) % DRING;
    };
    last(std::integral_constant<int, 2>{});
    last(std::integral_constant<int, 1>{});
    last(std::integral_constant<int, 0>{});
    static_assert(DRING == 4, "the walk's last stages");

    // add the wavefronts' sums (in a part of the ring that the wavefront alone has used); entry (token, rank row) of thread tid: token tid / 16, row tid % 16
    float *const sums = reinterpret_cast<float *>(mine);
#pragma unroll
    for (int r = 0; r < 4; ++r) sums[(4 * g + r) * 16 + m] = acc[r];
    __syncthreads();
    if (tid >= 256) return;
    const int ti = tid >> 4, jr = it.a + (tid & 15);
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < W; ++q) v += reinterpret_cast<const float *>(ring + q * (DRING * DSTAGE))[tid];
    const int tix[1] = {ti};
    int tok[1];
    tile_tokens(a, it, tix, tok);
    if (ti < it.n_tok && jr < it.rank) reinterpret_cast<__bf16 *>(a.v)[(size_t)tok[0] * (2 * a.v_stride) + jr] = (__bf16)(a.scale * it.alpha * v);
}

// ---------------------------------------------------------------------------------------
// shrink of a longer launch: a block of 8 wavefronts per (panel, k slice, up to three projections that read the same x), a panel being up to 192 rows of one slot (the tiles of
// a prompt put together again).
// What bounded the kernel above there is what misses L2: At once per tile of 64 rows, and x once per projection, since the blocks of q, k and v drift apart by more than an L2 holds of what
// 32 units have on their way (7B mixed batch: 2.9 GB fetched, 1.7 of them x; 1.65 GB this way).  Here At comes in once per panel and x once per group, and a launch is then bound by what
// the units take in (45 to 60 bytes per ns each), or by the memory where many small ranks make x nearly everything.
// x and At travel through an LDS ring of three to six stages of 64 k that the requests write themselves, waited for by count, one barrier per stage.  A ring slot: 64 TT rows of x, then 16 NB
// rows of At per projection (NB: rank blocks of 16), rows of 128 bytes, 16-byte slot s of row r holding piece s ^ ((r / 2) % 8).  Wavefront w multiplies every fourth row block with one half of
// the rank blocks: with all of them per wavefront and two row blocks each, the operand reads out of LDS took longer than the loads (7B mixed batch 491 us, 443 this way).
// What it takes in from behind L2 bounds it: eight prompts on q of eight layers, 281 MB of x and 122 of At, 76 us; x alone 55 to 58, without products 75; one stage less on its way, or more of x by
// rings of their own for x and At, gains nothing, whole 256-byte pieces of the rows take longer (68 us for x alone).
// 192 rows: with 256 three projections of rank 64 leave no room for three stages.  The panels are dealt out to the XCDs two neighbours at a time, the costliest first: in runs of neighbours per XCD, as
// the kernel above takes its tiles, some XCDs got most of the rank-128 panels (443 -> 338 us); a panel's blocks, if it has several, run side by side on one XCD.
// Measured, shrink and reduce of a launch, run table -> panels: 7B mixed batch (14 projections) 491 -> 338 us, eight prompts on q of eight layers 89 -> 75, 13B batch 100 -> 82;
// q, k, v of 17650 tokens in 100 prompts 99.6 -> 78.8, of 8485 in 20 prompts 45 -> 38 (three slices); one projection of 4291 tokens 20.2 -> 19.3 (six slices).
// ---------------------------------------------------------------------------------------
namespace {
constexpr int PANEL_RING = 156 << 10;  // of the 160 KB of a unit: one block to a unit
static_assert(PANEL_SLOT_ROWS * SROW * 3 <= PANEL_RING, "three stages at least");
}
struct PanelArgs {
    const __bf16 *x, *at0;
    int64_t at1, at2;  // At of the block's projections: the first, and how many elements further the others lie
    const int32_t *tok_list;
    __bf16 *v;    // of the first projection; the next lie v_set floats further
    float *part;  // the slice's sums of the panel, as v; null: the slice is everything, the result goes to v
    uint64_t v_set, part_set;
    int h_in, v_stride;
    float scale;
};
template <int TT, int NB, int NP>
__device__ __forceinline__ void mfma_panel_body(const PanelArgs &a, const DevItem &it, int st_begin, int n_st, int phase, unsigned char *ring)
{
    constexpr int NBT = NB * NP;  // rank blocks of all projections
    constexpr int SLOT = (64 * TT + 16 * NBT) * SROW, FIT = PANEL_RING / SLOT, NST = FIT < 6 ? FIT : 6, PER_AT = NBT / 4;
    // a wavefront's products: TT row blocks (every fourth) with half of the rank blocks; where there is but one of those, half of the row blocks
    constexpr bool ODD = NBT % 4 != 0, HALF_ROWS = NBT == 1;
    constexpr int RB = HALF_ROWS ? (TT + 1) / 2 : TT, NQ = (NBT + 1) / 2, STEP = HALF_ROWS ? 8 : 4;  // STEP: between a wavefront's row blocks
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int rs = rank_storage(it.rank);
    const int lr = lane >> 3, piece = (lane & 7) ^ ((4 * (w & 1) + (lr >> 1)) & 7);
    const bool more = ODD && w < 2 * (NBT % 4);
    const __bf16 *src[TT + PER_AT + ODD];
    {
        int ti[TT], tok[TT];
#pragma unroll
        for (int q = 0; q < TT; ++q) ti[q] = 8 * w + 64 * q + lr;
        tile_tokens_of(a.tok_list, it, ti, it.tok0, tok);  // (rows past the panel's end repeat its last)
#pragma unroll
        for (int q = 0; q < TT; ++q) src[q] = a.x + (size_t)tok[q] * a.h_in;
    }
#pragma unroll
    for (int q = 0; q < PER_AT + ODD; ++q) {
        const int grp = min(w + 8 * q, 2 * NBT - 1), pj = NP == 1 ? 0 : grp / (2 * NB), r = 8 * (grp - 2 * NB * pj) + lr;  // (wavefront-uniform but for lr)
        const __bf16 *at = a.at0;
        if constexpr (NP > 1) at += pj == 1 ? a.at1 : 0;
        if constexpr (NP > 2) at += pj == 2 ? a.at2 : 0;
        src[TT + q] = at + (size_t)min(r, rs - 1) * a.h_in;  // (rows past the stored rank: never written)
    }
    auto request = [&](int st, int slot) {
        int s = st + phase;
        s -= s >= n_st ? n_st : 0;
        const int k = (st_begin + s) * SKD + piece * 8;
        unsigned char *dst = ring + slot * SLOT + 8 * w * SROW;
#pragma unroll
        for (int q = 0; q < TT; ++q) request16(src[q] + k, dst + 64 * q * SROW);
#pragma unroll
        for (int q = 0; q < PER_AT; ++q) request16(src[TT + q] + k, dst + (64 * TT + 64 * q) * SROW);
        if (more) request16(src[TT + PER_AT + ODD - 1] + k, dst + (64 * TT + 64 * PER_AT) * SROW);
    };
    floatx4 acc[RB][NQ];
#pragma unroll
    for (int t = 0; t < RB; ++t)
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[t][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int rb0 = w % STEP, q0 = HALF_ROWS ? 0 : (w >> 2) * NQ;
    auto row_live = [&](int t) { return RB * STEP == 4 * TT || rb0 + STEP * t < 4 * TT; };  // (uniform)
    auto rank_live = [&](int q) { return NQ * 2 == NBT || HALF_ROWS || q0 + q < NBT; };
    // the operands of a stage's two k steps: those of one are read while the products of the one before run.  (All of a stage's reads first and its products behind them, the wavefronts being in
    // step, leave LDS and the matrix cores waiting for each other, but what comes in bounds the launch, see above: 0.3 % of a pass over layers of rank 128 (16 prompts of 512 tokens 4096 wide 720 -> 712 us), nothing in the
    // mean of 90 batches of prompts.)
    bf16x8 xo[2][RB], ao[2][NQ];
    auto read = [&](int slot, auto ks_tag) {
        constexpr int KS = decltype(ks_tag)::value;
        const unsigned char *xs = ring + slot * SLOT + (16 * rb0 + m) * SROW, *as = ring + slot * SLOT + (64 * TT + 16 * q0 + m) * SROW;
        const int at = ((4 * KS + g) ^ ((m >> 1) & 7)) << 4;
#pragma unroll
        for (int t = 0; t < RB; ++t) xo[KS][t] = *reinterpret_cast<const bf16x8 *>(xs + (row_live(t) ? 16 * STEP * t : 0) * SROW + at);
#pragma unroll
        for (int q = 0; q < NQ; ++q) ao[KS][q] = *reinterpret_cast<const bf16x8 *>(as + (rank_live(q) ? 16 * q : 0) * SROW + at);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto products = [&](auto ks_tag) {
        constexpr int KS = decltype(ks_tag)::value;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int t = 0; t < RB; ++t) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo[KS][t], ao[KS][q], acc[t][q], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    using step0 = std::integral_constant<int, 0>;
    using step1 = std::integral_constant<int, 1>;
#pragma unroll
    for (int t = 0; t < RB; ++t) xo[1][t] = bf16x8{};  // (the products before the first stage add nothing)
#pragma unroll
    for (int q = 0; q < NQ; ++q) ao[1][q] = bf16x8{};
    auto multiply = [&](int slot) {
        read(slot, step0{});
        products(step1{});  // of the stage before
        read(slot, step1{});
        products(step0{});
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read when this wavefront is at the next barrier
    };
    auto wait = [&](auto left_tag) {
        constexpr int LEFT = decltype(left_tag)::value;
        if (more) wait_requests<LEFT *(TT + 1 + PER_AT)>();
        else wait_requests<LEFT *(TT + PER_AT)>();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < n_st) request(s, s);
    int slot = 0, fill = NST - 1;
    for (int st = 0; st < n_st - (NST - 1); ++st) {
        wait(std::integral_constant<int, NST - 2>{});
        request(st + NST - 1, fill);
        multiply(slot);
        fill = slot;
        slot = slot + 1 == NST ? 0 : slot + 1;
    }
    auto last = [&](auto left_tag) {
        constexpr int LEFT = decltype(left_tag)::value;
        if constexpr (LEFT < NST - 1) {
            if (n_st <= LEFT) return;
            wait(left_tag);
            multiply(slot);
            slot = slot + 1 == NST ? 0 : slot + 1;
        }
    };
    last(std::integral_constant<int, 4>{});
    last(std::integral_constant<int, 3>{});
    last(std::integral_constant<int, 2>{});
    last(std::integral_constant<int, 1>{});
    last(std::integral_constant<int, 0>{});
    static_assert(NST >= 3 && NST <= 6, "the walk's last stages");
    products(step1{});
    const float s_v = a.scale * it.alpha;
    int ti[4 * RB], rows[4 * RB];
#pragma unroll
    for (int t = 0; t < RB; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) ti[4 * t + r] = 16 * (rb0 + STEP * t) + 4 * g + r;
    if (!a.part) tile_tokens_of(a.tok_list, it, ti, it.tok0, rows);
#pragma unroll
    for (int t = 0; t < RB; ++t) {
        if (!row_live(t)) continue;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (!rank_live(q)) continue;
            const int qq = q0 + q, pj = NP == 1 ? 0 : qq / NB, jr = 16 * (qq - NB * pj) + m;  // a rank block of projection pj (wavefront-uniform)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * t + r;
                if (ti[i] < it.n_tok && jr < it.rank) {
                    if (a.part) a.part[pj * a.part_set + (size_t)ti[i] * a.v_stride + jr] = acc[t][q][r];
                    else a.v[2 * pj * a.v_set + (size_t)rows[i] * (2 * a.v_stride) + jr] = (__bf16)(s_v * acc[t][q][r]);
                }
            }
        }
    }
}

template <int N, typename... Copy>
__global__ __launch_bounds__(512) void mfma_panel_kernel(const DevItem *panels, PanelClasses cls, PanelShape<N> sh, TileBatchArgs<N> tb, Copy... copy)
{
    if constexpr (sizeof...(Copy) > 0)
        if ((... || (blockIdx.x >= copy.first_block))) return (copy_lists(copy, blockIdx.x, 512), ...);
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    int gi = 0;  // the first group whose blocks end behind this one (the groups of long rows come first)
#pragma unroll
    for (int step = N / 2; step > 0; step >>= 1)
        if ((int)blockIdx.x >= sh.end[gi + step - 1]) gi += step;
    const uint32_t grp = sh.group[gi];
    const int g0 = (int)(grp & 0xffu), gn = (int)(grp >> 8 & 0xffu), slices = (int)(grp >> 16);
    int slice, panel, first, n;
    if (!panel_of_block(cls, gn, slices, (int)blockIdx.x - (gi ? sh.end[gi - 1] : 0), slice, panel, first, n)) return;
    const DevItem it = panels[panel];
    const int pj = g0 + first;
    auto at_of = [&](int i) {
        const BatchProj &p = tb.p[pj + i];
        return reinterpret_cast<const __bf16 *>(p.proj_base + (int64_t)it.row * (p.h_in + p.h_out) * 2);
    };
    PanelArgs a;
    a.x = static_cast<const __bf16 *>(tb.p[pj].x);
    a.at0 = at_of(0), a.at1 = at_of(n > 1 ? 1 : 0) - a.at0, a.at2 = at_of(n > 2 ? 2 : 0) - a.at0;
    a.tok_list = tb.tok_list;
    a.v = reinterpret_cast<__bf16 *>(tb.v + (size_t)pj * tb.v_set);
    a.part = slices == 1 ? nullptr : tb.part + (size_t)pj * tb.part_set + ((size_t)slice * tb.n_rows + it.tok_off) * tb.v_stride;
    a.v_set = tb.v_set, a.part_set = tb.part_set;
    a.h_in = tb.p[pj].h_in, a.v_stride = tb.v_stride;
    a.scale = tb.scale;
    const int n_k = a.h_in / SKD, k_lo = n_k * slice / slices, n_st = n_k * (slice + 1) / slices - k_lo;
    const int phase = (int)((unsigned)(it.row * 5 + g0 * 7) % (unsigned)n_st);
    const int nb = panel_rank_blocks(it.rank), tt = (it.n_tok + 63) >> 6;
    auto go = [&](auto tt_tag, auto nb_tag) __attribute__((always_inline)) {
        constexpr int T = decltype(tt_tag)::value, B = decltype(nb_tag)::value, MOST = panel_projs(T, B);
        if constexpr (MOST >= 3) if (n == 3) return mfma_panel_body<T, B, 3>(a, it, k_lo, n_st, phase, ring);
        if constexpr (MOST >= 2) if (n == 2) return mfma_panel_body<T, B, 2>(a, it, k_lo, n_st, phase, ring);
        mfma_panel_body<T, B, 1>(a, it, k_lo, n_st, phase, ring);
    };
    auto with_rows = [&](auto tt_tag) __attribute__((always_inline)) {
        if (nb == 8) go(tt_tag, std::integral_constant<int, 8>{});
        else if (nb == 6) go(tt_tag, std::integral_constant<int, 6>{});
        else if (nb == 4) go(tt_tag, std::integral_constant<int, 4>{});
        else if (nb == 2) go(tt_tag, std::integral_constant<int, 2>{});
        else go(tt_tag, std::integral_constant<int, 1>{});
    };
    if (tt == 3) with_rows(std::integral_constant<int, 3>{});
    else if (tt == 2) with_rows(std::integral_constant<int, 2>{});
    else with_rows(std::integral_constant<int, 1>{});
}

// V[token][0..rank) = the sum of the slices' sums, for the rows of all panels.  Bound by its two trips to memory (the panel, then the sums): 4 to 9 us
template <int N>
__global__ __launch_bounds__(256) void mfma_panel_sum_kernel(const DevItem *panels, PanelShape<N> sh, TileBatchArgs<N> tb)
{
    // a block per (panel, 32 rows, projection); a thread sums one float4 column of four rows
    constexpr int PER = PANEL_ROWS / 32;
    const int pj = (int)blockIdx.y, slices = sh.slices[pj];
    if (slices == 1) return;
    const int panel = blockIdx.x / PER, part = blockIdx.x - panel * PER;
    const DevItem it = panels[panel];
    const int t0 = part * 32 + (threadIdx.x >> 5), j4 = threadIdx.x & 31;
    if ((part * 32 >= it.n_tok) | (j4 * 4 >= rank_storage(it.rank))) return;
    const int pitch = tb.v_stride >> 2;
    const float4 *src = reinterpret_cast<const float4 *>(tb.part + (size_t)pj * tb.part_set) + (size_t)it.tok_off * pitch + j4;
    int ti[4], tok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ti[i] = t0 + 8 * i;
    tile_tokens_of(tb.tok_list, it, ti, it.tok0, tok);
    float4 sum[4];
    for (int s = 0; s < slices; ++s) {
        float4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = src[((size_t)s * tb.n_rows + min(ti[i], it.n_tok - 1)) * pitch];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s == 0) sum[i] = v[i];
            else sum[i].x += v[i].x, sum[i].y += v[i].y, sum[i].z += v[i].z, sum[i].w += v[i].w;
        }
    }
    const float s_v = tb.scale * it.alpha;
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    __bf16 *const out = reinterpret_cast<__bf16 *>(tb.v + (size_t)pj * tb.v_set);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (ti[i] >= it.n_tok) continue;
        bf16x4_t o;
        o[0] = (__bf16)(s_v * sum[i].x), o[1] = (__bf16)(s_v * sum[i].y), o[2] = (__bf16)(s_v * sum[i].z), o[3] = (__bf16)(s_v * sum[i].w);
        reinterpret_cast<bf16x4_t *>(out + (size_t)tok[i] * (2 * tb.v_stride))[j4] = o;
    }
}

// V[token][0..rank) = sum over the tile's pieces of their partial sums, for the tiles worked on in pieces.
// (Atomic adds into V instead cost about 30 us per launch: device-scope fp32 atomics execute at the memory side.)
template <int N>
__global__ __launch_bounds__(256) void mfma_reduce_kernel(TileBatchArgs<N> tb)
{
    // 8 blocks per tile (and projection of the batch: blockIdx.y), 8 tokens each; a thread sums one
    // float4 column of one token
    const int tile = blockIdx.x >> 3;
    const ShrinkSum sm = tb.sums[tile];
    const DevItem it = tb.tiles[tile];  // (requested together with sm: one trip to memory, not two)
    const int ti = (blockIdx.x & 7) * 8 + (threadIdx.x >> 5), j4 = threadIdx.x & 31;
    if ((sm.n_pieces < 2) | (ti >= it.n_tok) | (j4 * 4 >= rank_storage(it.rank))) return;  // entries past the rank are never used
    const ApplyArgs a = tile_args(tb, (int)blockIdx.y);
    const size_t slot_f4 = (size_t)SHRINK_SLOT_ROWS * (a.v_stride >> 2);
    const float4 *src = reinterpret_cast<const float4 *>(tb.part + (size_t)blockIdx.y * tb.part_set) + (size_t)ti * (a.v_stride >> 2) + j4;
    // four pieces at a time: their loads are issued together (one after the other, a tile in seven pieces took
    // seven trips to memory: 6.5 us per launch on the stress configuration), and only the loads that are needed (loads of a
    // padded batch cost the mixed configuration, two to three pieces per tile, 1 to 2 us)
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    auto piece = [&](int pc) __attribute__((always_inline)) {
        return src[(size_t)(pc == 0 ? sm.first_slot : 2 * ((sm.first_slot >> 1) + pc)) * slot_f4];
    };
    auto add = [&](const float4 &v) __attribute__((always_inline)) { sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w; };
    for (int p0 = 0; p0 < sm.n_pieces; p0 += 4) {
        const int n = sm.n_pieces - p0;  // the same for the whole block: the branches below are scalar
        if (n >= 4) {
            const float4 v0 = piece(p0), v1 = piece(p0 + 1), v2 = piece(p0 + 2), v3 = piece(p0 + 3);
            add(v0); add(v1); add(v2); add(v3);
        } else if (n == 3) {
            const float4 v0 = piece(p0), v1 = piece(p0 + 1), v2 = piece(p0 + 2);
            add(v0); add(v1); add(v2);
        } else if (n == 2) {
            const float4 v0 = piece(p0), v1 = piece(p0 + 1);
            add(v0); add(v1);
        } else {
            add(piece(p0));
        }
    }
    // the sum goes out as the expand takes it: scaled and rounded to bf16 (rows of the same pitch as the fp32 ones)
    const float s_v = a.scale * it.alpha;
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    bf16x4_t o;
    o[0] = (__bf16)(s_v * sum.x), o[1] = (__bf16)(s_v * sum.y), o[2] = (__bf16)(s_v * sum.z), o[3] = (__bf16)(s_v * sum.w);
    reinterpret_cast<bf16x4_t *>(reinterpret_cast<__bf16 *>(a.v) + (size_t)tile_token(a, it, ti) * (2 * a.v_stride))[j4] = o;
}

// ---------------------------------------------------------------------------------------
// expand.  Block = 4 wavefronts, tile of up to 64 tokens x (128 * n_pass) columns in passes of
// 128 columns (the launcher picks n_pass: longer column runs amortise the staging of V, shorter ones
// sweep base_out faster and keep the chip full when there are few tiles); wavefront w owns token half w&1 and column half w>>1 of a pass (32 tokens x 64
// columns).  The scaled V tile is staged once in LDS as bf16.  The product is formed
// transposed (rows = output columns, columns = tokens): MFMA row r of column block b is column
// 16b + r, so the 16 lanes of a Bp operand load read 256 contiguous bytes.
// The read-modify-write of base_out does not use the MFMA register layout (a lane would touch
// 16 bytes of each of many rows, and every 128-byte line would be fetched by two instructions,
// which stalls L1 on the second): the wavefront parks its fp32 products in LDS and goes over
// base_out with 8 lanes per token row, whole 128-byte lines per instruction, for the load (issued
// three passes ahead), the add and the store.
// A compute unit holds two blocks and asks for 8 wavefronts x three passes x 4 KB of base_out ahead of what it is adding to (one pass ahead, 32 KB, is less than
// the rate of the memory times its latency), and a wavefront asks for nothing past its run: its place on the unit is held until the last answer is there.
// Measured on the 7B mixed batch (one pass ahead and on past the run 2003 us): the requests past the run left out 1911, two passes ahead 1890, three 1866, four 1860;
// the prefill batch 234, 223, 221, 219; a prompt of 1200 tokens projection by projection 391 -> 365 (three blocks per unit there before).
// ---------------------------------------------------------------------------------------
namespace {
constexpr int CS_ROW = 64 * 4 + 16;  // bytes per token row of a wavefront's parked products (padded)
constexpr int AHEAD = 3;             // passes of base_out on their way (the loop below is written for it)
}

// KS: MFMA k steps of 32 ranks.  As in the shrink, global loads are unconditional from clamped
// addresses: rank chunks past the stored rank re-read the last stored chunk and meet zeros in V.
template <int KS>
__device__ __forceinline__ void mfma_expand_body(const ApplyArgs &a, const DevItem &it, int col_run, int n_pass, unsigned char *vs,
                                                 unsigned char (*cs)[32 * CS_ROW])
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int th = w & 1, ch = w >> 1;
    const int rs = rank_storage(it.rank), rs8 = rs >> 3;
    const __bf16 *Bp = reinterpret_cast<const __bf16 *>(a.proj_base + (int64_t)it.row * a.row_bytes) + (size_t)rs * a.h_in;
    __bf16 *y = static_cast<__bf16 *>(a.y);

    // read-modify-write layout: instruction i covers token rows 32*th + 8*i + lane/8, 8 columns at 8*(lane%8)
    const int rt = lane >> 3, rc = lane & 7;
    // the token ids of the rows this thread updates and of the rows of V it stages, looked up together and
    // before anything else is requested
    constexpr int c8 = KS * 4;  // staged chunks (8 ranks) per token
    static_assert(LORA_TILE_TOKENS * c8 == 256 * KS, "a thread stages KS pieces");
    int rows[4 + KS], toks[4 + KS];
#pragma unroll
    for (int i = 0; i < 4; ++i) rows[i] = 32 * th + 8 * i + rt;
#pragma unroll
    for (int i = 0; i < KS; ++i) rows[4 + i] = (tid + 256 * i) / c8;
    tile_tokens(a, it, rows, toks);
    size_t yoff[4];
    bool yok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        yok[i] = rows[i] < it.n_tok;
        yoff[i] = (size_t)toks[i] * a.h_out + rc * 8;
    }
    const bool half_live = 32 * th < it.n_tok;
    const int col0 = col_run * n_pass * 128 + 64 * ch;

    // base_out of pass `cp`.  Read once and written once, both as streaming accesses: the rows then leave the caches
    // as they are written instead of lying there dirty until the next kernel's loads push them out (measured on the
    // kernels that follow: the tile shrink of the next projection or layer 93 -> 79 us on the mixed configuration,
    // 19.9 -> 17.3 us on the prefill one, for 0.6 us more in this kernel; either hint alone changes nothing)
    auto load_y = [&](int cp, uint4(&d)[4]) {
        const int nw0 = min(col0 + cp * 128, a.h_out - 64);
        typedef unsigned u32x4_nt __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4_nt t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt *>(y + yoff[i] + nw0));
            d[i] = make_uint4(t[0], t[1], t[2], t[3]);
        }
    };
    // Bp operands of the pass starting at column nw0: block b = columns nw0 + 16b .. +15, k step ks
    const __bf16 *bg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bg[ks] = Bp + ((size_t)min(4 * ks + g, rs8 - 1) * a.h_out + m) * 8;
    auto load_b = [&](int nw0, uint4(&d)[KS][4]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < 4; ++b) d[ks][b] = *reinterpret_cast<const uint4 *>(bg[ks] + (size_t)(nw0 + 16 * b) * 8);
    };

    uint4 yr[AHEAD + 1][4];
    uint4 br[KS][4];
    // columns past h_out: this wavefront's share of the block ends
    const int my_pass = min(n_pass, (a.h_out - col0 + 127) / 128);

    // stage s.V (written as bf16 by the shrink or the reduce): vs[token][rank].  A thread's KS pieces (8 ranks of one
    // token each) are all requested before the first is used: taken one after the other, each with its own trip to
    // memory, the staging took 4.6 us (rank 16) to 8.2 us (rank 128) of a block's 17 to 21 us on the prefill
    // configuration.  V is requested first
    // and the first pass's base_out and Bp behind it (loads complete in the order of their requests): those are
    // on their way while V is staged.
    {
        const uint4 *vr[KS];
        bool ok[KS];
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const int idx = tid + 256 * i, ti = idx / c8, j8 = idx - ti * c8;
            ok[i] = ti < it.n_tok;
            vr[i] = reinterpret_cast<const uint4 *>(reinterpret_cast<const __bf16 *>(a.v) + (size_t)toks[4 + i] * (2 * a.v_stride) + j8 * 8);
        }
        uint4 pc[KS];
#pragma unroll
        for (int i = 0; i < KS; ++i) pc[i] = vr[i][0];
        __builtin_amdgcn_sched_barrier(0);  // keep the scheduler from trading loads in flight for registers
        load_y(0, yr[0]);
        load_b(min(col0, a.h_out - 64), br);
#pragma unroll
        for (int p = 1; p < AHEAD; ++p)
            if (p < my_pass) load_y(p, yr[p]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const int idx = tid + 256 * i, ti = idx / c8, j8 = idx - ti * c8;
            const bf16x8 f = __builtin_bit_cast(bf16x8, pc[i]);
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (ok[i] && j8 * 8 + e < it.rank) ? f[e] : (__bf16)0.f;  // entries past the rank were never written
            *reinterpret_cast<bf16x8 *>(&vs[ti * VS_ROW + j8 * 16]) = o;
        }
    }
    __syncthreads();

    if (!half_live) return;  // this token half is empty (no barrier follows)
    unsigned char *my_cs = cs[w];

    // one pass of 128 columns; AT = cp % (AHEAD + 1) is a compile-time constant so that the base_out buffers
    // stay in registers
    auto pass = [&](auto at_tag, int cp) {
        constexpr int AT = decltype(at_tag)::value;
        const int nw0 = col0 + cp * 128;
        if (cp + AHEAD < my_pass) load_y(cp + AHEAD, yr[(AT + AHEAD) % (AHEAD + 1)]);  // ahead of this pass's products

        floatx4 acc[4][2];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) acc[b][tb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const bf16x8 aop = __builtin_bit_cast(bf16x8, br[ks][b]);
                const bf16x8 b0 = *reinterpret_cast<const bf16x8 *>(&vs[(32 * th + m) * VS_ROW + (4 * ks + g) * 16]);
                const bf16x8 b1 = *reinterpret_cast<const bf16x8 *>(&vs[(32 * th + 16 + m) * VS_ROW + (4 * ks + g) * 16]);
                acc[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, b0, acc[b][0], 0, 0, 0);
                acc[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, b1, acc[b][1], 0, 0, 0);
            }
        if (cp + 1 < my_pass) load_b(min(nw0 + 128, a.h_out - 64), br);  // next pass's Bp, into the registers just used

        // park the products: lane (g, m) holds, for block b and token block tb, columns 16b + 4g .. +3 of token 16tb + m
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
                *reinterpret_cast<floatx4 *>(&my_cs[(16 * tb + m) * CS_ROW + (16 * b + 4 * g) * 4]) = acc[b][tb];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a wavefront's LDS operations execute in order
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 p0 = *reinterpret_cast<const float4 *>(&my_cs[(8 * i + rt) * CS_ROW + rc * 32]);
            const float4 p1 = *reinterpret_cast<const float4 *>(&my_cs[(8 * i + rt) * CS_ROW + rc * 32 + 16]);
            float f[8];
            Chunk<__bf16> c;
            c.v = yr[AT][i];
            unpack_chunk(c, f);
            bf16x8 o;
            o[0] = (__bf16)(f[0] + p0.x); o[1] = (__bf16)(f[1] + p0.y); o[2] = (__bf16)(f[2] + p0.z); o[3] = (__bf16)(f[3] + p0.w);
            o[4] = (__bf16)(f[4] + p1.x); o[5] = (__bf16)(f[5] + p1.y); o[6] = (__bf16)(f[6] + p1.z); o[7] = (__bf16)(f[7] + p1.w);
            if (yok[i]) __builtin_nontemporal_store(o, reinterpret_cast<bf16x8 *>(y + yoff[i] + nw0));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();  // the next pass overwrites the parked products
    };
    for (int cp = 0;; cp += AHEAD + 1) {
        if (cp >= my_pass) break;
        pass(std::integral_constant<int, 0>{}, cp);
        if (cp + 1 >= my_pass) break;
        pass(std::integral_constant<int, 1>{}, cp + 1);
        if (cp + 2 >= my_pass) break;
        pass(std::integral_constant<int, 2>{}, cp + 2);
        if (cp + 3 >= my_pass) break;
        pass(std::integral_constant<int, 3>{}, cp + 3);
    }
}

// Blocks -> (projection, tile, column run).  What the launch is bound by is base_out, read and written, and the rate of that
// depends on the order: with the column runs as the fast index the blocks in flight cover whole rows of a few tiles
// (a read-modify-write of this shape alone: 5.6 TB/s in runs of 1024 columns, 6.2 in runs of 256), with the tiles as the fast
// index a column window of many (4.2 TB/s).  A tile's runs are numbered up to the next multiple of 8, so that a run -- the
// same columns of every tile -- always falls on the same XCD (block b runs on XCD b % 8) and a prompt's Bp is fetched from memory by one
// XCD per column run instead of by all eight; the blocks past the last run return at once.
template <int N> struct ExpandShape {
    int32_t blk_end[N];  // blocks of projections 0 .. p (entries past the batch repeat the last)
    int32_t runs[N];     // per projection: passes of 128 columns per run | blocks per tile (a multiple of 8) << 8
};
template <int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void mfma_expand_kernel(TileBatchArgs<N> tb, ExpandShape<N> sh)
{
    __shared__ __attribute__((aligned(16))) unsigned char vs[LORA_TILE_TOKENS * VS_ROW];
    __shared__ __attribute__((aligned(16))) unsigned char cs[4][32 * CS_ROW];
    int pj = 0;  // the first projection whose blocks end behind this one
    if (tb.n > 1) {
#pragma unroll
        for (int step = N / 2; step > 0; step >>= 1)
            if ((int)blockIdx.x >= sh.blk_end[pj + step - 1]) pj += step;
    }
    const int b = (int)blockIdx.x - (pj ? sh.blk_end[pj - 1] : 0);
    const ApplyArgs a = tile_args(tb, pj);
    const int n_pass = sh.runs[pj] & 0xff, width = sh.runs[pj] >> 8;
    const int tile = b / width, col_run = b - tile * width;
    if (col_run * n_pass * 128 >= a.h_out) return;  // padding
    const DevItem it = tb.tiles[tile];
    switch ((it.rank + 31) >> 5) {
    case 1: mfma_expand_body<1>(a, it, col_run, n_pass, vs, cs); break;
    case 2: mfma_expand_body<2>(a, it, col_run, n_pass, vs, cs); break;
    case 3: mfma_expand_body<3>(a, it, col_run, n_pass, vs, cs); break;
    default: mfma_expand_body<4>(a, it, col_run, n_pass, vs, cs); break;
    }
}

// The arguments of a batch are 2.4 KB; a group's calls, one after the other as a model's forward pass makes them, take them
// along as 0.25 KB instead (a short prompt called projection by projection: 288 us with the large ones, 282 us).
template <typename F> static void with_batch_size(const TileBatch &tb, F go)
{
    if (tb.n > GROUP_MAX_PROJS) {
        go(static_cast<const TileBatchArgs<BATCH_MAX_PROJS> &>(tb));
        return;
    }
    TileBatchArgs<GROUP_MAX_PROJS> g;
    static_cast<TileBatchHead &>(g) = tb;
    for (int i = 0; i < GROUP_MAX_PROJS; ++i) {
        g.group[i] = 0;  // (one group)
        g.p[i] = tb.p[std::min(i, tb.n - 1)];
    }
    go(g);
}

static ListCopy copy_behind(ListCopy c, unsigned blocks)
{
    c.first_block = blocks;
    return c;
}
template <int W> constexpr int direct_lds = W *DRING *DSTAGE;
constexpr int SHRINK_LDS = NSTAGE * LORA_TILE_TOKENS * XROW;

// A kernel's limit of LDS belongs to the device that is current when it is set
template <int N> static hipError_t prepare_shrinks()
{
    hipError_t e = allow_lds(mfma_shrink_direct_kernel<N, 4>, direct_lds<4>);
    if (e == hipSuccess) e = allow_lds(mfma_shrink_direct_kernel<N, 8>, direct_lds<8>);
    if (e == hipSuccess) e = allow_lds(mfma_shrink_direct_kernel<N, 4, ListCopy>, direct_lds<4>);
    if (e == hipSuccess) e = allow_lds(mfma_shrink_direct_kernel<N, 8, ListCopy>, direct_lds<8>);
    if (e == hipSuccess) e = allow_lds(mfma_panel_kernel<N>, PANEL_RING);
    if (e == hipSuccess) e = allow_lds(mfma_panel_kernel<N, ListCopy>, PANEL_RING);
    if (e == hipSuccess) e = allow_lds(mfma_shrink_kernel<N>, SHRINK_LDS);
    if (e == hipSuccess) e = allow_lds(mfma_shrink_kernel<N, ListCopy>, SHRINK_LDS);
    return e;
}
hipError_t prepare_mfma_kernels()
{
    const hipError_t e = prepare_shrinks<GROUP_MAX_PROJS>();
    return e == hipSuccess ? prepare_shrinks<BATCH_MAX_PROJS>() : e;
}

// k ranges are multiples of the 128-element stage.
hipError_t launch_mfma_shrink(const TileBatch &batch, const ListCopy &copy, hipStream_t st, const KernelTimer *tm)
{
    if (batch.n_tiles <= 0 || batch.n <= 0) return hipSuccess;
    if (batch.n > BATCH_MAX_PROJS) return hipErrorInvalidValue;
    if (batch.n_direct > 0) {
        with_batch_size(batch, [&](const auto &tb) {
            constexpr int N = sizeof(tb.p) / sizeof(tb.p[0]);
            auto go = [&](auto w_tag) {
                constexpr int W = decltype(w_tag)::value;
                const unsigned blocks = (unsigned)(tb.n_direct * tb.n);
                if (copy.pieces) {
                    auto first = tb;  // (this launch reads the lists where the host wrote them)
                    first.direct = where_written(copy, tb.direct), first.tok_list = where_written(copy, tb.tok_list);
                    launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_shrink_direct_kernel<N, W, ListCopy>, dim3(blocks + copy_blocks(copy, 64 * W)), dim3(64 * W), direct_lds<W>, st, first,
                             copy_behind(copy, blocks));
                } else {
                    launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_shrink_direct_kernel<N, W>, dim3(blocks), dim3(64 * W), direct_lds<W>, st, tb);
                }
            };
            if (tb.n_direct * tb.n <= 256) go(std::integral_constant<int, 8>{});  // (a block to a compute unit)
            else go(std::integral_constant<int, 4>{});
        });
        return hipGetLastError();
    }
    if (batch.n_panels > 0) {
        with_batch_size(batch, [&](const auto &tb) {
            constexpr int N = sizeof(tb.p) / sizeof(tb.p[0]);
            PanelShape<N> sh;
            int end = 0, groups = 0;
            bool sums = false;
            for (int i = 0; i < tb.n; ++groups) {
                const int gn = (int)(batch.group[i] >> 8);
                sh.group[groups] = (uint32_t)i | (uint32_t)gn << 8 | (uint32_t)batch.slices[i] << 16;
                sh.end[groups] = end += panel_blocks(batch.classes, gn) * batch.slices[i];
                for (int k = 0; k < gn; ++k, ++i) sh.slices[i] = batch.slices[i];
                sums |= sh.slices[i - 1] > 1;
            }
            for (int g = groups; g < N; ++g) sh.end[g] = end, sh.group[g] = sh.group[groups - 1];
            for (int i = tb.n; i < N; ++i) sh.slices[i] = 1;
            if (copy.pieces) {
                auto first = tb;
                first.panels = where_written(copy, tb.panels), first.tok_list = where_written(copy, tb.tok_list);
                launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_panel_kernel<N, ListCopy>, dim3(end + copy_blocks(copy, 512)), dim3(512), PANEL_RING, st, first.panels, batch.classes, sh, first,
                         copy_behind(copy, (unsigned)end));
            } else {
                launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_panel_kernel<N>, dim3(end), dim3(512), PANEL_RING, st, tb.panels, batch.classes, sh, tb);
            }
            if (sums) launch_k(tm, nullptr, LORA_K_MFMA_REDUCE, mfma_panel_sum_kernel<N>, dim3(tb.n_panels * (PANEL_ROWS / 32), tb.n), dim3(256), 0, st, tb.panels, sh, tb);
        });
        return hipGetLastError();
    }
    if (batch.n_runs <= 0) return hipSuccess;
    if (batch.n_runs % 8 != 0 || batch.quanta < 1) return hipErrorInvalidValue;
    with_batch_size(batch, [&](const auto &tb) {
        constexpr int N = sizeof(tb.p) / sizeof(tb.p[0]);
        if (copy.pieces) {
            auto first = tb;
            first.cuts = where_written(copy, tb.cuts), first.tiles = where_written(copy, tb.tiles), first.tok_list = where_written(copy, tb.tok_list);
            launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_shrink_kernel<N, ListCopy>, dim3(tb.n_runs * tb.n + copy_blocks(copy, 256)), dim3(256), SHRINK_LDS, st, first.cuts, first.tiles, tb.n_runs / 8,
                     tb.n, tb.quanta, tb.n_tiles, first, copy_behind(copy, (unsigned)(tb.n_runs * tb.n)));
        } else {
            launch_k(tm, nullptr, LORA_K_MFMA_SHRINK, mfma_shrink_kernel<N>, dim3(tb.n_runs * tb.n), dim3(256), SHRINK_LDS, st, tb.cuts, tb.tiles, tb.n_runs / 8, tb.n, tb.quanta, tb.n_tiles, tb);
        }
        if (tb.any_pieces) launch_k(tm, nullptr, LORA_K_MFMA_REDUCE, mfma_reduce_kernel<N>, dim3(tb.n_tiles * 8, tb.n), dim3(256), 0, st, tb);
    });
    return hipGetLastError();
}

// Longest column run, in passes (7B mixed batch 1898 us with 4, 1866 with 8, 1887 with 16).
constexpr int EXPAND_PASSES = 8;
hipError_t launch_mfma_expand(const TileBatch &batch, hipStream_t st, const KernelTimer *tm, hipEvent_t done)
{
    if (batch.n_tiles <= 0 || batch.n <= 0) return hipSuccess;
    if (batch.n > BATCH_MAX_PROJS) return hipErrorInvalidValue;
    // blocks per tile: the multiple of 8 that keeps a run within the limit; shorter runs (at least two passes) where that leaves the launch below 512 blocks (two per CU)
    int32_t shape[BATCH_MAX_PROJS];
    int64_t total = 0;
    for (int passes = EXPAND_PASSES;; passes >>= 1) {
        int64_t live = 0;
        total = 0;
        for (int i = 0; i < batch.n; ++i) {
            const int all = (batch.p[i].h_out + 127) / 128, width = (all + 8 * passes - 1) / (8 * passes) * 8;  // blocks per tile
            const int n_pass = std::max(std::min(2, all), (all + width - 1) / width);
            const int used = (all + n_pass - 1) / n_pass, padded = (used + 7) / 8 * 8;
            shape[i] = n_pass | padded << 8;
            live += (int64_t)batch.n_tiles * used;
            total += (int64_t)batch.n_tiles * padded;
        }
        if (live >= 512 || passes <= 2) break;
    }
    if (total > INT32_MAX) return hipErrorInvalidValue;
    with_batch_size(batch, [&](const auto &tb) {
        constexpr int N = sizeof(tb.p) / sizeof(tb.p[0]);
        ExpandShape<N> sh;
        int32_t end = 0;
        for (int i = 0; i < N; ++i) {
            if (i < tb.n) end += tb.n_tiles * (shape[i] >> 8);
            sh.blk_end[i] = end;
            sh.runs[i] = i < tb.n ? shape[i] : 0;
        }
        launch_k(tm, done, LORA_K_MFMA_EXPAND, mfma_expand_kernel<N>, dim3((unsigned)end), dim3(256), 0, st, tb, sh);
    });
    return hipGetLastError();
}

}  // namespace lora
