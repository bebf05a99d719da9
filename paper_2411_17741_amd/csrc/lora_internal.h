// Internal declarations shared by the host side and the gfx950 kernels of liblora_cache.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "lora_cache.h"

namespace lora {

// Pool layout.  Every slot owns `rs_class` consecutive *storage rows* (rs = rank rounded up
// to a multiple of 8); a slot's first row is the same number in every projection, so a slab
// is found without a table:
//     slab(layer, proj, slot) = pool + layer*layer_stride + proj_off[proj] + row(slot) * row_bytes(proj)
//     row_bytes(proj) = (h_in + h_out) * element size
// Inside a slab of an adapter of rank r (rs = rank_storage(r)):
//   At [rs][h_in]          rank-major: row j holds column j of A, contiguous along h_in
//   Bp [rs/8][h_out][8]    rank-packed: the 8 ranks of a granule are contiguous per output column
// Rows r..rs-1 are zero.  Only rs*(h_in+h_out) elements are ever read, whatever the slot's class.
inline __host__ __device__ int32_t rank_storage(int32_t r) { return (r + 7) & ~7; }

// Work item as the kernels read it (the public lora_item_t with the slot resolved).
struct DevItem {
    int32_t tok_off, n_tok;  // tokens: tok_list[tok_off .. tok_off+n_tok)
    int32_t row;             // first storage row of the slot
    int32_t rank;
    int32_t a;               // as in lora_item_t
    int32_t consecutive;     // 1: the tokens are tok0, tok0+1, ... (a prompt's tile): no lookup in tok_list at all
    float alpha;             // the cache entry's own factor
    int32_t tok0;            // tok_list[tok_off], so one-token items need no second lookup
};
static_assert(sizeof(DevItem) == sizeof(lora_item_t), "device items are uploaded in place of lora_item_t");
// token id of row ti (0 <= ti < n_tok) of a tile (tile kernels and lora_plan_dump alike)
inline __host__ __device__ int32_t tile_token_of(const int32_t *tok_list, const DevItem &it, int32_t ti)
{
    return (it.consecutive || ti == 0) ? it.tok0 + ti : tok_list[it.tok_off + ti];
}

// Token ids of N rows of a tile in one round of lookups (none for a tile of consecutive tokens).  Rows past the
// tile's last count as its last, the rows of an empty tile as token `dead`.  (A conditional lookup per row is a
// branch per row in a kernel, and after each the compiler waits for every load and store still outstanding.)
template <int N, typename Item>
inline __host__ __device__ void tile_tokens_of(const int32_t *tok_list, const Item &it, const int (&ti)[N], int32_t dead,
                                               int (&tok)[N])
{
    if (it.n_tok <= 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) tok[i] = dead;
    } else if (it.consecutive) {
#pragma unroll
        for (int i = 0; i < N; ++i) tok[i] = it.tok0 + (ti[i] < it.n_tok ? ti[i] : it.n_tok - 1);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) tok[i] = tok_list[it.tok_off + (ti[i] < it.n_tok ? ti[i] : it.n_tok - 1)];
    }
}

// The rows of lora_linear_plan: every token of the batch in one list without gaps -- the tokens of the tiles, tile by tile, then
// those of the GEMV groups, then those without an adapter -- cut into runs of LORA_TILE_TOKENS rows.  (Tiles padded to 64 rows of
// their own made 2944 rows of a 13B layer's 2560 tokens, 12 row panels of 256 instead of 10.)  Rows of one slot
// that follow each other are a segment, whichever run they fall into.
struct LinearRows {
    int32_t tok_off, n_tok;      // rows tok_off .. tok_off + n_tok of the list
    int32_t consecutive, tok0;   // as in DevItem
    int32_t first_seg, n_segs;   // the segments with rows among them
    int32_t pad[2];
};
static_assert(sizeof(LinearRows) == 32, "read with one 32-byte scalar load");
struct LinearSeg {
    int32_t r0, r1;  // rows [r0, r1)
    int32_t row;     // first storage row of the slot
    int32_t rank;
};

// GEMV work item: a batch of up to GEMV_BATCH tokens of one slot, named directly so that the kernels
// reach their data with one lookup.  A shrink item stands for GEMV_SHRINK_ROWS stored rank rows from
// `a` on (stored rows past the rank hold zeros, so an item is always whole); an expand item for one
// run of gemv_expand_width(rank) columns in every super-chunk of the projection, `a` being the
// run's offset inside the super-chunk in units of 64 columns.  Items name no projection: a launch
// runs them for every projection of its group.  Kernels and lora_plan_dump read `a` through the
// routines below.
constexpr int GEMV_BATCH = 4;              // tokens one GEMV work item handles
constexpr int GEMV_SHRINK_ROWS = 4;        // rank rows of a shrink item
constexpr int GEMV_SUPER_COLS = 1024;      // an expand item stands for one run of columns in every super-chunk of this width
struct GemvItem {
    int32_t tok[GEMV_BATCH];  // token ids, -1 = unused; used ones come first
    int32_t row;              // first storage row of the slot
    int32_t rank;
    int32_t a;
    float alpha;              // the cache entry's own factor
};
static_assert(sizeof(GemvItem) == 32, "items are read with one 32-byte scalar load");

// columns one expand wavefront covers: 64 times the largest power of two that keeps it within 16 KB of Bp
inline __host__ __device__ int32_t gemv_expand_width(int32_t rank)
{
    const int32_t q = 128 / rank_storage(rank);
    return q >= 16 ? 1024 : q >= 8 ? 512 : q >= 4 ? 256 : q >= 2 ? 128 : 64;
}
inline __host__ __device__ int32_t gemv_pack_shrink(int32_t j0) { return j0; }
inline __host__ __device__ int32_t gemv_pack_expand(int32_t col_in_super) { return col_in_super / 64; }
// stored rank rows [j0, j0 + n) of a shrink item
inline __host__ __device__ void gemv_shrink_rows(const GemvItem &it, int32_t &j0, int32_t &n)
{
    j0 = it.a;
    n = GEMV_SHRINK_ROWS;
}
// `width` output columns [c0, c1) from a * 64 on in super-chunk `sc` of a projection h_out wide (empty if c0 >= c1)
inline __host__ __device__ void gemv_cols(int32_t width, int32_t a, int32_t sc, int32_t h_out, int32_t &c0, int32_t &c1)
{
    c0 = sc * GEMV_SUPER_COLS + a * 64;
    const int32_t end = c0 + width, super_end = (sc + 1) * GEMV_SUPER_COLS;
    c1 = end < super_end ? end : super_end;
    if (c1 > h_out) c1 = h_out;
}
inline __host__ __device__ void gemv_expand_cols(const GemvItem &it, int32_t sc, int32_t h_out, int32_t &c0, int32_t &c1)
{
    gemv_cols(gemv_expand_width(it.rank), it.a, sc, h_out, c0, c1);
}

// A plan's work lists on their way from pinned host memory to the pool, by blocks behind those of the plan's first launch, which itself reads them where the host wrote them: no launch of their own
struct ListCopy {
    void *to;          // device
    const void *from;  // pinned host memory as the device sees it
    uint32_t pieces;   // of 16 bytes; 0: nothing to copy
    uint32_t first_block;
};
inline uint32_t copy_blocks(const ListCopy &c, uint32_t threads) { return (c.pieces + threads - 1) / threads; }
// a pointer into the lists in the pool as one to the same place where the host wrote them
template <typename T> inline const T *where_written(const ListCopy &c, const T *p) { return reinterpret_cast<const T *>(static_cast<const char *>(c.from) + (reinterpret_cast<const char *>(p) - static_cast<const char *>(c.to))); }

// A batch: the projections one launch serves.  They do not depend on each other (no output overlaps another entry's
// output or any entry's input), so that every phase is one launch for all of them.
constexpr int BATCH_MAX_PROJS = 64;        // of a batch with tiles
constexpr int GEMV_BATCH_MAX_PROJS = 120;  // of a batch with GEMV work alone
struct BatchProj {
    const char *proj_base;    // device: first slab of this (layer, projection)
    const void *x;            // device [T][h_in]
    void *y;                  // device [T][h_out], in/out
    int32_t h_in, h_out;
};

// One GEMV launch serves up to GEMV_MAX_PROJS projections that read the same activations (q, k, v;
// gate, up): block and unit numbers map to (projection, item) by the two routines below, which the
// kernels and lora_plan_dump share.  (A batch of several such groups: GemvBatch further down.)
constexpr int GEMV_MAX_PROJS = 4;
struct GemvProj {
    const char *proj_base;    // device: first slab of this (layer, projection)
    int64_t row_bytes;        // (h_in + h_out) * element size
    void *y;                  // device [T][h_out], in/out
    float *y32;               // when set, the update s.v.B goes there as fp32 ([token][h_out]) instead of into y
    unsigned long long *vw;   // hand-over words of this projection's intermediate (see gemv_kernels.hip)
    int32_t h_out;
    int32_t pad;
};
// What a wavefront needs to find its work item, apart from the rest: the kernels take it as leading
// scalar arguments, which the hardware hands over in registers at wavefront start (no load to wait for
// before the item's own load can go out).
struct GemvMap {
    const GemvItem *gs, *ge;  // device: shrink and expand items
    uint32_t n_gs;
    uint32_t n_proj_phase;    // n_proj | phase << 8; phase 0: shrink blocks then expand blocks in one launch; 1: shrink only; 2: expand only
    int32_t unit_end[GEMV_MAX_PROJS];      // expand units of projections 0 .. p (entries past the group repeat the last)
    uint32_t n_super_packed;               // super-chunks of projection p, ceil(h_out / GEMV_SUPER_COLS) (< 256), in byte p
    uint32_t super_magic[GEMV_MAX_PROJS];  // ceil(2^32 / n_super) (unused when n_super == 1)
};
struct GemvArgs {
    const void *x;            // device [T][h_in]
    int32_t *fault;           // raised when a bounded wait gives up
    int32_t h_in, n_ge;
    uint32_t epoch;           // one launch: the number its hand-over words carry (never 0); 0: two launches, no waiting
    float scale;
    GemvProj p[GEMV_MAX_PROJS];
};
// floor(v / n) for v < 2^24 and n <= 255 with magic = ceil(2^32 / n), n > 1
inline __host__ __device__ uint32_t gemv_div(uint32_t v, uint32_t n, uint32_t magic)
{
    return n == 1 ? v : (uint32_t)(((uint64_t)v * magic) >> 32);
}
inline uint32_t gemv_magic(uint32_t n) { return n > 1 ? (uint32_t)((((uint64_t)1 << 32) + n - 1) / n) : 0; }
// one of four values by an index 0..3 (as selects: an array indexed by a run-time number would live in scratch memory on the device)
template <typename T> inline __host__ __device__ T gemv_sel4(uint32_t i, T v0, T v1, T v2, T v3)
{
    return i == 0 ? v0 : (i == 1 ? v1 : (i == 2 ? v2 : v3));
}
// Shrink block b of a launch with n_proj * n_gs shrink blocks -> (item, projection).  Block b runs on
// XCD b % 8, each XCD behind its own L2: XCD j takes a run of consecutive (item, projection) pairs,
// items in list order with their projections side by side, the i-th pair of the run as block 8i + j --
// the items of a token batch and all their projections read the batch's x rows, which are then
// fetched from memory by one XCD instead of eight.
inline __host__ __device__ void gemv_shrink_block(uint32_t b, uint32_t n_gs, uint32_t n_proj, uint32_t &item, uint32_t &proj)
{
    const uint32_t nb = n_gs * n_proj, j = b & 7;
    const uint32_t pos = j * (nb >> 3) + (j < (nb & 7) ? j : (nb & 7)) + (b >> 3);
    item = n_proj == 1 ? pos : (n_proj == 2 ? pos >> 1 : (n_proj == 4 ? pos >> 2 : gemv_div(pos, 3u, 0x55555556u)));
    proj = pos - item * n_proj;
}
// Expand unit u (over all projections of the launch) -> (projection, item, super-chunk)
inline __host__ __device__ void gemv_expand_unit(uint32_t u, const GemvMap &m, uint32_t &proj, uint32_t &item, uint32_t &sc)
{
    proj = (u >= (uint32_t)m.unit_end[0]) + (u >= (uint32_t)m.unit_end[1]) + (u >= (uint32_t)m.unit_end[2]);  // < n_proj for u < unit_end[n_proj - 1]
    const uint32_t r = u - gemv_sel4<uint32_t>(proj, 0u, (uint32_t)m.unit_end[0], (uint32_t)m.unit_end[1], (uint32_t)m.unit_end[2]);
    const uint32_t n_super = (m.n_super_packed >> (8 * proj)) & 0xffu;
    item = gemv_div(r, n_super, gemv_sel4(proj, m.super_magic[0], m.super_magic[1], m.super_magic[2], m.super_magic[3]));
    sc = r - item * n_super;
}

// floor(v / n) for v < 2^24 and 1 <= n < 2^24 as (v * mul) >> shift.  With shift = 24 + ceil(log2 n) and
// mul = ceil(2^shift / n) = (2^shift + e) / n, e < n, the product is v / n + v * e / (n * 2^shift), and v * e < 2^shift: less than 1 / n too much
struct Div24 {
    uint32_t mul, shift;
};
inline Div24 div24_of(uint32_t n)
{
    uint32_t l = 0;
    while ((1u << l) < n) ++l;
    return Div24{(uint32_t)((((uint64_t)1 << (24 + l)) + n - 1) / n), 24 + l};
}
inline __host__ __device__ uint32_t div24(uint32_t v, Div24 d) { return (uint32_t)(((uint64_t)v * d.mul) >> d.shift); }

// The GEMV launch of a batch (several groups of projections, each with its own x).  Blocks
// [0, n_proj * shrink_blocks) are the shrink blocks, projection by projection; expand units go super-chunk by
// super-chunk of all projections, items innermost.
constexpr int GEMV_BATCH_MAX_SUPERS = 768;
struct GemvBatchMap {
    uint32_t n_gs, n_ge, n_proj, n_units;  // n_units = n_ge * super-chunks of all projections
    uint32_t shrink_blocks;                // per projection: n_gs, or (by_xcd) n_gs rounded up to a multiple of 8
    uint32_t by_xcd, phase;                // phase as in GemvMap::n_proj_phase
    Div24 div_shrink, div_ge;              // by shrink_blocks, by n_ge
};
// From this many shrink items up XCD j (blocks j, j + 8, ...) takes a run of a projection's items: the items of a token
// batch read the same x rows.  Fewer items are dealt out one by one, or some XCDs would have none.
constexpr uint32_t GEMV_BATCH_XCD_ITEMS = 64;
// shrink block b -> (projection, item); item >= n_gs: nothing to do
inline __host__ __device__ void gemv_batch_shrink(uint32_t b, const GemvBatchMap &m, uint32_t &proj, uint32_t &item)
{
    proj = div24(b, m.div_shrink);
    const uint32_t r = b - proj * m.shrink_blocks;
    item = m.by_xcd ? (r & 7) * (m.shrink_blocks >> 3) + (r >> 3) : r;
}
// expand unit u -> (number of the super-chunk, item)
inline __host__ __device__ void gemv_batch_unit(uint32_t u, const GemvBatchMap &m, uint32_t &super, uint32_t &item)
{
    super = div24(u, m.div_ge);
    item = u - super * m.n_ge;
}
// super-chunk number -> its projection (four to a word)
inline __host__ __device__ uint32_t gemv_super(const uint32_t *supers, uint32_t super) { return (supers[super >> 2] >> (8 * (super & 3))) & 0xffu; }
// A projection of the launch in 24 bytes, so that the arguments (4 KB at most) hold one request's projections of 17 layers of a 7B model in one launch: three addresses
// (48 bits) and, in the 16 bits above each, a third of h_in / 64 (22 bits) | h_out / 64 (12 bits) | number of its first super-chunk (14 bits).
struct GemvEntry {
    uint64_t w[3];  // x, y, proj_base
};
inline GemvEntry gemv_entry(const BatchProj &p, uint32_t first_super)
{
    const uint64_t f = (uint64_t)(p.h_in / 64) | (uint64_t)(p.h_out / 64) << 22 | (uint64_t)first_super << 34, low = ((uint64_t)1 << 48) - 1;
    const uint64_t a[3] = {reinterpret_cast<uint64_t>(p.x), reinterpret_cast<uint64_t>(p.y), reinterpret_cast<uint64_t>(p.proj_base)};
    GemvEntry e;
    for (int i = 0; i < 3; ++i) e.w[i] = (a[i] & low) | (f >> 16 * i & 0xffff) << 48;
    return e;
}
// an address as a pointer to global memory (from a bare integer the compiler makes one to any memory: flat loads, +1 % on decode launches)
inline __host__ __device__ char *global_pointer(uint64_t address)
{
#ifdef __HIP_DEVICE_COMPILE__
    return (char *)(__attribute__((address_space(1))) char *)address;
#else
    return reinterpret_cast<char *>(address);
#endif
}
inline __host__ __device__ BatchProj gemv_entry_proj(const GemvEntry &e, uint32_t &first_super)
{
    const uint64_t low = ((uint64_t)1 << 48) - 1, f = e.w[0] >> 48 | (e.w[1] >> 48) << 16 | (e.w[2] >> 48) << 32;
    BatchProj p;
    p.x = global_pointer(e.w[0] & low);
    p.y = global_pointer(e.w[1] & low);
    p.proj_base = global_pointer(e.w[2] & low);
    p.h_in = (int32_t)(f & 0x3fffff) * 64;
    p.h_out = (int32_t)(f >> 22 & 0xfff) * 64;
    first_super = (uint32_t)(f >> 34);
    return p;
}
// Wide work items, for launches that fill the chip with them (bf16): a shrink item is up to GEMV_WIDE_ROWS stored rank rows
// (8 or 16) and GEMV_WIDE_SHRINK_TOKENS tokens, an expand item the columns of a GemvItem and GEMV_WIDE_TOKENS tokens.  What bounds such
// a launch is what the compute units take in (6 to 8 TB/s over all of them): per slab row the items of 4 rows and 4 tokens
// take in the activations of their tokens once per 4 rows, and a slab once per 4 tokens.
constexpr int GEMV_WIDE_ROWS = 16, GEMV_WIDE_SHRINK_TOKENS = 8, GEMV_WIDE_TOKENS = 16;
struct GemvWideItem {
    int32_t row, rank, a;  // as in GemvItem
    float alpha;
    int32_t n_tok, pad[3];
    int32_t tok[GEMV_WIDE_TOKENS];  // entries from n_tok on repeat the first
};
static_assert(sizeof(GemvWideItem) == 96, "items are read in 16-byte pieces");
// stored rank rows of a wide shrink item
inline __host__ __device__ int32_t gemv_wide_rows(int32_t rank, int32_t j0) { return rank_storage(rank) - j0 >= GEMV_WIDE_ROWS ? GEMV_WIDE_ROWS : 8; }
// columns of a wide expand item: those of a GemvItem, half of them up to rank 32 (8 KB of Bp: with 16 KB and the base_out rows
// of 16 products a lane would need more than the 128 registers that four wavefronts per SIMD leave it)
inline __host__ __device__ int32_t gemv_wide_width(int32_t rank) { return rank <= 32 ? gemv_expand_width(rank) / 2 : gemv_expand_width(rank); }
inline __host__ __device__ void gemv_wide_cols(int32_t rank, int32_t a, int32_t sc, int32_t h_out, int32_t &c0, int32_t &c1)
{
    gemv_cols(gemv_wide_width(rank), a, sc, h_out, c0, c1);
}
struct GemvBatch {
    const GemvItem *gs, *ge;  // device: shrink and expand items
    const GemvWideItem *wgs, *wge;  // the same as wide items: what gemv_wide_kernel reads, with m for their numbers
    float *y32;               // as GemvProj::y32 (a batch of one, wide)
    unsigned long long *vw;   // hand-over words of projection 0; those of projection p lie vw_set words behind those of p - 1
    uint64_t vw_set;
    int32_t *fault;
    uint32_t epoch;           // as in GemvArgs
    float scale;
    GemvBatchMap m;
    uint32_t supers[GEMV_BATCH_MAX_SUPERS / 4];  // per super-chunk its projection
    GemvEntry p[GEMV_BATCH_MAX_PROJS];
};
static_assert(sizeof(GemvBatch) <= 3900, "kernel arguments are at most 4 KB");
inline __host__ __device__ BatchProj gemv_batch_proj(const GemvBatch &b, uint32_t proj, uint32_t &first_super) { return gemv_entry_proj(b.p[proj], first_super); }
inline __host__ __device__ uint32_t gemv_batch_super(const GemvBatch &b, uint32_t super) { return gemv_super(b.supers, super); }

// A batch of more projections or super-chunks than that, up to all projections of 32 layers of a 7B model: a projection in 16 bytes, which name its layer and which of up to
// GEMV_LONG_KINDS (pool offset, widths) it has; its super-chunks are found from the projection of every 16th by steps of a
// projection each (a few, where outputs are 4096 wide).  What it saves is a launch of 5 to 6 us: 224 projections of a 7B model, one request of rank 16 27.2 -> 21.8 us, of rank 64 59.1 -> 52.7,
// 64 requests 362 -> 352; 196 of a 13B model, eight of rank 32 87 -> 77; 1024 wide, one of rank 16 22.4 -> 19.6.
constexpr int GEMV_LONG_MAX_PROJS = 224, GEMV_LONG_MAX_SUPERS = 1536, GEMV_LONG_KINDS = 8, GEMV_LONG_STEP = 16;
struct GemvLongEntry {
    uint64_t w[2];  // x / 16, y / 16 (44 bits each) and above them 20 bits of: kind (3 bits) | layer (21 bits) | number of its first super-chunk (16 bits)
};
struct GemvLong {
    const void *shrink_items, *expand_items;  // device: GemvItem or GemvWideItem
    unsigned long long *vw;                   // as in GemvBatch, as far as `scale`
    uint64_t vw_set;
    int32_t *fault;
    uint32_t epoch;
    float scale;
    char *pool;
    uint64_t layer_stride;
    uint64_t off_h_out[GEMV_LONG_KINDS];  // of layer 0's first slab (48 bits) | h_out / 64
    int32_t h_in[GEMV_LONG_KINDS];
    GemvBatchMap m;
    uint32_t marks[GEMV_LONG_MAX_SUPERS / GEMV_LONG_STEP / 4];  // projections of super-chunks 0, 16, 32, ..., four to a word
    GemvLongEntry p[GEMV_LONG_MAX_PROJS];
};
static_assert(sizeof(GemvLong) <= 3900, "kernel arguments are at most 4 KB");
inline GemvLongEntry gemv_long_entry(const void *x, const void *y, uint32_t kind, uint32_t layer, uint32_t first_super)
{
    const uint64_t f = kind | (uint64_t)layer << 3 | (uint64_t)first_super << 24, low = ((uint64_t)1 << 44) - 1;
    return GemvLongEntry{{(reinterpret_cast<uint64_t>(x) >> 4 & low) | f << 44, (reinterpret_cast<uint64_t>(y) >> 4 & low) | f >> 20 << 44}};
}
inline __host__ __device__ uint32_t gemv_long_first(const GemvLongEntry &e) { return (uint32_t)(e.w[1] >> 48); }
inline __host__ __device__ BatchProj gemv_batch_proj(const GemvLong &b, uint32_t proj, uint32_t &first_super)
{
    const uint64_t w0 = b.p[proj].w[0], w1 = b.p[proj].w[1], low = ((uint64_t)1 << 44) - 1;
    const uint32_t f = (uint32_t)(w0 >> 44) | (uint32_t)(w1 >> 44 & 0xf) << 20, kind = f & (GEMV_LONG_KINDS - 1);
    const uint64_t off = b.off_h_out[kind];
    BatchProj p;
    p.x = global_pointer((w0 & low) << 4);
    p.y = global_pointer((w1 & low) << 4);
    p.proj_base = b.pool + (uint64_t)(f >> 3) * b.layer_stride + (off & (((uint64_t)1 << 48) - 1));
    p.h_in = b.h_in[kind];
    p.h_out = (int32_t)(off >> 48) * 64;
    first_super = gemv_long_first(b.p[proj]);
    return p;
}
inline __host__ __device__ uint32_t gemv_batch_super(const GemvLong &b, uint32_t super)
{
    const uint32_t mark = super / GEMV_LONG_STEP;
    uint32_t p = (b.marks[mark >> 2] >> (8 * (mark & 3))) & 0xffu;
    while (p + 1 < b.m.n_proj && gemv_long_first(b.p[p + 1]) <= super) ++p;
    return p;
}

// Arguments common to the apply kernels of one (layer, projection).
struct ApplyArgs {
    const char *proj_base;    // device: first slab of this (layer, projection)
    int64_t row_bytes;        // (h_in + h_out) * element size
    const int32_t *tok_list;  // device
    const void *x;            // device [T][h_in]
    void *y;                  // device [T][h_out], in/out
    float *v;                 // device, rows of v_stride floats, one per token: the tile path's shrink result, kept as
                              // bf16 entries s.v[j] (scale and alpha applied) at the front of the token's row
    int32_t h_in, h_out, v_stride;
    float scale;
    // when set, the GEMV expand writes its term s.v.B there as fp32 ([token][h_out]) instead of adding it to y,
    // and linear_tiles_kernel takes the term of its GEMV rows from there
    float *y32 = nullptr;
};

// Optional per-kernel timing: when a launch gets a KernelTimer it asks it for an event pair and
// launches through hipExtLaunchKernelGGL, which stamps the pair with the kernel's own start and
// end (no bracketing commands in the stream, so kernels are neither serialised nor padded).
struct KernelTimer {
    void *ctx;
    void (*pair)(void *ctx, int kind, hipEvent_t *start, hipEvent_t *stop);
};

// `done`, when set, is an event that stands for the end of this kernel: it rides on the kernel's own completion signal
// instead of being recorded behind it (a record is a packet of its own that the queue processes after the kernel:
// 4.0 us per call on the device, 1.6 us this way; measured with an empty kernel).  A timed launch carries the timer's
// events instead: with a timer the caller records.
template <typename K, typename... A>
inline void launch_k(const KernelTimer *tm, hipEvent_t done, int kind, K kernel, dim3 grid, dim3 block, unsigned lds, hipStream_t st, A... args)
{
    hipEvent_t s = nullptr, e = done;
    if (tm) tm->pair(tm->ctx, kind, &s, &e);
    if (e) hipExtLaunchKernelGGL(kernel, grid, block, lds, st, s, e, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, lds, st, args...);
}

// launches (all asynchronous on `st`); dtype is LORA_F32 or LORA_BF16; tm and done may be null (done: see launch_k)
// GEMV shrink and expand of the group's projections: phase 0 as one launch (a.epoch != 0: the expand
// wavefronts wait for the hand-over words to carry that number), phases 1 and 2 as two
// copy (pieces 0: none): lists that the launch copies, in phase 0 and without wide items only, by kernels of their own (the others take 0.2 to 0.4 % longer with the branch in them)
hipError_t launch_gemv(int dtype, const GemvMap &m, const GemvArgs &a, const ListCopy &copy, hipStream_t st, const KernelTimer *tm, hipEvent_t done);
hipError_t launch_gemv_batch(int dtype, const GemvBatch &b, bool wide, const ListCopy &copy, hipStream_t st, const KernelTimer *tm, hipEvent_t done);
hipError_t launch_gemv_long(int dtype, const GemvLong &b, bool wide, const ListCopy &copy, hipStream_t st, const KernelTimer *tm, hipEvent_t done);
// bytes of one projection's hand-over words for max_tokens tokens
size_t gemv_handover_bytes(int dtype, int64_t max_tokens);
// zeroes the hand-over words of tokens toks[0 .. n) (device list) in `sets` sets from `vw` on, vw_set words apart
hipError_t launch_gemv_clear(int dtype, unsigned long long *vw, uint64_t vw_set, int sets, const int32_t *toks, int n, hipStream_t st);
// Tile shrink.  Its work is the sequence of all tiles' k ranges, every tile's range divided into `quanta`
// equal parts (a part is a whole number of the kernel's k stages for every projection of the cache).  A plan
// cuts that sequence into n_runs runs of about equal cost (a tile's cost per part: its x rows plus its At
// rows); run r is worked on by one block per projection of the launch, all blocks of a launch being
// resident at once (two per compute unit), so that the launch ends when a run ends.  A run covers a tail of
// its first tile, whole tiles, and a head of its last tile; a piece that is not a whole tile leaves a partial
// sum in the scratch rows of (run, first or last piece) and mfma_reduce_kernel adds a tile's pieces up.
// Cuts lie on part boundaries at least SHRINK_MIN_PARTS parts from a tile's ends and from each other, or on a
// tile boundary; the last runs of a table may be empty (the table is padded to a multiple of 8 runs).
struct ShrinkCut {  // where run r starts (it ends where run r + 1 starts; entry n_runs = {n_tiles, 0})
    int32_t tile;
    int32_t part;   // 0 <= part < quanta
};
struct ShrinkSum {  // per tile, for the reduce: its pieces' partial sums
    int32_t first_slot;  // scratch slot of the first piece; piece j > 0 lies in slot 2 * (first_slot / 2 + j)
    int32_t n_pieces;    // 1: the tile was worked on whole, the shrink wrote the result itself
};
constexpr int SHRINK_MIN_PARTS = 2;
constexpr int SHRINK_SLOT_ROWS = LORA_TILE_TOKENS;  // rows (of v_stride floats) of one partial-sum slot
// scratch slot of the piece of tile `tile` in run `run` that starts in tile `first_tile`
inline __host__ __device__ int32_t shrink_slot(int32_t run, int32_t first_tile, int32_t tile) { return 2 * run + (tile != first_tile); }
// k stages (of stage_k elements) before part boundary `part` of a row of h_in elements
inline __host__ __device__ int32_t shrink_part_stage(int32_t part, int32_t quanta, int32_t h_in, int32_t stage_k)
{
    const int32_t n_st = (h_in + stage_k - 1) / stage_k;
    return (int32_t)(((int64_t)part * n_st + quanta / 2) / quanta);
}
constexpr int SHRINK_STAGE_K = 128;
// The tile shrink of a launch too short for runs (a few hundred tokens): a block per (projection, unit), a unit being 16 tokens of a
// tile x 16 rank rows over the whole of h_in, so that nothing is left to add up.  A unit is a DevItem of its tokens with a = its first rank row.
constexpr int DIRECT_TOKENS = 16, DIRECT_ROWS = 16;
constexpr int DIRECT_MAX_UNITS = 2048;  // of a plan; with more it carries none
// The tile shrink of a long launch: a block per (panel, k slice, up to three projections that read the same x).  A panel is a DevItem of up to PANEL_ROWS rows of one slot.
// A block's stage of 64 k holds the panel's rows (whole runs of 64) and the rank blocks of its projections, as many projections as fit into PANEL_SLOT_ROWS rows.  A plan's
// panels come in falling order of their rows there for one projection, so those that take one projection per block come first, then two, then three.
constexpr int PANEL_ROWS = 192, PANEL_SLOT_ROWS = 416;
inline __host__ __device__ constexpr int panel_rank_blocks(int rank) { return rank > 96 ? 8 : rank > 64 ? 6 : rank > 32 ? 4 : rank > 16 ? 2 : 1; }  // of 16, as the kernel's bodies come
inline __host__ __device__ constexpr int panel_projs(int runs, int rank_blocks)  // runs of 64 rows
{
    return (PANEL_SLOT_ROWS - 64 * runs) / (16 * rank_blocks) >= 3 ? 3 : (PANEL_SLOT_ROWS - 64 * runs) / (16 * rank_blocks);
}
// Neighbouring panels, mostly of one slot, are dealt out two at a time, to run side by side on one XCD: the second finds part of the first's At in its L2 (eight prompts on q of eight layers fetch
// 380 MB instead of 403).  By themselves, one at a time -> two: four prompts of 1024 tokens of rank 128 on seven projections of two layers 4096 wide 382 -> 370 us a pass, 2048 wide 211 -> 203, 16 of 512 tokens 725 -> 712; 90
// batches of prompts 1024 to 4096 wide 0.5 % in the mean, from 1.6 % worse to 5 % better.  (Four at a time: some XCDs get more of the costly ones.)
constexpr int PANEL_DEAL = 2;
struct PanelClasses {
    int32_t end[3];  // panels before end[c] take at most c + 1 projections per block
};
// blocks of one slice of a group of gn projections
inline __host__ __device__ int panel_blocks(const PanelClasses &c, int gn)
{
    return c.end[0] * gn + (c.end[1] - c.end[0]) * ((gn + 1) / 2) + (c.end[2] - c.end[1]) * ((gn + 2) / 3);
}
// Block i of a group of gn projections in `slices` slices -> slice, panel and its projections [first, first + n) of the group; false: past the end.  Class by class; within a class the
// (slice, panel) pairs are dealt out to the XCDs PANEL_DEAL at a time (block b runs on XCD b % 8), and the blocks of a pair, if there are several, run on one XCD side by side: eight times
// PANEL_DEAL pairs take turns (at a class's end eight or fewer).
inline __host__ __device__ bool panel_of_block(const PanelClasses &c, int gn, int slices, int i, int &slice, int &panel, int &first, int &n)
{
    for (int k = 0, lo = 0; k < 3; lo = c.end[k], ++k) {
        const int count = c.end[k] - lo, per = (gn + k) / (k + 1), blocks = count * slices * per;
        if (i < blocks) {
            const int many = 8 * PANEL_DEAL, whole = count * slices / many * many;  // pairs dealt out PANEL_DEAL at a time
            int pair, turn;
            if (i < whole * per) {
                const int row = i / (many * per), at = i - row * many * per, t = at >> 3;
                turn = t % per;
                pair = many * row + PANEL_DEAL * (at & 7) + t / per;
            } else {
                const int rest = i - whole * per, row = rest / (8 * per), at = rest - row * 8 * per, left = count * slices - whole - 8 * row, width = left < 8 ? left : 8;
                turn = at / width;
                pair = whole + 8 * row + at - turn * width;
            }
            slice = pair / count;
            panel = lo + pair - slice * count;
            first = turn * (k + 1);
            n = gn - first < k + 1 ? gn - first : k + 1;
            return true;
        }
        i -= blocks;
    }
    return false;
}
// The projections one launch of the tile kernels serves, and the run table the shrink works through for each of them:
// projections that read the same x are neighbours (a group); projection i's intermediate lies v_set floats behind that of
// i - 1, its partial sums part_set floats (2 * n_runs slots of SHRINK_SLOT_ROWS rows).
constexpr int GROUP_MAX_PROJS = 4;
struct TileBatchHead {
    int32_t n;
    int32_t n_runs, quanta;   // n_runs: a multiple of 8 (run r is worked on by XCD r / (n_runs / 8))
    int32_t n_tiles, v_stride;
    int32_t any_pieces;       // some tile is worked on in pieces: the reduce launch is needed
    float scale;
    const DevItem *tiles;     // device, n_tiles
    const DevItem *direct;    // device, n_direct units; n_direct = 0: the launch works through the run table
    int32_t n_direct;
    const DevItem *panels;    // device, n_panels panels; n_panels = 0: not by panels
    int32_t n_panels;
    int32_t n_rows;           // rows of all panels
    const ShrinkCut *cuts;    // device, n_runs + 1
    const ShrinkSum *sums;    // device, n_tiles
    const int32_t *tok_list;  // device
    float *v;                 // as ApplyArgs::v
    float *part;              // fp32 partial sums of the tiles worked on in pieces
    uint64_t v_set, part_set;
};
template <int N> struct TileBatchArgs : TileBatchHead {  // as the kernels take it: N is a group's size or a batch's
    uint32_t group[N];  // of projection i: first projection of its group | projections of the group << 8
    BatchProj p[N];
};
struct TileBatch : TileBatchArgs<BATCH_MAX_PROJS> {  // as a launcher takes it
    PanelClasses classes;
    uint8_t slices[BATCH_MAX_PROJS];  // k slices of projection i's panels (of all projections of a group)
};
// blocks of the panels' launch: per group (in the order of the projections) where its blocks end, and first projection | projections << 8 | slices << 16; per projection its slices
template <int N> struct PanelShape {
    int32_t end[N];
    uint32_t group[N];
    uint8_t slices[N];
};
static_assert(sizeof(TileBatchArgs<BATCH_MAX_PROJS>) + sizeof(PanelShape<BATCH_MAX_PROJS>) <= 3900, "kernel arguments are at most 4 KB");
// The LDS that the kernels of a file ask for at launch, made known on the current device: by every cache for its own (each device has
// limits of its own, and threads that create caches or make calls meanwhile share nothing).
template <typename K> hipError_t allow_lds(K *kernel, int bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}
hipError_t prepare_mfma_kernels();
hipError_t prepare_linear_kernels();
// copy (pieces 0: none): lists that the launch copies, as in the GEMV launches; tb's pointers are those into the pool
hipError_t launch_mfma_shrink(const TileBatch &tb, const ListCopy &copy, hipStream_t st, const KernelTimer *tm);
hipError_t launch_mfma_expand(const TileBatch &tb, hipStream_t st, const KernelTimer *tm, hipEvent_t done);
// What lora_linear_plan's kernels read of a plan (device): the list of rows, its runs, the segments of the rows with an adapter
// product (rows [0, add0)), and the rows [add0, add1) whose adapter term has been computed beforehand.
struct LinearList {
    const int32_t *tok;
    const LinearRows *rows;
    const LinearSeg *segs;
    int32_t n_rows, n_rt, add0, add1;
};
// y = x . Wt^T + adapter update for the rows of the list; a.v holds the shrink results
hipError_t launch_zero_rows(void *y, const int32_t *toks, int n, int h_out, hipStream_t st);  // y bf16 [..][h_out]
// The tiles of the grid's last, partly filled round are split along k over several blocks as far as split_scratch
// (device; LINEAR_SHARE_BYTES for every part of a tile) and split_state (device, zero between launches, one per split
// tile) have room; fault: raised when the bounded wait for the other parts gives up.
struct SplitState {
    uint32_t started, way, arrived, read;  // parts that run, have left their sums, have read the others'; way: how the tile is finished
};
constexpr size_t LINEAR_SHARE_BYTES = (size_t)256 * 256 * sizeof(float);  // a tile's accumulators
// How lora_linear_plan's product of n_rt runs of rows is cut into blocks: tiles of `rows` rows (64, 128: x 64 columns, 192, 256, 288: x 256) with a ring of so many
// stages, and how many of them, the last ones, are split along k into `parts` parts.
struct LinearShape {
    int rows, ring, tiles, split, parts;
};
LinearShape linear_shape(int n_rows, int h_in, int h_out, size_t split_scratch_bytes, int n_split_state, int n_cu);
hipError_t launch_linear_tiles(const ApplyArgs &a, const void *Wt, const LinearList &list, void *split_scratch,
                               size_t split_scratch_bytes, SplitState *split_state, int n_split_state, int32_t *fault, int n_cu,
                               hipStream_t st, const KernelTimer *tm, hipEvent_t done);
// a plan's work lists (bytes rounded up to 16) from pinned host memory as the device sees it to their place in the pool
hipError_t launch_upload(void *dst, const void *src, size_t bytes, hipStream_t st, hipEvent_t done);
// A [h_in][r] / B [r][h_out] (16-byte aligned; device memory, or pinned host memory as the device sees it: from_host)
// -> slab layout, for up to REPACK_MAX_PARTS parts of one adapter in one launch (unit_end, r, rs are set by the launcher)
constexpr int REPACK_MAX_PARTS = 32;
struct RepackPart {
    const void *A, *B;
    void *slab;
    int32_t h_in, h_out, unit_end, pad;
};
struct RepackTable {
    RepackPart p[REPACK_MAX_PARTS];
    int32_t n, r, rs, pad;
};
hipError_t launch_repack_parts(int dtype, RepackTable &t, int32_t rank, bool from_host, hipStream_t st);

}  // namespace lora
