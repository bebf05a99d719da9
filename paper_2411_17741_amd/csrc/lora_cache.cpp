// Host side of liblora_cache: pool layout, slot table (the adapter cache's entries and their
// metadata, paper section 4.2), fills from host memory, plans and the apply launches.
#include <algorithm>
#include <limits>
#include <cstdlib>
#include <cstring>
#include <new>
#include <optional>
#include <unordered_map>
#include <vector>

#include "lora_internal.h"

namespace {

thread_local int g_last_hip = 0;

#define HIP_TRY(expr)                          \
    do {                                       \
        hipError_t e_ = (expr);                \
        if (e_ != hipSuccess) {                \
            g_last_hip = (int)e_;              \
            return LORA_E_HIP;                 \
        }                                      \
    } while (0)

constexpr int N_INTERNAL_PLANS = 4;
constexpr int N_STAGES = 2;
// One staging buffer of a fill.  The link moves 16 MB in 0.3 ms; the repack launch behind them (about 15 us with its
// waits on both sides) is then a twentieth of that.
constexpr size_t STAGE_BYTES = (size_t)16 << 20;
constexpr int N_APPLY_EVENTS = 64;
constexpr size_t ALIGN = 256;
// Tile shrink: at most this many runs per projection (two resident blocks per compute unit of a 256-unit part), and
// the variants of the run tables a plan carries: one per number of projections served by one launch up to a group's,
// one with few runs for the small fixed scratch, and two with few runs for batches of many projections.
constexpr int SHRINK_MAX_RUNS = 512;
constexpr int SHRINK_VARIANT_SMALL = lora::GROUP_MAX_PROJS;
constexpr int SHRINK_VARIANT_BATCH = SHRINK_VARIANT_SMALL + 1;
constexpr int SHRINK_BATCH_RUNS[] = {64, 32};
constexpr int SHRINK_VARIANTS = SHRINK_VARIANT_BATCH + 2;
constexpr int SHRINK_BATCH_BLOCKS = 1024;  // a batch's launch has at most this many blocks, where a table is small enough
constexpr int N_LINEAR_SPLITS = 256;  // split tiles of lora_linear_plan (tiles of the last round: fewer than CUs)
// What the tokens of an adapter cost on the GEMV path and on the tile path, in microseconds of one projection's call (`width`: h_in + h_out): fitted
// to calls of one to four prompts of 16 to 2300 tokens at ranks 8 to 128 and widths of 1024 to 4096 (GEMV / tiles measured: 77 tokens of rank 32 at 4096 6.0 / 11.0 us,
// 430 of rank 32 11.9 / 11.5, 430 of rank 128 28.2 / 13.6, 1000 of rank 32 at 1024 12.6 / 10.6, 2300 of rank 8 at 2048 15.9 / 13.7).  Launches with
// enough work for wide items take 0.45 (rank 128) to 1.3 (rank 8) times what the items of four tokens take, which the first formula stands for.
constexpr double GEMV_FIXED_US = 4.0, TILE_FIXED_US = 10.5;
// Beside the base product: a shrink launch, the fp32 term of GEMV rows
constexpr double LINEAR_SHRINK_US = 3.0, LINEAR_TERM_US = 1.0;
// A plan whose own lists have no tiles is made with lists for such launches besides, where one can gain by them: 1 to 4 us more on the host (one prompt of 77 tokens
// 8.2 and 9.1, three of 5 to 400 tokens 11.7 and 15.6), in the same upload.  What a launch has to gain by them was fitted to lists with an upload of their own, 6 us: a list
// of projections nearly all of it, a base product its share if the plan serves every projection of every layer once.  (The choice looks at nothing but the cache, the plan
// and the launch, and the lists are there from the start: the same call gives the same bits, captured or not.)  Measured, us a pass with GEMV alone and as chosen:
// q, k, v, o of two layers, prompts of 11 to 1136 tokens at rank 64 180 and 88; all of two 13B layers, 73 tokens of rank 128 77 and 50; q, k, v of eight layers, 922
// one-token requests over 20 adapters 92 and 83; base product of q, k, v, o 4096 wide, 941 tokens 256 and 216, of q 5120 wide, 1543 tokens 132 and 115.  Of 120 drawn
// lists and products it picks the better way but for 0.5 % in the geometric mean.
constexpr double TILED_LISTS_US = 5.0, LINEAR_MIN_GAIN_US = 1.0, LISTS_COST_US = 6.0;
// More, where a GEMV launch runs as well (200 one-token requests beside prompts of 300 / 1000 / 2048 tokens, GEMV 22.2 / 28.4 / 53.8, with tiles 24.9 / 29.1 / 48.6 us)
constexpr double TILE_BESIDE_GEMV_US = 3.0;
double gemv_tokens_us(int32_t n_tok, int32_t rank, double width, bool wide)
{
    const double k = width / 2048.0;
    return (n_tok + 3) / 4 * (0.004 + 0.0037 * k + rank * (0.00067 + 0.00023 * k)) * (wide ? std::min(1.3, 0.4 + 7.0 / rank) : 1.0);
}
double tile_tokens_us(int32_t n_tok, int32_t rank, double width) { return n_tok * width * (3.0 / 7e6 + 5.4e-9 * rank); }
// the same summed up over a batch's tokens, for launches of several projections
struct PathCost {
    double each = 0, per_width = 0;
    void add_gemv(int32_t n_tok, int32_t rank, bool wide) { add(gemv_tokens_us(n_tok, rank, 0, wide), gemv_tokens_us(n_tok, rank, 2048, wide)); }
    // (a tile of few tokens costs its blocks no less: 8 tiles of 16 on 56 projections 5120 wide 115 us)
    void add_tile(int32_t n_tok, int32_t rank) { add(0, tile_tokens_us(std::max(n_tok, 40), rank, 2048)); }
    void add(double at_0, double at_2048) { each += at_0, per_width += (at_2048 - at_0) / 2048; }
    double us(int n, double sum_width) const { return n * each + per_width * sum_width; }
};
// A tile-shrink launch runs as mfma_shrink_direct_kernel up to so many bytes taken in by its units (64 h_in each): 4000 tokens of ranks 8 to 128, 4096 wide, one
// projection (0.22 GB) 33.3 us per call against 37.4 through the run table; 2300 tokens, mostly of rank 128 (0.27 GB), 67 against 60; eight prompts of ranks 16 to 128 with the
// base product (0.34 GB) 159 against 155.
constexpr int64_t DIRECT_SHRINK_MAX_BYTES = 225000000;
// lora_apply's lists, used by one launch, are read where the host writes them (pinned memory, over the link) up to so many wavefronts that read an item: no upload
// launch.  us a call with the upload and without: 16 fp32 tokens 16.5 and 8.4, 16 requests at 4096 x 4096 16.0 and 8.2, 64 requests (about 2000 wavefronts) 18.5 and 10.5, 200 requests
// (about 6000) 23.4 and 12.4.  So too while the link is busy: 64 requests beside copies or staged fills 19 and 12.3, beside fills by a kernel that reads host memory 139 and 101.
// The first launch of a plan does the same and copies the lists for those that follow, in blocks of its own: one to 200 requests on one projection 1 to 3.7 us a pass less than uploaded ahead,
// idle and beside copies, on as many projections as stay below the line 1 to 2.5; one request on all 224 projections of a 7B model 25.6 and 20.2.  With more wavefronts or wide
// items the lists are uploaded ahead of it (64 requests on q of 32 layers, 65000 wavefronts).
constexpr int64_t PINNED_LISTS_MAX_WAVES = 16384;
// So too a tile shrink of up to so many tiles over its projections, all the lists of a plan being copied then.  us a pass uploaded and copied: eight prompts of 512 tokens 1024 wide on 16 projections (1024 tiles)
// 133.5 and 130.4, on 32 (2048) 239 and 236; 64 of them on four (2048) 233 and 227; 256 of them 512 wide on one (2048) 337 and 322 to 328; 300 short prompts on seven (2100) 233 and
// 231.  Beside copies the same.  Beside fills by a kernel that reads host memory 434 and 417, 430 and 408, 430 and 420, 578 and 571.  Of more tiles it is 1 %, and short prompts lose it beside such fills: 300 on 14 (4200) 829 and
// 838 to 846, on 28 (8400) 1466 and 1497 to 1556.
constexpr int64_t PINNED_LISTS_MAX_TILES = 2048;
// And of up to so many blocks where it runs as mfma_shrink_direct_kernel: each begins with a trip over the link, two stay on a compute unit and those behind them make it again.  us a pass uploaded and copied, idle and
// beside copies: four prompts of 300 tokens on three projections 1024 wide, 681 blocks, 23.4 and 20.5, 25.0 and 21.6; on six, 1362 blocks, 29.9 and 29.6, 31.8 and 34.4; on 14, 3178 blocks, 51.1 and 53.7, 52.6 and
// 59.9; of 700 on two, 1052 blocks, 35.9 and 32.3, 35.7 and 32.3; of 1000 on two, 1496 blocks, 34.6 and 31.9, 34.0 and 37.1; on four, 2992 blocks, 48.9 and 54.1, 50.7 and 63.8.
constexpr int64_t PINNED_LISTS_MAX_DIRECT = 1536;
// Work of a batch's tile kernels (bytes of activations and outputs of the tile tokens) from which its GEMV launch goes to the side stream: fork and join cost
// 10 to 25 us, and what there is to gain is the tails of the kernels, a percent of a millisecond.  us forked and on one stream: whole 7B layers of 500 adapters at 4.8 GB 1795 and 1813,
// twice that 3507 and 3568, one layer (2.4 GB) 968 and 954; 13B with four prompts of 512 (1.6 GB) 876 and 797, with 5120 prompt tokens (4 GB) 1188 and 1200; 64 requests beside a prompt of
// 100 tokens 40.6 and 18.3.  Above the line q alone or q, k, v, o lose: 1417 and 1393 (7B, 4 layers), 512 requests beside 16000 prompt tokens 2769 and 2651.
constexpr double FORK_MIN_TILE_BYTES = 4e9;
// Applies that run together in one batch each have their own copy of the intermediate (a set): as many sets as fit into
// BATCH_SCRATCH_BYTES (0.2 % of the card's memory), a group's at least.  64 one-token requests: 4 MB for 64 sets.
constexpr size_t BATCH_SCRATCH_BYTES = (size_t)512 << 20;
// Sets past GEMV_BATCH_MAX_PROJS as far as all of them stay within this: 224 up to 290 tokens
constexpr size_t LONG_SCRATCH_BYTES = (size_t)64 << 20;

size_t align_up(size_t v, size_t a = ALIGN) { return (v + a - 1) / a * a; }

// Device memory an apply needs beside its inputs and outputs: the shrink results (one set per
// projection of a group), the partial sums that the runs of the tile shrink leave, and the tagged words through
// which the one-launch GEMV form hands its intermediate over.
struct Scratch {
    char *v;
    size_t v_set_bytes;
    int n_sets;
    char *vpart;
    int64_t vpart_rows;        // rows of the partial-sum scratch, shared by the projections of a group
    bool small;                // the fixed scratch, which holds the partial sums of the small run table only
    char *vtag;                // hand-over words of the GEMV phases, one set per projection of a group
    size_t vtag_set_bytes;
    uint32_t *epoch;           // host counter of the one-launch GEMV launches that have used vtag
    // the latest one-launch GEMV enqueued under stream capture with this scratch: capture, plan and sets
    // (a replayed launch finds its own number in the words it wrote the last time, unless another launch
    // of the graph has written them since)
    unsigned long long *cap_id;
    uint64_t *cap_plan;
    int *cap_sets;
};

// The same scratch as a fixed array in the library's image, for lora_apply_plan_static: one set,
// sized for LORA_STATIC_MAX_TOKENS tokens.  Every device the library runs on holds its own copy
// at its own address (found once per device with hipGetSymbolAddress; the array's name itself is
// no device address in host code).
constexpr size_t STATIC_V_BYTES = sizeof(float) * (size_t)LORA_STATIC_MAX_TOKENS * LORA_MAX_RANK;
constexpr int STATIC_SHRINK_RUNS = 128;
constexpr int64_t STATIC_VPART_ROWS = 2 * (int64_t)lora::SHRINK_SLOT_ROWS * STATIC_SHRINK_RUNS;  // = 4 x LORA_STATIC_MAX_TOKENS
constexpr size_t STATIC_VPART_BYTES = sizeof(float) * (size_t)STATIC_VPART_ROWS * LORA_MAX_RANK;
constexpr size_t STATIC_VTAG_BYTES = sizeof(uint64_t) * (size_t)LORA_STATIC_MAX_TOKENS * LORA_MAX_RANK;  // fp32 words; bf16 takes half
constexpr size_t STATIC_SCRATCH_BYTES = STATIC_V_BYTES + STATIC_VPART_BYTES + STATIC_VTAG_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
struct StaticScratch {
    char *ptr = nullptr;   // this device's copy of `scratch`
    uint32_t epoch = 0;    // one-launch GEMV launches that have used its hand-over words, over all caches of the process
    unsigned long long cap_id = 0;
    uint64_t cap_plan = 0;
    int cap_sets = 0;
};
StaticScratch g_static[MAX_DEVICES];

// Once per device, with that device current: the address of its copy, and tagged words that carry no
// launch number yet.
int static_scratch_setup(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return LORA_E_INVAL;
    StaticScratch &ss = g_static[device];
    if (ss.ptr) return LORA_OK;
    char *ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)));
    if (!ptr) return LORA_E_HIP;
    HIP_TRY(hipMemset(ptr + STATIC_V_BYTES + STATIC_VPART_BYTES, 0, STATIC_VTAG_BYTES));
    ss.ptr = ptr;
    return LORA_OK;
}
int esize_of(int dtype) { return dtype == LORA_BF16 ? 2 : 4; }

struct Slot {
    int32_t cls = 0;
    bool bound = false;
    int64_t adapter_id = 0;
    int32_t rank = 0;
    float alpha = 1.f;
    int32_t refcount = 0;
    int64_t use_count = 0, last_used = 0;
    int64_t last_by[2] = {0, 0};  // last_used by calls with the pool's scratch and by those with the fixed one (they may overlap)
    double req_freq = 0;   // requests that used the entry, halved every policy.freq_window requests
    int64_t req_last = 0;  // number of the last such request
    uint32_t generation = 0;  // bumped whenever the slot is bound to another adapter or evicted
    std::vector<uint8_t> part;  // [n_layers * n_proj] 1 = data enqueued
    int32_t parts_filled = 0;
    hipEvent_t fill_ev = nullptr;
    bool fill_pending = false;
};

struct Stage {
    char *dev = nullptr;
    hipEvent_t ev = nullptr;  // the repack that read this buffer is done: it may be overwritten
    bool pending = false;
};

}  // namespace

// The work lists of a batch cut one way (one threshold between tiles and GEMV groups), and where they lie behind `lists`
struct PlanLists {
    const char *lists = nullptr;  // where the kernels read them
    int32_t T = 0;
    int32_t n_tok_list = 0, n_tiles = 0, n_gs = 0, n_ge = 0;
    int32_t n_tile_tok = 0;  // tokens of all tiles = leading entries of tok_list
    // the tile shrink's run tables (cuts, then the tiles' piece records), per variant
    int32_t shrink_quanta = 1;
    int32_t shrink_runs[SHRINK_VARIANTS] = {0};
    bool shrink_pieces[SHRINK_VARIANTS] = {false};
    size_t off_cuts[SHRINK_VARIANTS] = {0}, off_sums[SHRINK_VARIANTS] = {0};
    uint64_t build_seq = 0;  // changes whenever the lists are rebuilt
    size_t off_tiles = 0, off_gs = 0, off_ge = 0;
    int32_t n_wgs = 0, n_wge = 0;  // the GEMV work as wide items (bf16 caches)
    size_t off_wgs = 0, off_wge = 0;
    // for lora_linear_plan: the list of every token of the batch, its runs of rows and its segments (lora::LinearList)
    size_t off_lin_tok = 0, off_lin_rows = 0, off_lin_segs = 0;
    int32_t n_lin_rows = 0, n_lin_segs = 0;
    size_t off_direct = 0;  // units of a short tile shrink (0 of them: too many for that)
    int32_t n_direct = 0;
    size_t off_panels = 0;  // panels of a long tile shrink
    int32_t n_panels = 0;
    lora::PanelClasses panel_classes{};
    int32_t panel_count[lora::PANEL_ROWS / 64 + 1][9] = {{0}};  // by runs of 64 rows and rank blocks
    double panel_sum_bytes = 0;  // of one slice's sums, written and read
    int64_t tile_rows = 0;       // rows the run table's kernel takes in per stage: 64 and the rank of every tile
};

struct lora_plan : PlanLists {  // (the lists that a call for one projection works through)
    bool in_use = false;
    bool internal = false;
    char *dev = nullptr;
    char *pinned = nullptr;
    const char *pinned_dev = nullptr;  // the same as the device sees it; the lists are in dev or there
    hipEvent_t ev_upload = nullptr;
    bool upload_pending = false;
    // Lists that are still where the host wrote them alone (`deferred`): the first launch that works through them copies them, and reads them there.  That launch is covered by
    // the fence of its call (upload_fence, -1: none); copying: the call that runs now has got to it, its fence is not published yet
    bool deferred = false, copying = false;
    int32_t upload_fence = -1;
    int32_t last_use[2] = {-1, -1};  // fences of the latest calls that used the plan, with the pool's scratch and with the fixed one (they may overlap)
    bool unfenced = false;  // calls without a fence (captured, or with fencing off) have read lists in dev, and no upload in the order of a caller's stream has come since
    int32_t mfma_min_used = 0;  // the threshold the work lists were made with
    size_t bytes = 0;           // of these lists
    // Where a call for one projection leaves the tokens that could be tiles to the GEMV kernels, launches that share the tile path's fixed cost, and the base product, which needs
    // no expand launch, may do better with tiles: what it takes to tell (for the threshold 16), and the lists for them, behind the plan's own, where some launch can gain by them
    bool has_tiled = false;
    PathCost gemv_cost[2], rest_cost[2], tile_cost;  // GEMV tokens [items, wide items] of the lists and of those with tiles; the tile tokens
    int32_t rest_groups = 0, rest_wgs = 0, tile_tok = 0, tile_segs = 0;
    PlanLists tiled;
    size_t tiled_bytes = 0;
    std::vector<int32_t> slots;        // distinct slots the batch names
    std::vector<uint32_t> generations;  // their generation at plan time
};

struct lora_cache {
    std::vector<lora_proj_t> proj;
    std::vector<int32_t> class_rank, class_slots, class_first;
    int32_t n_layers = 0, n_slots = 0, dtype = 0, esize = 0;
    int32_t max_tokens = 0, max_segments = 0, n_user_plans = 0, mfma_min = 0, flags = 0;
    int32_t direct_max = 0;      // units of a short tile shrink that a plan has room for
    bool small_scratch = false;  // the pool holds the scratch of a group of projections only
    bool mfma_min_auto = false;  // the configuration left the threshold to the library
    int32_t v_stride = 0;
    bool host_only = false;

    char *pool = nullptr;
    size_t pool_bytes = 0;
    size_t layer_stride = 0;
    std::vector<int32_t> slot_row;  // [n_slots] first storage row of the slot (same in every projection)
    std::vector<size_t> proj_off;   // [n_proj] byte offset of the projection's slabs inside a layer
    std::vector<size_t> row_bytes;  // [n_proj] (h_in + h_out) * element size
    int64_t total_rows = 0;
    size_t off_splits = 0, off_vpart = 0, off_vtag = 0, v_set_bytes = 0, vtag_set_bytes = 0;
    int n_sets = lora::GROUP_MAX_PROJS;  // copies of the intermediate buffers: projections of a batch
    uint32_t tag_epoch = 0;  // one-launch GEMV launches so far; the number the words of the latest one carry
    unsigned long long cap_id = 0;
    uint64_t cap_plan = 0;  // build number of the plan
    int cap_sets = 0;
    int64_t vpart_rows = 0;  // rows of the tile shrink's partial-sum scratch
    size_t vpart_bytes = 0;
    int fused_gemv = 0;  // 0 never, 1 by size, 2 always
    size_t off_v = 0, off_plans = 0, off_stage = 0, plan_cap = 0, stage_cap = 0, total = 0;

    std::vector<Slot> slots;
    std::unordered_map<int64_t, int32_t> id2slot;
    std::vector<lora_plan> plans;  // user plans first, then the internal ring
    uint64_t internal_next = 0, plan_builds = 0, user_next = 0;
    Stage stage[N_STAGES];
    bool direct_fill = false;
    uint64_t stage_next = 0;

    // Within a group the GEMV launch (decode tokens) and the tile kernels (prompts) touch different tokens and
    // different scratch: they run side by side, the GEMV launch on a stream of the cache's own between a fork
    // and a join event (default priority, like every stream here)
    hipStream_t side_stream = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // Uploads that a captured call needs and that must not become part of the graph.  Not the side stream's: one that a captured call has forked to stays in the capture until that ends, joined or not.
    // Made by the first call that needs it: with a third stream in the process the tile expand of 16 prompts of 512 tokens on eight projections 1024 wide takes 88.5 us instead of 83.7
    hipStream_t upload_stream = nullptr;
    int device = 0;  // the device that was current at lora_cache_create
    int n_cu = 256;  // its compute units
    bool fencing = true;
    int64_t apply_seq = 0;
    // Fences: every call that enqueues applies has one event that stands for its end.  It is held by its place in a
    // ring of the latest calls, by the stream it is the latest of and by the plan it is the latest use of; an event
    // that nobody holds is free (one event per call instead of one per holder: a record costs the device 4 us).
    struct Fence {
        hipEvent_t ev;
        int32_t holders;
    };
    std::vector<Fence> fences;
    size_t next_fence = 0;  // where the search for a free one starts
    int32_t ring[N_APPLY_EVENTS];  // index into fences, -1: none
    int64_t ring_seq[N_APPLY_EVENTS] = {};
    std::unordered_map<hipStream_t, int32_t> stream_fence;
    // raised by a kernel that gave up a bounded wait: one word of pinned host memory that the kernels
    // write through its device address, so the host sees it without a synchronisation
    int32_t *fault_host = nullptr, *fault_dev = nullptr;

    lora_cache_stats_t stats = {};
    lora_policy_t policy = {0.45, 0.10, 0.45, 0};  // section 4.2's F, R, S
    int64_t req_seq = 0;                           // requests seen by lora_cache_acquire

    // benchmark aid: event pairs around kernels
    bool timing = false;
    struct Timed {
        int kind;
        hipEvent_t start, stop;
    };
    std::vector<Timed> timed;
    std::vector<hipEvent_t> free_events;
};

namespace {

bool config_ok(const lora_cache_config_t *cfg)
{
    if (!cfg || cfg->n_proj < 1 || !cfg->proj || cfg->n_layers < 1 || cfg->n_classes < 1 || !cfg->class_rank ||
        !cfg->class_slots)
        return false;
    if (cfg->dtype != LORA_F32 && cfg->dtype != LORA_BF16) return false;
    if (cfg->max_tokens < 1 || cfg->max_segments < 1 || cfg->n_plans < 0 || cfg->mfma_min_tokens < 0) return false;
    for (int p = 0; p < cfg->n_proj; ++p)
        if (cfg->proj[p].h_in < 64 || cfg->proj[p].h_out < 64 || cfg->proj[p].h_in % 64 || cfg->proj[p].h_out % 64)
            return false;
    int64_t total_slots = 0;
    for (int c = 0; c < cfg->n_classes; ++c) {
        if (cfg->class_rank[c] < 1 || cfg->class_rank[c] > LORA_MAX_RANK || cfg->class_slots[c] < 0) return false;
        if (c && cfg->class_rank[c] <= cfg->class_rank[c - 1]) return false;
        total_slots += cfg->class_slots[c];
    }
    return total_slots >= 1 && total_slots * (int64_t)LORA_MAX_RANK < (int64_t)1 << 31;
}

// Fills every layout field of `c` from the config; used by bytes_required and create alike.  small_scratch: what a group
// of projections needs and no more -- no further sets, run tables and wide items for batches, staging for one part.
// max_sets: sets for batches at most; direct: plans have room for the units of a short tile shrink.
void compute_layout(lora_cache &c, const lora_cache_config_t *cfg, bool small_scratch, int max_sets = lora::GEMV_LONG_MAX_PROJS, bool direct = true)
{
    c.small_scratch = small_scratch;
    c.proj.assign(cfg->proj, cfg->proj + cfg->n_proj);
    c.class_rank.assign(cfg->class_rank, cfg->class_rank + cfg->n_classes);
    c.class_slots.assign(cfg->class_slots, cfg->class_slots + cfg->n_classes);
    c.n_layers = cfg->n_layers;
    c.dtype = cfg->dtype;
    c.esize = esize_of(cfg->dtype);
    c.max_tokens = cfg->max_tokens;
    c.max_segments = cfg->max_segments;
    c.n_user_plans = cfg->n_plans;
    c.mfma_min = cfg->dtype == LORA_BF16 ? (cfg->mfma_min_tokens ? cfg->mfma_min_tokens : LORA_MFMA_MIN_TOKENS) : 0;
    c.mfma_min_auto = cfg->dtype == LORA_BF16 && cfg->mfma_min_tokens == 0;
    c.flags = cfg->flags;
    c.host_only = (cfg->flags & LORA_CACHE_HOST_ONLY) != 0;
    c.direct_fill = (cfg->flags & LORA_CACHE_DIRECT_FILL) != 0;
    c.fused_gemv = (cfg->flags & LORA_CACHE_SPLIT_GEMV) ? 0 : ((cfg->flags & LORA_CACHE_FUSED_GEMV) ? 2 : 1);

    const int n_proj = cfg->n_proj, n_cls = cfg->n_classes;
    c.class_first.resize(n_cls);
    c.n_slots = 0;
    for (int k = 0; k < n_cls; ++k) {
        c.class_first[k] = c.n_slots;
        c.n_slots += c.class_slots[k];
    }
    c.slot_row.assign(c.n_slots, 0);
    c.total_rows = 0;
    for (int k = 0; k < n_cls; ++k)
        for (int s = 0; s < c.class_slots[k]; ++s) {
            c.slot_row[c.class_first[k] + s] = (int32_t)c.total_rows;
            c.total_rows += lora::rank_storage(c.class_rank[k]);
        }
    c.proj_off.assign(n_proj, 0);
    c.row_bytes.assign(n_proj, 0);
    size_t off = 0, max_part = 0, row_sum = 0;
    for (int p = 0; p < n_proj; ++p) {
        const size_t width = (size_t)c.proj[p].h_in + (size_t)c.proj[p].h_out;
        c.proj_off[p] = off;
        c.row_bytes[p] = width * c.esize;  // a multiple of 256 bytes: h_in, h_out are multiples of 64
        row_sum += c.row_bytes[p];
        off += (size_t)c.total_rows * c.row_bytes[p];
        max_part = std::max(max_part, (size_t)c.class_rank[n_cls - 1] * width * c.esize);
    }
    c.layer_stride = off;
    c.v_stride = LORA_MAX_RANK;  // the GEMV expand reads whole rows of 128 entries (masked past the rank)

    const size_t max_tiles = (size_t)c.max_tokens / LORA_TILE_TOKENS + 2 * (size_t)c.max_segments + 2;
    // GEMV items: per token batch up to 32 shrink + 16 expand items; batches <= groups + tokens/4
    const size_t max_batches = (size_t)c.max_segments + (size_t)c.max_tokens / lora::GEMV_BATCH + 1;
    const size_t max_items = max_tiles + max_batches * (LORA_MAX_RANK / 4 + 16);
    const size_t max_wide = c.dtype != LORA_BF16 || small_scratch ? 0
                                                 : ((size_t)c.max_segments + (size_t)c.max_tokens / lora::GEMV_WIDE_SHRINK_TOKENS + 1) * (LORA_MAX_RANK / lora::GEMV_WIDE_ROWS) +
                                                       ((size_t)c.max_segments + (size_t)c.max_tokens / lora::GEMV_WIDE_TOKENS + 1) * 16;
    // units of a short tile shrink: no more than a launch of the narrowest projection may have, nor than the tokens make
    size_t narrowest = SIZE_MAX;
    for (const auto &pr : c.proj) narrowest = std::min(narrowest, (size_t)pr.h_in);
    c.direct_max = c.dtype != LORA_BF16 || small_scratch || !direct ? 0
                       : (int32_t)std::min({(size_t)lora::DIRECT_MAX_UNITS, (size_t)DIRECT_SHRINK_MAX_BYTES / (64 * narrowest),
                                            ((size_t)c.max_tokens / lora::DIRECT_TOKENS + max_tiles) * (LORA_MAX_RANK / lora::DIRECT_ROWS)});
    const int n_tables = small_scratch ? SHRINK_VARIANT_BATCH : SHRINK_VARIANTS;
    c.plan_cap = align_up(sizeof(int32_t) * (size_t)c.max_tokens) + align_up(sizeof(lora_item_t) * max_items) +
                 align_up(sizeof(int32_t) * max_batches) + 4 * ALIGN + (max_wide ? align_up(sizeof(lora::GemvWideItem) * max_wide) + 2 * ALIGN : 0) +
                 (c.dtype == LORA_BF16 ? align_up(sizeof(int32_t) * (size_t)c.max_tokens) +
                                             align_up(sizeof(lora::LinearRows) * ((size_t)c.max_tokens / LORA_TILE_TOKENS + 2)) +
                                             align_up(sizeof(lora::LinearSeg) * (size_t)c.max_segments) : 0) +
                 align_up(sizeof(lora::DevItem) * (size_t)c.direct_max) +
                 n_tables * (align_up(sizeof(lora::ShrinkCut) * (SHRINK_MAX_RUNS + 1)) + align_up(sizeof(lora::ShrinkSum) * max_tiles));
    // fill staging: a buffer takes parts of an adapter until STAGE_BYTES (or the largest adapter) are in it
    c.stage_cap = small_scratch ? align_up(max_part) + ALIGN : align_up(std::max(max_part, std::min(STAGE_BYTES, (size_t)c.class_rank[n_cls - 1] * row_sum * c.n_layers)));

    size_t cur = align_up(c.layer_stride * (size_t)c.n_layers);
    c.off_splits = cur;
    cur += align_up(sizeof(lora::SplitState) * N_LINEAR_SPLITS);
    c.off_v = cur;
    c.v_set_bytes = align_up(sizeof(float) * (size_t)c.max_tokens * c.v_stride);
    c.vtag_set_bytes = align_up(lora::gemv_handover_bytes(c.dtype, c.max_tokens));
    {  // (sets past a common batch's are for launches that their own cost matters to: few tokens)
        const size_t set = c.v_set_bytes + c.vtag_set_bytes, room = std::max<size_t>(lora::GROUP_MAX_PROJS, BATCH_SCRATCH_BYTES / set);
        const size_t most = std::max(std::min<size_t>(lora::GEMV_BATCH_MAX_PROJS, room), std::min<size_t>(lora::GEMV_LONG_MAX_PROJS, LONG_SCRATCH_BYTES / set));
        c.n_sets = small_scratch ? lora::GROUP_MAX_PROJS : (int)std::min({(size_t)max_sets, (size_t)c.n_layers * c.proj.size() + lora::GROUP_MAX_PROJS, most});
    }
    cur += c.v_set_bytes * c.n_sets;
    // partial sums of the tile shrink: two slots per run and projection; a launch has at most SHRINK_MAX_RUNS blocks
    // for a group whatever its size, twice that for a batch, and a batch of few tiles has few runs (a piece is at
    // least two of the parts a tile's k range is cut into)
    {
        const int64_t tiles = std::max<int64_t>(1, ((int64_t)c.max_tokens + LORA_TILE_TOKENS - 1) / LORA_TILE_TOKENS);
        const int64_t runs = std::min<int64_t>((small_scratch ? 1 : 2) * SHRINK_MAX_RUNS, 16 * std::min(c.n_sets, lora::GEMV_BATCH_MAX_PROJS) * tiles);
        c.vpart_rows = c.dtype == LORA_BF16 ? 2 * lora::SHRINK_SLOT_ROWS * runs : 0;
    }
    c.off_vpart = cur;
    c.vpart_bytes = align_up(sizeof(float) * (size_t)c.vpart_rows * c.v_stride);
    // (the fused linear kernel parks the sums of its split tiles in the same region: a third more parts than a round of 256 blocks,
    // 256 KB each; less for caches of small batches)
    if (c.dtype == LORA_BF16 && small_scratch) {
        c.vpart_bytes = std::max(c.vpart_bytes, std::min<size_t>((size_t)48 << 20, align_up(sizeof(float) * (size_t)c.v_stride * 8 * (size_t)c.max_tokens)));
    } else if (c.dtype == LORA_BF16) {
        const size_t row_tiles = std::min<size_t>((size_t)c.max_tokens, (size_t)c.max_tokens / LORA_TILE_TOKENS + (size_t)c.max_segments) + 2;
        size_t col_tiles = 1;
        for (const auto &pr : c.proj) col_tiles = std::max(col_tiles, ((size_t)pr.h_out + 255) / 256);
        c.vpart_bytes = std::max(c.vpart_bytes, lora::LINEAR_SHARE_BYTES * std::min<size_t>(340, (row_tiles + 3) / 4 * col_tiles * 8));
    }
    cur += c.vpart_bytes;
    // the GEMV phases hand their intermediate over as 64-bit words, one row per token and projection of a group
    c.off_vtag = cur;
    cur += c.vtag_set_bytes * c.n_sets;
    c.off_plans = cur;
    cur += c.plan_cap * (size_t)(c.n_user_plans + N_INTERNAL_PLANS);
    c.off_stage = cur;
    cur += c.stage_cap * N_STAGES;
    c.total = cur;
}

// The layout for a pool of fewer bytes than are required: fewer sets for batches (down to those of a batch with tiles), then without the units of
// a short tile shrink and with as many sets as there is room for, then the small scratch.
void fit_layout(lora_cache &c, const lora_cache_config_t *cfg, size_t bytes)
{
    if (!(cfg->flags & LORA_CACHE_SMALL_SCRATCH)) {
        for (int direct = 1; direct >= 0; --direct)
            for (int sets = direct ? c.n_sets : std::min(c.n_sets, lora::BATCH_MAX_PROJS); sets >= (direct ? lora::BATCH_MAX_PROJS : lora::GROUP_MAX_PROJS); --sets) {
                lora_cache t;
                compute_layout(t, cfg, false, sets, direct != 0);
                if (t.total > bytes) continue;
                compute_layout(c, cfg, false, sets, direct != 0);
                return;
            }
    }
    compute_layout(c, cfg, true);
}

char *slab_ptr(const lora_cache &c, int32_t layer, int32_t proj, int32_t slot)
{
    return c.pool + (size_t)layer * c.layer_stride + c.proj_off[proj] + (size_t)c.slot_row[slot] * c.row_bytes[proj];
}

int class_of_slot(const lora_cache &c, int32_t slot)
{
    int k = (int)c.class_first.size() - 1;
    while (k > 0 && slot < c.class_first[k]) --k;
    return k;
}

void unbind(lora_cache &c, Slot &s)
{
    if (s.bound) {
        auto it = c.id2slot.find(s.adapter_id);
        if (it != c.id2slot.end() && &c.slots[it->second] == &s) c.id2slot.erase(it);
    }
    s.bound = false;
    s.adapter_id = 0;
    s.rank = 0;
    s.alpha = 1.f;
    s.use_count = 0;
    s.req_freq = 0;
    s.req_last = 0;
    s.refcount = 0;
    s.parts_filled = 0;
    std::fill(s.part.begin(), s.part.end(), 0);
    ++s.generation;
}

// Section 4.2's eviction score of every cached entry: F * frequency + R * recency + S * size.
// The paper gives no units: each term is scaled to [0, 1] over the cached entries (frequency and
// rank by the largest cached, recency as 1 - age / largest age, age counted in requests), so that
// the coefficients weigh comparable quantities.  Entries that are not cached get +inf.
std::vector<double> eviction_scores(const lora_cache &c)
{
    double max_f = 0, max_age = 0, max_rank = 0;
    for (const Slot &s : c.slots) {
        if (!s.bound) continue;
        max_f = std::max(max_f, s.req_freq);
        max_age = std::max(max_age, (double)(c.req_seq - s.req_last));
        max_rank = std::max(max_rank, (double)s.rank);
    }
    std::vector<double> score(c.slots.size(), std::numeric_limits<double>::infinity());
    for (size_t i = 0; i < c.slots.size(); ++i) {
        const Slot &s = c.slots[i];
        if (!s.bound) continue;
        const double f = max_f > 0 ? s.req_freq / max_f : 0.0;
        const double r = max_age > 0 ? 1.0 - (double)(c.req_seq - s.req_last) / max_age : 1.0;
        const double z = (double)s.rank / max_rank;
        score[i] = c.policy.w_freq * f + c.policy.w_recency * r + c.policy.w_size * z;
    }
    return score;
}

bool is_queued(const int64_t *ids, int32_t n, int64_t id)
{
    for (int32_t i = 0; i < n; ++i)
        if (ids[i] == id) return true;
    return false;
}

// The entry to evict for an adapter of `rank` (any rank if 0): lowest score among the entries
// no running request uses and whose slot is large enough; entries of queued requests only if
// there is no other (section 4.2).  Ties go to the lower slot.  -1 if every candidate is in use.
int32_t choose_victim(const lora_cache &c, int32_t rank, const int64_t *queued, int32_t n_queued)
{
    const std::vector<double> score = eviction_scores(c);
    for (int pass = 0; pass < 2; ++pass) {
        int32_t best = -1;
        for (int32_t i = 0; i < c.n_slots; ++i) {
            const Slot &s = c.slots[i];
            if (!s.bound || s.refcount > 0 || c.class_rank[s.cls] < rank) continue;
            if (pass == 0 && is_queued(queued, n_queued, s.adapter_id)) continue;
            if (best < 0 || score[i] < score[best]) best = i;
        }
        if (best >= 0) return best;
    }
    return -1;
}

// bytes of pool memory the entry of a slot holds: its rank's storage rows in every layer and projection
size_t entry_bytes(const lora_cache &c, const Slot &s)
{
    size_t per_row = 0;
    for (size_t p = 0; p < c.proj.size(); ++p) per_row += c.row_bytes[p];
    return (size_t)lora::rank_storage(s.rank) * per_row * (size_t)c.n_layers;
}

int slot_state(lora_cache &c, Slot &s)
{
    if (!s.bound) return LORA_SLOT_EMPTY;
    if (s.parts_filled < (int32_t)s.part.size()) return LORA_SLOT_FILLING;
    if (s.fill_pending && !c.host_only) {
        if (hipEventQuery(s.fill_ev) == hipSuccess) s.fill_pending = false;
        else return LORA_SLOT_FILLING;
    }
    return LORA_SLOT_READY;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

bool is_capturing(hipStream_t st)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return cs != hipStreamCaptureStatusNone;
}

// The tile shrink's run table for `max_runs` runs (header of ShrinkCut in lora_internal.h): cuts[0 .. n_runs] and one
// piece record per tile.  A tile's cost per part of its k range: its x rows (absent rows are still loaded) plus its
// stored At rows (measured: a rank-128 tile takes 1.8 times as long as a rank-16 one).
struct ShrinkRuns {
    std::vector<lora::ShrinkCut> cuts;
    std::vector<lora::ShrinkSum> sums;
    int n_runs = 0;
    bool any_pieces = false;
};
bool shrink_pieces_of(const lora::DevItem *tiles, int n_tiles, int quanta, ShrinkRuns &out)
{
    out.sums.assign((size_t)n_tiles, lora::ShrinkSum{0, 0});
    out.any_pieces = false;
    for (int r = 0; r < out.n_runs; ++r) {
        const lora::ShrinkCut from = out.cuts[r], to = out.cuts[r + 1];
        const int last_tile = std::min(to.part > 0 ? to.tile : to.tile - 1, n_tiles - 1);
        for (int t = from.tile; t <= last_tile; ++t) {
            const int lo = t == from.tile ? from.part : 0, hi = t == to.tile ? to.part : quanta;
            if (lo >= hi) continue;
            lora::ShrinkSum &sm = out.sums[t];
            const int32_t slot = lora::shrink_slot(r, from.tile, t);
            if (sm.n_pieces == 0) sm.first_slot = (lo == 0 && hi == quanta) ? 0 : slot;
            else if (slot != 2 * (sm.first_slot / 2 + sm.n_pieces)) return false;  // (cannot happen: later pieces start their runs)
            ++sm.n_pieces;
            if (sm.n_pieces > 1) out.any_pieces = true;
        }
    }
    for (int t = 0; t < n_tiles; ++t)
        if (out.sums[t].n_pieces < 1) return false;
    return true;
}
// Runs of about equal cost, at most max_runs of them (a multiple of 8).  A piece costs its parts times its tile's
// weight, plus a fixed amount.  Measured with every block of a launch resident from the start (two per compute unit):
// a block spends about 6.5 us beside its k loop (the item, the first three stages of loads that every block requests at
// once, the write of the result); a stage of 128 k takes it 1.4 us at rank 16, 1.6 us at rank 32, 1.9 us at rank 64 and
// 2.6 us at rank 128 when the launch is long (x arrives at the rate the memory gives, the higher ranks add their At
// loads).  The result is flat around these weights: a fixed amount of 3 to 6 stages and a stage offset of 30 to 60
// gave the same launch times to within 1 %.
// Tables of few runs, long ones: for a cost limit the sequence is walked once, every run taking pieces until the limit is reached; the limit starts
// at an equal share of everything and grows by half a part or one percent until max_runs suffice.  Tables of many runs, a few parts each: one pass, run r
// starts where r equal shares of the cost are behind it.  (That way the long ones end a part later, prefill batch 228.3 -> 229.4 us; a search for the limit in
// all seven tables of a plan took 40 to 100 us of the host.)
constexpr int SHRINK_SEARCH_RUNS = 128;
void build_shrink_runs(const lora::DevItem *tiles, int n_tiles, int quanta, int max_runs, ShrinkRuns &out)
{
    constexpr int MINP = lora::SHRINK_MIN_PARTS;
    constexpr double PIECE = 6 * (44 + LORA_TILE_TOKENS + 16);  // six stages at rank 16
    auto weight = [&](int t) { return 44.0 + tiles[t].n_tok + lora::rank_storage(tiles[t].rank); };  // rank 128 : rank 16 = 1.9
    double total = 0;
    for (int t = 0; t < n_tiles; ++t) total += weight(t) * quanta + PIECE;
    const double part = (total - n_tiles * PIECE) / ((double)n_tiles * quanta);  // the average part's cost
    if (max_runs > SHRINK_SEARCH_RUNS) {
        const double share = total / max_runs;
        out.cuts.assign(1, lora::ShrinkCut{0, 0});
        double before = 0, w = weight(0);  // cost of the tiles before tile t, weight of tile t
        for (int r = 1, t = 0; r < max_runs; ++r) {
            const double goal = share * r;
            while (t < n_tiles && before + w * quanta + PIECE <= goal) {
                before += w * quanta + PIECE;
                if (++t < n_tiles) w = weight(t);
            }
            const lora::ShrinkCut at = out.cuts.back();
            lora::ShrinkCut cut{t, t < n_tiles ? (int)((goal - before) / w) : 0};
            if (cut.part < MINP) cut.part = 0;
            if (cut.tile < at.tile || (cut.tile == at.tile && cut.part < at.part + MINP)) cut = lora::ShrinkCut{at.tile, at.part + MINP};  // a run takes something
            if (quanta - cut.part < MINP) cut = lora::ShrinkCut{cut.tile + 1, 0};  // no slivers: the rest of the tile
            if (cut.tile >= n_tiles) break;
            out.cuts.push_back(cut);
        }
    } else {
        for (double limit = std::max((total + 0.5 * max_runs * PIECE) / max_runs, MINP * part + PIECE);; limit += std::max(0.01 * limit, 0.5 * part)) {
            int t = 0, q = 0;
            out.cuts.clear();
            while (t < n_tiles && (int)out.cuts.size() < max_runs) {
                out.cuts.push_back(lora::ShrinkCut{t, q});
                double left = limit;
                for (bool first = true; t < n_tiles; first = false) {
                    const double w = weight(t), rest = w * (quanta - q) + PIECE;
                    if (rest <= left) {  // the rest of the tile
                        left -= rest;
                        ++t, q = 0;
                        continue;
                    }
                    int parts = left > PIECE ? (int)((left - PIECE) / w) : 0;  // what still fits
                    if (parts < MINP) {
                        if (!first) break;  // the run ends on the tile boundary
                        parts = MINP;       // a run takes something
                    }
                    if (quanta - q - parts < MINP) ++t, q = 0;  // no slivers: the rest of the tile
                    else q += parts;
                    break;
                }
            }
            if (t >= n_tiles) break;  // (the limit that takes everything in one run is reached in the end)
        }
    }
    out.n_runs = (int)((out.cuts.size() + 7) / 8 * 8);
    out.cuts.resize((size_t)out.n_runs + 1, lora::ShrinkCut{n_tiles, 0});
    if (!shrink_pieces_of(tiles, n_tiles, quanta, out)) out.n_runs = 0;  // (cannot happen: the cuts rise)
}

// Wide items (up to 16 rank rows and 8 or 16 tokens) from so many wide shrink items of a launch up, for several groups and for one:
// with fewer, the items of 4 rows and 4 tokens share the work out better.  One request on every projection of a 7B model,
// 64 items a launch: 59 us wide, 46 us not; 8 layers' q for 16 requests, about 300: 24.4 against 26.8 us; 64 requests on 32 layers'
// q 167 against 194 us, 512 on q, k, v, o of 8 layers 791 against 1084 us.  One projection by itself: 200 requests, about
// 350 items, 21.8 against 20.3 us; 512 requests, about 700, 34.8 against 37.5 us.
constexpr int GEMV_WIDE_MIN_ITEMS = 256, GEMV_WIDE_MIN_ITEMS_ONE_GROUP = 512;
int64_t wide_shrink_items(int32_t n_tok, int32_t rank)
{
    return (int64_t)((n_tok + lora::GEMV_WIDE_SHRINK_TOKENS - 1) / lora::GEMV_WIDE_SHRINK_TOKENS) *
           ((lora::rank_storage(rank) + lora::GEMV_WIDE_ROWS - 1) / lora::GEMV_WIDE_ROWS);
}

// `place` now holds fence `f` (-1: none) instead of the one it held
void hold_fence(lora_cache &c, int32_t &place, int32_t f)
{
    if (f >= 0) ++c.fences[f].holders;
    if (place >= 0) --c.fences[place].holders;
    place = f;
}
// a fence nobody holds; -1 if the runtime gives no more events
int32_t free_fence(lora_cache &c)
{
    for (size_t i = 0; i < c.fences.size(); ++i)
        if (c.fences[(c.next_fence + i) % c.fences.size()].holders == 0) {
            const int32_t f = (int32_t)((c.next_fence + i) % c.fences.size());
            c.next_fence = (size_t)f + 1;
            return f;
        }
    hipEvent_t ev = nullptr;
    const hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        g_last_hip = (int)e;
        return -1;
    }
    c.fences.push_back({ev, 0});
    return (int32_t)c.fences.size() - 1;
}

// the units a tile shrink of projections with sum_h_in input columns runs as, 0: through the run table
int32_t direct_shrink(int32_t n_units, int64_t sum_h_in)
{
    return n_units * 2 * (lora::DIRECT_TOKENS + lora::DIRECT_ROWS) * sum_h_in <= DIRECT_SHRINK_MAX_BYTES ? n_units : 0;
}

// may a tile shrink of n projections, sum_h_in input columns together, be the launch that lists travel with?
bool shrink_copies(const PlanLists *q, int n, int64_t sum_h_in)
{
    return q->n_tiles > 0 && (int64_t)q->n_tiles * n <= PINNED_LISTS_MAX_TILES && (int64_t)direct_shrink(q->n_direct, sum_h_in) * n <= PINNED_LISTS_MAX_DIRECT;
}
// does the GEMV launch of a batch of projections go to the side stream, if there is one?
bool gemv_beside_tiles(const lora_cache &c, const PlanLists *q, int64_t sum_h_in, int64_t sum_h_out)
{
    return q->n_tiles > 0 && q->n_gs > 0 && (double)q->n_tile_tok * c.esize * (double)(sum_h_in + 2 * sum_h_out) >= FORK_MIN_TILE_BYTES;
}

// Work lists on their way into a plan
struct ListBuild {
    lora_worklists_t w{};
    std::vector<int> group_order;
    int64_t n_gs = 0, n_ge = 0, n_wgs = 0, n_wge = 0;
    std::vector<lora::DevItem> direct, panels;
    ShrinkRuns shrink_runs[SHRINK_VARIANTS];
    std::vector<int32_t> lin_tok;
    std::vector<lora::LinearRows> lin_rows;
    std::vector<lora::LinearSeg> lin_segs;
    ~ListBuild() { lora_worklists_free(&w); }
    size_t size(const lora_cache &c, PlanLists &p, bool internal, bool tables, int32_t T, size_t room);
    void write(const lora_cache &c, const PlanLists &p, char *to) const;
};
// Everything but the writing: the bytes the lists take (panels only if they fit into `room`).  Without `tables` the tile shrink has panels alone.
size_t ListBuild::size(const lora_cache &c, PlanLists &p, bool internal, bool tables, int32_t T, size_t room)
{
    // resolve slots: the device copy of an item carries the slot's first storage row, the
    // entry's alpha and the item's first token
    auto stamp = [&](lora_item_t *items, int n) {
        for (int i = 0; i < n; ++i) {
            const Slot &s = c.slots[items[i].slot];
            lora::DevItem d;
            d.tok_off = items[i].tok_off;
            d.n_tok = items[i].n_tok;
            d.row = c.slot_row[items[i].slot];
            d.rank = items[i].rank;
            d.a = items[i].a;
            d.consecutive = 1;
            for (int t = 1; t < items[i].n_tok; ++t)
                if (w.tok_list[items[i].tok_off + t] != w.tok_list[items[i].tok_off] + t) d.consecutive = 0;
            d.alpha = s.alpha;
            d.tok0 = w.tok_list[items[i].tok_off];
            std::memcpy(&items[i], &d, sizeof(d));
        }
    };
    p.n_tile_tok = 0;
    for (int i = 0; i < w.n_tiles; ++i) p.n_tile_tok += w.tiles[i].n_tok;
    // GEMV work items.  A group is worked on in token batches (runs of up to GEMV_BATCH entries of its
    // part of tok_list), every batch with items of its own so that batches run side by side: per batch
    // one shrink item per GEMV_SHRINK_ROWS stored rank rows, and one expand item per run of
    // gemv_expand_width(rank) columns of a super-chunk (the launch repeats it for every super-chunk of
    // the projection).
    // Groups in order of rising rank, whatever the caller's slot numbering (measured on the decode configuration:
    // 10.0 us per layer, 10.5 us with the order reversed).
    group_order.resize((size_t)w.n_groups);
    for (int i = 0; i < w.n_groups; ++i) group_order[i] = i;
    std::stable_sort(group_order.begin(), group_order.end(),
                     [&](int x, int y) { return lora::rank_storage(w.groups[x].rank) < lora::rank_storage(w.groups[y].rank); });
    // how many there are (they are written straight to the staged copy further down)
    for (int gi = 0; gi < w.n_groups; ++gi) {
        const int32_t n = w.groups[gi].n_tok, rank = w.groups[gi].rank, batches = (n + lora::GEMV_BATCH - 1) / lora::GEMV_BATCH;
        n_gs += (int64_t)batches * (lora::rank_storage(rank) / lora::GEMV_SHRINK_ROWS);
        n_ge += (int64_t)batches * (lora::GEMV_SUPER_COLS / lora::gemv_expand_width(rank));
        n_wgs += wide_shrink_items(n, rank);
        n_wge += (int64_t)((n + lora::GEMV_WIDE_TOKENS - 1) / lora::GEMV_WIDE_TOKENS) * (lora::GEMV_SUPER_COLS / lora::gemv_wide_width(rank));
    }
    // the same work as wide items (lora_apply's own plans serve one projection: none where that would not take them)
    if (c.dtype != LORA_BF16 || c.small_scratch || (internal && n_wgs < GEMV_WIDE_MIN_ITEMS_ONE_GROUP)) n_wgs = n_wge = 0;
    stamp(w.tiles, w.n_tiles);
    // the units of a short tile shrink
    if (w.n_tiles > 0) {
        int64_t n = 0;
        auto blocks = [](int32_t v, int32_t by) { return (v + by - 1) / by; };
        for (int i = 0; i < w.n_tiles && n <= c.direct_max; ++i) {
            const lora::DevItem &t = reinterpret_cast<const lora::DevItem *>(w.tiles)[i];
            n += blocks(t.n_tok, lora::DIRECT_TOKENS) * blocks(t.rank, lora::DIRECT_ROWS);
        }
        for (int i = 0; i < w.n_tiles && n <= c.direct_max; ++i) {
            const lora::DevItem &t = reinterpret_cast<const lora::DevItem *>(w.tiles)[i];
            for (int32_t o = 0; o < t.n_tok; o += lora::DIRECT_TOKENS) {
                lora::DevItem d = t;
                d.tok_off += o;
                d.n_tok = std::min(lora::DIRECT_TOKENS, t.n_tok - o);
                d.tok0 = w.tok_list[d.tok_off];
                for (d.a = 0; d.a < t.rank; d.a += lora::DIRECT_ROWS) direct.push_back(d);
            }
        }
    }
    // the panels of a long tile shrink: neighbouring tiles of a slot put together, cut into equal parts of at most lora::PANEL_ROWS rows
    if (c.dtype == LORA_BF16) {
        const lora::DevItem *dev_tiles = reinterpret_cast<const lora::DevItem *>(w.tiles);  // stamped above
        for (int i = 0; i < w.n_tiles;) {
            int32_t n = 0;
            int j = i;
            for (; j < w.n_tiles && dev_tiles[j].row == dev_tiles[i].row && dev_tiles[j].tok_off == dev_tiles[i].tok_off + n; ++j) n += dev_tiles[j].n_tok;
            const int32_t parts = (n + lora::PANEL_ROWS - 1) / lora::PANEL_ROWS, rows = ((n + parts - 1) / parts + 15) / 16 * 16;
            for (int32_t o = 0; o < n; o += rows) {
                lora::DevItem d = dev_tiles[i];
                d.tok_off += o;
                d.n_tok = std::min(rows, n - o);
                d.tok0 = w.tok_list[d.tok_off];
                d.consecutive = 1;
                for (int32_t r = 1; r < d.n_tok && d.consecutive; ++r) d.consecutive = w.tok_list[d.tok_off + r] == d.tok0 + r;
                panels.push_back(d);
            }
            i = j;
        }
        auto runs_of = [](const lora::DevItem &d) { return (d.n_tok + 63) / 64; };
        auto key = [&](const lora::DevItem &d) {
            const int runs = runs_of(d), nb = lora::panel_rank_blocks(d.rank);
            return std::make_pair(lora::panel_projs(runs, nb), -(64 * runs + 16 * nb));
        };
        std::stable_sort(panels.begin(), panels.end(), [&](const lora::DevItem &x, const lora::DevItem &y) { return key(x) < key(y); });
        p.panel_classes = lora::PanelClasses{};
        std::memset(p.panel_count, 0, sizeof(p.panel_count));
        p.panel_sum_bytes = 0;
        for (const auto &d : panels) {
            const int runs = runs_of(d), nb = lora::panel_rank_blocks(d.rank);
            for (int k = lora::panel_projs(runs, nb) - 1; k < 3; ++k) ++p.panel_classes.end[k];
            ++p.panel_count[runs][nb];
            p.panel_sum_bytes += 8.0 * d.n_tok * lora::rank_storage(d.rank);
        }
        p.tile_rows = 0;
        for (int i = 0; i < w.n_tiles; ++i) p.tile_rows += LORA_TILE_TOKENS + (lora::rank_storage(dev_tiles[i].rank) + 15) / 16 * 16;
    }
    // the tile shrink's run tables
    {
        int32_t quanta = INT32_MAX;
        for (const auto &pr : c.proj) quanta = std::min(quanta, (pr.h_in + lora::SHRINK_STAGE_K - 1) / lora::SHRINK_STAGE_K);
        p.shrink_quanta = std::max(1, std::min(quanta, 1 << 14));
        const int64_t slots = std::min<int64_t>(SHRINK_MAX_RUNS, 2 * (int64_t)c.n_cu);
        const lora::DevItem *dev_tiles = reinterpret_cast<const lora::DevItem *>(w.tiles);  // stamped above
        int32_t widest = 0;
        for (const auto &pr : c.proj) widest = std::max(widest, pr.h_in);
        for (int v = 0; v < SHRINK_VARIANTS && tables && w.n_tiles > 0 && c.vpart_rows > 0; ++v) {
            if (internal && (v > 0 || direct_shrink((int32_t)direct.size(), widest) > 0)) break;  // (lora_apply's own plans serve one projection)
            if (v >= SHRINK_VARIANT_BATCH && c.small_scratch) break;
            if (v == SHRINK_VARIANT_SMALL && T > LORA_STATIC_MAX_TOKENS) continue;  // lora_apply_plan_static refuses such a batch
            const int n = v >= SHRINK_VARIANT_SMALL ? 1 : v + 1;
            int64_t max_runs = v >= SHRINK_VARIANT_BATCH ? SHRINK_BATCH_RUNS[v - SHRINK_VARIANT_BATCH] : slots / 8 / n * 8;
            max_runs = std::min(max_runs, (v == SHRINK_VARIANT_SMALL ? STATIC_VPART_ROWS : c.vpart_rows) / (2 * lora::SHRINK_SLOT_ROWS) / n / 8 * 8);
            build_shrink_runs(dev_tiles, w.n_tiles, p.shrink_quanta, (int)std::max<int64_t>(8, max_runs), shrink_runs[v]);
        }
    }

    p.T = T;
    p.n_tok_list = w.n_tok_list;
    p.n_tiles = w.n_tiles;
    p.n_gs = (int32_t)n_gs;
    p.n_ge = (int32_t)n_ge;
    p.n_wgs = (int32_t)n_wgs;
    p.n_wge = (int32_t)n_wge;
    p.off_tiles = align_up(sizeof(int32_t) * (size_t)w.n_tok_list);
    p.off_gs = p.off_tiles + align_up(sizeof(lora_item_t) * (size_t)w.n_tiles);
    p.off_ge = p.off_gs + align_up(sizeof(lora::GemvItem) * (size_t)n_gs);
    // the rows of lora_linear_plan (bf16 caches): tok_list, then the tokens that name no adapter
    if (c.dtype == LORA_BF16 && !internal) {
        std::vector<uint8_t> named((size_t)T, 0);
        lin_tok.assign(w.tok_list, w.tok_list + w.n_tok_list);
        for (int32_t t : lin_tok) named[t] = 1;
        for (int32_t t = 0; t < T; ++t)
            if (!named[t]) lin_tok.push_back(t);
        const lora::DevItem *dev_tiles = reinterpret_cast<const lora::DevItem *>(w.tiles);  // stamped above
        for (int i = 0; i < w.n_tiles; ++i) {
            const lora::DevItem &t = dev_tiles[i];
            if (lin_segs.empty() || lin_segs.back().row != t.row) lin_segs.push_back(lora::LinearSeg{t.tok_off, t.tok_off, t.row, t.rank});
            lin_segs.back().r1 = t.tok_off + t.n_tok;
        }
        size_t s = 0;
        for (int32_t r = 0; r < T; r += LORA_TILE_TOKENS) {
            lora::LinearRows d{};
            d.tok_off = r;
            d.n_tok = std::min<int32_t>(LORA_TILE_TOKENS, T - r);
            d.tok0 = lin_tok[r];
            d.consecutive = 1;
            for (int32_t i = 1; i < d.n_tok; ++i)
                if (lin_tok[r + i] != d.tok0 + i) d.consecutive = 0;
            while (s < lin_segs.size() && lin_segs[s].r1 <= r) ++s;
            d.first_seg = (int32_t)s;
            for (size_t e = s; e < lin_segs.size() && lin_segs[e].r0 < r + d.n_tok; ++e) ++d.n_segs;
            lin_rows.push_back(d);
        }
    }
    p.n_lin_rows = (int32_t)lin_rows.size();
    p.n_lin_segs = (int32_t)lin_segs.size();
    p.off_wgs = p.off_ge + align_up(sizeof(lora::GemvItem) * (size_t)n_ge);
    p.off_wge = p.off_wgs + align_up(sizeof(lora::GemvWideItem) * (size_t)n_wgs);
    p.off_lin_tok = p.off_wge + align_up(sizeof(lora::GemvWideItem) * (size_t)n_wge);
    p.off_lin_rows = p.off_lin_tok + align_up(sizeof(int32_t) * lin_tok.size());
    p.off_lin_segs = p.off_lin_rows + align_up(sizeof(lora::LinearRows) * lin_rows.size());
    p.off_direct = p.off_lin_segs + align_up(sizeof(lora::LinearSeg) * lin_segs.size());
    p.n_direct = (int32_t)direct.size();
    size_t bytes = p.off_direct + align_up(sizeof(lora::DevItem) * direct.size());
    for (int v = 0; v < SHRINK_VARIANTS; ++v) {
        p.shrink_runs[v] = shrink_runs[v].n_runs;
        p.shrink_pieces[v] = shrink_runs[v].any_pieces;
        p.off_cuts[v] = bytes;
        bytes += align_up(sizeof(lora::ShrinkCut) * shrink_runs[v].cuts.size());
        p.off_sums[v] = bytes;
        bytes += align_up(sizeof(lora::ShrinkSum) * shrink_runs[v].sums.size());
    }
    // (A plan's own lists have room for them: compute_layout counts 48 GEMV items for every fourth token, tokens in tiles make none, and there are no more panels than tiles.
    // Lists with tiles besides the plan's own may find none behind it; the plan then does without them.)
    if (bytes + align_up(sizeof(lora::DevItem) * panels.size()) > room) panels.clear();
    p.off_panels = bytes;
    p.n_panels = (int32_t)panels.size();
    return bytes + align_up(sizeof(lora::DevItem) * panels.size());
}
void ListBuild::write(const lora_cache &c, const PlanLists &p, char *to) const
{
    std::memcpy(to, w.tok_list, sizeof(int32_t) * (size_t)w.n_tok_list);
    std::memcpy(to + p.off_tiles, w.tiles, sizeof(lora_item_t) * (size_t)w.n_tiles);
    {
        lora::GemvItem *gs = reinterpret_cast<lora::GemvItem *>(to + p.off_gs), *ge = reinterpret_cast<lora::GemvItem *>(to + p.off_ge);
        lora::GemvWideItem *wgs = reinterpret_cast<lora::GemvWideItem *>(to + p.off_wgs), *wge = reinterpret_cast<lora::GemvWideItem *>(to + p.off_wge);
        for (int gi = 0; gi < w.n_groups; ++gi) {
            const lora_item_t &gr = w.groups[group_order[gi]];
            const int32_t *toks = w.tok_list + gr.tok_off, row = c.slot_row[gr.slot];
            const float alpha = c.slots[gr.slot].alpha;
            lora::GemvItem d;
            d.row = row, d.rank = gr.rank, d.alpha = alpha;
            for (int32_t b0 = 0; b0 < gr.n_tok; b0 += lora::GEMV_BATCH) {
                for (int t = 0; t < lora::GEMV_BATCH; ++t) d.tok[t] = b0 + t < gr.n_tok ? toks[b0 + t] : -1;
                for (int32_t j0 = 0; j0 < lora::rank_storage(gr.rank); j0 += lora::GEMV_SHRINK_ROWS) {
                    d.a = lora::gemv_pack_shrink(j0);
                    *gs++ = d;
                }
                for (int32_t col = 0, nc = lora::gemv_expand_width(gr.rank); col < lora::GEMV_SUPER_COLS; col += nc) {
                    d.a = lora::gemv_pack_expand(col);
                    *ge++ = d;
                }
            }
            if (n_wgs == 0) continue;
            lora::GemvWideItem wd{};
            wd.row = row, wd.rank = gr.rank, wd.alpha = alpha;
            auto take = [&](int32_t b0, int32_t most) {
                wd.n_tok = std::min(most, gr.n_tok - b0);
                for (int t = 0; t < lora::GEMV_WIDE_TOKENS; ++t) wd.tok[t] = toks[b0 + (t < wd.n_tok ? t : 0)];
            };
            for (int32_t b0 = 0; b0 < gr.n_tok; b0 += lora::GEMV_WIDE_SHRINK_TOKENS) {
                take(b0, lora::GEMV_WIDE_SHRINK_TOKENS);
                for (wd.a = 0; wd.a < lora::rank_storage(gr.rank); wd.a += lora::GEMV_WIDE_ROWS) *wgs++ = wd;
            }
            for (int32_t b0 = 0; b0 < gr.n_tok; b0 += lora::GEMV_WIDE_TOKENS) {
                take(b0, lora::GEMV_WIDE_TOKENS);
                for (int32_t col = 0, nc = lora::gemv_wide_width(gr.rank); col < lora::GEMV_SUPER_COLS; col += nc) {
                    wd.a = lora::gemv_pack_expand(col);
                    *wge++ = wd;
                }
            }
        }
    }
    if (!lin_tok.empty()) std::memcpy(to + p.off_lin_tok, lin_tok.data(), sizeof(int32_t) * lin_tok.size());
    if (!lin_rows.empty()) std::memcpy(to + p.off_lin_rows, lin_rows.data(), sizeof(lora::LinearRows) * lin_rows.size());
    if (!direct.empty()) std::memcpy(to + p.off_direct, direct.data(), sizeof(lora::DevItem) * direct.size());
    if (!panels.empty()) std::memcpy(to + p.off_panels, panels.data(), sizeof(lora::DevItem) * panels.size());
    if (!lin_segs.empty()) std::memcpy(to + p.off_lin_segs, lin_segs.data(), sizeof(lora::LinearSeg) * lin_segs.size());
    for (int v = 0; v < SHRINK_VARIANTS; ++v) {
        if (!shrink_runs[v].cuts.empty()) std::memcpy(to + p.off_cuts[v], shrink_runs[v].cuts.data(), sizeof(lora::ShrinkCut) * shrink_runs[v].cuts.size());
        if (!shrink_runs[v].sums.empty()) std::memcpy(to + p.off_sums[v], shrink_runs[v].sums.data(), sizeof(lora::ShrinkSum) * shrink_runs[v].sums.size());
    }
}

// Does a launch for n projections in n_groups groups, sum_width wide together (h_in + h_out), gain by the lists with tiles?
bool list_takes_tiles(const lora_plan &p, int n, int n_groups, double sum_width)
{
    auto wide = [&](int64_t n_wgs) { return n_wgs * n >= (n_groups > 1 ? GEMV_WIDE_MIN_ITEMS : GEMV_WIDE_MIN_ITEMS_ONE_GROUP) ? 1 : 0; };
    const double gemv = GEMV_FIXED_US + p.gemv_cost[wide(p.n_wgs)].us(n, sum_width);
    // More projections than a batch of tiles holds pay for its launches again, and long lists take less than estimated as GEMV: 224 projections of a 7B model, 32 requests of one adapter of rank 16
    // 108 us with tiles and 85 without, 48 of two 238 and 187; 2048 wide, 64 of two of rank 8 101 and 80; 256 requests of four 524 and 880
    const int launches = (n + lora::BATCH_MAX_PROJS - 1) / lora::BATCH_MAX_PROJS;
    const double tiled = launches * (TILE_FIXED_US + (p.rest_groups > 0 ? TILE_BESIDE_GEMV_US : 0.0)) + p.rest_cost[wide(p.rest_wgs)].us(n, sum_width) + p.tile_cost.us(n, sum_width);
    return tiled < (n > lora::GEMV_BATCH_MAX_PROJS ? 0.75 : 0.92) * gemv && tiled + TILED_LISTS_US < gemv;
}
// The same for the base product, which takes the tiles' term along: no expand launch, but a segment of rows costs its blocks 1.3 us for its Bp
bool product_takes_tiles(const lora_cache &c, const lora_plan &p, double width)
{
    const double gemv = GEMV_FIXED_US + LINEAR_TERM_US + p.gemv_cost[p.n_wgs >= GEMV_WIDE_MIN_ITEMS_ONE_GROUP].us(1, width);
    const double rest = p.rest_groups > 0 ? GEMV_FIXED_US + p.rest_cost[p.rest_wgs >= GEMV_WIDE_MIN_ITEMS_ONE_GROUP].us(1, width) : 0.0;
    const double segments = std::max(1.0, p.tile_segs * std::min(1.0, 256.0 / p.tile_tok));  // of a block
    const double tiled = rest + LINEAR_SHRINK_US + 0.4 * p.tile_cost.us(1, width) + 1.3 * segments;
    const double least = LINEAR_MIN_GAIN_US + LISTS_COST_US / (double)(c.n_layers * c.proj.size());
    return tiled + least < gemv;
}
// Does any launch of the cache's projections?  Either estimate rises evenly with the projections and their widths as long as the number of launches and the kind of GEMV items stay, so the
// ends say it: the narrowest and the widest projection, as many as one and two batches with tiles take before more is asked of a list (and the scratch has sets for), and as many as
// still take no wide items.
bool some_launch_takes_tiles(const lora_cache &c, const lora_plan &p)
{
    double ends[2] = {std::numeric_limits<double>::infinity(), 0};
    for (const auto &pr : c.proj) {
        const double width = (double)pr.h_in + pr.h_out;
        ends[0] = std::min(ends[0], width), ends[1] = std::max(ends[1], width);
    }
    auto list_gains = [&](int limit, int n_groups, double width) {
        const int most = std::min(limit, c.n_sets);
        const int from = n_groups > 1 ? GEMV_WIDE_MIN_ITEMS : GEMV_WIDE_MIN_ITEMS_ONE_GROUP;
        auto below_wide = [&](int32_t n_wgs) { return n_wgs > 0 ? std::max(1, std::min(most, (from - 1) / n_wgs)) : most; };
        for (int n : {most, below_wide(p.n_wgs), below_wide(p.rest_wgs)})
            if (list_takes_tiles(p, n, n_groups, n * width)) return true;
        return false;
    };
    for (double width : ends)
        if (product_takes_tiles(c, p, width) || list_gains(lora::GROUP_MAX_PROJS, 1, width) || list_gains(lora::BATCH_MAX_PROJS, 2, width) || list_gains(lora::GEMV_BATCH_MAX_PROJS, 2, width))
            return true;
    return false;
}

// Is there a user plan to make next while the lists of `p` travel with a call?  Where `p` is the only one that is not held, making it anew would have to wait for that call, and
// host and device would take turns; an upload ahead of the call is long done by then.
bool another_free(const lora_cache &c, const lora_plan &p)
{
    return std::any_of(c.plans.begin(), c.plans.begin() + c.n_user_plans, [&](const lora_plan &q) { return &q != &p && !q.in_use; });
}

// What is enqueued on `st` from here on comes behind the calls that may still read the lists in p.dev.
hipError_t wait_for_uses(lora_cache &c, const lora_plan &p, hipStream_t st)
{
    hipError_t e = hipSuccess;
    for (int32_t f : p.last_use)
        if (f >= 0 && e == hipSuccess) e = hipStreamWaitEvent(st, c.fences[f].ev, 0);
    return e;
}
void forget_uses(lora_cache &c, lora_plan &p)
{
    for (int32_t &f : p.last_use) hold_fence(c, f, -1);
}

// Are a plan's lists left with the host until the first launch that works through them, which copies them (or is preceded by their upload, if it is a launch that cannot)?  Only where a call for
// one of the cache's projections, or a list of some, makes such a launch.  Not on a stream that no apply has run on when others have: whoever makes plans on a stream of their own wants the lists in the
// pool by the time a call needs them.  And not over lists that calls without a fence, a graph's replays say, may still read: nothing but the order of `st` is known to keep from them.
bool lists_travel(const lora_cache &c, const lora_plan &p, bool few_waves, hipStream_t st)
{
    if (!c.fencing || !c.side_stream || p.bytes == 0 || p.unfenced) return false;
    if (!p.internal && (!another_free(c, p) || (!c.stream_fence.empty() && c.stream_fence.count(st) == 0))) return false;
    if (p.n_tiles == 0) return few_waves && c.fused_gemv != 0 && p.n_wgs < GEMV_WIDE_MIN_ITEMS;
    return std::any_of(c.proj.begin(), c.proj.end(), [&](const lora_proj_t &pr) {
        for (int n = 1; n <= lora::BATCH_MAX_PROJS; n *= 2)  // (a list of several may shrink another way than a call for one)
            if (shrink_copies(&p, n, n * pr.h_in) && !gemv_beside_tiles(c, &p, n * pr.h_in, n * pr.h_out)) return true;
        return false;
    });
}

// The upload of a plan's lists on `st`, behind what may still read those that lie there.
hipError_t upload_lists(lora_cache &c, lora_plan &p, hipStream_t st)
{
    if (const hipError_t e = wait_for_uses(c, p, st)) return e;
    forget_uses(c, p);
    const hipError_t e = lora::launch_upload(p.dev, p.pinned_dev, p.bytes + p.tiled_bytes, st, p.ev_upload);
    if (e == hipSuccess) p.upload_pending = true;
    else (void)hipStreamSynchronize(st);  // (the error may be an earlier call's, and the launch on its way)
    p.deferred = e != hipSuccess;
    return e;
}

// Validates a batch against the slot table and writes its work lists into plan `p`
// (pinned copy + upload on `st`).
int build_plan(lora_cache &c, lora_plan &p, int32_t T, const int32_t *seg_offsets, const int32_t *seg_slot,
               const int32_t *seg_rank, int32_t n_seg, hipStream_t st)
{
    if (T < 0 || T > c.max_tokens || n_seg < 0 || n_seg > c.max_segments) return LORA_E_INVAL;
    ListBuild lists;
    lora_worklists_t &w = lists.w;
    int rc = lora_index(T, seg_offsets, seg_slot, seg_rank, n_seg, c.mfma_min, &w);
    if (rc != LORA_OK) return rc;
    p.mfma_min_used = c.mfma_min;
    // With the threshold left to the library: the tile path costs two launches more per apply, which a batch with few tile tokens does
    // not earn back.  So: what its tokens cost either way; below, everything stays GEMV; else the batch pays for the tile launches
    // anyway and smaller pools of tokens become tiles too.
    bool may_tile = false;
    p.has_tiled = false;
    p.tiled_bytes = 0;
    if (c.mfma_min_auto && w.n_tiles > 0) {
        double mean_width = 0;
        for (const auto &pr : c.proj) mean_width += (double)pr.h_in + pr.h_out;
        mean_width /= (double)c.proj.size();
        std::unordered_map<int32_t, std::pair<int32_t, int32_t>> of_slot;  // slot -> (tile tokens, rank)
        for (int i = 0; i < w.n_tiles; ++i) {
            auto &e = of_slot[w.tiles[i].slot];
            e.first += w.tiles[i].n_tok;
            e.second = w.tiles[i].rank;
        }
        const bool other = w.n_groups > 0;
        double gemv_us = other ? 0.0 : GEMV_FIXED_US, tile_us = TILE_FIXED_US + (other ? TILE_BESIDE_GEMV_US : 0.0);
        int64_t n_wide = 0;
        for (int i = 0; i < w.n_groups; ++i) n_wide += wide_shrink_items(w.groups[i].n_tok, w.groups[i].rank);
        for (const auto &kv : of_slot) n_wide += wide_shrink_items(kv.second.first, kv.second.second);
        const bool wide = c.dtype == LORA_BF16 && !c.small_scratch && n_wide >= GEMV_WIDE_MIN_ITEMS_ONE_GROUP;
        for (const auto &kv : of_slot) {
            gemv_us += gemv_tokens_us(kv.second.first, kv.second.second, mean_width, wide);
            tile_us += tile_tokens_us(kv.second.first, kv.second.second, mean_width);
        }
        p.mfma_min_used = gemv_us < tile_us ? 0 : LORA_MFMA_MIN_TOKENS_MIXED;
        if (p.mfma_min_used == 0 && c.dtype == LORA_BF16 && !p.internal && !c.small_scratch) {
            may_tile = true;
            p.rest_groups = w.n_groups, p.rest_wgs = p.tile_tok = 0, p.tile_segs = (int32_t)of_slot.size();
            p.tile_cost = p.gemv_cost[0] = p.gemv_cost[1] = p.rest_cost[0] = p.rest_cost[1] = PathCost{};
            for (int i = 0; i < w.n_tiles; ++i) p.tile_cost.add_tile(w.tiles[i].n_tok, w.tiles[i].rank);
            for (int i = 0; i < w.n_groups; ++i) {
                p.rest_wgs += (int32_t)wide_shrink_items(w.groups[i].n_tok, w.groups[i].rank);
                for (int wide_items = 0; wide_items < 2; ++wide_items) p.rest_cost[wide_items].add_gemv(w.groups[i].n_tok, w.groups[i].rank, wide_items);
            }
            for (int wide_items = 0; wide_items < 2; ++wide_items) {
                p.gemv_cost[wide_items] = p.rest_cost[wide_items];
                for (const auto &kv : of_slot) p.gemv_cost[wide_items].add_gemv(kv.second.first, kv.second.second, wide_items);
            }
            for (const auto &kv : of_slot) p.tile_tok += kv.second.first;
        }
        lora_worklists_free(&w);
        rc = lora_index(T, seg_offsets, seg_slot, seg_rank, n_seg, p.mfma_min_used, &w);
        if (rc != LORA_OK) return rc;
    }

    p.slots.clear();
    p.generations.clear();
    auto check = [&](const lora_item_t &it) -> int {
        if (it.slot >= c.n_slots) return LORA_E_INVAL;
        const Slot &s = c.slots[it.slot];
        if (!s.bound) return LORA_E_STATE;
        if (s.rank != it.rank) return LORA_E_INVAL;
        if (p.slots.empty() || p.slots.back() != it.slot) {
            p.slots.push_back(it.slot);
        }
        return LORA_OK;
    };
    for (int i = 0; i < w.n_tiles && rc == LORA_OK; ++i) rc = check(w.tiles[i]);
    for (int i = 0; i < w.n_groups && rc == LORA_OK; ++i) rc = check(w.groups[i]);
    if (rc != LORA_OK) return rc;
    std::sort(p.slots.begin(), p.slots.end());
    p.slots.erase(std::unique(p.slots.begin(), p.slots.end()), p.slots.end());
    for (int32_t s : p.slots) p.generations.push_back(c.slots[s].generation);

    const size_t bytes = lists.size(c, p, p.internal, true, T, c.plan_cap);
    if (bytes > c.plan_cap) return LORA_E_NOMEM;
    std::optional<ListBuild> tiled;  // (a plan without room for them, or for their panels, does without)
    if (may_tile && some_launch_takes_tiles(c, p)) {
        tiled.emplace();
        rc = lora_index(T, seg_offsets, seg_slot, seg_rank, n_seg, LORA_MFMA_MIN_TOKENS_MIXED, &tiled->w);
        if (rc != LORA_OK) return rc;
        const size_t room = c.plan_cap - bytes;
        p.tiled_bytes = tiled->size(c, p.tiled, false, false, T, room);
        p.has_tiled = p.tiled_bytes <= room && p.tiled.n_panels > 0;
        if (!p.has_tiled) p.tiled_bytes = 0;
    }
    // A captured upload would re-read the staged copy on every replay; plans are made outside of captures.
    if (!c.host_only && is_capturing(st)) return LORA_E_STATE;
    // the staged copy may still be the source of an earlier upload; the device copy may still be read
    // by earlier applies
    if (p.upload_pending) {
        const hipError_t e = hipEventSynchronize(p.ev_upload);
        if (e != hipSuccess) {
            g_last_hip = (int)e;
            return LORA_E_HIP;
        }
        p.upload_pending = false;
    }
    if (p.upload_fence >= 0) {  // the launch that read the staged copy and copied it
        const hipError_t e = hipEventSynchronize(c.fences[p.upload_fence].ev);
        if (e != hipSuccess) {
            g_last_hip = (int)e;
            return LORA_E_HIP;
        }
        hold_fence(c, p.upload_fence, -1);
    }
    p.deferred = false;
    if (!c.host_only && p.lists == p.pinned_dev) {  // an earlier apply may still be reading it there
        for (int32_t f : p.last_use)
            if (f >= 0) HIP_TRY(hipEventSynchronize(c.fences[f].ev));
        forget_uses(c, p);
    }
    lists.write(c, p, p.pinned);
    p.bytes = bytes;
    p.build_seq = ++c.plan_builds;
    p.lists = p.dev;
    if (p.has_tiled) {
        tiled->write(c, p.tiled, p.pinned + bytes);
        p.tiled.build_seq = ++c.plan_builds;
        if (!c.host_only) p.tiled.lists = p.dev + bytes;
    }
    int64_t waves = 4 * (int64_t)p.n_gs;  // of a launch for the widest projection
    {
        int32_t supers = 0;
        for (const auto &pr : c.proj) supers = std::max(supers, (pr.h_out + lora::GEMV_SUPER_COLS - 1) / lora::GEMV_SUPER_COLS);
        waves += (int64_t)p.n_ge * supers;
    }
    const bool few_waves = p.n_tiles == 0 && waves <= PINNED_LISTS_MAX_WAVES;
    if (!c.host_only && c.fencing && p.internal && few_waves) {
        p.lists = p.pinned_dev;
    } else if (!c.host_only && lists_travel(c, p, few_waves, st)) {
        p.deferred = true;
    } else if (!c.host_only && bytes) {
        HIP_TRY(upload_lists(c, p, st));
        p.unfenced = false;
    }
    return LORA_OK;
}

// Makes `st` wait for every apply enqueued so far that named the slot.  The fences of the calls that
// used it last (with either scratch) sit in a ring; once such an entry has been taken over by a later call, the latest fence
// of every stream that ever ran applies stands in (stream order covers the older ones).
int wait_for_applies(lora_cache &c, const Slot &s, hipStream_t st)
{
    if (!c.fencing) return LORA_OK;
    bool all = false;
    for (int64_t used : s.last_by) {
        const int e = (int)(used % N_APPLY_EVENTS);
        if (used <= 0) continue;
        if (c.ring_seq[e] == used) HIP_TRY(hipStreamWaitEvent(st, c.fences[c.ring[e]].ev, 0));
        else all = true;
    }
    if (all)
        for (const auto &kv : c.stream_fence) HIP_TRY(hipStreamWaitEvent(st, c.fences[kv.second].ev, 0));
    return LORA_OK;
}

hipEvent_t take_event(lora_cache &c)
{
    if (!c.free_events.empty()) {
        hipEvent_t e = c.free_events.back();
        c.free_events.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// KernelTimer callback: two events from the pool, remembered with the kernel kind.
void timer_pair(void *ctx, int kind, hipEvent_t *start, hipEvent_t *stop)
{
    lora_cache &c = *static_cast<lora_cache *>(ctx);
    lora_cache::Timed t{kind, take_event(c), take_event(c)};
    if (!t.start || !t.stop) return;  // the launch then goes untimed
    c.timed.push_back(t);
    *start = t.start;
    *stop = t.stop;
}

}  // namespace

// ------------------------------------------------------------------------------------------
extern "C" {

const char *lora_strerror(int status)
{
    switch (status) {
        case LORA_OK: return "ok";
        case LORA_E_INVAL: return "invalid argument";
        case LORA_E_STATE: return "cache slot in the wrong state";
        case LORA_E_NOMEM: return "out of pool / plan / host memory";
        case LORA_E_HIP: return "HIP call failed";
        case LORA_E_NOTFOUND: return "adapter not cached";
        case LORA_E_FAULT: return "a kernel of an earlier apply gave up a bounded wait";
        default: return "unknown status";
    }
}

int lora_last_hip_error(void) { return g_last_hip; }

size_t lora_adapter_bytes(int32_t h_in, int32_t h_out, int32_t rank, int32_t dtype)
{
    if (h_in < 1 || h_out < 1 || rank < 1 || (dtype != LORA_F32 && dtype != LORA_BF16)) return 0;
    return (size_t)rank * ((size_t)h_in + (size_t)h_out) * esize_of(dtype);
}

size_t lora_cache_bytes_required(const lora_cache_config_t *cfg)
{
    if (!config_ok(cfg)) return 0;
    lora_cache tmp;
    compute_layout(tmp, cfg, (cfg->flags & LORA_CACHE_SMALL_SCRATCH) != 0);
    return tmp.total;
}

int lora_cache_create(const lora_cache_config_t *cfg, void *dev_pool, size_t dev_pool_bytes, lora_cache_t **out)
{
    if (!out) return LORA_E_INVAL;
    *out = nullptr;
    if (!config_ok(cfg)) return LORA_E_INVAL;
    lora_cache *c = new (std::nothrow) lora_cache;
    if (!c) return LORA_E_NOMEM;
    compute_layout(*c, cfg, (cfg->flags & LORA_CACHE_SMALL_SCRATCH) != 0);
    if (!c->host_only && dev_pool_bytes < c->total) fit_layout(*c, cfg, dev_pool_bytes);
    c->slots.resize(c->n_slots);
    for (int32_t s = 0; s < c->n_slots; ++s) {
        c->slots[s].cls = class_of_slot(*c, s);
        c->slots[s].part.assign((size_t)c->n_layers * c->proj.size(), 0);
    }
    c->plans.resize(c->n_user_plans + N_INTERNAL_PLANS);
    for (size_t i = 0; i < c->plans.size(); ++i) c->plans[i].internal = (int)i >= c->n_user_plans;
    if (c->host_only) {
        // plans are still built (and can be inspected with lora_plan_dump), only never uploaded
        for (auto &p : c->plans) {
            p.pinned = static_cast<char *>(std::malloc(c->plan_cap));
            if (!p.pinned) {
                lora_cache_destroy(c);
                return LORA_E_NOMEM;
            }
        }
        *out = c;
        return LORA_OK;
    }
    if (!dev_pool || (reinterpret_cast<uintptr_t>(dev_pool) & (ALIGN - 1))) {
        delete c;
        return LORA_E_INVAL;
    }
    if (dev_pool_bytes < c->total) {
        delete c;
        return LORA_E_NOMEM;
    }
    c->pool = static_cast<char *>(dev_pool);
    c->pool_bytes = dev_pool_bytes;
    if (hipGetDevice(&c->device) != hipSuccess) {
        g_last_hip = (int)hipGetLastError();
        delete c;
        return LORA_E_HIP;
    }
    {
        int n_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, c->device) == hipSuccess && n_cu > 0) c->n_cu = n_cu;
        else (void)hipGetLastError();
    }
    if (const int rc_s = static_scratch_setup(c->device)) {
        delete c;
        return rc_s;
    }
    if (c->dtype == LORA_BF16) {
        hipError_t e = lora::prepare_mfma_kernels();
        if (e == hipSuccess) e = lora::prepare_linear_kernels();
        if (e != hipSuccess) {
            g_last_hip = (int)e;
            delete c;
            return LORA_E_HIP;
        }
    }

    int rc = LORA_OK;
    // the tagged words must not carry a future launch number by accident: numbers start at 1
    if (hipHostMalloc(reinterpret_cast<void **>(&c->fault_host), 64, hipHostMallocMapped) != hipSuccess ||
        hipHostGetDevicePointer(reinterpret_cast<void **>(&c->fault_dev), c->fault_host, 0) != hipSuccess ||
        (*c->fault_host = 0, false) ||
        hipMemset(c->pool + c->off_vtag, 0, c->vtag_set_bytes * c->n_sets) != hipSuccess ||
        hipMemset(c->pool + c->off_splits, 0, sizeof(lora::SplitState) * N_LINEAR_SPLITS) != hipSuccess) {
        g_last_hip = (int)hipGetLastError();
        delete c;
        return LORA_E_HIP;
    }
    auto fail = [&](hipError_t e) {
        if (e != hipSuccess && rc == LORA_OK) {
            g_last_hip = (int)e;
            rc = LORA_E_HIP;
        }
    };
    for (size_t i = 0; i < c->plans.size() && rc == LORA_OK; ++i) {
        lora_plan &p = c->plans[i];
        p.dev = c->pool + c->off_plans + c->plan_cap * i;
        fail(hipHostMalloc(reinterpret_cast<void **>(&p.pinned), c->plan_cap, hipHostMallocMapped));
        if (rc == LORA_OK) fail(hipHostGetDevicePointer(reinterpret_cast<void **>(const_cast<char **>(&p.pinned_dev)), p.pinned, 0));
        fail(hipEventCreateWithFlags(&p.ev_upload, hipEventDisableTiming));
    }
    for (int i = 0; i < N_STAGES && rc == LORA_OK; ++i) {
        c->stage[i].dev = c->pool + c->off_stage + c->stage_cap * i;
        fail(hipEventCreateWithFlags(&c->stage[i].ev, hipEventDisableTiming));
    }
    std::fill(c->ring, c->ring + N_APPLY_EVENTS, -1);
    // what the ring, the plans (their latest uses, the copy of their lists) and a few streams hold; more streams, more events
    for (size_t i = 0; i < N_APPLY_EVENTS + 3 * c->plans.size() + 8 && rc == LORA_OK; ++i) {
        hipEvent_t ev = nullptr;
        fail(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        if (ev) c->fences.push_back({ev, 0});
    }
    if (rc == LORA_OK && !(c->flags & LORA_CACHE_NO_OVERLAP)) {
        fail(hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking));
        fail(hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming));
        fail(hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming));
    }
    if (rc != LORA_OK) {
        lora_cache_destroy(c);
        return rc;
    }
    *out = c;
    return LORA_OK;
}

int lora_cache_destroy(lora_cache_t *c)
{
    if (!c) return LORA_E_INVAL;
    if (c->host_only) {
        for (auto &p : c->plans) std::free(p.pinned);
    } else {
        for (auto &p : c->plans) {
            if (p.pinned) (void)hipHostFree(p.pinned);
            if (p.ev_upload) (void)hipEventDestroy(p.ev_upload);
        }
        for (auto &s : c->stage)
            if (s.ev) (void)hipEventDestroy(s.ev);
        for (auto &f : c->fences) (void)hipEventDestroy(f.ev);
        if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
        if (c->ev_join) (void)hipEventDestroy(c->ev_join);
        if (c->side_stream) (void)hipStreamDestroy(c->side_stream);
        if (c->upload_stream) (void)hipStreamDestroy(c->upload_stream);
        if (c->fault_host) (void)hipHostFree(c->fault_host);
        for (auto &s : c->slots)
            if (s.fill_ev) (void)hipEventDestroy(s.fill_ev);
        for (auto &t : c->timed) {
            (void)hipEventDestroy(t.start);
            (void)hipEventDestroy(t.stop);
        }
        for (auto &e : c->free_events) (void)hipEventDestroy(e);
    }
    delete c;
    return LORA_OK;
}

// The address under which the device sees pinned (page-locked, mapped) host memory, or null for
// any other kind of pointer.
static const void *device_view_of_pinned(const void *host)
{
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, host) != hipSuccess) {
        (void)hipGetLastError();  // pageable memory is reported as an error by some runtimes
        return nullptr;
    }
    return at.type == hipMemoryTypeHost ? at.devicePointer : nullptr;
}

// End of the pinned host allocation that `host` lies in, or null for any other kind of pointer.
static const char *pinned_end(const void *host)
{
    const void *dev = device_view_of_pinned(host);
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (!dev) return nullptr;
    if (hipMemGetAddressRange(&base, &size, const_cast<void *>(dev)) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return static_cast<const char *>(host) + (static_cast<const char *>(base) + size - static_cast<const char *>(dev));
}

int lora_cache_fill_slot(lora_cache_t *c, int32_t slot, int64_t adapter_id, int32_t rank, float alpha, int32_t layer,
                         int32_t proj, const void *host_A, const void *host_B, void *fill_stream)
{
    const lora_fill_part_t part{layer, proj, host_A, host_B};
    return lora_cache_fill_slot_parts(c, slot, adapter_id, rank, alpha, &part, 1, fill_stream);
}

// Copies parts [0, n) of an adapter into the slot's slabs by way of the staging buffers: as many parts as fit go into
// a buffer back to back (a part's arrays are multiples of 128 bytes), and one kernel repacks them all.  Arrays that
// follow each other in one pinned allocation travel as one copy: a copy has a fixed cost of several us on the engine,
// and an adapter of rank 16 is 256 copies of 128 KB (five adapters of ranks 8 to 128 on 128 parts each, 520 MB: 31.7 ms
// with two copies, a kernel and two events per part; copies of whole buffers: 10.2 ms, the link's rate is 9.1 ms).
static int fill_staged(lora_cache *c, int32_t slot, int32_t rank, const lora_fill_part_t *parts, int32_t n, hipStream_t st)
{
    auto bytes_of = [&](const lora_fill_part_t &q, size_t &a, size_t &b) {
        a = (size_t)rank * c->proj[q.proj].h_in * c->esize;
        b = (size_t)rank * c->proj[q.proj].h_out * c->esize;
    };
    std::vector<int32_t> in_buffer(c->proj.size() * (size_t)c->n_layers, -1);  // per part: the buffer that holds it
    for (int32_t i = 0, buffer = 0; i < n; ++buffer) {
        Stage &sg = c->stage[c->stage_next++ % N_STAGES];
        if (sg.pending) HIP_TRY(hipStreamWaitEvent(st, sg.ev, 0));
        lora::RepackTable t;
        t.n = 0;
        size_t used = 0;
        // the run of host bytes that is not enqueued yet, where it goes, and the end of the allocation it lies in
        const char *run = nullptr, *run_end = nullptr, *alloc_end = nullptr;
        char *to = nullptr;
        auto flush = [&]() -> hipError_t {
            if (!run) return hipSuccess;
            const hipError_t e = hipMemcpyAsync(to, run, (size_t)(run_end - run), hipMemcpyHostToDevice, st);
            run = nullptr;
            return e;
        };
        auto add = [&](const void *host, size_t bytes) -> hipError_t {
            const char *h = static_cast<const char *>(host);
            if (run && h == run_end && h + bytes <= alloc_end) {
                run_end = h + bytes;
            } else {
                const hipError_t e = flush();
                if (e != hipSuccess) return e;
                run = h;
                run_end = h + bytes;
                to = sg.dev + used;
                alloc_end = pinned_end(h);
            }
            used += bytes;
            return hipSuccess;
        };
        for (; i < n && t.n < lora::REPACK_MAX_PARTS; ++i) {
            size_t bytes_a, bytes_b;
            bytes_of(parts[i], bytes_a, bytes_b);
            if (used + bytes_a + bytes_b > c->stage_cap) break;  // (a buffer holds the largest part)
            int32_t &seen = in_buffer[(size_t)parts[i].layer * c->proj.size() + parts[i].proj];
            if (seen == buffer) break;  // the part once more: the later one counts, and a launch's blocks run in no order
            seen = buffer;
            lora::RepackPart &q = t.p[t.n++];
            q.A = sg.dev + used;
            q.B = sg.dev + used + bytes_a;
            q.slab = slab_ptr(*c, parts[i].layer, parts[i].proj, slot);
            q.h_in = c->proj[parts[i].proj].h_in;
            q.h_out = c->proj[parts[i].proj].h_out;
            HIP_TRY(add(parts[i].host_A, bytes_a));
            HIP_TRY(add(parts[i].host_B, bytes_b));
        }
        HIP_TRY(flush());
        HIP_TRY(lora::launch_repack_parts(c->dtype, t, rank, false, st));
        HIP_TRY(hipEventRecord(sg.ev, st));
        sg.pending = true;
    }
    return LORA_OK;
}

// The same without staging: pinned host memory is mapped into the device's address space, the repack kernel reads it over
// PCIe itself (fastest for a fill that has the device to itself; kernels that wait on PCIe reads slow concurrent applies
// down far more than copy engines do).  dev_view: the parts' A and B as the device sees them.
static int fill_direct(lora_cache *c, int32_t slot, int32_t rank, const lora_fill_part_t *parts, int32_t n,
                       const std::vector<const void *> &dev_view, hipStream_t st)
{
    for (int32_t i0 = 0; i0 < n; i0 += lora::REPACK_MAX_PARTS) {
        lora::RepackTable t;
        t.n = std::min<int32_t>(lora::REPACK_MAX_PARTS, n - i0);
        for (int32_t i = 0; i < t.n; ++i) {
            const lora_fill_part_t &q = parts[i0 + i];
            t.p[i].A = dev_view[2 * (size_t)(i0 + i)];
            t.p[i].B = dev_view[2 * (size_t)(i0 + i) + 1];
            t.p[i].slab = slab_ptr(*c, q.layer, q.proj, slot);
            t.p[i].h_in = c->proj[q.proj].h_in;
            t.p[i].h_out = c->proj[q.proj].h_out;
        }
        HIP_TRY(lora::launch_repack_parts(c->dtype, t, rank, true, st));
    }
    return LORA_OK;
}

int lora_cache_fill_slot_parts(lora_cache_t *c, int32_t slot, int64_t adapter_id, int32_t rank, float alpha,
                               const lora_fill_part_t *parts, int32_t n_parts, void *fill_stream)
{
    if (!c || slot < 0 || slot >= c->n_slots || rank < 1 || n_parts < 0 || (n_parts > 0 && !parts)) return LORA_E_INVAL;
    Slot &s = c->slots[slot];
    if (rank > c->class_rank[s.cls]) return LORA_E_INVAL;
    for (int32_t i = 0; i < n_parts; ++i) {
        const lora_fill_part_t &q = parts[i];
        if (q.layer < 0 || q.layer >= c->n_layers || q.proj < 0 || q.proj >= (int32_t)c->proj.size()) return LORA_E_INVAL;
        if (!c->host_only && (!q.host_A || !q.host_B)) return LORA_E_INVAL;
    }
    const bool was_bound = s.bound;
    if (s.bound) {
        if (s.adapter_id != adapter_id || s.rank != rank || s.alpha != alpha) return LORA_E_STATE;
        for (int32_t i = 0; i < n_parts; ++i)  // would overwrite data in use
            if (s.part[(size_t)parts[i].layer * c->proj.size() + parts[i].proj] && s.refcount > 0) return LORA_E_STATE;
    } else if (c->id2slot.find(adapter_id) != c->id2slot.end()) {
        return LORA_E_STATE;  // the adapter is already cached elsewhere
    }
    if (n_parts == 0) return LORA_OK;
    if (!s.bound) {
        s.bound = true;
        s.adapter_id = adapter_id;
        s.rank = rank;
        s.alpha = alpha;
        s.use_count = 0;
        ++s.generation;
        c->id2slot[adapter_id] = slot;
    }
    if (!c->host_only) {
        hipStream_t st = static_cast<hipStream_t>(fill_stream);
        // a HIP failure below must not leave a bound, empty entry behind
        struct Rollback {
            lora_cache *c;
            Slot *s;
            bool armed;
            ~Rollback()
            {
                if (armed) unbind(*c, *s);
            }
        } rollback{c, &s, !was_bound};
        // pinned host arrays as the device sees them (all parts, or the call takes the staged way)
        bool direct = c->direct_fill;
        std::vector<const void *> dev_view;
        if (direct) {
            dev_view.resize(2 * (size_t)n_parts);
            for (int32_t i = 0; i < n_parts && direct; ++i) {
                dev_view[2 * i] = device_view_of_pinned(parts[i].host_A);
                dev_view[2 * i + 1] = device_view_of_pinned(parts[i].host_B);
                if (!dev_view[2 * i] || !dev_view[2 * i + 1] ||
                    ((reinterpret_cast<uintptr_t>(dev_view[2 * i]) | reinterpret_cast<uintptr_t>(dev_view[2 * i + 1])) & 15))
                    direct = false;
            }
        }
        // applies enqueued earlier may still read this slot; an earlier fill of it (of the entry it held before, or of
        // the same part) may still be writing it on another stream
        if (int rc = wait_for_applies(*c, s, st)) return rc;
        if (s.fill_pending) HIP_TRY(hipStreamWaitEvent(st, s.fill_ev, 0));
        if (const int rc = direct ? fill_direct(c, slot, rank, parts, n_parts, dev_view, st) : fill_staged(c, slot, rank, parts, n_parts, st))
            return rc;
        if (!s.fill_ev) HIP_TRY(hipEventCreateWithFlags(&s.fill_ev, hipEventDisableTiming));
        HIP_TRY(hipEventRecord(s.fill_ev, st));
        s.fill_pending = true;
        rollback.armed = false;
    }
    for (int32_t i = 0; i < n_parts; ++i) {
        const lora_fill_part_t &q = parts[i];
        const size_t part = (size_t)q.layer * c->proj.size() + q.proj;
        if (!s.part[part]) {
            s.part[part] = 1;
            ++s.parts_filled;
        }
        ++c->stats.fills;
        c->stats.bytes_filled += (int64_t)rank * (c->proj[q.proj].h_in + c->proj[q.proj].h_out) * c->esize;
    }
    return LORA_OK;
}

int lora_cache_release_slot(lora_cache_t *c, int32_t slot)
{
    if (!c || slot < 0 || slot >= c->n_slots) return LORA_E_INVAL;
    Slot &s = c->slots[slot];
    if (s.refcount > 0) return LORA_E_STATE;
    if (s.bound) ++c->stats.evictions;
    unbind(*c, s);
    return LORA_OK;
}

int lora_cache_slot_ref(lora_cache_t *c, int32_t slot, int32_t delta)
{
    if (!c || slot < 0 || slot >= c->n_slots) return LORA_E_INVAL;
    Slot &s = c->slots[slot];
    if (!s.bound) return LORA_E_STATE;
    if (s.refcount + delta < 0) return LORA_E_STATE;
    s.refcount += delta;
    return LORA_OK;
}

int lora_cache_lookup(lora_cache_t *c, int64_t adapter_id, int32_t *slot, int32_t *rank)
{
    if (!c) return LORA_E_INVAL;
    auto it = c->id2slot.find(adapter_id);
    if (it == c->id2slot.end()) {
        ++c->stats.misses;
        return LORA_E_NOTFOUND;
    }
    ++c->stats.hits;
    if (slot) *slot = it->second;
    if (rank) *rank = c->slots[it->second].rank;
    return LORA_OK;
}

int lora_cache_slot_info(lora_cache_t *c, int32_t slot, lora_slot_info_t *out)
{
    if (!c || !out || slot < 0 || slot >= c->n_slots) return LORA_E_INVAL;
    Slot &s = c->slots[slot];
    out->adapter_id = s.adapter_id;
    out->rank = s.rank;
    out->class_rank = c->class_rank[s.cls];
    out->state = slot_state(*c, s);
    out->refcount = s.refcount;
    out->use_count = s.use_count;
    out->last_used = s.last_used;
    out->alpha = s.alpha;
    out->parts_filled = s.parts_filled;
    return LORA_OK;
}

int lora_cache_slot_state(lora_cache_t *c, int32_t slot, int32_t *state)
{
    if (!c || !state || slot < 0 || slot >= c->n_slots) return LORA_E_INVAL;
    *state = slot_state(*c, c->slots[slot]);
    return LORA_OK;
}

int lora_cache_find_free_slot(lora_cache_t *c, int32_t rank, int32_t *slot)
{
    if (!c || !slot || rank < 1) return LORA_E_INVAL;
    for (size_t k = 0; k < c->class_rank.size(); ++k) {
        if (c->class_rank[k] < rank) continue;
        for (int32_t s = c->class_first[k]; s < c->class_first[k] + c->class_slots[k]; ++s)
            if (!c->slots[s].bound) {
                *slot = s;
                return LORA_OK;
            }
    }
    return LORA_E_NOMEM;
}

int lora_cache_set_policy(lora_cache_t *c, const lora_policy_t *p)
{
    if (!c || !p || !(p->w_freq >= 0) || !(p->w_recency >= 0) || !(p->w_size >= 0) || p->freq_window < 0) return LORA_E_INVAL;
    c->policy = *p;
    return LORA_OK;
}

int lora_cache_get_policy(const lora_cache_t *c, lora_policy_t *p)
{
    if (!c || !p) return LORA_E_INVAL;
    *p = c->policy;
    return LORA_OK;
}

int lora_cache_score(lora_cache_t *c, int32_t slot, double *score)
{
    if (!c || !score || slot < 0 || slot >= c->n_slots) return LORA_E_INVAL;
    if (!c->slots[slot].bound) return LORA_E_STATE;
    *score = eviction_scores(*c)[slot];
    return LORA_OK;
}

int lora_cache_choose_victim(lora_cache_t *c, int32_t rank, const int64_t *queued_ids, int32_t n_queued, int32_t *slot)
{
    if (!c || !slot || rank < 0 || n_queued < 0 || (n_queued > 0 && !queued_ids)) return LORA_E_INVAL;
    const int32_t v = choose_victim(*c, rank, queued_ids, n_queued);
    if (v < 0) return LORA_E_NOMEM;
    *slot = v;
    return LORA_OK;
}

int lora_cache_acquire(lora_cache_t *c, int64_t adapter_id, int32_t rank, float alpha, int32_t pin,
                       const int64_t *queued_ids, int32_t n_queued, int32_t *slot, int32_t *hit)
{
    if (!c || !slot || !hit || rank < 1 || n_queued < 0 || (n_queued > 0 && !queued_ids)) return LORA_E_INVAL;
    if (rank > c->class_rank.back()) return LORA_E_INVAL;
    auto touch = [&](Slot &s) {
        ++c->req_seq;
        if (c->policy.freq_window > 0 && c->req_seq % c->policy.freq_window == 0)
            for (Slot &o : c->slots) o.req_freq *= 0.5;
        s.req_freq += 1.0;
        s.req_last = c->req_seq;
        if (pin) ++s.refcount;
    };
    auto it = c->id2slot.find(adapter_id);
    if (it != c->id2slot.end()) {
        Slot &s = c->slots[it->second];
        if (s.rank != rank) return LORA_E_INVAL;
        ++c->stats.hits;
        touch(s);
        *slot = it->second;
        *hit = 1;
        return LORA_OK;
    }
    int32_t where = -1;
    if (lora_cache_find_free_slot(c, rank, &where) != LORA_OK) {
        where = choose_victim(*c, rank, queued_ids, n_queued);
        if (where < 0) return LORA_E_NOMEM;  // every large-enough entry is used by a running request
        ++c->stats.evictions;
        unbind(*c, c->slots[where]);
    }
    ++c->stats.misses;
    Slot &s = c->slots[where];
    s.bound = true;
    s.adapter_id = adapter_id;
    s.rank = rank;
    s.alpha = alpha;
    s.use_count = 0;
    ++s.generation;
    c->id2slot[adapter_id] = where;
    touch(s);
    *slot = where;
    *hit = 0;
    return LORA_OK;
}

int lora_cache_resident_bytes(const lora_cache_t *c, size_t *bytes)
{
    if (!c || !bytes) return LORA_E_INVAL;
    size_t sum = 0;
    for (const Slot &s : c->slots)
        if (s.bound) sum += entry_bytes(*c, s);
    *bytes = sum;
    return LORA_OK;
}

int lora_cache_trim(lora_cache_t *c, size_t max_bytes, const int64_t *queued_ids, int32_t n_queued, int32_t *n_evicted)
{
    if (!c || n_queued < 0 || (n_queued > 0 && !queued_ids)) return LORA_E_INVAL;
    size_t held = 0;
    lora_cache_resident_bytes(c, &held);
    int32_t n = 0;
    int rc = LORA_OK;
    while (held > max_bytes) {
        const int32_t v = choose_victim(*c, 0, queued_ids, n_queued);
        if (v < 0) {
            rc = LORA_E_NOMEM;  // what is left is in use
            break;
        }
        held -= entry_bytes(*c, c->slots[v]);
        ++c->stats.evictions;
        unbind(*c, c->slots[v]);
        ++n;
    }
    if (n_evicted) *n_evicted = n;
    return rc;
}

int lora_cache_stats(const lora_cache_t *c, lora_cache_stats_t *out)
{
    if (!c || !out) return LORA_E_INVAL;
    *out = c->stats;
    return LORA_OK;
}

int lora_cache_slab(const lora_cache_t *c, int32_t layer, int32_t proj, int32_t slot, void **dev_ptr, size_t *bytes)
{
    if (!c || layer < 0 || layer >= c->n_layers || proj < 0 || proj >= (int32_t)c->proj.size() || slot < 0 ||
        slot >= c->n_slots)
        return LORA_E_INVAL;
    if (dev_ptr)
        *dev_ptr = c->pool ? slab_ptr(*c, layer, proj, slot) : nullptr;
    if (bytes) *bytes = (size_t)lora::rank_storage(c->class_rank[c->slots[slot].cls]) * c->row_bytes[proj];
    return LORA_OK;
}

int lora_cache_set_fencing(lora_cache_t *c, int32_t on)
{
    if (!c) return LORA_E_INVAL;
    c->fencing = on != 0;
    return LORA_OK;
}

int lora_cache_check_fault(lora_cache_t *c, void *stream, int32_t *fault)
{
    if (!c || !fault || c->host_only) return LORA_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamSynchronize(st));
    const int32_t v = __atomic_exchange_n(c->fault_host, 0, __ATOMIC_ACQ_REL);
    *fault = v ? 1 : 0;
    return LORA_OK;
}

int lora_cache_set_timing(lora_cache_t *c, int32_t on)
{
    if (!c || c->host_only) return LORA_E_INVAL;
    c->timing = on != 0;
    return LORA_OK;
}

int lora_cache_read_timing(lora_cache_t *c, double ms[LORA_K_COUNT], int64_t launches[LORA_K_COUNT])
{
    if (!c || !ms || !launches) return LORA_E_INVAL;
    for (int k = 0; k < LORA_K_COUNT; ++k) {
        ms[k] = 0.0;
        launches[k] = 0;
    }
    int rc = LORA_OK;
    for (auto &t : c->timed) {
        float el = 0.f;
        hipError_t e = hipEventSynchronize(t.stop);
        if (e == hipSuccess) e = hipEventElapsedTime(&el, t.start, t.stop);
        if (e == hipSuccess) {
            ms[t.kind] += el;
            ++launches[t.kind];
        } else {
            g_last_hip = (int)e;
            rc = LORA_E_HIP;
        }
        c->free_events.push_back(t.start);
        c->free_events.push_back(t.stop);
    }
    c->timed.clear();
    return rc;
}

int lora_plan_create(lora_cache_t *c, int32_t T, const int32_t *seg_offsets, const int32_t *seg_slot,
                     const int32_t *seg_rank, int32_t n_seg, void *stream, lora_plan_t **out)
{
    if (!c || !out) return LORA_E_INVAL;
    *out = nullptr;
    lora_plan *p = nullptr;
    for (int i = 0; i < c->n_user_plans && !p; ++i) {  // in turns: making one waits for the upload of the lists it held before
        lora_plan &q = c->plans[(c->user_next + i) % c->n_user_plans];
        if (!q.in_use) p = &q;
    }
    if (!p) return LORA_E_NOMEM;
    const int rc = build_plan(*c, *p, T, seg_offsets, seg_slot, seg_rank, n_seg, static_cast<hipStream_t>(stream));
    if (rc != LORA_OK) return rc;
    c->user_next = (uint64_t)(p - c->plans.data()) + 1;
    p->in_use = true;
    *out = p;
    return LORA_OK;
}

int lora_plan_destroy(lora_cache_t *c, lora_plan_t *p)
{
    if (!c || !p || p->internal || !p->in_use) return LORA_E_INVAL;
    if (p < c->plans.data() || p >= c->plans.data() + c->n_user_plans) return LORA_E_INVAL;
    p->in_use = false;
    return LORA_OK;
}

int lora_plan_info(const lora_plan_t *p, lora_plan_info_t *out)
{
    if (!p || !out || !p->in_use) return LORA_E_INVAL;
    out->T = p->T;
    out->mfma_min_tokens = p->mfma_min_used;
    out->n_tiles = p->n_tiles;
    out->n_tile_tokens = p->n_tile_tok;
    out->n_gemv_shrink_items = p->n_gs;
    out->n_gemv_expand_items = p->n_ge;
    return LORA_OK;
}

static int32_t supers_of(int32_t h_out) { return (h_out + lora::GEMV_SUPER_COLS - 1) / lora::GEMV_SUPER_COLS; }

// Block and unit numbers of a batch's GEMV launch for n projections, h_out[i] wide, with a plan's items or its wide items;
// shared by the launches and lora_plan_dump.  `marks` comes in zeroed: the projection of every step-th super-chunk, four to a word; first[i]: number of projection i's first super-chunk.
static int gemv_batch_map(const PlanLists *p, bool wide, int n, const int32_t *h_out, lora::GemvBatchMap &m, uint32_t *marks, int32_t max_supers, int step, uint32_t *first)
{
    m.n_gs = (uint32_t)(wide ? p->n_wgs : p->n_gs);
    m.n_ge = (uint32_t)(wide ? p->n_wge : p->n_ge);
    m.n_proj = (uint32_t)n;
    m.by_xcd = m.n_gs >= lora::GEMV_BATCH_XCD_ITEMS;
    m.shrink_blocks = m.by_xcd ? (m.n_gs + 7) & ~7u : m.n_gs;
    m.div_shrink = lora::div24_of(m.shrink_blocks);
    m.div_ge = lora::div24_of(m.n_ge);
    int32_t n_super = 0;
    for (int i = 0; i < n; ++i) {
        if (supers_of(h_out[i]) > 255) return LORA_E_INVAL;  // as a group's launch
        first[i] = (uint32_t)n_super;
        const int32_t end = n_super + supers_of(h_out[i]);
        if (end > max_supers) return LORA_E_INVAL;  // (the caller cuts batches by batch_limits)
        for (int32_t k = (n_super + step - 1) / step; k * step < end; ++k) marks[k >> 2] |= (uint32_t)i << (8 * (k & 3));
        n_super = end;
    }
    const int64_t units = (int64_t)m.n_ge * n_super;
    if (units >= (1 << 24) || (int64_t)m.shrink_blocks * n >= (1 << 24)) return LORA_E_INVAL;  // beyond the kernels' unit arithmetic
    m.n_units = (uint32_t)units;
    return LORA_OK;
}

static Scratch pool_scratch(lora_cache_t *c)
{
    return Scratch{c->pool + c->off_v, c->v_set_bytes, c->n_sets, c->pool + c->off_vpart, c->vpart_rows, false,
                   c->pool + c->off_vtag, c->vtag_set_bytes, &c->tag_epoch, &c->cap_id, &c->cap_plan, &c->cap_sets};
}

// How many projections, and super-chunks of projections, a batch with plan p may have: the scratch's sets, the partial sums of the
// smallest run table of the tile shrink, and the ranges of the GEMV launch's unit arithmetic.
static void batch_limits(const PlanLists *p, const Scratch &sc, bool long_batch, int32_t &max_projs, int32_t &max_supers)
{
    int64_t projs = std::min(sc.n_sets, long_batch ? lora::GEMV_LONG_MAX_PROJS : lora::GEMV_BATCH_MAX_PROJS);
    int64_t supers = long_batch ? lora::GEMV_LONG_MAX_SUPERS : lora::GEMV_BATCH_MAX_SUPERS;
    if (p->n_tiles > 0) {
        projs = std::min<int64_t>(projs, lora::BATCH_MAX_PROJS);
        projs = std::min(projs, sc.vpart_rows / (2 * lora::SHRINK_SLOT_ROWS * std::max<int64_t>(1, p->shrink_runs[SHRINK_VARIANTS - 1])));
        projs = std::max<int64_t>(projs, lora::GROUP_MAX_PROJS);  // (up to a group's size there are tables of their own)
    }
    if (p->n_gs > 0) {
        projs = std::max<int64_t>(1, std::min<int64_t>(projs, ((1 << 24) - 1) / (p->n_gs + 7)));
        supers = std::min<int64_t>(supers, ((1 << 24) - 1) / std::max({1, p->n_ge, p->n_wge}));
    }
    max_projs = (int32_t)projs;
    max_supers = (int32_t)supers;
}

static int tile_setup(const lora_cache_t *c, const PlanLists *p, int n, int64_t sum_h_in, const Scratch &sc, float scale, lora::TileBatch &tb);
static void choose_panels(const lora_cache_t *c, const PlanLists *p, const Scratch &sc, lora::TileBatch &tb);

// The units of a plan's own lists, or of those with tiles that it has besides
static int dump_units(lora_cache_t *c, const lora_plan_t *plan, bool tiled, int32_t proj, lora_plan_unit_t *units, int32_t cap_units, int32_t *n_units, int32_t *toks, int32_t cap_toks,
                      int32_t *n_toks)
{
    if (!c || !plan || !plan->in_use || !n_units || !n_toks || proj < 0 || proj >= (int32_t)c->proj.size() || cap_units < 0 ||
        cap_toks < 0 || (cap_units > 0 && !units) || (cap_toks > 0 && !toks))
        return LORA_E_INVAL;
    if (tiled && !plan->has_tiled) {
        *n_units = *n_toks = 0;
        return LORA_OK;
    }
    const PlanLists *const p = tiled ? &plan->tiled : plan;
    const size_t at = tiled ? plan->bytes : 0, bytes = tiled ? plan->tiled_bytes : plan->bytes;
    // the bytes the kernels read
    std::vector<char> copy;
    const char *buf = plan->pinned + at;
    if (!c->host_only && !plan->deferred) {
        copy.resize(bytes);
        if (plan->upload_pending) HIP_TRY(hipEventSynchronize(plan->ev_upload));
        if (plan->upload_fence >= 0) HIP_TRY(hipEventSynchronize(c->fences[plan->upload_fence].ev));
        if (bytes) HIP_TRY(hipMemcpy(copy.data(), plan->dev + at, bytes, hipMemcpyDeviceToHost));
        buf = copy.data();
    }
    const int32_t *tok_list = reinterpret_cast<const int32_t *>(buf);
    const lora::DevItem *tiles = reinterpret_cast<const lora::DevItem *>(buf + p->off_tiles);
    const lora::GemvItem *gs = reinterpret_cast<const lora::GemvItem *>(buf + p->off_gs);
    const lora::GemvItem *ge = reinterpret_cast<const lora::GemvItem *>(buf + p->off_ge);
    const int32_t *lin_tok = reinterpret_cast<const int32_t *>(buf + p->off_lin_tok);
    const lora::LinearRows *lin_rows = reinterpret_cast<const lora::LinearRows *>(buf + p->off_lin_rows);
    const lora::LinearSeg *lin_segs = reinterpret_cast<const lora::LinearSeg *>(buf + p->off_lin_segs);

    int32_t nu = 0, nt = 0;
    auto slot_of_row = [&](int32_t row) -> int32_t {
        auto it = std::upper_bound(c->slot_row.begin(), c->slot_row.end(), row);
        return (int32_t)(it - c->slot_row.begin()) - 1;
    };
    auto put_tok = [&](int32_t t) {
        if (nt < cap_toks) toks[nt] = t;
        ++nt;
    };
    auto put_unit = [&](int32_t kind, int32_t tok_off, int32_t n_tok, int32_t row, int32_t rank, int32_t lo, int32_t hi,
                        int32_t where, float alpha) {
        if (nu < cap_units) units[nu] = lora_plan_unit_t{kind, tok_off, n_tok, row >= 0 ? slot_of_row(row) : -1, rank, lo, hi, where, alpha};
        ++nu;
    };
    // tokens of a tile as the tile kernels find them: a run from tok0, or through the token list
    auto tile_tokens = [&](const lora::DevItem &it, const int32_t *list) {
        for (int32_t i = 0; i < it.n_tok; ++i) put_tok(lora::tile_token_of(list, it, i));
    };
    std::vector<int32_t> tile_off((size_t)p->n_tiles, 0);
    for (int32_t i = 0; i < p->n_tiles; ++i) {
        tile_off[i] = nt;
        tile_tokens(tiles[i], tok_list);
        put_unit(LORA_UNIT_TILE, tile_off[i], tiles[i].n_tok, tiles[i].row, tiles[i].rank, 0, 0, 0, tiles[i].alpha);
    }
    // the units of a short tile shrink
    const lora::DevItem *direct = reinterpret_cast<const lora::DevItem *>(buf + p->off_direct);
    for (int32_t i = 0; i < p->n_direct; ++i) {
        const int32_t off = nt;
        tile_tokens(direct[i], tok_list);
        put_unit(LORA_UNIT_DIRECT_SHRINK, off, direct[i].n_tok, direct[i].row, direct[i].rank, direct[i].a, std::min(direct[i].a + lora::DIRECT_ROWS, direct[i].rank),
                 direct_shrink(p->n_direct, c->proj[proj].h_in) > 0 ? 1 : 0, direct[i].alpha);
    }
    // the blocks of the shrink by panels, for groups of 1 to 4 projections, as the kernel maps them
    const lora::DevItem *panels = reinterpret_cast<const lora::DevItem *>(buf + p->off_panels);
    for (int gn = 1; gn <= lora::GROUP_MAX_PROJS; ++gn)
        for (int b = 0; b < lora::panel_blocks(p->panel_classes, gn) && p->n_panels > 0; ++b) {
            int slice, panel, first, n;
            if (!lora::panel_of_block(p->panel_classes, gn, 1, b, slice, panel, first, n)) continue;
            const int32_t off = nt;
            tile_tokens(panels[panel], tok_list);
            put_unit(LORA_UNIT_PANEL_SHRINK, off, panels[panel].n_tok, panels[panel].row, panels[panel].rank, first, first + n, gn, panels[panel].alpha);
        }
    // how a launch for 1 to 4 such projections that read the same x does the shrink
    for (int gn = 1; gn <= lora::GROUP_MAX_PROJS && p->n_tiles > 0; ++gn) {
        lora::TileBatch tb;
        const Scratch sc = pool_scratch(c);
        if (tile_setup(c, p, gn, (int64_t)gn * c->proj[proj].h_in, sc, 1.f, tb) != LORA_OK) continue;
        for (int i = 0; i < gn; ++i) tb.p[i].h_in = c->proj[proj].h_in, tb.group[i] = (uint32_t)gn << 8;
        choose_panels(c, p, sc, tb);
        put_unit(LORA_UNIT_SHRINK_WAY, nt, 0, -1, 0, tb.n_direct > 0 ? 0 : tb.n_panels > 0 ? 2 : 1, tb.n_panels > 0 ? tb.slices[0] : 1, gn, 0.f);
    }
    // the tile shrink's pieces for this projection's h_in, per run table, walked as the kernel walks them; and the
    // scratch slots the reduce adds up per tile
    for (int v = 0; v < SHRINK_VARIANTS && p->n_tiles > 0; ++v) {
        if (p->shrink_runs[v] == 0) continue;  // (no such table: the batch is too large for the call it serves)
        const lora::ShrinkCut *cuts = reinterpret_cast<const lora::ShrinkCut *>(buf + p->off_cuts[v]);
        const lora::ShrinkSum *sums = reinterpret_cast<const lora::ShrinkSum *>(buf + p->off_sums[v]);
        const int32_t quanta = p->shrink_quanta, h_in = c->proj[proj].h_in, SK = lora::SHRINK_STAGE_K;
        for (int32_t r = 0; r < p->shrink_runs[v]; ++r) {
            const lora::ShrinkCut from = cuts[r], to = cuts[r + 1];
            const int32_t last_tile = std::min(to.part > 0 ? to.tile : to.tile - 1, p->n_tiles - 1);
            for (int32_t t = from.tile; t <= last_tile; ++t) {
                const int32_t lo = t == from.tile ? from.part : 0, hi = t == to.tile ? to.part : quanta;
                if (lo >= hi) continue;
                const int32_t k_begin = lora::shrink_part_stage(lo, quanta, h_in, SK) * SK;
                const int32_t k_end = std::min(h_in, lora::shrink_part_stage(hi, quanta, h_in, SK) * SK);
                const bool whole = lo == 0 && hi == quanta;
                put_unit(LORA_UNIT_TILE_SHRINK, tile_off[t], tiles[t].n_tok, tiles[t].row, tiles[t].rank, k_begin, k_end,
                         (v << 20) | r, whole ? -1.f : (float)lora::shrink_slot(r, from.tile, t));
            }
        }
        for (int32_t t = 0; t < p->n_tiles; ++t)
            for (int32_t j = 0; j < sums[t].n_pieces && sums[t].n_pieces > 1; ++j)
                put_unit(LORA_UNIT_TILE_SUM, tile_off[t], tiles[t].n_tok, tiles[t].row, tiles[t].rank, j, sums[t].n_pieces, v << 20,
                         (float)(j == 0 ? sums[t].first_slot : 2 * (sums[t].first_slot / 2 + j)));
    }
    auto gemv_tokens = [&](const lora::GemvItem &it) -> int32_t {
        int32_t n = 0;
        for (int t = 0; t < lora::GEMV_BATCH; ++t)
            if (it.tok[t] >= 0) {
                put_tok(it.tok[t]);
                ++n;
            }
        return n;
    };
    // the GEMV launch of this projection alone: blocks and units mapped to items as the kernel maps them
    for (uint32_t b = 0; b < (uint32_t)p->n_gs; ++b) {
        uint32_t item, pj;
        lora::gemv_shrink_block(b, (uint32_t)p->n_gs, 1u, item, pj);
        int32_t j0, n;
        lora::gemv_shrink_rows(gs[item], j0, n);
        const int32_t off = nt, cnt = gemv_tokens(gs[item]);
        put_unit(LORA_UNIT_GEMV_SHRINK, off, cnt, gs[item].row, gs[item].rank, j0, j0 + n, (int32_t)b, gs[item].alpha);
    }
    lora::GemvMap gm{};
    const int32_t h_out = c->proj[proj].h_out, n_super = (h_out + lora::GEMV_SUPER_COLS - 1) / lora::GEMV_SUPER_COLS;
    for (int i = 0; i < lora::GEMV_MAX_PROJS; ++i) {
        gm.unit_end[i] = p->n_ge * n_super;
        gm.n_super_packed |= (uint32_t)n_super << (8 * i);
        gm.super_magic[i] = lora::gemv_magic((uint32_t)n_super);
    }
    for (uint32_t u = 0; u < (uint32_t)gm.unit_end[0]; ++u) {
        uint32_t pj, item, sc;
        lora::gemv_expand_unit(u, gm, pj, item, sc);
        int32_t c0, c1;
        lora::gemv_expand_cols(ge[item], (int32_t)sc, h_out, c0, c1);
        if (c0 >= c1) continue;  // the wavefront returns at once
        const int32_t off = nt, cnt = gemv_tokens(ge[item]);
        put_unit(LORA_UNIT_GEMV_EXPAND, off, cnt, ge[item].row, ge[item].rank, c0, c1, 0, ge[item].alpha);
    }
    // the GEMV launch of a batch: every projection of up to two layers, with the items above and with the wide ones, as the
    // kernels of a batch map blocks and units
    const lora::GemvWideItem *wgs = reinterpret_cast<const lora::GemvWideItem *>(buf + p->off_wgs);
    const lora::GemvWideItem *wge = reinterpret_cast<const lora::GemvWideItem *>(buf + p->off_wge);
    const int32_t n_proj = (int32_t)c->proj.size();
    int32_t widths[lora::GEMV_BATCH_MAX_PROJS], entries = 0, supers_left, max_entries;
    batch_limits(p, pool_scratch(c), false, max_entries, supers_left);
    for (; entries < std::min(max_entries, std::min(c->n_layers, 2) * n_proj); ++entries) {
        widths[entries] = c->proj[entries % n_proj].h_out;
        supers_left -= supers_of(widths[entries]);
        if (supers_left < 0) break;
    }
    for (int wide = 0; wide < 2; ++wide) {
        lora::GemvBatchMap m{};
        uint32_t supers[lora::GEMV_BATCH_MAX_SUPERS / 4] = {0}, first[lora::GEMV_BATCH_MAX_PROJS];
        if ((wide ? p->n_wgs : p->n_gs) == 0 || entries == 0 || gemv_batch_map(p, wide != 0, entries, widths, m, supers, lora::GEMV_BATCH_MAX_SUPERS, 1, first)) continue;
        auto put = [&](int32_t kind, const lora::GemvItem *it, const lora::GemvWideItem *w, int32_t lo, int32_t hi, uint32_t e) {
            const int32_t off = nt;
            int32_t cnt = w ? w->n_tok : gemv_tokens(*it);
            for (int32_t t = 0; w && t < cnt; ++t) put_tok(w->tok[t]);
            put_unit(kind, off, cnt, w ? w->row : it->row, w ? w->rank : it->rank, lo, hi, (int32_t)e, w ? w->alpha : it->alpha);
        };
        for (uint32_t b = 0; b < m.n_proj * m.shrink_blocks; ++b) {
            uint32_t e, item;
            lora::gemv_batch_shrink(b, m, e, item);
            if (item >= m.n_gs || (int32_t)e % n_proj != proj) continue;
            if (wide) {
                put(LORA_UNIT_WIDE_SHRINK, nullptr, wgs + item, wgs[item].a, wgs[item].a + lora::gemv_wide_rows(wgs[item].rank, wgs[item].a), e);
            } else {
                int32_t j0, n;
                lora::gemv_shrink_rows(gs[item], j0, n);
                put(LORA_UNIT_BATCH_SHRINK, gs + item, nullptr, j0, j0 + n, e);
            }
        }
        for (uint32_t u = 0; u < m.n_units; ++u) {
            uint32_t super, item;
            lora::gemv_batch_unit(u, m, super, item);
            uint32_t e = lora::gemv_super(supers, super), sc;
            if ((int32_t)e % n_proj != proj) continue;
            const lora::BatchProj q = lora::gemv_entry_proj(lora::gemv_entry({nullptr, nullptr, nullptr, c->proj[proj].h_in, widths[e]}, first[e]), sc);
            sc = super - sc;
            if (q.h_out != h_out) continue;  // (what the kernels decode is this projection's width)
            int32_t c0, c1;
            if (wide) lora::gemv_wide_cols(wge[item].rank, wge[item].a, (int32_t)sc, h_out, c0, c1);
            else lora::gemv_expand_cols(ge[item], (int32_t)sc, h_out, c0, c1);
            if (c0 >= c1) continue;
            if (wide) put(LORA_UNIT_WIDE_EXPAND, nullptr, wge + item, c0, c1, e);
            else put(LORA_UNIT_BATCH_EXPAND, ge + item, nullptr, c0, c1, e);
        }
    }
    // the rows of lora_linear_plan: per tile the rows that a segment makes of it (a row outside it is left out), then
    // the others in runs
    auto linear_row = [&](int32_t r) {
        int32_t ti[1] = {r % LORA_TILE_TOKENS}, tok[1];
        lora::tile_tokens_of(lin_tok, lin_rows[r / LORA_TILE_TOKENS], ti, -1, tok);
        put_tok(tok[0]);
    };
    auto segment_of = [&](int32_t r) -> const lora::LinearSeg * {
        const lora::LinearRows &lr = lin_rows[r / LORA_TILE_TOKENS];
        for (int32_t s = lr.first_seg; s < lr.first_seg + lr.n_segs; ++s)
            if (lin_segs[s].r0 <= r && r < lin_segs[s].r1) return lin_segs + s;
        return nullptr;
    };
    for (int32_t i = 0; i < p->n_tiles && p->n_lin_rows > 0; ++i) {
        const int32_t off = nt, r0 = tiles[i].tok_off;
        const lora::LinearSeg *seg = segment_of(r0);
        for (int32_t r = r0; r < r0 + tiles[i].n_tok; ++r)
            if (seg && segment_of(r) == seg) linear_row(r);
        put_unit(LORA_UNIT_LINEAR_ROWS, off, nt - off, seg ? seg->row : -1, seg ? seg->rank : 0, 0, 0, 2, tiles[i].alpha);
    }
    for (int32_t mark = 1; mark >= 0 && p->n_lin_rows > 0; --mark) {
        const int32_t from = mark ? p->n_tile_tok : p->n_tok_list, to = mark ? p->n_tok_list : p->T;
        for (int32_t r0 = from; r0 < to; r0 += LORA_TILE_TOKENS) {
            const int32_t off = nt;
            for (int32_t r = r0; r < std::min(to, r0 + LORA_TILE_TOKENS); ++r)
                if (!segment_of(r)) linear_row(r);
            put_unit(LORA_UNIT_LINEAR_ROWS, off, nt - off, -1, 0, 0, 0, mark, 0.f);
        }
    }
    if (p->n_lin_rows > 0) {
        const lora::LinearShape sh = lora::linear_shape(p->T, c->proj[proj].h_in, c->proj[proj].h_out, c->vpart_bytes, N_LINEAR_SPLITS, c->n_cu);
        put_unit(LORA_UNIT_LINEAR_SHAPE, nt, 0, -1, 0, sh.rows, sh.tiles, sh.split << 8 | sh.parts, (float)sh.ring);
    }
    *n_units = nu;
    *n_toks = nt;
    return LORA_OK;
}

int lora_plan_dump(lora_cache_t *c, const lora_plan_t *p, int32_t proj, lora_plan_unit_t *units, int32_t cap_units, int32_t *n_units, int32_t *toks, int32_t cap_toks, int32_t *n_toks)
{
    return dump_units(c, p, false, proj, units, cap_units, n_units, toks, cap_toks, n_toks);
}

int lora_plan_dump_tiled(lora_cache_t *c, const lora_plan_t *p, int32_t proj, lora_plan_unit_t *units, int32_t cap_units, int32_t *n_units, int32_t *toks, int32_t cap_toks, int32_t *n_toks)
{
    return dump_units(c, p, true, proj, units, cap_units, n_units, toks, cap_toks, n_toks);
}

static int validate_apply(lora_cache_t *c, lora_plan_t *p, int32_t layer, int32_t proj, const void *x, void *base_out)
{
    if (c->fault_host && __atomic_load_n(c->fault_host, __ATOMIC_ACQUIRE)) return LORA_E_FAULT;
    if (layer < 0 || layer >= c->n_layers || proj < 0 || proj >= (int32_t)c->proj.size()) return LORA_E_INVAL;
    if (p->T > 0 && (!x || !base_out || !aligned16(x) || !aligned16(base_out))) return LORA_E_INVAL;
    const size_t part = (size_t)layer * c->proj.size() + proj;
    for (size_t i = 0; i < p->slots.size(); ++i) {
        const Slot &s = c->slots[p->slots[i]];
        if (!s.bound || s.generation != p->generations[i] || !s.part[part]) return LORA_E_STATE;
    }
    return LORA_OK;
}

// shrink items up to which the one-launch GEMV form is chosen: measured faster than two launches up to
// 7726 items (2048 one-token requests over 300 adapters: 83 against 86 us); not measured beyond
constexpr int FUSED_GEMV_MAX_ITEMS = 8192;
// The same for a batch, whose shrink blocks are long done when its expand blocks are dispatched: one launch up to the range of the
// unit arithmetic (64 requests on 32 projections, 15808 items: 167 against 180 us; 512 requests, 91328 items: 792 against 803 us).
constexpr int FUSED_GEMV_MAX_BATCH_ITEMS = 1 << 24;
// The run table of a tile-shrink launch for a batch of n projections whose partial sums go to a scratch of `vpart_rows`
// rows: the table of a group's size, or, for more projections, the largest that keeps the launch within
// SHRINK_BATCH_BLOCKS blocks.
static int shrink_variant(const PlanLists *p, int n, int64_t vpart_rows, bool small)
{
    if (small) return SHRINK_VARIANT_SMALL;
    if (n <= lora::GROUP_MAX_PROJS) return n - 1;
    const int order[] = {0, 1, 2, 3, SHRINK_VARIANT_BATCH, SHRINK_VARIANT_BATCH + 1};  // falling number of runs
    for (int v : order)
        if (p->shrink_runs[v] * n <= SHRINK_BATCH_BLOCKS && 2 * (int64_t)lora::SHRINK_SLOT_ROWS * p->shrink_runs[v] * n <= vpart_rows) return v;
    return SHRINK_VARIANT_BATCH + 1;
}
// The tile kernels' arguments but for the projections; n: how many there are, sum_h_in: the sum of their input widths.
static int tile_setup(const lora_cache_t *c, const PlanLists *p, int n, int64_t sum_h_in, const Scratch &sc, float scale, lora::TileBatch &tb)
{
    if (n < 1 || n > lora::BATCH_MAX_PROJS || n > sc.n_sets) return LORA_E_INVAL;
    const int v = shrink_variant(p, n, sc.vpart_rows, sc.small);
    tb.n = n;
    tb.n_runs = p->shrink_runs[v];
    tb.n_direct = direct_shrink(p->n_direct, sum_h_in);
    if (p->n_tiles > 0 && tb.n_runs == 0 && tb.n_direct == 0 && (p->n_panels == 0 || sc.small)) return LORA_E_STATE;  // the plan carries no such table
    tb.quanta = p->shrink_quanta;
    tb.n_tiles = p->n_tiles;
    tb.v_stride = c->v_stride;
    tb.any_pieces = p->shrink_pieces[v] ? 1 : 0;
    tb.scale = scale;
    tb.direct = reinterpret_cast<const lora::DevItem *>(p->lists + p->off_direct);
    tb.tiles = reinterpret_cast<const lora::DevItem *>(p->lists + p->off_tiles);
    tb.cuts = reinterpret_cast<const lora::ShrinkCut *>(p->lists + p->off_cuts[v]);
    tb.sums = reinterpret_cast<const lora::ShrinkSum *>(p->lists + p->off_sums[v]);
    tb.tok_list = reinterpret_cast<const int32_t *>(p->lists);
    tb.v = reinterpret_cast<float *>(sc.v);
    tb.part = reinterpret_cast<float *>(sc.vpart);
    tb.v_set = sc.v_set_bytes / sizeof(float);
    tb.n_panels = 0;
    const int64_t rows_per_proj = 2 * (int64_t)lora::SHRINK_SLOT_ROWS * tb.n_runs;
    if (rows_per_proj * n > sc.vpart_rows) return LORA_E_NOMEM;
    tb.v_set = sc.v_set_bytes / sizeof(float);
    tb.part_set = (uint64_t)rows_per_proj * c->v_stride;
    return LORA_OK;
}
// The shrink of a launch by panels, where that is the shorter way, and into how many k slices: estimates in microseconds, fitted to launches of one to four projections, of a projection of
// four layers and of all seven of two, 300 to 7600 tokens in prompts of 16 to 2048 at ranks 16, 128 and 8 to 128, 2048 to 5120 wide (shrink and reduce of 173 of them by the run tables take 1.16 times
// what they take by the way chosen here in the geometric mean; the best number of slices would make it 1.18).
// By panels: a block takes 1.7 us and 2.4 ns per stage and row of it; what the blocks take in comes at 8.4 TB/s, x alone at 5.1; slices have to be added up.
// By the run table: 11 us with the reduce, 64 + rank rows per tile and stage at 10.4 TB/s.
static void choose_panels(const lora_cache_t *c, const PlanLists *p, const Scratch &sc, lora::TileBatch &tb)
{
    if (tb.n_direct > 0 || p->n_panels <= 0 || sc.small) return;
    struct Kind {  // groups alike
        int n_k, gn, many;
    } kinds[8];
    int n_kinds = 0, least_k = INT32_MAX;
    for (int i = 0; i < tb.n;) {
        const int n_k = tb.p[i].h_in / 64, gn = (int)(tb.group[i] >> 8);
        least_k = std::min(least_k, n_k);
        int k = 0;
        while (k < n_kinds && (kinds[k].n_k != n_k || kinds[k].gn != gn)) ++k;
        if (k == 8) k = 7;  // (a cache has few widths: the rest counts as the last kind)
        else if (k == n_kinds) kinds[n_kinds++] = Kind{n_k, gn, 0};
        ++kinds[k].many;
        i += gn;
    }
    double blocks = 0, stage_rows = 0, longest = 0, x_bytes = 0, run_bytes = 0;  // stage_rows: of all blocks, longest: of one
    for (int k = 0; k < n_kinds; ++k) {
        const Kind &q = kinds[k];
        for (int runs = 1; runs <= lora::PANEL_ROWS / 64; ++runs)
            for (int nb = 1; nb <= 8; ++nb) {
                const int count = p->panel_count[runs][nb];
                if (count == 0) continue;
                const int np = lora::panel_projs(runs, nb), full = q.gn / np, rest = q.gn % np;
                blocks += (double)q.many * count * (full + (rest > 0));
                stage_rows += (double)q.many * count * q.n_k * ((full + (rest > 0)) * 64 * runs + q.gn * 16 * nb);
                longest = std::max(longest, (double)q.n_k * (64 * runs + 16 * nb * std::min(np, q.gn)));
            }
        x_bytes += (double)q.many * q.n_k * 128 * p->n_tile_tok;
        run_bytes += (double)q.many * q.gn * q.n_k * 128 * p->tile_rows;
    }
    int best = 0;
    double best_us = tb.n_runs > 0 ? 10.8 + std::max(run_bytes / 10.4e6, x_bytes / 5.2e6) : std::numeric_limits<double>::infinity();
    for (int S : {1, 2, 3, 4, 6, 8, 12, 16}) {
        if (S > 1 && (least_k < 4 * S || (int64_t)S * tb.n * p->n_tile_tok > sc.vpart_rows)) break;
        const double n = blocks * S, avg = 1.7 + 0.0024 * stage_rows / n, all = n * avg / c->n_cu;
        double us = std::max({1.7 + 0.0024 * longest / S, 1.7 + stage_rows * 128 / 8.4e6, 1.7 + x_bytes / 5.1e6});
        if (n > 2 * c->n_cu) us = std::max(us, all + 1.4 * avg);
        else if (n > c->n_cu) us = std::max(us, 1.63 * avg);
        us += 0.9 + (S > 1 ? 4.1 + S * tb.n * p->panel_sum_bytes / 6.7e6 : 0);
        if (us < best_us) best_us = us, best = S;
    }
    if (best == 0) return;
    for (int i = 0; i < tb.n; ++i) tb.slices[i] = (uint8_t)best;
    tb.panels = reinterpret_cast<const lora::DevItem *>(p->lists + p->off_panels);
    tb.n_rows = p->n_tile_tok;
    tb.n_panels = p->n_panels;
    tb.classes = p->panel_classes;
    tb.part_set = (uint64_t)best * tb.n_rows * c->v_stride;
}
static lora::BatchProj batch_proj(const lora_cache_t *c, const lora_apply_desc_t &d)
{
    return lora::BatchProj{c->pool + (size_t)d.layer * c->layer_stride + c->proj_off[d.proj], d.x, d.base_out, c->proj[d.proj].h_in, c->proj[d.proj].h_out};
}

// One-launch GEMV form under stream capture, for n projections with plan p.  A graph freezes the launch number, so a
// replay could take the words its own launch wrote in the replay before for fresh ones.  Not when another launch of the
// same graph has written the same words in between (its number differs): that holds for every launch after the first of a
// capture that works on the same plan with at least as many projections.  Otherwise the words are cleared first, by a
// small kernel that becomes part of the graph.
static int clear_words_for_capture(lora_cache_t *c, const PlanLists *p, int n, hipStream_t st, const Scratch &sc)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    unsigned long long cap = 0;
    if (hipStreamGetCaptureInfo(st, &cs, &cap) != hipSuccess) {
        (void)hipGetLastError();
        cs = hipStreamCaptureStatusNone;
    }
    if (cs == hipStreamCaptureStatusNone) return LORA_OK;
    const bool covered = cap == *sc.cap_id && p->build_seq == *sc.cap_plan && n <= *sc.cap_sets;
    if (!covered) {
        const int32_t *toks = reinterpret_cast<const int32_t *>(p->lists) + p->n_tile_tok;
        HIP_TRY(lora::launch_gemv_clear(c->dtype, reinterpret_cast<unsigned long long *>(sc.vtag), sc.vtag_set_bytes / sizeof(unsigned long long), n, toks,
                                        p->n_tok_list - p->n_tile_tok, st));
    }
    *sc.cap_id = cap;
    *sc.cap_plan = p->build_seq;
    *sc.cap_sets = n;
    return LORA_OK;
}
// the one-launch form, for a launch of `items` shrink items? (after 2^32 - 1 launches the numbers would repeat)
static bool one_gemv_launch(const lora_cache_t *c, const Scratch &sc, int64_t items, int64_t max_items)
{
    return *sc.epoch < UINT32_MAX - 1 && (c->fused_gemv == 2 || (c->fused_gemv == 1 && items <= max_items));
}

// The GEMV part of a group of n projections that read the same x: one launch with the in-kernel
// hand-over when the part is small (the launch in between then costs more than the hand-over), else a
// shrink and an expand launch.  y32[i], when set, receives projection i's update as fp32 instead of y.
static int enqueue_gemv(lora_cache_t *c, const PlanLists *p, const lora::BatchProj *a, float *const *y32, int n, float scale,
                        hipStream_t st, const Scratch &sc, const lora::KernelTimer *tm, hipEvent_t done, const lora::ListCopy &copy)
{
    if (p->n_gs <= 0) return LORA_OK;
    lora::GemvArgs ga{};
    lora::GemvMap gm{};
    ga.x = a[0].x;
    gm.gs = reinterpret_cast<const lora::GemvItem *>(p->lists + p->off_gs);
    gm.ge = reinterpret_cast<const lora::GemvItem *>(p->lists + p->off_ge);
    gm.n_gs = (uint32_t)p->n_gs;
    gm.n_proj_phase = (uint32_t)n;
    ga.fault = c->fault_dev;
    ga.h_in = a[0].h_in;
    ga.n_ge = p->n_ge;
    ga.scale = scale;
    int64_t units = 0;
    for (int i = 0; i < lora::GEMV_MAX_PROJS; ++i) {
        const int k = std::min(i, n - 1);  // entries past the group repeat its last
        lora::GemvProj &q = ga.p[i];
        q.proj_base = a[k].proj_base;
        q.row_bytes = (int64_t)(a[k].h_in + a[k].h_out) * c->esize;
        q.y = a[k].y;
        q.y32 = y32 ? y32[k] : nullptr;
        q.vw = reinterpret_cast<unsigned long long *>(sc.vtag + (size_t)k * sc.vtag_set_bytes);
        q.h_out = a[k].h_out;
        const int32_t n_super = supers_of(a[k].h_out);
        if (n_super > 255) return LORA_E_INVAL;  // beyond the kernels' unit arithmetic
        gm.n_super_packed |= (uint32_t)n_super << (8 * i);
        gm.super_magic[i] = lora::gemv_magic((uint32_t)n_super);
        if (i < n) units += (int64_t)p->n_ge * n_super;
        gm.unit_end[i] = (int32_t)std::min<int64_t>(units, INT32_MAX);
    }
    if (units >= (1 << 24) || (int64_t)p->n_gs * n >= (1 << 24)) return LORA_E_INVAL;  // beyond the kernels' unit arithmetic
    if (one_gemv_launch(c, sc, (int64_t)p->n_gs * n, FUSED_GEMV_MAX_ITEMS)) {
        if (const int rc = clear_words_for_capture(c, p, n, st, sc)) return rc;
        ga.epoch = ++*sc.epoch;
    }
    HIP_TRY(lora::launch_gemv(c->dtype, gm, ga, copy, st, tm, done));
    return LORA_OK;
}

// wide items for a GEMV launch of n projections in n_groups groups?
static bool gemv_wide(const lora_cache_t *c, const PlanLists *p, const lora::BatchProj *projs, int n, int n_groups)
{
    if (c->dtype != LORA_BF16 || (int64_t)p->n_wgs * n < (n_groups > 1 ? GEMV_WIDE_MIN_ITEMS : GEMV_WIDE_MIN_ITEMS_ONE_GROUP)) return false;
    int64_t supers = 0;  // (a group may be beyond the batch kernels' unit arithmetic, a batch is cut to it)
    for (int i = 0; i < n; ++i) supers += supers_of(projs[i].h_out);
    return supers <= lora::GEMV_LONG_MAX_SUPERS && (n_groups > 1 || supers <= lora::GEMV_BATCH_MAX_SUPERS) && supers * p->n_wge < (1 << 24);
}

// The same for a batch of several groups.
static int enqueue_gemv_batch(lora_cache_t *c, const PlanLists *p, const lora::BatchProj *projs, float *y32, int n, int n_groups, float scale, hipStream_t st, const Scratch &sc,
                              const lora::KernelTimer *tm, hipEvent_t done, const lora::ListCopy &copy)
{
    if (p->n_gs <= 0) return LORA_OK;
    lora::GemvBatch b{};
    b.gs = reinterpret_cast<const lora::GemvItem *>(p->lists + p->off_gs);
    b.ge = reinterpret_cast<const lora::GemvItem *>(p->lists + p->off_ge);
    b.vw = reinterpret_cast<unsigned long long *>(sc.vtag);
    b.vw_set = sc.vtag_set_bytes / sizeof(unsigned long long);
    b.y32 = y32;
    b.fault = c->fault_dev;
    b.scale = scale;
    const bool wide = gemv_wide(c, p, projs, n, n_groups);
    b.wgs = reinterpret_cast<const lora::GemvWideItem *>(p->lists + p->off_wgs);
    b.wge = reinterpret_cast<const lora::GemvWideItem *>(p->lists + p->off_wge);
    int32_t widths[lora::GEMV_BATCH_MAX_PROJS];
    uint32_t first[lora::GEMV_BATCH_MAX_PROJS];
    for (int i = 0; i < n; ++i) widths[i] = projs[i].h_out;
    if (const int rc = gemv_batch_map(p, wide, n, widths, b.m, b.supers, lora::GEMV_BATCH_MAX_SUPERS, 1, first)) return rc;
    for (int i = 0; i < n; ++i) b.p[i] = lora::gemv_entry(projs[i], first[i]);
    if (one_gemv_launch(c, sc, (int64_t)p->n_gs * n, FUSED_GEMV_MAX_BATCH_ITEMS)) {
        if (const int rc = clear_words_for_capture(c, p, n, st, sc)) return rc;
        b.epoch = ++*sc.epoch;
    }
    HIP_TRY(lora::launch_gemv_batch(c->dtype, b, wide, copy, st, tm, done));
    return LORA_OK;
}

// A batch of more projections or super-chunks than GemvBatch holds, entries as the caller gave them (their addresses are what `projs` says)?
static bool gemv_long(const lora_cache_t *c, const PlanLists *p, const lora_apply_desc_t *descs, int n)
{
    int32_t kinds[lora::GEMV_LONG_KINDS], n_kinds = 0;
    int64_t supers = 0;
    for (int i = 0; i < n; ++i) {
        supers += supers_of(c->proj[descs[i].proj].h_out);
        int k = 0;
        while (k < n_kinds && kinds[k] != descs[i].proj) ++k;
        if (k == lora::GEMV_LONG_KINDS) return false;
        if (k == n_kinds) kinds[n_kinds++] = descs[i].proj;
    }
    return p->n_tiles == 0 && p->n_gs > 0 && n <= lora::GEMV_LONG_MAX_PROJS && supers <= lora::GEMV_LONG_MAX_SUPERS && c->n_layers <= 1 << 21 &&
           (n > lora::GEMV_BATCH_MAX_PROJS || supers > lora::GEMV_BATCH_MAX_SUPERS);
}
static int enqueue_gemv_long(lora_cache_t *c, const PlanLists *p, const lora::BatchProj *projs, const lora_apply_desc_t *const *descs, int n, int n_groups, float scale, hipStream_t st,
                             const Scratch &sc, const lora::KernelTimer *tm, hipEvent_t done, const lora::ListCopy &copy)
{
    lora::GemvLong b{};
    const bool wide = gemv_wide(c, p, projs, n, n_groups);
    b.shrink_items = p->lists + (wide ? p->off_wgs : p->off_gs);
    b.expand_items = p->lists + (wide ? p->off_wge : p->off_ge);
    b.vw = reinterpret_cast<unsigned long long *>(sc.vtag);
    b.vw_set = sc.vtag_set_bytes / sizeof(unsigned long long);
    b.fault = c->fault_dev;
    b.scale = scale;
    b.pool = c->pool;
    b.layer_stride = c->layer_stride;
    int32_t widths[lora::GEMV_LONG_MAX_PROJS], kinds[lora::GEMV_LONG_KINDS], n_kinds = 0;
    uint32_t first[lora::GEMV_LONG_MAX_PROJS];
    for (int i = 0; i < n; ++i) widths[i] = projs[i].h_out;
    if (const int rc = gemv_batch_map(p, wide, n, widths, b.m, b.marks, lora::GEMV_LONG_MAX_SUPERS, lora::GEMV_LONG_STEP, first)) return rc;
    for (int i = 0; i < n; ++i) {
        const lora_apply_desc_t &d = *descs[i];
        int k = 0;
        while (k < n_kinds && kinds[k] != d.proj) ++k;
        if (k == lora::GEMV_LONG_KINDS) return LORA_E_INVAL;  // (cannot happen: gemv_long)
        if (k == n_kinds) {
            kinds[n_kinds++] = d.proj;
            b.off_h_out[k] = (uint64_t)c->proj_off[d.proj] | (uint64_t)(projs[i].h_out / 64) << 48;
            b.h_in[k] = projs[i].h_in;
        }
        b.p[i] = lora::gemv_long_entry(d.x, d.base_out, (uint32_t)k, (uint32_t)d.layer, first[i]);
    }
    if (one_gemv_launch(c, sc, (int64_t)p->n_gs * n, FUSED_GEMV_MAX_BATCH_ITEMS)) {
        if (const int rc = clear_words_for_capture(c, p, n, st, sc)) return rc;
        b.epoch = ++*sc.epoch;
    }
    HIP_TRY(lora::launch_gemv_long(c->dtype, b, wide, copy, st, tm, done));
    return LORA_OK;
}

// The lists a launch for n projections in n_groups groups works through, sum_width wide together (h_in + h_out), and those of the base product
static const PlanLists *pick_lists(const lora_plan_t *p, int n, int n_groups, double sum_width)
{
    return p->has_tiled && list_takes_tiles(*p, n, n_groups, sum_width) ? &p->tiled : p;
}
static const PlanLists *pick_linear_lists(const lora_cache_t *c, const lora_plan_t *p, double width)
{
    return p->has_tiled && product_takes_tiles(*c, *p, width) ? &p->tiled : p;
}

// What a call needs of other streams: the plan's lists and its slots' weights.  A captured call waits here, on the host: a wait on an event from outside the capture does not become
// part of the graph, whose replays may run before that event.  (The event of a stream that is not the null stream can be asked about and waited for while this thread captures
// only in relaxed mode; elsewhere the capture is invalidated.)
// copies: the launch this is for copies the plan's lists itself; else lists that are still with the host are uploaded here (for a captured call on a stream that is in no capture: the upload is no part of the graph).
static int wait_for_inputs(lora_cache_t *c, lora_plan_t *p, hipStream_t st, bool copies)
{
    int capturing = -1;  // not known yet
    if (copies) {
        HIP_TRY(wait_for_uses(*c, *p, st));
    } else if (p->deferred) {
        capturing = is_capturing(st);
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (capturing && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return LORA_E_HIP;
        hipError_t e = capturing && !c->upload_stream ? hipStreamCreateWithFlags(&c->upload_stream, hipStreamNonBlocking) : hipSuccess;
        if (e == hipSuccess) e = upload_lists(*c, *p, capturing ? c->upload_stream : st);
        if (capturing) (void)hipThreadExchangeStreamCaptureMode(&mode);
        HIP_TRY(e);
    }
    auto wait = [&](hipEvent_t ev, bool &pending) {
        if (capturing < 0) capturing = is_capturing(st);
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (capturing && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return hipErrorStreamCaptureUnsupported;
        hipError_t e = capturing ? hipEventSynchronize(ev) : hipEventQuery(ev);
        if (capturing) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e == hipSuccess) pending = false;
        else e = hipStreamWaitEvent(st, ev, 0);
        return e;
    };
    if (p->upload_pending) HIP_TRY(wait(p->ev_upload, p->upload_pending));
    if (p->upload_fence >= 0) {
        bool pending = true;
        HIP_TRY(wait(c->fences[p->upload_fence].ev, pending));
        if (!pending) hold_fence(*c, p->upload_fence, -1);
    }
    for (int32_t sl : p->slots) {
        Slot &s = c->slots[sl];
        if (s.fill_pending) HIP_TRY(wait(s.fill_ev, s.fill_pending));
    }
    return LORA_OK;
}

static lora::ListCopy list_copy(const lora_plan_t *p)
{
    return lora::ListCopy{p->dev, p->pinned_dev, (uint32_t)((p->bytes + p->tiled_bytes + 15) / 16), 0};
}

// Applies descs[0 .. n), n <= the scratch's sets, that do not depend on each other: every phase is one launch for all of
// them.  Entries that read the same x (a group, at most GROUP_MAX_PROJS) are neighbours; group_n[i] is the size of the group that
// starts at entry i.  The tile shrink runs first, for all entries (x of a group is then fetched from memory once), each
// with its own copy of the intermediate buffers.
// `fence` (null: none) is to stand for the batch's end on `st`.
static int enqueue_batch(lora_cache_t *c, lora_plan_t *p, const PlanLists *q, const lora_apply_desc_t *descs, const uint8_t *group_n, int n, float scale, hipStream_t st,
                         const Scratch &sc, hipEvent_t fence, bool fenced)
{
    int64_t sum_h_in = 0, sum_h_out = 0, sum_supers = 0;
    for (int i = 0; i < n; ++i) {
        sum_h_in += c->proj[descs[i].proj].h_in;
        sum_h_out += c->proj[descs[i].proj].h_out;
        sum_supers += supers_of(c->proj[descs[i].proj].h_out);
    }
    // The GEMV launch and the tile kernels of a batch work on different tokens (rows of base_out) with different
    // scratch: when a batch has enough of both, the GEMV launch goes to the cache's side stream, forked off here and
    // joined again behind the tile expands (also under stream capture, where fork and join become edges of the graph).
    // Not while kernels are being timed: a kernel's duration is then its own, not that of two kernels sharing the memory.
    const lora::KernelTimer timer{c, timer_pair};
    const lora::KernelTimer *tm = c->timing && !is_capturing(st) ? &timer : nullptr;
    const bool fork = gemv_beside_tiles(*c, q, sum_h_in, sum_h_out) && c->side_stream != nullptr && c->side_stream != st && tm == nullptr;
    // Lists that are still with the host travel with the first launch, if a fence will stand for it: a tile shrink, unless the GEMV launch runs beside it, or a GEMV launch of not too many
    // wavefronts that read them over the link
    const bool gemv_copies = q == p && q->n_tiles == 0 && q->n_gs > 0 && 4 * (int64_t)q->n_gs * n + q->n_ge * sum_supers <= PINNED_LISTS_MAX_WAVES &&
                             (int64_t)q->n_wgs * n < GEMV_WIDE_MIN_ITEMS && one_gemv_launch(c, sc, (int64_t)q->n_gs * n, FUSED_GEMV_MAX_ITEMS);
    const bool copies = p->deferred && fenced && !c->timing && (q->n_tiles > 0 ? !fork && shrink_copies(q, n, sum_h_in) : gemv_copies);
    if (const int rc = wait_for_inputs(c, p, st, copies)) return rc;
    struct Lists {  // where a GEMV launch that copies them reads them
        lora_plan *p;
        ~Lists()
        {
            if (p) p->lists = p->dev;
        }
    } lists{copies && gemv_copies ? p : nullptr};
    const lora::ListCopy copy = copies ? list_copy(p) : lora::ListCopy{};
    if (lists.p) p->lists = p->pinned_dev;
    lora::TileBatch tb;
    if (q->n_tiles > 0)
        if (const int rc_s = tile_setup(c, q, n, sum_h_in, sc, scale, tb)) return rc_s;
    // groups of long rows first: their shrink blocks take the longest, and the launch should not end with them
    int n_groups = 0;
    uint8_t first[lora::GEMV_LONG_MAX_PROJS];
    lora::BatchProj projs[lora::GEMV_LONG_MAX_PROJS];
    const lora_apply_desc_t *at_desc[lora::GEMV_LONG_MAX_PROJS];
    for (int i = 0; i < n; i += group_n[i]) first[n_groups++] = (uint8_t)i;
    std::stable_sort(first, first + n_groups, [&](uint8_t g, uint8_t h) { return c->proj[descs[g].proj].h_in > c->proj[descs[h].proj].h_in; });
    for (int g = 0, i = 0; g < n_groups; ++g) {
        const int size = group_n[first[g]], at = i;
        for (int k = 0; k < size; ++k, ++i) {
            at_desc[i] = &descs[first[g] + k];
            projs[i] = batch_proj(c, *at_desc[i]);
            if (q->n_tiles > 0) tb.p[i] = projs[i], tb.group[i] = (uint32_t)at | (uint32_t)size << 8;
        }
    }
    if (q->n_tiles > 0) choose_panels(c, q, sc, tb);
    hipStream_t gemv_st = st;
    if (fork) {
        HIP_TRY(hipEventRecord(c->ev_fork, st));
        HIP_TRY(hipStreamWaitEvent(c->side_stream, c->ev_fork, 0));
        gemv_st = c->side_stream;
    }
    // everything that reads x
    if (copies) p->copying = true;  // until a fence stands for the launch (which may be on its way although the runtime returns an error: one that an earlier call of the thread has left)
    if (q->n_tiles > 0) {
        HIP_TRY(lora::launch_mfma_shrink(tb, copy, st, tm));
        if (copies) p->deferred = false;
    }
    const lora::ListCopy gemv_copy = lists.p ? copy : lora::ListCopy{};
    // joined behind the tile expands, whatever happens in between: a captured fork must not stay open
    struct Join {
        lora_cache_t *c;
        hipStream_t st;
        bool armed, rides;  // rides: the join event is the GEMV launch's own (not while capturing, where it must be an edge of the graph)
        hipError_t now()
        {
            if (!armed) return hipSuccess;
            armed = false;
            const hipError_t e = rides ? hipSuccess : hipEventRecord(c->ev_join, c->side_stream);
            return e == hipSuccess ? hipStreamWaitEvent(st, c->ev_join, 0) : e;
        }
        ~Join() { (void)now(); }
    } join{c, st, fork, false};
    // the fence rides on the group's last kernel, where that is the last thing on `st`
    const bool ride = fence && !fork && tm == nullptr && (q->n_tiles > 0 || q->n_gs > 0);
    const bool join_rides = fork && !is_capturing(st);
    const hipEvent_t gemv_done = join_rides ? c->ev_join : (ride && q->n_tiles == 0 ? fence : nullptr);
    if (const int rc_g = n_groups > 1 && gemv_long(c, q, descs, n) ? enqueue_gemv_long(c, q, projs, at_desc, n, n_groups, scale, gemv_st, sc, tm, gemv_done, gemv_copy)
                                       : n_groups == 1 && !gemv_wide(c, q, projs, n, 1) ? enqueue_gemv(c, q, projs, nullptr, n, scale, gemv_st, sc, tm, gemv_done, gemv_copy)
                                       : enqueue_gemv_batch(c, q, projs, nullptr, n, n_groups, scale, gemv_st, sc, tm, gemv_done, gemv_copy))
        return rc_g;
    if (lists.p) p->deferred = false;
    join.rides = join_rides;
    // the updates of base_out
    if (q->n_tiles > 0) HIP_TRY(lora::launch_mfma_expand(tb, st, tm, ride ? fence : nullptr));
    for (int i = 0; i < n; ++i) {
        const int64_t seq = ++c->apply_seq;
        ++c->stats.applies;
        for (int32_t sl : p->slots) {
            c->slots[sl].last_used = c->slots[sl].last_by[sc.small] = seq;
            ++c->slots[sl].use_count;
        }
    }
    HIP_TRY(join.now());
    if (fence && !ride) HIP_TRY(hipEventRecord(fence, st));
    return LORA_OK;
}

// The event that is to stand for the end of a call that enqueues applies on `st`: fills that come later and uploads
// into the same plan wait for it.  None (-1) without fencing and under capture.
static int take_fence(lora_cache_t *c, lora_plan_t *p, hipStream_t st, int32_t &f)
{
    f = -1;
    if (!c->fencing || is_capturing(st)) {
        p->unfenced = true;
        return LORA_OK;
    }
    f = free_fence(*c);
    return f < 0 ? LORA_E_HIP : LORA_OK;
}
static void publish_fence(lora_cache_t *c, lora_plan_t *p, hipStream_t st, int32_t f, bool fixed_scratch = false)
{
    if (f < 0) return;
    const int64_t seq = c->apply_seq;
    hold_fence(*c, c->ring[seq % N_APPLY_EVENTS], f);
    c->ring_seq[seq % N_APPLY_EVENTS] = seq;
    hold_fence(*c, c->stream_fence.try_emplace(st, -1).first->second, f);
    hold_fence(*c, p->last_use[fixed_scratch], f);
    if (p->copying) {
        p->copying = false;
        hold_fence(*c, p->upload_fence, f);
    }
}
// A call that fails has no fence to stand for launches of it that read the plan's lists: lists with the host are waited for, for those in the pool it counts as any call without a fence
struct CallGuard {
    lora_plan_t *p;
    hipStream_t st;
    bool done = false;
    ~CallGuard()
    {
        if (done) return;
        if (p->copying || p->lists == p->pinned_dev) (void)hipStreamSynchronize(st);
        p->copying = false;
        p->unfenced = true;
    }
};

// one projection as a call with a fence of its own
static int apply_fenced(lora_cache_t *c, lora_plan_t *p, const lora_apply_desc_t &d, float scale, hipStream_t st, const Scratch &sc)
{
    int32_t f;
    if (const int rc = take_fence(c, p, st, f)) return rc;
    CallGuard guard{p, st};
    const uint8_t one = 1;
    if (const int rc = enqueue_batch(c, p, p, &d, &one, 1, scale, st, sc, f < 0 ? nullptr : c->fences[f].ev, f >= 0)) return rc;
    publish_fence(c, p, st, f, sc.small);
    guard.done = true;
    return LORA_OK;
}

int lora_apply_plan(lora_cache_t *c, lora_plan_t *p, int32_t layer, int32_t proj, const void *x, void *base_out,
                    float scale, void *stream)
{
    if (!c || !p || !p->in_use || c->host_only) return LORA_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = validate_apply(c, p, layer, proj, x, base_out);
    if (rc != LORA_OK) return rc;
    return apply_fenced(c, p, {layer, proj, x, base_out}, scale, st, pool_scratch(c));
}

int lora_apply_plan_static(lora_cache_t *c, lora_plan_t *p, int32_t layer, int32_t proj, const void *x, void *base_out,
                           float scale, void *stream)
{
    if (!c || !p || !p->in_use || c->host_only) return LORA_E_INVAL;
    if (p->T > LORA_STATIC_MAX_TOKENS) return LORA_E_NOMEM;  // the fixed scratch does not hold this batch
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = validate_apply(c, p, layer, proj, x, base_out);
    if (rc != LORA_OK) return rc;
    StaticScratch &ss = g_static[c->device];  // set up by lora_cache_create on this device
    if (!ss.ptr) return LORA_E_STATE;
    const Scratch sc{ss.ptr, STATIC_V_BYTES, 1, ss.ptr + STATIC_V_BYTES, STATIC_VPART_ROWS, true,
                     ss.ptr + STATIC_V_BYTES + STATIC_VPART_BYTES, STATIC_VTAG_BYTES, &ss.epoch, &ss.cap_id, &ss.cap_plan, &ss.cap_sets};
    const bool timing = c->timing;
    c->timing = false;  // timed launches take events from a pool that may have to grow
    rc = apply_fenced(c, p, {layer, proj, x, base_out}, scale, st, sc);
    c->timing = timing;
    return rc;
}

int lora_linear_workspace_bytes(const lora_cache_t *c, const lora_plan_t *p, int32_t proj, size_t *bytes)
{
    if (!c || !p || !p->in_use || !bytes || proj < 0 || proj >= (int32_t)c->proj.size()) return LORA_E_INVAL;
    *bytes = p->n_tok_list > p->n_tile_tok ? (size_t)p->T * c->proj[proj].h_out * sizeof(float) : 0;
    return LORA_OK;
}

int lora_linear_plan(lora_cache_t *c, lora_plan_t *p, int32_t layer, int32_t proj, const void *x, const void *Wt, void *y,
                     float scale, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!c || !p || !p->in_use || c->host_only || c->dtype != LORA_BF16) return LORA_E_INVAL;
    if (workspace) {
        size_t need = 0;
        if (lora_linear_workspace_bytes(c, p, proj, &need) != LORA_OK || !aligned16(workspace) || workspace_bytes < need) return LORA_E_INVAL;
    }
    int rc = validate_apply(c, p, layer, proj, x, y);
    if (rc != LORA_OK) return rc;
    if (p->T > 0 && (!Wt || !aligned16(Wt))) return LORA_E_INVAL;
    if (p->T == 0) return LORA_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const lora::KernelTimer timer{c, timer_pair};
    const lora::KernelTimer *tm = c->timing && !is_capturing(st) ? &timer : nullptr;
    const lora::BatchProj bp = batch_proj(c, {layer, proj, x, y});
    lora::ApplyArgs a;
    a.proj_base = bp.proj_base;
    a.row_bytes = (int64_t)c->row_bytes[proj];
    const PlanLists *const q = pick_linear_lists(c, p, (double)bp.h_in + bp.h_out);
    a.tok_list = reinterpret_cast<const int32_t *>(q->lists);
    a.x = x;
    a.y = y;
    a.v = reinterpret_cast<float *>(c->pool + c->off_v);
    a.h_in = c->proj[proj].h_in;
    a.h_out = c->proj[proj].h_out;
    a.v_stride = c->v_stride;
    a.scale = scale;
    int32_t f;
    if (const int rc_f = take_fence(c, p, st, f)) return rc_f;
    CallGuard guard{p, st};
    const bool copies = p->deferred && f >= 0 && !c->timing && shrink_copies(q, 1, a.h_in);  // (as in enqueue_batch)
    if (const int rc_w = wait_for_inputs(c, p, st, copies)) return rc_w;
    // shrink of the tiles (x is read, v written), then the adapter term of the GEMV tokens: as fp32 into the caller's workspace
    // (row = token), or, without one, into their zeroed output rows (rounded to the output type on the way).  One after the
    // other: the GEMV launch on the side stream, between a fork off the last base product and a join into the next, waits 10 us at
    // both for 20 us of shrink and reduce beside it (a 13B layer 2034 us, 2015 us this way).
    const int32_t n_gemv_tok = q->n_tok_list - q->n_tile_tok;
    if (q->n_tiles > 0) {
        lora::TileBatch tb;
        if (const int rc_s = tile_setup(c, q, 1, a.h_in, pool_scratch(c), scale, tb)) return rc_s;
        tb.p[0] = bp;
        tb.group[0] = 1u << 8;
        choose_panels(c, q, pool_scratch(c), tb);
        if (copies) p->copying = true;
        HIP_TRY(lora::launch_mfma_shrink(tb, copies ? list_copy(p) : lora::ListCopy{}, st, tm));
        if (copies) p->deferred = false;
    }
    if (n_gemv_tok > 0) {
        a.y32 = static_cast<float *>(workspace);
        if (!a.y32) HIP_TRY(lora::launch_zero_rows(y, a.tok_list + q->n_tile_tok, n_gemv_tok, a.h_out, st));
        float *const y32 = a.y32;
        if (const int rc_g = gemv_wide(c, q, &bp, 1, 1) ? enqueue_gemv_batch(c, q, &bp, y32, 1, 1, scale, st, pool_scratch(c), tm, nullptr, {})
                                                        : enqueue_gemv(c, q, &bp, &y32, 1, scale, st, pool_scratch(c), tm, nullptr, {}))
            return rc_g;
    }
    // base product of every token + adapter product of the tiles (+ the term just computed for the others)
    const lora::LinearList list{reinterpret_cast<const int32_t *>(q->lists + q->off_lin_tok), reinterpret_cast<const lora::LinearRows *>(q->lists + q->off_lin_rows),
                                reinterpret_cast<const lora::LinearSeg *>(q->lists + q->off_lin_segs),
                                q->T, q->n_lin_rows, q->n_tile_tok, q->n_tok_list};
    // (the partial sums of split tiles go where the tile shrink's partial sums went: that kernel is done)
    HIP_TRY(lora::launch_linear_tiles(a, Wt, list, c->pool + c->off_vpart, c->vpart_bytes, reinterpret_cast<lora::SplitState *>(c->pool + c->off_splits),
                                      N_LINEAR_SPLITS, c->fault_dev, c->n_cu, st, tm, tm || f < 0 ? nullptr : c->fences[f].ev));
    if (tm && f >= 0) HIP_TRY(hipEventRecord(c->fences[f].ev, st));
    const int64_t seq = ++c->apply_seq;
    ++c->stats.applies;
    for (int32_t sl : p->slots) {
        c->slots[sl].last_used = c->slots[sl].last_by[0] = seq;
        ++c->slots[sl].use_count;
    }
    publish_fence(c, p, st, f);
    guard.done = true;
    return LORA_OK;
}

int lora_apply_plan_multi(lora_cache_t *c, lora_plan_t *p, const lora_apply_desc_t *descs, int32_t n, float scale,
                          void *stream)
{
    if (!c || !p || !p->in_use || c->host_only || n < 0 || (n > 0 && !descs)) return LORA_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    for (int32_t i = 0; i < n; ++i) {
        const int rc = validate_apply(c, p, descs[i].layer, descs[i].proj, descs[i].x, descs[i].base_out);
        if (rc != LORA_OK) return rc;
    }
    int32_t f;
    if (const int rc_f = take_fence(c, p, st, f)) return rc_f;
    CallGuard guard{p, st};
    // Entries that do not depend on each other go as one batch: no output of the batch may overlap an input of it (an
    // earlier entry's: it may not have been read yet; a later one's: it would be read too early) or another output (both
    // would be updated from what was there before).  Within a batch neighbours that read the same x (q, k, v; gate, up)
    // form groups.  An entry that overwrites its own input is a batch by itself.
    struct Range {
        const char *lo, *hi;
        bool meets(const Range &o) const { return lo < o.hi && o.lo < hi; }
    };
    const size_t e = c->esize;
    Range in[lora::GEMV_LONG_MAX_PROJS], out[lora::GEMV_LONG_MAX_PROJS];  // distinct inputs of the batch's groups; outputs of its entries, by address (they do not overlap)
    uint8_t group_n[lora::GEMV_LONG_MAX_PROJS];
    const Scratch scratch = pool_scratch(c);
    int32_t max_projs, max_supers;
    batch_limits(p, scratch, p->n_tiles == 0, max_projs, max_supers);
    for (int32_t i = 0; i < n;) {
        int32_t m = 0, n_in = 0, last = 0, supers = 0;  // last: entry the latest group starts at
        for (; i + m < n && m < max_projs; ++m) {
            const lora_apply_desc_t &d = descs[i + m];
            const lora_proj_t &pr = c->proj[d.proj];
            const char *x0 = static_cast<const char *>(d.x), *y0 = static_cast<const char *>(d.base_out);
            const Range x{x0, x0 + (size_t)p->T * pr.h_in * e}, y{y0, y0 + (size_t)p->T * pr.h_out * e};
            const bool same_x = m > 0 && d.x == descs[i + m - 1].x && pr.h_in == c->proj[descs[i + m - 1].proj].h_in;
            auto behind = [&](const Range &r) { return std::upper_bound(out, out + m, r.lo, [](const char *lo, const Range &o) { return lo < o.hi; }); };  // the first output that ends behind r.lo
            auto meets_out = [&](const Range &r) { const Range *o = behind(r); return o != out + m && o->lo < r.hi; };
            bool ok = !y.meets(x) && !meets_out(y) && (same_x || !meets_out(x)), known = false;
            for (int32_t k = 0; k < n_in && ok; ++k) {
                ok = !in[k].meets(y);
                known |= in[k].lo == x.lo && in[k].hi == x.hi;
            }
            supers += supers_of(pr.h_out);
            const bool joins_only_group = same_x && last == 0 && m < lora::GROUP_MAX_PROJS;
            if (m > 0 && (!ok || (supers > max_supers && !joins_only_group))) break;
            Range *const at = out + (behind(y) - out);
            std::copy_backward(at, out + m, out + m + 1);
            *at = y;
            if (same_x && group_n[last] < lora::GROUP_MAX_PROJS) {
                ++group_n[last];
            } else {
                last = m;
                group_n[m] = 1;
                if (!known) in[n_in++] = x;
            }
            if (!ok) {
                ++m;
                break;
            }
        }
        double sum_width = 0;
        int n_groups = 0;
        for (int k = 0; k < m; ++k) sum_width += (double)c->proj[descs[i + k].proj].h_in + c->proj[descs[i + k].proj].h_out;
        for (int k = 0; k < m; k += group_n[k]) ++n_groups;
        const PlanLists *const q = pick_lists(p, m, n_groups, sum_width);
        int32_t most = m, most_supers = INT32_MAX;
        if (q != p || (p->n_tiles == 0 && !gemv_long(c, q, descs + i, m))) batch_limits(q, scratch, false, most, most_supers);
        for (int at = 0; at < m;) {  // (a batch with tiles holds fewer projections, one of more kinds of projections than a long one tells apart too)
            int k = 0;
            for (int32_t left = most_supers; at + k < m; k += group_n[at + k]) {
                for (int e = 0; e < group_n[at + k]; ++e) left -= supers_of(c->proj[descs[i + at + k + e].proj].h_out);
                if (k > 0 && (k + group_n[at + k] > most || left < 0)) break;
            }
            const int rc = enqueue_batch(c, p, q, descs + i + at, group_n + at, k, scale, st, scratch, f >= 0 && i + at + k == n ? c->fences[f].ev : nullptr, f >= 0);
            if (rc != LORA_OK) return rc;
            at += k;
        }
        i += m;
    }
    if (n > 0) publish_fence(c, p, st, f);
    guard.done = true;
    return LORA_OK;
}

int lora_apply(lora_cache_t *c, int32_t layer, int32_t proj, const void *x, void *base_out, int32_t T,
               const int32_t *seg_offsets, const int32_t *seg_slot, const int32_t *seg_rank, int32_t n_seg, float scale,
               void *stream)
{
    if (!c || c->host_only) return LORA_E_INVAL;
    lora_plan &p = c->plans[c->n_user_plans + (c->internal_next % N_INTERNAL_PLANS)];
    int rc = build_plan(*c, p, T, seg_offsets, seg_slot, seg_rank, n_seg, static_cast<hipStream_t>(stream));
    if (rc != LORA_OK) return rc;
    ++c->internal_next;
    p.in_use = true;
    rc = lora_apply_plan(c, &p, layer, proj, x, base_out, scale, stream);
    p.in_use = false;
    return rc;
}

}  // extern "C"
