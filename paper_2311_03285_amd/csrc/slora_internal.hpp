// Internal declarations shared by the host logic (pool, scheduler) and the kernel launchers.
#pragma once

#include <cstdint>
#include <string>
#include <unordered_map>
#include <vector>

#include "slora.h"

namespace slora {

// ---------------------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------------------
int32_t fail(int32_t code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();
const char *last_error_cstr();

// ---------------------------------------------------------------------------------------
// work items (device-visible, 32 bytes)
// ---------------------------------------------------------------------------------------
// One record type serves the four work lists; `a` and `b` mean
//   vector shrink : a = first page j0 of the A list, b = number of pages
//   vector expand : a = first column (element index),  b = number of columns
//   MFMA   expand : a = first column (element index),  b = number of columns, of a run of tiles
// (the MFMA shrink has its own record, MsItem)
struct Item {
    int32_t arena_off; // adapter's first entry in the page-list arena ([slot][A r][B r])
    int32_t rank;      // r of the adapter
    int32_t a;
    int32_t b;
    int32_t pos0;      // first position in the sorted token list (also the row of v)
    int32_t ntok;      // tokens handled by this item (MFMA expand: by its first tile)
    int32_t tile;      // MFMA lists: number of the (adapter, 32-token) tile, shared by shrink and expand; vector expand: 1 if no other item of
                       // the group reads these B rows
    int32_t run;       // MFMA expand: tiles the workgroup walks from `tile` on + 256 * tokens of the last one; vector lists: the first of
                       // the item's entries where v is handed over inside a launch, rank after rank, token after token
};
static_assert(sizeof(Item) == 32, "Item must stay 32 bytes");

// MFMA shrink item: up to kMsTok tokens of one adapter x up to kMsRanks of its ranks x a range
// of H.  The range is the whole of H, or one of n_parts shares of it: then the workgroups of a
// tile leave their partial sums in the slot's scratch and a second kernel adds them up in the
// order of the shares.
struct MsItem {
    int32_t arena_off; // adapter's first entry in the page-list arena
    int32_t rank;      // r of the adapter
    int32_t j0, nj;    // first rank (a multiple of kMsRanks) and number of ranks
    int32_t pos0, ntok; // first position in the sorted token list, tokens
    int32_t tile;      // v tile (32 tokens) of the first token; the item covers up to 4 consecutive tiles
    int32_t c0, c1;    // granules [c0, c1) of H, kMsGranule elements each
    int32_t part, n_parts;
    int32_t sync;      // number of the tile among those the join kernel finishes (-1: the shrink finishes it)
    int32_t part_off;  // floats from the slot's partial area to the tile's partial sums
    int32_t pad[3];
};
static_assert(sizeof(MsItem) == 64, "MsItem must stay 64 bytes");

// Per-launch arguments for up to SLORA_MAX_MULTI slots handled by one grid.
struct MultiArgs {
    const void *x[SLORA_MAX_MULTI];
    void *y[SLORA_MAX_MULTI];   // fp32 rows, or rows of the pool's storage type (16-bit y variant)
    float *v[SLORA_MAX_MULTI];
    int32_t slot[SLORA_MAX_MULTI];
    int32_t n; // slots in this launch; workgroup b handles item b / n for slot entry b % n
    int64_t vfrag_off; // floats from v[k] to the slot's v tiles in MFMA operand layout
    int64_t vexp_off;  // floats from v[k] to the per-row exponents of the tiles (binary16 pools)
    int64_t part_off;  // floats from v[k] to the partial sums of split tiles
};

// The lists of a launch in which the shrink hands v over to the expand
struct ChainLists {
    const Item *shrink, *expand;
    uint32_t n_shrink; // shrink items; then the expand items
    uint32_t turn;     // a slot moves on by one XCD every 2^turn items
    uint64_t *hand;    // words {value, number of the launch} of the first slot,
    int64_t hand_slot; // those of a slot
    uint32_t launch;
    int32_t polls;     // reads before a wavefront computes what it waits for
};

// Which kernels one call of a plan takes.  The expand follows the shrink whose v it reads.
struct Route {
    bool wide = false;  // a dual plan's groups of many tokens on the MFMA kernels
    bool small = false; // both stages in the one-launch kernel for small batches
    bool chain = false; // an apply: both vector stages in one launch that hands v over
    bool gang = false;        // vector groups of many tokens: the shrink for them,
    bool gang_expand = false; // the expand's longer items
    bool fused = false; // an apply: launch_fused serves the groups of the one-launch decode kernel
    int32_t sub = 0;    // MFMA shrink: a workgroup takes kMsTok >> sub tokens of an item
    int32_t parts = 1;  // MFMA expand: workgroups that share a run of tiles
};

// Tile constants the scheduler and the kernels must agree on.
constexpr int kShrinkTok = 4;     // tokens per vector-shrink item (x rows staged in LDS)
constexpr int kShrinkPages = 4;   // pages per vector-shrink item, unless the caller names a number
constexpr int kExpandTok = 4;     // tokens per vector-expand item (accumulators in registers)
constexpr int kSmallRanks = 32;   // most ranks of an adapter in a batch that runs in the one-launch kernel for small batches
constexpr int kExpandColsMax = 1024; // most columns per vector-expand item (a multiple of 512, <= 4096; measured best on cfg4: 1024)
constexpr int kSplitWaves = 4;    // rank-split expand: wavefronts of a workgroup, and parts of a sum over the ranks
constexpr int kGangTok = 8;       // tokens per item of the shrink for groups of many tokens,
constexpr int kGangPages = 16;    // pages, at most
constexpr int kGangFrom = 1400, kGangExpandFrom = 2000; // least workgroups of the small items at which a call takes them (see route)
constexpr bool gang_pays(int64_t small_items, int64_t large_items) { return 2 * large_items <= small_items; }
constexpr int kOwnRanks = 32;     // rank-split expand of groups of many tokens: up to this many ranks a wavefront forms whole sums,
constexpr int kGangOwnTok = 16;   // of that many tokens an item;
constexpr int kGangExpandTok = 8; // tokens per item of more ranks
// ... items whose tokens go through the 4x4x1 matrix instruction, four at a time: all that share the ranks out over the wavefronts, of the others those that leave
// a wavefront three or four tokens.  It takes the time of two tokens' fmaf, rows in f16 need a conversion that v_fma_mix does without, and up to 8 ranks half
// a block is all there is.  us of the call, fmaf / matrix instruction: 8 tokens of rank 16, H = 6144, 4 slots 30.5 / 32.9, 7 of rank 9, H = 5120, 4 slots 22.6 / 25.9, 5
// of rank 17, H = 3072 27.2 / 30.1; 12 of rank 9 in f16 28.5 / 29.7, of rank 16 25.1 / 25.9, of rank 32, H = 8192 42.6 / 43.4; in bf16 12 of rank 24, H = 6144 35.1 / 32.6, 9 of
// rank 24, H = 3072 33.5 / 31.9; 30 of rank 24 40.0 / 32.1.  Up to 8 ranks with y in fp32 16 of rank 1, H = 5120 16.6 / 18.3, 9 of rank 4, H = 8192 20.2 / 21.4, in 16 bits
// 13 of rank 4, H = 6144 19.5 / 17.9, 30 of rank 8, H = 5120 23.9 / 21.8, 12 of rank 4 16.5 / 16.3.
constexpr bool fours_pay(int dtype, bool y16, int32_t rank, int32_t tok)
{
    return rank > kOwnRanks ? tok > kExpandTok : rank > 8 ? tok > (dtype == SLORA_F16 ? 12 : 8) : y16 && tok > 8;
}
constexpr int kChainMaxH = 8192;  // widest rows whose sums the one-launch kernel that hands v over forms: a wavefront holds one in registers
constexpr int kMfmaTok = 32;      // tokens per v tile = per MFMA-expand item (one 32-row MFMA block)
constexpr int kMsTok = 128;       // most tokens per MFMA-shrink item
constexpr int kMsRanks = 128;     // ranks per MFMA-shrink item (up to four blocks of 32)
constexpr int kMsSubs = 3;        // a workgroup takes an item's tokens whole, in halves or in quarters
constexpr int kMsGranule = 128;   // shares of H are whole runs of this many elements
// LDS of the MFMA shrink for a tile of `blocks` 32-row blocks (token rows and page rows): a ring of
// pieces of 32 rows x 128 bytes per block, at most 80 KiB - two workgroups per compute unit
constexpr int kMsBlockBytes = 32 * 128;
constexpr int ms_stages(int blocks) { return blocks <= 2 ? 8 : 80 * 1024 / kMsBlockBytes / blocks; }
constexpr int ms_lds_bytes(int blocks) { return ms_stages(blocks) * blocks * kMsBlockBytes; }
constexpr int kMfmaExpandCols = 256; // columns per MFMA-expand item (4 wavefronts x 64)
constexpr int kMfmaRunMax = 16;  // most 32-token tiles an MFMA-expand workgroup walks
constexpr int kRankPad = 32;      // v rows are zero-padded to a multiple of this many ranks

// ---------------------------------------------------------------------------------------
// pool
// ---------------------------------------------------------------------------------------
enum PageState : uint8_t { kFree = 0, kKv = 1, kAdapter = 2 };

struct Adapter {
    int32_t rank;
    int64_t arena_off; // into the arena, n_slots*2*rank entries
};

// A set of buffers that one plan (or one page write) uses and then hands back to the pool: a
// pinned host image, its device copy, and the v scratch.  Nothing is freed when a user lets
// go: the set waits in the pool's idle list with `order` recorded on the stream that used it
// last and is handed out again once that event has completed, so a steady stream of batches
// (Sec. 4.1: a new batch every iteration) allocates nothing and never waits for the device.
struct Buffers {
    void *h = nullptr;     // pinned host memory
    size_t h_cap = 0;
    void *d = nullptr;     // device copy of h
    size_t d_cap = 0;
    float *v = nullptr;    // device scratch for v = x*A, and behind its v_cap floats
    size_t v_cap = 0;
    uint64_t *hand = nullptr; // words {value, number of a launch} in which a launch hands v over; none has a number that was not given out yet,
    size_t hand_cap = 0;
    bool hand_clear = false;  // once they have been cleared, which the first such launch does
    size_t hand_refused = SIZE_MAX; // from this many on there was no memory for them
    uint32_t launch = 0;   // number of the latest such launch
    std::vector<void *> outgrown; // device buffers replaced while work that names them may be in flight
    void *order = nullptr; // hipEvent_t: last use of the set, or a hand-over point between streams
};

// Makes the pool's device current for the calling scope and restores the caller's device.
class DeviceScope {
public:
    explicit DeviceScope(int device);
    ~DeviceScope();
    int32_t status() const { return rc_; }
private:
    int prev_ = -1;
    bool switched_ = false;
    int32_t rc_ = 0;
};

} // namespace slora

struct slora_pool {
    int32_t H = 0;
    int64_t n_pages = 0;
    int32_t dtype = 0;
    void *dev_base = nullptr;
    int32_t n_slots = 0;
    int32_t max_rank = 0;
    int device = -1;

    std::vector<uint8_t> state;                       // per page
    std::unordered_map<int32_t, slora::Adapter> adapters;
    std::vector<int32_t> arena;                       // host image of all page lists
    std::unordered_map<int64_t, std::vector<int64_t>> free_lists; // length -> offsets
    int32_t *d_arena = nullptr;                       // device image
    int64_t d_arena_cap = 0;                          // entries
    std::vector<int32_t *> retired_arenas;            // outgrown device images, freed with the pool
    int64_t dirty_lo = 0, dirty_hi = 0;               // [lo, hi) not yet on the device
    // allocator: pages are handed out from a stack of released pages first (entries are checked
    // when popped: a page may have been taken by index meanwhile), then from the never-used tail
    std::vector<int32_t> released;
    int64_t fresh = 0;                                // pages >= fresh never entered `released`
    int64_t n_free = 0;
    uint64_t unload_generation = 0;
    int64_t live_plans = 0;
    int64_t mfma_min_tokens = 16;
    int64_t mfma_min_tiles = 32;
    int64_t xcd_group = 0;                            // accepted, no effect
    int64_t hand_polls = 256;                         // reads of v in a launch that hands it over before a wavefront computes it for itself
    int64_t upload_groups = 32;                       // workgroups of an adapter upload from host memory
    int64_t fuse_decode = 1;                          // 0: never, 1: when the batch has enough small groups, 2: always
    int64_t shrink_pages = 0;                         // a caller's pages of A per vector-shrink item (its x rows are staged once for all of them); 0: kShrinkPages, or more
    int64_t mfma_split_bytes = 1 << 20;               // MFMA shrink: a tile's H range is cut into shares of about this many row bytes
    int64_t mfma_split_min_h = 1024;                  // ... but no share is shorter than this many elements of H

    // recycled buffer sets (plans, page writes) and the stream that carries work-list uploads
    std::vector<slora::Buffers *> idle_sets;
    int64_t sets_made = 0;                            // buffer sets ever allocated (steady state: constant)
    int64_t device_allocs = 0;                        // hipMalloc / hipHostMalloc calls made for them
    int64_t hand_overs = 0;                           // applies that handed v over inside a launch
    void *static_scratch = nullptr;                   // this GPU's copy of the library's static scratch
    void *upload_stream = nullptr;                    // hipStream_t, created on first use
    void *arena_event = nullptr;                      // hipEvent_t: the device page-list image is complete after it
    int32_t uploads(void **out);                      // the upload stream
    bool arena_done = true;                           // ... which is known to have happened
    int32_t arena_ready(void *stream);                // await_arena, unless it has happened
    int32_t await_arena(void *stream);                // make `stream` wait for the latest page-list upload

    int32_t take_set(slora::Buffers **out, size_t h_bytes, size_t d_bytes); // an idle set whose last use has completed, or a new one
    void give_set(slora::Buffers *set, void *last_stream);                  // record `order` on last_stream, park the set
    // room for v and, if there is memory for them, for the words of launches on `stream` that hand it over
    int32_t grow_v(slora::Buffers *set, size_t floats, size_t words, void *stream);
    bool next_launch(slora::Buffers *set, void *stream); // the number of the next such launch
    void free_sets();

    int32_t sync_device();                            // push dirty arena range
    void set_state(int64_t page, uint8_t to);         // ownership change with free-count / stack upkeep
    int32_t take(int64_t n, uint8_t as, int32_t *out); // n free pages -> state `as`
};

struct slora_plan {
    slora_pool *pool = nullptr;
    uint64_t generation = 0;
    int32_t T = 0;        // tokens in the batch
    int32_t T_act = 0;    // tokens that have an adapter of rank > 0
    int32_t v_stride = 0; // floats per row of v
    int32_t max_shrink_tok = 0;
    int32_t n_mfma_tiles = 0;
    int32_t expand_threads = 64; // workgroup size of the vector expand (columns per item / 8)
    int32_t max_expand_tok = 0;
    bool small = false;          // small calls on the plan may take the one-launch kernel for small batches
    int32_t expand_split = 0;    // small batch: 512-column items, ranks split over four wavefronts
    int64_t sum_rank = 0;
    int32_t n_groups = 0, n_groups_vec = 0, n_groups_mfma = 0;

    // host image
    std::vector<int32_t> tok_idx;                     // sorted position -> token index
    std::vector<slora::Item> vs_items, ve_items, me_items;
    std::vector<slora::Item> vf_items; // decode groups for the one-launch kernel (their two-stage items end vs / ve)
    int32_t n_vs_head = 0, n_ve_head = 0; // items of vs / ve that belong to other groups
    // A dual plan's groups of many tokens are in both kernels' lists: in vs / ve between the plain groups'
    // items and n_vs_head / n_ve_head, and in the MFMA lists.  fp32-y applies take the latter (wide).
    bool dual = false;
    int64_t reread = 0, reread_min = 0; // bytes of pages the vector kernels would read again, per slot; what it takes per call
    int32_t n_vs_plain = 0, n_ve_plain = 0;
    int32_t most_slots = 0;   // most slots of a call so far, and
    size_t most_words = 0;    // the words that they may take
    // of the vector items that a call which hands v over runs: on a wide route (without those of groups on the MFMA kernels), on another
    struct Chain {
        int64_t words = 0; // per slot, a value of v each
        int64_t work = 0;  // ranks times tokens of all expand items
        int32_t tok = 0;   // most tokens of a shrink item
        bool shared = false; // pages that several items read: a group of more than kExpandTok tokens
    } chain[2];
    const Chain &chain_of(const slora::Route &r) const { return chain[r.wide ? 0 : 1]; }
    bool mfma_on(const slora::Route &r) const { return !dual || r.wide; }
    // items of the two vector lists that a call runs beside the other kernels
    size_t n_vs(const slora::Route &r) const { return r.wide ? (size_t)n_vs_plain : r.fused ? (size_t)n_vs_head : vs_items.size(); }
    size_t n_ve(const slora::Route &r) const { return r.wide ? (size_t)n_ve_plain : r.fused ? (size_t)n_ve_head : ve_items.size(); }
    // The vector lists once more, in larger items, if the expand is rank-split and a group has more than kExpandTok tokens
    std::vector<slora::Item> gs_items, gv_items; // shrink: groups of more than that; vector-shrink items of the others
    std::vector<slora::Item> ge_items;           // expand: all groups
    int32_t n_gs_plain = 0, n_ge_plain = 0;      // without a dual plan's groups of many tokens
    int32_t max_gv_tok = 0;                      // most tokens of an item of gv
    bool fours[2] = {false, false};              // an item of ge is one of fours_pay, for y in fp32 and in 16 bits
    size_t n_gs(const slora::Route &r) const { return r.wide ? (size_t)n_gs_plain : gs_items.size(); }
    size_t n_ge(const slora::Route &r) const { return r.wide ? (size_t)n_ge_plain : ge_items.size(); }
    // ... of the one that hands v over
    int64_t chain_wgs(const slora::Route &r) const { return (int64_t)(n_vs(r) + n_ve(r)); }
    bool chain_pays(int32_t n, const slora::Route &r) const; // ... which an apply of n slots may take
    size_t most_chain_words(int32_t n) const; // its words in a call of up to n slots, if any may take it
    // workgroups of the vector kernels, per slot
    size_t shrink_wgs(const slora::Route &r) const { return r.gang ? n_gs(r) + gv_items.size() : n_vs(r); }
    size_t expand_wgs(const slora::Route &r) const { return r.gang_expand ? n_ge(r) : n_ve(r); }
    std::vector<slora::MsItem> ms_items;
    std::vector<slora::MsItem> mj_items; // one record per split tile, for the kernel that joins the shares
    // MFMA shrink with kMsTok >> sub tokens per workgroup: workgroups per slot, LDS of the largest tile
    int64_t ms_wgs[slora::kMsSubs] = {};
    int32_t ms_lds[slora::kMsSubs] = {};
    int32_t me_run = 1;        // most tiles of a run of the MFMA expand list
    int32_t me_stages = 0;     // most 32-rank stages of V that an MFMA expand workgroup holds in one of its two LDS buffers
    int32_t n_sync = 0;        // tiles that the join kernel finishes: those in several shares, all of a dual plan
    int64_t part_floats = 0;   // partial sums of the split tiles, per slot
    int32_t n_rank_blocks = 1; // kMsRanks-blocks per row of v (exponent sets per tile)

    // device image: tok_idx and the four lists in one buffer of the plan's buffer set
    slora::Buffers *set = nullptr;
    int32_t *d_tok_idx = nullptr;
    slora::Item *d_vs = nullptr, *d_ve = nullptr, *d_me = nullptr, *d_vf = nullptr, *d_gs = nullptr, *d_gv = nullptr, *d_ge = nullptr;
    slora::MsItem *d_ms = nullptr, *d_mj = nullptr;

    // scratch for v = x*A (set->v, or the library's static scratch), per slot: T_act * v_stride floats (vector path rows), n_mfma_tiles * (v_stride/16) *
    // pieces KiB of MFMA operand fragments, 32 row exponents (bytes) per tile and rank block, and the
    // partial sums of split tiles
    int64_t vfrag_floats(int32_t dtype) const
    {
        return (int64_t)n_mfma_tiles * (v_stride / 16) * pieces(dtype) * 256;
    }
    // 16-bit pieces that carry v to the MFMA expand: three where the vector kernels would keep it in fp32
    int32_t pieces(int32_t dtype) const { return dual || dtype != SLORA_F16 ? 3 : 2; }
    int64_t vexp_floats() const { return (int64_t)n_mfma_tiles * n_rank_blocks * 8; } // one byte per row
    int64_t v_slot_floats(int32_t dtype, bool mfma) const
    {
        return (int64_t)T_act * v_stride + (mfma ? vfrag_floats(dtype) + vexp_floats() + part_floats : 0);
    }
    int64_t v_total_floats(int32_t n, int32_t dtype, bool mfma) const { return (int64_t)n * v_slot_floats(dtype, mfma); }
    // scratch of any call with at most n slots, whatever the type of y: a plan's buffer is grown once
    int64_t v_most_floats(int32_t n, int32_t dtype) const;
    int64_t me_wgs() const { return (int64_t)n_mfma_tiles * ((pool->H + slora::kMfmaExpandCols - 1) / slora::kMfmaExpandCols); } // one per tile
    // The kernels of a call with n slots.  A dual plan's MFMA form is taken only where it fits the static scratch,
    // so that an apply gives the same bits wherever v is kept.
    slora::Route route(int32_t n, bool apply, bool y16) const;
    // The latest shrink whose launches succeeded.  Written together, after them: a call that fails on the
    // way must not change how an expand reads the v that is there.
    float *v_used = nullptr; // where it left v
    int32_t v_slots = 0;     // its n
    slora::Route v_route;    // and its kernels: the layout of v (fused: v of those groups never reached memory)

    // Stream order.  Every launch of a plan reads its work lists and reads or writes its v, so
    // all of a plan's work is kept in ONE order: when a call names another stream than the
    // previous one, the new stream first waits for an event recorded on the old one.
    void *last_stream = nullptr; // hipStream_t of the latest upload or launch
    bool order_recorded = false; // set->order already marks the end of the work on last_stream

    int32_t upload(bool once, void *stream); // once: for a single call, on `stream`
    int32_t enter(void *stream);
    void fill_args(slora::MultiArgs &a, int32_t n, float *v, const slora::Route &r) const;
};

namespace slora {

// scheduler (plan.cpp)
// call_slots: slots of the plan's only call, if that is known; 0: calls may have as many as the pool
int32_t build_plan(slora_pool *pool, slora_plan *plan, const int32_t *ids, int32_t T,
                   const int32_t *seg_offsets, int32_t n_seg, int32_t call_slots);

// kernel launchers (kernels.hip); all return a SLORA_* code
int32_t launch_write_pages(slora_pool *pool, const int32_t *d_idx, int64_t n, const void *d_src,
                           void *stream, int32_t max_groups = 0); // max_groups > 0 caps the grid
int32_t launch_copy(void *dst, const void *src, size_t bytes, void *stream); // 16-byte aligned; src may be pinned host memory
bool stream_captures(void *stream); // whether a HIP graph captures it
int32_t launch_clear(void *dst, size_t bytes, void *stream); // whole multiples of 16 bytes
int32_t launch_gather(slora_pool *pool, int64_t arena_entry, int32_t rank, void *dev_out, void *stream);
int32_t static_scratch_address(int device, void **out); // `device` must be current
int32_t launch_shrink(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, const Route &route);
int32_t launch_expand(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route);
// both stages of the vector groups that are not in launch_fused
int32_t launch_chain(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route);
// the groups of the one-launch decode kernel or, on a small route, the whole batch
int32_t launch_fused(slora_plan *plan, int32_t n, const MultiArgs &args, void *stream, bool y16, const Route &route);

} // namespace slora
